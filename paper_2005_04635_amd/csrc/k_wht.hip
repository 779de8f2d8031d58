// Blocked Walsh-Hadamard transform for the gate-level comparison path (H^n of Algorithms 1 and 2).
//
// H^n factorises over qubits, and any set of qubits can be transformed together once their amplitudes are in one
// workgroup.  So instead of n passes over the state (one per qubit, Algorithm 1 literally), the qubits are split into
// groups and each group takes one pass, over tiles of 2^B amplitudes:
//   - the low group, qubits 0 .. B-1: a tile is 2^B contiguous amplitudes;
//   - high groups of r <= B - c qubits: a tile is 2^r rows (stride 2^q0) by 2^c contiguous columns, and segments of
//     2^c amplitudes are at least 64 bytes, 128 where two groups can have it.
// The groups commute, so the two transforms of a conventional iteration, H^n (2|0><0| - I) H^n, visit them in opposite
// orders and the group in the middle is transformed, phase-shifted and transformed again while its tile is on chip;
// likewise the last group of one iteration and the first of the next, with the scale and the next oracle's flips in
// between.  k iterations of a state of g groups take 2k(g - 1) + 1 passes (2kg and k launches for the oracle
// otherwise), and a state of one group takes all k iterations in one launch.
//
// Butterflies are unnormalised, (a, b) -> (a + b, a - b), in binary64; the storage type is rounded once per pass.  The
// normalisation of an iteration is the exact power of two 2^-n (2^(-n/2) for H^n alone, exact for even n).  The phase
// shift is applied as I - 2|0><0|, which touches index 0 only, and its sign goes into the scale.
//
// What bounds a pass: HBM (two transfers of every amplitude), then LDS.  A tile lives in registers, 16 or 32 amplitudes
// per thread, so that a round in registers takes four or five stages, and 14 qubits need two or three rounds with an
// exchange through LDS between them (eight amplitudes per thread with the tile in LDS took four rounds for 12).  A complex
// exchange sends the real and the imaginary parts in turn through 2^B words, which lets a tile of 2^14 fit the 160 KiB;
// there only one workgroup fits a CU, and its next tile is loaded meanwhile.
//
// On MI355X, n = 25 complex64: 116 us for a pass that goes one way (4.6 TB/s), 175 and 197 us for the low and the high
// group there and back, whose 28 and 22 binary64 stages and four exchanges are not hidden behind the one tile in flight;
// four iterations 3200 -> 1640 us (24 passes of 133 us before).  n = 22: 242 -> 45 us per iteration; n = 12, in one
// launch: 12.5 -> 2.8; n = 28, 13 passes of four iterations at 4.3 TB/s for 24: 6.1 -> 3.3 ms per iteration.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "stream.h"
#include "wht.h"

namespace grover {
namespace {


// Amplitudes per thread, log2, for tiles of 2^B: a round's window of local bits.  Three windows, one of them at bit 4,
// cover bits 0 .. 4 + 2 value_bits - 1.
constexpr int value_bits(int B) { return B <= 12 ? 4 : 5; }

constexpr uint32_t kMaxTileBits = 14;
constexpr int kAnyCols = -1;

// What a pass does.
enum Kind {
    kLow,       // the low group once; the oracle's flips before it, the scale after it
    kLowBack,   // the low group, the scale and the oracle's flips, the low group again
    kHigh,      // a high group once; the scale after it
    kHighBack,  // the last high group, the phase shift, the same group again
    kAll,       // all iterations of a state that is one tile
};

struct WhtArgs {
    void *state;
    const uint64_t *marks;
    uint64_t m;
    uint64_t tiles;
    uint64_t iters;   // of the one-group kernel
    double scale;
    uint32_t top;     // bits of a tile's local index in use: the tile's B, or n where the state is smaller
    uint32_t c;       // low local bits that are columns; the stages are on bits c .. top-1
    uint32_t q0;      // qubit of local bit c
    uint32_t flips;   // whether kLow flips
};

// Storage <-> the binary64 parts held in registers.
template <class T>
struct Wht;
template <>
struct Wht<C64> {
    using E = float2;
    static constexpr int kParts = 2, kStride = 1, kBytes = 8;
    static constexpr bool kPrefetch = true;
    __device__ static void in(E x, double *re, double *im) { *re = x.x, *im = x.y; }
    __device__ static E out(double re, double im) { return make_float2(float(re), float(im)); }
};
template <>
struct Wht<C128> {
    using E = double2;
    static constexpr int kParts = 2, kStride = 1, kBytes = 16;
    static constexpr bool kPrefetch = false;  // two tiles do not fit the registers
    __device__ static void in(E x, double *re, double *im) { *re = x.x, *im = x.y; }
    __device__ static E out(double re, double im) { return make_double2(re, im); }
};
template <>
struct Wht<F64Real> {
    using E = double;
    static constexpr int kParts = 1, kStride = 1, kBytes = 8;
    static constexpr bool kPrefetch = true;
    __device__ static void in(E x, double *re, double *) { *re = x; }
    __device__ static E out(double re, double) { return re; }
};
// The real or the imaginary parts of a complex state, which no step of an iteration mixes: a workgroup for each.
template <class R>
struct PartOf {};
template <class R>
struct Wht<PartOf<R>> {
    using E = R;
    static constexpr int kParts = 1, kStride = 2, kBytes = 2 * int(sizeof(R));
    static constexpr bool kPrefetch = false;
    __device__ static void in(E x, double *re, double *) { *re = double(x); }
    __device__ static E out(double re, double) { return R(re); }
};
// Orders LDS accesses only: loads of the next tile stay in flight across it.
__device__ __forceinline__ void lds_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A tile of 2^B amplitudes, 2^v to a thread, v = value_bits(B).  In the layout S, value k of thread t is local index
// spot<S>(t) | k << S: the thread holds the bits S .. S+v-1 of the index.  Three layouts are in use: 4 (loads and stores
// of 16 neighbours, stages 4 .. 3+v), 0 (stages 0 .. 3) and B - v (stages 4+v .. B-1, and the stores of a pass that goes
// one way).
// C: columns of the tile of a high group, log2 (kAnyCols: those of the arguments); 0 for contiguous amplitudes.  kPart:
// the state may be smaller than the tile.
template <class T, int B, int C, bool kPart>
struct Tile {
    using W = Wht<T>;
    using E = typename W::E;
    static constexpr bool kRows = C != 0;
    static constexpr int kValBits = value_bits(B), kVals = 1 << kValBits;
    static constexpr uint32_t kMid = 4 + kValBits;  // the first stage of the top layout
    static constexpr int kThreads = 1 << (B - kValBits);
    static constexpr int kTop = B - kValBits;
    static constexpr int kWords = (1 << B) + (1 << (B - 5));

    double x[W::kParts][kVals];

    template <int S>
    static __device__ __forceinline__ uint32_t spot(uint32_t t)
    {
        return ((t >> S) << (S + kValBits)) | (t & ((1u << S) - 1u));
    }

    // LDS word of a local index: one word in 32 is left out, so that threads 32 words apart fall on different banks.
    // The word of spot | k << S is the sum of the two words, as the two have no bit in common.
    static __device__ __forceinline__ constexpr uint32_t word(uint32_t e) { return e + (e >> 5); }

    // Butterflies of the stages s with lo <= s < hi that lie in the layout S.
    template <int S>
    __device__ __forceinline__ void stages(uint32_t lo, uint32_t hi)
    {
#pragma unroll
        for (int b = 0; b < kValBits; ++b) {
            if (uint32_t(S + b) < lo || uint32_t(S + b) >= hi)
                continue;
#pragma unroll
            for (int p = 0; p < W::kParts; ++p) {
                __builtin_amdgcn_sched_barrier(0);  // a stage in place: nothing else's results beside it
#pragma unroll
                for (int k = 0; k < kVals; ++k) {
                    if (k & (1 << b))
                        continue;
                    const double u = x[p][k], v = x[p][k | (1 << b)];
                    x[p][k] = u + v;
                    x[p][k | (1 << b)] = u - v;
                }
            }
        }
    }

    // From layout F to layout S.
    template <int F, int S>
    __device__ __forceinline__ void exchange(double *buf)
    {
        const uint32_t t = fresh_tid();
        double *const from = buf + word(spot<F>(t));
        double *const to = buf + word(spot<S>(t));
#pragma unroll
        for (int p = 0; p < W::kParts; ++p) {
#pragma unroll
            for (int k = 0; k < kVals; ++k)
                from[word(uint32_t(k) << F)] = x[p][k];
            lds_sync();
#pragma unroll
            for (int k = 0; k < kVals; ++k)
                x[p][k] = to[word(uint32_t(k) << S)];
            lds_sync();
        }
    }

    // All stages c .. top-1, from layout 4 to the top one.
    __device__ __forceinline__ void forward(uint32_t c, uint32_t top, double *buf)
    {
        stages<4>(c, top < kMid ? top : kMid);
        if (c < 4u) {
            exchange<4, 0>(buf);
            stages<0>(c, top < 4u ? top : 4u);
            exchange<0, kTop>(buf);
        } else {
            exchange<4, kTop>(buf);
        }
        stages<kTop>(c < kMid ? kMid : c, top);
    }

    // The same in the opposite order, from the top layout to layout 4.
    __device__ __forceinline__ void backward(uint32_t c, uint32_t top, double *buf)
    {
        stages<kTop>(c < kMid ? kMid : c, top);
        if (c < 4u) {
            exchange<kTop, 0>(buf);
            stages<0>(c, top < 4u ? top : 4u);
            exchange<0, 4>(buf);
        } else {
            exchange<kTop, 4>(buf);
        }
        stages<4>(c, top < kMid ? top : kMid);
    }

    __device__ __forceinline__ void scaled(double s)
    {
#pragma unroll
        for (int p = 0; p < W::kParts; ++p)
#pragma unroll
            for (int k = 0; k < kVals; ++k)
                x[p][k] *= s;
    }

    __device__ __forceinline__ void negate_first()
    {
#pragma unroll
        for (int p = 0; p < W::kParts; ++p)
            x[p][0] = -x[p][0];
    }

    // Negates the values whose bit in `table` (one per local index) is set, in layout S.
    template <int S>
    __device__ __forceinline__ void flip(const uint32_t *table)
    {
        const uint32_t e0 = spot<S>(fresh_tid());
#pragma unroll
        for (int k = 0; k < kVals; ++k) {
            if (k % 4 == 0)
                __builtin_amdgcn_sched_barrier(0);
            const uint32_t e = e0 | uint32_t(k) << S;
            if ((table[e >> 5] >> (e & 31u)) & 1u) {
#pragma unroll
                for (int p = 0; p < W::kParts; ++p)
                    x[p][k] = -x[p][k];
            }
        }
    }

    // Offset in the state of a local index, from the tile's first amplitude; additive over disjoint bits.  Made anew
    // for each load and store: as many offsets as a thread has values do not fit beside the values.
    struct Offsets {
        uint32_t c, q0;
        __device__ __forceinline__ explicit Offsets(const WhtArgs &a) : c(C == kAnyCols ? a.c : uint32_t(C)), q0(a.q0)
        {
            asm volatile("" : "+s"(q0));
        }
        __device__ __forceinline__ uint64_t operator()(uint32_t e) const
        {
            return kRows ? (uint64_t(e >> c) << q0) | (e & ((1u << c) - 1u)) : e;
        }
    };

    // First amplitude of tile t: consecutive tiles are neighbours along the columns.
    static __device__ __forceinline__ uint64_t first(const WhtArgs &a, uint64_t t)
    {
        if (!kRows)
            return t << a.top;
        const uint32_t chunk_bits = a.q0 - a.c;
        return ((t >> chunk_bits) << (a.q0 + a.top - a.c)) | ((t & ((uint64_t(1) << chunk_bits) - 1u)) << a.c);
    }

    // Where part `part` of an amplitude is, in units of E.
    static __device__ __forceinline__ uint64_t place(const WhtArgs &a, uint64_t tile, uint32_t part, uint64_t offset)
    {
        return (first(a, tile) + offset) * W::kStride + part;
    }

    // A state of at most one tile (kPart): its bytes as a buffer, of which loads beyond the end give zero and stores there
    // do nothing, so that no value needs a condition.
    static __device__ __forceinline__ __amdgpu_buffer_rsrc_t small_state(const WhtArgs &a)
    {
        return buffer_rsrc(a.state, (uint32_t(sizeof(E)) * uint32_t(W::kStride)) << a.top);
    }
    template <int S>
    static __device__ __forceinline__ uint32_t small_place(uint32_t part, int k)
    {
        return ((spot<S>(threadIdx.x) | uint32_t(k) << S) * uint32_t(W::kStride) + part) * uint32_t(sizeof(E));
    }
    static __device__ __forceinline__ E load_bytes(__amdgpu_buffer_rsrc_t rs, uint32_t off)
    {
        E v;
        if constexpr (sizeof(E) == 4) {
            const auto w = __builtin_amdgcn_raw_buffer_load_b32(rs, off, 0, 0);
            __builtin_memcpy(&v, &w, 4);
        } else {
            static_assert(sizeof(E) == 8, "a part of an amplitude, or a real one");
            const auto w = __builtin_amdgcn_raw_buffer_load_b64(rs, off, 0, 0);
            __builtin_memcpy(&v, &w, 8);
        }
        return v;
    }
    static __device__ __forceinline__ void store_bytes(E v, __amdgpu_buffer_rsrc_t rs, uint32_t off)
    {
        if constexpr (sizeof(E) == 4) {
            unsigned w;
            __builtin_memcpy(&w, &v, 4);
            __builtin_amdgcn_raw_buffer_store_b32(w, rs, off, 0, 0);
        } else {
            unsigned w __attribute__((ext_vector_type(2)));
            __builtin_memcpy(&w, &v, 8);
            __builtin_amdgcn_raw_buffer_store_b64(w, rs, off, 0, 0);
        }
    }

    template <int S>
    static __device__ __forceinline__ void load(const WhtArgs &a, uint64_t tile, uint32_t part, E (&raw)[kVals])
    {
        if constexpr (kPart) {
            const auto rs = small_state(a);
#pragma unroll
            for (int k = 0; k < kVals; ++k)
                raw[k] = load_bytes(rs, small_place<S>(part, k));
            return;
        }
        const uint32_t e0 = spot<S>(fresh_tid());
        const Offsets offset(a);
        const E *const p = static_cast<const E *>(a.state) + place(a, tile, part, offset(e0));
#pragma unroll
        for (int k = 0; k < kVals; ++k) {
            raw[k] = p[offset(uint32_t(k) << S) * W::kStride];
            if (k % 4 == 3)
                __builtin_amdgcn_sched_barrier(0);  // keeps few of the addresses in registers at a time
        }
    }

    template <int S>
    __device__ __forceinline__ void store(const WhtArgs &a, uint64_t tile, uint32_t part) const
    {
        if constexpr (kPart) {
            const auto rs = small_state(a);
#pragma unroll
            for (int k = 0; k < kVals; ++k)
                store_bytes(W::out(x[0][k], x[W::kParts - 1][k]), rs, small_place<S>(part, k));
            return;
        }
        const uint32_t e0 = spot<S>(fresh_tid());
        const Offsets offset(a);
        E *const p = static_cast<E *>(a.state) + place(a, tile, part, offset(e0));
#pragma unroll
        for (int k = 0; k < kVals; ++k) {
            p[offset(uint32_t(k) << S) * W::kStride] = W::out(x[0][k], x[W::kParts - 1][k]);
            if (k % 4 == 3)
                __builtin_amdgcn_sched_barrier(0);
        }
    }

    __device__ __forceinline__ void widen(const E (&raw)[kVals])
    {
#pragma unroll
        for (int k = 0; k < kVals; ++k)
            W::in(raw[k], &x[0][k], &x[W::kParts - 1][k]);
        // here, not where the next tile's loads need the registers
#pragma unroll
        for (int p = 0; p < W::kParts; ++p)
#pragma unroll
            for (int k = 0; k < kVals; ++k)
                asm volatile("" : "+v"(x[p][k]));
    }
};

// The marks of [base, base + 2^top) as one bit per local index; returns whether there are any.  `mine` is mark
// threadIdx.x, read once per workgroup.
template <int B>
__device__ __forceinline__ bool mark_bits(const WhtArgs &a, uint64_t base, uint64_t mine, uint32_t *table, uint32_t *any)
{
    constexpr uint64_t kThreads = 1u << (B - value_bits(B));
    if (threadIdx.x < (1u << (B - 5)))  // 2^B bits
        table[threadIdx.x] = 0u;
    if (threadIdx.x == 0)
        *any = 0u;
    lds_sync();
    uint64_t i = threadIdx.x, end = a.m;
    if (a.m > 16u * kThreads) {  // a long list: from the first mark at or above base
        uint64_t lo = 0, hi = a.m;
        while (lo < hi) {
            const uint64_t mid = (lo + hi) / 2;
            if (a.marks[mid] < base)
                lo = mid + 1;
            else
                hi = mid;
        }
        i += lo;
        end = a.m - lo < (uint64_t(1) << a.top) ? a.m : lo + (uint64_t(1) << a.top);
    }
    for (; i < end; i += kThreads) {
        const uint64_t d = (i == threadIdx.x ? mine : a.marks[i]) - base;
        if ((d >> a.top) == 0u) {
            atomicOr(&table[d >> 5], 1u << (d & 31u));
            *any = 1u;
        }
    }
    lds_sync();
    return *any != 0u;
}

// Number of this block in an order that gives four consecutive numbers to one XCD (blocks go round the 8 XCDs in launch
// order): the two halves of a 128-byte line and the two parts of its amplitudes meet in one L2.  Longer runs would put
// the XCDs a power of two apart in memory, on the same channels (16 MiB
// states, H^n: n = 20 complex128 20.6 us, 29.6 with an eighth of the tiles in a row; n = 21 real 18.6 and 27.7).
__device__ __forceinline__ unsigned four_by_xcd()
{
    const unsigned b = blockIdx.x;
    return gridDim.x % 32u == 0u ? (b & ~31u) | (b & 7u) << 2 | (b >> 3 & 3u) : b;
}

// A pass (T: the storage, or the parts of one; kKind: what it does; C: columns of a high group's tile, log2).
template <class T, int B, Kind kKind, int C>
__global__ __launch_bounds__(1 << (B - value_bits(B)), 2) void wht_kernel(WhtArgs a)
{
    constexpr bool kRows = C != 0;
    constexpr bool kPart = B == 10;
    using Tl = Tile<T, B, C, kPart>;
    // the largest tile leaves room for one workgroup per CU: it takes several tiles, and loads the next one early
    constexpr bool kSeveral = B == int(kMaxTileBits) && Wht<T>::kStride == 1, kPrefetch = kSeveral && Wht<T>::kPrefetch;
    __shared__ double buf[Tl::kWords];
    __shared__ uint32_t table[kRows ? 1 : 1 << (B - 5)];
    __shared__ uint32_t any;
    const uint32_t c = C == kAnyCols ? a.c : uint32_t(C), top = kPart ? a.top : uint32_t(B);
    const bool flips = !kRows && (kKind != kLow || a.flips) && a.m > 0;
    const uint64_t mine = flips && threadIdx.x < a.m ? a.marks[threadIdx.x] : 0u;
    typename Tl::E raw[Tl::kVals];
    Tl tl;
    constexpr unsigned kStride = unsigned(Wht<T>::kStride);
    const unsigned number = four_by_xcd();
    uint64_t tile = number / kStride;
    const uint32_t part = kStride == 1u ? 0u : number % kStride;
    if (kPrefetch)
        Tl::template load<4>(a, tile, part, raw);
#pragma unroll 1
    do {
        if (!kPrefetch)
            Tl::template load<4>(a, tile, part, raw);
        tl.widen(raw);
        const uint64_t next = tile + gridDim.x / kStride;
        if (kPrefetch && next < a.tiles)
            Tl::template load<4>(a, next, part, raw);
        const bool marked = flips && mark_bits<B>(a, tile << top, mine, table, &any);
        if constexpr (kKind == kAll) {
#pragma unroll 1
            for (uint64_t it = 0; it < a.iters; ++it) {
                if (marked)
                    tl.template flip<4>(table);
                tl.forward(c, top, buf);
                if (threadIdx.x == 0)
                    tl.negate_first();
                tl.backward(c, top, buf);
                tl.scaled(a.scale);
            }
            tl.template store<4>(a, tile, part);
        } else if constexpr (kKind == kLowBack || kKind == kHighBack) {
            tl.forward(c, top, buf);
            if constexpr (kRows) {
                if (tile == 0 && threadIdx.x == 0)
                    tl.negate_first();
            } else {
                tl.scaled(a.scale);
                if (marked)
                    tl.template flip<Tl::kTop>(table);
            }
            tl.backward(c, top, buf);
            tl.template store<4>(a, tile, part);
        } else {
            if (marked)
                tl.template flip<4>(table);
            if (kPart && top <= Tl::kMid) {  // no stage in the top layout: nor the exchange to it
                tl.template stages<4>(c, top);
                tl.template exchange<4, 0>(buf);
                tl.template stages<0>(c, top < 4u ? top : 4u);
                tl.scaled(a.scale);
                tl.template store<0>(a, tile, part);
                return;
            }
            tl.forward(c, top, buf);
            if (a.scale != 1.0)
                tl.scaled(a.scale);
            tl.template store<Tl::kTop>(a, tile, part);
        }
        tile = next;
    } while (kSeveral && tile < a.tiles);
}

// How the n qubits are split: the low group takes `bits` of them, the others go evenly to `highs` groups.
struct Split {
    uint32_t bits = 0, highs = 0;
};

// One group up to n = 14: a workgroup's iteration in registers then costs less than two launches (n = 14 complex64 7.9 us,
// 13.7 in two groups).  Above, as few groups as tiles of 2^14 and segments of 64 bytes allow (n = 25 complex64, two
// groups 381 us per iteration; three, as n = 26 scaled, 420), and the smallest tile that does it: more and smaller
// workgroups hide each other's loads (n = 23 complex64, 2^13 against 2^14: 87 and 98 us for the first iteration).  Three
// groups keep 2^12, below which segments would be no longer.  H^n alone, for which one workgroup has no later passes to
// save, goes to two groups from n = 14 on (`alone`; n = 14 complex64 6.6 us, 8.3 in one group).  States below 2^11 have a
// kernel of one wave, whose loads and stores need no conditions, and no third layout up to n = 8 (n = 9 complex64, H^n 2.9
// us; 4.1 in the padded tile of 2^11, 3.1 with the tile in LDS).
constexpr Split split(uint32_t n, uint32_t elem, bool alone)
{
    Split s;
    if (n <= (alone ? kMaxTileBits - 1u : kMaxTileBits)) {
        s.bits = std::max(n, 10u);
        return s;
    }
    const uint32_t cols = elem == 16u ? 2u : 3u;  // columns of a 64-byte segment, log2
    for (s.highs = 1;; ++s.highs) {
        // n - bits <= highs * (bits - cols)
        s.bits = (n + s.highs * cols + s.highs) / (s.highs + 1u);
        if (s.bits > kMaxTileBits)
            continue;
        s.bits = std::max(s.bits, s.highs == 1u ? 11u : 12u);
        return s;
    }
}

// Qubits of high group g = 1 .. s.highs.
constexpr uint32_t high_bits(const Split &s, uint32_t n, uint32_t g)
{
    const uint32_t rest = n - s.bits;
    return rest / s.highs + (g <= rest % s.highs ? 1u : 0u);
}

// Whether the real and the imaginary parts go to workgroups of their own: where the tiles are too few to fill the
// chip, half the work of each takes less time than the lines read twice, which caches hold at these sizes (n = 18
// complex64 10.5 us per iteration against 17.2; at n = 20 the two are equal).
constexpr bool by_parts(const Split &s)
{
    return s.highs == 0u || (s.highs == 1u && s.bits <= 11u);
}

// Whether some n has a pass of this kind in tiles of 2^bits and, in high groups, segments of 2^c (kAnyCols: any): only
// those are compiled.
template <class T>
constexpr bool reached(Kind kind, uint32_t bits, int c)
{
    for (uint32_t n = 1; n <= kMaxQubits; ++n)
        for (const bool alone : {false, true}) {
            const Split s = split(n, uint32_t(Wht<T>::kBytes), alone);
            if (s.bits != bits || (!std::is_same<T, F64Real>::value && by_parts(s) != (Wht<T>::kStride == 2)))
                continue;
            if ((kind == kLow && (alone || s.highs > 0u)) || (kind == kLowBack && !alone && s.highs > 0u) ||
                (kind == kAll && !alone && s.highs == 0u))
                return true;
            for (uint32_t g = 1; g <= s.highs; ++g)
                if (kind == (alone || g < s.highs ? kHigh : kHighBack) &&
                    (c == kAnyCols || uint32_t(c) == s.bits - high_bits(s, n, g)))
                    return true;
        }
    return false;
}

template <class T, Kind kKind, int B, int C>
const void *kernel_if_reached()
{
    if constexpr (reached<T>(kKind, B, C))
        return reinterpret_cast<const void *>(&wht_kernel<T, B, kKind, C>);
    return nullptr;
}

// The kernel for tiles of 2^B and segments of 2^c.  The columns are a constant of the kernel where a workgroup has more
// than two waves: stages left out at run time cost registers and moves.
template <class T, Kind kKind, int B>
const void *kernel_of(uint32_t c)
{
    if constexpr (kKind != kHigh && kKind != kHighBack) {
        return kernel_if_reached<T, kKind, B, 0>();
    } else if constexpr (B <= 11) {
        return kernel_if_reached<T, kKind, B, kAnyCols>();
    } else {
        switch (c) {
        case 2: return kernel_if_reached<T, kKind, B, 2>();
        case 3: return kernel_if_reached<T, kKind, B, 3>();
        case 4: return kernel_if_reached<T, kKind, B, 4>();
        case 5: return kernel_if_reached<T, kKind, B, 5>();
        default: return nullptr;
        }
    }
}

template <class T, Kind kKind>
const void *kernel(uint32_t bits, uint32_t c)
{
    switch (bits) {
    case 10: return kernel_of<T, kKind, 10>(c);
    case 11: return kernel_of<T, kKind, 11>(c);
    case 12: return kernel_of<T, kKind, 12>(c);
    case 13: return kernel_of<T, kKind, 13>(c);
    case 14: return kernel_of<T, kKind, 14>(c);
    default: return nullptr;
    }
}
static_assert(kMaxTileBits == 14, "the largest of `kernel`");

// Every split has its kernels: high groups in tiles of 2^12 and more have segments of 2^2 to 2^5.
constexpr bool splits_covered()
{
    for (uint32_t n = 1; n <= kMaxQubits; ++n)
        for (const uint32_t elem : {8u, 16u})
            for (const bool alone : {false, true}) {
                const Split s = split(n, elem, alone);
                if (s.bits < 10u || s.bits > kMaxTileBits || (s.highs == 0u && n > s.bits))
                    return false;
                for (uint32_t g = 1; g <= s.highs; ++g) {
                    const uint32_t r = high_bits(s, n, g), c = s.bits - r;
                    if (r < 1u || r > s.bits || (s.bits > 11u && (c < 2u || c > 5u)))
                        return false;
                }
            }
    return true;
}
static_assert(splits_covered(), "a number of qubits without a kernel");

// One pass of group g (0: the low one).
template <class T, Kind kKind>
hipError_t pass(grover_ctx *c, const Split &s, uint32_t g, double scale = 1.0, bool flips = false, uint64_t iters = 1)
{
    WhtArgs a{};
    a.state = c->state;
    a.marks = c->marks_dev;
    a.m = c->marks.size();
    a.iters = iters;
    a.scale = scale;
    a.flips = flips;
    a.top = std::min(s.bits, c->n);
    if (g > 0) {
        const uint32_t rest = c->n - s.bits;
        a.c = s.bits - high_bits(s, c->n, g);
        a.q0 = s.bits + (g - 1u) * (rest / s.highs) + std::min(g - 1u, rest % s.highs);
    }
    a.tiles = c->N >> a.top;
    const void *fn = kernel<T, kKind>(s.bits, a.c);
    if (!fn)
        return hipErrorInvalidValue;
    const uint64_t grid = s.bits == kMaxTileBits && Wht<T>::kStride == 1 ? std::min<uint64_t>(a.tiles, uint64_t(c->cu_count))
                                                                         : a.tiles * Wht<T>::kStride;
    void *args[] = {&a};
    return hipLaunchKernel(fn, dim3(unsigned(grid)), dim3(1u << (s.bits - uint32_t(value_bits(int(s.bits))))), args, 0, c->stream);
}

template <class T>
hipError_t hadamard_all_blocked(grover_ctx *c, const Split &s)
{
    // 2^(-n/2): exact for even n; for odd n 2^(-(n+1)/2) * sqrt(2) rounded once to binary64
    const int n = int(c->n);
    const double scale = (n % 2 == 0) ? std::ldexp(1.0, -n / 2) : std::ldexp(std::sqrt(2.0), -(n + 1) / 2);
    hipError_t e = pass<T, kLow>(c, s, 0, s.highs == 0u ? scale : 1.0);
    for (uint32_t g = 1; g <= s.highs && e == hipSuccess; ++g)
        e = pass<T, kHigh>(c, s, g, g == s.highs ? scale : 1.0);
    return e;
}

template <class T>
hipError_t gate_iterate_blocked(grover_ctx *c, const Split &s, uint64_t k)
{
    const double scale = -std::ldexp(1.0, -int(c->n));
    if (k == 0)
        return hipSuccess;
    if (s.highs == 0)
        return pass<T, kAll>(c, s, 0, scale, true, k);
    hipError_t e = pass<T, kLow>(c, s, 0, 1.0, true);
    for (uint64_t it = 0; it < k && e == hipSuccess; ++it) {
        for (uint32_t g = 1; g < s.highs && e == hipSuccess; ++g)
            e = pass<T, kHigh>(c, s, g);
        if (e == hipSuccess)
            e = pass<T, kHighBack>(c, s, s.highs);
        for (uint32_t g = s.highs - 1u; g > 0u && e == hipSuccess; --g)
            e = pass<T, kHigh>(c, s, g);
        if (e == hipSuccess)
            e = it + 1 < k ? pass<T, kLowBack>(c, s, 0, scale) : pass<T, kLow>(c, s, 0, scale);
    }
    return e;
}

}  // namespace

hipError_t launch_hadamard_all_blocked(grover_ctx *c)
{
    const Split s = split(c->n, uint32_t(elem_bytes(c->dtype)), true);
    const bool parts = by_parts(s);
    switch (c->dtype) {
    case GROVER_F64_REAL: return hadamard_all_blocked<F64Real>(c, s);
    case GROVER_C64: return parts ? hadamard_all_blocked<PartOf<float>>(c, s) : hadamard_all_blocked<C64>(c, s);
    case GROVER_C128: return parts ? hadamard_all_blocked<PartOf<double>>(c, s) : hadamard_all_blocked<C128>(c, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_gate_iterate_blocked(grover_ctx *c, uint64_t k)
{
    const Split s = split(c->n, uint32_t(elem_bytes(c->dtype)), false);
    const bool parts = by_parts(s);
    switch (c->dtype) {
    case GROVER_F64_REAL: return gate_iterate_blocked<F64Real>(c, s, k);
    case GROVER_C64: return parts ? gate_iterate_blocked<PartOf<float>>(c, s, k) : gate_iterate_blocked<C64>(c, s, k);
    case GROVER_C128: return parts ? gate_iterate_blocked<PartOf<double>>(c, s, k) : gate_iterate_blocked<C128>(c, s, k);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace grover
