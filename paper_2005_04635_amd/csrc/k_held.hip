// On-chip iteration of one state by a team of workgroups: the held form of grover_iterate (complex64), and the
// fused form's kernel for states that fit on chip (binary64, complex64 and complex128 storage, binary64 sums).
// The state stays in registers and LDS for all k iterations of one call (Algorithm 5's loop of Algorithm 3's
// oracle sign and Eq. 2 / Algorithm 4's inversion about the mean), held by a team of T workgroups of 512
// threads (T a power of two).  Member `rank` owns the vectors [rank * per, (rank + 1) * per), per = nvec / T;
// thread tid the vectors rank * per + e * 512 + tid, e < NE = per / 512 (or the one vector tid < per when
// per < 512).  The launch loads the state, forms the oracle-signed sum of it in the order the iterations add
// theirs (so consecutive calls compose bit for bit), runs k iterations with one team barrier each, and stores
// the state back.
//
// What bounds it: the update's instructions (a complex64 part takes a binary64 subtraction, the rounding
// conversion, the widening one and the addition to the sum) and the team barrier's latency.  512 threads leave
// each 256 VGPRs, so up to 48 vectors per thread stay in registers (16 more in LDS: 512 KiB per workgroup,
// 128 MiB on 256) and a wave's share of the reduction, which every wave pays, is spread over more vectors than
// with 1024 threads.  NE is a template parameter, so the sweep has no branches.  Up to 16 complex64 vectors per
// thread are held widened to binary64 (values that a binary32 represents), which saves one of five
// instructions per part.  One optimal search (or 801 iterations at n = 24), 1024-thread workgroups of at most 16
// vectors and the earlier barrier (n = 24 and complex128: the streaming fused kernel) -> this kernel on MI355X:
// complex64 n = 16 (binary32 update) 0.634 -> 0.349 ms, n = 20 3.48 -> 2.10, n = 24 14.1 -> 6.44 (8.0 us per
// iteration); complex128 n = 21 4.61 -> 1.96 ms (2.4 us per iteration).
#include <algorithm>
#include <type_traits>

#include "stream.h"

namespace grover {
namespace {

constexpr int kChipBlock = 512;
constexpr int kChipRegE = 48;  // vectors per thread in registers when NE = 64, the other 16 in LDS (128 KiB)

struct ChipArgs {
    void *state;
    const uint64_t *marks;
    uint64_t m;
    uint64_t per;  // vectors per member: nvec / team
    uint64_t iters;
    double scale;  // 2 / N, a power of two: S * scale rounds as 2S / N
    GridSync *sync;
    uint64_t *partials;  // team slots
    uint64_t gen0;
    uint64_t timeout_ticks;
    uint32_t team;
    uint32_t xcds;   // blocks b with b % 8 < xcds form the team, rank (b / 8) * xcds + b % 8; the others end at once
    uint32_t probe;  // 1: one team barrier only (residency check)
};

// A storage vector as `parts` numbers, part p of amplitude amp(p); imag(p): an imaginary part.  H: the type
// that a held part has; widen: complex64 parts held as binary64 values that binary32 represents.
template <class T, bool U32, bool WIDE>
struct Held {
    static constexpr int parts = T::EPV * (T::kComplex ? 2 : 1);
    using H = typename std::conditional<std::is_same<T, C64>::value && !WIDE, float, double>::type;
    __device__ static constexpr int amp(int p) { return T::kComplex ? p / 2 : p; }
    __device__ static constexpr bool imag(int p) { return T::kComplex && (p & 1); }
    // one part of c' = 2S/N - c, rounded once to the storage (U32: one binary32 subtraction from 2S/N in binary32)
    __device__ static inline H update(H c, double m, float m32)
    {
        if constexpr (U32)
            return m32 - c;
        else if constexpr (std::is_same<T, C64>::value)
            return H(float(m - double(c)));
        else
            return m - c;
    }
    __device__ static inline void get(const typename T::vec &v, H (&x)[parts])
    {
        if constexpr (parts == 4) {
            x[0] = v.x;
            x[1] = v.y;
            x[2] = v.z;
            x[3] = v.w;
        } else {
            x[0] = v.x;
            x[1] = v.y;
        }
    }
    __device__ static inline typename T::vec vec(const H (&x)[parts])
    {
        if constexpr (parts == 4)
            return make_float4(float(x[0]), float(x[1]), float(x[2]), float(x[3]));
        else
            return make_double2(x[0], x[1]);
    }
    // A vector's parts into the sum, amplitude by amplitude.  The empty asm hides that a binary32 part is still
    // the value that was widened here: else the compiler keeps the widened values of all of them for the next
    // iteration, which is what `widen` does where there is room, and spills elsewhere.
    __device__ static inline void add(H (&x)[parts], AccF64 &acc)
    {
#pragma unroll
        for (int p = 0; p < parts; ++p) {
            if (imag(p))
                acc.i += double(x[p]);
            else
                acc.r += double(x[p]);
            if constexpr (std::is_same<H, float>::value)
                asm volatile("" : "+v"(x[p]));
        }
    }
    __device__ static inline void step(H (&x)[parts], double mr, double mi, float mr32, float mi32, AccF64 &acc)
    {
#pragma unroll
        for (int p = 0; p < parts; ++p)
            x[p] = imag(p) ? update(x[p], mi, mi32) : update(x[p], mr, mr32);
        add(x, acc);
    }
    // Marked amplitudes (bit a of `bits`: amplitude a of the vector) are handled around the sweep, which then
    // treats every amplitude alike: their held values are negated before it (exactly), which makes the update
    // 2S/N + c, their correct new value, and the sum is corrected after it by -2c' (so it holds s c').
    __device__ static inline void negate(H (&x)[parts], unsigned bits)
    {
#pragma unroll
        for (int p = 0; p < parts; ++p)
            x[p] = (bits >> amp(p)) & 1u ? -x[p] : x[p];
    }
    __device__ static inline void correct(const H (&x)[parts], unsigned bits, AccF64 &acc)
    {
#pragma unroll
        for (int p = 0; p < parts; ++p)
            if ((bits >> amp(p)) & 1u) {
                if (imag(p))
                    acc.i += -2.0 * double(x[p]);
                else
                    acc.r += -2.0 * double(x[p]);
            }
    }
};

// Marked bits of a thread's vectors, two per vector: bits 2 r, 2 r + 1 of word r / 16 for position r.
template <int NE>
struct MarkBits {
    static constexpr int words = (NE + 15) / 16;
    uint32_t w[words];
    __device__ inline unsigned at(int r) const { return (w[r / 16] >> (2 * (r % 16))) & 3u; }
    // a position in LDS, r >= kChipRegE: all in the last word
    __device__ inline unsigned in_lds(int r) const { return (w[words - 1] >> (2 * (r % 16))) & 3u; }
    __device__ inline void set(unsigned r, unsigned b)
    {
#pragma unroll
        for (int i = 0; i < words; ++i)
            w[i] |= int(r / 16u) == i ? b << (2u * (r % 16u)) : 0u;
    }
};

// Position r of a thread holds vector e = r ^ swap, swap the same in every lane of a wave and chosen so that the
// wave's first marked vector is at position 0: the few instructions for marks are then spent on position 0
// alone, unless the wave holds marks in other rows too (`rest`, a bit per position).
template <class T, bool U32, int NE>
__global__ __launch_bounds__(kChipBlock) void chip_iterate_kernel(ChipArgs a)
{
    constexpr int RE = NE > kChipRegE ? kChipRegE : NE, LE = NE - RE;
    static_assert(LE == 0 || (LE <= 16 && RE % 16 == 0), "the LDS positions' marked bits fill one word");
    constexpr bool kWide = std::is_same<T, C64>::value && !U32 && NE <= 16;
    using X = Held<T, U32, kWide>;
    using V = typename T::vec;
    __shared__ TeamShared<kChipBlock> sh;
    __shared__ V held[LE > 0 ? LE * kChipBlock : 1];
    const unsigned q = blockIdx.x & 7u, rank = (blockIdx.x >> 3) * a.xcds + q;
    if (q >= a.xcds || rank >= a.team)
        return;
    const Team tm{a.sync, a.partials, a.team, rank, a.timeout_ticks};
    uint64_t gen = a.gen0;
    if (a.probe) {
        double zr = 0.0, zi = 0.0;
        (void)team_sum<kChipBlock>(zr, zi, tm, ++gen, sh);
        return;
    }
    // A launch enqueued behind a failure (a wait that gave up, or input rejected on the device) leaves the
    // state as it is.  Thread 0 reads the error word (other threads might read it later and differ) and the
    // workgroup barrier before the first sum hands the answer on.
    uint32_t error = 0u;
    if (threadIdx.x == 0)
        error = __hip_atomic_load(&a.sync->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const unsigned tid = threadIdx.x, wave = tid / kWave;
    const uint64_t per = a.per, base = uint64_t(rank) * per;
    const bool active = NE > 1 || tid < per;
    V *st = static_cast<V *>(a.state) + base;

    // this member's slice of the sorted marked list, and from it the wave's swap and the threads' marked bits
    const uint64_t lo = a.m > 0 ? lower_bound_u64(a.marks, 0, a.m, base * T::EPV) : 0;
    const uint64_t hi = a.m > 0 ? lower_bound_u64(a.marks, lo, a.m, (base + per) * T::EPV) : 0;
    MarkBits<NE> mk{};
    unsigned swap = 0u;
    bool marked = false;  // this wave holds marked amplitudes (the same in every lane)
    uint64_t rest = 0;    // positions above 0 that hold marks in some lane of this wave
    if (hi - lo <= 512u) {
        for (uint64_t i = lo; i < hi; ++i) {
            const uint64_t x = a.marks[i];
            const unsigned v = unsigned(x / T::EPV - base), e = v / kChipBlock, owner = v % kChipBlock;
            if (owner / kWave == wave) {
                if (!marked)
                    swap = e;
                marked = true;
                const unsigned r = e ^ swap;
                if (owner == tid)
                    mk.set(r, 1u << unsigned(x % T::EPV));
                rest |= r > 0u ? uint64_t(1) << r : 0u;
            }
        }
    } else {
#pragma unroll 1
        for (unsigned r = 0; r < unsigned(NE); ++r) {
            const unsigned b = active ? marked_bits<T::EPV>(a.marks, lo, hi, (base + uint64_t(r) * kChipBlock + tid) * T::EPV) : 0u;
            mk.set(r, b);
            if (__any(b != 0u)) {
                marked = true;
                rest |= r > 0u ? uint64_t(1) << r : 0u;
            }
        }
    }
    // the same in every lane of a wave: kept in scalar registers
    swap = __builtin_amdgcn_readfirstlane(swap);
    const unsigned is_marked = __builtin_amdgcn_readfirstlane(marked ? 1u : 0u);
    const uint32_t rest_lo = __builtin_amdgcn_readfirstlane(uint32_t(rest)), rest_hi = __builtin_amdgcn_readfirstlane(uint32_t(rest >> 32));
    auto in_rest = [&](int r) { return ((r < 32 ? rest_lo >> r : rest_hi >> (r - 32)) & 1u) != 0u; };
    const bool has_rest = (rest_lo | rest_hi) != 0u;

    typename X::H x[RE][X::parts];
    V *mine = held + tid;
    // byte offset of position r's vector in this member's share
    const auto rs = buffer_rsrc(st, uint32_t(per * 16u));
    auto at = [&](unsigned r, unsigned t16) { return (r ^ swap) * (kChipBlock * 16u) + t16; };
    AccF64 acc0;
    auto correct_all = [&](AccF64 &acc) {
        X::correct(x[0], mk.at(0), acc);
        if (has_rest) {
#pragma unroll
            for (int r = 1; r < RE; ++r)
                if (in_rest(r))
                    X::correct(x[r], mk.at(r), acc);
#pragma unroll 1
            for (int r = RE; r < NE; ++r)
                if (in_rest(r)) {
                    typename X::H y[X::parts];
                    X::get(mine[(r - RE) * kChipBlock], y);
                    X::correct(y, mk.in_lds(r), acc);
                }
        }
    };
    if (active) {
#pragma unroll
        for (int r = 0; r < RE; ++r)
            X::get(bload16<kBufNT, V>(rs, at(r, tid * 16u)), x[r]);
#pragma unroll 4
        for (int r = RE; r < NE; ++r)
            mine[(r - RE) * kChipBlock] = bload16<kBufNT, V>(rs, at(r, tid * 16u));
#pragma unroll
        for (int r = 0; r < RE; ++r)
            X::add(x[r], acc0);
#pragma unroll 2
        for (int r = RE; r < NE; ++r) {
            typename X::H y[X::parts];
            X::get(mine[(r - RE) * kChipBlock], y);
            X::add(y, acc0);
        }
        if (is_marked)
            correct_all(acc0);
    }
    double sr = acc0.r, si = acc0.i;
    if (__syncthreads_or(error != 0u))
        return;
    if (!team_sum<kChipBlock>(sr, si, tm, ++gen, sh))
        return;
    for (uint64_t it = 0; it < a.iters; ++it) {
        const double mr = sr * a.scale, mi = si * a.scale;
        const float mr32 = float(mr), mi32 = float(mi);
        AccF64 acc;
        if (active) {
            if (is_marked) {
                X::negate(x[0], mk.at(0));
                if (has_rest) {
#pragma unroll
                    for (int r = 1; r < RE; ++r)
                        if (in_rest(r))
                            X::negate(x[r], mk.at(r));
#pragma unroll 1
                    for (int r = RE; r < NE; ++r)
                        if (in_rest(r)) {
                            typename X::H y[X::parts];
                            X::get(mine[(r - RE) * kChipBlock], y);
                            X::negate(y, mk.in_lds(r));
                            mine[(r - RE) * kChipBlock] = X::vec(y);
                        }
                }
            }
#pragma unroll
            for (int r = 0; r < RE; ++r)
                X::step(x[r], mr, mi, mr32, mi32, acc);
#pragma unroll 4
            for (int r = RE; r < NE; ++r) {
                typename X::H y[X::parts];
                X::get(mine[(r - RE) * kChipBlock], y);
                X::step(y, mr, mi, mr32, mi32, acc);
                mine[(r - RE) * kChipBlock] = X::vec(y);
            }
            if (is_marked)
                correct_all(acc);
        }
        sr = acc.r;
        si = acc.i;
        if (!team_sum<kChipBlock>(sr, si, tm, ++gen, sh))
            return;
    }
    if (active) {
        unsigned t16 = tid * 16u;
        asm volatile("" : "+v"(t16));  // offsets computed again, not kept in registers since the loads
#pragma unroll
        for (int r = 0; r < RE; ++r)
            bstore16<kBufNT>(X::vec(x[r]), rs, at(r, t16));
#pragma unroll 4
        for (int r = RE; r < NE; ++r)
            bstore16<kBufNT>(mine[(r - RE) * kChipBlock], rs, at(r, t16));
    }
}

template <class T, bool U32>
const void *chip_kernel(uint64_t ne)
{
    switch (ne) {
    case 1: return reinterpret_cast<const void *>(&chip_iterate_kernel<T, U32, 1>);
    case 2: return reinterpret_cast<const void *>(&chip_iterate_kernel<T, U32, 2>);
    case 4: return reinterpret_cast<const void *>(&chip_iterate_kernel<T, U32, 4>);
    case 8: return reinterpret_cast<const void *>(&chip_iterate_kernel<T, U32, 8>);
    case 16: return reinterpret_cast<const void *>(&chip_iterate_kernel<T, U32, 16>);
    case 32: return reinterpret_cast<const void *>(&chip_iterate_kernel<T, U32, 32>);
    case 64: return reinterpret_cast<const void *>(&chip_iterate_kernel<T, U32, 64>);
    default: return nullptr;
    }
}

uint64_t pow2_at_least(uint64_t x)
{
    uint64_t t = 1;
    while (t < x)
        t <<= 1;
    return t;
}

}  // namespace

// Team size of the held form for a complex64 state of nvec vectors on a device whose largest power-of-two
// team is max_team; 0 when the state does not fit.  About 4 vectors per thread up to 64 workgroups, then at
// most 32: the update's share of an iteration shrinks with the team, while the barrier costs about the same up
// to 64 members (1.0 us at 8, 1.36 at 64 within half of the XCDs) and 0.5-0.7 us more from 128 on.
uint32_t held_team_size(uint64_t nvec, uint32_t max_team)
{
    const uint64_t t16 = pow2_at_least((nvec + 16u * kChipBlock - 1) / (16u * kChipBlock));
    if (t16 <= 128 && t16 <= max_team) {
        uint64_t t4 = pow2_at_least((nvec + 4u * kChipBlock - 1) / (4u * kChipBlock));
        t4 = std::min<uint64_t>(t4, std::min<uint64_t>(64, max_team));
        return uint32_t(std::max(t16, t4));
    }
    const uint64_t t32 = pow2_at_least((nvec + 32u * kChipBlock - 1) / (32u * kChipBlock));
    return t32 <= max_team ? uint32_t(t32) : 0u;
}

// Team size of the fused form's on-chip kernel for a state of nvec vectors, 0 when the streaming kernel serves
// it: binary64 sums, 8 to 64 vectors per thread.  Binary64 and complex128 storage takes two instructions
// per part, so 32 vectors per thread and a team of 64 (0.4 + 1.4 us per iteration) beat 8 and 256 (0.1 + 2.1);
// complex64, four or five, spreads over as many as there are.
uint32_t chip_team_size(uint32_t dtype, uint32_t accum, uint64_t nvec, int cu_count)
{
    if (accum != GROVER_ACC_F64 || dtype == GROVER_CBF16 || nvec < 8u * kChipBlock)
        return 0u;
    uint64_t max_team = 1;
    while (max_team * 2 <= uint64_t(std::min(cu_count, 256)))
        max_team <<= 1;
    const uint64_t slots = nvec / kChipBlock;  // a power of two
    uint64_t team = std::min(slots / 8u, max_team);
    if (dtype != GROVER_C64 && team > 64u && slots <= 64u * 32u)
        team = 64u;
    return slots / team <= 64u ? uint32_t(team) : 0u;
}

hipError_t launch_chip(const ChipLaunch &L)
{
    ChipArgs a;
    a.state = L.state;
    a.marks = L.marks;
    a.m = L.m;
    a.per = L.N / elems_per_vec(L.dtype) / L.team;
    a.iters = L.k;
    a.scale = 2.0 / double(L.N);
    a.sync = L.sync;
    a.partials = L.partials;
    a.gen0 = L.gen0;
    a.timeout_ticks = L.timeout_ticks;
    a.team = L.team;
    a.probe = L.probe ? 1u : 0u;
    // Blocks go round the 8 XCDs: a team inside one XCD (up to 16 members) or one half of them (up to 128) has
    // a shorter way between its members (team_sum), at the price of blocks that end at once.
    a.xcds = L.team <= 16u ? 1u : L.team <= 128u ? 4u : 8u;
    while (a.xcds < 8u && uint64_t(L.team + a.xcds - 1u) / a.xcds * 8u > uint64_t(L.cu_count))
        a.xcds *= 2u;
    const unsigned grid = a.xcds < 8u ? (L.team + a.xcds - 1u) / a.xcds * 8u : L.team;
    const uint64_t ne = std::max<uint64_t>(1, a.per / kChipBlock);
    const void *fn = nullptr;
    switch (L.dtype) {
    case GROVER_F64_REAL: fn = chip_kernel<F64Real, false>(ne); break;
    case GROVER_C64: fn = L.update == GROVER_UPDATE_F32 ? chip_kernel<C64, true>(ne) : chip_kernel<C64, false>(ne); break;
    case GROVER_C128: fn = chip_kernel<C128, false>(ne); break;
    }
    if (!fn)
        return hipErrorInvalidValue;
    void *args[] = {&a};
    return hipLaunchCooperativeKernel(fn, dim3(grid), dim3(kChipBlock), args, 0, L.stream);
}

hipError_t launch_held_iterate(grover_ctx *c, uint64_t k, uint64_t timeout_ticks, bool probe)
{
    ChipLaunch L;
    L.state = c->state;
    L.dtype = c->dtype;
    L.update = c->update;
    L.N = c->N;
    L.marks = c->marks_dev;
    L.m = c->marks.size();
    L.k = k;
    L.team = c->held_team;
    L.cu_count = c->cu_count;
    L.partials = c->partials;
    L.sync = c->sync;
    L.gen0 = c->generation;
    L.timeout_ticks = timeout_ticks;
    L.probe = probe;
    L.stream = c->stream;
    const hipError_t e = launch_chip(L);
    if (e == hipSuccess)
        c->generation += probe ? 1u : k + 1u;
    return e;
}

}  // namespace grover
