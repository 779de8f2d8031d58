// Device code for states held on chip by a team of workgroups of B threads for all iterations: the single-state
// kernel (held form, and fused form on chip) and the batched kernel's resident phases.  Member `rank` owns the
// contiguous vectors [base, base + per), thread tid the vectors e * B + tid, e < NE = per / B (or the one vector
// tid < per when per < B): the first RE positions in registers, the others in the thread's own LDS slots (no
// other thread touches them, so they need no workgroup barrier).  NE and RE are template parameters, so the
// sweep has no branches.
#pragma once

#include <type_traits>

#include "stream.h"

namespace grover {

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
    // The same with the oracle's signs, s = -1 for a marked amplitude (bit a of `bits`: amplitude a of the vector): the
    // products with s are exact, so c' = 2S/N - s c and the addition of s c' round once, as above, in as many
    // instructions.  Position 0, where a wave with marks in one row has them, takes them in every wave, which needs no
    // branch.  On MI355X, against a branch around the sweep for negations and corrections: a search at n = 10 binary64
    // with 10^4 shots 16.2 -> 15.3 us, n = 16 complex64 with binary32 updates 326 -> 302 us, n = 24 complex64 6.44 -> 6.29
    // ms, 1024 searches of n = 8 .. 20 23.7 -> 22.8 ms.
    __device__ static inline double sign(unsigned bits, int p)
    {
        const unsigned hi = ((bits << (31 - amp(p))) & 0x80000000u) | 0x3FF00000u;  // of +-1.0
        return __longlong_as_double((long long)((unsigned long long)hi << 32));
    }
    // As in `add`: in branches, the compiler would widen all vectors ahead of them.
    __device__ static inline void own(H (&x)[parts])
    {
        if constexpr (std::is_same<H, float>::value)
#pragma unroll
            for (int p = 0; p < parts; ++p)
                asm volatile("" : "+v"(x[p]));
    }
    __device__ static inline void add_signed(H (&x)[parts], unsigned bits, AccF64 &acc)
    {
        own(x);
#pragma unroll
        for (int p = 0; p < parts; ++p) {
            if (imag(p))
                acc.i = __builtin_fma(sign(bits, p), double(x[p]), acc.i);
            else
                acc.r = __builtin_fma(sign(bits, p), double(x[p]), acc.r);
        }
        own(x);
    }
    __device__ static inline void step_signed(H (&x)[parts], unsigned bits, double mr, double mi, float mr32, float mi32,
                                              AccF64 &acc)
    {
#pragma unroll
        for (int p = 0; p < parts; ++p) {
            const double s = sign(bits, p), m = imag(p) ? mi : mr;
            if constexpr (U32)
                x[p] = __builtin_fmaf(-float(s), x[p], imag(p) ? mi32 : mr32);
            else if constexpr (std::is_same<T, C64>::value)
                x[p] = H(float(__builtin_fma(-s, double(x[p]), m)));
            else
                x[p] = __builtin_fma(-s, x[p], m);
        }
        add_signed(x, bits, acc);
    }
    // Marks in further rows are handled around the sweep, which treats their amplitudes as unmarked: the held values are
    // negated before it (exactly), which makes the update 2S/N + c, their correct new value, and the sum is corrected
    // after it by -2c' (so it holds s c').  A second sweep with signs everywhere, in a branch, spills.
    __device__ static inline void negate(H (&x)[parts], unsigned bits)
    {
#pragma unroll
        for (int p = 0; p < parts; ++p) {
            const unsigned flip = (bits << (31 - amp(p))) & 0x80000000u;
            if constexpr (std::is_same<H, float>::value)
                x[p] = __uint_as_float(__float_as_uint(x[p]) ^ flip);
            else
                x[p] = __longlong_as_double(__double_as_longlong(x[p]) ^ (long long)((unsigned long long)flip << 32));
        }
    }
    __device__ static inline void correct(H (&x)[parts], unsigned bits, AccF64 &acc)
    {
        own(x);
#pragma unroll
        for (int p = 0; p < parts; ++p) {
            // -2 or 0 (an unmarked amplitude that is not finite has made the sum so already)
            const unsigned hi = unsigned(int(bits << (31 - amp(p))) >> 31) & 0xC0000000u;
            const double k = __longlong_as_double((long long)((unsigned long long)hi << 32));
            if (imag(p))
                acc.i = __builtin_fma(k, double(x[p]), acc.i);
            else
                acc.r = __builtin_fma(k, double(x[p]), acc.r);
        }
        own(x);
    }
};

// Marked bits of a thread's vectors, two per vector: bits 2 r, 2 r + 1 of word r / 16 for position r.
template <int NE>
struct MarkBits {
    static constexpr int words = (NE + 15) / 16;
    uint32_t w[words];
    // The same bits, unknown to the compiler: what is derived from them (signs) is then made anew where it is used, not
    // kept in registers for all iterations.
    __device__ inline MarkBits fresh() const
    {
        MarkBits k = *this;
#pragma unroll
        for (int i = 0; i < words; ++i)
            asm volatile("" : "+v"(k.w[i]));
        return k;
    }
    __device__ inline unsigned at(int r) const { return (w[r / 16] >> (2 * (r % 16))) & 3u; }
    // a position in LDS: all in the last word
    __device__ inline unsigned in_lds(int r) const { return (w[words - 1] >> (2 * (r % 16))) & 3u; }
    __device__ inline void set(unsigned r, unsigned b)
    {
#pragma unroll
        for (int i = 0; i < words; ++i)
            w[i] |= int(r / 16u) == i ? b << (2u * (r % 16u)) : 0u;
    }
};

// First index of the sorted list marks[0, m) whose mark is >= x, m if none is.  Called by a whole wave: 64 probes a
// step, as a list is far away and a step's loads travel together.
__device__ inline uint64_t wave_lower_bound(const uint64_t *marks, uint64_t m, uint64_t x)
{
    const uint64_t lane = threadIdx.x % kWave;
    uint64_t lo = 0, len = m;  // the answer lies in [lo, lo + len]
    while (len > 0) {
        const uint64_t step = (len + kWave - 1u) / kWave;
        const uint64_t below = uint64_t(__popcll(__ballot(lane * step < len && marks[lo + lane * step] < x)));
        if (below == 0)
            break;
        const uint64_t end = below * step < len ? below * step : len;
        lo += (below - 1u) * step + 1u;
        len = end - ((below - 1u) * step + 1u);
    }
    return lo;
}

// Where a wave of a B-thread member finds its marked amplitudes.  Position r of a thread holds vector e = r ^ swap,
// swap the same in every lane of a wave and chosen so that a wave whose marks lie in one row has them at position 0:
// instructions for marks are then spent on position 0 alone, unless the wave holds marks in other rows too (in_rest, a
// bit per position).
template <int NE, int B, int EPV>
struct WaveMarks {
    // LDS words that `find` needs: a bit per amplitude of the member
    static constexpr unsigned kWords = unsigned(NE) * B * EPV / 32u;
    MarkBits<NE> mk{};
    unsigned swap = 0u;
    unsigned any = 0u;  // this wave holds marked amplitudes (the same in every lane, as swap and rest)
    uint32_t rest_lo = 0u, rest_hi = 0u;
    __device__ inline bool in_rest(int r) const { return ((r < 32 ? rest_lo >> r : rest_hi >> (r - 32)) & 1u) != 0u; }
    __device__ inline bool has_rest() const { return (rest_lo | rest_hi) != 0u; }
    // Calls f(r) for the positions r in [BEGIN, END) of the groups of four that hold marks beyond the first row.  The
    // groups are tested where they are used: conditions kept for all iterations do not fit the scalar registers.
    template <int BEGIN, int END, class F>
    __device__ inline void each_rest(F f) const
    {
        uint32_t lo = rest_lo, hi = rest_hi;
        asm volatile("" : "+s"(lo), "+s"(hi));
#pragma unroll
        for (int g = BEGIN / 4; g * 4 < END; ++g)
            if (((g < 8 ? lo : hi) >> (4 * (g % 8))) & 0xFu)
#pragma unroll
                for (int r = g * 4 > BEGIN ? g * 4 : BEGIN; r < END && r < g * 4 + 4; ++r)
                    f(r);
    }
    // From the sorted list marks[0, m), for the vectors [base, base + per) of the member; called by the whole workgroup.
    // Up to 16 marks are held by the lanes of every wave, which goes through those of its own; more are scattered into the
    // LDS words.  On MI355X, one iteration of a call on one workgroup (n = 10 binary64, 64 marks; n = 14 complex64, 300
    // and 1024 marks): every mark gone through by every wave up to 128 of them, then a binary search of the list per
    // vector 8.8, 28.8 and 32.9 us; a search per vector always 3.6, 19.5, 20.9; this 2.7, 7.2, 7.5.
    __device__ inline void find(const uint64_t *marks, uint64_t m, uint64_t base, uint64_t per, uint32_t *words)
    {
        const unsigned tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
        uint64_t lo = 0, hi = m;
        if (m > uint64_t(kWave)) {
            lo = wave_lower_bound(marks, m, base * EPV);
            hi = lo + wave_lower_bound(marks + lo, m - lo, (base + per) * EPV);
        }
        const uint64_t mine = hi - lo <= uint64_t(kWave) && lane < hi - lo ? marks[lo + lane] : ~uint64_t(0);
        const uint64_t v = mine / EPV - base;  // huge when the mark lies before the member, or there is none
        uint64_t rows = 0;                     // positions that hold marks
        if (__builtin_expect(hi - lo <= uint64_t(kWave) && __popcll(__ballot(v < per)) <= 16, 1)) {
            uint64_t todo = __ballot(v < per && unsigned(v) % B / kWave == wave);
            if (todo != 0)
                swap = unsigned(__builtin_amdgcn_readlane(int(v), __builtin_ctzll(todo))) / B;
            for (; todo != 0; todo &= todo - 1u) {
                const int k = __builtin_ctzll(todo);
                const unsigned at = unsigned(__builtin_amdgcn_readlane(int(v), k));
                const unsigned amp = unsigned(__builtin_amdgcn_readlane(int(mine % EPV), k));
                const unsigned r = (at / B) ^ swap;
                if (at % kWave == lane)
                    mk.set(r, 1u << amp);
                rows |= uint64_t(1) << r;
            }
        } else {
            for (unsigned w = tid; w < kWords; w += B)
                words[w] = 0u;
            __syncthreads();
#pragma unroll 4
            for (uint64_t i = lo + tid; i < hi; i += B) {
                const uint64_t d = marks[i] - base * EPV;
                if (d < per * EPV)
                    atomicOr(&words[d / 32u], 1u << (d % 32u));
            }
            __syncthreads();
#pragma unroll
            for (int e = 0; e < NE; ++e) {
                const unsigned w = words[tid * EPV / 32u + unsigned(e) * (B * EPV / 32u)];
                const unsigned b = (w >> (tid * EPV % 32u)) & ((1u << EPV) - 1u);
                mk.w[e / 16] |= b << (2 * (e % 16));
                rows |= __ballot(b != 0u) != 0u ? uint64_t(1) << e : 0u;
            }
            if (rows != 0u && (rows & (rows - 1u)) == 0u) {  // one row: to position 0
                swap = unsigned(__builtin_ctzll(rows));
                unsigned b = 0u;
#pragma unroll
                for (int i = 0; i < MarkBits<NE>::words; ++i) {
                    b |= int(swap / 16u) == i ? (mk.w[i] >> (2u * (swap % 16u))) & 3u : 0u;
                    mk.w[i] = 0u;
                }
                mk.w[0] = b;
                rows = 1u;
            }
        }
        // the same in every lane of a wave: kept in scalar registers
        swap = __builtin_amdgcn_readfirstlane(swap);
        any = __builtin_amdgcn_readfirstlane(rows != 0u ? 1u : 0u);
        rest_lo = __builtin_amdgcn_readfirstlane(uint32_t(rows) & ~1u);
        rest_hi = __builtin_amdgcn_readfirstlane(uint32_t(rows >> 32));
    }
};

// All iterations of one member's share, and the store back.  The state is loaded (kLoad) or starts as `fill`;
// its oracle-signed sum is formed in the order the iterations add theirs, so consecutive calls compose bit for
// bit.  `begin` is asked once, by the whole workgroup, before the first sum; `reduce` is the team's (or the
// workgroup's) sum.  Returns false, nothing stored, when either says so.  `words`: LDS of WaveMarks::find; `mine`: the
// thread's LDS slots, B apart.
template <class T, bool U32, bool WIDE, int NE, int RE, int B, bool kLoad, class Begin, class Reduce>
__device__ __forceinline__ bool held_run(typename T::vec *st, uint64_t base, uint64_t per, const uint64_t *marks,
                                         uint64_t m, uint64_t iters, double scale, const typename T::vec &fill,
                                         uint32_t *words, typename T::vec *mine, Begin begin, Reduce reduce)
{
    using X = Held<T, U32, WIDE>;
    using V = typename T::vec;
    constexpr int LE = NE - RE;
    static_assert(LE == 0 || (LE <= 16 && RE % 16 + LE <= 16), "the LDS positions' marked bits lie in one word");
    const unsigned tid = threadIdx.x;
    const bool active = NE > 1 || tid < per;
    WaveMarks<NE, B, T::EPV> wm;
    wm.find(marks, m, base, per, words);
    const bool has_rest = NE > 1 && wm.has_rest();

    typename X::H x[RE][X::parts];
    // byte offset of position r's vector in this member's share
    const auto rs = buffer_rsrc(st, uint32_t(per * 16u));
    auto at = [&](unsigned r, unsigned t16) { return (r ^ wm.swap) * unsigned(B * 16) + t16; };
    AccF64 acc0;
    // The sum of a wave with marks in several rows: from +c' to s c'.  Where that is not finite (an infinite amplitude,
    // or c' or -2 c' near the largest finite value), the sum is formed again with the signs.
    auto correct_rest = [&](AccF64 &acc) {
        const MarkBits<NE> mk = wm.mk.fresh();
        wm.template each_rest<1, RE>([&](int r) { X::correct(x[r], mk.at(r), acc); });
#pragma unroll 1
        for (int r = RE; r < NE; ++r)
            if (wm.in_rest(r)) {
                typename X::H y[X::parts];
                X::get(mine[(r - RE) * B], y);
                X::correct(y, mk.in_lds(r), acc);
            }
        if (__builtin_expect(__any(!isfinite(acc.r) || !isfinite(acc.i)), 0)) {
            acc = AccF64();
#pragma unroll
            for (int r = 0; r < RE; ++r) {
                X::add_signed(x[r], mk.at(r), acc);
                __builtin_amdgcn_sched_barrier(0);  // one vector's signs and temporaries at a time
            }
#pragma unroll 1
            for (int r = RE; r < NE; ++r) {
                typename X::H y[X::parts];
                X::get(mine[(r - RE) * B], y);
                X::add_signed(y, mk.in_lds(r), acc);
            }
        }
    };
    if (active) {
#pragma unroll
        for (int r = 0; r < RE; ++r)
            X::get(kLoad ? bload16<kBufNT, V>(rs, at(r, tid * 16u)) : fill, x[r]);
#pragma unroll 4
        for (int r = RE; r < NE; ++r)
            mine[(r - RE) * B] = kLoad ? bload16<kBufNT, V>(rs, at(r, tid * 16u)) : fill;
        X::add_signed(x[0], wm.mk.at(0), acc0);
#pragma unroll
        for (int r = 1; r < RE; ++r)
            X::add(x[r], acc0);
#pragma unroll 2
        for (int r = RE; r < NE; ++r) {
            typename X::H y[X::parts];
            X::get(mine[(r - RE) * B], y);
            X::add(y, acc0);
        }
        if (has_rest)
            correct_rest(acc0);
    }
    double sr = acc0.r, si = acc0.i;
    if (!begin() || !reduce(sr, si))
        return false;
    for (uint64_t it = 0; it < iters; ++it) {
        const double mr = sr * scale, mi = si * scale;
        const float mr32 = float(mr), mi32 = float(mi);
        AccF64 acc;
        if (active) {
            if (has_rest) {
                const MarkBits<NE> mk = wm.mk.fresh();
                wm.template each_rest<1, RE>([&](int r) { X::negate(x[r], mk.at(r)); });
#pragma unroll 1
                for (int r = RE; r < NE; ++r)
                    if (wm.in_rest(r)) {
                        typename X::H y[X::parts];
                        X::get(mine[(r - RE) * B], y);
                        X::negate(y, mk.in_lds(r));
                        mine[(r - RE) * B] = X::vec(y);
                    }
            }
            X::step_signed(x[0], wm.mk.at(0), mr, mi, mr32, mi32, acc);
#pragma unroll
            for (int r = 1; r < RE; ++r)
                X::step(x[r], mr, mi, mr32, mi32, acc);
#pragma unroll 4
            for (int r = RE; r < NE; ++r) {
                typename X::H y[X::parts];
                X::get(mine[(r - RE) * B], y);
                X::step(y, mr, mi, mr32, mi32, acc);
                mine[(r - RE) * B] = X::vec(y);
            }
            if (has_rest)
                correct_rest(acc);
        }
        sr = acc.r;
        si = acc.i;
        if (!reduce(sr, si))
            return false;
    }
    if (active) {
        unsigned t16 = tid * 16u;
        asm volatile("" : "+v"(t16));  // offsets computed again, not kept in registers since the loads
#pragma unroll
        for (int r = 0; r < RE; ++r)
            bstore16<kBufNT>(X::vec(x[r]), rs, at(r, t16));
#pragma unroll 4
        for (int r = RE; r < NE; ++r)
            bstore16<kBufNT>(mine[(r - RE) * B], rs, at(r, t16));
    }
    return true;
}

}  // namespace grover
