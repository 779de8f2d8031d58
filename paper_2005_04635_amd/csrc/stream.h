// Device code shared by the held, batched and phase kernels: the team barrier that also reduces the
// iteration's sum, the marked-tile table, and one streaming pass of a team's share of a state.  A "team"
// is T workgroups of one launch (rank 0 .. T-1) that iterate one state together.  The single-state fused
// kernel keeps its own copy of the same pass and barrier specialised to the whole grid: written against
// these generic helpers (team rank and size as run-time values) the compiler scheduled the tile loop's
// loads less well and the n = 28 iteration ran 4 % slower on MI355X.
#pragma once

#include "internal.h"

namespace grover {

constexpr int kStreamTile = 4096;   // 16-byte vectors per tile: kStreamTile / B per thread of a B-thread workgroup
constexpr int kMarkWords = 1024;    // LDS bitmap of a workgroup's tiles that hold marked amplitudes
constexpr int kTileMarks = 8;       // marks of one tile held in registers

// LDS of a workgroup's part in a team barrier (B threads).
template <int B>
struct TeamShared {
    double red[2][2 * (B / kWave)];  // wave sums of re, then of im; block_allsum alternates the two sets
    double sum[2];
    int failed;
};

// Where a team's barrier lives: its error word (GridSync), its member slots (team_words() 64-bit words: two
// sets by the generation's parity), the number of workgroups T, this workgroup's rank, and the wait limit.
struct Team {
    GridSync *sync;
    uint64_t *partials;
    unsigned size;
    unsigned rank;
    uint64_t timeout_ticks;
};

// A binary64 value travels as 16 bytes {tag, high, tag, low}: two self-validating 64-bit words, each carrying
// 32 bits of the value and the barrier generation (mod 2^32).  A reader that sees the current tag in both has
// both halves of this generation's value, and no memory fence (which on this GPU writes back or invalidates a
// whole L2) is needed to order the value against a separate flag.  Slots are zeroed before a launch and
// generations start at 1.  Device-scope (sc1) 16-byte buffer accesses.
constexpr int kBufDevice = 16;  // sc1

__device__ inline void put_value(__amdgpu_buffer_rsrc_t slots, uint32_t off, double x, uint32_t tag)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(x);
    u32x4 w;
    w.x = tag;
    w.y = unsigned(b >> 32);
    w.z = tag;
    w.w = unsigned(b);
    __builtin_amdgcn_raw_buffer_store_b128(w, slots, off, 0, kBufDevice);
}

// Bounded wait for the values of generation `tag` at the byte offsets off[q] that use[q] names (the others read as
// zero): the loads of a round are issued together.  Gives up when the error word is set or the wall-clock limit
// passes (then setting the error word); both are looked at in the first round and every 16th, the error word by a
// load issued with that round's others (on its own it would add a memory round trip to nearly every barrier: the
// first round mostly comes too early).  The clock is first read in the 16th round, for the same reason: the
// limit counts from there, and a limit of zero gives up in the first round unless all is there already (kernels that
// are to give up at a limit of zero in any case look at it before their first barrier).
template <int NV>
__device__ inline bool wait_offsets(__amdgpu_buffer_rsrc_t slots, const uint32_t (&off)[NV], const bool (&use)[NV],
                                    uint32_t tag, uint32_t *error, uint64_t timeout_ticks, double (&x)[NV])
{
    uint64_t t0 = 0;
    const auto error_word = buffer_rsrc(error, 4u);
    u32x4 w[NV];
    for (unsigned round = 0;; ++round) {
        const bool look = (round & 15u) == 0u;
        uint32_t failed = 0u;
        bool ready = true;
        asm volatile("" ::: "memory");  // the loads are of this round (volatile ones would be of system scope)
#pragma unroll
        for (int q = 0; q < NV; ++q)
            w[q] = __builtin_amdgcn_raw_buffer_load_b128(slots, off[q], 0, kBufDevice);
        if (look)
            failed = __builtin_amdgcn_raw_buffer_load_b32(error_word, 0u, 0, kBufDevice);
#pragma unroll
        for (int q = 0; q < NV; ++q)
            ready = ready && (!use[q] || (w[q].x == tag && w[q].z == tag));
        if (ready)
            break;
        if (look) {
            if (failed != 0u)
                return false;
            bool late = timeout_ticks == 0u;
            if (round >= 16u) {
                const uint64_t now = wall_clock64();
                if (round == 16u)
                    t0 = now;
                late = late || now - t0 > timeout_ticks;
            }
            if (late) {
                __hip_atomic_store(error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return false;
            }
        }
    }
#pragma unroll
    for (int q = 0; q < NV; ++q)
        x[q] = use[q] ? __longlong_as_double((long long)(((unsigned long long)w[q].y << 32) | w[q].w)) : 0.0;
    return true;
}

// The same for NV values at off + q * stride.
template <int NV>
__device__ inline bool wait_values(__amdgpu_buffer_rsrc_t slots, uint32_t off, uint32_t stride, uint32_t tag,
                                   uint32_t *error, uint64_t timeout_ticks, double (&x)[NV])
{
    uint32_t offs[NV];
    bool use[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        offs[q] = off + uint32_t(q) * stride;
        use[q] = true;
    }
    return wait_offsets<NV>(slots, offs, use, tag, error, timeout_ticks, x);
}

// This thread's index in the workgroup, computed afresh: what is derived from it (lane masks, slot offsets) is
// then recomputed at each barrier in a few instructions instead of being kept in registers across the sweep, where
// it costs held state or spills.
__device__ inline unsigned fresh_tid()
{
    unsigned t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t;
}

// Adds the wave values that `red` holds (re of waves 0 .. W-1, then im): lane W - 1 gets the sum of re, lane
// 2 W - 1 that of im.  Called by one whole wave.
template <int B>
__device__ inline double add_wave_values(const double *red, unsigned lane)
{
    constexpr unsigned W = B / kWave;
    double p = lane < 2 * W ? red[lane] : 0.0;
    if (W > 1)
        p += dpp_row_shifted<0x111>(p);
    if (W > 2)
        p += dpp_row_shifted<0x112>(p);
    if (W > 4)
        p += dpp_row_shifted<0x114>(p);
    if (W > 8)
        p += dpp_row_shifted<0x118>(p);
    return p;
}

// Each wave's sums of (re, im) into red.
template <int B>
__device__ inline void put_wave_values(double xr, double xi, double *red, unsigned tid)
{
    const unsigned lane = tid % kWave, wave = tid / kWave;
    const double v = half_totals(fold_pair(xr, xi));
    if (lane == 31)
        red[wave] = v;
    if (lane == 63)
        red[B / kWave + wave] = v;
}

// Workgroup sum of (a, b) for every thread with one workgroup barrier: wave sums, then every wave adds the
// wave values by the same fixed tree (the same bits everywhere).  The wave values alternate between two sets
// by `parity`: a set is rewritten two calls later, after the next call's barrier, which every thread reaches
// only after reading it.
template <int B>
__device__ inline void block_allsum(double &a, double &b, unsigned parity, TeamShared<B> &sh)
{
    if constexpr (B == kWave) {  // one wave: no exchange
        const double v = half_totals(fold_pair(a, b));
        a = lane_value(v, 31);
        b = lane_value(v, 63);
    } else {
        double *red = sh.red[parity & 1u];
        const unsigned tid = fresh_tid();
        put_wave_values<B>(a, b, red, tid);
        __syncthreads();
        const double p = add_wave_values<B>(red, tid % kWave);
        a = lane_value(p, B / kWave - 1);
        b = lane_value(p, 2 * (B / kWave) - 1);
    }
}

// Team-wide sum of (xr, xi) at barrier generation `gen` (1, 2, ... per barrier object; slots zeroed before
// the launch).  Returns false when the wait gave up (time limit, or another workgroup gave up); every thread
// of the workgroup gets the same answer and the sum in (xr, xi).
//
// An all-gather: every member publishes its partial in its own slot of the generation's parity; then, in every
// member, wave 0 waits for the members' values of this generation and adds them in a fixed order, so every
// member computes the same sum bit for bit after one memory round trip.  A member rewrites a slot of parity p
// only at generation g + 2: its partial for g + 1 depends on the sum of g, so its reads of generation g have
// returned before it publishes g + 1, and g + 2 follows only after every member's g + 1 has been seen.
// (Arrivals counted with one atomic per member serialise at the counter's address.)  The team's workgroups
// share no other memory within a launch, so the barrier orders nothing but these values.
//
// What bounds it is latency: 0.3 us for the workgroup's own sum and hand-out (512 threads), the rest the store
// and the load that first sees it.  Bare barriers on MI355X (blocks go round the 8 XCDs, so a team of
// consecutive blocks spans them all), this form against the one before it (two 8-byte words per value at 32
// bytes per member, lane-read wave totals, sleeping polls; 1024 threads): T = 32 1.55 / 2.52 us, T = 64 1.65 /
// 2.67, T = 128 1.98 / 3.22, T = 256 2.05 / 3.73.  Slots 64 bytes apart: at 32, four members' stores land on
// one line that every XCD polls (T = 64 1.88 us).  A team inside one half of the XCDs saves the trip between
// the halves: T = 64 1.36 us, T = 32 1.20.  Above 128 members two levels are faster than one wave's four
// polls per lane (T = 256 2.70 us): members of equal rank % 8 (one XCD when ranks are block numbers)
// meet at the first of them, which publishes their sum, and every member adds the 8 group sums.
template <int B>
__device__ bool team_sum(double &xr, double &xi, const Team &tm, uint64_t gen, TeamShared<B> &sh)
{
    constexpr unsigned W = B / kWave;
    const uint32_t tag = uint32_t(gen);
    const unsigned tid = fresh_tid(), lane = tid % kWave, wave = tid / kWave;
    // sh.red[0] is read by wave 0 only between the two workgroup barriers below; a wave writes it again only
    // in the next call, after the second.  sh.sum and sh.failed are written again only after the first barrier
    // of the next call, which every thread reaches after reading them here.
    put_wave_values<B>(xr, xi, sh.red[0], tid);
    __syncthreads();
    if (wave == 0) {
        const unsigned stride = team_stride(tm.size);
        const bool two = team_two_level(tm.size);
        const unsigned part = (lane >> 5) * 16u;  // lanes 32 .. 63 handle im
        const unsigned groups = 8u, per_group = tm.size / groups;
        const unsigned pos = two ? (tm.rank % groups) * per_group + tm.rank / groups : tm.rank;
        uint64_t *set = tm.partials + uint64_t(gen & 1u) * tm.size * (stride / 8u);
        const auto slots = buffer_rsrc(set, tm.size * stride);
        const double p = add_wave_values<B>(sh.red[0], lane);
        if (lane == W - 1u || lane == 2u * W - 1u)
            put_value(slots, pos * stride + (lane == W - 1u ? 0u : 16u), p, tag);
        double v = 0.0;
        bool ok = true;
        if (two) {
            const auto sums = buffer_rsrc(tm.partials + 2u * tm.size * (stride / 8u) + uint64_t(gen & 1u) * groups * kGroupWords,
                                          groups * uint32_t(kGroupWords) * 8u);
            const unsigned m = lane & 31u;
            double x[1] = {0.0};
            if (tm.rank < groups) {  // the group's first member; per_group <= 32
                if (m < per_group)
                    ok = wait_values<1>(slots, (pos + m) * stride + part, 0u, tag, &tm.sync->error, tm.timeout_ticks, x);
                const double g = half_totals(x[0]);
                const bool all_ok = __all(ok);
                if (m == 31u && all_ok)
                    put_value(sums, tm.rank * uint32_t(kGroupWords) * 8u + part, g, tag);
                x[0] = 0.0;
            }
            if (ok && m < groups)
                ok = wait_values<1>(sums, m * uint32_t(kGroupWords) * 8u + part, 0u, tag, &tm.sync->error,
                                    tm.timeout_ticks, x);
            v = x[0];
        } else if (tm.size <= 32u) {
            const unsigned m = lane & 31u;
            double x[1] = {0.0};
            if (m < tm.size)
                ok = wait_values<1>(slots, m * stride + part, 0u, tag, &tm.sync->error, tm.timeout_ticks, x);
            v = x[0];
        } else {
            double ar = 0.0, ai = 0.0;
            for (unsigned m = lane; m < tm.size && ok; m += kWave) {
                double x[2] = {0.0, 0.0};
                ok = wait_values<2>(slots, m * stride, 16u, tag, &tm.sync->error, tm.timeout_ticks, x);
                ar += x[0];
                ai += x[1];
            }
            v = fold_pair(ar, ai);
        }
        v = half_totals(v);
        const bool failed = __any(!ok);
        if (lane == 31u)
            sh.sum[0] = v;
        if (lane == 63u)
            sh.sum[1] = v;
        if (lane == 0u)
            sh.failed = failed;
    }
    __syncthreads();
    xr = sh.sum[0];
    xi = sh.sum[1];
    return !sh.failed;
}

// First index q >= start with marks[q] >= x in the sorted list marks[0, m), given that every entry before
// `start` is < x: exponential steps from `start`, then a binary search in the last step.  Tiles are visited
// in increasing order, so each search starts where the previous tile's ended and costs O(log gap).
__device__ inline uint64_t gallop_lower_bound(const uint64_t *marks, uint64_t start, uint64_t m, uint64_t x)
{
    if (start >= m || marks[start] >= x)
        return start;
    uint64_t lo = start, step = 1;  // invariant: marks[lo] < x
    while (lo + step < m && marks[lo + step] < x) {
        lo += step;
        step <<= 1;
    }
    const uint64_t hi = lo + step < m ? lo + step : m;
    return lower_bound_u64(marks, lo + 1, hi, x);
}

// Marked bits of the EPV amplitudes starting at element i, from up to kTileMarks marks held in registers
// (padded with ~0, which never equals an amplitude index).
template <int EPV>
__device__ inline unsigned bits_from_regs(const uint64_t (&mk)[kTileMarks], uint64_t i)
{
    unsigned bits = 0;
#pragma unroll
    for (int q = 0; q < kTileMarks; ++q) {
        const uint64_t d = mk[q] - i;  // wraps to a huge value when mk[q] < i
        bits |= d < uint64_t(EPV) ? 1u << unsigned(d) : 0u;
    }
    return bits;
}

// One team member's view of a state: its tiles are t = rank + j * size, j = 0, 1, ... (tiles of
// kStreamTile 16-byte vectors).  At any moment the team streams one contiguous window of the state, spread
// over all HBM channels, while each tile stays with the same workgroup (hence XCD) in every iteration.
template <class T>
struct Share {
    typename T::vec *st;
    uint64_t nvec;
    const uint64_t *marks;  // the state's sorted marked list
    uint64_t m;
    uint64_t rank;
    uint64_t size;
    __device__ uint64_t ntiles() const { return (nvec + kStreamTile - 1) / kStreamTile; }
    __device__ uint64_t count() const { return rank < ntiles() ? (ntiles() - rank + size - 1) / size : 0; }
};

// Table of this workgroup's tiles that hold marked amplitudes (bit j = tile rank + j * size), built by the
// whole workgroup.  Returns false when it cannot be used (too many tiles, or a marked list so long that
// scanning it per workgroup costs more than checking every tile); every tile then takes the checked path.
template <int B, class T>
__device__ bool build_mark_table(const Share<T> &sh, uint32_t *table)
{
    const bool use = sh.count() <= uint64_t(kMarkWords) * 32u && sh.m <= uint64_t(64) * B;
    if (use) {
        for (unsigned w = threadIdx.x; w < kMarkWords; w += B)
            table[w] = 0u;
        __syncthreads();
        for (uint64_t q = threadIdx.x; q < sh.m; q += B) {
            const uint64_t t = sh.marks[q] / T::EPV / kStreamTile;
            if (t % sh.size == sh.rank) {
                const uint64_t j = t / sh.size;
                atomicOr(&table[j >> 5], 1u << (j & 31));
            }
        }
    }
    __syncthreads();
    return use;
}

enum PassMode { kAccumulate, kUpdate, kFill };

// One pass over the workgroup's tiles.  kUpdate: c' = 2S/N - s c written back (nontemporal) and s c' added
// to the accumulator; kAccumulate: s c added; kFill: `fill` written everywhere and s * fill added.  The
// per-thread order of the sum is identical in all modes, so a fresh sum of a stored state equals, bit for
// bit, the sum the pass that wrote it produced.  U32: the update in binary32 from 2S/N rounded to binary32
// (complex64 storage only); otherwise in binary64.
template <int B, class T, class A, PassMode MODE, bool U32 = false>
__device__ inline void stream_pass(const Share<T> &sh, const uint32_t *table, bool use_table, double mr, double mi,
                                   const typename T::vec &fill, A &acc)
{
    using V = typename T::vec;
    constexpr int kUnroll = kStreamTile / B;
    const float mr32 = float(mr), mi32 = float(mi);
    auto update = [&](V &v, unsigned bits) {
        if constexpr (U32)
            update_vec_f32(v, mr32, mi32, bits, acc);
        else
            update_vec<T>(v, mr, mi, bits, acc);
    };
    const unsigned tid = fresh_tid();
    const uint64_t cnt = sh.count();
    uint64_t mp = 0;  // marked entries before this position lie in tiles already visited
    auto plain = [&](uint64_t j) {  // a full tile without marked amplitudes
        const uint64_t v0 = (sh.rank + j * sh.size) * kStreamTile;
        return v0 + kStreamTile <= sh.nvec && !(use_table ? ((table[j >> 5] >> (j & 31)) & 1u) != 0u : sh.m > 0);
    };
    // The next plain tile's loads are issued before this one is updated: with 512 threads, two waves per SIMD are
    // too few to keep loads in flight by themselves.
    bool ahead = false;
    V y[kUnroll];
    for (uint64_t j = 0; j < cnt; ++j) {
        const uint64_t t = sh.rank + j * sh.size;
        const uint64_t v0 = t * kStreamTile;
        if (plain(j)) {
            V x[kUnroll];
            if (MODE != kFill) {
#pragma unroll
                for (int u = 0; u < kUnroll; ++u)
                    x[u] = ahead ? y[u] : load16<true>(sh.st + v0 + u * B + tid);
                ahead = j + 1 < cnt && plain(j + 1);
                if (ahead) {
#pragma unroll
                    for (int u = 0; u < kUnroll; ++u)
                        y[u] = load16<true>(sh.st + v0 + sh.size * kStreamTile + u * B + tid);
                }
            }
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                if (MODE == kUpdate) {
                    update(x[u], 0u);
                    store16<true>(x[u], sh.st + v0 + u * B + tid);
                } else if (MODE == kFill) {
                    store16<true>(fill, sh.st + v0 + u * B + tid);
                    accum_vec<T>(fill, 0u, acc);
                } else {
                    accum_vec<T>(x[u], 0u, acc);
                }
            }
        } else {
            // Ragged tail of the state, or a tile that may hold marked amplitudes: each amplitude's sign
            // comes from the tile's slice [mp, mq) of the sorted marked list.
            mp = gallop_lower_bound(sh.marks, mp, sh.m, v0 * T::EPV);
            const uint64_t mq = gallop_lower_bound(sh.marks, mp, sh.m, (v0 + kStreamTile) * T::EPV);
            const bool in_regs = mq - mp <= uint64_t(kTileMarks);
            uint64_t mk[kTileMarks];
#pragma unroll
            for (int q = 0; q < kTileMarks; ++q)
                mk[q] = in_regs && mp + q < mq ? sh.marks[mp + q] : ~uint64_t(0);
            V x[kUnroll];
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const uint64_t v = v0 + u * B + tid;
                if (v < sh.nvec)
                    x[u] = MODE == kFill ? fill : load16<true>(sh.st + v);
            }
#pragma unroll
            for (int u = 0; u < kUnroll; ++u) {
                const uint64_t v = v0 + u * B + tid;
                if (v < sh.nvec) {
                    const unsigned bits = in_regs ? bits_from_regs<T::EPV>(mk, v * T::EPV)
                                                  : marked_bits<T::EPV>(sh.marks, mp, mq, v * T::EPV);
                    if (MODE == kUpdate) {
                        update(x[u], bits);
                        store16<true>(x[u], sh.st + v);
                    } else {
                        if (MODE == kFill)
                            store16<true>(x[u], sh.st + v);
                        accum_vec<T>(x[u], bits, acc);
                    }
                }
            }
            mp = mq;
        }
    }
}

}  // namespace grover
