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
// complex64 n = 16 (binary32 update) 0.635 -> 0.32 ms, n = 20 3.49 -> 2.04, n = 24 14.1 -> 5.87 (7.3 us per
// iteration); complex128 n = 21 4.61 -> 1.91 ms (2.4 us per iteration).
#include <algorithm>

#include "held.h"

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

template <class T, bool U32, int NE>
__global__ __launch_bounds__(kChipBlock) void chip_iterate_kernel(ChipArgs a)
{
    constexpr int RE = NE > kChipRegE ? kChipRegE : NE, LE = NE - RE;
    constexpr bool kWide = std::is_same<T, C64>::value && !U32 && NE <= 16;
    using V = typename T::vec;
    __shared__ TeamShared<kChipBlock> sh;
    __shared__ V held[LE > 0 ? LE * kChipBlock : 1];
    __shared__ uint32_t words[WaveMarks<NE, kChipBlock, T::EPV>::kWords];
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
    // A limit of zero gives up here: at the barriers, members that arrive together would not have to wait.
    uint32_t error = 0u;
    if (threadIdx.x == 0) {
        if (a.timeout_ticks == 0u)
            __hip_atomic_store(&a.sync->error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        error = __hip_atomic_load(&a.sync->error, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const uint64_t base = uint64_t(rank) * a.per;
    (void)held_run<T, U32, kWide, NE, RE, kChipBlock, true>(
        static_cast<V *>(a.state) + base, base, a.per, a.marks, a.m, a.iters, a.scale, V{}, words,
        held + threadIdx.x,
        [&]() { return !__syncthreads_or(error != 0u); },
        [&](double &r, double &i) { return team_sum<kChipBlock>(r, i, tm, ++gen, sh); });
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
