// Batched searches in one persistent launch (many independent instances of Algorithm 5, complex64 states,
// binary64 sums, the update in binary64 or binary32).  The grid (one workgroup of 512 threads per CU, all
// co-resident) works through a sequence of phases, each with its own queue ordered by decreasing work N * k and
// its own team size T:
//   - in a phase with T > 1 the grid is split into teams of T workgroups; a team's leader takes the next
//     instance and publishes it through the team barrier, and the team iterates it with one team barrier per
//     iteration (which also reduces the sum).  The state is either held on chip by the team for all iterations
//     (resident phases: the instance fits T * 512 threads * the phase's vectors per thread, up to 32, all in
//     registers) or streamed from memory every iteration, as the fused single-instance kernel does;
//   - in a phase with T = 1 every workgroup takes instances alone: held on chip when the state fits (n <= 15),
//     otherwise streamed with workgroup-level sums only.
// Team sizes do not increase from one phase to the next and each divides the previous one, so the members
// of a team always come from one team of the previous phase (they finish it together) and no grid-wide
// barrier is needed between phases.  Which phases exist and their parameters is the tiling the host
// chooses; each instance starts from the uniform superposition.
//
// What bounds an iteration of a resident instance at n = 20 (T = 32): 2.2 us of update instructions (five per
// part, 32 vectors per thread, 4.2 cycles per instruction and SIMD), 1.2 us for the team barrier.  512 threads
// rather than 1024: all 32 vectors sit in registers (the other half of 16 went through LDS), and half the waves
// pay the reduction.  Two workgroups of 16 vectors per CU, to update one instance while another waits, do not
// overlap: a second workgroup on the CU lengthened the barrier from 1.4 to 2.9 us (T = 64), whatever the waves'
// priorities and the pace of the polls, and an n = 20 iteration to 4.5 us.  1024 searches of n = 8 .. 20: 32.2 -> 22.9
// ms on MI355X.
#include "batch.h"
#include "held.h"
#include "stream.h"

namespace grover {
namespace {

struct BatchArgs {
    float4 *state;
    const uint64_t *marks;
    const BatchInstance *inst;
    const uint32_t *queue;
    uint64_t qoff[kBatchMaxPhases + 1];
    uint32_t team[kBatchMaxPhases];
    uint32_t resident[kBatchMaxPhases];
    uint32_t nphases;
    uint32_t probe;
    unsigned long long *heads;
    GridSync *sync;
    uint64_t *partials;
    uint64_t timeout_ticks;
};

// Sets an error word (the team's, which its members' barrier waits poll, or the workgroup's own), which
// the host reads after the run and reports as a failure.
__device__ inline void flag_error(GridSync *word)
{
    if (threadIdx.x == 0)
        __hip_atomic_store(&word->error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ inline float4 uniform_vec(double amp)
{
    const float af = float(amp);
    return make_float4(af, 0.0f, af, 0.0f);
}

// One instance streamed by the T workgroups of a team (or by one).  Returns false when a barrier gave up.
template <bool U32, class Reduce>
__device__ bool run_streamed(const BatchArgs &a, const BatchInstance &I, unsigned rank, unsigned size, uint32_t *table,
                             Reduce reduce)
{
    const Share<C64> share{a.state + I.state_off, I.nvec, a.marks + I.marks_off, I.m, rank, size};
    const bool use_table = build_mark_table<kBatchBlock>(share, table);
    AccF64 acc0;
    stream_pass<kBatchBlock, C64, AccF64, kFill>(share, table, use_table, 0.0, 0.0, uniform_vec(I.amp), acc0);
    double sr = acc0.r, si = acc0.i;
    if (!reduce(sr, si))
        return false;
    const float4 none{};
    for (uint64_t it = 0; it < I.iters; ++it) {
        const double mr = (sr * 2.0) / I.N, mi = (si * 2.0) / I.N;
        AccF64 acc;
        stream_pass<kBatchBlock, C64, AccF64, kUpdate, U32>(share, table, use_table, mr, mi, none, acc);
        sr = acc.r;
        si = acc.i;
        if (!reduce(sr, si))
            return false;
    }
    return true;
}

// One instance held on chip by a team for all its iterations (member `rank` owns the contiguous vectors
// [rank * per, (rank + 1) * per), per = nvec / T a power of two), from the uniform state, in registers; written to
// memory once, at the end.  Returns false when a barrier gave up.
template <bool U32, int NE, class Reduce>
__device__ __forceinline__ bool run_held_ne(const BatchArgs &a, const BatchInstance &I, uint64_t base, uint64_t per,
                                            uint32_t *words, Reduce reduce)
{
    static_assert(WaveMarks<NE, kBatchBlock, 2>::kWords <= unsigned(kMarkWords), "the table holds a bit per amplitude");
    // 2/N is a power of two, so S * (2/N) rounds to the same binary64 value as 2S / N
    return held_run<C64, U32, !U32 && NE <= 16, NE, NE, kBatchBlock, false>(
        a.state + I.state_off + base, base, per, a.marks + I.marks_off, I.m, I.iters, 2.0 / I.N, uniform_vec(I.amp),
        words, static_cast<float4 *>(nullptr), []() { return true; }, reduce);
}

template <bool U32, class Reduce>
__device__ __forceinline__ bool run_held(const BatchArgs &a, const BatchInstance &I, uint64_t base, uint64_t per,
                                         uint32_t *words, Reduce reduce)
{
    switch (per < uint64_t(kBatchBlock) ? 1u : unsigned(per / kBatchBlock)) {
    case 1: return run_held_ne<U32, 1>(a, I, base, per, words, reduce);
    case 2: return run_held_ne<U32, 2>(a, I, base, per, words, reduce);
    case 4: return run_held_ne<U32, 4>(a, I, base, per, words, reduce);
    case 8: return run_held_ne<U32, 8>(a, I, base, per, words, reduce);
    case 16: return run_held_ne<U32, 16>(a, I, base, per, words, reduce);
    case 32: return run_held_ne<U32, 32>(a, I, base, per, words, reduce);
    default: return false;
    }
}

// kStreams = false compiles the kernel without the streamed paths, for tilings that hold every state on
// chip: the held loops then get the registers to themselves.  The host launches that instantiation only
// when no phase streams, so its streamed branches are never taken; were one taken, the kernel would report
// it through the error word instead of computing.  U32: the update in binary32 from 2S/N rounded to
// binary32; otherwise in binary64.
template <bool kStreams, bool U32>
__global__ __launch_bounds__(kBatchBlock) void batch_kernel(BatchArgs a)
{
    __shared__ TeamShared<kBatchBlock> sh;
    __shared__ uint32_t table[kMarkWords];  // of build_mark_table or WaveMarks::find
    const uint32_t grid = gridDim.x;
    if (a.probe) {
        const Team tm{a.sync, a.partials, grid, blockIdx.x, a.timeout_ticks};
        double zr = 0.0, zi = 0.0;
        (void)team_sum<kBatchBlock>(zr, zi, tm, 1u, sh);
        return;
    }
    // A limit of zero gives up before the first team's barrier (team sizes do not increase): at the barriers, members that
    // arrive together would not have to wait.
    if (a.timeout_ticks == 0u && a.nphases > 0u && a.team[0] > 1u) {
        flag_error(a.sync);
        return;
    }
    const unsigned major = xcd_major_block();
    for (uint32_t p = 0; p < a.nphases; ++p) {
        const uint64_t q0 = a.qoff[p], count = a.qoff[p + 1] - q0;
        const unsigned T = a.team[p];
        // a team of the whole grid meets in two levels by XCD, which ranks by launch order give (team_sum)
        const unsigned block = T == grid ? blockIdx.x : major;
        const unsigned teams = grid / T, team_id = block / T;
        if (count == 0 || team_id >= teams)
            continue;
        const Team tm{a.sync + uint64_t(p) * grid + team_id,
                      a.partials + uint64_t(p) * kBatchSlotWords * grid + uint64_t(team_id) * team_words(T), T, block % T,
                      a.timeout_ticks};
        uint64_t gen = 0;
        unsigned parity = 0;
        auto reduce = [&](double &r, double &i) {
            if (T == 1u) {
                block_allsum<kBatchBlock>(r, i, parity++, sh);
                return true;
            }
            return team_sum<kBatchBlock>(r, i, tm, ++gen, sh);
        };
        for (;;) {
            // the leader takes the next instance and contributes its index to a sum (exact in binary64: one
            // integer below 2^53 plus zeros), which hands it to every member
            double zr = 0.0, zi = 0.0;
            if (tm.rank == 0 && threadIdx.x == 0)
                zr = double(atomicAdd(&a.heads[p], 1ull));
            if (!reduce(zr, zi))
                return;
            const uint64_t qv = uint64_t(zr);  // the same in every lane; made scalar, as the instance's fields are
            const uint64_t q = __builtin_amdgcn_readfirstlane(uint32_t(qv)) |
                               (uint64_t(__builtin_amdgcn_readfirstlane(uint32_t(qv >> 32))) << 32);
            if (q >= count)
                break;
            const BatchInstance I = a.inst[a.queue[q0 + q]];
            bool ok;
            if (T == 1u ? I.nvec <= kBatchAloneVecs : a.resident[p] != 0u) {
                const uint64_t per = I.nvec / T;
                ok = run_held<U32>(a, I, uint64_t(tm.rank) * per, per, table, reduce);
            } else if (kStreams) {
                ok = run_streamed<U32>(a, I, tm.rank, T, table, reduce);
            } else {
                ok = false;
            }
            if (!ok) {
                flag_error(tm.sync);
                return;
            }
        }
    }
}

// Zeroes the phase heads, the team barriers and the member slots (whose generation tags the barriers
// compare against) before a run — a kernel, not a memset, so that the pair of launches can be captured into
// a graph and replayed.
__global__ void batch_reset_kernel(unsigned long long *heads, uint64_t nheads, uint64_t *sync_words, uint64_t nwords,
                                   uint64_t *slots, uint64_t nslots)
{
    const uint64_t i = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
    if (i < nheads)
        heads[i] = 0ull;
    for (uint64_t w = i; w < nwords; w += stride)
        sync_words[w] = 0u;
    for (uint64_t w = i; w < nslots; w += stride)
        slots[w] = 0u;
}

}  // namespace

const void *batch_kernel_fn(bool streams, bool u32)
{
    if (u32)
        return streams ? reinterpret_cast<const void *>(&batch_kernel<true, true>)
                       : reinterpret_cast<const void *>(&batch_kernel<false, true>);
    return streams ? reinterpret_cast<const void *>(&batch_kernel<true, false>)
                   : reinterpret_cast<const void *>(&batch_kernel<false, false>);
}

hipError_t launch_batch(const BatchLaunch &L)
{
    BatchArgs a;
    a.state = static_cast<float4 *>(L.state);
    a.marks = L.marks;
    a.inst = L.inst;
    a.queue = L.queue;
    for (int p = 0; p <= kBatchMaxPhases; ++p)
        a.qoff[p] = L.qoff[p];
    for (int p = 0; p < kBatchMaxPhases; ++p) {
        a.team[p] = L.team[p];
        a.resident[p] = L.resident[p];
    }
    a.nphases = L.nphases;
    a.probe = L.probe;
    a.heads = L.heads;
    a.sync = L.sync;
    a.partials = L.partials;
    a.timeout_ticks = L.timeout_ticks;
    unsigned long long *heads = L.heads;
    uint64_t nheads = kBatchMaxPhases;
    uint64_t *words = reinterpret_cast<uint64_t *>(L.sync);
    uint64_t nwords = uint64_t(kBatchMaxPhases) * uint64_t(L.grid) * sizeof(GridSync) / sizeof(uint64_t);
    uint64_t *slots = L.partials;
    uint64_t nslots = uint64_t(kBatchMaxPhases) * uint64_t(L.grid) * kBatchSlotWords;
    void *ra[] = {&heads, &nheads, &words, &nwords, &slots, &nslots};
    hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(&batch_reset_kernel), dim3(256), dim3(256), ra, 0,
                                   L.stream);
    if (e != hipSuccess)
        return e;
    void *args[] = {&a};
    return hipLaunchCooperativeKernel(batch_kernel_fn(L.streams != 0u, L.update != 0u), dim3(L.grid),
                                      dim3(kBatchBlock), args, 0, L.stream);
}

}  // namespace grover
