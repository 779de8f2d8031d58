// Measurement (Background, step 6).  The paper plots outcome probabilities but gives no sampling procedure;
// this library samples by inverse transform over an integer CDF so that the result is a function of the
// state's bits alone:
//   p_i = re^2 + im^2 (binary64, no fused multiply-add), q_i = floor(p_i 2^62), Q_i = q_0 + ... + q_i,
//   t_j = floor(U_j Q_{N-1} / 2^53), shot j -> the smallest i with Q_i > t_j.
// Integer addition is associative, so any grouping yields exactly the sequential prefix sums Q_i, and they need
// not be stored: a shot finds its CDF block (one or several tiles of 4096 amplitudes) among the blocks' prefix sums,
// its group of 16 or 64 among the block's, and adds up the group's q_i itself.  What is kept is one prefix sum per
// group, so the state is read once and little is written.  At n = 28 complex64 on MI355X, 10^6 shots of a searched
// state: 1.21 ms (block totals 0.33, their scan 0.11, the CDF written 0.74, searches 0.04) -> 0.45 ms.  States of
// up to kSmallN amplitudes (complex128: half) are sampled by one launch, every workgroup building the whole CDF in its
// LDS (four launches and their gaps before; 10^4 shots at n = 10: 11 -> 5.5 us).
#include "internal.h"

namespace grover {
namespace {

constexpr int kGroupBlock = 256;      // group sums: 256-thread workgroups striding over the CDF blocks
constexpr int kScanBlock = 1024;      // scan of the block totals: one workgroup
constexpr uint64_t kTile = 4096;      // amplitudes a workgroup takes at a time
// Tiles per CDF block: one for small states, so that there are workgroups enough; eight from 2^25 amplitudes on, which
// keeps the one workgroup that scans the blocks' totals to 8192 of them at n = 28 (65536: 0.05 ms).
constexpr uint64_t tiles_per_block(uint64_t N) { return N >= (uint64_t(1) << 25) ? 8u : 1u; }
// Amplitudes per group, G.  Smaller groups shorten the searches' last step, where a thread adds up its group's q (10^6
// shots of a spread state: 64 per group 0.03 ms more than 16), but their sums have to be written among the reads (2
// GiB: 64 per group 0.40 ms for the pass, 16 0.48, none 0.35): 16, one 128-byte line (`wide`, complex128: 8), while
// the state is small.
constexpr int group_size(uint64_t N, bool wide) { return N >= (uint64_t(1) << 25) ? 64 : wide ? 8 : 16; }
constexpr unsigned kKeepWords = 2048;  // group sums a workgroup collects in LDS before it writes them (16 KiB)
constexpr uint64_t kSmallN = 16384;   // one launch up to here (128 KiB of LDS; complex128, whose loads take longer: half)
constexpr uint64_t small_limit(bool wide) { return wide ? kSmallN / 2 : kSmallN; }
constexpr int kSmallBlock = 1024;
constexpr int kSearchBlock = 256;

__device__ inline double pval(double r, double m) { return __dadd_rn(__dmul_rn(r, r), __dmul_rn(m, m)); }
__device__ inline uint64_t qval(double r, double m) { return (uint64_t)__dmul_rn(pval(r, m), 0x1p62); }

// q of amplitude e of a storage vector
template <class T>
__device__ inline uint64_t qval_of(const typename T::vec &x, int e)
{
    return qval(T::re(x, e), T::im(x, e));
}

// floor(p 2^62) from the bits of p >= 0, for p < 4 (`top`, the high word of p, below kTopLimit): the significand with
// its leading bit at bit 63, shifted down.  About half the time of the conversion, which has no instruction.
constexpr uint32_t kTopLimit = 0x40100000u;  // high word of 4.0
__device__ inline uint64_t q_from_bits(double p, uint32_t &top)
{
    const uint64_t b = uint64_t(__double_as_longlong(p));
    top = uint32_t(b >> 32);
    const uint32_t down = 1024u - (top >> 20);  // 0 for [2, 4), 1 for [1, 2), ...
    const uint64_t m = (b << 11) | (uint64_t(1) << 63);
    return down < 64u ? m >> down : 0u;
}

// Sum of q over the amplitudes of two storage vectors.
template <class T>
__device__ inline uint64_t q_of_pair(const typename T::vec &x, const typename T::vec &y)
{
    uint64_t q = 0;
    uint32_t most = 0;
#pragma unroll
    for (int e = 0; e < T::EPV; ++e) {
        uint32_t t0, t1;
        q += q_from_bits(pval(T::re(x, e), T::im(x, e)), t0);
        q += q_from_bits(pval(T::re(y, e), T::im(y, e)), t1);
        most = max(most, max(t0, t1));
    }
    if (__any(most >= kTopLimit)) {  // an amplitude of magnitude 2 or more, infinite or NaN: as the conversion has it
        q = 0;
#pragma unroll
        for (int e = 0; e < T::EPV; ++e)
            q += qval_of<T>(x, e) + qval_of<T>(y, e);
    }
    return q;
}

// Inclusive scan of one uint64 per lane across the wave, by lane shuffles (six steps).
__device__ inline uint64_t wave_inclusive_scan(uint64_t x)
{
    const unsigned lane = threadIdx.x % kWave;
#pragma unroll
    for (unsigned off = 1; off < kWave; off <<= 1) {
        const uint64_t y = __shfl_up(x, off, kWave);
        if (lane >= off)
            x += y;
    }
    return x;
}

// Sum over aligned groups of L lanes (L = 2, 4, 8 or 16), in every lane, by DPP moves within a row.
template <int kCtrl>
__device__ inline uint64_t dpp_u64(uint64_t x)
{
    const unsigned lo = unsigned(__builtin_amdgcn_update_dpp(0, int(unsigned(x)), kCtrl, 0xf, 0xf, true));
    const unsigned hi = unsigned(__builtin_amdgcn_update_dpp(0, int(unsigned(x >> 32)), kCtrl, 0xf, 0xf, true));
    return (uint64_t(hi) << 32) | lo;
}
template <int L>
__device__ inline uint64_t group_sum(uint64_t x)
{
    static_assert(L == 2 || L == 4 || L == 8 || L == 16, "groups within a row of 16 lanes");
    x += dpp_u64<0xB1>(x);  // quad_perm 1,0,3,2
    if (L > 2)
        x += dpp_u64<0x4E>(x);  // quad_perm 2,3,0,1
    if (L > 4)
        x += dpp_u64<0x141>(x);  // row_half_mirror: the other quad of the half row
    if (L > 8)
        x += dpp_u64<0x140>(x);  // row_mirror: the other half row
    return x;
}

// Per CDF block: the inclusive prefix sums of its groups (within the block) and its total.  A workgroup reads a
// tile in rows of 256 x 2 adjacent vectors (32 bytes per thread, all rows in flight), sums the lanes of a group
// (complex128: of half a group) by DPP, and wave 0 collects the group sums from LDS and scans them, one
// or four per lane, from the block's sum so far.  Bound by reading the state.  The results of several tiles are
// collected in LDS and written together: written tile by tile among the reads, the 1.6 % of the bytes that groups of
// 64 have cost a quarter of the time (2 GiB: 0.43 ms).
template <class T, int G>
__global__ __launch_bounds__(kGroupBlock, T::EPV == 1 ? 4 : 8) void group_sums_kernel(const void *state, uint64_t nb, uint64_t tiles,
                                                                 uint64_t *group_prefix, uint64_t *block_sums)
{
    using V = typename T::vec;
    constexpr int R = int(kTile) / T::EPV / kGroupBlock / 2;  // rows
    constexpr unsigned kGroups = unsigned(kTile) / G;         // groups of a tile
    constexpr int kPer = int(kGroups) / kWave;                // groups of a lane in the scan
    constexpr int kLanes = G / T::EPV / 2;                    // lanes of a group
    constexpr int L = kLanes < 16 ? kLanes : 16;
    constexpr int kParts = kLanes / L;                        // LDS entries per group
    constexpr int kRowParts = kGroupBlock / L;
    constexpr unsigned kKeep = kKeepWords / kGroups;          // tiles collected
    // double-buffered by tile: a set is written again two tiles later, after the next tile's barrier, which wave 0
    // passes only after reading it
    __shared__ uint64_t gs[2][kGroups * kParts];
    __shared__ uint64_t kept[kKeep][kGroups];
    const V *st = static_cast<const V *>(state);
    const unsigned tid = threadIdx.x;
    uint64_t so_far = 0;     // wave 0: the block's sum before this tile
    uint64_t b = blockIdx.x, i = 0;  // block, and tile of the block
    for (unsigned n = 0, p = 0; b < nb; p ^= 1u) {  // n: tiles in `kept`
        // the state has more than small_limit amplitudes, two tiles and more, so every tile is full
        const V *from = st + (b * tiles + i) * (kTile / T::EPV) + 2u * tid;
        V x[R][2];
#pragma unroll
        for (int u = 0; u < R; ++u) {
            x[u][0] = load16<true>(from + u * 2 * kGroupBlock);
            x[u][1] = load16<true>(from + u * 2 * kGroupBlock + 1);
        }
#pragma unroll
        for (int u = 0; u < R; ++u) {
            const uint64_t q = group_sum<L>(q_of_pair<T>(x[u][0], x[u][1]));
            if (tid % L == 0)
                gs[p][u * kRowParts + tid / L] = q;
        }
        __syncthreads();
        if (tid < kWave) {
            uint64_t q[kPer], sum = 0;
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                q[j] = 0;
#pragma unroll
                for (int k = 0; k < kParts; ++k)
                    q[j] += gs[p][(tid * kPer + j) * kParts + k];
                sum += q[j];
            }
            const uint64_t incl = wave_inclusive_scan(sum) + so_far;
            uint64_t run = incl - sum;
#pragma unroll
            for (int j = 0; j < kPer; ++j) {
                run += q[j];
                kept[n][tid * kPer + j] = run;
            }
            so_far = i + 1u < tiles ? __shfl(incl, kWave - 1, kWave) : 0u;
        }
        ++n;
        const uint64_t last_b = b, last_i = i;
        if (++i == tiles) {
            i = 0;
            b += gridDim.x;
        }
        if (n == kKeep || b >= nb) {
            __syncthreads();
            // tile j of `kept` is the (n - 1 - j)-th before (last_b, last_i)
            const uint64_t end = (last_b / gridDim.x) * tiles + last_i;  // number of the last tile in this workgroup's order
            for (unsigned j = tid; j < n * kGroups; j += kGroupBlock) {
                const uint64_t t = end - (n - 1u - j / kGroups);
                const uint64_t tb = blockIdx.x + (t / tiles) * gridDim.x;
                group_prefix[(tb * tiles + t % tiles) * kGroups + j % kGroups] = kept[j / kGroups][j % kGroups];
                if (j % kGroups == kGroups - 1 && t % tiles == tiles - 1u)
                    block_sums[tb] = kept[j / kGroups][j % kGroups];
            }
            __syncthreads();
            n = 0;
        }
    }
}

// Single workgroup: block_sums[b] <- sum of block_sums[0 .. b-1] for b <= nb.  Chunks of 8 entries per thread (a
// 64-byte run each, the next chunk's loaded ahead), scanned across the workgroup with a running base.
__global__ __launch_bounds__(kScanBlock) void scan_block_totals_kernel(uint64_t *block_sums, uint64_t nb)
{
    constexpr int kRun = 8, kWaves = kScanBlock / kWave;
    constexpr uint64_t kChunk = uint64_t(kScanBlock) * kRun;
    __shared__ uint64_t wt[2][kWaves];
    const unsigned lane = threadIdx.x % kWave, wave = threadIdx.x / kWave;
    uint64_t base = 0;
    unsigned p = 0;
    uint64_t next[kRun];
    auto load = [&](uint64_t c) {
        const uint64_t j0 = c + uint64_t(threadIdx.x) * kRun;
#pragma unroll
        for (int i = 0; i < kRun; ++i)
            next[i] = j0 + i < nb ? block_sums[j0 + i] : 0u;
    };
    load(0);
    for (uint64_t c = 0; c < nb; c += kChunk, p ^= 1u) {
        const uint64_t j0 = c + uint64_t(threadIdx.x) * kRun;
        uint64_t x[kRun], sum = 0;
#pragma unroll
        for (int i = 0; i < kRun; ++i) {
            x[i] = next[i];
            sum += x[i];
        }
        load(c + kChunk);
        const uint64_t incl = wave_inclusive_scan(sum);
        if (lane == kWave - 1)
            wt[p][wave] = incl;
        __syncthreads();
        uint64_t before = 0, all = 0;
#pragma unroll
        for (unsigned w = 0; w < unsigned(kWaves); ++w) {
            const uint64_t t = wt[p][w];
            before += w < wave ? t : 0u;
            all += t;
        }
        uint64_t run = base + before + incl - sum;
#pragma unroll
        for (int i = 0; i < kRun; ++i) {
            if (j0 + i < nb)
                block_sums[j0 + i] = run;
            run += x[i];
        }
        base += all;
    }
    if (threadIdx.x == 0)
        block_sums[nb] = base;
}

// t_j = floor(U_j Q_{N-1} / 2^53) of shot j
__device__ inline uint64_t shot_threshold(const uint64_t *u53, uint64_t seed, int on_device, uint64_t j, uint64_t total)
{
    const uint64_t U = on_device ? (splitmix64(seed, j) >> 11) : (u53[j] & ((uint64_t(1) << 53) - 1u));
    const uint64_t hi = __umul64hi(U, total);
    const uint64_t lo = U * total;
    return (hi << 11) | (lo >> 53);
}

// One thread per shot: the block whose prefix sums enclose t, the group within it, then the amplitude.  n = 28, 10^6
// shots: 0.04-0.07 ms.
template <class T, int G>
__global__ __launch_bounds__(kSearchBlock) void search_kernel(const void *state, uint64_t tiles, const uint64_t *block_prefix, uint64_t nb,
                              const uint64_t *group_prefix, const uint64_t *u53, uint64_t seed, int on_device,
                              uint64_t shots, uint64_t *out, uint32_t *err)
{
    using V = typename T::vec;
    constexpr int W = G < 16 ? G : 16;       // amplitudes added up at a time (the state holds whole groups)
    constexpr uint64_t kVecs = W / T::EPV;
    const V *st = static_cast<const V *>(state);
    const uint64_t total = block_prefix[nb];
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
    for (uint64_t j = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; j < shots; j += stride) {
        if (total == 0) {
            if (j == 0)
                *err = 1u;
            out[j] = 0;
            continue;
        }
        uint64_t t = shot_threshold(u53, seed, on_device, j, total);
        // the last block whose exclusive prefix is <= t: t < total, so it holds a q > 0 beyond t
        uint64_t a = 0, b = nb - 1;
        while (a < b) {
            const uint64_t mid = a + ((b - a + 1) >> 1);
            if (block_prefix[mid] <= t)
                a = mid;
            else
                b = mid - 1;
        }
        const uint64_t block = a;
        t -= block_prefix[block];
        const uint64_t groups = tiles * (kTile / G), *gp = group_prefix + block * groups;
        uint64_t g = 0, h = groups - 1;  // the first group whose inclusive prefix exceeds t
        while (g < h) {
            const uint64_t mid = (g + h) >> 1;
            if (gp[mid] > t)
                h = mid;
            else
                g = mid + 1;
        }
        if (g > 0)
            t -= gp[g - 1];
        // the amplitude, W at a time
        uint64_t v = (block * groups + g) * (G / T::EPV), run = 0, index = 0;
        bool found = false;
        for (int part = 0; part < G / W && !found; ++part, v += kVecs) {
            V x[kVecs];
#pragma unroll
            for (uint64_t u = 0; u < kVecs; ++u)
                x[u] = st[v + u];
            uint64_t q[W];
            uint32_t most = 0;
#pragma unroll
            for (int i = 0; i < W; ++i) {
                uint32_t top;
                q[i] = q_from_bits(pval(T::re(x[i / T::EPV], i % T::EPV), T::im(x[i / T::EPV], i % T::EPV)), top);
                most = max(most, top);
            }
            if (most >= kTopLimit) {
#pragma unroll
                for (int i = 0; i < W; ++i)
                    q[i] = qval_of<T>(x[i / T::EPV], i % T::EPV);
            }
#pragma unroll
            for (int i = 0; i < W; ++i) {
                run += q[i];
                if (!found && run > t) {
                    found = true;
                    index = v * T::EPV + i;
                }
            }
        }
        out[j] = index;
    }
}

// States of up to small_limit amplitudes: every workgroup builds the CDF in LDS (1024 threads, each the vectors of one
// contiguous run of kSmallN / 1024 amplitudes or fewer) and serves its shots from there.  n = 10, 10^4 shots: one
// launch of about 4 us instead of four kernels.
template <class T>
__global__ __launch_bounds__(kSmallBlock) void small_sample_kernel(const void *state, uint64_t N, const uint64_t *u53,
                                                                   uint64_t seed, int on_device, uint64_t shots,
                                                                   uint64_t *out, uint32_t *err)
{
    using V = typename T::vec;
    constexpr int kWaves = kSmallBlock / kWave;
    constexpr int kMost = int(small_limit(T::kBytes == 16)) / kSmallBlock / T::EPV;  // vectors per thread
    __shared__ uint64_t cdf[kSmallN];
    __shared__ uint64_t wt[kWaves];
    const V *st = static_cast<const V *>(state);
    const unsigned tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const uint64_t nvec = N / T::EPV;
    const uint64_t per = (nvec + kSmallBlock - 1) / kSmallBlock;  // a power of two
    uint64_t q[kMost > 0 ? kMost : 1][T::EPV], sum = 0;
#pragma unroll
    for (int u = 0; u < (kMost > 0 ? kMost : 1); ++u) {
        const uint64_t v = uint64_t(tid) * per + u;
#pragma unroll
        for (int e = 0; e < T::EPV; ++e)
            q[u][e] = 0;
        if (uint64_t(u) < per && v < nvec) {
            const V x = st[v];
#pragma unroll
            for (int e = 0; e < T::EPV; ++e) {
                q[u][e] = qval_of<T>(x, e);
                sum += q[u][e];
            }
        }
    }
    const uint64_t incl = wave_inclusive_scan(sum);
    if (lane == kWave - 1)
        wt[wave] = incl;
    __syncthreads();
    uint64_t run = incl - sum, total = 0;
#pragma unroll
    for (unsigned w = 0; w < unsigned(kWaves); ++w) {
        const uint64_t t = wt[w];
        run += w < wave ? t : 0u;
        total += t;
    }
#pragma unroll
    for (int u = 0; u < (kMost > 0 ? kMost : 1); ++u) {
        const uint64_t v = uint64_t(tid) * per + u;
        if (uint64_t(u) < per && v < nvec)
#pragma unroll
            for (int e = 0; e < T::EPV; ++e) {
                run += q[u][e];
                cdf[v * T::EPV + e] = run;
            }
    }
    __syncthreads();
    const uint64_t stride = uint64_t(gridDim.x) * kSmallBlock;
    for (uint64_t j = uint64_t(blockIdx.x) * kSmallBlock + tid; j < shots; j += stride) {
        if (total == 0) {
            if (j == 0)
                *err = 1u;
            out[j] = 0;
            continue;
        }
        const uint64_t t = shot_threshold(u53, seed, on_device, j, total);
        uint64_t a = 0, b = N - 1;
        while (a < b) {
            const uint64_t mid = (a + b) >> 1;
            if (cdf[mid] > t)
                b = mid;
            else
                a = mid + 1;
        }
        out[j] = a;
    }
}

struct Kernels {
    const void *groups, *search, *small;
};

template <class T, int G>
Kernels kernels_of()
{
    return {reinterpret_cast<const void *>(&group_sums_kernel<T, G>),
            reinterpret_cast<const void *>(&search_kernel<T, G>),
            reinterpret_cast<const void *>(&small_sample_kernel<T>)};
}

template <class T>
Kernels kernels_for(uint64_t N)
{
    constexpr bool wide = T::kBytes == 16;
    return group_size(N, wide) == 64 ? kernels_of<T, 64>() : kernels_of<T, group_size(0, wide)>();
}

Kernels kernels_for(uint32_t dtype, uint64_t N)
{
    switch (dtype) {
    case GROVER_F64_REAL: return kernels_for<F64Real>(N);
    case GROVER_C64: return kernels_for<C64>(N);
    case GROVER_CBF16: return kernels_for<CBF16>(N);
    default: return kernels_for<C128>(N);
    }
}

uint64_t block_count(uint64_t N) { return N / (kTile * tiles_per_block(N)); }  // N > kTile: whole blocks

}  // namespace

// Words of the sampler's workspaces: the groups' prefix sums and the blocks' (with the total); 0 for a state that
// is sampled without them.
size_t sample_group_words(uint32_t dtype, uint64_t N)
{
    const bool wide = dtype == GROVER_C128;
    return N <= small_limit(wide) ? 0 : size_t(N / uint64_t(group_size(N, wide)));
}
size_t sample_block_words(uint64_t N) { return size_t(block_count(N) + 1); }

hipError_t launch_sample(grover_ctx *c, const uint64_t *u53_dev, uint64_t seed, bool device_uniforms,
                         uint64_t shots, uint64_t *out_dev)
{
    if (shots == 0)
        return hipSuccess;
    const Kernels k = kernels_for(c->dtype, c->N);
    const void *state = c->state;
    uint64_t N = c->N;
    int on_dev = device_uniforms ? 1 : 0;
    uint32_t *err = c->flag_dev;
    const uint64_t cus = uint64_t(c->cu_count > 0 ? c->cu_count : 256);
    if (N <= small_limit(c->dtype == GROVER_C128)) {
        const uint64_t want = (shots + kSmallBlock - 1) / kSmallBlock;
        void *a[] = {&state, &N, &u53_dev, &seed, &on_dev, &shots, &out_dev, &err};
        return hipLaunchKernel(k.small, dim3(unsigned(want < cus ? want : cus)), dim3(kSmallBlock), a, 0, c->stream);
    }
    uint64_t nb = block_count(N), tiles = tiles_per_block(N);
    uint64_t *gp = c->group_prefix, *bs = c->block_sums;
    // a few workgroups per CU, each striding over the CDF blocks
    const uint64_t cap = cus * 8u;
    const unsigned grid = unsigned(nb < cap ? nb : cap);
    void *a1[] = {&state, &nb, &tiles, &gp, &bs};
    hipError_t e = hipLaunchKernel(k.groups, dim3(grid), dim3(kGroupBlock), a1, 0, c->stream);
    if (e != hipSuccess)
        return e;
    void *a2[] = {&bs, &nb};
    e = hipLaunchKernel(reinterpret_cast<const void *>(&scan_block_totals_kernel), dim3(1), dim3(kScanBlock), a2, 0,
                        c->stream);
    if (e != hipSuccess)
        return e;
    const uint64_t want = (shots + kSearchBlock - 1) / kSearchBlock;
    const unsigned sgrid = unsigned(want < 65535 ? want : 65535);
    void *a3[] = {&state, &tiles, &bs, &nb, &gp, &u53_dev, &seed, &on_dev, &shots, &out_dev, &err};
    return hipLaunchKernel(k.search, dim3(sgrid), dim3(kSearchBlock), a3, 0, c->stream);
}

}  // namespace grover
