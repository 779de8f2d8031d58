// Generalized iteration with per-iteration phases, and its adjoint (reverse sweep) for the gradient.
//
// Iteration j (1 .. K) of schedule b applies O(phi_j) then D(theta_j), with
//   O(phi):   c_i <- e^{i phi} c_i on the marked indices (Algorithm 3 is phi = pi),
//   D(theta): c_i <- (1 - e^{i theta}) S / N - c_i with S the sum of the state (Eq. 2 is theta = pi),
// from the uniform superposition; the loss is L = 1 - sum over marked i of |c_i|^2.
//
// Forward: one pass per iteration, fused as in the plain kernel: the pass that writes c' = alpha - O c also
// accumulates the sum T of c' and the sum Mk of its marked entries, so the next iteration's
// S = sum O(phi') c' = T + (e^{i phi'} - 1) Mk needs no extra pass.  Every `every`-th state is also written
// to a checkpoint buffer.
//
// Adjoint: lambda = dL/d(conj c) starts as -g c on the marked entries (g = upstream gradient of L) and is
// carried back through the inverses of the unitary steps, D(theta)^-1 = D(-theta) and O(phi)^-1 = O(-phi),
// while the state is rebuilt backwards with the same inverses.  Step j needs the sums of c_j and
// lambda_j and yields, with y = O(phi_j) c_{j-1} = D(-theta_j) c_j and nu = D(-theta_j) lambda_j,
//   dL/dtheta_j = -2 Im( conj(sum lambda_j) * sum c_j ) / N,
//   dL/dphi_j   = -2 Im( sum over marked of conj(nu) * y ),
//   c_{j-1} = O(-phi_j) y,  lambda_{j-1} = O(-phi_j) nu,
// all in one pass that also accumulates the sums for step j - 1.  Where j - 1 is a checkpoint the state is
// re-read from it (the uniform state for j - 1 = 0) instead of being rebuilt, which bounds the drift of the
// rebuilt state to `every` steps.
//
// Storage is complex64 (float re, im); phases, sums and the element arithmetic are binary64.  A team of
// `team_size` workgroups iterates one schedule at a time, with one team barrier per iteration that also
// reduces six binary64 values; teams take schedules b = team, team + teams, ...
#include <algorithm>
#include <iterator>

#include "held.h"
#include "phase.h"

namespace grover {
namespace {

constexpr int kPV = 6;  // values a barrier reduces
constexpr int kStreamBlock = 1024;
constexpr int kStreamUnroll = kStreamTile / kStreamBlock;  // 16-byte vectors per thread per tile

struct C2 {
    double re, im;
};

__device__ inline C2 cmul(C2 a, C2 b) { return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }

struct PhaseShared {
    double red[kPV * (kStreamBlock / kWave)];  // wave sums, value by value
    double sum[kPV];
    int failed;
};

struct PhaseTeam {
    PhaseSync *sync;
    uint64_t *partials;  // [2][size][16]: kPV values as 16 tagged bytes each
    unsigned size;
    unsigned rank;
    uint64_t timeout_ticks;
};

// Team-wide sum of v[0 .. NV) (the other entries are left as they are), an all-gather as in the batched
// kernels' barrier (team_sum): every member publishes its partials in its slot of the generation's parity, 16
// tagged bytes per value; in every member wave 0 awaits the members' values and adds them in a fixed order, so
// all members compute identical sums.  Slots are double-buffered by parity (a slot is rewritten two generations
// later, after every member has read it).  Every thread gets the sums; false when the wait gave up.
//
// The first four values travel together through a wave's rows of 16 lanes: a wave's four sums take one fold and
// four row shifts, the workgroup's wave values of a value lie in one row, and a row gathers one value of 64
// members with four loads per lane.  Further values (only the marked amplitudes contribute to them: a wave that
// holds none passes `more` false and skips their sums) take one load per lane each, waited for together with the
// others.  LDS words are written again only after the first workgroup barrier of the next call, which every
// thread reaches after reading them.
template <int B, int NV>
__device__ bool team_sum_n(double (&v)[kPV], const PhaseTeam &tm, uint64_t gen, PhaseShared &sh, bool more = true)
{
    static_assert(NV >= 4 && NV <= kPV, "values per barrier");
    constexpr int kMore = NV - 4;
    constexpr unsigned kW = B / kWave;
    static_assert(kW == 8 || kW == 16, "a row per value");
    const uint32_t tag = uint32_t(gen);
    const unsigned tid = fresh_tid(), lane = tid % kWave, wave = tid / kWave;
    const unsigned row = lane / 16u, in_row = lane % 16u;
    const unsigned q = (row & 1u) * 2u + (row >> 1);  // the value of a row (fold_quad's order)
    {
        const double t = row_totals(fold_quad(v[0], v[1], v[2], v[3]));
        if (in_row == 15u)
            sh.red[q * kW + wave] = t;
    }
    if constexpr (kMore > 0) {
        double t = 0.0;
        if (more)
            t = half_totals(fold_pair(v[4], kMore > 1 ? v[kPV - 1] : 0.0));
        if (lane == 31u)
            sh.red[4u * kW + wave] = t;
        if (kMore > 1 && lane == 63u)
            sh.red[5u * kW + wave] = t;
    }
    __syncthreads();
    if (wave == 0) {
        const auto slots = buffer_rsrc(tm.partials + uint64_t(gen & 1u) * tm.size * 16u, tm.size * 128u);
        {
            const double t = row_totals(in_row < kW ? sh.red[q * kW + in_row] : 0.0);
            if (in_row == 15u)
                put_value(slots, tm.rank * 128u + q * 16u, t, tag);
        }
        if constexpr (kMore > 0) {
            const double t = row_totals(row < unsigned(kMore) && in_row < kW ? sh.red[(4u + row) * kW + in_row] : 0.0);
            if (in_row == 15u && row < unsigned(kMore))
                put_value(slots, tm.rank * 128u + (4u + row) * 16u, t, tag);
        }
        bool ok = true;
        double w = 0.0, u[2] = {0.0, 0.0};
        for (unsigned m0 = 0; m0 < tm.size && ok; m0 += kWave) {
            uint32_t off[4 + kMore];
            bool use[4 + kMore];
            double x[4 + kMore];
#pragma unroll
            for (unsigned i = 0; i < 4u; ++i) {
                const unsigned m = m0 + in_row + 16u * i;
                off[i] = m * 128u + q * 16u;
                use[i] = m < tm.size;
            }
#pragma unroll
            for (unsigned i = 0; i < unsigned(kMore); ++i) {
                off[4 + i] = (m0 + lane) * 128u + (4u + i) * 16u;
                use[4 + i] = m0 + lane < tm.size;
            }
            ok = wait_offsets<4 + kMore>(slots, off, use, tag, &tm.sync->error, tm.timeout_ticks, x);
            w += (x[0] + x[1]) + (x[2] + x[3]);
#pragma unroll
            for (int i = 0; i < kMore; ++i)
                u[i] += x[4 + i];
        }
        w = row_totals(w);
        if (in_row == 15u)
            sh.sum[q] = w;
        if constexpr (kMore > 0) {
            const double t = half_totals(fold_pair(u[0], u[1]));
            if (lane == 31u)
                sh.sum[4] = t;
            if (lane == 63u)
                sh.sum[5] = t;
        }
        const bool failed = __any(!ok);
        if (lane == 0)
            sh.failed = failed;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < NV; ++i)
        v[i] = sh.sum[i];
    return sh.failed == 0;
}

struct PhaseArgs {
    float4 *state;   // [B][nvec]
    float4 *lambda;  // [B][nvec]
    float4 *ckpt;    // [B][nck][nvec]
    const uint64_t *marks;
    uint64_t m;
    uint64_t nvec;
    uint64_t per;  // on-chip form: vectors per member
    double N;
    float amp;  // uniform amplitude rounded to binary32
    uint32_t B, K, every, nck;
    const double *phi, *theta;  // [B][K]
    double *loss;               // [B]
    double *aux;                // [B][2] sum of the final state (forward -> adjoint)
    const double *dloss;        // [B]
    double *dphi, *dtheta;      // [B][K]
    PhaseSync *sync;            // one per team
    uint64_t *partials;         // [teams][2][T][16]
    uint32_t team_size;
    uint32_t probe;  // 1: only meet once at a barrier of the whole grid (residency check)
    uint64_t timeout_ticks;
};

// A limit of zero gives up before the first barrier: at the barriers, members that arrive together would not have to wait.
__device__ inline bool gives_up(const PhaseArgs &a, const PhaseTeam &tm)
{
    if (a.timeout_ticks == 0u && threadIdx.x == 0)
        __hip_atomic_store(&tm.sync->error, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return a.timeout_ticks == 0u;
}

// Marked entries of one tile: the slice [mp, mq) of the sorted list, held in registers when short.
struct TileMarks {
    uint64_t mp, mq;
    bool in_regs;
    uint64_t mk[kTileMarks];
    __device__ void load(const uint64_t *marks, uint64_t m, uint64_t v0)
    {
        mp = gallop_lower_bound(marks, mp, m, v0 * 2u);
        mq = gallop_lower_bound(marks, mp, m, (v0 + kStreamTile) * 2u);
        in_regs = mq - mp <= uint64_t(kTileMarks);
#pragma unroll
        for (int q = 0; q < kTileMarks; ++q)
            mk[q] = in_regs && mp + q < mq ? marks[mp + q] : ~uint64_t(0);
    }
    __device__ unsigned bits(const uint64_t *marks, uint64_t v) const
    {
        return in_regs ? bits_from_regs<2>(mk, v * 2u) : marked_bits<2>(marks, mp, mq, v * 2u);
    }
};

__device__ inline C2 lo(const float4 &x) { return {double(x.x), double(x.y)}; }
__device__ inline C2 hi(const float4 &x) { return {double(x.z), double(x.w)}; }
__device__ inline float4 pack(C2 a, C2 b) { return make_float4(float(a.re), float(a.im), float(b.re), float(b.im)); }

// The team-rank-th share of one state: tiles t = rank + j * size (kStreamTile vectors each).
__device__ inline uint64_t share_tiles(uint64_t nvec, unsigned rank, unsigned size)
{
    const uint64_t nt = (nvec + kStreamTile - 1) / kStreamTile;
    return rank < nt ? (nt - rank + size - 1) / size : 0;
}

// Does local tile j of this workgroup's share hold a marked amplitude?  From the LDS table when it could be
// built, otherwise assume it may (the tile then finds its marks by search).
__device__ inline bool tile_marked(const PhaseArgs &a, const uint32_t *table, bool use_table, uint64_t j)
{
    return use_table ? ((table[j >> 5] >> (j & 31)) & 1u) != 0u : a.m > 0;
}

// The table of this workgroup's tiles that hold marked amplitudes; every schedule shares the marked set and
// the tile assignment, so it is built once per launch.
__device__ inline bool build_phase_table(const PhaseArgs &a, const PhaseTeam &tm, uint32_t *table)
{
    const Share<C64> share{nullptr, a.nvec, a.marks, a.m, tm.rank, tm.size};
    return build_mark_table<kStreamBlock>(share, table);
}

// Forward pass over a team's share.  mode 0: write the uniform state; mode 1: c' = alpha - O(phi) c.
// Accumulates v = {sum re, sum im, marked sum re, marked sum im, marked |c|^2, 0} of the values stored.
__device__ void forward_pass(const PhaseArgs &a, float4 *st, float4 *ck, const PhaseTeam &tm, const uint32_t *table,
                             bool use_table, int mode, C2 alpha, C2 ephi, double (&v)[kPV])
{
    const unsigned tid = threadIdx.x;
    const uint64_t cnt = share_tiles(a.nvec, tm.rank, tm.size);
    TileMarks tmk;
    tmk.mp = 0;
    for (uint64_t j = 0; j < cnt; ++j) {
        const uint64_t v0 = (tm.rank + j * tm.size) * uint64_t(kStreamTile);
        const bool fast = !tile_marked(a, table, use_table, j) && v0 + kStreamTile <= a.nvec;
        if (!fast)
            tmk.load(a.marks, a.m, v0);
        float4 x[kStreamUnroll];
#pragma unroll
        for (int u = 0; u < kStreamUnroll; ++u) {
            const uint64_t vi = v0 + u * kStreamBlock + tid;
            if (fast || vi < a.nvec)
                x[u] = mode == 0 ? make_float4(a.amp, 0.0f, a.amp, 0.0f) : load16<true>(st + vi);
        }
#pragma unroll
        for (int u = 0; u < kStreamUnroll; ++u) {
            const uint64_t vi = v0 + u * kStreamBlock + tid;
            if (!fast && vi >= a.nvec)
                continue;
            const unsigned bits = fast ? 0u : tmk.bits(a.marks, vi);
            float4 out;
            if (mode == 0) {
                out = x[u];
            } else {
                C2 c0 = lo(x[u]), c1 = hi(x[u]);
                if (bits & 1u)
                    c0 = cmul(ephi, c0);
                if (bits & 2u)
                    c1 = cmul(ephi, c1);
                out = pack({alpha.re - c0.re, alpha.im - c0.im}, {alpha.re - c1.re, alpha.im - c1.im});
            }
            store16<true>(out, st + vi);
            if (ck)
                store16<true>(out, ck + vi);
            const C2 r0 = lo(out), r1 = hi(out);
            v[0] += r0.re + r1.re;
            v[1] += r0.im + r1.im;
            if (bits & 1u) {
                v[2] += r0.re;
                v[3] += r0.im;
                v[4] += r0.re * r0.re + r0.im * r0.im;
            }
            if (bits & 2u) {
                v[2] += r1.re;
                v[3] += r1.im;
                v[4] += r1.re * r1.re + r1.im * r1.im;
            }
        }
        if (!fast)
            tmk.mp = tmk.mq;
    }
}

__global__ __launch_bounds__(kStreamBlock) void phase_forward_kernel(PhaseArgs a)
{
    __shared__ PhaseShared sh;
    __shared__ uint32_t table[kMarkWords];
    const unsigned T = a.team_size, teams = gridDim.x / T, team_id = xcd_major_block() / T;
    if (team_id >= teams)
        return;
    const PhaseTeam tm{a.sync + team_id, a.partials + uint64_t(team_id) * 32u * T, T, xcd_major_block() % T,
                       a.timeout_ticks};
    uint64_t gen = 0;
    if (a.probe) {
        double v[kPV] = {};
        (void)team_sum_n<kStreamBlock, kPV>(v, tm, ++gen, sh);
        return;
    }
    if (gives_up(a, tm))
        return;
    const bool use_table = build_phase_table(a, tm, table);
    for (uint32_t b = team_id; b < a.B; b += teams) {
        float4 *st = a.state + uint64_t(b) * a.nvec;
        double v[kPV] = {};
        forward_pass(a, st, nullptr, tm, table, use_table, 0, {0.0, 0.0}, {1.0, 0.0}, v);
        if (!team_sum_n<kStreamBlock, kPV>(v, tm, ++gen, sh))
            return;
        for (uint32_t k = 1; k <= a.K; ++k) {
            const double ph = a.phi[uint64_t(b) * a.K + k - 1], th = a.theta[uint64_t(b) * a.K + k - 1];
            const C2 ephi{cos(ph), sin(ph)}, eth{cos(th), sin(th)};
            // S = sum of O(phi) c = T + (e^{i phi} - 1) Mk;  alpha = (1 - e^{i theta}) S / N
            const C2 S = {v[0] + (ephi.re - 1.0) * v[2] - ephi.im * v[3], v[1] + (ephi.re - 1.0) * v[3] + ephi.im * v[2]};
            const C2 f = cmul({1.0 - eth.re, -eth.im}, S);
            const C2 alpha{f.re / a.N, f.im / a.N};
            float4 *ck = (k % a.every == 0 && k < a.K)
                             ? a.ckpt + (uint64_t(b) * a.nck + (k / a.every - 1u)) * a.nvec
                             : nullptr;
            double w[kPV] = {};
            forward_pass(a, st, ck, tm, table, use_table, 1, alpha, ephi, w);
            if (!team_sum_n<kStreamBlock, kPV>(w, tm, ++gen, sh))
                return;
#pragma unroll
            for (int q = 0; q < kPV; ++q)
                v[q] = w[q];
        }
        if (tm.rank == 0 && threadIdx.x == 0) {
            a.loss[b] = 1.0 - v[4];
            a.aux[2u * b] = v[0];
            a.aux[2u * b + 1u] = v[1];
        }
    }
}

// Adjoint seed: lambda = -g c on the marked entries, 0 elsewhere; accumulates its sum into v[2], v[3].
__device__ void lambda_seed_pass(const PhaseArgs &a, const float4 *st, float4 *lam, const PhaseTeam &tm,
                                 const uint32_t *table, bool use_table, double g, double (&v)[kPV])
{
    const unsigned tid = threadIdx.x;
    const uint64_t cnt = share_tiles(a.nvec, tm.rank, tm.size);
    TileMarks tmk;
    tmk.mp = 0;
    for (uint64_t j = 0; j < cnt; ++j) {
        const uint64_t v0 = (tm.rank + j * tm.size) * uint64_t(kStreamTile);
        const bool marked = tile_marked(a, table, use_table, j);
        if (marked)
            tmk.load(a.marks, a.m, v0);
#pragma unroll
        for (int u = 0; u < kStreamUnroll; ++u) {
            const uint64_t vi = v0 + u * kStreamBlock + tid;
            if (vi >= a.nvec)
                continue;
            const unsigned bits = !marked || tmk.mq == tmk.mp ? 0u : tmk.bits(a.marks, vi);
            float4 out = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            if (bits) {
                const float4 x = st[vi];
                const C2 c0 = lo(x), c1 = hi(x);
                const C2 l0 = (bits & 1u) ? C2{-g * c0.re, -g * c0.im} : C2{0.0, 0.0};
                const C2 l1 = (bits & 2u) ? C2{-g * c1.re, -g * c1.im} : C2{0.0, 0.0};
                out = pack(l0, l1);
                const C2 r0 = lo(out), r1 = hi(out);
                v[2] += r0.re + r1.re;
                v[3] += r0.im + r1.im;
            }
            store16<true>(out, lam + vi);
        }
        if (marked)
            tmk.mp = tmk.mq;
    }
}

// One reverse step over a team's share (see the file comment).  src: the checkpoint to re-read c_{j-1}
// from, or null with anchor set for the uniform state, or anchor clear to rebuild from the state.
// Accumulates v = {sum c_{j-1}, sum lambda_{j-1}, sum over marked of conj(nu) y}.
__device__ void reverse_pass(const PhaseArgs &a, float4 *st, float4 *lam, const float4 *src, bool anchor,
                             const PhaseTeam &tm, const uint32_t *table, bool use_table, C2 beta_c, C2 beta_l,
                             C2 ephi, double (&v)[kPV])
{
    const unsigned tid = threadIdx.x;
    const uint64_t cnt = share_tiles(a.nvec, tm.rank, tm.size);
    const C2 emphi{ephi.re, -ephi.im};
    TileMarks tmk;
    tmk.mp = 0;
    for (uint64_t j = 0; j < cnt; ++j) {
        const uint64_t v0 = (tm.rank + j * tm.size) * uint64_t(kStreamTile);
        const bool fast = !tile_marked(a, table, use_table, j) && v0 + kStreamTile <= a.nvec;
        if (!fast)
            tmk.load(a.marks, a.m, v0);
        float4 xc[kStreamUnroll], xl[kStreamUnroll];
#pragma unroll
        for (int u = 0; u < kStreamUnroll; ++u) {
            const uint64_t vi = v0 + u * kStreamBlock + tid;
            if (fast || vi < a.nvec) {
                if (!anchor)
                    xc[u] = load16<true>(st + vi);
                else
                    xc[u] = src ? load16<true>(src + vi) : make_float4(a.amp, 0.0f, a.amp, 0.0f);
                xl[u] = load16<true>(lam + vi);
            }
        }
#pragma unroll
        for (int u = 0; u < kStreamUnroll; ++u) {
            const uint64_t vi = v0 + u * kStreamBlock + tid;
            if (!fast && vi >= a.nvec)
                continue;
            const unsigned bits = fast ? 0u : tmk.bits(a.marks, vi);
            C2 cp[2], lp[2];
            const C2 cin[2] = {lo(xc[u]), hi(xc[u])}, lin[2] = {lo(xl[u]), hi(xl[u])};
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const bool mk = (bits >> e) & 1u;
                C2 y;
                if (anchor) {
                    cp[e] = cin[e];
                    y = mk ? cmul(ephi, cin[e]) : cin[e];
                } else {
                    y = {beta_c.re - cin[e].re, beta_c.im - cin[e].im};
                    cp[e] = mk ? cmul(emphi, y) : y;
                }
                const C2 nu{beta_l.re - lin[e].re, beta_l.im - lin[e].im};
                lp[e] = mk ? cmul(emphi, nu) : nu;
                if (mk) {
                    // conj(nu) * y
                    v[4] += nu.re * y.re + nu.im * y.im;
                    v[5] += nu.re * y.im - nu.im * y.re;
                }
            }
            const float4 oc = pack(cp[0], cp[1]), ol = pack(lp[0], lp[1]);
            store16<true>(oc, st + vi);
            store16<true>(ol, lam + vi);
            v[0] += double(oc.x) + double(oc.z);
            v[1] += double(oc.y) + double(oc.w);
            v[2] += double(ol.x) + double(ol.z);
            v[3] += double(ol.y) + double(ol.w);
        }
        if (!fast)
            tmk.mp = tmk.mq;
    }
}

__global__ __launch_bounds__(kStreamBlock) void phase_adjoint_kernel(PhaseArgs a)
{
    __shared__ PhaseShared sh;
    __shared__ uint32_t table[kMarkWords];
    const unsigned T = a.team_size, teams = gridDim.x / T, team_id = xcd_major_block() / T;
    if (team_id >= teams)
        return;
    const PhaseTeam tm{a.sync + team_id, a.partials + uint64_t(team_id) * 32u * T, T, xcd_major_block() % T,
                       a.timeout_ticks};
    uint64_t gen = 0;
    if (a.probe) {
        double v[kPV] = {};
        (void)team_sum_n<kStreamBlock, kPV>(v, tm, ++gen, sh);
        return;
    }
    if (gives_up(a, tm))
        return;
    const bool leader = tm.rank == 0 && threadIdx.x == 0;
    const bool use_table = build_phase_table(a, tm, table);
    for (uint32_t b = team_id; b < a.B; b += teams) {
        float4 *st = a.state + uint64_t(b) * a.nvec;
        float4 *lam = a.lambda + uint64_t(b) * a.nvec;
        double v[kPV] = {};
        lambda_seed_pass(a, st, lam, tm, table, use_table, a.dloss[b], v);
        if (!team_sum_n<kStreamBlock, kPV>(v, tm, ++gen, sh))
            return;
        C2 sc{a.aux[2u * b], a.aux[2u * b + 1u]}, sl{v[2], v[3]};
        for (uint32_t k = a.K; k >= 1; --k) {
            const uint64_t pk = uint64_t(b) * a.K + k - 1;
            const double ph = a.phi[pk], th = a.theta[pk];
            if (leader)  // -2 Im(conj(sum lambda) * sum c) / N
                a.dtheta[pk] = -2.0 * (sl.re * sc.im - sl.im * sc.re) / a.N;
            const C2 emth{cos(th), -sin(th)};
            const C2 om{1.0 - emth.re, -emth.im};
            const C2 fc = cmul(om, sc), fl = cmul(om, sl);
            const C2 beta_c{fc.re / a.N, fc.im / a.N}, beta_l{fl.re / a.N, fl.im / a.N};
            const bool anchor = (k - 1u) % a.every == 0u;
            const float4 *src = (anchor && k - 1u > 0u)
                                    ? a.ckpt + (uint64_t(b) * a.nck + ((k - 1u) / a.every - 1u)) * a.nvec
                                    : nullptr;
            double w[kPV] = {};
            reverse_pass(a, st, lam, src, anchor, tm, table, use_table, beta_c, beta_l, {cos(ph), sin(ph)}, w);
            if (!team_sum_n<kStreamBlock, kPV>(w, tm, ++gen, sh))
                return;
            if (leader)  // -2 Im(sum over marked of conj(nu) y)
                a.dphi[pk] = -2.0 * w[5];
            sc = {w[0], w[1]};
            sl = {w[2], w[3]};
        }
    }
}

// ------------------------------------------------------------------------------ on-chip form
// For states small enough to stay on chip the same iteration and reverse sweep run with each state held in its
// team's registers for all K steps, so that the only memory traffic is the checkpoints, the final state and the
// reads of the checkpoints in the reverse sweep.  Team size T (a power of two, set by the host from the state
// size): member `rank` owns the contiguous vectors [rank * per, (rank + 1) * per), per = nvec / T, and thread tid
// the vectors rank * per + e * 512 + tid, e < NE = per / 512 (or, when per < 512, the one vector tid < per).
// Forward: up to 32 vectors per thread; adjoint: up to 16 of the state and 16 of the adjoint state.  The marked
// set is the same for every schedule and step, so each wave finds its marks once per launch (WaveMarks).
//
// What bounds a step is the update's instructions (five per part: 2.2 us with 32 vectors per thread) and the team
// barrier (1.2-1.5 us).  512 threads rather than 1024 keep all held vectors in registers (half of them went through
// LDS) and halve the waves that pay the reduction.
constexpr int kHeldBlock = 512;

// e^{i phi_k} and e^{i theta_k} of one schedule for a chunk of kTrigChunk steps, computed once by the
// workgroup's threads (step k0 + i by thread i) into LDS instead of at every step by every thread: on chip a
// step costs a few microseconds, and binary64 sine and cosine plus the loads of the phases would be a large
// part of that.  Entry i holds {cos phi, sin phi, cos theta, sin theta} of step k0 + i (0-based).  Called by
// every thread at the same step; the barrier at its end publishes the table, and the table is rewritten
// only after the next team barrier, which every thread reaches after its last read of the old entries.
constexpr uint32_t kTrigChunk = 512;

struct TrigTable {
    double v[4][kTrigChunk];
};

__device__ inline void fill_trig(const PhaseArgs &a, uint32_t b, uint32_t k0, TrigTable &t)
{
    for (uint32_t i = threadIdx.x; i < kTrigChunk && k0 + i < a.K; i += kHeldBlock) {
        const uint64_t pk = uint64_t(b) * a.K + k0 + i;
        double sp, cp, sth, cth;
        sincos(a.phi[pk], &sp, &cp);
        sincos(a.theta[pk], &sth, &cth);
        t.v[0][i] = cp;
        t.v[1][i] = sp;
        t.v[2][i] = cth;
        t.v[3][i] = sth;
    }
    __syncthreads();
}

// A held vector's four parts {re, im, re, im}.
using Vec4 = float[4];

__device__ inline void unpack(const float4 &v, Vec4 &x)
{
    x[0] = v.x;
    x[1] = v.y;
    x[2] = v.z;
    x[3] = v.w;
}
__device__ inline float4 packed(const Vec4 &x) { return make_float4(x[0], x[1], x[2], x[3]); }

// A vector's parts into (sr, si).  The empty asm hides that the parts are still the values widened here: else the
// compiler keeps all the widened values for the next step, which there are no registers for.  It takes the sums
// too, so that the additions stay ahead of it and need no copies of the parts.
__device__ inline void add_parts(Vec4 &x, double &sr, double &si)
{
    sr += double(x[0]) + double(x[2]);
    si += double(x[1]) + double(x[3]);
    asm("" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(sr), "+v"(si));
}

// Makes the parts other values to the compiler in this branch, so that it does not merge the branch's widening
// conversions with another branch's and compute all of them ahead of both.
template <int NE>
__device__ inline void own_values(Vec4 (&x)[NE])
{
#pragma unroll
    for (int r = 0; r < NE; ++r)
#pragma unroll
        for (int p = 0; p < 4; ++p)
            asm volatile("" : "+v"(x[r][p]));
}

// One step of one vector without marked amplitudes: c' = m - c.
__device__ inline void plain_step(Vec4 &x, C2 m, double &sr, double &si)
{
#pragma unroll
    for (int p = 0; p < 4; ++p)
        x[p] = float((p & 1 ? m.im : m.re) - double(x[p]));
    add_parts(x, sr, si);
}

// One forward step of a vector that may hold marked amplitudes: c' = alpha - O(phi) c; the stored values' sums go to
// w ({sum, marked sum, marked |c|^2}, as forward_pass).
__device__ inline void marked_forward(Vec4 &x, unsigned bits, C2 alpha, C2 ephi, double (&w)[kPV])
{
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const C2 c{double(x[2 * e]), double(x[2 * e + 1])};
        const C2 o = (bits >> e) & 1u ? cmul(ephi, c) : c;
        x[2 * e] = float(alpha.re - o.re);
        x[2 * e + 1] = float(alpha.im - o.im);
    }
#pragma unroll
    for (int e = 0; e < 2; ++e)
        if ((bits >> e) & 1u) {
            const C2 r{double(x[2 * e]), double(x[2 * e + 1])};
            w[2] += r.re;
            w[3] += r.im;
            w[4] += r.re * r.re + r.im * r.im;
        }
    add_parts(x, w[0], w[1]);
}

template <int NE, bool kRest>
__global__ __launch_bounds__(kHeldBlock) void phase_forward_held_kernel(PhaseArgs a)
{
    __shared__ PhaseShared sh;
    __shared__ TrigTable trig;
    __shared__ uint32_t words[WaveMarks<NE, kHeldBlock, 2>::kWords];
    const unsigned T = a.team_size, teams = gridDim.x / T, team_id = xcd_major_block() / T;
    if (team_id >= teams)
        return;
    const PhaseTeam tm{a.sync + team_id, a.partials + uint64_t(team_id) * 32u * T, T, xcd_major_block() % T,
                       a.timeout_ticks};
    uint64_t gen = 0;
    if (a.probe) {
        double v[kPV] = {};
        (void)team_sum_n<kHeldBlock, 4>(v, tm, ++gen, sh);
        return;
    }
    if (gives_up(a, tm))
        return;
    const unsigned tid = threadIdx.x;
    const uint64_t per = a.per, base = uint64_t(tm.rank) * per;
    const bool active = NE > 1 || tid < per;
    WaveMarks<NE, kHeldBlock, 2> wm;
    wm.find(a.marks, a.m, base, per, words);
    const double inv_n = 1.0 / a.N;  // N is a power of two: x * (1/N) rounds as x / N
    auto at = [&](unsigned r, unsigned t16) { return (r ^ wm.swap) * unsigned(kHeldBlock * 16) + t16; };
    auto store = [&](float4 *to, Vec4 (&x)[NE]) {
        const auto rs = buffer_rsrc(to, uint32_t(per * 16u));
        const unsigned t16 = fresh_tid() * 16u;
#pragma unroll
        for (int r = 0; r < NE; ++r)
            bstore16<kBufNT>(packed(x[r]), rs, at(r, t16));
    };
    for (uint32_t b = team_id; b < a.B; b += teams) {
        float4 *st = a.state + uint64_t(b) * a.nvec + base;
        Vec4 x[NE];
        double v[kPV] = {};
        if (active) {
            // the sums of the uniform state, as the first pass of the streamed form computes them
#pragma unroll
            for (int r = 0; r < NE; ++r) {
                unpack(make_float4(a.amp, 0.0f, a.amp, 0.0f), x[r]);
                v[0] += double(a.amp) + double(a.amp);
            }
            if (wm.any)
#pragma unroll
                for (int r = 0; r < (kRest ? NE : 1); ++r)
#pragma unroll
                    for (int e = 0; e < 2; ++e)
                        if ((wm.mk.at(r) >> e) & 1u) {
                            v[2] += double(a.amp);
                            v[4] += double(a.amp) * double(a.amp);
                        }
        }
        // the next step needs the total and the marked sum (4 values); the last one also the marked |c|^2
        if (!team_sum_n<kHeldBlock, 4>(v, tm, ++gen, sh))
            return;
        for (uint32_t k = 1; k <= a.K; ++k) {
            const uint32_t i = (k - 1u) % kTrigChunk;
            if (i == 0u)
                fill_trig(a, b, k - 1u, trig);
            const C2 ephi{trig.v[0][i], trig.v[1][i]}, eth{trig.v[2][i], trig.v[3][i]};
            const C2 S = {v[0] + (ephi.re - 1.0) * v[2] - ephi.im * v[3], v[1] + (ephi.re - 1.0) * v[3] + ephi.im * v[2]};
            const C2 f = cmul({1.0 - eth.re, -eth.im}, S);
            const C2 alpha{f.re * inv_n, f.im * inv_n};
            double w[kPV] = {};
            if (active) {
                if (wm.any)
                    marked_forward(x[0], wm.mk.at(0), alpha, ephi, w);
                else
                    plain_step(x[0], alpha, w[0], w[1]);
#pragma unroll
                for (int r = 1; r < NE; ++r) {
                    if (kRest && wm.in_rest(r))
                        marked_forward(x[r], wm.mk.at(r), alpha, ephi, w);
                    else
                        plain_step(x[r], alpha, w[0], w[1]);
                }
                if (k % a.every == 0 && k < a.K)
                    store(a.ckpt + (uint64_t(b) * a.nck + (k / a.every - 1u)) * a.nvec + base, x);
            }
            if (!(k == a.K ? team_sum_n<kHeldBlock, 5>(w, tm, ++gen, sh, wm.any != 0u)
                           : team_sum_n<kHeldBlock, 4>(w, tm, ++gen, sh)))
                return;
#pragma unroll
            for (int q = 0; q < kPV; ++q)
                v[q] = w[q];
        }
        // the final state goes to memory: the adjoint starts from it, and it is the result
        if (active)
            store(st, x);
        if (tm.rank == 0 && tid == 0) {
            a.loss[b] = 1.0 - v[4];
            a.aux[2u * b] = v[0];
            a.aux[2u * b + 1u] = v[1];
        }
    }
}

// One reverse step of one pair of vectors (state xc, adjoint state xl) that may hold marked amplitudes, as
// reverse_pass: with anchor set xc is c_{j-1} already (a checkpoint or the uniform state) instead of being rebuilt.
__device__ inline void marked_reverse(Vec4 &xc, Vec4 &xl, bool anchor, unsigned bits, C2 beta_c, C2 beta_l, C2 ephi,
                                      double (&w)[kPV])
{
    const C2 emphi{ephi.re, -ephi.im};
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const bool mk = (bits >> e) & 1u;
        const C2 c{double(xc[2 * e]), double(xc[2 * e + 1])}, l{double(xl[2 * e]), double(xl[2 * e + 1])};
        C2 y;
        if (anchor) {
            y = mk ? cmul(ephi, c) : c;
        } else {
            y = {beta_c.re - c.re, beta_c.im - c.im};
            const C2 o = mk ? cmul(emphi, y) : y;
            xc[2 * e] = float(o.re);
            xc[2 * e + 1] = float(o.im);
        }
        const C2 nu{beta_l.re - l.re, beta_l.im - l.im};
        const C2 p = mk ? cmul(emphi, nu) : nu;
        xl[2 * e] = float(p.re);
        xl[2 * e + 1] = float(p.im);
        if (mk)  // Im(conj(nu) y), the only part the gradient uses
            w[4] += nu.re * y.im - nu.im * y.re;
    }
    add_parts(xc, w[0], w[1]);
    add_parts(xl, w[2], w[3]);
}

__device__ inline void plain_reverse(Vec4 &xc, Vec4 &xl, bool anchor, C2 beta_c, C2 beta_l, double (&w)[kPV])
{
    if (anchor)
        add_parts(xc, w[0], w[1]);
    else
        plain_step(xc, beta_c, w[0], w[1]);
    plain_step(xl, beta_l, w[2], w[3]);
}

template <int NE, bool kRest>
__global__ __launch_bounds__(kHeldBlock) void phase_adjoint_held_kernel(PhaseArgs a)
{
    __shared__ PhaseShared sh;
    __shared__ TrigTable trig;
    __shared__ uint32_t words[WaveMarks<NE, kHeldBlock, 2>::kWords];
    const unsigned T = a.team_size, teams = gridDim.x / T, team_id = xcd_major_block() / T;
    if (team_id >= teams)
        return;
    const PhaseTeam tm{a.sync + team_id, a.partials + uint64_t(team_id) * 32u * T, T, xcd_major_block() % T,
                       a.timeout_ticks};
    uint64_t gen = 0;
    if (a.probe) {
        double v[kPV] = {};
        (void)team_sum_n<kHeldBlock, 5>(v, tm, ++gen, sh);
        return;
    }
    if (gives_up(a, tm))
        return;
    const unsigned tid = threadIdx.x;
    const bool leader = tm.rank == 0 && tid == 0;
    const uint64_t per = a.per, base = uint64_t(tm.rank) * per;
    const bool active = NE > 1 || tid < per;
    WaveMarks<NE, kHeldBlock, 2> wm;
    wm.find(a.marks, a.m, base, per, words);
    const double inv_n = 1.0 / a.N;
    auto at = [&](unsigned r, unsigned t16) { return (r ^ wm.swap) * unsigned(kHeldBlock * 16) + t16; };
    auto load = [&](const float4 *from, Vec4 (&x)[NE]) {
        const auto rs = buffer_rsrc(from, uint32_t(per * 16u));
        const unsigned t16 = fresh_tid() * 16u;
#pragma unroll
        for (int r = 0; r < NE; ++r)
            unpack(bload16<kBufNT, float4>(rs, at(r, t16)), x[r]);
    };
    for (uint32_t b = team_id; b < a.B; b += teams) {
        float4 *st = a.state + uint64_t(b) * a.nvec + base;
        const double g = a.dloss[b];
        Vec4 xc[NE], xl[NE];
        double v[kPV] = {};
        // c_{k-1} of an anchor step k ((k - 1) % every == 0), loaded before the barrier that precedes the step so
        // that the loads travel while it waits; the state they replace is no longer needed then
        auto anchor_step = [&](uint32_t k) { return (k - 1u) % a.every == 0u; };
        auto fetch_anchor = [&](uint32_t k) {
            if (k - 1u > 0u) {
                load(a.ckpt + (uint64_t(b) * a.nck + ((k - 1u) / a.every - 1u)) * a.nvec + base, xc);
            } else {
#pragma unroll
                for (int r = 0; r < NE; ++r)
                    unpack(make_float4(a.amp, 0.0f, a.amp, 0.0f), xc[r]);
            }
        };
        // the final state of the forward run, and the seed lambda = -g c on the marked entries
        if (active) {
            load(st, xc);
#pragma unroll
            for (int r = 0; r < NE; ++r) {
                unpack(make_float4(0.0f, 0.0f, 0.0f, 0.0f), xl[r]);
                if (r == 0 ? wm.any != 0u : kRest && wm.in_rest(r)) {
                    const unsigned bits = wm.mk.at(r);
#pragma unroll
                    for (int p = 0; p < 4; ++p)
                        xl[r][p] = (bits >> (p / 2)) & 1u ? float(-g * double(xc[r][p])) : 0.0f;
                    add_parts(xl[r], v[2], v[3]);
                }
            }
            if (anchor_step(a.K))
                fetch_anchor(a.K);
        }
        if (!team_sum_n<kHeldBlock, 4>(v, tm, ++gen, sh))  // the seed's sum, in v[2], v[3]
            return;
        C2 sc{a.aux[2u * b], a.aux[2u * b + 1u]}, sl{v[2], v[3]};
        for (uint32_t k = a.K; k >= 1; --k) {
            const uint64_t pk = uint64_t(b) * a.K + k - 1;
            // the table covers the chunk of step k - 1 (0-based); refilled on entering a chunk from above
            const uint32_t i = (k - 1u) % kTrigChunk;
            if (k == a.K || i == kTrigChunk - 1u)
                fill_trig(a, b, k - 1u - i, trig);
            if (leader)  // -2 Im(conj(sum lambda) * sum c) / N
                a.dtheta[pk] = -2.0 * (sl.re * sc.im - sl.im * sc.re) / a.N;
            const C2 emth{trig.v[2][i], -trig.v[3][i]};
            const C2 om{1.0 - emth.re, -emth.im};
            const C2 fc = cmul(om, sc), fl = cmul(om, sl);
            const C2 beta_c{fc.re * inv_n, fc.im * inv_n}, beta_l{fl.re * inv_n, fl.im * inv_n};
            const bool anchor = anchor_step(k);
            double w[kPV] = {};
            if (active) {
                const C2 ephi{trig.v[0][i], trig.v[1][i]};
                if (wm.any)
                    marked_reverse(xc[0], xl[0], anchor, wm.mk.at(0), beta_c, beta_l, ephi, w);
                else
                    plain_reverse(xc[0], xl[0], anchor, beta_c, beta_l, w);
                if constexpr (kRest) {
#pragma unroll
                    for (int r = 1; r < NE; ++r) {
                        if (wm.in_rest(r))
                            marked_reverse(xc[r], xl[r], anchor, wm.mk.at(r), beta_c, beta_l, ephi, w);
                        else
                            plain_reverse(xc[r], xl[r], anchor, beta_c, beta_l, w);
                    }
                } else {
                    if (anchor) {
                        own_values<NE>(xc);
#pragma unroll
                        for (int r = 1; r < NE; ++r)
                            add_parts(xc[r], w[0], w[1]);
                    } else {
#pragma unroll
                        for (int r = 1; r < NE; ++r)
                            plain_step(xc[r], beta_c, w[0], w[1]);
                    }
#pragma unroll
                    for (int r = 1; r < NE; ++r)
                        plain_step(xl[r], beta_l, w[2], w[3]);
                }
                if (k > 1u && anchor_step(k - 1u))
                    fetch_anchor(k - 1u);
            }
            // sum c, sum lambda and Im(sum over marked of conj(nu) y): 5 values
            if (!team_sum_n<kHeldBlock, 5>(w, tm, ++gen, sh, wm.any != 0u))
                return;
            if (leader)  // -2 Im(sum over marked of conj(nu) y)
                a.dphi[pk] = -2.0 * w[4];
            sc = {w[0], w[1]};
            sl = {w[2], w[3]};
        }
        // back at the uniform state: written out, as the streamed form leaves it
        if (active) {
            const auto rs = buffer_rsrc(st, uint32_t(per * 16u));
            const unsigned t16 = fresh_tid() * 16u;
#pragma unroll
            for (int r = 0; r < NE; ++r)
                bstore16<kBufNT>(packed(xc[r]), rs, at(r, t16));
        }
    }
}

// Zeroes the team barriers and the member slots (whose generation tags the barriers compare against)
// before a launch — a kernel, so that launches can be captured and replayed.
__global__ void phase_reset_kernel(uint64_t *words, uint64_t nwords, uint64_t *slots, uint64_t nslots)
{
    const uint64_t stride = uint64_t(gridDim.x) * blockDim.x;
    for (uint64_t w = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; w < nwords; w += stride)
        words[w] = 0u;
    for (uint64_t w = uint64_t(blockIdx.x) * blockDim.x + threadIdx.x; w < nslots; w += stride)
        slots[w] = 0u;
}

}  // namespace

namespace {

template <int NE>
const void *held_kernel(bool adjoint, bool rest)
{
    if constexpr (NE <= int(kPhaseHeldAdjointVecs / kHeldBlock))
        if (adjoint)
            return rest ? reinterpret_cast<const void *>(&phase_adjoint_held_kernel<NE, true>)
                        : reinterpret_cast<const void *>(&phase_adjoint_held_kernel<NE, false>);
    return rest ? reinterpret_cast<const void *>(&phase_forward_held_kernel<NE, true>)
                : reinterpret_cast<const void *>(&phase_forward_held_kernel<NE, false>);
}

}  // namespace

uint32_t phase_block(bool held) { return held ? kHeldBlock : kStreamBlock; }

// The on-chip kernels are compiled per number of vectors a thread holds (a member holds `per` of them, at most
// kPhaseHeldForwardVecs or kPhaseHeldAdjointVecs), with and without code for a wave whose marks lie in several
// rows (phase_rest): a few marked amplitudes in a state rarely do, and the branch at every vector costs a sweep
// its scheduling.
const void *phase_kernel_fn(bool adjoint, bool held, uint64_t per, bool rest)
{
    if (held)
        switch (per / kHeldBlock) {
        case 0:
        case 1: return held_kernel<1>(adjoint, false);
        case 2: return held_kernel<2>(adjoint, rest);
        case 4: return held_kernel<4>(adjoint, rest);
        case 8: return held_kernel<8>(adjoint, rest);
        case 16: return held_kernel<16>(adjoint, rest);
        default: return adjoint ? held_kernel<16>(adjoint, rest) : held_kernel<32>(adjoint, rest);
        }
    return adjoint ? reinterpret_cast<const void *>(&phase_adjoint_kernel)
                   : reinterpret_cast<const void *>(&phase_forward_kernel);
}

// Does some wave of a member of `per` vectors hold marked amplitudes in two rows?
bool phase_rest(const std::vector<uint64_t> &marks, uint64_t per)
{
    // sorted marks: a wave's marks in one row are adjacent, so remember the last row of each wave of the member
    uint64_t member = ~uint64_t(0);
    int64_t row[kHeldBlock / kWave];
    for (const uint64_t i : marks) {
        const uint64_t v = i / 2, at = v % per;
        if (v / per != member) {
            member = v / per;
            std::fill(std::begin(row), std::end(row), -1);
        }
        const unsigned wave = unsigned(at % kHeldBlock) / kWave;
        const int64_t e = int64_t(at / kHeldBlock);
        if (row[wave] >= 0 && row[wave] != e)
            return true;
        row[wave] = e;
    }
    return false;
}

hipError_t launch_phase(const PhaseLaunch &L, bool adjoint)
{
    PhaseArgs a;
    a.state = static_cast<float4 *>(L.state);
    a.lambda = static_cast<float4 *>(L.lambda);
    a.ckpt = static_cast<float4 *>(L.ckpt);
    a.marks = L.marks;
    a.m = L.m;
    a.nvec = L.nvec;
    a.per = L.per;
    a.N = L.N;
    a.amp = L.amp;
    a.B = L.B;
    a.K = L.K;
    a.every = L.every;
    a.nck = L.nck;
    a.phi = L.phi;
    a.theta = L.theta;
    a.loss = L.loss;
    a.aux = L.aux;
    a.dloss = L.dloss;
    a.dphi = L.dphi;
    a.dtheta = L.dtheta;
    a.sync = L.sync;
    a.partials = L.partials;
    a.team_size = L.team_size;
    a.probe = L.probe;
    a.timeout_ticks = L.timeout_ticks;
    uint64_t *words = reinterpret_cast<uint64_t *>(L.sync);
    uint64_t nwords = uint64_t(L.teams_alloc) * sizeof(PhaseSync) / sizeof(uint64_t);
    uint64_t *slots = L.partials;
    uint64_t nslots = uint64_t(L.grid) * 32u;
    void *ra[] = {&words, &nwords, &slots, &nslots};
    hipError_t e = hipLaunchKernel(reinterpret_cast<const void *>(&phase_reset_kernel), dim3(64), dim3(256), ra, 0,
                                   L.stream);
    if (e != hipSuccess)
        return e;
    void *args[] = {&a};
    return hipLaunchCooperativeKernel(phase_kernel_fn(adjoint, L.held != 0u, L.per, L.rest != 0u), dim3(L.grid),
                                      dim3(phase_block(L.held != 0u)), args, 0, L.stream);
}

}  // namespace grover
