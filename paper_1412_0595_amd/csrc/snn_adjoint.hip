// Reverse-time adjoint kernels (gfx950): gradient of a loss on one
// population's time-averaged voltage with respect to every synaptic weight
// g and every instance's g_scale, exact for the discrete forward map with
// the spike raster held fixed.
//
// With the raster fixed, the loss population sees the rest of the network
// only through recorded spike times, so the backward pass touches only its
// neurons and the projections into it.  The forward keeps a checkpoint every K
// steps and the bitmask raster; the backward works through groups of whole
// segments, as many as its tape holds (one at least, so memory stays
// O(T/K + K)), the last group first:
//
//  k_adj_deliver  the group's delivered increments, a block per (instance,
//                 step): they depend on the raster alone
//  k_adj_states   the loss neurons' states, a lane per (segment, neuron) from
//                 the segment's checkpoint; bit-identical to the forward
//  k_adj_reverse  the adjoint: every step's transposed Jacobian, steps in
//                 parallel, then the chain of its products with the adjoint
//  k_adj_gather   the weight gradients, a block per 64 pre neurons
//
// Only k_adj_states and the chain are serial in time, and only over one
// segment and over a 4-vector's products.  (One block per instance that
// recomputed a segment step by step, one lane per neuron that reversed it, one
// wavefront per word that read the raster a step at a time took 8.9, 6.0 and
// 2.6 us per step of 64 instances of 200 loss neurons: 35.0 ms for 2 000 steps,
// 8.3 ms as above.)
#include <algorithm>

#include "snn_device.h"

namespace snn {

// d/dx [x / (e^x - 1)] = (e^x - 1 - x e^x) / (e^x - 1)^2, by its Taylor
// series -1/2 + x/6 - x^3/180 where the closed form cancels (|x| < 1e-3).
__device__ __forceinline__ double dxexpm1_ratio(double x)
{
    if (fabs(x) < 1e-3) return -0.5 + x * (1.0 / 6.0) - x * x * x * (1.0 / 180.0);
    const double em1 = expm1(x);
    return (em1 * (1.0 - x) - x) / (em1 * em1);
}

// One Euler substep (x' = x + hs f(x, I)) of the state x = (v, m, h, n) and of
// its derivatives: D (x by the state at the step's start) and dI (x by the
// injected current) are multiplied by the substep's Jacobian.
__device__ __forceinline__ void hh_substep_jvp(const Seg &S, double hs, double hc, double iin, double (&x)[4],
                                               double (&D)[4][4], double (&dI)[4])
{
    const double v = x[0], m = x[1], h = x[2], n = x[3];
    const HHRates r = hh_rates(v);
    const double dam = -0.25 * 1.28 * dxexpm1_ratio((-52.0 - v) * 0.25);
    const double dbm = 0.2 * 1.4 * dxexpm1_ratio((v + 25.0) * 0.2);
    const double dah = -r.ah * (1.0 / 18.0);
    const double ez = exp((-25.0 - v) * 0.2);
    const double dbh = 0.2 * 4.0 * ez / ((ez + 1.0) * (ez + 1.0));
    const double dan = -0.2 * 0.16 * dxexpm1_ratio((-50.0 - v) * 0.2);
    const double dbn = -r.bn * 0.025;
    const double m2 = m * m, n3 = n * n * n;
    // v' = v + hc (I - I_ion)
    const double vv = 1.0 - hc * (S.gna * m2 * m * h + S.gk * n3 * n + S.gl);
    const double vm = -hc * 3.0 * S.gna * m2 * h * (v - S.ena);
    const double vh = -hc * S.gna * m2 * m * (v - S.ena);
    const double vn = -hc * 4.0 * S.gk * n3 * (v - S.ek);
    // x' = x + hs (a (1 - x) - b x)
    const double mv = hs * (dam * (1.0 - m) - dbm * m), mm = 1.0 - hs * (r.am + r.bm);
    const double hv = hs * (dah * (1.0 - h) - dbh * h), hh = 1.0 - hs * (r.ah + r.bh);
    const double nv = hs * (dan * (1.0 - n) - dbn * n), nn = 1.0 - hs * (r.an + r.bn);
#pragma unroll
    for (int j = 0; j < 5; ++j) {
        double *d[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) d[i] = j < 4 ? &D[i][j & 3] : &dI[i];
        const double dv = *d[0];
        *d[0] = vv * dv + vm * *d[1] + vh * *d[2] + vn * *d[3] + (j < 4 ? 0.0 : hc);
        *d[1] = mv * dv + mm * *d[1];
        *d[2] = hv * dv + hh * *d[2];
        *d[3] = nv * dv + nn * *d[3];
    }
    const double n2 = n * n;
    const double iion = S.gna * (m2 * m * h) * (v - S.ena) + S.gk * (n2 * n2) * (v - S.ek) + S.gl * (v - S.el);
    x[0] = v + hc * (iin - iion);
    x[1] = m + hs * (r.am * (1.0 - m) - r.bm * m);
    x[2] = h + hs * (r.ah * (1.0 - h) - r.bh * h);
    x[3] = n + hs * (r.an * (1.0 - n) - r.bn * n);
}

// ---------------------------------------------------------------------------
// Increments delivered to the loss population at every step of the group:
// block (b, k) sums instance b's at step t_a + k in LDS, on the forward's
// 2^-40 uS grid (integer sums: the order does not matter).  Its spiking rows
// are listed in LDS and dealt out over the wavefronts; beyond kAdjList rows
// the wavefronts walk the words themselves.
// ---------------------------------------------------------------------------
constexpr int kAdjList = 1024;
constexpr int kAdjSteps = 32768;   // steps per launch (a grid's second dimension is 16 bits)

__global__ __launch_bounds__(256) void k_adj_deliver(AdjArgs a)
{
    extern __shared__ long long s_inc[];      // [n_in][n]
    __shared__ int2 s_rows[kAdjList];         // (input, row)
    __shared__ uint32_t s_n;
    const int b = blockIdx.x, k = a.k_first + blockIdx.y;
    const int64_t t = a.t_a + k;
    const Seg &S = a.segs[a.loss_seg[b]];
    const int n = S.n, n_in = S.n_in;
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x >> 6, nwb = blockDim.x >> 6;
    const double s_fix = (double)a.gscale[b] * kFixOne;
    for (int i = threadIdx.x; i < n_in * n; i += blockDim.x) s_inc[i] = 0;
    if (threadIdx.x == 0) s_n = 0;
    __syncthreads();
    auto add_row = [&](int q, int32_t i) {
        const Proj &P = a.projs[S.in_proj[q]];
        const int32_t *rp = a.rp_pool + P.rp_base;
        const int32_t *col = a.col_pool + P.syn_base;
        const float *w = a.w_pool + P.syn_base;
        const int32_t k1 = rp[i + 1];
        for (int32_t kk = rp[i] + lane; kk < k1; kk += kWave)
            atomicAdd((unsigned long long *)&s_inc[q * n + col[kk]], (unsigned long long)fix_increment(s_fix, w[kk]));
    };
    if (t > 0) {
        for (int q = 0; q < n_in; ++q) {
            const Seg &pre = a.segs[a.projs[S.in_proj[q]].pre_seg];
            const int nw = (pre.n + kWave - 1) / kWave;
            const uint64_t *bits = a.raster + (t - 1) * a.n_waves + pre.base / kWave;
            for (int wd = threadIdx.x; wd < nw; wd += blockDim.x) {
                uint64_t word = bits[wd];
                if (word == 0) continue;
                uint32_t at = atomicAdd(&s_n, (uint32_t)__popcll(word));
                for (; word && at < (uint32_t)kAdjList; word &= word - 1, ++at)
                    s_rows[at] = make_int2(q, wd * kWave + __builtin_ctzll(word));
            }
        }
        __syncthreads();
        if (s_n <= (uint32_t)kAdjList) {
            for (int i = wid; i < (int)s_n; i += nwb) {
                const int2 e = s_rows[i];
                add_row(__builtin_amdgcn_readfirstlane(e.x), __builtin_amdgcn_readfirstlane(e.y));
            }
        } else {
            for (int q = 0; q < n_in; ++q) {
                const Seg &pre = a.segs[a.projs[S.in_proj[q]].pre_seg];
                const int nw = (pre.n + kWave - 1) / kWave;
                const uint64_t *bits = a.raster + (t - 1) * a.n_waves + pre.base / kWave;
                for (int wd = wid; wd < nw; wd += nwb)
                    for (uint64_t word = uniform_u64(bits[wd]); word; word &= word - 1)
                        add_row(q, wd * kWave + __builtin_ctzll(word));
            }
        }
        __syncthreads();
    }
    long long *out = reinterpret_cast<long long *>(a.tape_g) + (int64_t)k * a.n_in_max * a.n_loss + a.loss_base[b];
    for (int i = threadIdx.x; i < n_in * n; i += blockDim.x) out[(int64_t)(i / n) * a.n_loss + i % n] = s_inc[i];
}

// ---------------------------------------------------------------------------
// States of the loss neurons at the start of every step of the group: lane
// (s, c) steps neuron c through segment s from its checkpoint.  The tape's
// increments become the delivered conductances.  Bound by the dependent chain
// of the substeps (0.6 us each); the next step's increments are loaded a step
// ahead.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void k_adj_states(AdjArgs a)
{
    const int64_t N = a.n_loss, c = (int64_t)blockIdx.x * kWave + threadIdx.x;
    if (c >= N) return;
    const int sg = blockIdx.y;
    const int b = a.loss_owner[c];
    const Seg &S = a.segs[a.loss_seg[b]];
    const int64_t j = c - a.loss_base[b], gi = S.base + j, P = a.n_pad;
    const int k0 = sg * a.seg_steps, k1 = min(k0 + a.seg_steps, a.K);
    const float *cs = a.ckpt_state + (int64_t)sg * 8 * P;
    const int64_t *cg = a.ckpt_G + sg * a.g_stride;
    const double hc = a.hs * S.inv_c;
    float vh = cs[gi], vl = cs[P + gi], mh = cs[2 * P + gi], ml = cs[3 * P + gi];
    float hh = cs[4 * P + gi], hl = cs[5 * P + gi], nh = cs[6 * P + gi], nl = cs[7 * P + gi];
    int64_t g[kMaxIn] = {0, 0, 0, 0}, inc[kMaxIn] = {0, 0, 0, 0};
    const long long *tg = reinterpret_cast<const long long *>(a.tape_g);
#pragma unroll
    for (int q = 0; q < kMaxIn; ++q)
        if (q < S.n_in) {
            g[q] = cg[S.in_G[q] + j];
            inc[q] = tg[((int64_t)k0 * a.n_in_max + q) * N + c];
        }
    for (int k = k0; k < k1; ++k) {
        int64_t gin[kMaxIn];
        const int kn = min(k + 1, k1 - 1);
#pragma unroll
        for (int q = 0; q < kMaxIn; ++q)
            if (q < S.n_in) {
                gin[q] = g[q] + inc[q];
                inc[q] = tg[((int64_t)kn * a.n_in_max + q) * N + c];
            }
        double v = (double)vh + (double)vl, m = (double)mh + (double)ml;
        double h = (double)hh + (double)hl, n = (double)nh + (double)nl;
        a.tape_x[((int64_t)k * 4 + 0) * N + c] = v;
        a.tape_x[((int64_t)k * 4 + 1) * N + c] = m;
        a.tape_x[((int64_t)k * 4 + 2) * N + c] = h;
        a.tape_x[((int64_t)k * 4 + 3) * N + c] = n;
        const double iin = syn_current(S, gin, v);
#pragma unroll
        for (int q = 0; q < kMaxIn; ++q)
            if (q < S.n_in) {
                a.tape_g[((int64_t)k * a.n_in_max + q) * N + c] = (double)gin[q] * kFixInv;
                g[q] = fix_decay(gin[q], S.in_decay[q]);
            }
        for (int s = 0; s < a.substeps; ++s) hh_substep(S, a.hs, hc, iin, v, m, h, n);
        pair_split(v, vh, vl);
        pair_split(m, mh, ml);
        pair_split(h, hh, hl);
        pair_split(n, nh, nl);
    }
    // the recomputation must reproduce the next checkpoint bit for bit
    if (a.first_seg + sg + 1 < a.n_seg) {
        const float *ns = cs + 8 * P;
        const int64_t *ng = cg + a.g_stride;
        uint32_t bad = 0;
        bad += __float_as_uint(ns[gi]) != __float_as_uint(vh);
        bad += __float_as_uint(ns[P + gi]) != __float_as_uint(vl);
        bad += __float_as_uint(ns[2 * P + gi]) != __float_as_uint(mh);
        bad += __float_as_uint(ns[3 * P + gi]) != __float_as_uint(ml);
        bad += __float_as_uint(ns[4 * P + gi]) != __float_as_uint(hh);
        bad += __float_as_uint(ns[5 * P + gi]) != __float_as_uint(hl);
        bad += __float_as_uint(ns[6 * P + gi]) != __float_as_uint(nh);
        bad += __float_as_uint(ns[7 * P + gi]) != __float_as_uint(nl);
#pragma unroll
        for (int q = 0; q < kMaxIn; ++q)
            if (q < S.n_in) bad += ng[S.in_G[q] + j] != g[q];
        if (bad) atomicAdd(a.mismatch, bad);
    }
}

// ---------------------------------------------------------------------------
// Reverse the group: a block takes kRevNeurons loss neurons, the last steps
// first, as many at a time as it has threads for.  A thread per (step, neuron) carries the
// derivatives of the state after the step by the state before it (4 x 4) and
// by the injected current through the substeps, into LDS; then a lane per
// neuron follows the chain of the adjoint (lv, lm, lh, ln) through the steps.
// The derivatives are most of the arithmetic and independent of each other;
// the chain is 20 multiply-adds a step.  About 200 VGPRs, two wavefronts per
// SIMD: blocks of four, so that one's chain runs beside the other's maps.
// Eight neurons by 32 steps keep the most chains apart; a group of up to 8 or
// 4 steps would leave most of such a block idle, so it takes 32 or 64 neurons
// by as many steps (backward of 300 networks with 100 loss neurons each: one
// step 93.5 -> 42.0 us, four 110 -> 53.7, five 116 -> 68.3); 32 only where that
// leaves blocks for the chip (100 loss neurons, five steps: 37 us by 8, 42 by
// 32; 4 000: 50 either way).
// ---------------------------------------------------------------------------
constexpr int kRevThreads = 256, kRevMap = 21, kRevWide = 4096;

template <int kRevNeurons>
__global__ __launch_bounds__(kRevThreads) void k_adj_reverse(AdjArgs a)
{
    extern __shared__ double s_map[];      // [step][entry][neuron]
    constexpr int kRevSteps = kRevThreads / kRevNeurons;
    const int64_t N = a.n_loss;
    const int nn = threadIdx.x % kRevNeurons, st = threadIdx.x / kRevNeurons;
    const int64_t c = (int64_t)blockIdx.x * kRevNeurons + nn;
    const bool mine = c < N, chain = mine && st == 0;
    const Seg &S = a.segs[a.loss_seg[mine ? a.loss_owner[c] : 0]];
    const double hc = a.hs * S.inv_c;
    double lv = 0.0, lm = 0.0, lh = 0.0, ln = 0.0, src = 0.0, lG[kMaxIn] = {0.0, 0.0, 0.0, 0.0};
    if (chain) {
        lv = a.lam[c];
        lm = a.lam[N + c];
        lh = a.lam[2 * N + c];
        ln = a.lam[3 * N + c];
#pragma unroll
        for (int q = 0; q < kMaxIn; ++q)
            if (q < S.n_in) lG[q] = a.lam[(4 + q) * N + c];
        src = a.dvbar[c] / (double)a.T;
    }
    for (int hi = a.K; hi > 0; hi -= kRevSteps) {
        const int lo = max(hi - kRevSteps, 0), k = lo + st;
        if (mine && k < hi) {
            double x[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) x[v] = a.tape_x[((int64_t)k * 4 + v) * N + c];
            const double v0 = x[0];
            double iin = S.i_ext, gsum = 0.0;
#pragma unroll
            for (int q = 0; q < kMaxIn; ++q)
                if (q < S.n_in) {
                    const double g = a.tape_g[((int64_t)k * a.n_in_max + q) * N + c];
                    iin += g * (S.in_erev[q] - v0);
                    gsum += g;
                }
            double D[4][4] = {{1.0, 0.0, 0.0, 0.0}, {0.0, 1.0, 0.0, 0.0}, {0.0, 0.0, 1.0, 0.0}, {0.0, 0.0, 0.0, 1.0}};
            double dI[4] = {0.0, 0.0, 0.0, 0.0};
            for (int s = 0; s < a.substeps; ++s) hh_substep_jvp(S, a.hs, hc, iin, x, D, dI);
            // I = I_ext + sum_q Ginj_q (E_q - V(t-1)): the current's own share of V
            double *M = s_map + (int64_t)st * kRevMap * kRevNeurons + nn;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
#pragma unroll
                for (int j = 0; j < 4; ++j) M[(4 * j + i) * kRevNeurons] = D[i][j] - (j == 0 ? gsum * dI[i] : 0.0);
                M[(16 + i) * kRevNeurons] = dI[i];
            }
            M[20 * kRevNeurons] = v0;
        }
        __syncthreads();
        if (chain)
            for (int kk = hi - 1; kk >= lo; --kk) {
                const double *M = s_map + (int64_t)(kk - lo) * kRevMap * kRevNeurons + nn;
                double e[kRevMap];
#pragma unroll
                for (int v = 0; v < kRevMap; ++v) e[v] = M[v * kRevNeurons];
                lv += src;    // V at the end of this step enters Vbar
                const double pv = e[0] * lv + e[1] * lm + e[2] * lh + e[3] * ln;
                const double pm = e[4] * lv + e[5] * lm + e[6] * lh + e[7] * ln;
                const double ph = e[8] * lv + e[9] * lm + e[10] * lh + e[11] * ln;
                const double pn = e[12] * lv + e[13] * lm + e[14] * lh + e[15] * ln;
                const double li = e[16] * lv + e[17] * lm + e[18] * lh + e[19] * ln;
                // G(t) = d_q Ginj_q, Ginj_q(t) = G_q(t-1) + deliveries
#pragma unroll
                for (int q = 0; q < kMaxIn; ++q)
                    if (q < S.n_in) {
                        lG[q] = S.in_decay[q] * lG[q] + li * (S.in_erev[q] - e[20]);
                        a.lg[((int64_t)kk * a.n_in_max + q) * N + c] = lG[q];
                    }
                lv = pv;
                lm = pm;
                lh = ph;
                ln = pn;
            }
        __syncthreads();
    }
    if (chain) {
        a.lam[c] = lv;
        a.lam[N + c] = lm;
        a.lam[2 * N + c] = lh;
        a.lam[3 * N + c] = ln;
#pragma unroll
        for (int q = 0; q < kMaxIn; ++q)
            if (q < S.n_in) a.lam[(4 + q) * N + c] = lG[q];
    }
}

// ---------------------------------------------------------------------------
// Weight and g_scale gradients of the group: a block per 64 rows of one
// projection into the loss population, a quarter of the rows per wavefront.
// The rows' spike words of the group's steps are held in LDS (kGatherSteps at
// a time); for a row, a ballot over 64 of them gives its spikes, and each
// lane sums lambda_Ginj(t)[post] over the spikes of its synapses:
// g_scale * sum is added to dL/dg, g * sum to dL/dg_scale.  The sums run in
// double over a segment and are added segment by segment, the last first, so
// the gradient does not depend on how many segments a group has.  Each
// synapse belongs to one lane, so no atomics on dg.
// ---------------------------------------------------------------------------
constexpr int kGatherSteps = 2048;

__global__ __launch_bounds__(256) void k_adj_gather(AdjArgs a)
{
    __shared__ uint64_t s_words[kGatherSteps];
    __shared__ uint64_t s_any;
    const int lane = threadIdx.x & (kWave - 1), wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int4 it = a.gitems[blockIdx.x];
    const int b = it.x, q = it.y, wd = it.w;
    const Seg &L = a.segs[a.loss_seg[b]];
    const Proj &P = a.projs[L.in_proj[q]];
    const Seg &pre = a.segs[P.pre_seg];
    const double s = (double)a.gscale[b];
    const int64_t lb = a.loss_base[b];
    const int32_t *rp = a.rp_pool + P.rp_base;
    const int32_t *col = a.col_pool + P.syn_base;
    const float *w = a.w_pool + P.syn_base;
    float *dg = a.dg + P.syn_base;
    const int64_t lstride = (int64_t)a.n_in_max * a.n_loss;
    const double *lg = a.lg + (int64_t)q * a.n_loss + lb;
    const uint64_t *bits = a.raster + pre.base / kWave + wd;
    const int32_t row_l = min(wd * kWave + lane, P.n_pre - 1);
    const int32_t b0 = rp[row_l], b1 = rp[row_l + 1];
    double acc = 0.0;
    for (int sg = (a.K - 1) / a.seg_steps; sg >= 0; --sg) {
        const int k_end = min((sg + 1) * a.seg_steps, a.K);
        for (int ka = sg * a.seg_steps; ka < k_end; ka += kGatherSteps) {
            const int nk = min(kGatherSteps, k_end - ka);
            __syncthreads();
            if (threadIdx.x == 0) s_any = 0;
            __syncthreads();
            uint64_t any = 0;
            for (int k = threadIdx.x; k < nk; k += blockDim.x) {
                const int64_t t = a.t_a + ka + k;
                const uint64_t x = t > 0 ? bits[(t - 1) * a.n_waves] : 0ull;
                s_words[k] = x;
                any |= x;
            }
            if (any) atomicOr((unsigned long long *)&s_any, (unsigned long long)any);
            __syncthreads();
            // rows wid, wid + 4, ... that spiked
            uint64_t rows = uniform_u64(s_any) & (0x1111111111111111ull << wid);
            for (; rows; rows &= rows - 1) {
                const int r = __builtin_ctzll(rows);
                const int32_t r0 = __builtin_amdgcn_readlane(b0, r), r1 = __builtin_amdgcn_readlane(b1, r);
                for (int32_t kb = r0; kb < r1; kb += kWave) {
                    const int32_t kk = min(kb + lane, r1 - 1);
                    const double *lc = lg + col[kk];
                    double sum = 0.0;
                    for (int k = 0; k < nk; k += kWave) {
                        const uint64_t x = k + lane < nk ? s_words[k + lane] : 0ull;
                        uint64_t m = __ballot((x >> r) & 1ull);
                        for (; m; m &= m - 1) sum += lc[(int64_t)(ka + k + __builtin_ctzll(m)) * lstride];
                    }
                    if (kb + lane < r1) {
                        dg[kk] = (float)((double)dg[kk] + s * sum);
                        acc += (double)w[kk] * sum;
                    }
                }
            }
        }
    }
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) acc += __shfl_down(acc, d, kWave);
    if (lane == 0 && acc != 0.0) atomicAdd(&a.ds[b], acc);
}

__global__ void k_gather_vbar(const Seg *segs, const int32_t *loss_seg, const int64_t *loss_base,
                              const int32_t *loss_owner, int64_t n_loss, const double *vsum, double inv_T, double *vbar)
{
    const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= n_loss) return;
    const int b = loss_owner[c];
    const Seg &S = segs[loss_seg[b]];
    vbar[c] = vsum[S.base + (c - loss_base[b])] * inv_T;
}

hipError_t launch_adj_group(const AdjArgs &a, int max_inc, hipStream_t s)
{
    if (a.n_loss == 0 || a.K <= 0) return hipSuccess;
    AdjArgs d = a;
    for (d.k_first = 0; d.k_first < a.K; d.k_first += kAdjSteps)
        hipLaunchKernelGGL(k_adj_deliver, dim3((unsigned)a.n_inst, (unsigned)std::min(a.K - d.k_first, kAdjSteps)),
                           dim3(256), 8 * (size_t)max_inc, s, d);
    const int segs = (a.K + a.seg_steps - 1) / a.seg_steps;
    hipLaunchKernelGGL(k_adj_states, dim3((unsigned)((a.n_loss + kWave - 1) / kWave), (unsigned)segs), dim3(kWave), 0,
                       s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t lds = sizeof(double) * kRevThreads * kRevMap;
    auto reverse = [&](auto kernel, int neurons) {
        e = hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e == hipSuccess)
            hipLaunchKernelGGL(kernel, dim3((unsigned)((a.n_loss + neurons - 1) / neurons)), dim3(kRevThreads), lds, s, a);
    };
    if (a.K <= kRevThreads / 64) reverse(k_adj_reverse<64>, 64);
    else if (a.K <= kRevThreads / 32 && a.n_loss >= kRevWide) reverse(k_adj_reverse<32>, 32);
    else reverse(k_adj_reverse<8>, 8);
    if (e != hipSuccess) return e;
    if (a.n_gitems > 0) hipLaunchKernelGGL(k_adj_gather, dim3((unsigned)a.n_gitems), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t launch_gather_vbar(const Seg *segs, const int32_t *loss_seg, const int64_t *loss_base,
                              const int32_t *loss_owner, int64_t n_loss, const double *vsum, double inv_T,
                              double *vbar, hipStream_t s)
{
    const int64_t blocks = (n_loss + 255) / 256;
    if (blocks == 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_vbar, dim3((unsigned)blocks), dim3(256), 0, s, segs, loss_seg, loss_base, loss_owner,
                       n_loss, vsum, inv_T, vbar);
    return hipGetLastError();
}

}  // namespace snn
