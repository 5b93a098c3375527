// Resident stepping (gfx950): many steps in one launch, the network's state
// in LDS.
//
// Instances are independent, so an instance is a cluster of blocks that steps
// by itself: a block owns a contiguous range of the words (64 neurons) of
// every population, keeps their state and conductances in LDS for the whole
// launch, and delivers by pulling in the slices of the spiking rows that end
// on its own neurons, with LDS atomics.  All that leaves a block during the
// steps are its spike words: each goes out as two 8-byte values, half the word
// and the step's tag, stored and polled with relaxed agent-scope atomics, so a
// value that carries the awaited tag is also the data (no flags, no fences).
// An instance in one block needs none of that.
//
// A step of a small network is a chain of latencies, not work, and the chain
// is what this kernel shortens: spike words, a list of the spiking rows in LDS
// (so that the waves share them evenly), slice bounds, synapses, LDS sums,
// update.  Deliveries go into two alternating sums, so a wave need not wait
// for the others' updates before it delivers the next step; and the first
// Euler substep of the gates and the ionic current do not depend on the step's
// input, so they run, like the sources' draws, while the words travel.
#include <algorithm>

#include "snn_device.h"

namespace snn {

namespace {

using CResBlock = const __attribute__((address_space(4))) ResBlock;
using CResWord = const __attribute__((address_space(4))) ResWord;
using CSeg = const __attribute__((address_space(4))) Seg;

constexpr int kResPoll = 4;    // half words a lane asks for at once
constexpr int kResState = 5;   // doubles of state per neuron in LDS

// The constants of a Traub-Miles population, in scalar registers.
struct HHConst {
    double gna, ena, gk, ek, gl, el;
};

// Poisson draw of step t for lane's neuron j.
__device__ __forceinline__ bool poisson_spike(CSeg &S, int32_t j, int64_t t)
{
    const uint32_t w = philox_first_word((uint32_t)j, (uint32_t)((uint64_t)t & 0xffffffffu),
                                         (uint32_t)((uint64_t)t >> 32), (uint32_t)S.pop,
                                         (uint32_t)(S.seed & 0xffffffffu), (uint32_t)(S.seed >> 32));
    return (uint64_t)w < S.thresh;
}

// One batch of kSlotsN slots of up to 64 entries of one slice each, from the
// slice in progress [k, k1) and the lanes left in rem; all loads before the
// atomics.  Past the last slice a slot repeats its entries and adds nothing.
template <int kSlotsN>
__device__ __forceinline__ void slots_to_lds(unsigned long long *s_g, const int32_t *col, const float *w, int32_t b0,
                                             int32_t b1, int32_t go, double s, int lane, uint64_t &rem, int32_t &k,
                                             int32_t &k1, int32_t &g0)
{
    int32_t sk[kSlotsN], se[kSlotsN], sg[kSlotsN];
#pragma unroll
    for (int u = 0; u < kSlotsN; ++u) {
        if (k >= k1 && rem) {
            const int r = __builtin_ctzll(rem);
            rem &= rem - 1;
            k = __builtin_amdgcn_readlane(b0, r);
            k1 = __builtin_amdgcn_readlane(b1, r);
            g0 = __builtin_amdgcn_readlane(go, r);
        }
        sk[u] = k;
        se[u] = k1;
        sg[u] = g0;
        k += kWave;
    }
    int32_t c[kSlotsN];
    float g[kSlotsN];
#pragma unroll
    for (int u = 0; u < kSlotsN; ++u) {
        const uint32_t kk = (uint32_t)min(sk[u] + lane, se[u] - 1);
        c[u] = col[kk];
        g[u] = w[kk];
    }
#pragma unroll
    for (int u = 0; u < kSlotsN; ++u)
        if (sk[u] + lane < se[u]) atomicAdd(s_g + (sg[u] + c[u]), (unsigned long long)fix_increment(s, g[u]));
}

// Adds slices into the block's sums: lane l holds its slice's bounds [b0, b1)
// (relative to the instance's first synapse; empty: none) and the LDS index
// of the slice's column 0.
__device__ __forceinline__ void slices_to_lds(unsigned long long *s_g, const int32_t *col, const float *w, int32_t b0,
                                              int32_t b1, int32_t go, double s, int lane)
{
    uint64_t rem = __ballot(b1 > b0);
    int32_t k = 0, k1 = 0, g0 = 0;
    while (rem || k < k1) {
        if (__popcll(rem) + (k < k1 ? 1 : 0) <= 2 && k1 - k <= kWave)
            slots_to_lds<2>(s_g, col, w, b0, b1, go, s, lane, rem, k, k1, g0);
        else
            slots_to_lds<8>(s_g, col, w, b0, b1, go, s, lane, rem, k, k1, g0);
    }
}

}  // namespace

// One block's part of a cluster for n steps from step t0.
template <int FEAT>
__global__ __launch_bounds__(1024) void k_resident(ResArgs a)
{
    extern __shared__ __align__(16) char s_mem[];
    __shared__ uint32_t s_fail, s_cnt[3];   // rows listed per step, of three in turn
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int nt = (int)blockDim.x, nw = nt >> 6;
    constexpr bool kIzhOn = (FEAT & kFeatIzh) != 0, kRec = (FEAT & kFeatRec) != 0;

    CResBlock &B = ((CResBlock *)a.blocks)[blockIdx.x];
    const int n_state = B.n_state, n_poi = B.n_poi, n_words = B.n_words, n_g = B.n_g;
    const int64_t w_first = B.w_first;      // the instance's first spike word
    const bool multi = B.n_blocks > 1;
    CResWord *words = (CResWord *)a.words + B.word0;
    const double s_fix = (double)a.gscale[B.inst] * kFixOne;
    const int32_t *col = a.col_pool + B.syn_first;
    const float *wt = a.w_pool + B.syn_first;
    uint64_t *xw = a.xbuf + B.x_off;        // kResRing slots of 2 n_words tagged halves

    // LDS: conductances, the deliveries of two alternating steps, neuron
    // state, recorded sums, feeds, spike words of two steps, each word's feeds,
    // the rows (neuron of the instance) listed for three steps in turn
    unsigned long long *s_g = reinterpret_cast<unsigned long long *>(s_mem);
    unsigned long long *s_acc = s_g + n_g;
    double *s_state = reinterpret_cast<double *>(s_acc + 2 * n_g);
    double *s_vsum = s_state + n_state * kResState * kWave;
    ResFeed *s_feed = reinterpret_cast<ResFeed *>(s_vsum + (kRec ? n_state * kWave : 0));
    uint64_t *s_word = reinterpret_cast<uint64_t *>(s_feed + B.n_feed);
    uint32_t *s_wfeed = reinterpret_cast<uint32_t *>(s_word + 2 * n_words);
    uint32_t *s_list = s_wfeed + n_words;

    const int64_t t0 = a.t0, t_end = a.t0 + a.n;
    if (threadIdx.x == 0) s_fail = s_cnt[0] = s_cnt[1] = s_cnt[2] = 0;
    for (int i = threadIdx.x; i < 2 * n_g; i += nt) s_acc[i] = 0;
    for (int i = threadIdx.x; i < B.n_feed; i += nt) s_feed[i] = a.feeds[B.feed0 + i];
    for (int i = threadIdx.x; i < n_words; i += nt) s_wfeed[i] = a.wfeeds[B.wfeed0 + i];
    __syncthreads();

    // A word of step t: to the cluster (a single block: to its own list l) and
    // the records.
    auto publish = [&](int64_t t, int l, int64_t gw, uint64_t ball) {
        const int rel = (int)(gw - w_first);
        if (multi) {
            if (lane < 2) {
                const uint64_t tag = (uint64_t)(uint32_t)(a.tag0 + (uint32_t)(t - t0)) << 32;
                __hip_atomic_store(xw + (t & (kResRing - 1)) * 2 * n_words + 2 * rel + lane,
                                   tag | (uint32_t)(ball >> (32 * lane)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        } else {
            if (lane == 0) s_word[(t & 1) * n_words + rel] = ball;
            if (ball != 0 && s_wfeed[rel] != 0) {
                uint32_t at = 0;
                if (lane == 0) at = atomicAdd(&s_cnt[l], (uint32_t)__popcll(ball));
                at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + (uint32_t)__popcll(ball & ((1ull << lane) - 1ull));
                if (((ball >> lane) & 1ull) && at < (uint32_t)kResList) s_list[l * kResList + at] = rel * kWave + lane;
            }
        }
        if (lane == 0) {
            if (a.raster) a.raster[(t % a.raster_steps) * a.n_waves + gw] = ball;
            if (t == t_end - 1) a.bits[(t & 1) * a.n_waves + gw] = ball;
        }
    };
    // The block's Poisson words of step t (the last waves first: the first
    // ones have the longer share of the neurons).
    auto sources = [&](int64_t t, int l) {
        for (int w = nw - 1 - wid; w < n_poi; w += nw) {
            CResWord &W = words[n_state + w];
            CSeg &S = ((CSeg *)a.segs)[W.seg];
            const int64_t gid = W.gw * kWave + lane;
            const int32_t j = (int32_t)(gid - S.base);
            const bool spike = j < S.n && poisson_spike(S, j, t);
            publish(t, l, W.gw, __ballot(spike));
            if (spike) atomicAdd(&a.counts[gid], 1);
        }
    };
    // Traub-Miles: the part of a step's first substep that its input does not
    // enter, from (v, m, h, n) to LDS: v, the gates after it, the ionic current.
    auto hh_ahead = [&](CSeg &S, double *x, double v, double m, double h, double n) {
        const HHConst P{S.gna, S.ena, S.gk, S.ek, S.gl, S.el};
        x[0] = v;
        x[4 * kWave] = hh_gates(P, a.hs, v, m, h, n);
        x[kWave] = m;
        x[2 * kWave] = h;
        x[3 * kWave] = n;
    };

    // ---- state in, the sources' first step
    for (int w = wid; w < n_state; w += nw) {
        CResWord &W = words[w];
        CSeg &S = ((CSeg *)a.segs)[W.seg];
        const int64_t gid = W.gw * kWave + lane;
        const int32_t jj = min((int32_t)(gid - S.base), S.n - 1);
        double *x = s_state + w * kResState * kWave + lane;
#pragma unroll
        for (int q = 0; q < kMaxIn; ++q)
            if (q < S.n_in) s_g[W.g_off[q] + lane] = (unsigned long long)a.G[S.in_G[q] + jj];
        if constexpr (kRec) s_vsum[w * kWave + lane] = S.record_vbar ? a.vsum[gid] : 0.0;
        const double v = pair_load(a.vh, a.vl, gid), m = pair_load(a.mh, a.ml, gid);
        if (!kIzhOn || S.kind == kHH) {
            hh_ahead(S, x, v, m, pair_load(a.hh, a.hl, gid), pair_load(a.nh, a.nl, gid));
        } else {
            x[0] = v;
            x[kWave] = m;
        }
    }
    int l_prev = 0, l_cur = 1, l_next = 2;   // lists of S(t - 1), S(t), S(t + 1)
    sources(t0, l_cur);

    const int h_share = (2 * n_words + nw - 1) / nw;
    const int h_begin = wid * h_share, h_end = min(h_begin + h_share, 2 * n_words);
    // Adds the slices of the rows that its lanes hold (neurons of the
    // instance; -1: none).
    auto deliver_rows = [&](unsigned long long *acc, int32_t row) {
        const uint32_t e = row >= 0 ? s_wfeed[row >> 6] : 0u;      // first feed, number of feeds
        const uint32_t f0 = e >> 16, nf = e & 0xffffu;
        for (uint32_t r = 0; __any(r < nf); ++r) {
            int32_t b0 = 0, b1 = 0, go = 0;
            if (r < nf) {
                const ResFeed F = s_feed[f0 + r];
                const int64_t at = (int64_t)(row - F.word0 * kWave) * F.stride;
                b0 = F.bounds[at] + F.syn;
                b1 = F.bounds[at + 1] + F.syn;
                go = F.g0;
            }
            slices_to_lds(acc, col, wt, b0, b1, go, s_fix, lane);
        }
    };

    for (int64_t t = t0; t < t_end; ++t) {
        // ---- the rows of S(t - 1): a lane per half word, each wave an equal
        // share of them (a single block has listed them as it published)
        uint32_t *pw = reinterpret_cast<uint32_t *>(s_word + ((t + 1) & 1) * n_words);
        if (multi || t == t0) {
            for (int i0 = h_begin; i0 < h_end; i0 += kResPoll * kWave) {
                uint32_t half[kResPoll];
                if (t == t0) {
                    const uint32_t *src = reinterpret_cast<const uint32_t *>(a.bits + ((t + 1) & 1) * a.n_waves + w_first);
#pragma unroll
                    for (int u = 0; u < kResPoll; ++u) {
                        const int i = i0 + u * kWave + lane;
                        half[u] = i < h_end && !a.skip_first ? src[i] : 0u;
                    }
                } else {
                    // A ring slot is written again kResRing steps later: its
                    // writer has then seen a later step's words of every block,
                    // each published after its block had read the slot.
                    const uint32_t tag = a.tag0 + (uint32_t)(t - 1 - t0);
                    const uint64_t *src = xw + ((t - 1) & (kResRing - 1)) * 2 * n_words;
                    const int64_t since = wall_clock64();
                    for (uint32_t tries = 1;; ++tries) {
                        uint64_t x[kResPoll];
#pragma unroll
                        for (int u = 0; u < kResPoll; ++u)
                            if (i0 + u * kWave < h_end)
                                x[u] = __hip_atomic_load(src + min(i0 + u * kWave + lane, h_end - 1), __ATOMIC_RELAXED,
                                                         __HIP_MEMORY_SCOPE_AGENT);
                        bool here = true;
#pragma unroll
                        for (int u = 0; u < kResPoll; ++u) {
                            half[u] = 0u;
                            if (i0 + u * kWave < h_end) {
                                here &= (uint32_t)(x[u] >> 32) == tag;
                                if (i0 + u * kWave + lane < h_end) half[u] = (uint32_t)x[u];
                            }
                        }
                        if (__all(here)) break;
                        // the blocks are resident together (cooperative launch),
                        // so a wait this long is a fault: flag it and end
                        if ((tries & 1023u) == 0 && wall_clock64() - since > a.max_wait) {
                            s_fail = 1;
#pragma unroll
                            for (int u = 0; u < kResPoll; ++u) half[u] = 0u;
                            break;
                        }
                    }
                }
#pragma unroll
                for (int u = 0; u < kResPoll; ++u) {
                    const int i = i0 + u * kWave + lane;
                    uint32_t h = half[u];
                    if (i < h_end) pw[i] = h;
                    if (h != 0 && s_wfeed[i >> 1] != 0) {
                        uint32_t at = atomicAdd(&s_cnt[l_prev], (uint32_t)__popc(h));
                        for (; h != 0 && at < (uint32_t)kResList; h &= h - 1, ++at)
                            s_list[l_prev * kResList + at] = i * 32 + __builtin_ctz(h);
                    }
                }
            }
        }
        __syncthreads();

        // ---- deliver them: a row per lane, dealt out over the waves
        unsigned long long *acc = s_acc + (t & 1) * n_g;
        const int n_rows = (int)s_cnt[l_prev];
        if (threadIdx.x == 0) s_cnt[l_next] = 0;
        if (n_rows <= kResList) {
            for (int base = 0; base < n_rows; base += nt) {
                const int i = base + lane * nw + wid;
                deliver_rows(acc, i < n_rows ? (int32_t)s_list[l_prev * kResList + i] : -1);
            }
        } else {
            // more rows than the list holds: from the words, row by row of a
            // lane's half word
            for (int i0 = h_begin; i0 < h_end; i0 += kWave) {
                const int i = i0 + lane;
                uint32_t h = i < h_end ? pw[i] : 0u;
                for (; __any(h != 0); h &= h - 1) deliver_rows(acc, h != 0 ? i * 32 + __builtin_ctz(h) : -1);
            }
        }
        __syncthreads();
        if (multi && s_fail) {
            if (threadIdx.x == 0) atomicOr(&a.st->overflow, 4u);
            return;
        }

        // ---- update the block's neurons, one word per wave at a time
        for (int w = wid; w < n_state; w += nw) {
            CResWord &W = words[w];
            CSeg &S = ((CSeg *)a.segs)[W.seg];
            const int64_t gid = W.gw * kWave + lane;
            const int32_t j = (int32_t)(gid - S.base), n_in = S.n_in;
            const bool active = j < S.n;
            double *x = s_state + w * kResState * kWave + lane;
            double v = x[0];
            const double v0 = v;
            double iin = S.i_ext;
#pragma unroll
            for (int q = 0; q < kMaxIn; ++q)
                if (q < n_in) {
                    const int32_t at = W.g_off[q] + lane;
                    const int64_t g = (int64_t)(s_g[at] + acc[at]);
                    acc[at] = 0;
                    iin += (double)g * kFixInv * (S.in_erev[q] - v0);
                    s_g[at] = (unsigned long long)fix_decay(g, S.in_decay[q]);
                }
            bool spike;
            double m = x[kWave], h = 0.0, n = 0.0;      // (Izhikevich: m is u)
            const bool is_hh = !kIzhOn || S.kind == kHH;
            if (is_hh) {
                h = x[2 * kWave];
                n = x[3 * kWave];
                const HHConst P{S.gna, S.ena, S.gk, S.ek, S.gl, S.el};
                const double hc = a.hs * S.inv_c;
                v = fma(hc, iin - x[4 * kWave], v);     // the first substep, begun by hh_ahead
                for (int k = 1; k < a.substeps; ++k) hh_substep(P, a.hs, hc, iin, v, m, h, n);
                spike = active && (v0 < 0.0) && (v >= 0.0);
            } else {
                const float4 pr = a.izp[S.izp_base + min(j, S.n - 1)];
                for (int k = 0; k < a.substeps; ++k) izh_substep((double)pr.x, (double)pr.y, a.hs, iin, v, m);
                spike = active && v >= kIzhPeak;
                if (active && fits_fp32(v0) && !fits_fp32(v)) atomicAdd(&a.nan_count[S.inst], 1);
                if (spike) {
                    v = (double)pr.z;
                    m = m + (double)pr.w;
                }
            }
            publish(t, l_cur, W.gw, __ballot(spike));
            if (is_hh && active && fits_fp32(v0) && !fits_fp32(v)) atomicAdd(&a.nan_count[S.inst], 1);
            if (spike) atomicAdd(&a.counts[gid], 1);
            if (kRec && S.record_vbar) s_vsum[w * kWave + lane] += v;
            // the state is held as fp32 pairs between steps
            float vh, vl, mh, ml, hh, hl, nh, nl;
            pair_split(v, vh, vl);
            pair_split(m, mh, ml);
            pair_split(h, hh, hl);
            pair_split(n, nh, nl);
            if (t + 1 < t_end) {
                v = (double)vh + (double)vl;
                m = (double)mh + (double)ml;
                if (is_hh) {
                    hh_ahead(S, x, v, m, (double)hh + (double)hl, (double)nh + (double)nl);
                } else {
                    x[0] = v;
                    x[kWave] = m;
                }
            } else if (active) {
                a.vh[gid] = vh;
                a.vl[gid] = vl;
                a.mh[gid] = mh;
                a.ml[gid] = ml;
                if (is_hh) {
                    a.hh[gid] = hh;
                    a.hl[gid] = hl;
                    a.nh[gid] = nh;
                    a.nl[gid] = nl;
                }
#pragma unroll
                for (int q = 0; q < kMaxIn; ++q)
                    if (q < n_in) a.G[S.in_G[q] + j] = (int64_t)s_g[W.g_off[q] + lane];
                if (kRec && S.record_vbar) a.vsum[gid] = s_vsum[w * kWave + lane];
            }
        }
        if (t + 1 == t_end) break;
        sources(t + 1, l_next);
        const int l = l_prev;
        l_prev = l_cur;
        l_cur = l_next;
        l_next = l;
    }

    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.st->t_prop = t_end;
        a.st->t_neuron = t_end;
    }
}

// bounds[row][part] of one split projection: where each part of the post
// population starts in the row (columns ascend within a row).
__global__ void k_slice_bounds(ResSplit d, const int32_t *rp_pool, const int32_t *col_pool, const int32_t *starts,
                               int32_t *out)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t np = d.parts + 1;
    if (i >= (int64_t)d.n_pre * np) return;
    const int32_t row = (int32_t)(i / np), part = (int32_t)(i % np);
    const int32_t *rp = rp_pool + d.rp_base;
    const int32_t *col = col_pool + d.syn_base;
    int32_t lo = rp[row], hi = rp[row + 1];
    const int32_t lim = starts[d.start0 + part];
    while (lo < hi) {
        const int32_t mid = lo + (hi - lo) / 2;
        if (col[mid] < lim) lo = mid + 1; else hi = mid;
    }
    out[d.out0 + i] = lo;
}

hipError_t launch_slice_bounds(const ResSplit &d, const int32_t *rp_pool, const int32_t *col_pool,
                               const int32_t *starts, int32_t *out, hipStream_t s)
{
    const int64_t n = (int64_t)d.n_pre * (d.parts + 1);
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_slice_bounds, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, d, rp_pool, col_pool, starts,
                       out);
    return hipGetLastError();
}

namespace {

const void *resident_kernel(int feat)
{
    switch (feat) {
    case 0: return reinterpret_cast<const void *>(&k_resident<0>);
    case kFeatIzh: return reinterpret_cast<const void *>(&k_resident<kFeatIzh>);
    case kFeatRec: return reinterpret_cast<const void *>(&k_resident<kFeatRec>);
    case kFeatIzh | kFeatRec: return reinterpret_cast<const void *>(&k_resident<kFeatIzh | kFeatRec>);
    default: return nullptr;
    }
}

}  // namespace

bool resident_fits(int feat, int block, size_t lds, int blocks, bool together, int n_cu)
{
    const void *k = resident_kernel(feat);
    if (!k) return false;
    int per_cu = 0;
    if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, block, lds) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return per_cu > 0 && (!together || (int64_t)per_cu * n_cu >= blocks);
}

hipError_t launch_resident(const ResArgs &a, int feat, int blocks, int block, size_t lds, bool together, hipStream_t s)
{
    const void *k = resident_kernel(feat);
    if (!k) return hipErrorInvalidValue;
    ResArgs args = a;
    void *params[] = {&args};
    return together ? hipLaunchCooperativeKernel(k, dim3((unsigned)blocks), dim3((unsigned)block), params, (unsigned)lds, s)
                    : hipLaunchKernel(k, dim3((unsigned)blocks), dim3((unsigned)block), params, lds, s);
}

}  // namespace snn
