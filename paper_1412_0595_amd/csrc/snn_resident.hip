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
// (so that the waves share them evenly), synapses (a block's own, slice after
// slice; their bounds in LDS where these fit), LDS sums, voltage.  A step's
// last voltage needs the rates of all substeps but the first, whose gates and
// ionic current the step's input does not enter, and the last, whose gates
// only the next step uses: of three substeps' rates one lies before the spike
// words and two run after they have left, while they travel.  Waves without a
// neuron draw the sources (in short calls) and poll the words meanwhile.
//
// Time per step, step kernels -> here (2 000 steps a call): 1 100 neurons in 7
// blocks 7.0 -> 3.1 us, 21 000 neurons in 96 blocks 10.1 -> 4.4, 325 networks of
// 220 neurons 19.7 -> 5.0, 48 of 2 000 to 20 000 neurons 36 -> 19.  An
// exchange takes 0.8 to 2 of these, one evaluation of the rates 0.6.
#include <algorithm>

#include "snn_device.h"

namespace snn {

namespace {

using CResBlock = const __attribute__((address_space(4))) ResBlock;

using GlobalU64 = __attribute__((address_space(1))) uint64_t;
using GlobalI32 = __attribute__((address_space(1))) int32_t;   // (generic loads would wait for LDS and memory alike)

constexpr int kResPoll = 4;    // half words a lane asks for at once
constexpr int kResState = 5;   // doubles of state per neuron in LDS
constexpr int kResHelpers = 3; // waves without neurons that take the reading off the others

// A word's constants, in LDS: one round trip where the population record would
// take several scalar loads in turn.
struct NeuronRec {
    double gna, ena, gk, ek, gl, el;      // Traub-Miles
    double hc, i_ext;                     // dt / substeps / C
    double erev[kMaxIn], decay[kMaxIn];
    int32_t g_off[kMaxIn];                // LDS conductances, per incoming projection
    int32_t n_in, rel, active;            // inputs, word of the instance, lanes with a neuron
    int32_t izh, rec, izp, inst, seg;     // Izhikevich: place of its parameters
};
struct SourceRec {
    uint32_t seed_lo, seed_hi, pop;
    int32_t rel, active, j0;              // word of the instance, lanes with a source, its first source
    uint64_t thresh;
};
static_assert(sizeof(NeuronRec) == kResNeuronRec && sizeof(SourceRec) == kResSourceRec, "LDS sizes of the plan");

// A batch of kN slots of up to 64 entries of one slice each: the entries, and
// which of them the lane adds (bit u: slot u's).  Past the last slice a slot
// repeats its entries and adds nothing.
template <int kN>
struct SlotBatch {
    int2 e[kN];
    uint32_t add;
};

// The next slices of a wave's rows: the one in progress, [k, k1), and the
// lanes left in rem.
struct SliceWalk {
    int32_t b0, b1;      // lane l: its slice's bounds in the block's synapses (empty: none)
    uint64_t rem;
    int32_t k, k1;
};

template <int kN>
__device__ __forceinline__ bool load_slots(SlotBatch<kN> &B, SliceWalk &W, const int2 *syn, int lane)
{
    if (!W.rem && W.k >= W.k1) return false;
    B.add = 0;
#pragma unroll
    for (int u = 0; u < kN; ++u) {
        if (W.k >= W.k1 && W.rem) {
            const int r = __builtin_ctzll(W.rem);
            W.rem &= W.rem - 1;
            W.k = __builtin_amdgcn_readlane(W.b0, r);
            W.k1 = __builtin_amdgcn_readlane(W.b1, r);
        }
        const int32_t kk = W.k + lane;
        B.add |= (kk < W.k1 ? 1u : 0u) << u;
        B.e[u] = syn[(uint32_t)min(kk, W.k1 - 1)];
        W.k += kWave;
    }
    return true;
}

template <int kN>
__device__ __forceinline__ void add_slots(const SlotBatch<kN> &B, unsigned long long *s_g, double s)
{
    // (the empty asm keeps the wait for this batch ahead of the branches, so
    // that it does not cover the next batch's loads)
#pragma unroll
    for (int u = 0; u < kN; ++u) asm volatile("" ::"v"(B.e[u].x), "v"(B.e[u].y));
#pragma unroll
    for (int u = 0; u < kN; ++u)
        if ((B.add >> u) & 1u)
            atomicAdd(s_g + B.e[u].x, (unsigned long long)fix_increment(s, __int_as_float(B.e[u].y)));
}

// Adds slices into the block's conductances; a batch's loads are in flight
// while the one before is added.
__device__ __forceinline__ void slices_to_lds(unsigned long long *s_g, const int2 *syn, int32_t b0, int32_t b1, double s,
                                              int lane)
{
    SliceWalk W{b0, b1, __ballot(b1 > b0), 0, 0};
    if (__popcll(W.rem) <= 2 && !__any(b1 - b0 > kWave)) {
        SlotBatch<2> A;
        if (load_slots(A, W, syn, lane)) add_slots(A, s_g, s);
        return;
    }
    SlotBatch<8> A, B;
    if (!load_slots(A, W, syn, lane)) return;
    for (;;) {
        const bool more_b = load_slots(B, W, syn, lane);
        add_slots(A, s_g, s);
        if (!more_b) return;
        const bool more_a = load_slots(A, W, syn, lane);
        add_slots(B, s_g, s);
        if (!more_a) return;
    }
}

}  // namespace

// One block's part of a cluster for n steps from step t0.
template <int FEAT>
__global__ __launch_bounds__(1024) void k_resident(ResArgs a)
{
    extern __shared__ __align__(16) char s_mem[];
    __shared__ uint32_t s_fail, s_cnt[2], s_src[2];   // rows listed, source words taken; of alternating steps
    const int lane = threadIdx.x & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int nt = (int)blockDim.x, nw = nt >> 6;
    constexpr bool kIzhOn = (FEAT & kFeatIzh) != 0, kRec = (FEAT & kFeatRec) != 0;

    CResBlock &B = ((CResBlock *)a.blocks)[blockIdx.x];
    const int n_state = B.n_state, n_poi = B.n_poi, n_words = B.n_words, n_g = B.n_g;
    const int n_early = B.n_early, n_read = n_early + B.n_late;
    const int64_t w_first = B.w_first;      // the instance's first spike word
    const bool multi = B.n_blocks > 1;
    const bool late_feeds = B.late_feeds != 0;
    const bool drawn = a.drawn != nullptr;
    const double s_fix = (double)a.gscale[B.inst] * kFixOne;
    const int2 *syn = a.syn + B.syn0;
    uint64_t *xw = a.xbuf + B.x_off;        // kResRing slots of 2 n_words tagged halves

    // LDS: conductances, neuron state, recorded sums, feeds, the words'
    // constants, spike words of two steps, the words that the block reads
    // (sources' first) and the latters' places among the drawn, each word's
    // feeds, the listed rows (neurons of the
    // instance), slice bounds of the feeds that have them here
    unsigned long long *s_g = reinterpret_cast<unsigned long long *>(s_mem);
    double *s_state = reinterpret_cast<double *>(s_g + n_g);
    double *s_vsum = s_state + n_state * kResState * kWave;
    ResFeed *s_feed = reinterpret_cast<ResFeed *>(s_vsum + (kRec ? n_state * kWave : 0));
    NeuronRec *s_rec = reinterpret_cast<NeuronRec *>(s_feed + B.n_feed);
    SourceRec *s_src_rec = reinterpret_cast<SourceRec *>(s_rec + n_state);
    uint64_t *s_word = reinterpret_cast<uint64_t *>(s_src_rec + n_poi);
    uint32_t *s_read = reinterpret_cast<uint32_t *>(s_word + 2 * n_words);
    uint32_t *s_drawn = s_read + n_read;
    uint32_t *s_wfeed = s_drawn + n_early;
    uint32_t *s_list = s_wfeed + n_words;
    int32_t *s_bounds = reinterpret_cast<int32_t *>(s_list + kResList);

    const int64_t t0 = a.t0, t_end = a.t0 + a.n;
    if (threadIdx.x == 0) s_fail = s_cnt[0] = s_cnt[1] = s_src[0] = s_src[1] = 0;
    for (int i = threadIdx.x; i < B.n_feed; i += nt) s_feed[i] = a.feeds[B.feed0 + i];
    for (int i = threadIdx.x; i < n_words; i += nt) s_wfeed[i] = a.wfeeds[B.wfeed0 + i];
    for (int i = threadIdx.x; i < n_read; i += nt) s_read[i] = a.reads[B.read0 + i];
    for (int i = threadIdx.x; i < n_early; i += nt) s_drawn[i] = a.drawn_at[B.early0 + i];
    for (int w = threadIdx.x; w < n_state + n_poi; w += nt) {
        const ResWord &W = a.words[B.word0 + w];
        const Seg &S = a.segs[W.seg];
        const int32_t rel = (int32_t)(W.gw - w_first), j0 = (int32_t)(W.gw * kWave - S.base);
        const int32_t active = min(S.n - j0, kWave);
        if (w < n_state) {
            NeuronRec &R = s_rec[w];
            R.gna = S.gna;
            R.ena = S.ena;
            R.gk = S.gk;
            R.ek = S.ek;
            R.gl = S.gl;
            R.el = S.el;
            R.hc = a.hs * S.inv_c;
            R.i_ext = S.i_ext;
            for (int q = 0; q < kMaxIn; ++q) {
                R.erev[q] = q < S.n_in ? S.in_erev[q] : 0.0;
                R.decay[q] = q < S.n_in ? S.in_decay[q] : 0.0;
                R.g_off[q] = q < S.n_in ? W.g_off[q] : 0;
            }
            R.n_in = S.n_in;
            R.rel = rel;
            R.active = active;
            R.izh = S.kind == kIzh;
            R.rec = S.record_vbar;
            R.izp = (int32_t)S.izp_base + j0;
            R.inst = S.inst;
            R.seg = W.seg;
        } else {
            s_src_rec[w - n_state] = SourceRec{(uint32_t)S.seed, (uint32_t)(S.seed >> 32), (uint32_t)S.pop, rel, active, j0,
                                               S.thresh};
        }
    }
    for (int f = 0; f < B.n_feed; ++f) {
        const ResFeed F = a.feeds[B.feed0 + f];
        if (F.lds >= 0)
            for (int i = threadIdx.x; i <= F.n_pre; i += nt) s_bounds[F.lds + i] = F.bounds[i];
    }
    __syncthreads();

    // A word of step t: to the cluster (a single block: to its own words and,
    // with a membrane, list) and the records.
    auto publish = [&](int64_t t, bool list, int rel, uint64_t ball) __attribute__((always_inline)) {
        if (multi) {
            if (lane < 2) {
                const uint64_t tag = (uint64_t)(uint32_t)(a.tag0 + (uint32_t)(t - t0)) << 32;
                __hip_atomic_store(xw + (t & (kResRing - 1)) * 2 * n_words + 2 * rel + lane,
                                   tag | (uint32_t)(ball >> (32 * lane)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        } else {
            if (lane == 0) s_word[(t & 1) * n_words + rel] = ball;
            if (list && ball != 0 && s_wfeed[rel] != 0) {
                uint32_t at = 0;
                if (lane == 0) at = atomicAdd(&s_cnt[t & 1], (uint32_t)__popcll(ball));
                at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at) + (uint32_t)__popcll(ball & ((1ull << lane) - 1ull));
                if (((ball >> lane) & 1ull) && at < (uint32_t)kResList) s_list[at] = rel * kWave + lane;
            }
        }
        if (lane == 0) {
            if (a.raster) a.raster[(t % a.raster_steps) * a.n_waves + w_first + rel] = ball;
            if (t == t_end - 1 && (list || !multi)) a.bits[(t & 1) * a.n_waves + w_first + rel] = ball;
        }
    };
    // The block's Poisson words of step t, two at a time by the next free wave
    // (one draw's dependent products hide behind the other's).
    auto sources = [&](int64_t t) __attribute__((always_inline)) {
        while (n_poi > 0 && !drawn) {
            int w = 0;
            if (lane == 0) w = (int)atomicAdd(&s_src[t & 1], 2u);
            w = __builtin_amdgcn_readfirstlane(w);
            if (w >= n_poi) break;
            const int w2 = min(w + 1, n_poi - 1);
            auto draw = [&](const SourceRec &R) __attribute__((always_inline)) {
                return philox_first_word((uint32_t)(R.j0 + lane), (uint32_t)t, (uint32_t)((uint64_t)t >> 32), R.pop,
                                         R.seed_lo, R.seed_hi);
            };
            auto finish = [&](const SourceRec &R, uint32_t x) __attribute__((always_inline)) {
                const int rel = __builtin_amdgcn_readfirstlane(R.rel);
                const bool spike = lane < R.active && (uint64_t)x < R.thresh;
                publish(t, false, rel, __ballot(spike));
                if (spike) atomicAdd(&a.counts[(w_first + rel) * kWave + lane], 1);
            };
            const uint32_t x = draw(s_src_rec[w]), x2 = draw(s_src_rec[w2]);
            finish(s_src_rec[w], x);
            if (w2 > w) finish(s_src_rec[w2], x2);
        }
    };
    // Half words [i0, i0 + 64 kResPoll) of step t among those that the block
    // reads, up to `end`; waits for them.
    auto read_halves = [&](int64_t t, int i0, int end, uint32_t (&half)[kResPoll]) __attribute__((always_inline)) {
        if (t < t0) {
            const uint32_t *src = reinterpret_cast<const uint32_t *>(a.bits + (t & 1) * a.n_waves + w_first);
#pragma unroll
            for (int u = 0; u < kResPoll; ++u) {
                const int i = i0 + u * kWave + lane;
                half[u] = i < end && !a.skip_first ? src[2 * s_read[i >> 1] + (i & 1)] : 0u;
            }
            asm volatile("");
            return;
        }
        if (!multi && !drawn) {
            const uint32_t *src = reinterpret_cast<const uint32_t *>(s_word + (t & 1) * n_words);
#pragma unroll
            for (int u = 0; u < kResPoll; ++u) {
                const int i = i0 + u * kWave + lane;
                half[u] = i < end ? src[2 * s_read[i >> 1] + (i & 1)] : 0u;
            }
            return;
        }
        // A ring slot is written again kResRing steps later: its writer has
        // then seen a later step's words of every block that reads it, each
        // published after that block had read the slot.  (A block of sources
        // that nothing reads may fall further behind and find later tags;
        // it has no use for the words.)
        const uint32_t tag = a.tag0 + (uint32_t)(t - t0);
        const uint64_t *src = xw + (t & (kResRing - 1)) * 2 * n_words;
        const int64_t since = wall_clock64();
        const GlobalU64 *at[kResPoll];
#pragma unroll
        for (int u = 0; u < kResPoll; ++u) {
            const int i = min(i0 + u * kWave + lane, end - 1);
            at[u] = (const GlobalU64 *)src + 2 * s_read[i >> 1] + (i & 1);
            if (drawn && i < 2 * n_early)
                at[u] = (const GlobalU64 *)a.drawn + ((t - t0) * a.n_drawn + s_drawn[i >> 1]) * 2 + (i & 1);
        }
        for (uint32_t tries = 1;; ++tries) {
            uint64_t x[kResPoll];
#pragma unroll
            for (int u = 0; u < kResPoll; ++u)
                if (i0 + u * kWave < end) x[u] = __hip_atomic_load(at[u], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            bool here = true;
#pragma unroll
            for (int u = 0; u < kResPoll; ++u) {
                half[u] = 0u;
                if (i0 + u * kWave < end) {
                    here &= (int32_t)((uint32_t)(x[u] >> 32) - tag) >= 0;
                    if (i0 + u * kWave + lane < end) half[u] = (uint32_t)x[u];
                }
            }
            if (__all(here)) break;
            // the blocks are resident together (cooperative launch), so a
            // wait this long is a fault: flag it and end
            if ((tries & 1023u) == 0 && wall_clock64() - since > a.max_wait) {
                s_fail = 1;
#pragma unroll
                for (int u = 0; u < kResPoll; ++u) half[u] = 0u;
                break;
            }
        }
    };
    // Adds the slices of the rows that its lanes hold (neurons of the
    // instance; -1: none).
    auto deliver_rows = [&](int32_t row) __attribute__((always_inline)) {
        const uint32_t e = row >= 0 ? s_wfeed[row >> 6] : 0u;      // first feed, number of feeds
        const uint32_t f0 = e >> 16, nf = e & 0xffffu;
        for (uint32_t r = 0; __any(r < nf); ++r) {
            int32_t b0 = 0, b1 = 0;
            if (r < nf) {
                const ResFeed F = s_feed[f0 + r];
                const int32_t i = row - F.word0 * kWave;
                if (F.lds >= 0) {
                    b0 = s_bounds[F.lds + i];
                    b1 = s_bounds[F.lds + i + 1];
                } else {
                    const GlobalI32 *bd = (const GlobalI32 *)F.bounds + i;
                    b0 = bd[0];
                    b1 = bd[1];
                }
            }
            slices_to_lds(s_g, syn, b0, b1, s_fix, lane);
        }
    };
    // Lists the rows of half words [begin, end) of step t.
    auto list_rows = [&](int64_t t, int begin, int end) __attribute__((always_inline)) {
        for (int i0 = begin; i0 < end; i0 += kResPoll * kWave) {
            uint32_t half[kResPoll];
            read_halves(t, i0, end, half);
#pragma unroll
            for (int u = 0; u < kResPoll; ++u) {
                const int i = i0 + u * kWave + lane;
                if (i >= end) continue;
                const uint32_t rel = s_read[i >> 1];
                uint32_t h = half[u];
                reinterpret_cast<uint32_t *>(s_word + (t & 1) * n_words)[2 * rel + (i & 1)] = h;
                if (h != 0 && s_wfeed[rel] != 0) {
                    uint32_t at = atomicAdd(&s_cnt[t & 1], (uint32_t)__popc(h));
                    for (; h != 0 && at < (uint32_t)kResList; h &= h - 1, ++at)
                        s_list[at] = rel * kWave + (i & 1) * 32 + __builtin_ctz(h);
                }
            }
        }
    };
    // Delivers the listed rows of step t, dealt out over the waves; if there
    // were more than the list holds, those of the half words that the block
    // read.
    auto deliver_list = [&](int64_t t) __attribute__((always_inline)) {
        const int n_rows = (int)s_cnt[t & 1];
        if (threadIdx.x == 0) s_cnt[(t + 1) & 1] = s_src[t & 1] = 0;   // (t + 1's sources are drawn)
        if (n_rows <= kResList) {
            for (int base = 0; base < n_rows; base += nt) {
                const int i = base + lane * nw + wid;
                deliver_rows(i < n_rows ? (int32_t)s_list[i] : -1);
            }
            return;
        }
        const uint32_t *w = reinterpret_cast<const uint32_t *>(s_word + (t & 1) * n_words);
        for (int base = 0; base < 2 * n_read; base += nt) {
            const int i = base + lane * nw + wid;
            const uint32_t at = i < 2 * n_read ? 2 * s_read[i >> 1] + (i & 1) : 0u;
            uint32_t h = i < 2 * n_read && s_wfeed[at >> 1] != 0 ? w[at] : 0u;
            for (; __any(h != 0); h &= h - 1) deliver_rows(h != 0 ? at * 32 + __builtin_ctz(h) : -1);
        }
    };
    // a wave's share of half words [begin, end), as wave h of nh
    auto share = [&](int &begin, int &end, int h, int nh) __attribute__((always_inline)) {
        const int each = (end - begin + nh - 1) / nh, first = begin + h * each;
        end = min(first + each, end);
        begin = first;
    };
    // Traub-Miles: the part of a step's first substep that its input does not
    // enter, from (v, m, h, n) to LDS: v, the gates after it, the ionic current.
    auto hh_ahead = [&](const NeuronRec &P, double *x, double v, double m, double h, double n) __attribute__((always_inline)) {
        x[0] = v;
        x[4 * kWave] = hh_ionic(P, v, m, h, n);
        hh_gates(a.hs, v, m, h, n);
        x[kWave] = m;
        x[2 * kWave] = h;
        x[3 * kWave] = n;
    };

    // ---- state in
    for (int w = wid; w < n_state; w += nw) {
        const NeuronRec &R = s_rec[w];
        const Seg &S = a.segs[R.seg];
        const int64_t gid = (w_first + R.rel) * kWave + lane;
        const int32_t jj = min((int32_t)(gid - S.base), S.n - 1);
        double *x = s_state + w * kResState * kWave + lane;
#pragma unroll
        for (int q = 0; q < kMaxIn; ++q)
            if (q < S.n_in) s_g[R.g_off[q] + lane] = (unsigned long long)a.G[S.in_G[q] + jj];
        if constexpr (kRec) s_vsum[w * kWave + lane] = R.rec ? a.vsum[gid] : 0.0;
        const double v = pair_load(a.vh, a.vl, gid), m = pair_load(a.mh, a.ml, gid);
        if (!kIzhOn || !R.izh) {
            hh_ahead(R, x, v, m, pair_load(a.hh, a.hl, gid), pair_load(a.nh, a.nl, gid));
        } else {
            x[0] = v;
            x[kWave] = m;
        }
    }
    // The waves without a word to update (at least kResHelpers of them; else
    // all, after their updates) read the words; those beside a block of
    // neurons that only sources feed are read every kResCheck steps, which
    // keeps the cluster's blocks within the ring.
    const int n_upd = min(n_state, nw);
    const bool helpers = nw - n_upd >= kResHelpers;
    const int help_i = helpers ? wid - n_upd : wid, help_n = helpers ? nw - n_upd : nw;
    int e_begin = 0, e_end = 2 * n_early, r_begin = 0, r_end = 2 * n_read;
    share(e_begin, e_end, help_i, help_n);
    share(r_begin, r_end, help_i, help_n);
    // the next step whose starting state is also left as a checkpoint
    int64_t next_ckpt = a.ckpt_every > 0 ? (t0 / a.ckpt_every + 1) * a.ckpt_every : -1;
    const int64_t t_all = multi ? t0 : t0 - 1;   // every word is read up to this step, see below
    // (step t0 - 1 has only the part that follows its update)
    for (int64_t t = t0 - 1;; ++t) {
        // ---- the block's neurons up to the voltage after the step, one word
        // per wave at a time
        for (int w = t < t0 ? n_state : wid; w < n_state; w += nw) {
            const NeuronRec &R = s_rec[w];
            const int n_in = __builtin_amdgcn_readfirstlane(R.n_in), rel = __builtin_amdgcn_readfirstlane(R.rel);
            const bool active = lane < R.active;
            double *x = s_state + w * kResState * kWave + lane;
            double v = x[0], m = x[kWave];              // (Izhikevich: m is u)
            double h = x[2 * kWave], n = x[3 * kWave];
            const double iion = x[4 * kWave], v0 = v;
            double iin = R.i_ext;
            auto input = [&](int q) __attribute__((always_inline)) {
                const int32_t at = R.g_off[q] + lane;
                const int64_t g = (int64_t)s_g[at];
                iin += (double)g * kFixInv * (R.erev[q] - v0);
                s_g[at] = (unsigned long long)fix_decay(g, R.decay[q]);
            };
            if (n_in > 0) input(0);
            if (n_in > 1) input(1);
            if (n_in > 2) input(2);
            if (n_in > 3) input(3);
            bool spike;
            if (!kIzhOn || !__builtin_amdgcn_readfirstlane(R.izh)) {
                v = fma(R.hc, iin - iion, v);           // the first substep, begun by hh_ahead
                for (int k = 2; k < a.substeps; ++k) hh_substep(R, a.hs, R.hc, iin, v, m, h, n);
                const double vl = v;
                if (a.substeps > 1) v = fma(R.hc, iin - hh_ionic(R, v, m, h, n), v);
                spike = active && (v0 < 0.0) && (v >= 0.0);
                publish(t, true, rel, __ballot(spike));
                // the last substep's gates follow from its starting voltage vl
                x[2 * kWave] = h;
                x[3 * kWave] = n;
                x[4 * kWave] = vl;
                if (active && fits_fp32(v0) && !fits_fp32(v)) atomicAdd(&a.nan_count[R.inst], 1);
            } else {
                const float4 pr = a.izp[R.izp + min(lane, R.active - 1)];
                for (int k = 0; k < a.substeps; ++k) izh_substep((double)pr.x, (double)pr.y, a.hs, iin, v, m);
                spike = active && v >= kIzhPeak;
                publish(t, true, rel, __ballot(spike));
                if (active && fits_fp32(v0) && !fits_fp32(v)) atomicAdd(&a.nan_count[R.inst], 1);
                if (spike) {
                    v = (double)pr.z;
                    m = m + (double)pr.w;
                }
            }
            x[0] = v;
            x[kWave] = m;
            if (spike) atomicAdd(&a.counts[(w_first + rel) * kWave + lane], 1);
        }
        // ---- the rest of their step and the start of the next
        for (int w = t < t0 ? n_state : wid; w < n_state; w += nw) {
            const NeuronRec &R = s_rec[w];
            double *x = s_state + w * kResState * kWave + lane;
            double v = x[0], m = x[kWave], h = 0.0, n = 0.0;
            const bool is_hh = !kIzhOn || !__builtin_amdgcn_readfirstlane(R.izh);
            if (is_hh) {
                h = x[2 * kWave];
                n = x[3 * kWave];
                if (a.substeps > 1) hh_gates(a.hs, x[4 * kWave], m, h, n);
            }
            if (kRec && R.rec) s_vsum[w * kWave + lane] += v;
            // the state is held as fp32 pairs between steps
            float vh, vl, mh, ml, hh, hl, nh, nl;
            pair_split(v, vh, vl);
            pair_split(m, mh, ml);
            pair_split(h, hh, hl);
            pair_split(n, nh, nl);
            if (t + 1 == next_ckpt && next_ckpt < a.ckpt_end && lane < R.active) {
                const Seg &S = a.segs[R.seg];
                const int64_t gid = (w_first + R.rel) * kWave + lane;
                float *c = a.ckpt_state + (next_ckpt / a.ckpt_every) * 8 * a.n_waves * kWave + gid;
                int64_t *cg = a.ckpt_G + (next_ckpt / a.ckpt_every) * a.g_stride;
                const float pairs[8] = {vh, vl, mh, ml, hh, hl, nh, nl};
#pragma unroll
                for (int k = 0; k < 8; ++k)
                    if (k < 4 || is_hh) c[k * a.n_waves * kWave] = pairs[k];
#pragma unroll
                for (int q = 0; q < kMaxIn; ++q)
                    if (q < S.n_in) cg[S.in_G[q] + (gid - S.base)] = (int64_t)s_g[R.g_off[q] + lane];
            }
            if (t + 1 < t_end) {
                v = (double)vh + (double)vl;
                m = (double)mh + (double)ml;
                if (is_hh) {
                    hh_ahead(R, x, v, m, (double)hh + (double)hl, (double)nh + (double)nl);
                } else {
                    x[0] = v;
                    x[kWave] = m;
                }
            } else if (lane < R.active) {
                const Seg &S = a.segs[R.seg];
                const int64_t gid = (w_first + R.rel) * kWave + lane;
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
                    if (q < S.n_in) a.G[S.in_G[q] + (gid - S.base)] = (int64_t)s_g[R.g_off[q] + lane];
                if (kRec && R.rec) a.vsum[gid] = s_vsum[w * kWave + lane];
            }
        }
        if (t + 1 == next_ckpt) next_ckpt += a.ckpt_every;
        if (t + 1 == t_end) break;

        // ---- the next step's sources; deliver S(t).  An even number of steps
        // leaves its last words in the slot of `bits` that its first step was
        // delivered from, so no block writes them before its whole cluster has
        // read that slot: all await the first step's words of every block with
        // neurons, whether they need them or not, and sources, which are drawn
        // a step ahead, go there after the last step.
        sources(t + 1);
        if (help_i >= 0) {
            const bool all = t <= t_all || (multi && (late_feeds || (t & (kResCheck - 1)) == 0));
            list_rows(t, all ? r_begin : e_begin, all ? r_end : e_end);
        }
        __syncthreads();
        deliver_list(t);
        __syncthreads();
        if (multi && s_fail) {
            if (threadIdx.x == 0) atomicOr(&a.st->overflow, 4u);
            return;
        }
    }

    // the last step's source words, as this block sent them
    for (int w = multi && !drawn ? wid : n_poi; w < n_poi; w += nw) {
        const int rel = s_src_rec[w].rel;
        const uint64_t *x = xw + ((t_end - 1) & (kResRing - 1)) * 2 * n_words + 2 * rel;
        if (lane < 2)
            reinterpret_cast<uint32_t *>(a.bits + ((t_end - 1) & 1) * a.n_waves + w_first + rel)[lane] =
                (uint32_t)__hip_atomic_load(x + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        a.st->t_prop = t_end;
        a.st->t_neuron = t_end;
    }
}

// First entry of CSR row [lo, hi) with column >= lim (columns ascend).
__device__ __forceinline__ int32_t first_at(const int32_t *col, int32_t lo, int32_t hi, int32_t lim)
{
    while (lo < hi) {
        const int32_t mid = lo + (hi - lo) / 2;
        if (col[mid] < lim) lo = mid + 1; else hi = mid;
    }
    return lo;
}

// A block's slices of its feeds' rows: where each begins in the projection's
// CSR (from) and, one after another, in the block's own synapses (bounds).
__global__ __launch_bounds__(1024) void k_resident_bounds(const ResBlock *blocks, const ResSource *srcs,
                                                          const int32_t *rp_pool, const int32_t *col_pool,
                                                          int32_t *bounds, int32_t *from, int64_t *totals)
{
    __shared__ uint32_t s_sum[16];
    const ResBlock &B = blocks[blockIdx.x];
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x >> 6, nw = blockDim.x >> 6;
    int64_t total = 0;
    for (int f = 0; f < B.n_feed; ++f) {
        const ResSource &F = srcs[B.feed0 + f];
        const int32_t *rp = rp_pool + F.rp_base, *col = col_pool + F.syn_base;
        for (int32_t r0 = 0; r0 < F.n_pre; r0 += blockDim.x) {
            const int32_t r = r0 + threadIdx.x;
            uint32_t len = 0;
            if (r < F.n_pre) {
                const int32_t a = first_at(col, rp[r], rp[r + 1], F.c0), b = first_at(col, a, rp[r + 1], F.c1);
                from[F.bounds0 + r] = a;
                len = (uint32_t)(b - a);
            }
            const uint32_t incl = wave_incl_sum(len, lane);
            if (lane == kWave - 1) s_sum[wid] = incl;
            __syncthreads();
            uint32_t before = 0, all = 0;
            for (int w = 0; w < nw; ++w) {
                if (w < wid) before += s_sum[w];
                all += s_sum[w];
            }
            if (r < F.n_pre) bounds[F.bounds0 + r] = (int32_t)(total + before + incl - len);
            total += all;
            __syncthreads();
        }
        if (threadIdx.x == 0) bounds[F.bounds0 + F.n_pre] = (int32_t)total;
    }
    if (threadIdx.x == 0) totals[blockIdx.x] = total;
}

// The blocks' synapses (LDS conductance, weight) from the CSR pools; a
// wavefront per slice, grid (blocks, any).
__global__ __launch_bounds__(256) void k_resident_fill(const ResBlock *blocks, const ResSource *srcs,
                                                       const int32_t *col_pool, const float *w_pool,
                                                       const int32_t *bounds, const int32_t *from, int2 *syn)
{
    const ResBlock &B = blocks[blockIdx.x];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = (int)(blockIdx.y * (blockDim.x >> 6) + (threadIdx.x >> 6)), nw = (int)(gridDim.y * (blockDim.x >> 6));
    for (int f = 0; f < B.n_feed; ++f) {
        const ResSource &F = srcs[B.feed0 + f];
        const int32_t *col = col_pool + F.syn_base;
        const float *w = w_pool + F.syn_base;
        for (int32_t r = wave; r < F.n_pre; r += nw) {
            const int32_t b0 = bounds[F.bounds0 + r], b1 = bounds[F.bounds0 + r + 1], k0 = from[F.bounds0 + r];
            for (int32_t k = lane; k < b1 - b0; k += kWave)
                syn[B.syn0 + b0 + k] = make_int2(F.g0 + col[k0 + k], __float_as_int(w[k0 + k]));
        }
    }
}

hipError_t launch_resident_bounds(const ResBlock *blocks, int n, const ResSource *srcs, const int32_t *rp_pool,
                                  const int32_t *col_pool, int32_t *bounds, int32_t *from, int64_t *totals, hipStream_t s)
{
    hipLaunchKernelGGL(k_resident_bounds, dim3((unsigned)n), dim3(1024), 0, s, blocks, srcs, rp_pool, col_pool, bounds,
                       from, totals);
    return hipGetLastError();
}

hipError_t launch_resident_fill(const ResBlock *blocks, int n, const ResSource *srcs, const int32_t *col_pool,
                                const float *w_pool, const int32_t *bounds, const int32_t *from, int2 *syn, hipStream_t s)
{
    const int y = std::max(1, std::min(256, 4096 / n));
    hipLaunchKernelGGL(k_resident_fill, dim3((unsigned)n, (unsigned)y), dim3(256), 0, s, blocks, srcs, col_pool, w_pool,
                       bounds, from, syn);
    return hipGetLastError();
}

// The sources of a launch, before it: streams that several instances share
// (the runs of a sweep) are drawn once, all steps side by side; inside the
// launch each block would draw its own, step by step, beside its neurons (a
// sweep of 125 networks with 500 to 5 000 sources: 8.9 us a step, 7.0 with
// the draws ahead; 325 small ones 6.1 and 5.6).  A wavefront per word and
// kResDrawSteps steps.
__global__ __launch_bounds__(256) void k_resident_draw(ResArgs a, const ResDraw *draws, const int32_t *alias)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int64_t d = (int64_t)blockIdx.x * (blockDim.x >> 6) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (d >= a.n_drawn) return;
    const ResDraw &D = draws[d];
    uint64_t *out = const_cast<uint64_t *>(a.drawn);
    const int64_t k0 = (int64_t)blockIdx.y * kResDrawSteps, k1 = min(k0 + kResDrawSteps, a.n);
    const uint32_t seed_lo = D.seed_lo, seed_hi = D.seed_hi, pop = D.pop, j = (uint32_t)(D.j0 + lane);
    const uint64_t thresh = D.thresh;
    const bool active = lane < D.active;
    int32_t count = 0;
    for (int64_t k = k0; k < k1; ++k) {
        const int64_t t = a.t0 + k;
        const bool spike = active && (uint64_t)philox_first_word(j, (uint32_t)t, (uint32_t)((uint64_t)t >> 32), pop, seed_lo,
                                                                 seed_hi) < thresh;
        const uint64_t ball = __ballot(spike);
        count += spike ? 1 : 0;
        if (lane < 2)
            out[(k * a.n_drawn + d) * 2 + lane] =
                (uint64_t)(uint32_t)(a.tag0 + (uint32_t)k) << 32 | (uint32_t)(ball >> (32 * lane));
        // (of a ring shorter than the launch, its last round)
        if (a.raster && k >= a.n - a.raster_steps)
            for (int i = lane; i < D.n_alias; i += kWave)
                a.raster[(t % a.raster_steps) * a.n_waves + alias[D.alias0 + i]] = ball;
    }
    if (count)
        for (int i = 0; i < D.n_alias; ++i) atomicAdd(&a.counts[(int64_t)alias[D.alias0 + i] * kWave + lane], count);
}

// Their spike words of the launch's last step, after it (before, the slot may
// hold the words that its first step delivers).
__global__ void k_resident_last(ResArgs a, const ResDraw *draws, const int32_t *alias)
{
    const int64_t d = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (d >= a.n_drawn) return;
    const uint64_t *w = a.drawn + ((a.n - 1) * a.n_drawn + d) * 2;
    const uint64_t ball = (uint64_t)(uint32_t)w[0] | w[1] << 32;
    const ResDraw &D = draws[d];
    for (int i = 0; i < D.n_alias; ++i) a.bits[((a.t0 + a.n - 1) & 1) * a.n_waves + alias[D.alias0 + i]] = ball;
}

hipError_t launch_resident_last(const ResArgs &a, const ResDraw *draws, const int32_t *alias, hipStream_t s)
{
    if (a.n_drawn == 0) return hipSuccess;
    hipLaunchKernelGGL(k_resident_last, dim3((unsigned)((a.n_drawn + 63) / 64)), dim3(64), 0, s, a, draws, alias);
    return hipGetLastError();
}

hipError_t launch_resident_draw(const ResArgs &a, const ResDraw *draws, const int32_t *alias, hipStream_t s)
{
    if (a.n_drawn == 0) return hipSuccess;
    const dim3 grid((unsigned)((a.n_drawn + 3) / 4), (unsigned)((a.n + kResDrawSteps - 1) / kResDrawSteps));
    hipLaunchKernelGGL(k_resident_draw, grid, dim3(256), 0, s, a, draws, alias);
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

// (the attribute is the function's, so every network sets the same value)
bool resident_fits(int feat, int block, size_t lds, int blocks, bool together, int n_cu)
{
    const void *k = resident_kernel(feat);
    if (!k) return false;
    int per_cu = 0;
    if (hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kResLds) != hipSuccess ||
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
