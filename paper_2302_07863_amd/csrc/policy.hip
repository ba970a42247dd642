// Policy kernels of the BiLD library (gfx950): merge of the LM-head partial statistics, the fallback test
// (Section 3.3), the rollback test (Section 3.4), the commit of Algorithm 1 on the device, and the draws of the
// sampling variant (Appendix, "BiLD with Sampling") with the rejection-sampling acceptance of the methods the
// paper compares with (Section 4.2).
#include "policy_commit.h"

namespace bild {

// =====================================================================================
// Merge of the LM-head partials + policy + commit.  One workgroup.
//   mode 0  small step: token = argmax, fallback iff max p < alpha or n_max drafts pending
//   mode 1  review: nll_i = lse_i - z_i[draft_i]; r = first i with nll_i > alpha, else n;
//           y <- y[:draft_start + r] + [argmax of row r]; cache lengths follow
//   mode 2  plain greedy: always append
//   mode 3  no LM head: only advance the cache length by the rows consumed
//   mode 4  measurement: merge the statistics, commit nothing
// =====================================================================================
// LDS use of finish_body (from the start of the workgroup's LDS)
constexpr int kFinishLds = 3 * kMaxRows * 4;
// LDS of the sampling variant behind that: 16 waves x 16 bins, 1024 per-thread masses, a few scalars
constexpr int kDrawLds = 16 * 16 * 4 + 1024 * 4 + 128;

// Order-preserving integer image of a float: a < b  <=>  key(a) < key(b).
__device__ __forceinline__ uint32_t float_key(float f) {
    const uint32_t b = __float_as_uint(f);
    return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// Nucleus draw of the sampling variant (Appendix, BiLD with Sampling), by the whole workgroup (at most
// 1024 threads).  Nucleus = every token whose probability is at least that of the least likely member of
// the smallest top set reaching top_p; the draw walks the members in increasing id until their running mass
// exceeds u * mass.  The threshold is found exactly, as an integer key, by a radix search of 4 bits per
// sweep over the logits: with e_i = exp(z_i - m), K is the largest key with sum_{key_i >= K} e_i >= top_p * sum e_i.
// Returns the token to every thread.  `ws` is kDrawLds bytes of LDS.
// nucleus_search finds the threshold key and the nucleus' mass (in units of exp(z - m)); weighted_walk draws.
__device__ __forceinline__ void nucleus_search(const float* __restrict__ z, int V, float m, float top_p, char* ws,
                                               uint32_t& K_out, float& mass_out) {
    float* bins = (float*)ws;              // [16 waves][16]
    float* tmass = bins + 16 * 16;         // [1024]
    float* sc = tmass + 1024;              // scalars
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nthr = blockDim.x, nwv = nthr >> 6;
    uint32_t K = 0;
    float target = 0.f, mass = 0.f;
    // A row of up to 32 logits per thread stays in registers for all sweeps (one batch of loads); longer rows
    // are re-read from L2 every sweep, eight loads at a time.
    constexpr int CACHED = 32;
    const bool cached = V <= CACHED * nthr;
    float zc[CACHED];
    if (cached) {
#pragma unroll
        for (int c = 0; c < CACHED; ++c) {
            const int i = tid + c * nthr;
            zc[c] = i < V ? z[i] : -INFINITY;  // -inf: weight exp(-inf) = 0 and the lowest key
        }
    }
    for (int shift = 28; shift >= 0; shift -= 4) {
        float h[16], sure = 0.f;  // sure: members of every candidate of this sweep (their key is 16 steps or more above K)
#pragma unroll
        for (int j = 0; j < 16; ++j) h[j] = 0.f;
        auto take = [&](float zi) {
            const uint32_t k = float_key(zi);
            if (k >= K) {  // below K: excluded for good; the set still in play shrinks with every sweep
                const uint32_t q = (k - K) >> shift;
                const float e = expf(zi - m);
                if (q >= 16u) {
                    sure += e;
                } else {
#pragma unroll
                    for (int j = 0; j < 16; ++j) h[j] += (q == (uint32_t)j) ? e : 0.f;
                }
            }
        };
        if (cached) {
#pragma unroll
            for (int c = 0; c < CACHED; ++c) take(zc[c]);
        } else {
            for (int i0 = tid; i0 < V; i0 += nthr * 8) {
                float v[8];
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const int i = i0 + c * nthr;
                    v[c] = i < V ? z[i] : -INFINITY;
                }
#pragma unroll
                for (int c = 0; c < 8; ++c) take(v[c]);
            }
        }
        h[15] += sure;
#pragma unroll
        for (int j = 0; j < 16; ++j) {
            const float t = wave_sum(h[j]);
            if (lane == 0) bins[wave * 16 + j] = t;
        }
        __syncthreads();
        if (tid < 16) {  // bin totals over the waves, one bin per thread
            float t = 0.f;
            for (int w = 0; w < nwv; ++w) t += bins[w * 16 + tid];
            sc[8 + tid] = t;
        }
        __syncthreads();
        if (tid == 0) {
            if (shift == 28) {
                float all = 0.f;
                for (int j = 0; j < 16; ++j) all += sc[8 + j];
                sc[2] = top_p * all;
            }
            const float tgt = sc[2];
            float above = 0.f;  // mass of the members of candidate j = sum of bins j..15
            int pick = 0;
            float pick_mass = 0.f;
            for (int j = 15; j >= 0; --j) {
                above += sc[8 + j];
                if (j == 0 || above >= tgt) {
                    pick = j;
                    pick_mass = above;
                    break;
                }
            }
            sc[0] = __uint_as_float((uint32_t)pick);
            sc[1] = pick_mass;
        }
        __syncthreads();
        K += __float_as_uint(sc[0]) << shift;
        mass = sc[1];
        target = sc[2];
        __syncthreads();
    }
    (void)target;
    K_out = K;
    mass_out = mass;
}

// Inverse-CDF draw over the ids of a row, walked in increasing id: the first id whose running weight exceeds
// u * total.  weight(i) >= 0 is the (unnormalised) probability of id i, the same for every thread; `total` < 0
// means "add the weights up here" (wave sums in wave order).  Returns the token to every thread.
template <class W>
__device__ __forceinline__ int weighted_walk(W weight, int V, float total, float u, char* ws) {
    float* bins = (float*)ws;              // [16 waves][16]
    float* tmass = bins + 16 * 16;         // [1024]
    float* sc = tmass + 1024;              // scalars
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nthr = blockDim.x, nwv = nthr >> 6;
    __syncthreads();                       // the workspace may still be read by an earlier search or walk
    // ---- every thread owns a run of consecutive ids ----
    const int chunk = (V + nthr - 1) / nthr;
    const int i0 = min(tid * chunk, V), i1 = min(i0 + chunk, V);
    float mine = 0.f;
    for (int i = i0; i < i1; ++i) mine += weight(i);
    tmass[tid] = mine;
    const float wsum = wave_sum(mine);
    if (lane == 0) bins[wave] = wsum;
    __syncthreads();
    if (tid == 0) {
        float mass = total;
        if (mass < 0.f) {
            mass = 0.f;
            for (int w = 0; w < nwv; ++w) mass += bins[w];
        }
        const float t = u * mass;
        float run = 0.f;
        int w = 0;
        for (; w < nwv - 1; ++w) {  // the wave whose ids hold the target mass
            if (run + bins[w] > t) break;
            run += bins[w];
        }
        int th = w * 64;
        const int th_end = w * 64 + 63;
        for (; th < th_end; ++th) {
            if (run + tmass[th] > t) break;
            run += tmass[th];
        }
        sc[3] = __uint_as_float((uint32_t)th);
        sc[4] = run;
        sc[5] = t;
        sc[6] = __uint_as_float(0xFFFFFFFFu);
    }
    __syncthreads();
    const int owner = (int)__float_as_uint(sc[3]);
    if (tid == owner) {
        float run = sc[4];
        const float t = sc[5];
        int tok = -1, last = -1;
        for (int i = i0; i < i1; ++i) {
            const float wi = weight(i);
            if (wi > 0.f) {
                last = i;
                run += wi;
                if (run > t) {
                    tok = i;
                    break;
                }
            }
        }
        sc[6] = __uint_as_float((uint32_t)(tok >= 0 ? tok : last));
    }
    __syncthreads();
    int tok = (int)__float_as_uint(sc[6]);
    if (tok < 0) {  // rounding left the target beyond the last member: take the highest member id
        int best = -1;
        for (int i = tid; i < V; i += nthr)
            if (weight(i) > 0.f) best = max(best, i);
        for (int o = 32; o > 0; o >>= 1) best = max(best, __shfl_xor(best, o, 64));
        if (lane == 0) bins[wave] = __int_as_float(best);
        __syncthreads();
        for (int w = 0; w < nwv; ++w) tok = max(tok, __float_as_int(bins[w]));
    }
    return tok;
}

__device__ __forceinline__ int nucleus_draw(const float* __restrict__ z, int V, float m, float top_p, float u, char* ws) {
    uint32_t K;
    float mass;
    nucleus_search(z, V, m, top_p, ws, K, mass);
    return weighted_walk([&](int i) { const float zi = z[i]; return float_key(zi) >= K ? expf(zi - m) : 0.f; }, V, mass, u, ws);
}

// Merge of the LM-head partial statistics of the rows of a pass into (max, sum exp, argmax) per row, in LDS.  With at
// least as many waves as rows, every row gets nwv / T waves, each merging a contiguous share of the row's partials
// (lanes stride through it, eight loads in flight per lane), so that a single row with two thousand partials (250 112
// ids) costs one trip to memory instead of four; the shares are then joined in a fixed order.  More rows than waves: the
// rows are dealt to the waves.  A row's partials lie side by side: 16 bytes each, where one slot per row of every workgroup
// had a workgroup fetch a line of 128 bytes for each (1004 partials of one row: 2.6 us of the compute unit's bandwidth).
// `first` runs between the first requests and their use.  Ends with a barrier.
template <class First>
__device__ __forceinline__ void merge_partials(const FinishArgs& a, float* rm, float* rsum, int* ridx, First&& first) {
    __shared__ StatPart share[16];  // [row * wpr + share] (at most 16 waves)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nwv = blockDim.x >> 6;
    const int wpr = max(nwv / a.T, 1);              // waves per row
    const int per = (a.nparts + wpr - 1) / wpr;     // partials per share
    const int t0 = wave / wpr, c = wave - t0 * wpr;
    const int begin = min(c * per, a.nparts), end = min(begin + per, a.nparts);
    StatPart sp[8];
    load_parts(sp, a.part + (size_t)(a.row_off + min(t0, a.T - 1)) * a.part_ld, begin + lane, end);
    first();
    for (int t = t0; t < a.T; t += nwv) {           // (more than one turn only with one wave per row)
        const StatPart* row = a.part + (size_t)(a.row_off + t) * a.part_ld;
        Stat r = stat_neutral();
        for (int p0 = begin + lane;; p0 += 64 * 8) {
#pragma unroll
            for (int k = 0; k < 8; ++k)  // (pairwise, in the order of the partials)
                if (p0 + k * 64 < end) r = stat_merge(r, Stat{sp[k].m, sp[k].s, sp[k].idx});
            if (__builtin_amdgcn_readfirstlane(p0) + 64 * 8 >= end) break;
            load_parts(sp, row, p0 + 64 * 8, end);
        }
        if (t + nwv < a.T) load_parts(sp, row + (size_t)nwv * a.part_ld, begin + lane, end);
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) r = stat_merge(r, stat_shfl_xor(r, o));  // (an empty share stays neutral)
        if (lane == 0) {
            if (wpr == 1) {
                rm[t] = r.m;
                rsum[t] = r.s;
                ridx[t] = r.idx;
            } else {
                share[wave] = StatPart{r.m, r.s, r.idx, 0};
            }
        }
    }
    __syncthreads();
    if (wpr == 1) return;
    if (tid < a.T) {
        Stat r = stat_neutral();
        for (int c2 = 0; c2 < wpr; ++c2) {
            const StatPart q = share[tid * wpr + c2];
            r = stat_merge(r, Stat{q.m, q.s, q.idx});
        }
        rm[tid] = r.m;
        rsum[tid] = r.s;
        ridx[tid] = r.idx;
    }
    __syncthreads();
}

// draw(): the token of the sampling variant, drawn from what draw_bins_kernel and draw_split_kernel left; -1: none
struct NoDraw {
    __device__ __forceinline__ int operator()() const { return -1; }
};
template <bool SAMPLE, class Draw = NoDraw>
__device__ __forceinline__ void finish_body(const FinishArgs& a, char* lds, Draw&& draw = Draw()) {
    float* rm = (float*)lds;
    float* rsum = rm + kMaxRows;
    int* ridx = (int*)(rsum + kMaxRows);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int nthr = blockDim.x, nwv = nthr >> 6;
    // the control words the policy needs, requested now (nothing in this kernel writes them before they are used): their
    // trip from memory overlaps with the partials' instead of following it
    const Controls k(a);
    const int c_ylen = k.ylen, c_ds = k.ds;
    const float c_arb = k.arb;
    const bool failed = a.sync && a.sync[kPassSyncWords - 1] != 0u;
    float z_draft = 0.f;
    if (a.mode != 3)
        merge_partials(a, rm, rsum, ridx, [&] { if (a.mode == 1) z_draft = a.zt[a.row_off + min(lane, max(a.T - 2, 0))]; });
    // Sampling variant: the token that will be committed is drawn by the whole workgroup from the row the
    // policy selects (the last row of a step; row r of a review), at the position it will occupy.
    int drawn = draw();
    int r_given = -1;  // rejection-sampling acceptance: the index of the first refused draft (n: none), decided here
    if (SAMPLE && a.top_p > 0.f && a.mode <= 2) {
        int* sel = (int*)(lds + kFinishLds);  // [0] row, [1] position
        char* ws = lds + kFinishLds + 16;
        if (a.accept_mode == 1 && a.mode == 1) {
            // Review by the rejection rule (the acceptance of the speculative-decoding methods the paper compares
            // with, Section 4.2): draft x at position q, drawn from the small model's nucleus distribution p_S, is kept
            // iff u_acc[q] * p_S(x) < p_L(x); the first refused draft is replaced by a draw from the positive part of
            // p_L - p_S.  Every thread follows the same scalars; the searches and the walk use the whole workgroup.
            const int n = a.T - 1, V = a.vocab;
            int r = n;
            uint32_t KL = 0;
            float massL = 1.f;
            for (int i = 0; i < n; ++i) {
                const int pos = c_ds + i;
                const int x = a.y[pos];
                const float* zl = a.logits + (size_t)(a.row_off + i) * V;
                if (a.top_p < 1.f) nucleus_search(zl, V, rm[i], a.top_p, ws, KL, massL);
                else { KL = 0u; massL = rsum[i]; }
                const float zlx = zl[x];
                const float pl = float_key(zlx) >= KL ? expf(zlx - rm[i]) / massL : 0.f;
                const float4 sd = a.s_draw[pos];  // (max logit, threshold key, nucleus mass) of the small model's row
                const float zsx = a.s_ring[(size_t)i * V + x];
                const float ps = float_key(zsx) >= __float_as_uint(sd.y) ? expf(zsx - sd.x) / sd.z : 0.f;
                if (!(a.u_acc[pos] * ps < pl)) {
                    r = i;
                    break;
                }
            }
            r_given = r;
            const int pos = c_ds + r;
            const float* zl = a.logits + (size_t)(a.row_off + r) * V;
            if (r == n) {
                drawn = nucleus_draw(zl, V, rm[r], a.top_p, a.u[pos], ws);
            } else {  // (KL, massL) are those of row r, the last one searched
                const float4 sd = a.s_draw[pos];
                const float* zs = a.s_ring + (size_t)r * V;
                const uint32_t KS = __float_as_uint(sd.y);
                const float mL = rm[r], iL = 1.f / massL, mS = sd.x, iS = 1.f / sd.z;
                drawn = weighted_walk([&](int v) {
                    const float a_ = zl[v], b_ = zs[v];
                    const float pl = float_key(a_) >= KL ? expf(a_ - mL) * iL : 0.f;
                    const float ps = float_key(b_) >= KS ? expf(b_ - mS) * iS : 0.f;
                    return fmaxf(pl - ps, 0.f);
                }, V, -1.f, a.u[pos], ws);
            }
        } else {
            if (tid == 0) {
                int row = a.T - 1, pos = c_ylen;
                if (a.mode == 1) {
                    const int n = a.T - 1;
                    const float alpha = c_arb;
                    row = n;
                    for (int i = 0; i < n; ++i)
                        if ((rm[i] + logf(rsum[i])) - a.zt[a.row_off + i] > alpha) {
                            row = i;
                            break;
                        }
                    pos = c_ds + row;
                }
                sel[0] = row;
                sel[1] = pos;
            }
            __syncthreads();
            const int row = sel[0], pos = sel[1];
            const float* zr = a.logits + (size_t)(a.row_off + row) * a.vocab;
            if (a.accept_mode == 1 && a.mode == 0) {
                // the small model's step under the rejection rule: the review will need the distribution this token was
                // drawn from - keep the row's logits in the slot of its draft index and its (max, threshold, mass)
                uint32_t K;
                float mass;
                nucleus_search(zr, a.vocab, rm[row], a.top_p, ws, K, mass);
                drawn = weighted_walk([&](int i) { const float zi = zr[i]; return float_key(zi) >= K ? expf(zi - rm[row]) : 0.f; },
                                      a.vocab, mass, a.u[pos], ws);
                const int slot = min(max(c_ylen - c_ds, 0), kMaxRows - 1);
                float* dst = a.s_ring + (size_t)slot * a.vocab;
                for (int i = tid; i < a.vocab; i += nthr) dst[i] = zr[i];
                if (tid == 0) a.s_draw[pos] = make_float4(rm[row], __uint_as_float(K), mass, 0.f);
            } else {
                drawn = nucleus_draw(zr, a.vocab, rm[row], a.top_p, a.u[pos], ws);
            }
        }
    }
    // From here on wave 0 alone, lane t with row t: no barrier, no trip through LDS.
    if (tid >= 64) return;
    const int t = min(lane, max(a.T - 1, 0));
    const bool rows = a.mode != 3;
    commit(a, k, failed, rows ? ridx[t] : 0, rows ? rm[t] : 0.f, rows ? rsum[t] : 0.f, z_draft, drawn, r_given);
}

__global__ __launch_bounds__(256) void finish_kernel(const FinishArgs a) {
    __shared__ __attribute__((aligned(16))) char lds[kFinishLds];
    finish_body<false>(a, lds);
}

// Reviews of several rows: sixteen waves, so that the rows' partial statistics are merged side by side (a wave takes
// rows w, w + 16, ...: one trip to memory per row it has).
__global__ __launch_bounds__(1024) void finish_wide_kernel(const FinishArgs a) {
    __shared__ __attribute__((aligned(16))) char lds[kFinishLds];
    finish_body<false>(a, lds);
}

__global__ __launch_bounds__(1024) void finish_sample_kernel(const FinishArgs a) {
    __shared__ __attribute__((aligned(16))) char lds[kFinishLds + 16 + kDrawLds];
    finish_body<true>(a, lds);
}


// =====================================================================================
// Nucleus draw spread over the chip (sampling variant with the threshold rule of the review).
//
// The single-workgroup draw above sweeps a row of logits eight times on one compute unit (80 us at 32 128 ids, 650 us
// at 250 112).  Here the row is cut into slices (draw_per), one workgroup each, and every probability mass
// is an INTEGER: exp(z - max) in units of 2^-40, truncated.  Integer sums do not depend on the order of their terms,
// so the result is the same on every run; and the nucleus mass found by the threshold search equals the sum of the
// members' masses of the walk exactly, so the walk always ends inside the nucleus.
//
//   draw_bins_kernel   (slices)       merges the LM-head partials and applies the rollback test to find the row the token
//                      comes from (every workgroup for itself; the first leaves row, position, max and the merged statistics),
//                      then its slice's mass per bin of max - z
//   draw_split_kernel  (slices)       the bin the threshold lies in, from all slices' bins; its slice's mass in the bins
//                      before it and in the parts of this bin, and a list of the ids in it in the order of their parts
//   draw_pick_kernel   (1 workgroup)  the threshold key: where more ids are listed than there are threads those in the threshold's part
//                      of the bin only, then a radix search of the bits in which the candidates' keys differ; floor(u * mass) -> slice ->
//                      id by two integer prefix sums; then the policy and the commit of finish_body with that token
//
// Bound by launches and trips to memory.  A search by the four bytes of the key, a sweep over the row each, with a launch in front
// to merge and one behind for the members' masses, were seven launches: 4.7 + 4 x 4.6 + 4.7 + 7.5 us at 32 128 ids, 4.8 + 4 x 6.4 + 4.7
// + 7.9 at 250 112; these are 4.9 + 4.9 + 6.8 and 6.0 + 8.3 + 9.5 us for a peaked row and one row of statistics, 8.5 + 8.3 + 11.6 for the eleven of a review
// (every slice's workgroup merges all of them; the merge alone took 8.3 before), and 4.5 + 6.1 + 10.8 and 6.1 + 10.7 + 16.3 us where all logits lie within 1e-3 of each other.  A
// step of one layer, wall clock, seven launches / three: 32 128 ids peaked 64.5 / 52.8 us, flat 65.9 / 57.8; 250 112 ids 95.7 / 86.0 and 102.6 / 94.6.
// Bins by distance from the maximum divide what has any mass evenly, where a key's top byte is a sign and most of an exponent; they are as wide as
// the row asks for (draw_map), because with one width for all rows a flat row lies in a few of them: a list of all ids, swept by one
// workgroup, 288 and 1829 us a step.  What is left of that: many ids with two keys in one part, as a row of zeros of both signs (129 and 613 us).
// Workgroups of 1024 threads lost 3 us, slices of 4096 ids at 256 threads 2.
// =====================================================================================
typedef unsigned long long u64;

__device__ __forceinline__ u64 mass_units(float z, float m) { return (u64)(expf(z - m) * 1099511627776.f); }  // 2^40

// How a row's bins lie: the near ones up to twice ln(vocab / sum of exp(z - max)), which the mean distance of the row's mass from its
// maximum never exceeds, the far ones up to where there is no mass.
__device__ __forceinline__ DrawMap draw_map(float sum, int vocab) {
    DrawMap w;
    w.knee = fminf(fmaxf(1.3862944f * __builtin_amdgcn_logf((float)vocab * __builtin_amdgcn_rcpf(sum)), 0x1p-20f), 28.f);  // (2^-40 of the largest mass is 27.7 below it)
    w.near = (float)kDrawNear * __builtin_amdgcn_rcpf(w.knee);
    w.far = (float)(kDrawBins - kDrawNear) * __builtin_amdgcn_rcpf(fmaxf(28.f - w.knee, 1.f));
    return w;
}
// Place of an id among the bins: not decreasing where z falls (rounding keeps the order), so that an id in an earlier bin, or an
// earlier part of the same bin, has a larger key.  Ids without mass may be in any bin (NaN: the first).
__device__ __forceinline__ float draw_place(float z, float m, const DrawMap& w) {
    const float d = fmaxf(m - z, 0.f);
    return __builtin_fmaf(fmaxf(d - w.knee, 0.f), w.far, fminf(d * w.near, (float)kDrawNear));  // (the same in every kernel)
}
__device__ __forceinline__ int draw_bin(float place) { return (int)fminf(place, (float)(kDrawBins - 1)); }
__device__ __forceinline__ int draw_part(float place, int bin) { return draw_bin((place - (float)bin) * (float)kDrawBins); }

// Sum over the threads up to and with this one, in `all` over all: lane shifts inside a wavefront, the waves' totals through LDS
// (buf: a word per wave; it may be used again behind the caller's next barrier).
template <int CTRL, int ROWS>
__device__ __forceinline__ u64 dpp_add(u64 v) {
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)v, CTRL, ROWS, 0xF, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp(0, (int)(unsigned)(v >> 32), CTRL, ROWS, 0xF, false);
    return v + ((u64)hi << 32 | lo);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned dpp_add(unsigned v) {
    return v + (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
template <class T>
__device__ __forceinline__ T wave_prefix(T v) {
    v = dpp_add<0x111, 0xF>(v);  // row_shr:1, 2, 4, 8
    v = dpp_add<0x112, 0xF>(v);
    v = dpp_add<0x114, 0xF>(v);
    v = dpp_add<0x118, 0xF>(v);
    v = dpp_add<0x142, 0xA>(v);  // row_bcast:15 to rows 1 and 3
    return dpp_add<0x143, 0xC>(v);  // row_bcast:31 to rows 2 and 3
}
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t dpp_umax(uint32_t v) {
    return max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false));
}
__device__ __forceinline__ uint32_t wave_umax(uint32_t v) {  // (as wave_prefix: the last lane has it)
    v = dpp_umax<0x111, 0xF>(v);
    v = dpp_umax<0x112, 0xF>(v);
    v = dpp_umax<0x114, 0xF>(v);
    v = dpp_umax<0x118, 0xF>(v);
    v = dpp_umax<0x142, 0xA>(v);
    return (uint32_t)__builtin_amdgcn_readlane((int)dpp_umax<0x143, 0xC>(v), 63);
}
__device__ __forceinline__ u64 prefix_sum(u64 v, u64* buf, u64& all) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    v = wave_prefix(v);
    if (lane == 63) buf[wave] = v;
    __syncthreads();
    u64 before = 0;
    all = 0;
#pragma unroll
    for (int w = 0; w < kDrawThreads / 64; ++w) {
        const u64 t = buf[w];
        all += t;
        before += w < wave ? t : 0ull;
    }
    return v + before;
}

// This workgroup's slice of the row: ids first + c * kDrawThreads.  PER: of a thread (draw_per)
template <int PER>
__device__ __forceinline__ void load_slice(float (&z)[PER], const FinishArgs& a, int row, int first) {
    const float* zr = a.logits + (size_t)(a.row_off + row) * a.vocab;
#pragma unroll
    for (int c = 0; c < PER; ++c) z[c] = zr[min(first + c * kDrawThreads, a.vocab - 1)];
}

template <int PER>
__global__ __launch_bounds__(kDrawThreads) void draw_bins_kernel(const FinishArgs a) {
    __shared__ __attribute__((aligned(16))) char lds[kFinishLds];
    __shared__ u64 bins[kDrawBins];
    float* rm = (float*)lds;
    float* rsum = rm + kMaxRows;
    int* ridx = (int*)(rsum + kMaxRows);
    const int tid = threadIdx.x, lane = tid & 63;
    const Ctl* c = a.ctl;
    const int c_ylen = c->y_len, c_ds = c->draft_start, n = a.T - 1;
    const float c_arb = c->alpha_rb;
    DrawWs* ws = a.dws;
    const int first = (int)blockIdx.x * (PER * kDrawThreads) + tid;
    float z[PER], z_draft = 0.f;
    load_slice(z, a, n, first);  // (the row unless a draft is refused)
    bins[tid] = 0ull;
    merge_partials(a, rm, rsum, ridx, [&] { if (a.mode == 1) z_draft = a.zt[a.row_off + min(lane, max(n - 1, 0))]; });
    int row = n, pos = c_ylen;
    if (a.mode == 1) {  // review: the first draft whose cross-entropy exceeds the threshold (Section 3.4), else the row after the last
        const int t = min(lane, n);
        const u64 over = __builtin_amdgcn_ballot_w64(lane < n && (rm[t] + logf(rsum[t])) - z_draft > c_arb);
        row = over ? (int)__builtin_ctzll(over) : n;
        pos = c_ds + row;
        if (row != n) load_slice(z, a, row, first);
    }
    const float m = rm[row];
    const DrawMap map = draw_map(rsum[row], a.vocab);
#pragma unroll
    for (int k = 0; k < PER; ++k)
        if (first + k * kDrawThreads < a.vocab) {
            const u64 e = mass_units(z[k], m);
            if (e) atomicAdd(&bins[draw_bin(draw_place(z[k], m, map))], e);
        }
    __syncthreads();
    ws->bins(blockIdx.x)[tid] = bins[tid];
    if (blockIdx.x == 0) {
        if (tid < a.T) {
            StatPart sp;
            sp.m = rm[tid]; sp.s = rsum[tid]; sp.idx = ridx[tid]; sp.pad = 0;
            ws->merged[a.row_off + tid] = sp;
        }
        if (tid == 0) {
            ws->row = row;
            ws->pos = pos;
            ws->m = m;
            ws->map = map;
            ws->n = 0u;
        }
    }
}

template <int PER>
__global__ __launch_bounds__(kDrawThreads) void draw_split_kernel(const FinishArgs a) {
    __shared__ u64 parts[kDrawBins], buf[3][kDrawThreads / 64], found[2];
    __shared__ unsigned count[kDrawBins], base;
    __shared__ uint4 range[kDrawThreads / 64];
    __shared__ int at_bin;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nslices = (int)gridDim.x;
    DrawWs* ws = a.dws;
    const int first = (int)blockIdx.x * (PER * kDrawThreads) + tid;
    const float m = ws->m;
    const DrawMap map = ws->map;
    const int pos = ws->pos;
    float z[PER];
    load_slice(z, a, ws->row, first);
    const float u = a.u[pos];
    u64 mine = 0, total;  // of bin tid
    for (int s = 0; s < nslices; s += 8) {
        u64 v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = ws->bins(min(s + k, nslices - 1))[tid];
#pragma unroll
        for (int k = 0; k < 8; ++k) mine += s + k < nslices ? v[k] : 0ull;
    }
    parts[tid] = 0ull;
    count[tid] = 0u;
    if (tid == 0) at_bin = kDrawBins;  // (no mass, or a target above all of it: every id is a member)
    const u64 upto = prefix_sum(mine, buf[0], total);
    const u64 target = (u64)ceil((double)a.top_p * (double)total);
    if (upto >= target && upto - mine < target) {  // one thread at most
        at_bin = tid;
        found[0] = upto - mine;
        found[1] = upto;
    }
    __syncthreads();
    const int b = at_bin;
    u64 mass = 0;
    int part[PER];       // of the id if it lies in the bin, else -1
    unsigned rank[PER];  // among the slice's ids in that part
    uint32_t least = 0u, largest = 0u;  // key of this thread's (the least: its complement)
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        part[k] = -1;
        if (first + k * kDrawThreads < a.vocab) {
            const float place = draw_place(z[k], m, map);
            const int bin = draw_bin(place);
            if (bin <= b) {
                const u64 e = mass_units(z[k], m);
                mass += bin < b ? e : 0ull;
                if (bin == b && e != 0ull) {
                    part[k] = draw_part(place, b);
                    atomicAdd(&parts[part[k]], e);
                    rank[k] = atomicAdd(&count[part[k]], 1u);
                    least = max(least, ~float_key(z[k]));
                    largest = max(largest, float_key(z[k]));
                }
            }
        }
    }
    __syncthreads();  // (`count` and `parts` are complete)
    const unsigned own = count[tid];
    u64 in_parts = wave_prefix(parts[tid]);
    mass = wave_prefix(mass);
    unsigned before = wave_prefix(own);
    least = wave_umax(least);
    largest = wave_umax(largest);
    if (lane == 63) {
        buf[1][wave] = in_parts;
        buf[2][wave] = mass;
        range[wave] = make_uint4(before, least, largest, 0u);
    }
    before -= own;
    __syncthreads();
    u64 slice = 0;
    unsigned listed = 0;
#pragma unroll
    for (int w = 0; w < kDrawThreads / 64; ++w) {
        const uint4 r = range[w];
        in_parts += w < wave ? buf[1][w] : 0ull;
        before += w < wave ? r.x : 0u;
        slice += buf[2][w];
        listed += r.x;
        least = max(least, r.y);
        largest = max(largest, r.z);
    }
    count[tid] = before;
    ws->parts(nslices, blockIdx.x)[tid] = in_parts;
    unsigned* starts = ws->starts(nslices, blockIdx.x);
    if (tid == 0) {
        base = listed ? atomicAdd(&ws->n, listed) : 0u;
        starts[kDrawBins] = base + listed;
        ws->slice[blockIdx.x] = slice;
        ws->range[blockIdx.x] = make_uint2(least, largest);
        if (blockIdx.x == 0) {
            ws->u = u;
            ws->bin = b;
            ws->target = target;
            ws->above = b == kDrawBins ? total : found[0];
            ws->upto = b == kDrawBins ? total : found[1];
        }
    }
    __syncthreads();
    const unsigned at = base;
    starts[tid] = at + before;
    uint2* list = ws->list(nslices) + at;
#pragma unroll
    for (int k = 0; k < PER; ++k)
        if (part[k] >= 0) list[count[part[k]] + rank[k]] = make_uint2(__float_as_uint(z[k]), (unsigned)(first + k * kDrawThreads));
}

template <int PER>
__global__ __launch_bounds__(kDrawThreads) void draw_pick_kernel(const FinishArgs a, const int nslices) {
    __shared__ __attribute__((aligned(16))) char lds[kFinishLds];
    __shared__ u64 bins[kDrawBins], slice[kDrawMaxSlices], buf[2][kDrawThreads / 64], found[2];
    constexpr int IDS = PER * kDrawThreads;
    __shared__ float zs[IDS + kDrawThreads];  // (a word between a thread's ids and the next one's)
    __shared__ uint2 range[kDrawThreads / 64];
    __shared__ uint2 cand[kDrawThreads];  // where the list has candidate tid, or (more of them than threads) those of slice tid
    __shared__ int at_bin, token;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    // (requested ahead of the policy's words and the statistics: one trip for all of it)
    const DrawWs* ws = a.dws;
    const int row = ws->row, n = (int)ws->n;
    const float m = ws->m, u = ws->u;
    const u64 target = ws->target;
    u64 above = ws->above, upto = ws->upto;
    const uint2* list = ws->list(nslices);
    uint2 own = list[min(tid, a.vocab - 1)];  // this thread's candidate
    const u64 of_slice = ws->slice[tid];
    finish_body<false>(a, lds, [&]() -> int {
        slice[tid] = tid < nslices ? of_slice : 0ull;
        if (tid == 0) token = ((const int*)lds)[2 * kMaxRows + row];  // (argmax; stays only where no id has any mass)
        int many = n;  // candidates
        u64 in_part = 0;  // (more ids listed than there are threads) mass of slice tid in the candidates' part of the bin
        uint32_t least = 0u, largest = 0u;  // candidates' keys (the least: its complement), or those of all ids in the bin
        // (wavefronts with candidates as a whole, surplus lanes with `there` false)
        auto each = [&](auto&& f) {
            if (many <= kDrawThreads) {
                if (wave * 64 < many) f(own, tid < many);
                return;
            }
            for (int s = wave; s < nslices; s += kDrawThreads / 64) {  // (so many ids so close together)
                const unsigned from = cand[s].x, to = cand[s].y;
                for (unsigned i = from & ~1u; i < to; i += 64 * 2 * 8) {
                    uint4 e[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) e[k] = *(const uint4*)(list + min(i + (k * 64 + lane) * 2, (unsigned)(a.vocab - 1) & ~1u));
#pragma unroll
                    for (int k = 0; k < 8; ++k) {
                        const unsigned j = i + (k * 64 + lane) * 2;
                        if (i + k * 128 >= to) break;
                        f(make_uint2(e[k].x, e[k].y), j >= from && j < to);
                        f(make_uint2(e[k].z, e[k].w), j + 1 < to);
                    }
                }
            }
        };
        if (n > kDrawThreads) {  // the part of the bin that the threshold lies in: its ids are the candidates
            u64 sum = 0, all;    // of the parts up to and with part tid
            for (int s = 0; s < nslices; s += 8) {
                u64 v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = ws->parts(nslices, min(s + k, nslices - 1))[tid];
#pragma unroll
                for (int k = 0; k < 8; ++k) sum += s + k < nslices ? v[k] : 0ull;
            }
            bins[tid] = sum;
            if (tid == 0) {
                at_bin = 0;
                found[0] = above;
                found[1] = upto;
            }
            __syncthreads();
            const u64 upto_part = above + sum, upto_last = above + (tid ? bins[tid - 1] : 0ull);
            if (upto_part >= target && upto_last < target) {  // exactly one thread
                at_bin = tid;
                found[0] = upto_last;
                found[1] = upto_part;
            }
            __syncthreads();
            const int part = at_bin;
            above = found[0];
            upto = found[1];
            unsigned from = 0u, to = 0u;
            if (tid < nslices) {  // members in the parts before it, to their slices
                const u64* p = ws->parts(nslices, tid);
                const unsigned* st = ws->starts(nslices, tid);
                const u64 before = part ? p[part - 1] : 0ull;
                in_part = p[part] - before;
                slice[tid] += before;
                from = st[part];
                to = st[part + 1];
            }
            const unsigned first = (unsigned)prefix_sum(to - from, buf[0], all) - (to - from);
            many = (int)all;
            if (many <= kDrawThreads) {
                for (unsigned i = from; i < to; ++i) cand[first + i - from].x = i;
                __syncthreads();
                own = list[min(cand[min(tid, max(many - 1, 0))].x, (unsigned)a.vocab - 1u)];
            } else {
                cand[tid] = make_uint2(from, to);
                const uint2 r = ws->range[min(tid, nslices - 1)];
                least = r.x;
                largest = r.y;
                __syncthreads();
            }
        }
        uint32_t K = 0u;
        if (n > 0) {
            if (many <= kDrawThreads && tid < many) {
                least = ~float_key(__uint_as_float(own.x));
                largest = float_key(__uint_as_float(own.x));
            }
            least = wave_umax(least);
            largest = wave_umax(largest);
            if (lane == 0) range[wave] = make_uint2(least, largest);
            __syncthreads();
            for (const uint2& r : range) {
                least = max(least, r.x);
                largest = max(largest, r.y);
            }
            const uint32_t kmin = ~least, kmax = largest;
            // The largest key whose members' mass reaches the target, as its distance from the least: eight bits at a time
            uint32_t D = 0u;
            const int bits = kmax == kmin ? 0 : 32 - __builtin_clz(kmax - kmin);
            for (int shift = (bits + 7) / 8 * 8 - 8; shift >= 0; shift -= 8) {
                bins[tid] = 0ull;
                __syncthreads();
                each([&](const uint2& e, bool there) {
                    const float z = __uint_as_float(e.x);
                    const uint32_t k = float_key(z) - kmin;
                    if (there && (shift == 24 || ((k ^ D) >> (shift + 8)) == 0u)) atomicAdd(&bins[(k >> shift) & 255u], mass_units(z, m));
                });
                __syncthreads();
                u64 all;
                const u64 mine = bins[kDrawBins - 1 - tid];
                const u64 s = above + prefix_sum(mine, buf[shift >> 3 & 1], all);
                if (s >= target && s - mine < target) {  // exactly one thread
                    at_bin = kDrawBins - 1 - tid;
                    found[0] = s - mine;
                    found[1] = s;
                }
                __syncthreads();
                D |= (uint32_t)at_bin << shift;
                above = found[0];
                upto = found[1];
            }
            K = kmin + D;
            // the candidates that are members to their slices (a slice's ids lie together: a sum over the wavefront for each slice in it)
            if (many > kDrawThreads && bits == 0) slice[tid] += in_part;  // (all of them are)
            else each([&](const uint2& e, bool there) {
                const float z = __uint_as_float(e.x);
                const bool member = there && float_key(z) >= K;
                const u64 units = member ? mass_units(z, m) : 0ull;
                for (u64 left = __builtin_amdgcn_ballot_w64(member); left != 0ull;) {
                    const unsigned s = __builtin_amdgcn_readlane(e.y, (int)__builtin_ctzll(left)) / IDS;
                    const bool here = member && e.y / IDS == s;
                    const u64 sum = wave_prefix(here ? units : 0ull);
                    if (lane == 63) atomicAdd(&slice[s], sum);
                    left &= ~__builtin_amdgcn_ballot_w64(here);
                }
            });
        }
        __syncthreads();
        // target of the walk: the first member (ids increasing) whose running mass exceeds u * mass, i.e. exceeds t = floor(u * mass)
        const u64 t = (u64)((double)u * (double)upto);
        if (tid == 0) {
            at_bin = 0;
            found[0] = 0;
        }
        u64 all;
        {
            const u64 mine = slice[tid];
            const u64 s = prefix_sum(mine, buf[0], all);
            if (s - mine <= t && t < s) {  // exactly one thread (the masses add up to `upto` > t exactly)
                at_bin = tid;
                found[0] = s - mine;
            }
        }
        __syncthreads();
        const u64 rem = t - found[0];  // mass to pass inside the slice, whose ids j * PER .. are thread j's
        const int base = at_bin * IDS, i0 = base + tid * PER;
        float z[PER];
        load_slice(z, a, row, base + tid);
#pragma unroll
        for (int c = 0; c < PER; ++c) {
            const int i = tid + c * kDrawThreads;
            zs[i + i / PER] = z[c];
        }
        __syncthreads();
        u64 e[PER], tot = 0;
#pragma unroll
        for (int c = 0; c < PER; ++c) z[c] = zs[tid * (PER + 1) + c];
#pragma unroll
        for (int c = 0; c < PER; ++c) {
            e[c] = (i0 + c < a.vocab && float_key(z[c]) >= K) ? mass_units(z[c], m) : 0ull;
            tot += e[c];
        }
        const u64 s = prefix_sum(tot, buf[1], all);
        if (s - tot <= rem && rem < s) {
            u64 run = s - tot;
            int c = -1;
#pragma unroll
            for (int j = 0; j < PER; ++j) {
                run += e[j];
                c = c < 0 && run > rem ? j : c;
            }
            token = i0 + c;
        }
        __syncthreads();
        return token;
    });
}

// What the host changes between passes.  As a kernel's arguments it costs its enqueueing, about 3 us and no wait; as a copy
// (pageable or pinned) with the synchronization that keeps its source valid it cost 15 us, and 22 us more per piece of tokens.
// The tokens come over the host link: one per thread, so that all of them cost one trip.
__global__ __launch_bounds__(256) void ctl_kernel(const CtlArgs a) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < a.n) a.dst[i] = a.src[i];
    else if (i < a.n + a.n2) a.dst2[i - a.n] = a.src2[i - a.n];
    if (blockIdx.x == 0) {
        int* c = (int*)a.ctl;
        constexpr int words = sizeof(Ctl) / 4;
        static_assert(offsetof(Ctl, alpha_rb) == 28 && words <= 256, "one word per thread");
        if (threadIdx.x < words && (!a.thresholds_only || threadIdx.x == 6 || threadIdx.x == 7))
            c[threadIdx.x] = threadIdx.x < 8 ? a.head[threadIdx.x & 7] : threadIdx.x == words - 1 ? a.seq : 0;
    }
}

hipError_t launch_ctl(const CtlArgs& a, hipStream_t st) {
    if (!a.ctl || a.n < 0 || a.n2 < 0) return hipErrorInvalidValue;
    hipLaunchKernelGGL(ctl_kernel, dim3((a.n + a.n2 + 255) / 256 + (a.n + a.n2 == 0)), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_finish_draw(const FinishArgs& a, hipStream_t st) {
    if (!(a.top_p > 0.f) || a.mode > 2 || a.accept_mode != 0 || !a.logits || !a.u || !a.dws || a.vocab < 1 || a.T < 1 || a.T > kMaxRows)
        return hipErrorInvalidValue;
    const int ns = draw_slices(a.vocab);
    if (ns > kDrawMaxSlices) return hipErrorInvalidValue;
    FinishArgs f = a;  // the commit merges one "partial" per row: the statistics draw_bins_kernel left
    f.part = a.dws->merged;  // (address arithmetic only: dws is a device pointer)
    f.nparts = f.part_ld = 1;
    if (draw_per(a.vocab) == kDrawFew) {
        hipLaunchKernelGGL(draw_bins_kernel<kDrawFew>, dim3(ns), dim3(kDrawThreads), 0, st, a);
        hipLaunchKernelGGL(draw_split_kernel<kDrawFew>, dim3(ns), dim3(kDrawThreads), 0, st, a);
        hipLaunchKernelGGL(draw_pick_kernel<kDrawFew>, dim3(1), dim3(kDrawThreads), 0, st, f, ns);
    } else {
        hipLaunchKernelGGL(draw_bins_kernel<kDrawMany>, dim3(ns), dim3(kDrawThreads), 0, st, a);
        hipLaunchKernelGGL(draw_split_kernel<kDrawMany>, dim3(ns), dim3(kDrawThreads), 0, st, a);
        hipLaunchKernelGGL(draw_pick_kernel<kDrawMany>, dim3(1), dim3(kDrawThreads), 0, st, f, ns);
    }
    return hipGetLastError();
}

hipError_t launch_finish(const FinishArgs& a, hipStream_t st) {
    if (a.top_p > 0.f && a.mode <= 2) {
        if (!a.logits || !a.u || a.vocab < 1) return hipErrorInvalidValue;
        if (a.accept_mode == 1 && (!a.u_acc || !a.s_ring || !a.s_draw)) return hipErrorInvalidValue;
        hipLaunchKernelGGL(finish_sample_kernel, dim3(1), dim3(1024), 0, st, a);
        return hipGetLastError();
    }
    if (a.mode != 3 && (a.T > 4 || a.nparts > 1024)) hipLaunchKernelGGL(finish_wide_kernel, dim3(1), dim3(1024), 0, st, a);
    else hipLaunchKernelGGL(finish_kernel, dim3(1), dim3(256), 0, st, a);
    return hipGetLastError();
}

}  // namespace bild
