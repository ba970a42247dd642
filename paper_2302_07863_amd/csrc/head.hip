// LM head over 1 .. 32 rows: the vocabulary matrix streamed once, softmax statistics of every row.
//
// Bound: the matrix' way from memory.  A workgroup per compute unit at most stays for the whole sweep: it norms and splits the rows once,
// each of its eight waves the inputs it multiplies, and keeps them in operand registers (up to eight rows one operand holds the high
// parts in its columns 0 .. 7 and the low parts in 8 .. 15); then it takes one group of feature tiles after the other, two batches
// of weights always on their way, also while the waves' sums of a group are joined through LDS.  Statistics run on in the waves that
// own a row tile, so that a row has one partial per workgroup, and where the caller wants the row's result the last workgroup to
// arrive joins them, which spares a launch.
//
// us per launch, floor at 6.1 TB/s / workgroups of eight feature tiles that each stage all rows / now: 32 128 x 512, 1 and 32 rows 5.4 /
// 10.3, 16.6 / 11.3, 13.9; 250 112 x 512 42 / 52.8, 80.3 / 43.9, 45.3; 250 112 x 1024, 1, 21, 32 rows 84 / 109, 133, 141 / 91, 93, 95;
// 131 072 x 2048, 1, 21 rows 88 / 103, 136 / 94, 103.  bild_head_stats where this kernel joins and the host polls, one row: 512 x 16 000 ids 21.7 -> 16.6,
// 2048 x 32 000 40.3 -> 32.0 (the short workgroups and the merge with the host polling 17.1, 35.7: where they are taken, see head_stats.hip).  Sums against 64 bits as before: rms of lse 4.1e-7, 6.3e-7, 6.4e-7 at 1000,
// 32 128 and 250 112 ids (4.0e-7, 6.4e-7, 6.3e-7).
//
// fp32 models (F32): tiles of sixteen inputs, rows and weights as they are, four fp32 products a tile of sixteen rows, which take a compute unit
// 32 bytes a clock of weights with up to sixteen rows and 16 with more (19 and 10 TB/s over the chip): the matrix' way from memory still.  A row
// of 2048 and 4096 inputs takes 64 and 128 registers; 17 rows and more of the latter do not fit, and up to sixteen of them spill 40 registers (164 bytes a
// lane): 4096 x 50 000 takes 173 us, 134 at a large copy's rate (taken only where the short workgroups are slower still, head_route).  50 000 ids, 1, 16, 32 rows, short workgroups / now (floor
// 17, 34, 67 us): 512 wide 34.5, 38.7, 50.1 / 32.0, 34.1, 42.0; 1024 53.6, 58.4, 98.7 / 46.5, 51.2, 59.7; 2048 98, 130, 191 / 86, 89, 106 (more: head_route).
#include "head.h"

#include <algorithm>

#include "last_in.h"

namespace bild {

constexpr int kHeadWaves = 8;

// KP: input tiles per wave at most; RW feature tiles per group; U input tiles per batch
template <int KP, int RW, int U, int NT, bool PACK, bool F32 = false>
__global__ __launch_bounds__(64 * kHeadWaves, 1) void head_kernel(const float* __restrict__ h_x, const void* __restrict__ h_w, const float* __restrict__ h_gain, const int h_ldx,
                                                                 const int h_tn, const int h_tk, const int h_T, const HeadArgs a0) {
    constexpr int P = PACK || F32 ? 1 : 2, BATCHES = KP / U, UNITS = RW * NT;
    constexpr int KT = F32 ? 16 : 32, Q = F32 ? 1 : 2;  // inputs of a tile; a lane's, in fours
    static_assert(KP % U == 0 && UNITS <= kHeadWaves && kHeadWaves % NT == 0, "whole batches; a wave keeps one row tile's statistics");
    extern __shared__ __attribute__((aligned(16))) char smem[];
    f32x4* red = (f32x4*)smem;                                    // [wave][RW * NT][64]
    float* rsum = (float*)(smem + kHeadWaves * UNITS * 1024);     // [wave][32]
    StatPart* wstat = (StatPart*)(rsum + kHeadWaves * 32);        // [wave][16]
    unsigned* share = (unsigned*)(wstat + kHeadWaves * 16);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int tok = lane & 15, g = lane >> 4, T = h_T;
    const int tk = h_tk, tn = h_tn, groups = (tn + RW - 1) / RW, per = (tk + kHeadWaves - 1) / kHeadWaves;
    const int k0 = min(wave * per, tk - 1), n = max(0, min(per, tk - wave * per));

    // ---- rows and gain requested (JC input tiles at a time, what the registers hold), behind them the first weights ----
    constexpr int JC = KP * NT > 8 ? 4 : KP;
    float4 xv[JC][NT][Q], gv[JC][Q];
    const __amdgpu_buffer_rsrc_t xr = make_rsrc(h_x, 0xFFFFFFFFu), gr = make_rsrc(h_gain, 0xFFFFFFFFu);
    auto fetch = [&](int j0) {
#pragma unroll
        for (int j = 0; j < JC; ++j) {
            const int kt = k0 + min(j0 + j, max(n - 1, 0));
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                const int row = min(PACK ? tok & 7 : i * 16 + tok, T - 1);
#pragma unroll
                for (int p = 0; p < Q; ++p) xv[j][i][p] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(xr, (row * h_ldx + g * 4 * Q) * 4, kt * (KT * 4) + p * 16, 0));
            }
#pragma unroll
            for (int p = 0; p < Q; ++p) gv[j][p] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(gr, g * 16 * Q, kt * (KT * 4) + p * 16, 0));
        }
    };
    fetch(0);
    uint4 W0[U][RW], W1[U][RW];
    auto request = [&](uint4 (&W)[U][RW], int grp, int batch) {
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            const __amdgpu_buffer_rsrc_t w = make_rsrc((const char*)h_w + (size_t)min(grp * RW + r, tn - 1) * tk * kTileBytes, 0xFFFFFFFFu);
#pragma unroll
            for (int u = 0; u < U; ++u) W[u][r] = buf_load(w, (unsigned)lane * 16u, (k0 + min(batch * U + u, max(n - 1, 0))) * kTileBytes);
        }
    };
    int grp = (int)blockIdx.x;
    const int step = (int)gridDim.x;
    // batch b of the sweep, counted over the groups
    auto ask = [&](uint4 (&W)[U][RW], int gg, int b) {  // (b: within group gg and the one after it)
        const int at = b < BATCHES ? gg : gg + step;
        if (at < groups) request(W, at, b < BATCHES ? b : b - BATCHES);
    };
    ask(W0, grp, 0);
    ask(W1, grp, 1);
    const HeadArgs a = a0;
    const int pos0 = (a.pos_ptr ? *a.pos_ptr : 0) + a.pos_add;
    int target = -1;
    {
        const int t = (wave % NT) * 16 + tok, ti = pos0 + t + 1;
        if (t < T && ti < *a.ylen_ptr) target = a.y[ti];
    }
    // ---- operands ----
    uint4 X[KP][NT][P];
    {
        float ss[NT];
#pragma unroll
        for (int i = 0; i < NT; ++i) ss[i] = 0.f;
#pragma unroll
        for (int j = 0; j < KP; ++j) {
            const int c = j % JC;
            if (j > 0 && c == 0) fetch(j);
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                constexpr int Z = Q - 1;
                float v[8] = {xv[c][i][0].x, xv[c][i][0].y, xv[c][i][0].z, xv[c][i][0].w, xv[c][i][Z].x, xv[c][i][Z].y, xv[c][i][Z].z, xv[c][i][Z].w};
                const float gg[8] = {gv[c][0].x, gv[c][0].y, gv[c][0].z, gv[c][0].w, gv[c][Z].x, gv[c][Z].y, gv[c][Z].z, gv[c][Z].w};
                float sq = 0.f;
#pragma unroll
                for (int q = 0; q < 4 * Q; ++q) {
                    sq += v[q] * v[q];
                    v[q] = j < n ? v[q] * gg[q] : 0.f;  // (inputs past this wave's last count for nothing)
                }
                ss[i] += j < n ? sq : 0.f;
                if constexpr (F32) {
                    X[j][i][0] = make_uint4(__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3]));
                    continue;
                }
                uint32_t hi[4], lo[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) split_bf16x2(v[2 * q], v[2 * q + 1], hi[q], lo[q]);
                if constexpr (PACK) {
                    const bool low = tok >= 8;
                    X[j][i][0] = make_uint4(low ? lo[0] : hi[0], low ? lo[1] : hi[1], low ? lo[2] : hi[2], low ? lo[3] : hi[3]);
                } else {
                    X[j][i][0] = make_uint4(hi[0], hi[1], hi[2], hi[3]);
                    X[j][i][P - 1] = make_uint4(lo[0], lo[1], lo[2], lo[3]);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            ss[i] = quad_rows_sum(ss[i]);
            if (g == 0) rsum[wave * 32 + i * 16 + tok] = ss[i];
        }
    }
    f32x4 acc[RW][NT];
    auto multiply = [&](const uint4 (&W)[U][RW], auto batch) {
        constexpr int B = decltype(batch)::value;
        if constexpr (F32) {
            auto part = [](const uint4& v, int q) { return __uint_as_float(q == 0 ? v.x : q == 1 ? v.y : q == 2 ? v.z : v.w); };
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int q = 0; q < 4; ++q)
#pragma unroll
                    for (int i = 0; i < NT; ++i)
#pragma unroll
                        for (int r = 0; r < RW; ++r) acc[r][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(part(W[u][r], q), part(X[B * U + u][i][0], q), acc[r][i], 0, 0, 0);
        } else
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll
                    for (int r = 0; r < RW; ++r)
                        acc[r][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, W[u][r]), __builtin_bit_cast(bf16x8, X[B * U + u][i][p]), acc[r][i], 0, 0, 0);
    };
    Stat st = stat_neutral();
    float lost = 0.f;  // (fp32) of the running sum
    float scale = 1.f;
    bool first = true;
    const int nt = wave % NT, t = nt * 16 + tok;
    auto clear = [&] {
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int i = 0; i < NT; ++i) acc[r][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    };
    // the waves' sums of group `gg` joined, its logits counted
    auto join = [&](int gg) {
        if (!first) lds_barrier();  // (the group before has been read)
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int i = 0; i < NT; ++i) red[(wave * UNITS + r * NT + i) * 64 + lane] = acc[r][i];
        lds_barrier();
        if (first) {
            float p[kHeadWaves], s = 0.f;
#pragma unroll
            for (int w = 0; w < kHeadWaves; ++w) p[w] = rsum[w * 32 + (PACK ? tok & 7 : t)];
#pragma unroll
            for (int w = 0; w < kHeadWaves; ++w) s += p[w];
            scale = __builtin_amdgcn_rsqf(s * __builtin_amdgcn_rcpf((float)(tk * KT)) + a.eps);
        }
        first = false;
        const int tile = gg * RW + wave / NT;
        if (wave >= UNITS || tile >= tn) return;
        f32x4 p[kHeadWaves];
#pragma unroll
        for (int w = 0; w < kHeadWaves; ++w) p[w] = red[(w * UNITS + wave) * 64 + lane];
        f32x4 c = p[0];
#pragma unroll
        for (int w = 1; w < kHeadWaves; ++w) c += p[w];
        const int n0 = tile * 16 + g * 4;
        float z[4], top = -INFINITY;
        int at = 0x7FFFFFFF;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            if constexpr (PACK) c[v] += dpp_f<0x128, 0xF>(0.f, c[v]);
            z[v] = c[v] * scale * a.scale;
            if (t < T && n0 + v < a.vocab) {
                if (n0 + v == target) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(z[v]), make_rsrc(a.zt, sizeof(float) * kMaxRows), t * 4, 0, kPartAux);
                if (a.dbg) a.dbg[(size_t)t * a.vocab + n0 + v] = z[v];
            } else {
                z[v] = -INFINITY;
            }
            if (z[v] > top) {  // (strict: equal maxima keep the lower id)
                top = z[v];
                at = n0 + v;
            }
        }
        if (top > st.m) st.idx = at;
        const float m = fmaxf(st.m, top), base = m == -INFINITY ? 0.f : m;
        float e[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) e[v] = fexp_full(z[v] - base);
        const float f = fexp_full(st.m - base), add = (e[0] + e[1]) + (e[2] + e[3]);
        if constexpr (F32) {  // (a sum of as many groups: what an addition loses goes into the next)
            const float y = add - lost * f, kept = st.s * f, sum = kept + y;
            lost = (sum - kept) - y;
            st.s = sum;
        } else {
            st.s = st.s * f + add;
        }
        st.m = m;
    };
    if constexpr (BATCHES == 1) {  // a group per batch
#pragma unroll 1
        for (; grp < groups; grp += 2 * step) {
            clear();
            multiply(W0, std::integral_constant<int, 0>{});
            if (grp + 2 * step < groups) request(W0, grp + 2 * step, 0);
            join(grp);
            if (grp + step >= groups) break;
            clear();
            multiply(W1, std::integral_constant<int, 0>{});
            if (grp + 3 * step < groups) request(W1, grp + 3 * step, 0);
            join(grp + step);
        }
    } else {
        static_assert(BATCHES == 1 || BATCHES == 2 || BATCHES == 4 || BATCHES == 8, "two buffers");
#pragma unroll 1
        for (; grp < groups; grp += step) {
            clear();
            multiply(W0, std::integral_constant<int, 0>{});
            ask(W0, grp, 2);
            multiply(W1, std::integral_constant<int, 1 % BATCHES>{});
            ask(W1, grp, 3);
            if constexpr (BATCHES >= 4) {
                multiply(W0, std::integral_constant<int, 2 % BATCHES>{});
                ask(W0, grp, 4);
                multiply(W1, std::integral_constant<int, 3 % BATCHES>{});
                ask(W1, grp, 5);
            }
            if constexpr (BATCHES == 8) {
                multiply(W0, std::integral_constant<int, 4 % BATCHES>{});
                ask(W0, grp, 6);
                multiply(W1, std::integral_constant<int, 5 % BATCHES>{});
                ask(W1, grp, 7);
                multiply(W0, std::integral_constant<int, 6 % BATCHES>{});
                ask(W0, grp, 8);
                multiply(W1, std::integral_constant<int, 7 % BATCHES>{});
                ask(W1, grp, 9);
            }
            join(grp);
        }
    }
    // ---- the workgroup's partials ----
    if constexpr (F32) st.s -= lost;
    {  // lanes of a row
        Stat x, y;
        uint32_t p, q;
        auto both = [&](const Stat& u, const Stat& v) {
            const float m = fmaxf(u.m, v.m), base = m == -INFINITY ? 0.f : m;
            return Stat{m, u.s * fexp_full(u.m - base) + v.s * fexp_full(v.m - base), (u.m > v.m || (u.m == v.m && u.idx < v.idx)) ? u.idx : v.idx};
        };
        pair_xor16(__float_as_uint(st.m), p, q); x.m = __uint_as_float(p); y.m = __uint_as_float(q);
        pair_xor16(__float_as_uint(st.s), p, q); x.s = __uint_as_float(p); y.s = __uint_as_float(q);
        pair_xor16((uint32_t)st.idx, p, q); x.idx = (int)p; y.idx = (int)q;
        st = both(x, y);
        pair_xor32(__float_as_uint(st.m), p, q); x.m = __uint_as_float(p); y.m = __uint_as_float(q);
        pair_xor32(__float_as_uint(st.s), p, q); x.s = __uint_as_float(p); y.s = __uint_as_float(q);
        pair_xor32((uint32_t)st.idx, p, q); x.idx = (int)p; y.idx = (int)q;
        st = both(x, y);
    }
    if (g == 0) wstat[wave * 16 + tok] = StatPart{st.m, st.s, st.idx, 0};
    lds_barrier();
    const int row = (int)threadIdx.x;
    const __amdgpu_buffer_rsrc_t part = make_rsrc(a.part, 0xFFFFFFFFu);
    if (row < T) {
        Stat r = stat_neutral();
#pragma unroll
        for (int u = 0; u < RW; ++u) {
            const StatPart p = wstat[(u * NT + (row >> 4)) * 16 + (row & 15)];
            r = stat_merge<true>(r, Stat{p.m, p.s, p.idx});
        }
        const StatPart o = {r.m, r.s, r.idx, 0};
        typedef unsigned v4u __attribute__((ext_vector_type(4)));
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, o), part, (row * a.part_ld + (int)blockIdx.x) * (int)sizeof(StatPart), 0, kPartAux);
    }
    if (!a.out || !last_in(a.arrived, (unsigned)step, share)) return;
    for (int r0 = wave; r0 < T; r0 += kHeadWaves) {
        StatPart sp[8];
        Stat r = stat_neutral();
        for (int p0 = lane; p0 < step; p0 += 512) {
#pragma unroll
            for (int k = 0; k < 8; ++k)
                sp[k] = __builtin_bit_cast(StatPart, __builtin_amdgcn_raw_buffer_load_b128(part, (r0 * a.part_ld + min(p0 + k * 64, step - 1)) * (int)sizeof(StatPart), 0, kPartAux));
            take_parts(r, sp, p0, step);
        }
        r = join_parts(r);
        const int tg = pos0 + r0 + 1 < *a.ylen_ptr ? a.y[pos0 + r0 + 1] : -1;
        const float zt = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(make_rsrc(a.zt, sizeof(float) * kMaxRows), r0 * 4, 0, kPartAux));
        if (lane == 0) put_row_stats(a.out, r0, r.m, r.s, r.idx, tg >= 0 && tg < a.vocab, zt, a.done, a.call);
    }
}

// Feature tiles per group: as many as the registers hold, unless fewer leave less to the last round of groups.
static int head_tiles(const TMat& W, int T, bool f32) {
    const int per = (W.tk + kHeadWaves - 1) / kHeadWaves, most = per <= 4 ? 4 : f32 && (per > 16 || (per > 8 && T > 16)) ? 1 : 2;
    if (f32 ? per > (T > 16 ? 16 : 32) : per > 8) return 0;  // (wider rows do not fit the registers beside the weights: 4096 x 65 536 ids 138 us for 8 rows against 119)
    int best = most;
    auto rounds = [&](int rw) { return ((W.tn + rw - 1) / rw + 255) / 256 * rw; };
    for (int rw = most; rw >= 1; rw /= 2)
        if (rounds(rw) < rounds(best)) best = rw;
    return best;
}
int head_groups(const TMat& W, int T, bool f32) {
    const int rw = head_tiles(W, T, f32);
    return rw ? std::min((W.tn + rw - 1) / rw, 256) : 0;
}

// (input tiles per wave, feature tiles, input tiles per batch)
#define BILD_HEAD_EACH(X) X(2, 4, 2) X(2, 2, 2) X(2, 1, 2) X(4, 4, 2) X(4, 2, 2) X(4, 1, 4) X(8, 2, 4) X(8, 1, 4)
// (fp32 models: tiles of sixteen inputs)
#define BILD_HEAD_F32(X) X(16, 2, 4) X(16, 1, 4) X(32, 1, 4)

hipError_t head_init() {
    static hipError_t done = [] {
#define BILD_F(KPV, RWV, UV) (const void*)head_kernel<KPV, RWV, UV, 1, true>, (const void*)head_kernel<KPV, RWV, UV, 1, false>,
#define BILD_F2(KPV, RWV, UV) (const void*)head_kernel<KPV, RWV, UV, 2, false>,
#define BILD_F3(KPV, RWV, UV) (const void*)head_kernel<KPV, RWV, UV, 1, false, true>, (const void*)head_kernel<KPV, RWV, UV, KPV * RWV >= 32 ? 1 : 2, false, true>,
        const void* fns[] = {BILD_HEAD_EACH(BILD_F) BILD_HEAD_EACH(BILD_F2) BILD_HEAD_EACH(BILD_F3) BILD_HEAD_F32(BILD_F3)};
#undef BILD_F
#undef BILD_F2
#undef BILD_F3
        return raise_lds_limit(fns, 160 * 1024);
    }();
    return done;
}

hipError_t launch_head(const HeadArgs& a, hipStream_t st) {
    if (hipError_t e = head_init(); e != hipSuccess) return e;
    const int rw = head_tiles(a.W, a.T, a.f32), per = (a.W.tk + kHeadWaves - 1) / kHeadWaves, kp = per <= 2 ? 2 : per <= 4 ? 4 : per <= 8 ? 8 : per <= 16 ? 16 : 32;
    if (!rw || a.T < 1 || a.T > kMaxRows || !a.x || !a.gain || !a.part || !a.zt || !a.y || !a.ylen_ptr || a.ldx < a.W.k || a.ldx % 4 || (a.out && !a.arrived) ||
        a.part_ld < head_groups(a.W, a.T, a.f32) || (size_t)a.part_ld * sizeof(StatPart) * kMaxRows >= (size_t)1 << 31)
        return hipErrorInvalidValue;
    const int nt = a.T > 16 ? 2 : 1;
    const size_t smem = (size_t)kHeadWaves * (rw * nt * 1024 + 32 * 4 + 16 * sizeof(StatPart)) + 16;
    const dim3 grid(head_groups(a.W, a.T, a.f32)), block(64 * kHeadWaves);
#define BILD_L(KPV, RWV, UV, NTV, PV) hipLaunchKernelGGL((head_kernel<KPV, RWV, UV, NTV, PV>), grid, block, smem, st, a.x, a.W.w, a.gain, a.ldx, a.W.tn, a.W.tk, a.T, a)
#define BILD_X3(KPV, RWV, UV)                                                                                                                                      \
    if (kp == KPV && rw == RWV) {                                                                                                                                  \
        if (nt == 1) hipLaunchKernelGGL((head_kernel<KPV, RWV, UV, 1, false, true>), grid, block, smem, st, a.x, a.W.w, a.gain, a.ldx, a.W.tn, a.W.tk, a.T, a);     \
        else hipLaunchKernelGGL((head_kernel<KPV, RWV, UV, KPV * RWV >= 32 ? 1 : 2, false, true>), grid, block, smem, st, a.x, a.W.w, a.gain, a.ldx, a.W.tn, a.W.tk, a.T, a); \
        return hipGetLastError();                                                                                                                                  \
    }
    if (a.f32) {
        BILD_HEAD_EACH(BILD_X3) BILD_HEAD_F32(BILD_X3)
        return hipErrorInvalidValue;
    }
#define BILD_X(KPV, RWV, UV)                              \
    if (kp == KPV && rw == RWV && nt == 1) {              \
        if (a.T <= 8) BILD_L(KPV, RWV, UV, 1, true);      \
        else BILD_L(KPV, RWV, UV, 1, false);              \
        return hipGetLastError();                         \
    }
#define BILD_X2(KPV, RWV, UV)                             \
    if (kp == KPV && rw == RWV && nt == 2) {              \
        BILD_L(KPV, RWV, UV, 2, false);                   \
        return hipGetLastError();                         \
    }
    BILD_HEAD_EACH(BILD_X) BILD_HEAD_EACH(BILD_X2)
    return hipErrorInvalidValue;
}

}  // namespace bild
