// GEMM of bf16 models over 2 .. 32 rows (a review of drafts): y[T][N] = f(x) W^T, weights streamed once.
//
// Bound: the weights' way from memory.  What stands beside it is the activations' way from L2: every workgroup of a projection
// reads all T rows of its inputs, which for 32 rows is as much as four feature tiles' weights.  A workgroup therefore
//   - has RW feature tiles, so many that about one workgroup per compute unit results (more tiles share one reading of x);
//   - splits the inputs over its eight waves: a wave needs only its own inputs of x, so x goes straight into operand registers, in
//     the order the matrix core wants (tile planes, written once by the producer), with no LDS, no conversion and no barrier on the
//     way; the waves' sums are joined through LDS once at the end;
//   - has a slice of the inputs only, where the matrix has few feature tiles and the rows are many, and the last of a group's slices
//     joins them (last_in.h);
//   - keeps two batches of tiles, weights and activations, on their way all the time, also across its feature groups where
//     there are more groups than workgroups (LM head).
// Up to eight rows one operand holds the high parts of the rows in its columns 0 .. 7 and the low parts in 8 .. 15 (PACK): half the
// loads of x and half the products.
//
// 7B shape, us per launch with rows staged in every workgroup and now (floor at 5.5 TB/s): 32 rows q, k, v 33.4, 23.1 (18.3); gated FFN
// input 46.5, 39.7 (32.8); residual projections, mean of two, 28.6, 18.1 (11.2); 11 rows 20.4, 38.3, 16.2.  The whole pass over 1024
// keys, 2, 4, 8, 12, 16, 32 rows: 3406, 3443, 3592, 3869, 4045, 5053 -> 3156, 3160, 3177, 3367, 3379, 3742 us (attn_split.hip included).
// Without slices the 32-row residual projections take 25.3; sliced q, k, v 34.6 instead of 30.6; workgroups that begin at the same
// inputs 2 % more in all; the sums of squares fetched one load after the other in front of the weights 2.5 us a launch.
#include "gemm_thin.h"

#include <algorithm>

#include "last_in.h"

namespace bild {

constexpr int kThinWaves = 8;
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
// input tiles per batch
constexpr int thin_batch(int loads) { return loads <= 2 ? 8 : loads <= 4 ? 4 : loads <= 6 ? 3 : 2; }

template <int RW, int NT, int EPI, int ROPE, bool GATED, bool PACK, bool SLICED>
__global__ __launch_bounds__(64 * kThinWaves, 1) void thin_kernel(const ThinArgs a) {
    constexpr int XL = PACK ? 1 : 2 * NT, U = thin_batch(RW + XL);
    constexpr bool NORM = EPI != EPI_RESID;
    constexpr int UNIT = GATED ? 2 : 1, UNITS = RW / UNIT * NT;  // joined at once: a tile (pair) of sixteen rows
    constexpr int TL = PACK ? 8 : NT * 16;                       // rows an operand has
    extern __shared__ __attribute__((aligned(16))) char smem[];
    f32x4* red = (f32x4*)smem;                              // [wave][RW * NT][64]
    float* rsum = (float*)(smem + kThinWaves * RW * NT * 1024);  // [wave][32]
    StatPart* wstat = (StatPart*)(rsum + kThinWaves * 32);  // [wave][16]
    unsigned* share = (unsigned*)(wstat + kThinWaves * 16);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int tok = lane & 15, g = lane >> 4;
    const int tk = a.W.tk, groups = (a.W.tn + RW - 1) / RW;
    // this workgroup's input tiles and, of those, this wave's
    const int slices = SLICED ? (int)gridDim.y : 1, slice = SLICED ? (int)blockIdx.y : 0, run = SLICED ? (tk + slices - 1) / slices : tk;
    const int ks = min(slice * run, tk - 1), ke = min(tk, slice * run + run), per = (run + kThinWaves - 1) / kThinWaves;
    const int k0 = min(ks + wave * per, tk - 1), n = max(0, min(per, ke - ks - wave * per));
    const int batches = ((per + U - 1) / U + 1) & ~1;  // (two buffers: an even number)

    // ---- the rows' sums of squares: requested first, all at once, they come from L2 ----
    constexpr int SP = kThinWaves * (64 / TL), SL = kMaxSsqParts / SP;  // parts a load covers, loads
    float sv[SL];
    if constexpr (NORM) {
        const int t = min(lane % TL, a.T - 1), p0 = wave * (64 / TL) + lane / TL;
#pragma unroll
        for (int i = 0; i < SL; ++i) sv[i] = a.ssq[(size_t)min(p0 + i * SP, a.ssq_parts - 1) * kMaxRows + t];
    }
    const __amdgpu_buffer_rsrc_t xs = make_rsrc(a.xp, 0xFFFFFFFFu);
    const unsigned xo = PACK ? (unsigned)((tok >> 3) * kTileBytes + (g * 16 + (tok & 7)) * 16) : (unsigned)lane * 16u;
    // (workgroups begin at different places of their inputs, or all of them would want the same lines of x at once)
    const int turn = n > 0 ? (int)(blockIdx.x % (unsigned)n) : 0;
    uint4 W0[U][RW], X0[U][XL], W1[U][RW], X1[U][XL];
    auto request = [&](uint4 (&W)[U][RW], uint4 (&X)[U][XL], int grp, int batch) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int j = min(batch * U + u, max(n - 1, 0)) + turn, kt = k0 + (j >= n ? max(j - n, 0) : j);
#pragma unroll
            for (int r = 0; r < RW; ++r)
                W[u][r] = buf_load(make_rsrc((const char*)a.W.w + (size_t)min(grp * RW + r, a.W.tn - 1) * tk * kTileBytes, 0xFFFFFFFFu), (unsigned)lane * 16u, kt * kTileBytes);
#pragma unroll
            for (int x = 0; x < XL; ++x) X[u][x] = buf_load(xs, xo, ((x >> 1) * tk + kt) * (2 * kTileBytes) + (x & 1) * kTileBytes);
        }
    };
    f32x4 acc[RW][NT];
    auto multiply = [&](const uint4 (&W)[U][RW], const uint4 (&X)[U][XL], int batch) {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (batch * U + u < n) {
#pragma unroll
                for (int x = 0; x < XL; ++x)
#pragma unroll
                    for (int r = 0; r < RW; ++r)
                        acc[r][x >> 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, W[u][r]), __builtin_bit_cast(bf16x8, X[u][x]), acc[r][x >> 1], 0, 0, 0);
            }
    };
    int grp = (int)blockIdx.x;
    request(W0, X0, grp, 0);
    request(W1, X1, grp, 1);
    if constexpr (NORM) {
        const int p0 = wave * (64 / TL) + lane / TL;
        float ss = 0.f;
#pragma unroll
        for (int i = 0; i < SL; ++i) ss += p0 + i * SP < a.ssq_parts ? sv[i] : 0.f;
        // one part per lane and wave to one per row and wave; joined behind the first barrier
        if constexpr (PACK) ss += dpp_f<0x128, 0xF>(0.f, ss);  // row_ror:8
        if constexpr (TL <= 16) {
            ss = quad_rows_sum(ss);
        } else {
            uint32_t lo, hi;
            pair_xor32(__float_as_uint(ss), lo, hi);
            ss = __uint_as_float(lo) + __uint_as_float(hi);
        }
        if (lane < TL) rsum[wave * 32 + lane] = ss;
    }
    const int pos0 = (EPI == EPI_QKV || EPI == EPI_LMHEAD) && a.pos_ptr ? *a.pos_ptr : 0;
    Stat st = stat_neutral();  // (LM head: of this wave's unit, over the groups)
    int target = -1;
    if constexpr (EPI == EPI_LMHEAD) {
        const int t = (wave % NT) * 16 + tok, ti = pos0 + t + 1;
        if (t < a.T && ti < *a.ylen_ptr) target = a.y[ti];
    }
    float scale[NT];
    bool first = true;
#pragma unroll 1
    for (; grp < groups; grp += (int)gridDim.x) {
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int i = 0; i < NT; ++i) acc[r][i] = f32x4{0.f, 0.f, 0.f, 0.f};
        const int ahead = grp + (int)gridDim.x;
#pragma unroll 1
        for (int b = 0; b < batches; b += 2) {
            const bool more = b + 2 < batches;
            multiply(W0, X0, b);
            if (more || ahead < groups) request(W0, X0, more ? grp : ahead, more ? b + 2 : 0);
            multiply(W1, X1, b + 1);
            if (more || ahead < groups) request(W1, X1, more ? grp : ahead, more ? b + 3 : 1);
        }
        float4 old[(UNITS + kThinWaves - 1) / kThinWaves];
        if constexpr (EPI == EPI_RESID) {
#pragma unroll
            for (int u = wave, j = 0; j < (UNITS + kThinWaves - 1) / kThinWaves; u += kThinWaves, ++j)
                old[j] = ld_act4(a.out + (size_t)min((u % NT) * 16 + tok, a.T - 1) * a.ldo + min(grp * RW + u / NT, a.W.tn - 1) * 16 + g * 4);
        }
        if (!first) lds_barrier();  // (the group before has been read)
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int i = 0; i < NT; ++i) red[(wave * (RW * NT) + r * NT + i) * 64 + lane] = acc[r][i];
        lds_barrier();
        if (NORM && first) {
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                float p[kThinWaves], s = 0.f;
                const int t = PACK ? tok & 7 : i * 16 + tok;
#pragma unroll
                for (int w = 0; w < kThinWaves; ++w) p[w] = rsum[w * 32 + t];
#pragma unroll
                for (int w = 0; w < kThinWaves; ++w) s += p[w];
                scale[i] = __builtin_amdgcn_rsqf(s * __builtin_amdgcn_rcpf((float)tk * 32.f) + a.eps);
            }
        }
        first = false;
        constexpr int MINE = (UNITS + kThinWaves - 1) / kThinWaves;  // units per wave
        f32x4 c[MINE][UNIT];
#pragma unroll
        for (int j = 0; j < MINE; ++j) {
            const int u = wave + j * kThinWaves;
            if (u >= UNITS) break;
            const int nt = u % NT, r0 = u / NT * UNIT;
#pragma unroll
            for (int q = 0; q < UNIT; ++q) {
                f32x4 p[kThinWaves];
#pragma unroll
                for (int w = 0; w < kThinWaves; ++w) p[w] = red[(w * (RW * NT) + (r0 + q) * NT + nt) * 64 + lane];
                c[j][q] = p[0];
#pragma unroll
                for (int w = 1; w < kThinWaves; ++w) c[j][q] += p[w];
                if constexpr (PACK) {
#pragma unroll
                    for (int v = 0; v < 4; ++v) c[j][q][v] += dpp_f<0x128, 0xF>(0.f, c[j][q][v]);
                }
            }
        }
        if constexpr (SLICED) {  // (a group per workgroup)
            static_assert(UNIT == 1 && EPI != EPI_LMHEAD, "one sum per unit");
            const __amdgpu_buffer_rsrc_t sums = make_rsrc(a.sums, kThinSums * sizeof(float));
            auto place = [&](int u, int s) { return ((((int)blockIdx.x * UNITS + u) * slices + s) * 64 + lane) * 16; };
#pragma unroll
            for (int j = 0; j < MINE; ++j)
                if (wave + j * kThinWaves < UNITS)
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, c[j][0]), sums, place(wave + j * kThinWaves, slice), 0, kPartAux);
            if (!last_in(a.arrived + blockIdx.x, (unsigned)slices, share)) return;
#pragma unroll
            for (int j = 0; j < MINE; ++j) {
                if (wave + j * kThinWaves >= UNITS) break;
                f32x4 p[8];  // (at most so many slices)
#pragma unroll
                for (int s = 0; s < 8; ++s) p[s] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(sums, place(wave + j * kThinWaves, min(s, slices - 1)), 0, kPartAux));
                c[j][0] = p[0];
#pragma unroll
                for (int s = 1; s < 8; ++s)
                    if (s < slices) c[j][0] += p[s];
            }
        }
#pragma unroll
        for (int j = 0; j < MINE; ++j) {
            const int u = wave + j * kThinWaves;
            if (u >= UNITS) break;
            const int nt = u % NT, tile = grp * RW + u / NT * UNIT;
            if (tile >= a.W.tn) continue;
            f32x4 (&c_)[UNIT] = c[j];
            if constexpr (NORM) {
#pragma unroll
                for (int q = 0; q < UNIT; ++q) c_[q] *= NT == 1 || nt == 0 ? scale[0] : scale[NT - 1];
            }
            const int t = nt * 16 + tok, n0 = (GATED ? tile >> 1 : tile) * 16 + g * 4;
            const bool ok = t < a.T;
            if constexpr (EPI == EPI_STORE) {
                if (ok) st_act4(a.out + (size_t)t * a.ldo + n0, make_float4(c_[0][0], c_[0][1], c_[0][2], c_[0][3]));
            } else if constexpr (EPI == EPI_ACT) {
                float o[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    if constexpr (GATED) o[v] = (a.act == BILD_ACT_GATED_GELU ? gelu_tanh_f(c_[0][v]) : silu_f(c_[0][v])) * c_[UNIT - 1][v];
                    else o[v] = fmaxf(c_[0][v], 0.f);
                }
                if (ok) put_tile_planes(a.np, a.np_tk, t, n0, o);
            } else if constexpr (EPI == EPI_RESID) {
                const float xn[4] = {old[j].x + c_[0][0], old[j].y + c_[0][1], old[j].z + c_[0][2], old[j].w + c_[0][3]};
                const float4 gn = *(const float4*)(a.np_gain + n0);
                const float w[4] = {xn[0] * gn.x, xn[1] * gn.y, xn[2] * gn.z, xn[3] * gn.w};
                const float sq = quad_rows_sum(xn[0] * xn[0] + xn[1] * xn[1] + xn[2] * xn[2] + xn[3] * xn[3]);
                if (ok) {
                    st_act4(a.out + (size_t)t * a.ldo + n0, make_float4(xn[0], xn[1], xn[2], xn[3]));
                    put_tile_planes(a.np, a.np_tk, t, n0, w);
                    if (g == 0) a.np_ssq[(size_t)tile * kMaxRows + t] = sq;
                }
            } else if constexpr (EPI == EPI_QKV) {
                const int seg = n0 < a.q_dim ? 0 : (n0 < a.q_dim + a.i_dim ? 1 : 2), pos = pos0 + t;
                const int nn = n0 - (seg == 0 ? 0 : (seg == 1 ? a.q_dim : a.q_dim + a.i_dim));
                float v4[4] = {c_[0][0], c_[0][1], c_[0][2], c_[0][3]};
                if (!ok) continue;
                if (ROPE && seg < 2) {
                    const double2* tb = a.rope + ((size_t)pos * a.d_head + nn % a.d_head) / 2;
#pragma unroll
                    for (int p2 = 0; p2 < 2; ++p2) {
                        const double2 cs = tb[p2];
                        const float x0 = v4[2 * p2], x1 = v4[2 * p2 + 1];
                        v4[2 * p2] = (float)((double)x0 * cs.x - (double)x1 * cs.y);
                        v4[2 * p2 + 1] = (float)((double)x0 * cs.y + (double)x1 * cs.x);
                    }
                }
                if (seg == 0) {
                    st_act4(a.q_out + (size_t)t * a.i_dim + nn, make_float4(v4[0], v4[1], v4[2], v4[3]));
                } else if (seg == 1) {
                    st_u64((uint16_t*)a.k_cache + (size_t)pos * a.i_dim + nn, pack_bf16x2(v4[0], v4[1]), pack_bf16x2(v4[2], v4[3]));
                } else {
#pragma unroll
                    for (int v = 0; v < 4; ++v) st_u16((uint16_t*)a.v_cache + (size_t)(nn + v) * a.vcap + pos, (uint16_t)f2bf(v4[v]));
                }
            } else {  // EPI_LMHEAD
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float z = c_[0][v] * a.scale;
                    if (ok && n0 + v < a.vocab) {
                        stat_push(st, z, n0 + v);
                        if (t >= a.first) {
                            if (n0 + v == target) a.zt[t - a.first] = z;
                            if (a.dbg) a.dbg[(size_t)(t - a.first) * a.vocab + n0 + v] = z;
                        }
                    }
                }
            }
        }
    }
    if constexpr (EPI == EPI_LMHEAD) {
        static_assert(UNITS <= kThinWaves && kThinWaves % NT == 0, "a wave keeps one row tile's statistics");
        st = stat_quad_rows(st);
        if (g == 0) wstat[wave * 16 + tok] = StatPart{st.m, st.s, st.idx, 0};
        lds_barrier();
        const int t = (int)threadIdx.x;
        if (t >= a.first && t < a.T) {
            Stat r = stat_neutral();
#pragma unroll
            for (int u = t >> 4; u < UNITS; u += NT) {
                const StatPart p = wstat[u * 16 + (t & 15)];
                r = stat_merge(r, Stat{p.m, p.s, p.idx});
            }
            a.part[(size_t)(t - a.first) * a.part_ld + blockIdx.x] = StatPart{r.m, r.s, r.idx, 0};
        }
    }
}

// Feature tiles per workgroup: so many that a workgroup per compute unit results, at most what the registers hold (a larger matrix's
// workgroups take one group after the other).
// More than eight rows: x is as much as 2 (9 .. 16 rows) or 4 feature tiles' weights, and it is the L2s' rate that a workgroup
// with fewer tiles waits for.  The residual projections then take four tiles and a slice of the inputs, as many slices
// as compute units allow; below four input tiles per wave the joining costs more than it saves.
ThinShape thin_shape(const TMat& W, int epi, int act, int T) {
    const int pair = epi == EPI_ACT && act != BILD_ACT_RELU ? 2 : 1, want = (W.tn / pair + 255) / 256;
    auto plain = [&](int rw) { return ThinShape{rw, std::min((W.tn + rw - 1) / rw, 256), 1}; };
    auto sliced = [&](int rw) {
        ThinShape s = {rw, (W.tn + rw - 1) / rw, 1};
        while (s.slices < 8 && s.groups * s.slices * 2 <= 256 && W.tk >= 4 * kThinWaves * s.slices * 2) s.slices *= 2;
        return s;
    };
    if (epi == EPI_LMHEAD) return plain(W.tn >= 2 * 256 ? 4 : 1);
    if (pair == 2) return plain(2 * std::min(want, 3));
    if (epi == EPI_RESID && T > 8) {
        const ThinShape s = sliced(4);
        if (s.slices > 1 && s.groups * s.slices >= 192) return s;
    }
    return plain(epi == EPI_QKV ? std::min(want, 3) : 1);
}

#define BILD_THIN_EACH(X)                                                                                              \
    X(1, EPI_STORE, 0, false) X(1, EPI_RESID, 0, false) X(1, EPI_QKV, 0, false) X(2, EPI_QKV, 0, false)                \
    X(3, EPI_QKV, 0, false) X(1, EPI_QKV, 1, false) X(2, EPI_QKV, 1, false) X(3, EPI_QKV, 1, false)                    \
    X(1, EPI_ACT, 0, false) X(2, EPI_ACT, 0, true) X(4, EPI_ACT, 0, true) X(6, EPI_ACT, 0, true)                       \
    X(1, EPI_LMHEAD, 0, false) X(4, EPI_LMHEAD, 0, false)

hipError_t gemm_thin_init() {
    static hipError_t done = [] {
#define BILD_F(RWV, EPIV, ROPEV, GV)                                                                                   \
    (const void*)thin_kernel<RWV, 1, EPIV, ROPEV, GV, true, false>, (const void*)thin_kernel<RWV, 1, EPIV, ROPEV, GV, false, false>, \
        (const void*)thin_kernel<RWV, 2, EPIV, ROPEV, GV, false, false>,
        const void* fns[] = {BILD_THIN_EACH(BILD_F)
                             (const void*)thin_kernel<4, 1, EPI_RESID, 0, false, false, true>, (const void*)thin_kernel<4, 2, EPI_RESID, 0, false, false, true>};
#undef BILD_F
        return raise_lds_limit(fns, 160 * 1024);
    }();
    return done;
}

hipError_t launch_gemm_thin(const ThinArgs& a, hipStream_t st) {
    if (hipError_t e = gemm_thin_init(); e != hipSuccess) return e;
    const bool norm = a.epi != EPI_RESID, gated = a.epi == EPI_ACT && a.act != BILD_ACT_RELU, rope = a.epi == EPI_QKV && a.rope;
    if (a.T < 1 || a.T > kMaxRows || !a.xp || !a.W.w || a.W.tk < 1 || a.W.tn < 1 || (norm && (!a.ssq || a.ssq_parts < 1 || a.ssq_parts > kMaxSsqParts)) ||
        ((a.epi == EPI_RESID || a.epi == EPI_STORE) && !a.out) || (a.epi == EPI_RESID && (!a.np || !a.np_gain || !a.np_ssq)) ||
        (a.epi == EPI_ACT && (!a.np || (gated && a.W.tn % 2))) || (a.epi == EPI_QKV && (!a.q_out || !a.k_cache || !a.v_cache || !a.pos_ptr)) ||
        (a.epi == EPI_LMHEAD && (!a.part || !a.ylen_ptr || a.first < 0 || a.first >= a.T)))
        return hipErrorInvalidValue;
    const ThinShape sh = thin_shape(a.W, a.epi, a.act, a.T);
    if (sh.slices > 1 && (!a.sums || !a.arrived || sh.groups > kThinArrivals)) return hipErrorInvalidValue;
    const int nt = a.T > 16 ? 2 : 1;
    const size_t smem = (size_t)kThinWaves * (sh.rw * nt * 1024 + 32 * 4 + 16 * sizeof(StatPart)) + 16;
    const dim3 grid(sh.groups, sh.slices), block(64 * kThinWaves);
#define BILD_S(RWV, NTV, EPIV, ROPEV)                                                                                    \
    if (sh.rw == RWV && nt == NTV && a.epi == EPIV && rope == (ROPEV != 0)) {                                            \
        hipLaunchKernelGGL((thin_kernel<RWV, NTV, EPIV, ROPEV, false, false, true>), grid, block, smem, st, a);          \
        return hipGetLastError();                                                                                        \
    }
    if (sh.slices > 1) {
        BILD_S(4, 1, EPI_RESID, 0) BILD_S(4, 2, EPI_RESID, 0)
        return hipErrorInvalidValue;
    }
#undef BILD_S
#define BILD_L(RWV, EPIV, ROPEV, GV)                                                                                     \
    if (sh.rw == RWV && a.epi == EPIV && rope == (ROPEV != 0) && gated == GV) {                                          \
        if (a.T <= 8) hipLaunchKernelGGL((thin_kernel<RWV, 1, EPIV, ROPEV, GV, true, false>), grid, block, smem, st, a); \
        else if (nt == 1) hipLaunchKernelGGL((thin_kernel<RWV, 1, EPIV, ROPEV, GV, false, false>), grid, block, smem, st, a); \
        else hipLaunchKernelGGL((thin_kernel<RWV, 2, EPIV, ROPEV, GV, false, false>), grid, block, smem, st, a);         \
        return hipGetLastError();                                                                                        \
    }
    BILD_THIN_EACH(BILD_L)
#undef BILD_L
    return hipErrorInvalidValue;
}

}  // namespace bild
