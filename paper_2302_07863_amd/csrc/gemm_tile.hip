// GEMM of bf16 models for passes over MANY rows (more than 32): the encoder, the cross K/V of a source and the prompt
// prefill of a decoder-only model - everything a request has to wait for before its first token (Section 3.2 conditions
// both models on the input x; Section 4.1 measures latency end to end per example).
//
//   y[M][N] = f(x[M][K]) W^T   with the RMSNorm scale, the residual add, the activation / gating, the Q/K/V split with RoPE
//   and the cache append fused behind the products.
//
// Activations arrive as "tile planes": the kernel that produced them has split every value once into a high and a low bf16
// part (times the gain of this projection's norm) and stored both in the order of the matrix-core B operand,
//   [row / 16][input / 32][high, low][1 KiB: lane l holds row l % 16, inputs 8 (l / 16) .. + 7],
// so that a wavefront fetches an operand of 16 rows x 32 inputs with one contiguous 1 KiB load, exactly as it fetches
// a weight tile, and nothing is converted, transposed or staged here.  (Converting fp32 activations in every workgroup was
// most of what these passes cost: a 512-row pass over a 1024-wide projection repeats the conversion 16 to 64 times.)
//
// Bound: matrix cores for large products (two MFMAs per tile, high and low part), otherwise the 64 bytes a clock a compute
// unit takes from L2.  A wave owns 64 rows x 16 FT features; the operands of its next step are requested while the current
// one is multiplied.  Waves of a workgroup share nothing in the loop (no barrier, no LDS): either they own different
// features of the same rows (the rows' operands then come from the vector cache), or, where a product has too few tiles
// to occupy the chip, they take slices of the inputs and add their sums in LDS at the end, in a fixed order.
#include <algorithm>

#include "kernel_common.h"

namespace bild {

constexpr int kTileWaves = 4;
__host__ __device__ constexpr int tile_sums(int rt) { return rt * 16 * kTileWaves > 256 ? rt * 16 * kTileWaves : 256; }

// Three workgroups per compute unit (see the shared form below)
constexpr bool tile_lean(int rt, int epi, bool gated) { return rt == 4 && (epi == EPI_QKV || gated); }

// One workgroup per compute unit (sliced inputs, 24 tiles of sums and more a wave)
constexpr bool tile_alone(int rt, int ft, bool share) { return !share && rt * ft >= 24; }

// Row block and feature group of a workgroup.  Workgroups go to the eight dies in turn; the dies form a grid of a.gr row
// shares x 8 / a.gr feature shares (launch_gemm_tile), and a die walks the row blocks of its share before the next feature
// group, so that the weights of a group come from memory once and are then in that die's L2 while the rows pass.
// (Row blocks outermost, a 22016 x 4096 projection over 1023 rows streamed its 180 MB once per row block: 424 us against
// 323 with the same tiles.)
__device__ __forceinline__ bool tile_block(const TileGemmArgs& a, int& rb, int& fg) {
    const int die = (int)blockIdx.x & 7, j = (int)blockIdx.x >> 3;
    const int gf = 8 / a.gr, rper = (a.rbs + a.gr - 1) / a.gr;
    const int q = j / rper;
    rb = (j - q * rper) * a.gr + die / gf;
    fg = q * gf + die % gf;
    return rb < a.rbs && fg < a.fgs;
}

// FT: feature tiles per wave.  GATED: feature tiles 2j / 2j+1 hold gate and linear branch of output block j.
// SPLIT: the waves of a workgroup (also) slice the inputs, a.wk of them per feature group.
template <int RT, int FT, int EPI, int ROPE, bool GATED, bool SPLIT, bool SHARE>
__global__ __launch_bounds__(256, SHARE && tile_lean(RT, EPI, GATED) ? 3 : tile_alone(RT, FT, SHARE) ? 1 : 2) void gemm_tile_kernel(const TileGemmArgs a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr bool norm = EPI != EPI_RESID;  // residual-adding projections read un-normalised input
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int WK = SPLIT ? a.wk : 1, wkid = SPLIT ? wave & (WK - 1) : 0, wn = SPLIT ? wave >> a.lwk : wave;
    const int WN = SPLIT ? kTileWaves >> a.lwk : kTileWaves;
    const int tok_l = lane & 15, kq = lane >> 4;
    int rb, fg;
    if (!tile_block(a, rb, fg)) return;
    const int r0 = rb * (RT * 16), tile0 = (fg * WN + wn) * FT;
    const int tk = a.W.tk;
    const int rt_last = (a.M - 1) >> 4;
    const unsigned lane16 = (unsigned)lane * 16u;
    // operands by buffer loads: base and size in scalar registers, one lane offset, a scalar offset per tile (from the
    // first tile of this wave, so that offsets stay small however long the pass)
    const int wt0 = min(tile0, a.W.tn - 1), xt0 = r0 >> 4;
    const __amdgpu_buffer_rsrc_t wr = make_rsrc((const char*)a.W.w + (size_t)wt0 * tk * kTileBytes, (size_t)(a.W.tn - wt0) * tk * kTileBytes);
    const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.xp + (size_t)xt0 * tk * (2 * kTileBytes), (size_t)(rt_last + 1 - xt0) * tk * (2 * kTileBytes));
    int woff[FT], xoff[RT];
#pragma unroll
    for (int f = 0; f < FT; ++f) woff[f] = (min(tile0 + f, a.W.tn - 1) - wt0) * tk * kTileBytes;
#pragma unroll
    for (int r = 0; r < RT; ++r) xoff[r] = min(r, rt_last - xt0) * tk * (2 * kTileBytes);

    const int per = SPLIT ? (tk + WK - 1) >> a.lwk : tk;
    const int kb = wkid * per, ke = min(tk, kb + per);
    f32x4 acc[FT][RT];
#pragma unroll
    for (int f = 0; f < FT; ++f)
#pragma unroll
        for (int r = 0; r < RT; ++r) acc[f][r] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](const uint4 (&W)[FT], const uint4 (&X)[RT][2]) {
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int f = 0; f < FT; ++f)
                    acc[f][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, W[f]), __builtin_bit_cast(bf16x8, X[r][p]),
                                                                        acc[f][r], 0, 0, 0);
    };
    float* nss = (float*)smem;              // [at least 256] sums of squares: of the input rows, or (EPI_RESID) of the output rows
    f32x4* red = (f32x4*)(nss + tile_sums(RT));
    // Sums of squares of the rows from the producer's partial sums: 256 / rows threads share a row's parts, eight requests at
    // a time (one after the other they were up to 64 dependent trips to memory); added up behind the products.
    constexpr int ROWS = RT * 16, SHARES = 256 / ROWS;
    float ssum = 0.f;
    auto row_sums = [&]() {
        if (!norm) return;
        if (SHARES * ROWS < 256 && tid >= SHARES * ROWS) return;
        const float* sp = a.ssq + min(r0 + tid % ROWS, a.M - 1);
        for (int p0 = tid / ROWS; p0 < a.ssq_parts; p0 += 8 * SHARES) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = sp[(size_t)min(p0 + u * SHARES, a.ssq_parts - 1) * a.ssq_ld];
#pragma unroll
            for (int u = 0; u < 8; ++u) ssum += p0 + u * SHARES < a.ssq_parts ? v[u] : 0.f;
        }
        nss[tid] = ssum;  // [share][row]
    };
    auto row_scale = [&](int tl) {  // 1/rms of row tl of the block
        float sum = 0.f;
#pragma unroll
        for (int h = 0; h < SHARES; ++h) sum += nss[h * ROWS + tl];
        return rsqrtf(sum / (float)a.W.k + a.eps);
    };
    // With sliced inputs a wave finishes 1 / WK of the row tiles: what it adds to is requested ahead of the products.
    // (not where a wave has so many sums)
    constexpr bool AHEAD = FT <= 4;
    float4 old[AHEAD ? FT : 1], gain[AHEAD ? FT : 1];
    if constexpr (EPI == EPI_RESID && AHEAD) {
#pragma unroll
        for (int f = 0; f < FT; ++f) {
            const int n0 = min(tile0 + f, a.W.tn - 1) * 16 + kq * 4;
            gain[f] = *(const float4*)(a.np_gain + n0);
            if (SPLIT) old[f] = *(const float4*)(a.x + (size_t)min(r0 + wkid * 16 + tok_l, a.M - 1) * a.ldx + n0);
        }
    }
    if constexpr (SHARE) {
        // The rows' operands go through LDS: in step k each wave stores its part of a later step's.
        // Four row tiles, but for an FFN without gate: of step k + 2, so that the first row tile of step k + 1 is read ahead of the
        // barrier between the two and a step begins with products; the requests are spread among the products (all at once they
        // hold up the wave that issues them); registers for three workgroups per compute unit unless the epilogue needs them.  1023
        // rows: 12288 features 176 -> 167 us; 4096 features, 4096 and 11008 inputs, one workgroup per compute unit, on average 157
        // -> 149; 11264 features, gated, 86 -> 83 (1531 rows x 4096 x 1024 without gate: 31.9 -> 32.2, and 1 % off the encoder).
        // Else of step k + 1, requests in one go.  Eight row tiles have room for two steps ahead (the other way 280 -> 285 us at 22016
        // features, 1531 rows x 49152 x 1024 291 -> 307; spread as well 310).
        constexpr int UPW = 2 * RT / kTileWaves;  // 1 KiB units a wave fetches per step
        constexpr int SLOT = 2 * RT * kTileBytes;
        constexpr bool SPREAD = tile_lean(RT, EPI, GATED) || (RT == 4 && EPI == EPI_RESID);
        constexpr int AH = SPREAD ? 2 : 1;        // steps from the store to the use
        char* xs = (char*)red;                    // [2 AH][RT][2][1 KiB]
        constexpr int D = RT == 8 ? 2 : RT == 6 || tile_lean(RT, EPI, GATED) ? 3 : 4;  // steps requested ahead (spread: one less of the weights)
        uint4 W[D][FT], XR[D][UPW], B[2][2];
        int xu[UPW];
#pragma unroll
        for (int u = 0; u < UPW; ++u) {
            const int unit = wave * UPW + u;
            xu[u] = min(unit >> 1, rt_last - xt0) * tk * (2 * kTileBytes) + (unit & 1) * kTileBytes;
        }
        auto request_w = [&](uint4 (&Wd)[FT], int k, int f) { Wd[f] = buf_load(wr, lane16, woff[f] + min(k, tk - 1) * kTileBytes); };
        auto request_x = [&](uint4 (&Xd)[UPW], int k, int u) { Xd[u] = buf_load(xr, lane16, xu[u] + min(k, tk - 1) * (2 * kTileBytes)); };
        static_assert(UPW + FT <= 2 * RT, "a request per half row tile");
        auto store_x = [&](const uint4 (&Xd)[UPW], int k) {
#pragma unroll
            for (int u = 0; u < UPW; ++u) *(uint4*)(xs + (k & (2 * AH - 1)) * SLOT + (wave * UPW + u) * kTileBytes + lane16) = Xd[u];
        };
        auto frag = [&](int k, int r) {
            const char* xb = xs + (k & (2 * AH - 1)) * SLOT + r * 2 * kTileBytes + lane16;
            B[r & 1][0] = *(const uint4*)xb;
            B[r & 1][1] = *(const uint4*)(xb + kTileBytes);
        };
        auto compute = [&](const uint4 (&Wc)[FT], uint4 (&Xn)[UPW], uint4 (&Wn)[FT], int k, bool more) {
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                if (AH == 1 && r == 0) frag(k, 0);
                if (AH == 2 || r + 1 < RT) frag(r + 1 < RT ? k : k + 1, r + 1 < RT ? r + 1 : 0);  // read ahead of the products of this row tile
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int p = 0; p < 2; ++p) {
#pragma unroll
                    for (int f = 0; f < FT; ++f)
                        acc[f][r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, Wc[f]), __builtin_bit_cast(bf16x8, B[r & 1][p]), acc[f][r], 0, 0, 0);
                    __builtin_amdgcn_sched_barrier(0);
                    const int i = r * 2 + p;
                    if (SPREAD && more && i < UPW + FT) {
                        if (i < UPW) request_x(Xn, k + AH + D, i); else request_w(Wn, k + D - 1, i - UPW);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        // (in the order of the loop: the memory counter retires requests in order, and the waits of the loop hold for both ways into it)
        uint4 X0[AH][UPW];
#pragma unroll
        for (int i = 0; i < AH; ++i)
#pragma unroll
            for (int u = 0; u < UPW; ++u) request_x(X0[i], i, u);
#pragma unroll
        for (int d = 0; d < D; ++d) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int u = 0; u < UPW; ++u) request_x(XR[d], d + AH, u);
            __builtin_amdgcn_sched_barrier(0);
            if (d >= SPREAD)
#pragma unroll
                for (int f = 0; f < FT; ++f) request_w(W[d - SPREAD], d - SPREAD, f);
        }
        __builtin_amdgcn_sched_barrier(0);
        row_sums();
#pragma unroll
        for (int i = 0; i < AH; ++i) store_x(X0[i], i);
        lds_barrier();
        if constexpr (AH == 2) frag(0, 0);
        int k = 0;
        for (; k + D <= tk; k += D) {
#pragma unroll
            for (int j = 0; j < D; ++j) {
                store_x(XR[j], k + j + AH);
                if constexpr (!SPREAD) {
#pragma unroll
                    for (int u = 0; u < UPW; ++u) request_x(XR[j], k + j + AH + D, u);
                }
                __builtin_amdgcn_sched_barrier(0);
                compute(W[j], XR[j], W[(j + D - 1) % D], k + j, true);
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (!SPREAD) {
#pragma unroll
                    for (int f = 0; f < FT; ++f) request_w(W[j], k + j + D, f);
                }
                lds_barrier();
            }
        }
#pragma unroll
        for (int j = 0; j < D - 1; ++j) {  // the steps left over; their operands are on the way
            if (k + j < tk) {
                store_x(XR[j], k + j + AH);
                compute(W[j], XR[j], W[(j + D - 1) % D], k + j, false);
                lds_barrier();
            }
        }
    } else {
        // Steps requested ahead: a small step's loads do not cover their trip from L2, a large one's (12 KiB a wave) already fill the
        // compute unit's queue.  Encode of 40, 77, 201, 512, 1531 tokens, T5 shapes, us: three or four ahead and a request past the end of
        // a wave's few steps for each 1018, 1125, 1373, 2028, 4562; without those 985, 1086, 1326, 1951, 4424 (998, 1109, 1336, 1992, 4482
        // before, that run); by size as here 975, 1065, 1326, 1959, 4416; 8, 6, 5, 3 by size 996, 1079, 1333, 2041, 4440 (that run).
        // Six steps of 32 rows take 174 to 182 registers with two feature tiles and 142 to 150 with one (128 with four steps): two or three
        // waves a SIMD fit instead of four.  These forms are launched with a workgroup per compute unit at most (tile_shape), one wave a
        // SIMD, two beside the pair's other encoder.
        constexpr int LOADS = RT * 2 + FT, D = LOADS <= 6 ? 6 : LOADS == 8 ? 5 : LOADS <= 10 ? 4 : tile_alone(RT, FT, SHARE) ? 3 : 2;
        uint4 W[D][FT], X[D][RT][2];
        auto request = [&](int d, int k) {
#pragma unroll
            for (int f = 0; f < FT; ++f) W[d][f] = buf_load(wr, lane16, woff[f] + k * kTileBytes);
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                X[d][r][0] = buf_load(xr, lane16, xoff[r] + k * (2 * kTileBytes));
                X[d][r][1] = buf_load(xr, lane16 + kTileBytes, xoff[r] + k * (2 * kTileBytes));
            }
        };
#pragma unroll
        for (int d = 0; d < D; ++d) request(d, min(kb + d, ke - 1));
        row_sums();
        int k = kb;
        for (; k + 2 * D <= ke; k += D) {
#pragma unroll
            for (int j = 0; j < D; ++j) {
                multiply(W[j], X[j]);
                __builtin_amdgcn_sched_barrier(0);
                request(j, k + j + D);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        // (nothing past the end is asked for: a wave of sliced inputs has a few steps)
#pragma unroll
        for (int j = 0; j < D; ++j)
            if (k + j < ke) {
                multiply(W[j], X[j]);
                __builtin_amdgcn_sched_barrier(0);
                if (k + j + D < ke) request(j, k + j + D);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
        for (int j = 0; j < D - 1; ++j)
            if (k + j + D < ke) multiply(W[j], X[j]);
    }
    if constexpr (SPLIT) {
#pragma unroll
        for (int f = 0; f < FT; ++f)
#pragma unroll
            for (int r = 0; r < RT; ++r) red[((wave * RT + r) * FT + f) * 64 + lane] = acc[f][r];
    }
    if (norm || SPLIT) __syncthreads();

    const int pos0 = EPI == EPI_QKV ? (a.pos_ptr ? *a.pos_ptr : 0) + a.pos_add : 0;
    // ---- epilogue of one row tile: lane holds features tile*16 + kq*4 + v of row r*16 + tok_l ----
    auto finish = [&](int r, f32x4 (&c)[FT]) {
        const int tl = r * 16 + tok_l, t = r0 + tl;
        float ss = 0.f;
        const float sc = norm ? row_scale(tl) : 1.f;
        const bool row_ok = t < a.M;
        if constexpr (GATED) {
#pragma unroll
            for (int p = 0; p < FT / 2; ++p) {
                if (!row_ok || tile0 + 2 * p + 1 >= a.W.tn) continue;
                float o[4];
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const float g = c[2 * p][v] * sc, u = c[2 * p + 1][v] * sc;
                    o[v] = (a.act == BILD_ACT_GATED_GELU ? gelu_tanh_f(g) : silu_f(g)) * u;
                }
                put_tile_planes(a.np, a.np_tk, t, ((tile0 >> 1) + p) * 16 + kq * 4, o);
            }
            return;
        }
#pragma unroll
        for (int f = 0; f < FT; ++f) {
            if (!row_ok || tile0 + f >= a.W.tn) continue;
            const int n0 = (tile0 + f) * 16 + kq * 4;
            float v4[4] = {c[f][0] * sc, c[f][1] * sc, c[f][2] * sc, c[f][3] * sc};
            if constexpr (EPI == EPI_RESID) {
                float4* px = (float4*)(a.x + (size_t)t * a.ldx + n0);
                const float4 o = SPLIT && AHEAD && r == wkid ? old[AHEAD ? f : 0] : *px;
                const float xn[4] = {o.x + v4[0], o.y + v4[1], o.z + v4[2], o.w + v4[3]};
                *px = make_float4(xn[0], xn[1], xn[2], xn[3]);
                const float4 gn = AHEAD ? gain[AHEAD ? f : 0] : *(const float4*)(a.np_gain + n0);
                const float w[4] = {xn[0] * gn.x, xn[1] * gn.y, xn[2] * gn.z, xn[3] * gn.w};
                put_tile_planes(a.np, a.np_tk, t, n0, w);
                ss += xn[0] * xn[0] + xn[1] * xn[1] + xn[2] * xn[2] + xn[3] * xn[3];
            } else if constexpr (EPI == EPI_ACT) {
                const float o[4] = {fmaxf(v4[0], 0.f), fmaxf(v4[1], 0.f), fmaxf(v4[2], 0.f), fmaxf(v4[3], 0.f)};
                put_tile_planes(a.np, a.np_tk, t, n0, o);
            } else {  // EPI_QKV; several layers' K/V projections side by side when a.layer_n < N
                const int layer = n0 / a.layer_n, nl = n0 - layer * a.layer_n;
                const int pos = pos0 + t;
                const int seg = nl < a.q_dim ? 0 : (nl < a.q_dim + a.i_dim ? 1 : 2);
                const int nn = nl - (seg == 0 ? 0 : (seg == 1 ? a.q_dim : a.q_dim + a.i_dim));
                if (ROPE && seg < 2) {  // pairs (2i, 2i+1) of a head; the table holds cos and sin in double precision
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
                    *(float4*)(a.q_out + (size_t)t * a.i_dim + nn) = make_float4(v4[0], v4[1], v4[2], v4[3]);
                } else if (seg == 1) {  // K: [position][I]
                    uint16_t* kc = (uint16_t*)a.k_cache + (size_t)layer * a.kv_layer;
                    st_u64(kc + (size_t)pos * a.i_dim + nn, pack_bf16x2(v4[0], v4[1]), pack_bf16x2(v4[2], v4[3]));
                } else {  // V: transposed, [I][vcap] with the position contiguous
                    uint16_t* vc = (uint16_t*)a.v_cache + (size_t)layer * a.kv_layer;
#pragma unroll
                    for (int v = 0; v < 4; ++v) vc[(size_t)(nn + v) * a.vcap + pos] = (uint16_t)f2bf(v4[v]);
                }
            }
        }
        if constexpr (EPI == EPI_RESID) {
            ss = quad_rows_sum(ss);
            if (kq == 0) nss[wn * (RT * 16) + tl] = ss;
        }
    };
    if constexpr (SPLIT) {
        for (int r = wkid; r < RT; r += WK) {  // the row tiles are dealt to the slices
            f32x4 c[FT];
#pragma unroll
            for (int f = 0; f < FT; ++f) {
                const f32x4* src = red + (((wn << a.lwk) * RT + r) * FT + f) * 64 + lane;
                c[f] = src[0];
                for (int w = 1; w < WK; ++w) c[f] += src[w * RT * FT * 64];
            }
            finish(r, c);
        }
    } else {
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            f32x4 c[FT];
#pragma unroll
            for (int f = 0; f < FT; ++f) c[f] = acc[f][r];
            finish(r, c);
        }
    }
    if constexpr (EPI == EPI_RESID) {
        __syncthreads();
        if (tid < RT * 16 && r0 + tid < a.M) {
            float sum = 0.f;
            for (int w = 0; w < WN; ++w) sum += nss[w * (RT * 16) + tid];
            a.np_ssq[(size_t)fg * a.ssq_ld + r0 + tid] = sum;
        }
    }
}

// Embedding of many rows: the fp32 residual stream, its tile planes (times the first norm's gain) and the rows' sums of squares.
__global__ __launch_bounds__(256) void embed_tile_kernel(const EmbedArgs a, char* np, int np_tk) {
    __shared__ float part[4];
    const int t = (int)blockIdx.x, tid = threadIdx.x;
    const int base = (a.base_ptr ? *a.base_ptr : 0) + a.base_add, pos = base + t;
    const int row = (int)(((long long)a.tokens[pos] + a.tie_shift) % a.vocab);
    const double lg = log2(10000.0);
    float ss = 0.f;
    for (int k4 = tid; k4 < a.d / 4; k4 += 256) {
        const int k = k4 * 4;
        const char* p = (const char*)a.E.w + ((size_t)(row >> 4) * a.E.tk + (k >> 5)) * kTileBytes + ((row & 15) + 16 * ((k & 31) >> 3)) * 16 + (k & 7) * 2;
        const uint2 raw = *(const uint2*)p;
        const float e[4] = {bf2f(raw.x & 0xFFFFu), bf2f(raw.x >> 16), bf2f(raw.y & 0xFFFFu), bf2f(raw.y >> 16)};
        float v[4], w[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            float pterm = 0.f;
            if (a.sinusoidal) {
                if (a.pe) {
                    pterm = a.pe[(size_t)pos * a.d + k + j];
                } else {
                    const double ang = (double)pos * exp2(-(double)(2 * ((k + j) >> 1)) / (double)a.d * lg);
                    pterm = (float)(((k + j) & 1) ? cos(ang) : sin(ang));
                }
            }
            v[j] = __builtin_fmaf(e[j], a.embed_scale, pterm);
            ss += v[j] * v[j];
            w[j] = v[j] * a.nx_gain[k + j];
        }
        *(float4*)(a.x + (size_t)t * a.d + k) = make_float4(v[0], v[1], v[2], v[3]);
        put_tile_planes(np, np_tk, t, k, w);
    }
    const float tot = wave_sum(ss);
    if ((tid & 63) == 0) part[tid >> 6] = tot;
    __syncthreads();
    if (tid == 0) a.nx_ssq[t] = part[0] + part[1] + part[2] + part[3];
}

hipError_t launch_embed_tiles(const EmbedArgs& a, char* np, hipStream_t st) {
    if (!a.nx_gain || !a.nx_ssq || !np || a.d % 32 || a.T < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(embed_tile_kernel, dim3(a.T), dim3(256), 0, st, a, np, a.d / 32);
    return hipGetLastError();
}

__global__ __launch_bounds__(256) void row_tile_kernel(const RowCopyArgs a, const float* gain, char* np, int np_tk, float* ssq) {
    __shared__ float part[4];
    const int t = (int)blockIdx.x, tid = threadIdx.x;
    const float4* src = (const float4*)(a.src + (size_t)((a.src_row_ptr ? *a.src_row_ptr : 0) + a.src_row_add + t) * a.d);
    float4* dst = (float4*)(a.dst + (size_t)((a.dst_row_ptr ? *a.dst_row_ptr : 0) + a.dst_row_add + t) * a.d);
    float ss = 0.f;
    for (int i = tid; i < a.d / 4; i += 256) {
        const float4 v = src[i], g = *(const float4*)(gain + i * 4);
        if (a.dst) dst[i] = v;
        ss += v.x * v.x + v.y * v.y + v.z * v.z + v.w * v.w;
        const float w[4] = {v.x * g.x, v.y * g.y, v.z * g.z, v.w * g.w};
        put_tile_planes(np, np_tk, t, i * 4, w);
    }
    const float tot = wave_sum(ss);
    if ((tid & 63) == 0) part[tid >> 6] = tot;
    __syncthreads();
    if (tid == 0) ssq[t] = part[0] + part[1] + part[2] + part[3];
}

hipError_t launch_row_tiles(const RowCopyArgs& a, const float* gain, char* np, float* ssq, hipStream_t st) {
    if (!gain || !np || !ssq || a.d % 32 || a.T < 1) return hipErrorInvalidValue;
    hipLaunchKernelGGL(row_tile_kernel, dim3(a.T), dim3(256), 0, st, a, gain, np, a.d / 32, ssq);
    return hipGetLastError();
}

// cos and sin of position * base^(-2i / d_head), in double precision
__global__ __launch_bounds__(64) void rope_table_kernel(double2* table, int half, double base) {
    const int pos = (int)blockIdx.x;
    for (int i = threadIdx.x; i < half; i += 64) {
        const double fr = exp2(-(double)(2 * i) / (double)(2 * half) * log2(base));
        double sn, cs;
        sincos((double)pos * fr, &sn, &cs);
        table[(size_t)pos * half + i] = make_double2(cs, sn);
    }
}

hipError_t launch_rope_table(double2* table, int positions, int d_head, float base, hipStream_t st) {
    if (!table || positions < 1 || d_head < 2) return hipErrorInvalidValue;
    hipLaunchKernelGGL(rope_table_kernel, dim3(positions), dim3(64), 0, st, table, d_head / 2, (double)base);
    return hipGetLastError();
}

// Launch shapes.  `us` is what one step (32 inputs; with sliced inputs 32 per slice) of a workgroup takes when it has a
// compute unit to itself, measured over 64 .. 1531 rows x 512 .. 49152 features x 512 .. 11008 inputs: it follows the bytes
// a step pulls (8 to 48 KiB at 45 to 60 bytes a ns).  Workgroups that share a compute unit or follow each other on it take 0.8
// of that each.  The shape with the smallest total is taken: the wide shared tiles where there are enough of them, else
// smaller tiles and sliced inputs.  (1023 x 22016 x 4096: 285 us, 1.3 PFLOP/s issued of the 1.75 the matrix cores keep up on
// random operands; 512 x 1024 x 4096: 18.5 us; 64 x 1024 x 1024: 5.2 us.)
// Shapes of 96 rows x 192 or 256 features (shared) and of 48 x 128 (sliced, one workgroup per compute unit, `once` us for joining 24 tiles of sums) are
// for products that they cut into one round where the others make a round and a bit of another: 1531 rows, features x inputs, us, best of the others /
// with: 3072 x 1024 (256 workgroups of 96 x 192) 31.4 / 25.4, 4096 x 1024 (256 of 96 x 256) 31.0 / 27.4, 1024 x 4096 (256 of 48 x 128) 42.5 / 34.1, but
// 1024 x 1024 16.4 / 17.6.  Measured beside them and not taken: sliced, 96 x 64 as 48 x 128; 64 x 96, which gains 1 us at 512 x 3072 x 1024 alone; 64 x 128.
// One round is 32 workgroups on the busiest die, not 256 of them (features x inputs, rows, us, best of the others / with, 33 to 44 on that
// die): 768 x 3072, 2016 rows 29.5 / 44.4; 5632 x 1024 gated, 1056 28.4 / 38.0; 3072 x 1024, 2016 31.2 / 41.9; 4096 x 4096, 1056 97 / 105.
// Weights from memory are no reason against them: 12288 x 4096 rotary, 80, 352, 432 rows 43.7, 98.9, 100.5 / 40.2, 76.7, 92.8; 22016 x 4096 gated, 40 55.2 / 47.9;
// 4096 x 4096, 320 44.6 / 34.8; 4096 x 11008, 320 105.7 / 72.7; 6144 x 2048 rotary, 704 53.7 / 45.5; 2048 x 5504, 640 54.0 / 41.3; 11008 x 2048 gated, 464 51.5 / 45.1.
// The epilogue of so many sums is dear where there are few inputs, with the rotation in double precision above all, so there is a least number of input
// tiles (`from`, with rotation `turned`).  Ratio to the others, 1200 products of 128 to 11008 inputs drawn at random, 96 x 256: rotary 1.21 to 1.34 up to 1024 inputs,
// 1.07 to 1.16 at 1280 and 1536, 0.98 to 1.03 at 2048, 0.95 to 1.06 at 2560 to 3072, 0.88 to 0.94 at 4096; the others 0.96 to 1.14 up to 640, 0.77 to 1.00 from 768 on.
// 96 x 192: rotary 0.85 to 1.04 up to 768, 0.73 to 1.00 from 1024 on; the others 0.56 to 0.92.  48 x 128 (by its cost from 2560 inputs on) 0.67 to 0.98.
struct TileShape {
    int rt, ft, wk;
    bool share;
    float us, once;
    int from, turned;  // > 0: only where it makes one round, and from so many input tiles on
};
// Row shares of the dies (see tile_block): every feature share fetches all its rows, every row share all its weights; least bytes into the
// eight L2s, without leaving dies idle where there are few row blocks or feature groups.  Returns the workgroups of the busiest die.
static long die_shares(const TileGemmArgs& a, int rbs, int fgs, int& best) {
    long least = 0, most = 0;
    for (int gr = 1; gr <= 8; gr *= 2) {
        const int gf = 8 / gr;
        const long slots = (long)((rbs + gr - 1) / gr) * ((fgs + gf - 1) / gf);
        const long cost = (long)(gf * (long)a.M * 4 + gr * (long)a.W.n * 2) * (slots * 8 * 4 > 5 * (long)rbs * fgs ? 4 : 1) * 16 + slots;
        if (gr == 1 || cost < least) { least = cost; most = slots; best = gr; }
    }
    return most;
}
static TileShape tile_shape(const TileGemmArgs& a) {
    static const TileShape shapes[] = {{8, 4, 1, true, 0.94f, 0.f, 0, 0}, {4, 4, 1, true, 0.57f, 0.f, 0, 0}, {4, 4, 2, false, 0.84f, 0.f, 0, 0},
                                       {4, 4, 4, false, 0.80f, 0.f, 0, 0}, {4, 2, 4, false, 0.69f, 0.f, 0, 0}, {4, 1, 4, false, 0.60f, 0.f, 0, 0},
                                       {2, 4, 4, false, 0.56f, 0.f, 0, 0}, {2, 2, 4, false, 0.42f, 0.f, 0, 0}, {2, 1, 4, false, 0.36f, 0.f, 0, 0},
                                       {6, 4, 1, true, 0.83f, 0.f, 24, 128}, {6, 3, 1, true, 0.75f, 0.f, 1, 32}, {3, 8, 4, false, 0.70f, 11.f, 1, 1}};
    const bool gated = a.epi == EPI_ACT && a.act != BILD_ACT_RELU;
    const TileShape* best = nullptr;
    float least = 0.f;
    for (const TileShape& t : shapes) {
        if (gated && t.ft % 2) continue;
        const int rows = t.rt * 16, feats = t.ft * (kTileWaves / t.wk);
        const int rbs = (a.M + rows - 1) / rows, fgs = (a.W.tn + feats - 1) / feats, rounds = (rbs * fgs + 255) / 256;
        int gr;
        if (t.from > 0 && (a.W.tk < (a.rope ? t.turned : t.from) || die_shares(a, rbs, fgs, gr) > 32)) continue;
        const float us = (float)((a.W.tk + t.wk - 1) / t.wk) * t.us * (rounds == 1 ? 1.f : 0.8f * (float)rounds) + t.once;
        if (!best || us < least) { best = &t; least = us; }
    }
    return *best;
}

int tile_gemm_parts(const TileGemmArgs& a) {
    const TileShape t = tile_shape(a);
    const int per = t.ft * (kTileWaves / t.wk);
    return (a.W.tn + per - 1) / per;
}

void tile_gemm_shape(const TileGemmArgs& a, int (&out)[5]) {
    const TileShape t = tile_shape(a);
    const int rows = t.rt * 16;
    int gr;
    const long most = die_shares(a, (a.M + rows - 1) / rows, tile_gemm_parts(a), gr);
    const int o[5] = {rows, t.ft * (kTileWaves / t.wk) * 16, t.wk, t.share, (int)most};
    std::copy(o, o + 5, out);
}

hipError_t gemm_tile_init() {
    static hipError_t done = [] {
#define BILD_T(RTV, FTV, EPIV, ROPEV, GV, SP, SH) (const void*)gemm_tile_kernel<RTV, FTV, EPIV, ROPEV, GV, SP, SH>
#define BILD_TF(EPIV, ROPEV)                                                                                                 \
    BILD_T(8, 4, EPIV, ROPEV, false, false, true), BILD_T(4, 4, EPIV, ROPEV, false, false, true),                            \
    BILD_T(2, 4, EPIV, ROPEV, false, true, false), BILD_T(2, 2, EPIV, ROPEV, false, true, false),                            \
    BILD_T(2, 1, EPIV, ROPEV, false, true, false), BILD_T(4, 4, EPIV, ROPEV, false, true, false),                            \
    BILD_T(4, 2, EPIV, ROPEV, false, true, false), BILD_T(4, 1, EPIV, ROPEV, false, true, false),                            \
    BILD_T(6, 4, EPIV, ROPEV, false, false, true), BILD_T(6, 3, EPIV, ROPEV, false, false, true),                            \
    BILD_T(3, 8, EPIV, ROPEV, false, true, false)
        const void* fns[] = {BILD_TF(EPI_RESID, 0), BILD_TF(EPI_ACT, 0), BILD_TF(EPI_QKV, 0), BILD_TF(EPI_QKV, 1),
                             BILD_T(8, 4, EPI_ACT, 0, true, false, true), BILD_T(4, 4, EPI_ACT, 0, true, false, true),
                             BILD_T(2, 4, EPI_ACT, 0, true, true, false), BILD_T(2, 2, EPI_ACT, 0, true, true, false),
                             BILD_T(4, 4, EPI_ACT, 0, true, true, false), BILD_T(4, 2, EPI_ACT, 0, true, true, false),
                             BILD_T(6, 4, EPI_ACT, 0, true, false, true), BILD_T(3, 8, EPI_ACT, 0, true, true, false)};
#undef BILD_TF
#undef BILD_T
        return raise_lds_limit(fns, 160 * 1024);
    }();
    return done;
}

hipError_t launch_gemm_tile(const TileGemmArgs& a0, hipStream_t st) {
    if (hipError_t e = gemm_tile_init(); e != hipSuccess) return e;
    TileGemmArgs a = a0;
    const TileShape t = tile_shape(a);
    a.wk = t.wk;
    a.lwk = a.wk == 4 ? 2 : a.wk - 1;
    const bool gated = a.epi == EPI_ACT && a.act != BILD_ACT_RELU;
    const bool norm = a.epi != EPI_RESID;
    if (a.M < 1 || !a.xp || a.W.tk < 1 || (norm && (!a.ssq || a.ssq_parts < 1))) return hipErrorInvalidValue;
    if ((a.epi == EPI_RESID && (!a.x || !a.np || !a.np_gain || !a.np_ssq)) || (a.epi == EPI_ACT && !a.np)) return hipErrorInvalidValue;
    if (a.epi == EPI_QKV && (!a.k_cache || !a.v_cache || a.layer_n < 1 || (a.q_dim > 0 && !a.q_out))) return hipErrorInvalidValue;
    const int rows = t.rt * 16;
    a.fgs = tile_gemm_parts(a);
    a.rbs = (a.M + rows - 1) / rows;
    const dim3 grid((unsigned)(8 * die_shares(a, a.rbs, a.fgs, a.gr))), block(64 * kTileWaves);
    // (shared forms: what the largest needs; 16 KiB for 64 rows without spreading: 1531 x 1024 inputs the same, 1290 an encode 0.7 % slower)
    const size_t smem = (size_t)tile_sums(t.rt) * 4 + (t.share ? (size_t)32 * 1024 : a.wk > 1 ? (size_t)kTileWaves * t.rt * t.ft * 1024 : 0);
#define BILD_T(RTV, FTV, EPIV, ROPEV, GV, SP, SH)                                                                            \
    do {                                                                                                                     \
        hipLaunchKernelGGL((gemm_tile_kernel<RTV, FTV, EPIV, ROPEV, GV, SP, SH>), grid, block, smem, st, a);                 \
        return hipGetLastError();                                                                                            \
    } while (0)
#define BILD_TF(EPIV, ROPEV)                                                                                                 \
    do {                                                                                                                     \
        if (t.share && t.rt == 8) BILD_T(8, 4, EPIV, ROPEV, false, false, true);                                             \
        if (t.share && t.rt == 6 && t.ft == 4) BILD_T(6, 4, EPIV, ROPEV, false, false, true);                                \
        if (t.share && t.rt == 6) BILD_T(6, 3, EPIV, ROPEV, false, false, true);                                             \
        if (t.rt == 3) BILD_T(3, 8, EPIV, ROPEV, false, true, false);                                                        \
        if (t.share) BILD_T(4, 4, EPIV, ROPEV, false, false, true);                                                          \
        if (t.rt == 2 && t.ft == 4) BILD_T(2, 4, EPIV, ROPEV, false, true, false);                                           \
        if (t.rt == 2 && t.ft == 2) BILD_T(2, 2, EPIV, ROPEV, false, true, false);                                           \
        if (t.rt == 2) BILD_T(2, 1, EPIV, ROPEV, false, true, false);                                                        \
        if (t.ft == 4) BILD_T(4, 4, EPIV, ROPEV, false, true, false);                                                        \
        if (t.ft == 2) BILD_T(4, 2, EPIV, ROPEV, false, true, false);                                                        \
        BILD_T(4, 1, EPIV, ROPEV, false, true, false);                                                                       \
    } while (0)
    switch (a.epi) {
        case EPI_RESID: BILD_TF(EPI_RESID, 0); break;
        case EPI_ACT:
            if (!gated) BILD_TF(EPI_ACT, 0);
            if (t.share && t.rt == 8) BILD_T(8, 4, EPI_ACT, 0, true, false, true);
            if (t.share && t.rt == 6) BILD_T(6, 4, EPI_ACT, 0, true, false, true);
            if (t.rt == 3) BILD_T(3, 8, EPI_ACT, 0, true, true, false);
            if (t.share) BILD_T(4, 4, EPI_ACT, 0, true, false, true);
            if (t.rt == 2 && t.ft == 4) BILD_T(2, 4, EPI_ACT, 0, true, true, false);
            if (t.rt == 2) BILD_T(2, 2, EPI_ACT, 0, true, true, false);
            if (t.ft == 4) BILD_T(4, 4, EPI_ACT, 0, true, true, false);
            BILD_T(4, 2, EPI_ACT, 0, true, true, false);
            break;
        case EPI_QKV:
            if (a.rope) BILD_TF(EPI_QKV, 1); else BILD_TF(EPI_QKV, 0);
            break;
        default: break;
    }
#undef BILD_TF
#undef BILD_T
    return hipErrorInvalidValue;
}

}  // namespace bild
