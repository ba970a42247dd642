// Attention of bf16 models over a long cache, up to 32 query rows.
//
// Bound: the trip of keys and values from memory and the instruction chain behind it.  A workgroup has one head and a range of its
// keys (about one workgroup per compute unit), a wave 32 keys at a time: it asks for its keys and values first and for the queries
// behind them, straight into operand registers, so that nothing is staged; the waves' results are joined through LDS, and the
// workgroups' by the last one of a head to arrive (last_in.h), which spares a kernel for joining, or a projection that joins while it
// stages.  Up to eight rows one operand holds the high parts of the queries (and weights) in its columns 0 .. 7 and the low parts in
// 8 .. 15, as in pass_kernel.hip.
//
// 7B shape over 1064 keys, us per layer: 8 rows 9.6 + 4.8 for the kernel that joined -> 11.3, 32 rows 12.1 + 4.9 -> 14.6; one row 8.6 and
// a projection of 10.0 that joined -> 10.7 and 8.3.  More than eight splits of a head cost a second round of reads when they are
// joined (16 heads, 1064 keys: 664 us a pass with 8 splits, 692 with 16; 4137 keys 791, 756): they are taken from 2049 keys on.
#include "attn_split.h"

#include <algorithm>

#include "last_in.h"

namespace bild {

// R: row tiles; PACK: up to eight rows
template <int DH32, int R, bool PACK>
__global__ __launch_bounds__(512, 1) void attn_split_kernel(const void* __restrict__ h_k, const void* __restrict__ h_v, const float* __restrict__ h_q, const int* __restrict__ h_len,
                                                            const int h_dim, const int h_vcap, const int h_geom, const float h_scale, const AttnSplitArgs a0) {
    // (the first requests' arguments arrive in scalar registers, the structure is fetched for the rest)
    AttnSplitArgs a = a0;
    a.k = h_k; a.v = h_v; a.q = h_q; a.len_ptr = h_len; a.i_dim = h_dim; a.vcap = h_vcap; a.scale = h_scale;
    a.T = h_geom & 63; a.splits = (h_geom >> 6) & 31; a.waves = (h_geom >> 11) & 15; a.causal = h_geom >> 15;
    constexpr int DT16 = DH32 * 2, DH = DH32 * 32, P = PACK ? 1 : 2;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), nw = a.waves;
    const int tok = lane & 15, g = lane >> 4, h = (int)blockIdx.x, split = (int)blockIdx.y;
    f32x4* co = (f32x4*)smem;                            // [wave][R * DT16][64]
    float* cm = (float*)(co + nw * R * DT16 * 64);       // [wave][R * 16] maxima, then sums
    float* cl = cm + nw * R * 16;
    unsigned* share = (unsigned*)(cl + nw * R * 16);
    const __amdgpu_buffer_rsrc_t kr = make_rsrc((const char*)a.k + (size_t)h * DH * 2, 0xFFFFFFFFu),
                                 vr = make_rsrc((const char*)a.v + (size_t)h * DH * a.vcap * 2, 0xFFFFFFFFu), qr = make_rsrc(a.q + h * DH, 0xFFFFFFFFu);
    const int ko = (tok * a.i_dim + g * 8) * 2, vo = (tok * a.vcap + g * 4) * 2;
    uint4 K[2][DH32], V[DT16];
    auto load = [&](int blk) {
        const int key = min(blk, (a.vcap >> 5) - 1) * 32;  // (blocks past the last key are read, inside the cache, and dropped)
#pragma unroll
        for (int ab = 0; ab < 2; ++ab)
#pragma unroll
            for (int ks = 0; ks < DH32; ++ks) K[ab][ks] = buf_load(kr, (unsigned)ko, ((key + ab * 16) * a.i_dim + ks * 32) * 2);
#pragma unroll
        for (int dt = 0; dt < DT16; ++dt) {
            const int off = (dt * 16 * a.vcap + key) * 2;
            const uint2 x = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(vr, vo, off, 0));
            const uint2 y = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(vr, vo + 32, off, 0));
            V[dt] = make_uint4(x.x, x.y, y.x, y.y);
        }
    };
    float m_run[R], l_run[R];
    f32x4 O[R][DT16];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        m_run[r] = -INFINITY;
        l_run[r] = 0.f;
#pragma unroll
        for (int dt = 0; dt < DT16; ++dt) O[r][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    // this wave's blocks of 32 keys: every (splits x waves)th, so that the first is known before the number of keys is
    const int mine = split + wave * a.splits, step = nw * a.splits;
    load(mine);
    __builtin_amdgcn_sched_barrier(0);
    const int len = *a.len_ptr, nkeys = a.causal ? len + a.T : len, nblk = (nkeys + 31) >> 5;
    if (mine < nblk) {
        // high and low parts of eight values in operand order
        auto parts = [&](const float (&v)[8], bf16x8 (&o)[P]) {
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) split_bf16x2(v[2 * j], v[2 * j + 1], hi[j], lo[j]);
            if constexpr (PACK) {
                const bool low = tok >= 8;
                o[0] = __builtin_bit_cast(bf16x8, make_uint4(low ? lo[0] : hi[0], low ? lo[1] : hi[1], low ? lo[2] : hi[2], low ? lo[3] : hi[3]));
            } else {
                o[0] = __builtin_bit_cast(bf16x8, make_uint4(hi[0], hi[1], hi[2], hi[3]));
                o[P - 1] = __builtin_bit_cast(bf16x8, make_uint4(lo[0], lo[1], lo[2], lo[3]));
            }
        };
        bf16x8 Q[R][DH32][P];
        int lim[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int row = min(PACK ? tok & 7 : r * 16 + tok, a.T - 1);
            lim[r] = a.causal ? len + row : nkeys - 1;
            float4 qv[DH32][2];
#pragma unroll
            for (int ks = 0; ks < DH32; ++ks)
#pragma unroll
                for (int p = 0; p < 2; ++p) qv[ks][p] = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(qr, (row * a.i_dim + g * 8) * 4, ks * 128 + p * 16, 0));
#pragma unroll
            for (int ks = 0; ks < DH32; ++ks) {
                const float v[8] = {qv[ks][0].x * a.scale, qv[ks][0].y * a.scale, qv[ks][0].z * a.scale, qv[ks][0].w * a.scale,
                                    qv[ks][1].x * a.scale, qv[ks][1].y * a.scale, qv[ks][1].z * a.scale, qv[ks][1].w * a.scale};
                parts(v, Q[r][ks]);
            }
        }
        const int safe = a.causal ? len : nkeys - 1;  // keys every row sees
#pragma unroll 1
        for (int blk = mine; blk < nblk; blk += step) {
            bf16x8 W[R][P];
#pragma unroll
            for (int r = 0; r < R; ++r) {
                f32x4 s[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                for (int ks = 0; ks < DH32; ++ks)
#pragma unroll
                    for (int p = 0; p < P; ++p)
#pragma unroll
                        for (int ab = 0; ab < 2; ++ab) s[ab] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, K[ab][ks]), Q[r][ks][p], s[ab], 0, 0, 0);
                float p[8];
#pragma unroll
                for (int v = 0; v < 8; ++v) {
                    p[v] = s[v >> 2][v & 3];
                    if constexpr (PACK) p[v] += dpp_f<0x128, 0xF>(0.f, p[v]);
                }
                if (blk * 32 + 31 > safe) {
#pragma unroll
                    for (int v = 0; v < 8; ++v)
                        if (blk * 32 + (v >> 2) * 16 + g * 4 + (v & 3) > lim[r]) p[v] = -INFINITY;
                }
                float top = m_run[r];
#pragma unroll
                for (int v = 0; v < 8; ++v) top = fmaxf(top, p[v]);
                const float m_new = quad_rows_max(top), base = m_new == -INFINITY ? 0.f : m_new;
                float sum = 0.f;
#pragma unroll
                for (int v = 0; v < 8; ++v) {
                    p[v] = fexp(p[v] - base);
                    sum += p[v];
                }
                const float f = fexp(m_run[r] - base);
                l_run[r] = l_run[r] * f + quad_rows_sum(sum);
#pragma unroll
                for (int dt = 0; dt < DT16; ++dt) O[r][dt] *= f;
                m_run[r] = m_new;
                parts(p, W[r]);
            }
#pragma unroll
            for (int dt = 0; dt < DT16; ++dt)
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int p = 0; p < P; ++p) O[r][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, V[dt]), W[r][p], O[r][dt], 0, 0, 0);
            if (blk + step < nblk) load(blk + step);
        }
    }
    // ---- the waves' results (every wave's: one without keys has a maximum of minus infinity and zeros) ----
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (g == 0) {
            cm[wave * (R * 16) + r * 16 + tok] = m_run[r];
            cl[wave * (R * 16) + r * 16 + tok] = l_run[r];
        }
#pragma unroll
        for (int dt = 0; dt < DT16; ++dt) co[(wave * (R * DT16) + r * DT16 + dt) * 64 + lane] = O[r][dt];
    }
    lds_barrier();
    const __amdgpu_buffer_rsrc_t part = make_rsrc(a.part, kAttnSplitFloats * sizeof(float));
    constexpr int UNITS = R * DT16, ROOM = UNITS * 1024 + R * 128;  // bytes per workgroup: the units, then (maximum, sum) per row
    const int at = (h * a.splits + split) * ROOM;
    for (int u = wave; u < UNITS; u += nw) {
        const int r = u / DT16;
        float M = -INFINITY, L = 0.f;
        f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
        float w[8], l[8];
        f32x4 p[8];
#pragma unroll
        for (int v = 0; v < 8; ++v) {  // (four waves: the surplus reads are of the last wave and dropped)
            const int c = min(v, nw - 1);
            w[v] = cm[c * (R * 16) + r * 16 + tok];
            l[v] = cl[c * (R * 16) + r * 16 + tok];
            p[v] = co[(c * UNITS + u) * 64 + lane];
        }
#pragma unroll
        for (int v = 0; v < 8; ++v) M = fmaxf(M, w[v]);
        const float base = M == -INFINITY ? 0.f : M;
#pragma unroll
        for (int v = 0; v < 8; ++v) {
            w[v] = v < nw ? fexp(w[v] - base) : 0.f;
            L += l[v] * w[v];
            o += p[v] * w[v];
        }
        if constexpr (PACK) {
#pragma unroll
            for (int v = 0; v < 4; ++v) o[v] += dpp_f<0x128, 0xF>(0.f, o[v]);
        }
        if (a.splits > 1) {
            typedef unsigned v4u __attribute__((ext_vector_type(4)));
            typedef unsigned v2u __attribute__((ext_vector_type(2)));
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, o), part, at + u * 1024 + lane * 16, 0, kPartAux);
            if (u % DT16 == 0 && g == 0) __builtin_amdgcn_raw_buffer_store_b64(v2u{__float_as_uint(M), __float_as_uint(L)}, part, at + UNITS * 1024 + (r * 16 + tok) * 8, 0, kPartAux);
        } else {
            const int t = r * 16 + tok, n = h * DH + (u % DT16) * 16 + g * 4;
            const float inv = 1.f / L, x[4] = {o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv};
            if (t < a.T) {
                if (a.ob_t) put_tile_planes(a.ob_t, a.i_dim >> 5, t, n, x);
                else st_act4(a.out + (size_t)t * a.i_dim + n, make_float4(x[0], x[1], x[2], x[3]));
            }
        }
    }
    if (a.splits == 1 || !last_in(a.arrived + h, (unsigned)a.splits, share)) return;
    const int head = h * a.splits * ROOM;
    for (int u = wave; u < UNITS; u += nw) {
        const int r = u / DT16;
        float M = -INFINITY, L = 0.f;
        f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int s0 = 0; s0 < a.splits; s0 += 8) {
            uint2 ml[8];
            f32x4 p[8];
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const int c = head + min(s0 + s, a.splits - 1) * ROOM;
                ml[s] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(part, UNITS * 1024 + (r * 16 + tok) * 8, c, kPartAux));
                p[s] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(part, u * 1024 + lane * 16, c, kPartAux));
            }
            float top = M;
#pragma unroll
            for (int s = 0; s < 8; ++s) top = fmaxf(top, __uint_as_float(ml[s].x));
            const float base = top == -INFINITY ? 0.f : top, f = fexp_full(M - base);
            M = top;
            L *= f;
            o *= f;
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const float w = s0 + s < a.splits ? fexp_full(__uint_as_float(ml[s].x) - base) : 0.f;
                L += __uint_as_float(ml[s].y) * w;
                o += p[s] * w;
            }
        }
        const int t = r * 16 + tok, n = h * DH + (u % DT16) * 16 + g * 4;
        const float inv = 1.f / L, x[4] = {o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv};
        if (t < a.T) {
            if (a.ob_t) put_tile_planes(a.ob_t, a.i_dim >> 5, t, n, x);
            else st_act4(a.out + (size_t)t * a.i_dim + n, make_float4(x[0], x[1], x[2], x[3]));
        }
    }
}

void attn_split_shape(int heads, int d_head, int i_dim, int vcap, int keys, int* splits, int* waves) {
    *splits = *waves = 0;
    if ((d_head != 64 && d_head != 128) || heads < 1 || heads > kAttnSplitHeads || !cache_in_int(vcap, i_dim, 2)) return;
    const int blocks = (keys + 31) / 32;
    int s = 1;
    while (heads * s * 2 <= 256 && s < 16 && blocks > s * (s < 8 ? 4 : 8)) s *= 2;
    *splits = s;
    *waves = (blocks + s - 1) / s <= 4 ? 4 : 8;
}

template <int DH32, int R, bool PACK>
static hipError_t launch_split(const AttnSplitArgs& a, hipStream_t st) {
    const size_t smem = (size_t)a.waves * R * (DH32 * 2 * 1024 + 128) + 16;
    hipLaunchKernelGGL((attn_split_kernel<DH32, R, PACK>), dim3(a.heads, a.splits), dim3(64 * a.waves), smem, st, a.k, a.v, a.q, a.len_ptr, a.i_dim, a.vcap,
                       a.T | a.splits << 6 | a.waves << 11 | (a.causal ? 1 << 15 : 0), a.scale, a);
    return hipGetLastError();
}
hipError_t attn_split_init() {
    static hipError_t done = [] {
        const void* fns[] = {(const void*)attn_split_kernel<2, 1, true>, (const void*)attn_split_kernel<2, 1, false>, (const void*)attn_split_kernel<2, 2, false>,
                             (const void*)attn_split_kernel<4, 1, true>, (const void*)attn_split_kernel<4, 1, false>, (const void*)attn_split_kernel<4, 2, false>};
        return raise_lds_limit(fns, 160 * 1024);
    }();
    return done;
}
hipError_t launch_attn_split(const AttnSplitArgs& a, hipStream_t st) {
    if (hipError_t e = attn_split_init(); e != hipSuccess) return e;
    if (a.T < 1 || a.T > kMaxRows || (a.d_head != 64 && a.d_head != 128) || a.splits < 1 || a.heads * a.splits > kAttnSplitGroups || a.heads > kAttnSplitHeads ||
        (a.waves != 4 && a.waves != 8) || a.splits > 16 || a.vcap < 32 || a.vcap % 32 || !cache_in_int(a.vcap, a.i_dim, 2) || !a.q || !a.k || !a.v || !a.len_ptr || (!a.out && !a.ob_t) || (a.splits > 1 && (!a.part || !a.arrived)))
        return hipErrorInvalidValue;
#define BILD_D(DHV) (a.T <= 8 ? launch_split<DHV, 1, true>(a, st) : a.T <= 16 ? launch_split<DHV, 1, false>(a, st) : launch_split<DHV, 2, false>(a, st))
    return a.d_head == 64 ? BILD_D(2) : BILD_D(4);
#undef BILD_D
}

}  // namespace bild
