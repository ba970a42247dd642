// Attention of bf16 models for MANY query rows (more than 32: encoder, prompt prefill), between the projections of
// gemm_tile.hip: q in fp32, K [position][I] and V^T [I][capacity] as the projection left them, output as tile planes.
//
// One workgroup per (head, 64 query rows); each of its four waves owns 16 rows and walks ALL keys, 64 at a time, so nothing
// is merged across waves.  The 64 keys' K and V^T go through LDS once for the four waves (two buffers, the next block is
// on its way while the current one is multiplied), in matrix-core A-operand order: every LDS access is 16 contiguous bytes
// per lane.  q stays in registers as the B operand, high and low bf16 part, times 1/sqrt(d_head) and log2(e), so that
// probabilities are bare base-2 exponentials.  The score tile leaves the matrix core in the B-operand order of the second
// product (contraction index 8g + j is key 4g + j of the first 16 keys for j < 4, of the second 16 for j >= 4), so
// probabilities never cross lanes.
//
// Bound: vector ALU (the exponentials and the split of P, about 130 instructions per 64 keys and 16 rows against 32
// matrix instructions).  The kernel before it gave 32 rows to eight waves that split the keys and merged: each such
// workgroup fetched all K/V for 32 rows and paid staging and merge of q, m, l, O in LDS.
#include "kernel_common.h"

namespace bild {

template <int DH32, bool REL>
__global__ __launch_bounds__(256, 2) void attn_tile_kernel(const AttnArgs a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    constexpr int DT16 = DH32 * 2, KB = 4 * DH32 * 1024, BUF = 2 * KB;  // bytes of K (and of V^T) per 64 keys
    constexpr float kLog2e = 1.4426950408889634f;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tok_l = lane & 15, g = lane >> 4;
    const int h = (int)blockIdx.x, I = a.i_dim, dh = a.d_head, T = a.T;
    const int rb = a.causal ? (int)(gridDim.y - 1 - blockIdx.y) : (int)blockIdx.y;  // (the longest causal rows start first)
    const int r0 = rb * 64, rw = r0 + wave * 16;
    const int base = a.causal ? *a.len_ptr + a.base_add : 0;
    const int nkeys = a.causal ? min(base + T, base + r0 + 64) : a.nkeys_fixed;  // keys any row of this workgroup sees
    const int nblk = (nkeys + 63) >> 6;
    const int t = min(rw + tok_l, T - 1);
    const int lim = a.causal ? base + t : nkeys - 1;             // last key this lane's row sees
    const int lim_min = a.causal ? base + min(rw, T - 1) : nkeys - 1;  // ... the wave's first row: blocks up to it need no mask
    float* relb = (float*)(smem + 2 * BUF);
    const int nrel = 2 * a.rel_d + 1;

    const __amdgpu_buffer_rsrc_t kr = make_rsrc((const uint16_t*)a.k + (size_t)h * dh, 0xFFFFFFFFu);
    const __amdgpu_buffer_rsrc_t vr = make_rsrc((const uint16_t*)a.v + (size_t)h * dh * a.vcap, 0xFFFFFFFFu);
    // this wave fetches the K of keys 16 wave .. + 15 of a block and a quarter of its V^T
    uint4 K0[DH32], K1[DH32];
    uint2 V0[DH32][2], V1[DH32][2];
    auto request = [&](uint4 (&Kn)[DH32], uint2 (&Vn)[DH32][2], int blk) {
        const int key = min(blk * 64 + wave * 16 + tok_l, a.vcap - 1);  // (the caches hold whole blocks of 32 positions)
#pragma unroll
        for (int ks = 0; ks < DH32; ++ks)
            Kn[ks] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(kr, (key * I + min(ks * 32 + g * 8, dh - 8)) * 2, 0, 0));
#pragma unroll
        for (int i = 0; i < DH32; ++i) {
            const int u = wave * DH32 + i, b2 = u / DT16, dt = u % DT16;  // unit: 32 keys x 16 dims
            const int d = min(dt * 16 + tok_l, dh - 1);
            const int k0 = min(blk * 64 + b2 * 32, a.vcap - 32) + g * 4;
            Vn[i][0] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(vr, (d * a.vcap + k0) * 2, 0, 0));
            Vn[i][1] = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(vr, (d * a.vcap + k0 + 16) * 2, 0, 0));
        }
    };
    auto store = [&](const uint4 (&Kn)[DH32], const uint2 (&Vn)[DH32][2], int buf) {
        char* kb = smem + buf * BUF + lane * 16;
#pragma unroll
        for (int ks = 0; ks < DH32; ++ks) *(uint4*)(kb + (wave * DH32 + ks) * 1024) = Kn[ks];
#pragma unroll
        for (int i = 0; i < DH32; ++i)
            *(uint4*)(kb + KB + (wave * DH32 + i) * 1024) = make_uint4(Vn[i][0].x, Vn[i][0].y, Vn[i][1].x, Vn[i][1].y);
    };
    request(K0, V0, 0);
    __builtin_amdgcn_sched_barrier(0);
    request(K1, V1, min(1, nblk - 1));
    bf16x8 Qh[DH32], Ql[DH32];
    {
        const float sc = a.scale * kLog2e;
#pragma unroll
        for (int ks = 0; ks < DH32; ++ks) {
            const int d0 = ks * 32 + g * 8;
            const float* qp = a.q + (size_t)t * I + h * dh + min(d0, dh - 8);
            const float4 q0 = *(const float4*)qp, q1 = *(const float4*)(qp + 4);
            const float z = d0 < dh ? sc : 0.f;
            uint32_t hi[4], lo[4];
            split_bf16x2(q0.x * z, q0.y * z, hi[0], lo[0]);
            split_bf16x2(q0.z * z, q0.w * z, hi[1], lo[1]);
            split_bf16x2(q1.x * z, q1.y * z, hi[2], lo[2]);
            split_bf16x2(q1.z * z, q1.w * z, hi[3], lo[3]);
            Qh[ks] = __builtin_bit_cast(bf16x8, make_uint4(hi[0], hi[1], hi[2], hi[3]));
            Ql[ks] = __builtin_bit_cast(bf16x8, make_uint4(lo[0], lo[1], lo[2], lo[3]));
        }
    }
    if constexpr (REL)
        for (int i = tid; i < nrel; i += 256) relb[i] = a.rel_bias[(size_t)h * nrel + i] * kLog2e;
    const int qpos = (a.causal ? base : a.base_add) + t;

    // m_run is subtracted in the accumulators the products start from; it follows the row's maximum only when that has
    // grown by more than 2^6 (or for the first block), so most blocks neither rescale O nor subtract: probabilities stay below
    // 64, the quotient is the same.  The row sums are one more product, with a tile of ones: of the weights' high and low bf16
    // parts (17 bits or more), not of the weights themselves, accumulated in fp32.  O is made of the same parts, so that what a
    // weight loses cancels in the quotient: error of an output row against 64 bits, sums of the weights / of their parts, scores of
    // standard deviation 0.5, 2, 5 (simulated, 60 rows each, 2-norms): 8 keys 1.68e-6 / 1.58e-6, 9.7e-7 / 9.1e-7, 4.7e-7 / 4.5e-7;
    // 512 keys 2.43e-6 / 2.42e-6, 1.65e-6 / 1.61e-6, 9.6e-7 / 9.2e-7; 1531 keys 2.39e-6 / 2.39e-6, 1.73e-6 / 1.71e-6, 9.5e-7 / 9.1e-7;
    // 4097 keys 2.54e-6 / 2.54e-6, 1.92e-6 / 1.91e-6, 1.09e-6 / 1.08e-6; the worst row never larger.
    float m_run = 0.f;
    f32x4 O[DT16], L = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int dt = 0; dt < DT16; ++dt) O[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bf16x8 ones = __builtin_bit_cast(bf16x8, make_uint4(0x3F803F80u, 0x3F803F80u, 0x3F803F80u, 0x3F803F80u));
    auto block = [&](int blk) {
        const char* kb = smem + (blk & 1) * BUF + lane * 16;
        const int key0 = blk * 64;
        if (a.causal && key0 > base + min(rw + 15, T - 1)) return;  // (wave-uniform) no row of this wave sees the block
        // All operands of the block are read ahead and the products dealt round the accumulators: left to itself the compiler
        // reads each operand in front of its use and chains the four products of a tile, so that one wave waits for LDS and
        // for the matrix core most of the time (39 us at 1531 rows, whatever else was taken out of the loop).
        bf16x8 Ak[4][DH32];
#pragma unroll
        for (int ks = 0; ks < DH32; ++ks)
#pragma unroll
            for (int c = 0; c < 4; ++c) Ak[c][ks] = __builtin_bit_cast(bf16x8, *(const uint4*)(kb + (c * DH32 + ks) * 1024));
        f32x4 s[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) s[c] = f32x4{-m_run, -m_run, -m_run, -m_run};
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < DH32; ++ks) {
#pragma unroll
            for (int c = 0; c < 4; ++c) s[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ak[c][ks], Ql[ks], s[c], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int c = 0; c < 4; ++c) s[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Ak[c][ks], Qh[ks], s[c], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        bf16x8 Av[2][DT16];
#pragma unroll
        for (int b2 = 0; b2 < 2; ++b2)
#pragma unroll
            for (int dt = 0; dt < DT16; ++dt) Av[b2][dt] = __builtin_bit_cast(bf16x8, *(const uint4*)(kb + KB + (b2 * DT16 + dt) * 1024));
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (REL) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int dist = max(-a.rel_d, min(a.rel_d, key0 + c * 16 + g * 4 + v - qpos));
                    s[c][v] += relb[a.rel_d + dist];
                }
        }
        if (key0 + 63 > lim_min) {
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    if (key0 + c * 16 + g * 4 + v > lim) s[c][v] = -INFINITY;
        }
        float tmax = s[0][0];
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) tmax = fmaxf(tmax, s[c][v]);
        if (blk == 0 || __builtin_amdgcn_ballot_w64(tmax > 6.f)) {
            tmax = quad_rows_max(tmax);
            const float up = blk == 0 ? tmax : fmaxf(tmax, 0.f);  // (block 0: every row sees key 0)
            const float f = __builtin_amdgcn_exp2f(-up);
            m_run += up;
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int v = 0; v < 4; ++v) s[c][v] -= up;
#pragma unroll
            for (int dt = 0; dt < DT16; ++dt) O[dt] *= f;
            L *= f;
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) s[c][v] = __builtin_amdgcn_exp2f(s[c][v]);
#pragma unroll
        for (int b2 = 0; b2 < 2; ++b2) {
            uint32_t ph[4], pl[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) split_bf16x2(s[b2 * 2 + (j >> 1)][(j & 1) * 2], s[b2 * 2 + (j >> 1)][(j & 1) * 2 + 1], ph[j], pl[j]);
            const bf16x8 Ph = __builtin_bit_cast(bf16x8, make_uint4(ph[0], ph[1], ph[2], ph[3]));
            const bf16x8 Pl = __builtin_bit_cast(bf16x8, make_uint4(pl[0], pl[1], pl[2], pl[3]));
            __builtin_amdgcn_sched_barrier(0);
            L = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, Ph, L, 0, 0, 0);
#pragma unroll
            for (int dt = 0; dt < DT16; ++dt) O[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Av[b2][dt], Ph, O[dt], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            L = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, Pl, L, 0, 0, 0);
#pragma unroll
            for (int dt = 0; dt < DT16; ++dt) O[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Av[b2][dt], Pl, O[dt], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    store(K0, V0, 0);
    lds_barrier();
    for (int blk = 0; blk < nblk; blk += 2) {  // (blocks past the end are requested again, never multiplied)
        request(K0, V0, min(blk + 2, nblk - 1));
        __builtin_amdgcn_sched_barrier(0);
        block(blk);
        store(K1, V1, 1);
        lds_barrier();
        request(K1, V1, min(blk + 3, nblk - 1));
        __builtin_amdgcn_sched_barrier(0);
        if (blk + 1 < nblk) block(blk + 1);
        store(K0, V0, 0);
        lds_barrier();
    }
    const float inv = 1.f / L[0];
    if (rw + tok_l < T) {
#pragma unroll
        for (int dt = 0; dt < DT16; ++dt) {
            const int d0 = dt * 16 + g * 4;
            if (d0 >= dh) continue;
            const float w[4] = {O[dt][0] * inv, O[dt][1] * inv, O[dt][2] * inv, O[dt][3] * inv};
            put_tile_planes(a.ob_t, I >> 5, rw + tok_l, h * dh + d0, w);
        }
    }
}

hipError_t attn_tile_init() {
    static hipError_t done = [] {
        const void* fns[] = {(const void*)attn_tile_kernel<1, false>, (const void*)attn_tile_kernel<2, false>, (const void*)attn_tile_kernel<4, false>,
                             (const void*)attn_tile_kernel<1, true>, (const void*)attn_tile_kernel<2, true>, (const void*)attn_tile_kernel<4, true>};
        return raise_lds_limit(fns, 160 * 1024);
    }();
    return done;
}

hipError_t launch_attention_tile(const AttnArgs& a, hipStream_t st) {
    if (hipError_t e = attn_tile_init(); e != hipSuccess) return e;
    if (a.T < 1 || !a.ob_t || !a.len_ptr || a.heads < 1 || a.d_head < 8 || a.d_head > 128 || a.d_head % 8 || a.vcap < 32 || a.vcap % 32 ||
        (!a.causal && (a.nkeys_fixed < 1 || a.nkeys_fixed > a.vcap)) || (a.rel_bias && a.rel_d < 1))
        return hipErrorInvalidValue;
    const int dh32 = a.d_head <= 32 ? 1 : (a.d_head <= 64 ? 2 : 4);
    const size_t smem = (size_t)dh32 * 16 * 1024 + (a.rel_bias ? (size_t)(2 * a.rel_d + 1) * 4 : 0);
    if (smem > 160 * 1024) return hipErrorInvalidValue;
    const dim3 grid((unsigned)a.heads, (unsigned)((a.T + 63) / 64)), block(256);
#define BILD_AT(DHV, RV)                                                                                                     \
    do {                                                                                                                     \
        hipLaunchKernelGGL((attn_tile_kernel<DHV, RV>), grid, block, smem, st, a);                                           \
        return hipGetLastError();                                                                                            \
    } while (0)
    if (a.rel_bias) {
        if (dh32 == 1) BILD_AT(1, true);
        if (dh32 == 2) BILD_AT(2, true);
        BILD_AT(4, true);
    }
    if (dh32 == 1) BILD_AT(1, false);
    if (dh32 == 2) BILD_AT(2, false);
    BILD_AT(4, false);
#undef BILD_AT
}

}  // namespace bild
