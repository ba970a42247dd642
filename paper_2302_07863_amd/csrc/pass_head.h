// LM head and policy inside the pass kernel on one die (pass_kernel.hip), for passes of one row.
//
// The workgroups of the other dies have nothing to do in such a pass.  Here they ask for their part of the vocabulary matrix while the
// layers run, up to two units of feature tiles each (10 tiles x 16 KiB of a 512-wide bf16 model: a 32 128-id head lies in registers as a
// whole), wait for the final hidden state, which the owners of its features hand over past their die's L2, multiply, and hand over one
// (max, sum, argmax) a wave; the first of them joins these and runs the policy.  What follows the last layer is then two hand-overs, a
// product and a join instead of two launches that each begin with a trip to memory.  us a step, with the host's wait, head and policy as kernels / here, one
// card: T5-small shape 82.9 / 79.5, mT5-small shape 145.6 / 136.8 (250 112 ids: seven units a workgroup, of which two are there in time), fp32 256 wide, two
// layers, 1024 ids 40.6 / 37.0.  Of the 13 us behind the T5-small shape's layers 0.9 are the hidden state's way, 1.5 the product and its statistics, 0.8 to 2.5 the
// partials' way from the last of 224 workgroups, 1.2 the host's copy.  Tried: all of that rehearsed on zeros while the layers run, for the
// instructions' sake, and the weights 7.6 us later, out of the way of the first layer's (0.9 us there, which then came in the next one): no gain.
//
// The hidden state and the partials have two places that take turns (a pass fills the other one's with "not there yet"; nobody looks
// there before the next kernel).  Rank and turn are one count's, which goes on from pass to pass: 32 a pass on die 0, 256 a pass on the others (the
// last of the 224 to start adds what is left).  So nobody has to have started for the pass to be counted: other streams' kernels may
// have any compute unit of these dies, as when head and policy were kernels.  The first workgroup (rank 0) has the parts of those that have not started when it has
// done its own; who starts behind that does its part once more, the same words in the same place, and ends.  A workgroup waits
// for the hidden state 64 times as often as others for theirs, 0.3 s: die 0 may be in use too.  Whoever hands something over there has given up before
// that if it cannot, and the flag is looked at here.
#pragma once
#include "pass_walk.h"
#include "policy_commit.h"

namespace bild {

// (a kernel of its own: in one with the other passes, those take 0.5 us more)
template <bool FP32>
struct HeadWalk : Walk<true, FP32, 1> {
    static constexpr bool HEAD = true;
    bool odd;  // whose turn it is
    // (the flag is in memory before anything that comes of it is handed over)
    __device__ __forceinline__ void give_up() {
        Walk<true, FP32, 1>::give_up();
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    }
};

template <bool F32>
struct HeadCut {
    static constexpr int RW = F32 ? 4 : 10;         // feature tiles of a unit
    static constexpr int NV = (RW * 16 + 63) / 64;  // waves with its logits
};

// The final norm's gain for the last layer's owners, in place of what other passes ask for there (and don't use).
__device__ __forceinline__ const float* final_gain(const float* other) { return other; }
__device__ __forceinline__ const float* final_gain(const float*, const PassHead& h) { return h.gain; }

// Four features from n0 of the final hidden state (of the lanes of the waves that have some), past the die's L2.
template <class Walk>
__device__ __forceinline__ void publish_final(Walk& c, const PassArgs& a, const PassHead& h, bool mine, int n0, const float4& x, const float4& gain) {
    if (!mine) return;
    const float w[4] = {x.x * gain.x, x.y * gain.y, x.z * gain.z, x.w * gain.w};
    const float ss = quad_rows_sum(x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w);
    const Rsrc out = whole(a.scratch + h.at + (c.odd ? h.bytes : 0)), other = whole(a.scratch + h.at + (c.odd ? 0 : h.bytes));
    const v4u none = {kNotThere, kNotThere, kNotThere, kNotThere};
    v4u v = {__float_as_uint(w[0]), __float_as_uint(w[1]), __float_as_uint(w[2]), __float_as_uint(w[3])};
    int off = (n0 >> 4) * tile_bytes(true, 1, true) + (n0 & 15) * 4;  // (as put_planes() lays them out; the sum of squares behind them)
    if constexpr (!Walk::F32) {
        v = query_parts(f32x4{w[0], w[1], w[2], w[3]});
        off = (n0 >> 5) * tile_bytes(true, 1, false) + ((n0 >> 4) & 1) * 128 + c.g * 16;
    }
    if (c.tok == 1) {
        v = v4u{__float_as_uint(ss), __float_as_uint(ss), __float_as_uint(ss), __float_as_uint(ss)};
        off = Walk::F32 ? (n0 >> 4) * tile_bytes(true, 1, true) + 64 : (n0 >> 5) * tile_bytes(true, 1, false) + ((n0 >> 4) & 1) * 128 + 64;
    }
    if (c.tok == 0 || (c.tok == 1 && c.g == 0)) {
        __builtin_amdgcn_raw_buffer_store_b128(v, out, off, 0, 17);
        __builtin_amdgcn_raw_buffer_store_b128(none, other, off, 0, 17);
    }
}

template <class Cut, class Walk>
__device__ __forceinline__ void head_part(Walk& c, const PassArgs& a, const PassHead& h) {
    constexpr bool F32 = Walk::F32;
    constexpr int N = Cut::KD, RW = HeadCut<F32>::RW, NV = HeadCut<F32>::NV;
    unsigned* const others = h.started + kPassOthers;
    if (threadIdx.x == 0) {
        const unsigned n = __hip_atomic_fetch_add(others, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if ((int)(n & 255u) == h.groups - 1) __hip_atomic_fetch_add(others, 256u - (unsigned)h.groups, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // (the last one)
        *(unsigned*)c.lds = n;
    }
    lds_barrier();
    const unsigned before = (unsigned)__builtin_amdgcn_readfirstlane(*(volatile int*)c.lds);
    const int rank = (int)(before & 255u);
    const bool odd = c.odd = (before >> 8) & 1u;
    lds_barrier();
    const int units = (h.tn + RW - 1) / RW, workers = min(units, h.groups);
    if (rank >= workers) return;
    const int tk = a.d >> Walk::KS, S = tile_bytes(true, 1, F32), clear = odd ? -h.bytes : h.bytes;
    char* const mem = a.scratch + h.at + (odd ? h.bytes : 0);
    const Run r = run_of(c.wave, tk);
    const int n = workers * NV;  // partials
    // The part of workgroup `who`.
    auto part = [&](auto several, const int who) {
        constexpr bool MORE = decltype(several)::value;
        uint4 W[MORE ? 2 : 1][N * RW];
        request<N, RW>(c, W[0], h.w, who, tk, h.tn);
        if constexpr (MORE) request<N, RW>(c, W[1], h.w, min(who + h.groups, units - 1), tk, h.tn);
        const Rsrc xs = whole(mem), count = whole(others);
        // ---- the final hidden state ----
        uint4 X;
        unsigned sum = 0u;
        {
            const int beside = F32 ? c.tok : c.tok & 3, last = max(r.n - 1, 0), from = r.n > 0 ? r.k0 * S : 0;
            const int at = (F32 ? c.g * 16 : (c.tok & 4) ? (c.g & 1) * 128 + 64 : (c.g >> 1) * 128 + (c.g & 1) * 32 + (c.tok >> 3) * 16) + min(beside, last) * S;
            const int most = c.spins > 1 << 24 ? 1 << 30 : 64 * c.spins;
            int tries = 0;
            unsigned seen = 0u, lost = 0u;
            bool missing;
            do {
                asm volatile("" ::: "memory");
                X = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xs, at, from, Walk::kIn));
                if constexpr (F32) sum = __builtin_amdgcn_raw_buffer_load_b32(xs, min(c.g, last) * S + 64, from, Walk::kIn);
                if (rank == 0) seen = __builtin_amdgcn_raw_buffer_load_b32(count, 0, 0, Walk::kIn);
                if ((tries & 15) == 15) lost = __builtin_amdgcn_raw_buffer_load_b32(whole(c.failed), 0, 0, Walk::kIn);
                const unsigned m = max(max(max(X.x, X.y), max(X.z, X.w)), sum);
                missing = __builtin_amdgcn_ballot_w64(m == kNotThere) != 0ull && !c.dead;
                if (__builtin_amdgcn_readfirstlane(lost) != 0u) c.dead = true, missing = false;  // (nobody may be left who would hand it over)
                if (missing) __builtin_amdgcn_s_sleep(4);  // (0.1 us)
            } while (missing && ++tries < most);
            if (missing) c.give_up();
            if (rank == 0 && threadIdx.x == 0) *(unsigned*)(c.lds + kMl + 512) = seen - before;  // (behind the waves' statistics)
        }
        if constexpr (F32) c.ss = quad_rows_sum(c.g < r.n ? __uint_as_float(sum) : 0.f);
        else c.ss = (c.tok & 3) < r.n ? __uint_as_float(X.x) : 0.f;
        uint4 x[N];  // (bf16: an operand per tile, whose high parts' row and low parts' row alone are not zero)
#pragma unroll
        for (int j = 0; j < N; ++j) {
            if constexpr (F32) {
                x[j] = from_lane<0>(X, j);
            } else {
                const bool on = (c.tok & 7) == j;
                x[j] = make_uint4(on ? X.x : 0u, on ? X.y : 0u, on ? X.z : 0u, on ? X.w : 0u);
            }
        }
        float factor = 0.f;
        Stat st = stat_neutral();  // of this lane's logits
        auto unit = [&](uint4 (&w)[N * RW], int u, auto first) {
            constexpr bool FIRST = decltype(first)::value;
            f32x4 acc[RW];
#pragma unroll
            for (int q = 0; q < RW; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < N; ++j)
                if (j < r.n) {
#pragma unroll
                    for (int q = 0; q < RW; ++q) {
                        const uint4 v = w[j * RW + q];
                        if constexpr (F32) {
                            acc[q][0] = __builtin_fmaf(__uint_as_float(v.x), __uint_as_float(x[j].x), acc[q][0]);
                            acc[q][1] = __builtin_fmaf(__uint_as_float(v.y), __uint_as_float(x[j].y), acc[q][1]);
                            acc[q][2] = __builtin_fmaf(__uint_as_float(v.z), __uint_as_float(x[j].z), acc[q][2]);
                            acc[q][3] = __builtin_fmaf(__uint_as_float(v.w), __uint_as_float(x[j].w), acc[q][3]);
                        } else {
                            acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf(x[j]), as_bf(v), acc[q], 0, 0, 0);
                        }
                    }
                }
            if constexpr (MORE) {
                __builtin_amdgcn_sched_barrier(0);
                if (u + 2 * h.groups < units) request<N, RW>(c, w, h.w, u + 2 * h.groups, tk, h.tn);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (!F32) {
#pragma unroll
                for (int q = 0; q < RW; ++q) acc[q][0] = (acc[q][0] + acc[q][1]) + (acc[q][2] + acc[q][3]);
            }
            leave<RW, FIRST, true>(c, acc);
            if (c.wave >= NV) return;
            if constexpr (FIRST) factor = norm_factor(c, a.d, a.eps) * h.scale;
            const int i = c.wave * 64 + c.lane, tile = min(i >> 4, RW - 1), id = (u * RW + tile) * 16 + (i & 15);
            float p[kPassWaves];
#pragma unroll
            for (int v = 0; v < kPassWaves; ++v) p[v] = *(const float*)(c.lds + kRed + c.red + ((v * RW + tile) * 16 + (i & 15)) * 4);
            float z = p[0];
#pragma unroll
            for (int v = 1; v < kPassWaves; ++v) z += p[v];
            z = i < RW * 16 && id < h.vocab ? z * factor : -INFINITY;
            if (z > st.m) st.idx = id;  // (ids rise)
            const float m = fmaxf(st.m, z), base = m == -INFINITY ? 0.f : m;
            st.s = st.s * fexp_full(st.m - base) + fexp_full(z - base);
            st.m = m;
        };
        unit(W[0], who, std::true_type{});
        if constexpr (MORE) {
            for (int u = who + h.groups; u < units; u += 2 * h.groups) {
                unit(W[1], u, std::false_type{});
                if (u + h.groups >= units) break;
                unit(W[0], u + h.groups, std::false_type{});
            }
        }
        if (c.wave < NV) {
            const Stat o = join_parts(st);
            if (c.lane == 0) {
                const int off = h.rec + (who * NV + c.wave) * 16;
                __builtin_amdgcn_raw_buffer_store_b128(v4u{__float_as_uint(o.m), __float_as_uint(o.s), (unsigned)o.idx, 0u}, whole(mem), off, 0, 17);
                __builtin_amdgcn_raw_buffer_store_b128(v4u{kNotThere, kNotThere, kNotThere, kNotThere}, whole(mem + clear), off, 0, 17);
            }
        }
    };
    for (int who = rank; who < workers;) {
        if (units > h.groups) part(std::true_type{}, who);
        else part(std::false_type{}, who);
        if (rank != 0) return;
        // (the first one: then the parts of those that have not started)
        who = max(who + 1, __builtin_amdgcn_readfirstlane(*(volatile int*)(c.lds + kMl + 512)));
        lds_barrier();
    }
    // ---- the partials' join and the policy ----
    const Controls k(h.f);
    static_assert(256 * NV <= 2 * kPassThreads, "two partials a thread");
    uint4 p[2];
    int tries = 0;
    bool missing;
    do {
        asm volatile("" ::: "memory");
        unsigned m = 0u;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            p[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(whole(mem), h.rec + min((int)threadIdx.x + i * kPassThreads, n - 1) * 16, 0, Walk::kIn));
            m = max(max(m, max(p[i].x, p[i].y)), max(p[i].z, p[i].w));
        }
        missing = __builtin_amdgcn_ballot_w64(m == kNotThere) != 0ull && !c.dead;
    } while (missing && ++tries < c.spins);
    if (missing) c.give_up();
    const unsigned failed = __builtin_amdgcn_raw_buffer_load_b32(whole(c.failed), 0, 0, 17);  // (set before what came of it was handed over)
    Stat s = stat_neutral();
#pragma unroll
    for (int i = 0; i < 2; ++i)
        if ((int)threadIdx.x + i * kPassThreads < n) s = stat_merge<true>(s, Stat{__uint_as_float(p[i].x), __uint_as_float(p[i].y), (int)p[i].z});
    s = join_parts(s);
    StatPart* const all = (StatPart*)(c.lds + kMl);
    if (c.lane == 0) all[c.wave] = StatPart{s.m, s.s, s.idx, c.dead || failed != 0u};
    lds_barrier();
    if (c.wave != 0) return;
    StatPart q = {-INFINITY, 0.f, 0x7FFFFFFF, 0};
    if (c.lane < kPassWaves) q = all[c.lane];
    const bool lost = __builtin_amdgcn_ballot_w64(q.pad != 0) != 0ull;
    s = join_parts(Stat{q.m, q.s, q.idx});
    commit<true>(h.f, k, lost, s.idx, s.m, s.s, 0.f, -1, -1);
}

}  // namespace bild
