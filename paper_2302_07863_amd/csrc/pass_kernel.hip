// One decoder pass of a narrow model in ONE kernel: embedding and all layers for up to 16 rows (bf16; fp32 up to 256 wide, on one die).
//
// Such a pass is a chain of 45 (T5-small shape) to 171 (T5-large shape) dependent stages, each far too small to use the
// chip for long.  As kernels of their own they cost 3.5 - 8 us each: 1.5 us of launch, a trip to memory for the activations and
// a longer one for the weights, which can only be asked for once the kernel runs.  Here workgroups stay for the whole pass (one
// per compute unit at most) and walk the stages:
//
//   - hand-over.  Results are their own flags: the memory they are handed over in is filled with words that no result has, and who
//     needs a piece reads it until none of them is left.  Three layers' memory takes turns: who produces a piece for layer l fills its
//     place for layer l + 2.  What was there, of layer l - 1, has been read by then, because layer l's results come from it; and the
//     filling has been seen before somebody looks there, because its producer has waited for a later read since and what it
//     produced then for layer l + 1 is what the reader has seen before.  Nothing is counted, nothing waits for a store to be acknowledged, and the read that finds the flag
//     has brought the data: between two dies 0.65 - 0.8 us from a store to its reader, 0.3 us on one die, where publish, count, poll
//     and read back took 1.8 us over the chip.  A read misses its die's L2 only after somebody has written the line, so waiting
//     workgroups stay off the fabric.  A line that is polled before it is written has to be taken away from eight L2s and
//     fetched again, 0.3 us: where a stage's results cannot be there yet its readers sleep first.  A reader whose part in between is
//     the others' (who owns features has none of the FFN's input, as in the T5-large shape and in one-row passes of the mT5-large one)
//     sleeps until just before the results of two stages on (out_nap, qkv_nap: 1.7 to 3.9 us, see there).  One that has a part in between has a
//     shorter nap: q, k, v and the FFN's input projection 0.25 us, its output projection 0.4, behind a gated input projection 0.65
//     (measured while the T5-large shape's owners had a part of everything, one row, without / with: q, k, v 413 / 413, input 413 / 412, output
//     418 / 406; two to eight rows gain 2, 5 to 10 and 10 us by the three; mT5-large shape, eight rows, output 550 / 538, one row 480 / 479.  Twice
//     as long loses 5 to 20 us everywhere, naps in front of the other stages gain nothing or 2 us);
//   - what belongs together lies together: a row's sums of squares beside its planes (a line that all producers write is taken
//     away from its readers by each of them: 623 -> 714 us when the sums had two lines of their own), a head's query, keys
//     and values of the new rows, which it needs before they can be read from the caches.  Sixteen features' high and low parts
//     are one store, and with one row their sum of squares lies in the same line and comes by the same load: a line that is written
//     twice is fetched twice (one row, T5-large shape, 441 -> 411 us; in a kernel of hand-overs alone 2.0 -> 1.3 us a stage);
//   - weights depend on nothing: they are requested while a workgroup has nothing else to do, those of the FFN and of the next
//     layer during the cross-attention (a wave's loads come back in order, so a request just before a wait delays what follows);
//   - eight waves share a feature tile's inputs; activations arrive as high and low bf16 parts in the order of the matrix core's
//     operand, so that no stage has anything to convert or to share: load, multiply, add up over the waves in LDS in wave order;
//   - a workgroup that owns sixteen features of the residual stream owns them in all layers: they stay in its registers (fp32);
//   - the cross query is worked out by the workgroup of the head that uses it, which saves a hand-over.
//
// A model small enough for the 32 compute units of one die (pass_die_groups: T5-small, mT5-small) walks there: what is handed over
// then only goes to that die's L2 and back, at 1.25 TB/s for the weights instead of the chip's 4.8, which a layer of 7 MB in 13 us
// does not notice.  Workgroups of the other dies end at once, or, in a pass of one row, have the LM head and the policy (pass_head.h).
//
// fp32 models keep fp32 everywhere: activations travel as they are, sixteen rows in a matrix-core operand, attention in blocks of sixteen
// keys (a block's 64 fp32 products take 0.85 us of a wave's SIMD for 32 keys); one row's projections run on the vector ALU (multiply).
//
// Per pass, us, as separate kernels, with counters (and flags on one die) and with results as flags, 512 source tokens: T5-small shape one row 147, 97, 96;
// mT5-small shape 206, 121, 117; T5-large shape 1, 2, 4, 8, 11, 16 rows 676, 785, 853, 986, -, 1211 / 623, 631, 624, 638, 702, 713 / 447,
// 448, 456, 475, 544, 552; mT5-large shape 1 and 8 rows 726, 1045 / 644, 666 / 443, 462.  fp32, 256 wide, 32 source tokens, as separate kernels
// and now: 2 layers, one row 68, 40.5 (49.7 with the matrix cores for it, 43.5 with blocks of 32 keys); 4 layers, 1, 4, 11 rows 120, 145,
// 154, 63, 74, 78.
// Loads of several tiles, one store and one line a producer (multiply, put_planes), with head and policy, before / with: T5-large shape,
// 1, 2, 4, 8 rows 455, 455, 465, 479 / 412, 429, 455, 474; mT5-large shape 514, 511, 523, 537 / 477, 497, 515, 532; T5-small 97 / 96; fp32, 4
// layers, one row 60.4 / 57.5.
//
// A workgroup that has polled `spins` times in vain flags the pass as failed and walks on without waiting again (nothing
// handed over is ever used as an address), so every workgroup ends.  The policy kernel then commits nothing and the host runs
// the pass again as separate kernels; after some passes it tries this kernel again.  That happens only if the workgroups cannot
// all be resident, because of another process' kernel of the same kind, for instance.
#include "pass_head.h"

namespace bild {

// Attention of one head over its keys for all rows: the waves take blocks of 32 keys in turn; (max, sum, O) joined through LDS.
template <bool CAUSAL, bool PACK, class Walk>
struct Attend {
    const Rsrc kr, vr;
    const int I, cap, nkeys, nblk;  // (causal: the keys of earlier passes)
    static constexpr bool F32 = Walk::F32, ONE = Walk::ROOM1;
    // blocks of sixteen or (bf16) twice sixteen keys; pieces of sixteen keys' rows and of a block's values
    static constexpr int AB = F32 ? 1 : 2, BK = 16 * AB, KC = F32 ? 4 : 2, VC = 4;
    uint4 K0[AB][KC], K1[AB][KC], V0[VC], V1[VC];
    // The waves' (max, sum) have a place for each of the two attentions: a wave without keys of the sequence waits for nothing and may leave
    // the next layer's while others still read those of this layer's cross-attention.
    static constexpr int kTops = kMl + (CAUSAL ? 0 : kMlBytes);

    __device__ __forceinline__ void load(const Walk& c, uint4 (&Kr)[AB][KC], uint4 (&Vr)[VC], int blk) const {
        const int key0 = min(blk, nblk - 1) * BK;
        constexpr int E = Walk::ESZ;
#pragma unroll
        for (int ab = 0; ab < AB; ++ab)
#pragma unroll
            for (int ks = 0; ks < KC; ++ks) Kr[ab][ks] = buf_load(kr, (unsigned)((ab * 16 + c.tok) * I * E + c.g * 16), key0 * I * E + ks * 64);
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) {
            const int off = ((dt * 16 + c.tok) * cap + c.g * (ONE ? 8 : 4)) * E;
            if constexpr (F32 || ONE) {
                Vr[dt] = buf_load(vr, (unsigned)off, key0 * E);
            } else {
                const uint2 va = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(vr, off, key0 * 2, 0));
                const uint2 vb = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(vr, off + 32, key0 * 2, 0));
                Vr[dt] = make_uint4(va.x, va.y, vb.x, vb.y);
            }
        }
    }
    // One row: the query is the first operand, so that a product's columns are keys and its rows all the query (high parts in the lane
    // groups 0 and 1, low parts in 2 and 3): after one exchange of the halves each lane has ONE of the wave's 64 keys (two blocks),
    // where the other order leaves sixteen scores to each of the four lanes of the row's column and the same work to all columns.
    // The weights reach the second product's order through LDS, its result is a feature per lane.  With head and policy, us: T5-large
    // shape 412 -> 381, mT5-large 477 -> 441, T5-small on one die 96 -> 87.5; for two rows the two chains of maxima and sums take more
    // than the columns save (420 -> 438), for four 443 -> 498.
    __device__ __forceinline__ void run_one(Walk& c, const Fresh& fresh, int len, const float* relb, int rel_d, void* out, int h) {
        constexpr int IN = Walk::kIn;
        const bool odd = c.g & 1, upper = c.g >= 2;
        char* const w = c.lds + kP + c.wave * 256;  // the weights' high parts and their low parts
        bf16x8 Q[2];
        float m_run = -INFINITY, l_run = 0.f;  // (the sum: this lane's)
        f32x4 O[4];
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) O[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        // of four tiles' values this lane's: tile g's, high and low parts added
        auto mine = [&](const f32x4 (&v)[4]) {
            const float a = odd ? v[1][0] : v[0][0], b = odd ? v[3][0] : v[2][0];
            const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
            return __uint_as_float(x[0]) + __uint_as_float(x[1]);
        };
        // a block of keys to the lower lanes and one to the upper ones, either may be missing; keys behind `lim` are not seen
        auto step = [&](bool lower_has, int lower_key, int lower_lim, bool upper_has, int upper_key, int upper_lim, bool first) {
            f32x4 s[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) s[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (lower_has) {
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                    for (int ab = 0; ab < 2; ++ab) s[ab] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Q[ks], as_bf(K0[ab][ks]), s[ab], 0, 0, 0);
            }
            if (upper_has) {
#pragma unroll
                for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                    for (int ab = 0; ab < 2; ++ab) s[2 + ab] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(Q[ks], as_bf(K1[ab][ks]), s[2 + ab], 0, 0, 0);
            }
            const int key = (upper ? upper_key : lower_key) + (odd ? 16 : 0) + c.tok, lim = upper ? (upper_has ? upper_lim : -1) : (lower_has ? lower_lim : -1);
            float z = mine(s);
            if (CAUSAL && relb) z += relb[rel_d + max(-rel_d, min(rel_d, key - len))];
            if (key > lim) z = -INFINITY;
            const float m_new = fmaxf(m_run, wave_max(z)), base = m_new == -INFINITY ? 0.f : m_new;
            const float p = fexp(z - base);
            if (first) {
                l_run = p;
            } else {
                const float f = fexp(m_run - base);
                l_run = l_run * f + p;
#pragma unroll
                for (int dt = 0; dt < 4; ++dt) O[dt] *= f;
            }
            m_run = m_new;
            uint32_t hi, lo;
            split_bf16x2(p, 0.f, hi, lo);
            *(uint16_t*)(w + c.lane * 2) = (uint16_t)hi;
            *(uint16_t*)(w + 128 + c.lane * 2) = (uint16_t)lo;
            asm volatile("" ::: "memory");
            const char* const wr = w + (c.tok >> 3) * 128 + c.g * 16;
            const bf16x8 wl = as_bf(*(const uint4*)wr), wu = as_bf(*(const uint4*)(wr + 64));
            asm volatile("" ::: "memory");
            if (lower_has) {
#pragma unroll
                for (int dt = 0; dt < 4; ++dt) O[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wl, as_bf(V0[dt]), O[dt], 0, 0, 0);
            }
            if (upper_has) {
#pragma unroll
                for (int dt = 0; dt < 4; ++dt) O[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wu, as_bf(V1[dt]), O[dt], 0, 0, 0);
            }
        };
        if constexpr (CAUSAL) {
            const bool newest = c.wave == (nblk & (kPassWaves - 1)), old = c.wave < nblk;
            if (old || newest) {
                uint4 qv[2], kn[2];
                unsigned vn[4];
                int n = 0;
                bool missing;
#pragma unroll 1
                do {
                    asm volatile("" ::: "memory");
                    unsigned m = 0u;
                    auto see = [&](const uint4& v) { m = max(max(m, max(v.x, v.y)), max(v.z, v.w)); };
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks) qv[ks] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(fresh.q, query_piece<true>(c, ks, 0), 0, IN));
                    if (newest) {
#pragma unroll
                        for (int ks = 0; ks < 2; ++ks) kn[ks] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(fresh.k, ks * 64 + c.g * 16, 0, IN));
#pragma unroll
                        for (int dt = 0; dt < 4; ++dt) {
                            vn[dt] = __builtin_amdgcn_raw_buffer_load_b32(fresh.v, (dt * 16 + c.tok) * 4, 0, IN);
                            m = max(m, vn[dt]);
                        }
                        see(kn[0]);
                        see(kn[1]);
                    }
                    see(qv[0]);
                    see(qv[1]);
                    missing = __builtin_amdgcn_ballot_w64(m == kNotThere) != 0ull && !c.dead;
                } while (missing && ++n < c.spins);
                if (missing) c.give_up();
                Q[0] = as_bf(qv[0]);
                Q[1] = as_bf(qv[1]);
                if (newest) {
#pragma unroll
                    for (int ks = 0; ks < 2; ++ks) {
                        K1[0][ks] = kn[ks];
                        K1[1][ks] = make_uint4(0u, 0u, 0u, 0u);
                    }
#pragma unroll
                    for (int dt = 0; dt < 4; ++dt) V1[dt] = make_uint4(c.g == 0 ? vn[dt] >> 16 : 0u, 0u, 0u, 0u);  // (one key: lane group 0's first)
                }
                step(old, c.wave * BK, nkeys - 1, newest, len, len, true);
                for (int blk = c.wave + kPassWaves; blk < nblk; blk += kPassWaves) {
                    load(c, K0, V0, blk);
                    step(true, blk * BK, nkeys - 1, false, 0, 0, false);
                }
            }
        } else {
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) Q[ks] = as_bf(*(const uint4*)(c.lds + kQ + query_piece<true>(c, ks, 0)));
            for (int blk = c.wave; blk < nblk; blk += 2 * kPassWaves) {
                step(true, blk * BK, nkeys - 1, blk + kPassWaves < nblk, (blk + kPassWaves) * BK, nkeys - 1, blk == c.wave);
                if (blk + 2 * kPassWaves < nblk) load(c, K0, V0, blk + 2 * kPassWaves);
                if (blk + 3 * kPassWaves < nblk) load(c, K1, V1, blk + 3 * kPassWaves);
            }
        }
        float* const cm = (float*)(c.lds + kTops);  // the waves' maxima and sums
        c.red = kRedBytes - c.red;
        float* const co = (float*)(c.lds + kRed + c.red) + c.lane;
        const float sum = wave_sum(l_run);
        co[c.wave * 64] = mine(O);
        if (c.lane == 0) {
            cm[c.wave] = m_run;
            cm[kPassWaves + c.wave] = sum;
        }
        lds_barrier();
        if (c.wave == 0) {
            // (a wave without keys has left a maximum of minus infinity and zeros)
            float m[kPassWaves], l[kPassWaves], p[kPassWaves], M = -INFINITY, L = 0.f, o = 0.f;
#pragma unroll
            for (int v = 0; v < kPassWaves; ++v) {
                m[v] = cm[v];
                l[v] = cm[kPassWaves + v];
                p[v] = co[v * 64];
            }
#pragma unroll
            for (int v = 0; v < kPassWaves; ++v) M = fmaxf(M, m[v]);
#pragma unroll
            for (int v = 0; v < kPassWaves; ++v) {
                m[v] = fexp(m[v] - M);
                L += l[v] * m[v];
                o += p[v] * m[v];
            }
            o *= 1.f / L;
            // eight features' high parts to a quad of lanes, their low parts to the next; the quads' first lanes store
            uint32_t h01, h23, l01, l23;
            split_bf16x2(dpp_f<0x00, 0xF>(0.f, o), dpp_f<0x55, 0xF>(0.f, o), h01, l01);
            split_bf16x2(dpp_f<0xAA, 0xF>(0.f, o), dpp_f<0xFF, 0xF>(0.f, o), h23, l23);
            auto from = [](auto ctrl, uint32_t v) { return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, decltype(ctrl)::value, 0xF, 0xF, true); };
            using Next = std::integral_constant<int, 0x104>;  // row_shl:4: the lane four on
            using Last = std::integral_constant<int, 0x114>;  // row_shr:4
            const bool low = c.lane & 4;
            const uint32_t n01 = from(Next{}, h01), n23 = from(Next{}, h23), p01 = from(Last{}, l01), p23 = from(Last{}, l23);  // (of all lanes)
            const v4u v = {low ? p01 : h01, low ? p23 : h23, low ? l01 : n01, low ? l23 : n23};
            const int off = h * 256 + (c.lane >> 2) * 16;
            if ((c.lane & 3) == 0) {
                __builtin_amdgcn_raw_buffer_store_b128(v, whole(out), off, 0, Walk::kOut);
                __builtin_amdgcn_raw_buffer_store_b128(v4u{kNotThere, kNotThere, kNotThere, kNotThere}, whole((const char*)out + c.clear), off, 0, Walk::kOut);
            }
        }
    }
    // Up to eight rows are packed as in multiply().  Causal: query, keys and values of this pass' rows are handed over in `fresh`,
    // a block of keys of its own that one wave takes; else the query lies in LDS.
    __device__ __forceinline__ void run(Walk& c, const Fresh& fresh, float scale, int len, const float* relb, int rel_d, void* out, int h) {
        if constexpr (ONE) return run_one(c, fresh, len, relb, rel_d, out, h);
        constexpr int P = PACK ? 1 : 2, IN = Walk::kIn;
        bf16x8 Q[2][P];  // scaled, high parts (columns 0 .. 7 if packed) and low parts, as they were handed over
        uint4 Qf[4];     // fp32: scaled, inputs c * 16 + g * 4 ..
        const bool low = c.tok >= 8;
        const int row = PACK ? c.t8 : c.t;
        // high and low parts of eight values in operand order
        auto parts = [&](const float (&v)[8], bf16x8 (&o)[P]) {
            uint32_t hi[4], lo[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) split_bf16x2(v[2 * j], v[2 * j + 1], hi[j], lo[j]);
            if constexpr (PACK) {
                o[0] = as_bf(make_uint4(low ? lo[0] : hi[0], low ? lo[1] : hi[1], low ? lo[2] : hi[2], low ? lo[3] : hi[3]));
            } else {
                o[0] = as_bf(make_uint4(hi[0], hi[1], hi[2], hi[3]));
                o[1] = as_bf(make_uint4(lo[0], lo[1], lo[2], lo[3]));
            }
        };
        auto scale_query = [&](const float4 (&qv)[4]) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                Qf[i] = make_uint4(__float_as_uint(qv[i].x * scale), __float_as_uint(qv[i].y * scale), __float_as_uint(qv[i].z * scale), __float_as_uint(qv[i].w * scale));
        };
        auto take_query = [&](const uint4 (&qv)[4]) {
#pragma unroll
            for (int i = 0; i < 2 * P; ++i) Q[i / P][i % P] = as_bf(qv[i]);
        };
        float m_run = -INFINITY, l_run = 0.f;
        f32x4 O[4];
#pragma unroll
        for (int dt = 0; dt < 4; ++dt) O[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
        // NB blocks at once, whose keys begin at `key`: one maximum, one rescaling; keys behind `lim` (of this lane's row) are not seen
        auto process = [&](auto nb, const uint4 (*const (&Kr)[decltype(nb)::value])[KC], const uint4* const (&Vr)[decltype(nb)::value], const int (&key)[decltype(nb)::value], bool edge, int lim, bool first) {
            constexpr int NB = decltype(nb)::value;
            f32x4 s[NB][AB];
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int ab = 0; ab < AB; ++ab) s[b][ab] = f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (F32) {
#pragma unroll
                for (int ks = 0; ks < KC; ++ks)
#pragma unroll
                    for (int b = 0; b < NB; ++b)
#pragma unroll
                        for (int ab = 0; ab < AB; ++ab) products(s[b][ab], s[b][ab], Kr[b][ab][ks], Qf[ks]);
            } else
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll
                    for (int b = 0; b < NB; ++b)
#pragma unroll
                        for (int ab = 0; ab < AB; ++ab) s[b][ab] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf(Kr[b][ab][ks]), Q[ks][p], s[b][ab], 0, 0, 0);
            if constexpr (PACK) {
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int v = 0; v < 4 * AB; ++v) s[b][v >> 2][v & 3] += dpp_f<0x128, 0xF>(0.f, s[b][v >> 2][v & 3]);
            }
            if (CAUSAL && relb) {
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int v = 0; v < 4 * AB; ++v)
                        s[b][v >> 2][v & 3] += relb[rel_d + max(-rel_d, min(rel_d, key[b] + (v >> 2) * 16 + c.g * 4 + (v & 3) - (len + row)))];
            }
            if (edge) {
#pragma unroll
                for (int b = 0; b < NB; ++b)
#pragma unroll
                    for (int v = 0; v < 4 * AB; ++v)
                        if (key[b] + (v >> 2) * 16 + c.g * 4 + (v & 3) > lim) s[b][v >> 2][v & 3] = -INFINITY;
            }
            float tmax = m_run;
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma unroll
                for (int v = 0; v < 4 * AB; ++v) tmax = fmaxf(tmax, s[b][v >> 2][v & 3]);
            const float m_new = quad_rows_max(tmax), base = m_new == -INFINITY ? 0.f : m_new;
            bf16x8 W[NB][P];
            uint4 Wf[NB];
            float psum = 0.f;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                float p[8] = {};
#pragma unroll
                for (int v = 0; v < 4 * AB; ++v) {
                    p[v] = fexp(s[b][v >> 2][v & 3] - base);
                    psum += p[v];
                }
                if constexpr (F32) {
                    Wf[b] = make_uint4(__float_as_uint(p[0]), __float_as_uint(p[1]), __float_as_uint(p[2]), __float_as_uint(p[3]));
                } else {
                    parts(p, W[b]);
                }
            }
            psum = quad_rows_sum(psum);
            if (first) {
                l_run = psum;
            } else {
                const float f = fexp(m_run - base);
                l_run = l_run * f + psum;
#pragma unroll
                for (int dt = 0; dt < 4; ++dt) O[dt] *= f;
            }
            m_run = m_new;
#pragma unroll
            for (int b = 0; b < NB; ++b)
                if constexpr (F32) {
#pragma unroll
                    for (int dt = 0; dt < 4; ++dt) products(O[dt], O[dt], Vr[b][dt], Wf[b]);
                } else
#pragma unroll
                for (int p = 0; p < P; ++p)
#pragma unroll
                    for (int dt = 0; dt < 4; ++dt) O[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf(Vr[b][dt]), W[b][p], O[dt], 0, 0, 0);
        };
        using One = std::integral_constant<int, 1>;
        using Two = std::integral_constant<int, 2>;
        if constexpr (CAUSAL) {
            const bool newest = c.wave == (nblk & (kPassWaves - 1));
            if (c.wave < nblk || newest) {
                constexpr int QL = F32 ? 4 : 2 * P;
                uint4 qv[4];
                float4 vn[4];
                uint4 kn[KC];
                int n = 0;
                bool missing;
#pragma unroll 1
                do {
                    asm volatile("" ::: "memory");
                    unsigned m = 0u;
                    auto see = [&](unsigned a, unsigned b, unsigned d, unsigned e) { m = max(max(m, max(a, b)), max(d, e)); };
#pragma unroll
                    for (int i = 0; i < QL; ++i) qv[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(fresh.q, row * 256 + (F32 ? i * 64 + c.g * 16 : query_piece<PACK>(c, i / P, i % P)), 0, IN));
                    if (newest) {
#pragma unroll
                        for (int ks = 0; ks < KC; ++ks) kn[ks] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(fresh.k, c.t * (64 * Walk::ESZ) + ks * 64 + c.g * 16, 0, IN));
#pragma unroll
                        for (int dt = 0; dt < 4; ++dt) vn[dt] = ldf4<IN>(fresh.v, ((dt * 16 + c.tok) * fresh.room + min(c.g * 4, fresh.room - 4)) * 4);
#pragma unroll
                        for (int ks = 0; ks < KC; ++ks) see(kn[ks].x, kn[ks].y, kn[ks].z, kn[ks].w);
#pragma unroll
                        for (int dt = 0; dt < 4; ++dt) see(__float_as_uint(vn[dt].x), __float_as_uint(vn[dt].y), __float_as_uint(vn[dt].z), __float_as_uint(vn[dt].w));
                    }
#pragma unroll
                    for (int i = 0; i < QL; ++i) see(qv[i].x, qv[i].y, qv[i].z, qv[i].w);
                    missing = __builtin_amdgcn_ballot_w64(m == kNotThere) != 0ull && !c.dead;
                } while (missing && ++n < c.spins);
                if (missing) c.give_up();
                if constexpr (F32) scale_query({__builtin_bit_cast(float4, qv[0]), __builtin_bit_cast(float4, qv[1]), __builtin_bit_cast(float4, qv[2]), __builtin_bit_cast(float4, qv[3])});
                else take_query(qv);
                if (c.wave < nblk) process(One{}, {K0}, {V0}, {c.wave * BK}, c.wave * BK + BK - 1 >= nkeys, nkeys - 1, true);
                for (int blk = c.wave + kPassWaves; blk < nblk; blk += kPassWaves) {
                    load(c, K0, V0, blk);
                    process(One{}, {K0}, {V0}, {blk * BK}, blk * BK + BK - 1 >= nkeys, nkeys - 1, false);
                }
                if (newest) {
#pragma unroll
                    for (int ks = 0; ks < KC; ++ks) {
                        K0[0][ks] = kn[ks];
                        if constexpr (AB == 2) K0[AB - 1][ks] = make_uint4(0u, 0u, 0u, 0u);
                    }
#pragma unroll
                    for (int dt = 0; dt < 4; ++dt) {
                        const uint4 v = __builtin_bit_cast(uint4, vn[dt]);
                        if constexpr (F32) {
                            V0[dt] = v;
                        } else {  // (bf16 values in the upper halves)
                            V0[dt] = make_uint4(__builtin_amdgcn_perm(v.y, v.x, 0x07060302u), __builtin_amdgcn_perm(v.w, v.z, 0x07060302u), 0u, 0u);
                        }
                    }
                    process(One{}, {K0}, {V0}, {len}, true, len + row, c.wave >= nblk);
                }
            }
        } else {
            if constexpr (F32) {
                const float* q = (const float*)(c.lds + kQ) + row * kQLd;
                scale_query({*(const float4*)(q + c.g * 4), *(const float4*)(q + 16 + c.g * 4), *(const float4*)(q + 32 + c.g * 4), *(const float4*)(q + 48 + c.g * 4)});
            } else {
                uint4 qv[4];
#pragma unroll
                for (int i = 0; i < 2 * P; ++i) qv[i] = *(const uint4*)(c.lds + kQ + row * kQLd * 4 + query_piece<PACK>(c, i / P, i % P));
                take_query(qv);
            }
            if constexpr (F32) {  // (one set of registers)
                for (int blk = c.wave; blk < nblk; blk += kPassWaves) {
                    process(One{}, {K0}, {V0}, {blk * BK}, blk * BK + BK - 1 >= nkeys, nkeys - 1, blk == c.wave);
                    if (blk + kPassWaves < nblk) load(c, K0, V0, blk + kPassWaves);
                }
            } else {
                for (int blk = c.wave; blk < nblk; blk += 2 * kPassWaves) {
                    const bool first = blk == c.wave;
                    if (blk + kPassWaves < nblk) process(Two{}, {K0, K1}, {V0, V1}, {blk * BK, (blk + kPassWaves) * BK}, (blk + kPassWaves) * BK + BK - 1 >= nkeys, nkeys - 1, first);
                    else process(One{}, {K0}, {V0}, {blk * BK}, blk * BK + BK - 1 >= nkeys, nkeys - 1, first);
                    if (blk + 2 * kPassWaves < nblk) load(c, K0, V0, blk + 2 * kPassWaves);
                    if (blk + 3 * kPassWaves < nblk) load(c, K1, V1, blk + 3 * kPassWaves);
                }
            }
        }
        float* cm = (float*)(c.lds + kTops);
        float* cl = cm + kPassWaves * 16;
        if (c.g == 0) {
            cm[c.wave * 16 + c.tok] = m_run;
            cl[c.wave * 16 + c.tok] = l_run;
        }
        leave<4, false, false>(c, O);
        if (c.wave < 4) {
            // (all of it read at once and without a test: a wave without keys has left a maximum of minus infinity and zeros)
            float w[kPassWaves], l[kPassWaves], M = -INFINITY, L = 0.f;
            f32x4 p[kPassWaves], o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int v = 0; v < kPassWaves; ++v) {
                w[v] = cm[v * 16 + c.tok];
                l[v] = cl[v * 16 + c.tok];
                p[v] = *(const f32x4*)(c.lds + kRed + c.red + ((v * 4 + c.wave) * 64 + c.lane) * 16);
            }
#pragma unroll
            for (int v = 0; v < kPassWaves; ++v) M = fmaxf(M, w[v]);
#pragma unroll
            for (int v = 0; v < kPassWaves; ++v) {
                w[v] = fexp(w[v] - M);
                L += l[v] * w[v];
                o += p[v] * w[v];
            }
            if constexpr (PACK) {
#pragma unroll
                for (int v = 0; v < 4; ++v) o[v] += dpp_f<0x128, 0xF>(0.f, o[v]);
            }
            const float inv = 1.f / L;
            const float r[4] = {o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv};
            put_planes<PACK, false>(c, out, h * 64 + c.wave * 16 + c.g * 4, r);
        }
    }
};

// How the projections are cut: feature tiles per workgroup of q, k, v (QT), of the residual stream (OT), of the FFN (FT, pairs of
// tiles where it is gated), input tiles per wave of the model's width (KD) and of the FFN's hidden state (KF).
struct ChipCut {
    static constexpr int QT = 1, OT = 1, FT = 2, KD = 4, KF = 16;
};
struct DieCut {
    static constexpr int QT = 4, OT = 2, FT = 6, KD = 2, KF = 8;
};
struct DieCutF32 {
    static constexpr int QT = 2, OT = 1, FT = 4, KD = 2, KF = 8;
};
__host__ __device__ inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Workgroups [0, workers) do the projections; the first of them own sixteen features (OT times) of the residual stream each: wave
// q holds those of tile q.
template <bool GATED, bool PACK, class Cut, class Walk, class... Head>
__device__ __forceinline__ void worker(Walk& c, const PassArgs& a, int groups, const Head&... head) {
    int T = a.T, d = a.d, I = a.I, F = a.F;
    constexpr int QT = Cut::QT, OT = Cut::OT, FT = Cut::FT, KD = Cut::KD, KF = Cut::KF;
    constexpr bool CHIP = Walk::kOut != 0;
    // EARLY: input tiles of the FFN's output projection asked for before the self-attention's results are waited for, WQ: where the next
    // layer's first weights are asked for (see there).  Over the chip 0, 0: with 4 to 16 of 16 early T5-large 372 -> 371 .. 390 us.  On one
    // die, EARLY 0, 4, 8 and WQ 0, 1, 2: T5-small shape 87 (0, 0), 85 (0, 1), 84 (4, 1), 82.5 (4, 2), 85.5 (8, 2), mT5-small 152, 144, 143.5, 146, 146.
    // WQ, 12 layers, one row, 1 / 2: without gate, 512 wide, d_ff 512, 1024, 1408, 2048 125.7, 134, 135.4, 139 / 125.3, 134, 134, 136, 256 wide, d_ff 512, 704,
    // 1024 118.3, 119, 119.5 / 117, 118, 118.5 (four rows up to 1.5 % the other way, d_ff 2048 2 % this way); gated the two lie within 1 % of each other (512 wide,
    // d_ff 512 127, 128, six heads and 1024 130.7, 131.8, eight heads and 1024 137.4, 136.6; 256 wide 121 either way).
    // fp32, whose weights are twice as large and whose rows travel whole: 0, 0 too (256 wide, d_ff 1024, 12 layers, 1, 2, 4, 11 rows 139.5, 182, 183, 188 with
    // 4, 2 and 133, 175, 176, 181; gated, d_ff 512, 139, 174, 175, 180 with 4, 1 and 135, 171, 172, 176).
    constexpr int EARLY = CHIP || Walk::F32 ? 0 : 4, WQ = CHIP || Walk::F32 ? 0 : GATED ? 1 : 2;
    // Naps of workgroups whose part in between is the others' (see the head of this file), in turns of 95 ns: from their own result to
    // what comes of it two stages on.  By width and rows; measured optima (none / best, us, 12 layers): 256 wide 1, 8 rows 15, 20 turns (149 / 149,
    // 171 / 167), 512 20, 22 (154 / 152, 188 / 182), 768 23, 26 (167 / 163, 213 / 203), 1024 27, 31 (189 / 183, 244 / 230), gated 29, 34 (190 / 185, 248 /
    // 234); two turns more here than in those measurements, whose naps also read their length.  Two turns too short or four too long lose
    // half of it where d_ff is 4 d.  d_ff is not part of it: with three or six turns less in front of q, k, v (256 to 1024 wide) passes of 1 to 8 rows take -0.4 to +0.7 %
    // at d_ff of 1 to 2 d, -0.5 to +2.5 % at 2.75 d and -1.1 to +2.6 % at 4 d, eleven rows -1.3 to +0.2 %.  Over the chip only: on one die, where a hand-over takes 0.3 us, 256-wide models of a narrow FFN lost by it (d_ff 256, 12 layers, one,
    // two, four rows 126, 134, 134 us with, 116, 123, 123 without; gated, d_ff 128, 128, 139, 137 and 118, 125, 124; fp32, d_ff 512, 145, 176, 176 and 137, 174, 175).
    constexpr int RI = Walk::KNOWN <= 1 ? 0 : Walk::KNOWN == 2 ? 1 : Walk::KNOWN == 4 ? 2 : Walk::KNOWN == 8 ? 3 : 4;
    constexpr int OUT_A[] = {14, 16, 16, 18, 20}, OUT_B[] = {15, 14, 14, 14, 17}, QKV_A[] = {18, 22, 18, 20, 20}, QKV_B[] = {8, 5, 14, 14, 16};
    auto out_nap = [&] { return OUT_A[RI] + ((OUT_B[RI] * d + 512) >> 10) + (!GATED ? 0 : RI ? 4 : 2); };
    auto qkv_nap = [&] { return QKV_A[RI] + ((QKV_B[RI] * d + 512) >> 10); };
    constexpr bool RD = Walk::template side<KD>() > 1, RF = Walk::template side<KF>() > 1;  // (tiles beside each other: sums by row)
    const int base = groups - a.heads;  // the workgroups with a head each follow
    const int len = *a.len_ptr;
    auto nd = [&] { return d >> 4; };
    auto tq = [&] { return 3 * (I >> 4); };
    auto tf = [&] { return GATED ? F >> 3 : F >> 4; };  // tiles
    auto no = [&] { return ceil_div(nd(), OT); };
    auto nq = [&] { return ceil_div(tq(), QT); };
    auto nf = [&] { return ceil_div(tf(), FT); };       // workgroups
    // This workgroup's part of q, k, v and of the FFN: the last workgroups' (pass_last), so that those that own features of the residual stream have
    // as few other weights to ask for as there are compute units for: an owner that also had its part of the FFN's input asked for 224
    // KB in front of the cross-attention's results, which came 2.6 us after they were handed over (1.5 now).
    const bool back = !CHIP || a.last;
    const int uq = c.wg - (back ? base - nq() : 0), uf = c.wg - (back ? base - nf() : 0);
    const bool owner = c.wg < no(), qkv = uq >= 0 && uq < nq(), ffn = uf >= 0 && uf < nf();
    const bool apart = CHIP && back && no() + nf() <= base;  // who owns features has no part of the FFN's input
    uint4 Wq[KD * QT], Wo[KD * OT], Wi[KD * FT], Wf[KF * OT];
    float4 next_gain = make_float4(0.f, 0.f, 0.f, 0.f);
    float4 x = make_float4(0.f, 0.f, 0.f, 0.f);  // (owners, waves below OT) the residual stream of this lane's row, features n0 .. n0 + 3
    const bool mine = c.wave < OT && c.wg * OT + c.wave < nd();
    auto n0 = [&] { return (c.wg * OT + c.wave) * 16 + c.g * 4; };
    // the gain of the norm that reads x next, requested before the wait for what is added to it
    auto gain = [&](const float* g) { return ldf4(whole(g), mine ? n0() * 4 : 0); };
    auto publish = [&](const float4& gn, char* planes) {
        if (mine) {
            const float w[4] = {x.x * gn.x, x.y * gn.y, x.z * gn.z, x.w * gn.w};
            const float ss = quad_rows_sum(x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w);
            put_planes<PACK, true>(c, planes, n0(), w, ss);
            if (!Walk::ROOM1 && c.g == 0) {
                const int off = Walk::F32 ? (n0() >> 4) * tile_bytes(true, c.R, true) + c.R * 64 + c.tok * 4
                                          : (n0() >> 5) * tile_bytes(true, c.R, false) + c.R * 128 + (c.tok * 2 + ((n0() >> 4) & 1)) * 4;
                if (c.tok < T) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(ss), whole(planes), off, 0, Walk::kOut);
                if (c.tok < c.R) __builtin_amdgcn_raw_buffer_store_b32(kNotThere, whole(planes + c.clear), off, 0, Walk::kOut);
            }
        }
    };
    auto add = [&](auto row) {
        const f32x4 s = total<OT, PACK, decltype(row)::value>(c, c.wave);
        x = make_float4(x.x + s[0], x.y + s[1], x.z + s[2], x.w + s[3]);
    };
    const CLayer* L = (const CLayer*)(uintptr_t)a.layers;
    char* z = c.scratch(a);  // this layer's hand-over buffers
    if (owner) {
        const int pos = len + c.t;
        const float4 gn = gain(L->ln1);
        if (mine) {
            if (a.emb) {
                int er = a.tokens[pos] + a.tie_shift;
                er = er >= a.vocab ? er - a.vocab : er;
                const char* p = (const char*)a.emb + ((size_t)(er >> 4) * (d >> c.KS) + (n0() >> c.KS)) * kTileBytes;
                float4 e;
                if constexpr (Walk::F32) {
                    e = *(const float4*)(p + ((er & 15) + 16 * ((n0() & 15) >> 2)) * 16);
                } else {
                    const uint2 raw = *(const uint2*)(p + ((er & 15) + 16 * ((n0() & 31) >> 3)) * 16 + (n0() & 7) * 2);
                    e = make_float4(bf2f(raw.x & 0xFFFFu), bf2f(raw.x >> 16), bf2f(raw.y & 0xFFFFu), bf2f(raw.y >> 16));
                }
                float4 pe = make_float4(0.f, 0.f, 0.f, 0.f);
                if (a.pe) pe = *(const float4*)(a.pe + (size_t)pos * d + n0());
                const float sc = a.embed_scale;
                x = make_float4(__builtin_fmaf(e.x, sc, pe.x), __builtin_fmaf(e.y, sc, pe.y), __builtin_fmaf(e.z, sc, pe.z), __builtin_fmaf(e.w, sc, pe.w));
            } else {
                x = *(const float4*)(a.x_in + (size_t)pos * d + n0());
            }
        }
        publish(gn, z + a.at.x1);
    }
    if (qkv) request<KD, QT>(c, Wq, L->wqkv, uq, d >> c.KS, tq());
    for (int l = 0; l < a.n_layers; ++l) {
        L = (const CLayer*)(uintptr_t)a.layers + l;
        const bool last = l + 1 == a.n_layers;
        // (addresses are worked out where they are needed: kept across the loop they would not fit the registers)
        asm volatile("" : "+v"(c.lane));
        asm volatile("" : "+s"(T), "+s"(d), "+s"(I), "+s"(F));
        c.place(T, a.room);
        // ---- q, k, v (a workgroup's tiles are of one of the three) ----
        if (qkv) {
            const char* xs = pinned(z + a.at.x1);
            const int seg = uq * QT * 16 / I;
            char* kept = pinned(seg == 1 ? L->kc : L->vc);
            char* out = pinned(z + (seg == 0 ? a.at.q : seg == 1 ? a.at.k : a.at.v));
            f32x4 acc[QT];
            if (apart && !owner) c.rest(l ? qkv_nap() : 0);  // (the first layer's come from the embedding)
            else c.template nap<250>();
            multiply<KD, QT, PACK, true>(c, acc, Wq, xs, d >> c.KS);
            leave<QT, true, RD>(c, acc);
            if (c.wave < QT) {
                const float f = norm_factor(c, d, a.eps);
                const f32x4 s = total<QT, PACK, RD>(c, c.wave) * f;
                const int nn = (uq * QT + c.wave) * 16 + c.g * 4 - seg * I, pos = len + c.tok;
                const Rsrc o = whole(out), n = whole(out + c.clear), kv = whole(kept);
                const int hd = nn >> 6, f0 = nn & 63;
                if (seg == 0) {
                    const int off = Walk::F32 ? ((hd * c.R + c.tok) * 64 + f0) * 4 : (hd * c.R + c.tok) * 256 + (f0 >> 4) * 64 + c.g * 16;
                    v4u v = {__float_as_uint(s[0]), __float_as_uint(s[1]), __float_as_uint(s[2]), __float_as_uint(s[3])};
                    if constexpr (!Walk::F32) v = query_parts(s * a.att_scale);
                    if (c.tok < T) __builtin_amdgcn_raw_buffer_store_b128(v, o, off, 0, Walk::kOut);
                    if (c.tok < c.R) __builtin_amdgcn_raw_buffer_store_b128(v4u{kNotThere, kNotThere, kNotThere, kNotThere}, n, off, 0, Walk::kOut);
                } else if (Walk::F32 && seg == 1) {
                    const int off = ((hd * c.R + c.tok) * 64 + f0) * 4;
                    const v4u v = {__float_as_uint(s[0]), __float_as_uint(s[1]), __float_as_uint(s[2]), __float_as_uint(s[3])};
                    if (c.tok < T) {
                        __builtin_amdgcn_raw_buffer_store_b128(v, o, off, 0, Walk::kOut);
                        __builtin_amdgcn_raw_buffer_store_b128(v, kv, (pos * I + nn) * 4, 0, Walk::kOut);
                    }
                    if (c.tok < c.R) __builtin_amdgcn_raw_buffer_store_b128(v4u{kNotThere, kNotThere, kNotThere, kNotThere}, n, off, 0, Walk::kOut);
                } else if (seg == 1) {
                    const int off = ((hd * c.R + c.tok) * 64 + f0) * 2;
                    const unsigned k01 = pack_bf16x2(s[0], s[1]), k23 = pack_bf16x2(s[2], s[3]);
                    if (c.tok < T) {
                        st8<Walk::kOut>(o, off, k01, k23);
                        st8<Walk::kOut>(kv, (pos * I + nn) * 2, k01, k23);
                    }
                    if (c.tok < c.R) st8<Walk::kOut>(n, off, kNotThere, kNotThere);
                } else {
                    const int room = Walk::ROOM1 ? 1 : fresh_room(c.R), off = ((hd * 64 + f0) * room + c.tok) * 4;
                    if constexpr (Walk::ROOM1) {
                        unsigned b[4];
#pragma unroll
                        for (int v = 0; v < 4; ++v) b[v] = f2bf(s[v]);
                        if (c.tok == 0) {
                            __builtin_amdgcn_raw_buffer_store_b128(v4u{b[0] << 16, b[1] << 16, b[2] << 16, b[3] << 16}, o, off, 0, Walk::kOut);
#pragma unroll
                            for (int v = 0; v < 4; ++v) __builtin_amdgcn_raw_buffer_store_b16((unsigned short)b[v], kv, ((nn + v) * a.vcap + pos) * 2, 0, Walk::kOut);
                            __builtin_amdgcn_raw_buffer_store_b128(v4u{kNotThere, kNotThere, kNotThere, kNotThere}, n, off, 0, Walk::kOut);
                        }
                    } else
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const unsigned b = Walk::F32 ? __float_as_uint(s[v]) : f2bf(s[v]);
                        if (c.tok < room) __builtin_amdgcn_raw_buffer_store_b32(c.tok < T ? (Walk::F32 ? b : b << 16) : 0u, o, off + v * room * 4, 0, Walk::kOut);
                        if (c.tok < T) {
                            if constexpr (Walk::F32) __builtin_amdgcn_raw_buffer_store_b32(b, kv, ((nn + v) * a.vcap + pos) * 4, 0, Walk::kOut);
                            else __builtin_amdgcn_raw_buffer_store_b16((unsigned short)b, kv, ((nn + v) * a.vcap + pos) * 2, 0, Walk::kOut);
                        }
                        if (c.tok < room) __builtin_amdgcn_raw_buffer_store_b32(kNotThere, n, off + v * room * 4, 0, Walk::kOut);
                    }
                }
            }
        }
        // ---- output projection ----
        // Requests go out where the workgroup has several microseconds before it is needed again (a wave's loads come back in
        // order: what is asked for late delays the next stage's activations): here, while the heads work, and below.
        if (owner) {
            request<KD, OT>(c, Wo, L->wo, c.wg, I >> c.KS, nd());
            const float4 gn = gain(a.cross ? L->lnc : L->ln2);
            if (a.cross) request<KF, OT, 0, EARLY>(c, Wf, L->wout, c.wg, F >> c.KS, nd());
            if (!a.cross) {
                next_gain = gain(last ? final_gain(L->ln2, head...) : L[1].ln1);
                request<KF, OT>(c, Wf, L->wout, c.wg, F >> c.KS, nd());
            }
            const char* xs = pinned(z + a.at.a1);
            char* ox = pinned(z + a.at.x2);
            f32x4 acc[OT];
            multiply<KD, OT, PACK, false>(c, acc, Wo, xs, I >> c.KS);
            leave<OT, false, RD>(c, acc);
            if (mine) add(std::bool_constant<RD>{});
            publish(gn, ox);
        }
        const char* xf = z + a.at.x2;  // what the FFN reads
        if (a.cross) {
            // ---- output projection of the cross-attention ----
            if (owner) {
                request<KD, OT>(c, Wo, L->cwo, c.wg, I >> c.KS, nd());
                const float4 gn = gain(L->ln2);
                next_gain = gain(last ? final_gain(L->ln2, head...) : L[1].ln1);
                if (ffn) request<KD, FT>(c, Wi, L->win, uf, d >> c.KS, tf());
                request<KF, OT, EARLY, KF>(c, Wf, L->wout, c.wg, F >> c.KS, nd());
                if (qkv && !last && WQ == 0) request<KD, QT>(c, Wq, L[1].wqkv, uq, d >> c.KS, tq());
                const char* xs = pinned(z + a.at.a2);
                char* ox = pinned(z + a.at.x3);
                f32x4 acc[OT];
                multiply<KD, OT, PACK, false>(c, acc, Wo, xs, I >> c.KS);
                leave<OT, false, RD>(c, acc);
                if (mine) add(std::bool_constant<RD>{});
                publish(gn, ox);
            }
            xf = z + a.at.x3;
        }
        // ---- FFN ----
        if (ffn) {
            if (!owner || !a.cross) request<KD, FT>(c, Wi, L->win, uf, d >> c.KS, tf());
            const char* xs = pinned(xf);
            char* out = pinned(z + a.at.h);
            constexpr int FW = GATED ? FT / 2 : FT;  // waves with results
            f32x4 acc[FT];
            c.template nap<250>();
            multiply<KD, FT, PACK, true>(c, acc, Wi, xs, d >> c.KS);
            leave<FT, true, RD>(c, acc);
            const int tile = uf * FW + c.wave;  // of the hidden state
            if (c.wave < FW && tile < F >> 4) {
                const float r = norm_factor(c, d, a.eps);
                float w[4];
                if constexpr (GATED) {
                    const f32x4 s = total<FT, PACK, RD>(c, 2 * c.wave) * r, u = total<FT, PACK, RD>(c, 2 * c.wave + 1) * r;
#pragma unroll
                    for (int v = 0; v < 4; ++v) w[v] = (a.act == BILD_ACT_GATED_GELU ? gelu_tanh_f(s[v]) : silu_f(s[v])) * u[v];
                } else {
                    const f32x4 s = total<FT, PACK, RD>(c, c.wave) * r;
#pragma unroll
                    for (int v = 0; v < 4; ++v) w[v] = fmaxf(s[v], 0.f);
                }
                put_planes<PACK, false>(c, out, tile * 16 + c.g * 4, w);
            }
        }
        if (qkv && !last && (!owner || !a.cross || WQ == 1)) request<KD, QT>(c, Wq, L[1].wqkv, uq, d >> c.KS, tq());
        const char* hidden = z + a.at.h;
        z = c.next(z, a.at.layer);
        c.walk_on(a.at.layer);
        if (owner) {
            const char* xs = pinned(hidden);
            char* ox = pinned(z + a.at.x1);
            f32x4 acc[OT];
            if (apart) c.rest(out_nap());
            else c.template nap<GATED ? 650 : 400>();
            multiply<KF, OT, PACK, false>(c, acc, Wf, xs, F >> c.KS);
            leave<OT, false, RF>(c, acc);
            if (mine) add(std::bool_constant<RF>{});
            if (!last) publish(next_gain, ox);
            else if constexpr (Walk::HEAD) publish_final(c, a, head..., mine, n0(), x, next_gain);
            if (qkv && !last && a.cross && WQ == 2) request<KD, QT>(c, Wq, L[1].wqkv, uq, d >> c.KS, tq());
        }
    }
    if (owner && mine && c.tok < T) {
        *(float4*)(a.x_out + (size_t)c.tok * d + n0()) = x;
        if (a.x_keep) *(float4*)(a.x_keep + (size_t)(len + c.tok) * d + n0()) = x;
    }
}

// The last `heads` workgroups: a head each, of the self-attention and of the cross-attention (query included).
template <bool GATED, bool PACK, class Cut, class Walk>
__device__ __forceinline__ void header(Walk& c, const PassArgs& a, int groups) {
    constexpr int KD = Cut::KD;
    constexpr bool RD = Walk::template side<KD>() > 1;
    const int base = groups - a.heads, h = c.wg - base;
    int T = a.T, d = a.d, I = a.I;
    const int len = *a.len_ptr, nsrc = a.cross ? *a.nsrc_ptr : 0;
    const float* relb = nullptr;
    if (a.rel_bias) {
        float* r = (float*)(c.lds + kRel);
        const int n = 2 * a.rel_d + 1;
        for (int i = threadIdx.x; i < n; i += kPassThreads) r[i] = a.rel_bias[(size_t)h * n + i];
        relb = r;
    }
    uint4 Wc[KD * 4];  // of the cross query
    const CLayer* L = (const CLayer*)(uintptr_t)a.layers;
    char* z = c.scratch(a);
    if (a.cross) request<KD, 4>(c, Wc, L->cwq, h, d >> c.KS, I >> 4);
    if (a.rel_bias) lds_barrier();  // (a wave reads biases that others have left, and the first scores come before any other barrier)
    for (int l = 0; l < a.n_layers; ++l, z = c.next(z, a.at.layer), c.walk_on(a.at.layer)) {
        L = (const CLayer*)(uintptr_t)a.layers + l;
        asm volatile("" : "+v"(c.lane));
        asm volatile("" : "+s"(T), "+s"(d), "+s"(I));
        c.place(T, a.room);
        Attend<true, PACK, Walk> self = {whole(L->kc + (size_t)h * 64 * c.ESZ), whole(L->vc + (size_t)h * 64 * a.vcap * c.ESZ), I, a.vcap, len, (len + Walk::BK - 1) / Walk::BK, {}, {}, {}, {}};
        if (c.wave < self.nblk) self.load(c, self.K0, self.V0, c.wave);
        // the cross-attention's keys and values while the heads have nothing else to do
        Attend<false, PACK, Walk> cross = {whole(L->ck + (size_t)h * 64 * c.ESZ), whole(L->cv + (size_t)h * 64 * a.scap * c.ESZ), I, a.scap, nsrc, (nsrc + Walk::BK - 1) / Walk::BK, {}, {}, {}, {}};
        if (a.cross) {
            cross.load(c, cross.K0, cross.V0, c.wave);
            if (!Walk::F32 && cross.nblk > kPassWaves) cross.load(c, cross.K1, cross.V1, c.wave + kPassWaves);
        }
        {
            const int room = Walk::ROOM1 ? 1 : fresh_room(c.R);
            const Fresh fresh = {whole(pinned(z + a.at.q + h * c.R * 256)), whole(pinned(z + a.at.k + h * c.R * 64 * c.ESZ)), whole(pinned(z + a.at.v + h * room * 256)), room};
            char* out = pinned(z + a.at.a1);
            const float sc = a.att_scale;
            self.run(c, fresh, sc, len, relb, a.rel_d, out, h);
            if (!a.cross) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (waves without keys wait for nothing else)
        }
        if (a.cross) {
            const char* xs = pinned(z + a.at.x2);
            char* out = pinned(z + a.at.a2);
            const float sc = a.att_scale;
            f32x4 acc[4];
            multiply<KD, 4, PACK, true>(c, acc, Wc, xs, d >> c.KS);
            leave<4, true, RD>(c, acc);
            if (c.wave < 4) {
                const f32x4 s = total<4, PACK, RD>(c, c.wave) * norm_factor(c, d, a.eps);
                if constexpr (Walk::F32) *(f32x4*)((float*)(c.lds + kQ) + c.tok * kQLd + c.wave * 16 + c.g * 4) = s;
                else *(v4u*)(c.lds + kQ + c.tok * kQLd * 4 + c.wave * 64 + c.g * 16) = query_parts(s * sc);
            }
            lds_barrier();
            cross.run(c, Fresh{}, sc, len, nullptr, 0, out, h);
            if (l + 1 < a.n_layers) request<KD, 4>(c, Wc, L[1].cwq, h, d >> c.KS, I >> 4);
        }
    }
}

template <bool GATED, bool DIE, bool F32, int ROOM>
__global__ __launch_bounds__(kPassThreads, 1) void pass_kernel(const PassArgs a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    using Cut = std::conditional_t<F32, DieCutF32, std::conditional_t<DIE, DieCut, ChipCut>>;
    constexpr bool PACK = !F32 && ROOM <= 8;
    Walk<DIE, F32, ROOM> c;
    c.lds = smem;
    c.failed = a.sync + kPassSyncWords - 1;
    c.spins = a.spins;
    c.wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    c.lane = (int)threadIdx.x & 63;
    c.wg = (int)blockIdx.x;
    if constexpr (DIE) {  // the workgroups of die 0 in the order in which they get here
        if (__builtin_amdgcn_s_getreg((3 << 11) | 20) != 0) return;
        if (threadIdx.x == 0) {
            unsigned rank;
            asm volatile("global_atomic_add %0, %1, %2, off sc0\n\ts_waitcnt vmcnt(0)" : "=v"(rank) : "v"(a.sync), "v"(1u) : "memory");
            *(unsigned*)smem = rank;
        }
        lds_barrier();
        c.wg = __builtin_amdgcn_readfirstlane(*(volatile int*)smem);
        if (c.wg >= a.groups) return;
        lds_barrier();
    }
    c.place(a.T, a.room);
    c.dead = false;
    if (c.wg < a.groups - a.heads) worker<GATED, PACK, Cut>(c, a, a.groups);
    else header<GATED, PACK, Cut>(c, a, a.groups);
}

// The same on one die for one row, with LM head and policy (pass_head.h): die 0 walks the layers, the others have the head.
template <bool GATED, bool F32>
__global__ __launch_bounds__(kPassThreads, 1) void pass_head_kernel(const PassArgs a, const PassHead head) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    using Cut = std::conditional_t<F32, DieCutF32, DieCut>;
    constexpr bool PACK = !F32;
    HeadWalk<F32> c;
    c.lds = smem;
    c.failed = a.sync + kPassSyncWords - 1;
    c.spins = a.spins;
    c.wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    c.lane = (int)threadIdx.x & 63;
    c.dead = false;
    c.place(1, 1);
    if (__builtin_amdgcn_s_getreg((3 << 11) | 20) != 0) {
        head_part<Cut>(c, a, head);
        return;
    }
    if (threadIdx.x == 0) {
        unsigned n;
        asm volatile("global_atomic_add %0, %1, %2, off sc0\n\ts_waitcnt vmcnt(0)" : "=v"(n) : "v"(head.started), "v"(1u) : "memory");
        *(unsigned*)smem = n;
    }
    lds_barrier();
    const unsigned before = (unsigned)__builtin_amdgcn_readfirstlane(*(volatile int*)smem);  // (32 a pass)
    c.wg = (int)(before & 31u);
    c.odd = (before >> 5) & 1u;
    if (c.wg >= a.groups) return;
    lds_barrier();
    if (c.wg < a.groups - a.heads) worker<GATED, PACK, Cut>(c, a, a.groups, head);
    else header<GATED, PACK, Cut>(c, a, a.groups);
}

template <class Cut>
static int cut_groups(int d, int heads, int F, bool gated) {
    return std::max(std::max(ceil_div(3 * heads * 4, Cut::QT), ceil_div(gated ? F / 8 : F / 16, Cut::FT)), ceil_div(d / 16, Cut::OT)) + heads;
}
template <class Cut>
static bool cut_fits(int d, int I, int F, int inputs) {
    return ceil_div(std::max(d, I) / inputs, kPassWaves) <= Cut::KD && ceil_div(F / inputs, kPassWaves) <= Cut::KF;
}

// Sizes the kernel is made for: runs of inputs that fit the registers, the workgroups on the chip at once.  Wider models: pass_wide.hip.
// last: see pass_last.  Apart, a pass may take every compute unit there is (one row of the mT5-large shape, 64 + 176 + 16): another stream's
// kernel on one of them then holds it up until that ends or the workgroups give up and it runs again as kernels.  The arrangement with the first ones
// leaves 48 of 256 free at the mT5-large shape and takes 360 us instead of 342 for one row there; a state takes either only while it is alone inside a call.
int pass_groups(int d, int heads, int d_head, int F, bool gated, int cus, bool last) {
    if (d_head != 64 || d % 256 != 0 || F % 32 != 0 || !cut_fits<ChipCut>(d, heads * 64, F, 32)) return 0;
    const int g = cut_groups<ChipCut>(d, heads, F, gated), apart = d / 16 + ceil_div(gated ? F / 8 : F / 16, ChipCut::FT) + heads;
    return last && apart <= cus ? std::max(g, apart) : g <= cus ? g : 0;
}
// Whether the FFN's input and q, k, v are the last workgroups' over the chip, apart from the owners of features, or the first ones'.  It pays where the
// weights of a pass come from memory (`bytes` of them, which the 256 MiB of the last-level cache do not hold from pass to pass), one row always, more
// rows where the FFN's output weights, which an owner asks for as well, are many.  us, 64 source tokens, first / last, 1, 2, 4, 8, 11 rows, 1024
// wide, 16 heads: d_ff 4096, 8 layers (256 MiB) 118, 135, 142, 150, 177 / 120, 136, 144, 152, 181, 9 layers 139, 155, 163, 173, 206 / 133, 154, 162,
// 171, 205, 24 layers 370, 406, 426, 449, 539 / 344, 389, 412, 431, 528; 24 layers of 3584 360, 399, 418, 442, 530 / 336, 386, 409, 430, 517, of 3072 349, 389,
// 406, 428, 510 / 327, 383, 402, 423, 496 (512 tokens 356, 404, 419, 435, 515 / 346, 402, 421, 440, 511), of 2560 342, 382, 395, 415, 494 / 326, 381, 399, 419, 485 (512
// tokens 423 / 436 for eight rows), of 2048 332, 371, 381, 400, 474 / 321, 379, 392, 415, 474; gated, 2816, 24 layers 360, 410, 423, 445, 526 / 342, 410, 428, 447, 529, 8 layers 122, 142, 147, 153,
// 179 / 122, 142, 148, 157, 186.  768 wide, d_ff 3072, 12 layers (216 MiB) 157, 178, 187, 197, 230 / 158, 178, 186, 197, 231, 24 layers 319, 351, 369, 388, 456 / 303, 349, 362,
// 381, 454.  Narrower models, held by the cache, are 0 to 2 % faster with the last ones, gated ones above eight rows 2 to 4 % slower.
// The line lies where the two are about the same in requests, whose reviews by a larger model come in between and whose caches are read as well: rounds
// of eight small steps and a review, 64 source tokens, us a step that the last ones take more (+) or less, small model of 4, 5, 6, 7 layers with its head, by d_ff of
// 1024-wide models: 4096 (191, 223, 255, 287 MiB) +1.1, -1.4, -2.0, -4.8, as early exit +0.9, +1.8, +2.0, -4.6; gated, 2816 (193, 225, 258, 290 MiB) +0.4, 0, -0.8,
// -3.2, as early exit +0.2, 0, +0.7, -2.8; 768 wide, d_ff 3072, 8, 10, 11, 12 layers (191, 227, 245, 263 MiB) -0.6, -0.2, -1.8, -2.2, as early exit +1.7, -2.4, -1.1,
// -2.6; of steps of 80 to 130 us.  1024 wide, d_ff 2048, 7, 8, 9 layers (231, 255, 279 MiB) +1.3, +2.1, +0.7, as early exit +4.2, +1.9, +1.9: there the line could
// lie higher.  With 512 source tokens the six layers of the T5-large shape as early exit, three small steps between reviews, take 14.73 ms a request with the first
// ones and 14.55 with the last.
bool pass_last(int d, int F, bool gated, int T, size_t bytes) {
    if (d < 768) return !(gated && T > 8);
    return bytes > (size_t)250 << 20 && (T == 1 || F >= 3 * d);
}
// ... and of the form on one die: all of it on the 32 compute units of one.
int pass_die_groups(int d, int heads, int d_head, int F, bool gated, bool f32) {
    if (d_head != 64 || d % 256 != 0 || F % 32 != 0 || !(f32 ? cut_fits<DieCutF32>(d, heads * 64, F, 16) : cut_fits<DieCut>(d, heads * 64, F, 32))) return 0;
    const int g = f32 ? cut_groups<DieCutF32>(d, heads, F, gated) : cut_groups<DieCut>(d, heads, F, gated);
    return g <= 32 ? g : 0;
}

void pass_head_plan(PassHead& h, const PassPlan& at, int d, bool f32, int cus) {
    const int x = d / (f32 ? 16 : 32) * tile_bytes(true, 1, f32), nv = f32 ? HeadCut<true>::NV : HeadCut<false>::NV;
    h.groups = cus - cus / 8;  // (workgroups go to the eight dies in turn)
    h.at = 3 * at.layer;
    h.rec = (x + 255) / 256 * 256;
    h.bytes = (h.rec + h.groups * nv * 16 + 255) / 256 * 256;
}

PassPlan pass_plan(int room, int d, int I, int F, bool f32, bool wide) {
    PassPlan p;
    size_t at = 0;
    auto take = [&](size_t bytes) {
        const size_t r = at;
        at += (bytes + 255) / 256 * 256;
        return (int)r;
    };
    const int inputs = f32 ? 16 : 32;
    const size_t x = (size_t)(d / inputs) * (tile_bytes(true, room, f32) + (room > 16 ? 128 : 0)), i = (size_t)(I / inputs) * tile_bytes(false, room, f32);
    p.x1 = take(x); p.q = take((size_t)room * I * 4); p.k = take((size_t)room * I * (f32 ? 4 : 2)); p.v = take((size_t)fresh_room(room) * I * 4);
    p.a1 = take(i); p.x2 = take(x);
    p.a2 = wide ? 0 : take(i); p.x3 = wide ? 0 : take(x);  // (cross-attention)
    p.h = take((size_t)(F / inputs) * tile_bytes(false, room, f32));
    if (wide) {
        p.part = take((size_t)kWideSplits * room * I * 4);
        p.top = take((size_t)kWideSplits * room * (I / kWideHead) * 8);
    }
    p.layer = (int)at;
    return p;
}

hipError_t pass_init() {
    static hipError_t done = [] {
#define BILD_P(DV, FV, RV) (const void*)pass_kernel<false, DV, FV, RV>, (const void*)pass_kernel<true, DV, FV, RV>
        const void* fns[] = {BILD_P(true, false, 1), BILD_P(true, false, 2), BILD_P(true, false, 4), BILD_P(false, false, 1), BILD_P(false, false, 2), BILD_P(false, false, 4),
                             BILD_P(false, false, 8), BILD_P(false, false, 16), BILD_P(true, true, 1), BILD_P(true, true, 0),
                             (const void*)pass_head_kernel<false, false>, (const void*)pass_head_kernel<true, false>,
                             (const void*)pass_head_kernel<false, true>, (const void*)pass_head_kernel<true, true>};
#undef BILD_P
        return raise_lds_limit(fns, 160 * 1024);
    }();
    return done;
}

hipError_t launch_pass(const PassArgs& a, const PassHead* head, int grid, hipStream_t st) {
    if (hipError_t e = pass_init(); e != hipSuccess) return e;
    if (a.groups < 1 || grid < a.groups || a.T < 1 || a.T > kPassRows || a.room < a.T || (a.die && !a.f32 && a.T > kPassDieRows) || (a.f32 && !a.die) || !a.turn || !a.layers || !a.sync || !a.scratch || !a.x_out || !a.len_ptr ||
        (a.cross && !a.nsrc_ptr) || (head && (!a.die || a.room != 1 || !head->w || !head->gain || !head->started || grid != 256 || head->groups != grid - grid / 8 || !head->f.ctl)))
        return hipErrorInvalidValue;
    const size_t smem = kRel + (a.rel_bias ? (size_t)(2 * a.rel_d + 1) * 4 : 0);
    if (smem > 160 * 1024) return hipErrorInvalidValue;
    const bool gated = a.act != BILD_ACT_RELU;
#define BILD_PH(FV)                                                                                                           \
    do {                                                                                                                     \
        if (gated) hipLaunchKernelGGL((pass_head_kernel<true, FV>), dim3(grid), dim3(kPassThreads), smem, st, a, *head);     \
        else hipLaunchKernelGGL((pass_head_kernel<false, FV>), dim3(grid), dim3(kPassThreads), smem, st, a, *head);          \
        return hipGetLastError();                                                                                            \
    } while (0)
#define BILD_P(DV, FV, RV)                                                                                                   \
    do {                                                                                                                     \
        if (gated) hipLaunchKernelGGL((pass_kernel<true, DV, FV, RV>), dim3(grid), dim3(kPassThreads), smem, st, a);         \
        else hipLaunchKernelGGL((pass_kernel<false, DV, FV, RV>), dim3(grid), dim3(kPassThreads), smem, st, a);              \
        return hipGetLastError();                                                                                            \
    } while (0)
    if (head && a.f32) BILD_PH(true);
    if (head) BILD_PH(false);
    if (a.f32 && a.room == 1) BILD_P(true, true, 1);
    if (a.f32) BILD_P(true, true, 0);
    if (a.die && a.room == 1) BILD_P(true, false, 1);
    if (a.die && a.room == 2) BILD_P(true, false, 2);
    if (a.die && a.room == 4) BILD_P(true, false, 4);
    if (!a.die && a.room == 1) BILD_P(false, false, 1);
    if (!a.die && a.room == 2) BILD_P(false, false, 2);
    if (!a.die && a.room == 4) BILD_P(false, false, 4);
    if (!a.die && a.room == 8) BILD_P(false, false, 8);
    if (!a.die && a.room == 16) BILD_P(false, false, 16);
#undef BILD_P
#undef BILD_PH
    return hipErrorInvalidValue;
}

}  // namespace bild
