// One decoder pass of a wide bf16 model without cross-attention (above 1024 and up to 4096 wide, heads of 128) in ONE kernel, up to
// eight rows, or sixteen, or thirty-two (wide_rows): pass_kernel.hip's way of handing results over (its head explains it; nothing is counted, results are their own flags),
// for layers of 60 to 400 MB.
//
// Bound: the weights from memory.  As kernels of their own the six stages of a layer each end with a few microseconds in which the
// memory has little to do (the last workgroups, the launch, the trip for the activations, cold instructions) and attention keeps it
// idle for ten; here a workgroup per compute unit stays, and asks for the next stage's weights before that stage's activations exist:
//
//   - two pieces of a stage's weights wait in registers (8 to 16 KB a wave, up to 256 KB a compute unit), the rest follow while they
//     are multiplied.  A compute unit takes new requests only as fast as the old ones are answered, so a request that is not the
//     critical path's holds up what comes behind it: results are published BEFORE the next stage's weights are asked for, and the
//     other waves wait for that too (with the requests first, publishing took 2 to 13 us of each stage: 2048-wide, 16 layers, 527 us
//     either way because the weights then come later; 4096-wide, 8 layers, 708 -> 663);
//   - models up to 2048 wide ask for all of the FFN's first weights already when q, k and v are handed over, which keeps the memory
//     busy while the heads work (536 -> 455 us, with heads and projections together); so much of a 4096-wide model's would only delay the output projection's activations
//     (663 -> 685).  Asking for the FFN's second weights or the next layer's first ones a stage earlier loses for the same reason
//     (455 -> 466, 482);
//   - a head's keys are cut into ranges of at least 256 keys, eight at most, a workgroup each, whose waves take blocks of 32; the
//     ranges' results are handed over once more and each of the head's workgroups joins 128 / ranges of its features;
//   - a workgroup has the same sixteen features of the residual stream in all layers: they stay in registers.
//
// us per pass with the LM head, separate kernels / this, at 1064 positions: 2048-wide, 16 layers, 1, 2, 4, 8 rows 661, 731, 784, 805 /
// 437, 443, 462, 500; 4096-wide, 8 layers 772, 836, 838, 841 / 663, 667, 679, 714, of which the layers' weights alone take 270 and 530 at
// the 6.1 TB/s of a large copy.  Heads and projections apart, up to 1280 keys (see wide_kernel), before / with: 457, 461, 480, 514 / 442,
// 444, 462, 500; a load of several tiles' activations for one and two rows (run_few) 442, 444 / 437, 443 and at 200 positions 413, 420 /
// 409, 413.
// Nine to sixteen rows have high and low parts in operands of their own, twice the activations and products; the weights still take longer.  The 7B shape, nine, sixteen
// rows over 64, 1024, 4097 tokens, separate kernels / this, us: 3305, 3311, 3463, 3473, 3770, 3779 / 2837, 2843, 2918, 2927, 3239, 3246 (eight rows 2591, 2680, 2993); six
// layers of 2304 (without gate), 2560, 3072, 4096 (without gate) and of 1536 with a hidden state of 8192, twelve rows over 64 and 8100 tokens 336, 410, 452, 522, 387 and 501, 576, 618, 703, 458 / 338, 381, 415,
// 474, 322 and 466, 528, 582, 675, 424.  Seventeen to thirty-two have two row tiles (figures at wide_keys).
#include "pass_walk.h"

namespace bild {

// What the lane j on has (of sixteen; j is a constant once unrolled).
template <int J = 1>
__device__ __forceinline__ uint4 lanes_on(const uint4& v, int j) {
    if constexpr (J < 8) {
        if (j == 0) return v;
        if (j != J) return lanes_on<J + 1>(v, j);
        return make_uint4(__builtin_amdgcn_update_dpp(0, v.x, 0x100 + J, 0xF, 0xF, true), __builtin_amdgcn_update_dpp(0, v.y, 0x100 + J, 0xF, 0xF, true),
                          __builtin_amdgcn_update_dpp(0, v.z, 0x100 + J, 0xF, 0xF, true), __builtin_amdgcn_update_dpp(0, v.w, 0x100 + J, 0xF, 0xF, true));
    }
    return v;
}

// (a layout of its own where rows are few: a producer's sum of squares is not behind its features here)
template <int ROOM>
struct WideWalk : Walk<false, false, ROOM> {
    static constexpr bool ROOM1 = false;
    static constexpr bool PACKED = ROOM <= 8;  // high and low parts in one operand (multiply() in pass_walk.h); above eight rows one each
    static constexpr int P = PACKED ? 1 : 2;
    static constexpr int NT = ROOM == 32 ? 2 : 1;  // row tiles of sixteen
    float ss2;                                     // as ss, of the second row tile
    __device__ __forceinline__ int row(int u = 0) const { return NT > 1 ? min(u * 16 + this->tok, this->T - 1) : PACKED ? this->t8 : this->t; }
};
// (thirty-two rows' sums of squares take twice the place)
template <class Walk>
__device__ __forceinline__ int tile_size(const Walk& c, bool normed) {
    return tile_bytes(normed, c.R, false) + (Walk::NT > 1 && normed ? 128 : 0);
}
// The waves' results side by side in LDS, and the rows' factors (leave(), norm_factor() in pass_walk.h).  Two row tiles take both halves of that memory:
// a barrier behind every stage's results keeps the next one's away from them.
template <int RW, bool NORM, class Walk>
__device__ __forceinline__ void leave_rows(Walk& c, const f32x4 (&acc)[RW * Walk::NT]) {
    if constexpr (Walk::NT == 1) {
        leave<RW, NORM, false>(c, acc);
    } else {
        static_assert(kPassWaves * RW * Walk::NT * 1024 <= 2 * kRedBytes, "room for both row tiles' sums");
        if (NORM && c.g < 2) *(float*)(c.lds + kSq + (c.wave * 32 + c.g * 16 + c.tok) * 4) = c.g ? c.ss2 : c.ss;
#pragma unroll
        for (int q = 0; q < RW * Walk::NT; ++q) *(f32x4*)(c.lds + kRed + ((c.wave * RW * Walk::NT + q) * 64 + c.lane) * 16) = acc[q];
        lds_barrier();
    }
}
template <class Walk>
__device__ __forceinline__ float row_factor(const Walk& c, int d, float eps, int u) {
    if constexpr (Walk::NT == 1) return norm_factor(c, d, eps);
    float p[kPassWaves], s = 0.f;
#pragma unroll
    for (int v = 0; v < kPassWaves; ++v) p[v] = *(const float*)(c.lds + kSq + (v * 32 + u * 16 + c.tok) * 4);
#pragma unroll
    for (int v = 0; v < kPassWaves; ++v) s += p[v];
    return __builtin_amdgcn_rsqf(s * __builtin_amdgcn_rcpf((float)d) + eps);
}
// put_planes() of row tile u
template <bool PACK, bool NORM, class Walk>
__device__ __forceinline__ void put_rows(const Walk& c, void* planes, int n0, const float (&w)[4], int u) {
    if constexpr (Walk::NT == 1) {
        put_planes<PACK, NORM>(c, planes, n0, w);
    } else {
        const int row = u * 16 + c.tok, off = (n0 >> 5) * tile_size(c, NORM) + (((n0 >> 4) & 1) * 2 + (c.g >> 1)) * 16 * c.R + (c.g & 1) * 64 * c.R + row * 16;
        const v4u v = query_parts(f32x4{w[0], w[1], w[2], w[3]});  // (eight features' high parts to the even lane groups, their low parts to the odd ones)
        if (row < c.T) __builtin_amdgcn_raw_buffer_store_b128(v, whole(planes), off, 0, Walk::kOut);
        __builtin_amdgcn_raw_buffer_store_b128(v4u{kNotThere, kNotThere, kNotThere, kNotThere}, whole((const char*)planes + c.clear), off, 0, Walk::kOut);
    }
}

// A projection's weights on their way: N input tiles per wave at most, RW feature tiles, in pieces of CH input tiles of which two
// are requested before their activations are there.  The next piece's activations are requested ahead of the weights that follow
// (a wave's loads come back in order).
template <int N, int RW, int CH, bool NORM>
struct Stream {
    static constexpr int NC = (N + CH - 1) / CH, SQ = (CH + 3) / 4;
    uint4 W[NC > 1 ? 2 : 1][CH * RW];

    struct Where {
        Rsrc rs;
        int k0, n, tk, most;
    };
    // (tiles first .. end - 1; past the last one: that one again.  Without a request there: 4096-wide, 8 rows, 0.7 % more)
    __device__ __forceinline__ static Where where(int wave, const void* w, int first, int tk, int end) {
        const Run r = run_of(wave, tk);
        return {whole((const char*)w + (size_t)first * tk * kTileBytes), min(r.k0, tk - 1), r.n, tk, end - 1 - first};
    }
    __device__ __forceinline__ static void ask(int lane, uint4 (&w)[CH * RW], const Where& a, int i) {
#pragma unroll
        for (int j = 0; j < CH; ++j)
            if (i * CH + j < N) {
                const int k = a.k0 + min(i * CH + j, max(a.n - 1, 0));  // (past the wave's last tile: that one again, not used)
#pragma unroll
                for (int q = 0; q < RW; ++q) w[j * RW + q] = buf_load(a.rs, (unsigned)lane * 16u, ((RW == 1 ? 0 : min(q, a.most)) * a.tk + k) * kTileBytes);
            }
    }
    // (the registers hold nothing: without this they would be kept through the paths on which they are not filled anew)
    __device__ __forceinline__ void forget() {
#pragma unroll
        for (uint4 (&w)[CH * RW] : W)
#pragma unroll
            for (uint4& v : w) asm volatile("" : "=v"(v.x), "=v"(v.y), "=v"(v.z), "=v"(v.w));
    }
    template <class Walk>
    __device__ __forceinline__ void open(const Walk& c, const void* w, int first, int tk, int end) {
        const Where a = where(c.wave, w, first, tk, end);
        ask(c.lane, W[0], a, 0);
        if constexpr (NC > 1) ask(c.lane, W[1], a, 1);
    }
    // acc = W x over this wave's inputs
    template <class Walk>
    __device__ __forceinline__ void run(Walk& c, f32x4 (&acc)[RW * Walk::NT], const void* planes, const void* weights, int first, int tk, int end) {
        const Where a = where(c.wave, weights, first, tk, end);
        const int k0 = a.k0, n = a.n;
        const Rsrc xs = whole(planes);
        if constexpr (Walk::KNOWN == 1 || Walk::KNOWN == 2) return run_few(c, acc, xs, a);
        constexpr int P = Walk::P, NT = Walk::NT, XL = P * NT;  // loads of a tile
        const int S = tile_size(c, NORM);
        int at[NT];
#pragma unroll
        for (int u = 0; u < NT; ++u) at[u] = (Walk::PACKED ? (c.g * 2 + (c.tok >> 3)) * c.R + c.row() : c.g * c.R + c.row(u)) * 16;
        uint4 X[NC > 1 ? 2 : 1][CH * XL];
        v2u sq[NC > 1 ? 2 : 1][SQ * NT];
        float ss = 0.f, ss2 = 0.f;
        auto get = [&](uint4 (&x)[CH * XL], v2u (&s)[SQ * NT], int i) {
#pragma unroll
            for (int j = 0; j < CH; ++j)
                if (i * CH + j < N) {
#pragma unroll
                    for (int p = 0; p < XL; ++p) x[XL * j + p] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xs, at[p / P] + p % P * c.R * 64, (k0 + min(i * CH + j, max(n - 1, 0))) * S, Walk::kIn));
                }
            if constexpr (NORM) {  // (lane group g: tiles g, g + 4 of the piece)
#pragma unroll
                for (int u = 0; u < SQ * NT; ++u)
                    s[u] = __builtin_bit_cast(v2u, __builtin_amdgcn_raw_buffer_load_b64(xs, min(i * CH + u / NT * 4 + c.g, max(n - 1, 0)) * S + c.R * 128 + c.row(u % NT) * 8, k0 * S, Walk::kIn));
            }
        };
        auto missing = [&](const uint4 (&x)[CH * XL], const v2u (&s)[SQ * NT], int i) {
            unsigned m = 0u;
#pragma unroll
            for (int j = 0; j < CH * XL; ++j)
                if (i * CH + j / XL < N) m = max(max(m, max(x[j].x, x[j].y)), max(x[j].z, x[j].w));
            if constexpr (NORM) {
#pragma unroll
                for (int u = 0; u < SQ * NT; ++u) m = max(m, max(s[u].x, s[u].y));
            }
            return __builtin_amdgcn_ballot_w64(m == kNotThere) != 0ull && !c.dead;
        };
#pragma unroll
        for (int q = 0; q < RW * NT; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
        get(X[0], sq[0], 0);
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            uint4 (&x)[CH * XL] = X[i & 1];
            v2u (&s)[SQ * NT] = sq[i & 1];
            // (the first look apart: the wait of a loop would be for everything requested since)
            if (__builtin_expect(missing(x, s, i), 0)) {
                int tries = 0;
                bool more;
#pragma unroll 1
                do {
                    asm volatile("" ::: "memory");
                    get(x, s, i);
                    more = missing(x, s, i);
                } while (more && ++tries < c.spins);
                if (more) c.give_up();
            }
            __builtin_amdgcn_sched_barrier(0);
            if (i + 1 < NC) get(X[(i + 1) & 1], sq[(i + 1) & 1], i + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < CH; ++j)
                if (i * CH + j < N && i * CH + j < n) {
#pragma unroll
                    for (int p = 0; p < XL; ++p)
#pragma unroll
                        for (int q = 0; q < RW; ++q) acc[q * NT + p / P] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf(W[i & 1][j * RW + q]), as_bf(x[XL * j + p]), acc[q * NT + p / P], 0, 0, 0);
                }
            if constexpr (NORM) {
#pragma unroll
                for (int u = 0; u < SQ; ++u)
                    if (u * 4 + c.g < CH && i * CH + u * 4 + c.g < n) {
                        ss += __uint_as_float(s[u * NT].x) + __uint_as_float(s[u * NT].y);
                        if constexpr (NT > 1) ss2 += __uint_as_float(s[u * NT + NT - 1].x) + __uint_as_float(s[u * NT + NT - 1].y);
                    }
            }
            __builtin_amdgcn_sched_barrier(0);
            if (i + 2 < NC) ask(c.lane, W[i & 1], a, i + 2);
        }
        if constexpr (NORM) c.ss = quad_rows_sum(ss);
        if constexpr (NORM && NT > 1) c.ss2 = quad_rows_sum(ss2);
    }
    // One or two rows: a load brings eight tiles' activations, or four tiles' (see multiply() in pass_walk.h for what a load takes
    // however few of its bytes differ): columns (tile, row) of a tile's high and low parts, which move down to the rows' own for its
    // products.  What is in the other columns then is no row's.  All of a wave's activations are asked for at once, its tiles'
    // sums of squares in a load or two.
    template <class Walk>
    __device__ __forceinline__ void run_few(Walk& c, f32x4 (&acc)[RW], const Rsrc xs, const Where& a) {
        constexpr int R = Walk::KNOWN, SIDE = 8 / R, NX = (N + SIDE - 1) / SIDE, NS = NORM ? (N * R + 15) / 16 : 0;
        const int S = tile_bytes(NORM, R, false), last = max(a.n - 1, 0), row = min(c.tok & (R - 1), c.T - 1);
        const int at = ((c.g * 2 + (c.tok >> 3)) * R + row) * 16, beside = (c.tok & 7) / R;
        uint4 X[NX];
        v2u sq[NS + 1];
        auto get = [&] {
#pragma unroll
            for (int i = 0; i < NX; ++i) X[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xs, at + min(i * SIDE + beside, last) * S, a.k0 * S, Walk::kIn));
#pragma unroll
            for (int i = 0; i < NS; ++i) sq[i] = __builtin_bit_cast(v2u, __builtin_amdgcn_raw_buffer_load_b64(xs, min((i * 16 + c.tok) / R, last) * S + R * 128 + row * 8, a.k0 * S, Walk::kIn));
        };
        auto missing = [&] {
            unsigned m = 0u;
#pragma unroll
            for (int i = 0; i < NX; ++i) m = max(max(m, max(X[i].x, X[i].y)), max(X[i].z, X[i].w));
#pragma unroll
            for (int i = 0; i < NS; ++i) m = max(m, max(sq[i].x, sq[i].y));
            return __builtin_amdgcn_ballot_w64(m == kNotThere) != 0ull && !c.dead;
        };
        get();
        if (__builtin_expect(missing(), 0)) {
            int tries = 0;
            bool more;
#pragma unroll 1
            do {
                asm volatile("" ::: "memory");
                get();
                more = missing();
            } while (more && ++tries < c.spins);
            if (more) c.give_up();
        }
        if constexpr (NORM) {
            float ss = 0.f;
#pragma unroll
            for (int i = 0; i < NS; ++i) ss += (i * 16 + c.tok) / R < a.n ? __uint_as_float(sq[i].x) + __uint_as_float(sq[i].y) : 0.f;
            ss += dpp_f<0x128, 0xF>(0.f, ss);  // row_ror
            ss += dpp_f<0x124, 0xF>(0.f, ss);
            ss += dpp_f<0x122, 0xF>(0.f, ss);
            if constexpr (R == 1) ss += dpp_f<0x121, 0xF>(0.f, ss);
            c.ss = ss;
        }
#pragma unroll
        for (int q = 0; q < RW; ++q) acc[q] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int j = 0; j < CH; ++j)
                if (i * CH + j < N && i * CH + j < a.n) {
                    const int tile = i * CH + j;
                    const uint4 x = lanes_on(X[tile / SIDE], tile % SIDE * R);
#pragma unroll
                    for (int q = 0; q < RW; ++q) acc[q] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf(W[i & 1][j * RW + q]), as_bf(x), acc[q], 0, 0, 0);
                }
            __builtin_amdgcn_sched_barrier(0);
            if (i + 2 < NC) ask(c.lane, W[i & 1], a, i + 2);
        }
    }
};

// One key range of a head: the waves of the head's workgroups take blocks of 32 keys in turn.
template <class Walk>
struct Range {
    const Rsrc kr, vr;
    const int I, cap, nblk;  // (blocks of the keys of earlier passes)
    uint4 K[2][4], V[8];

    __device__ __forceinline__ void load(const Walk& c, int blk) {
        const int key = min(blk, max(nblk - 1, 0)) * 32;
#pragma unroll
        for (int ab = 0; ab < 2; ++ab)
#pragma unroll
            for (int ks = 0; ks < 4; ++ks) K[ab][ks] = buf_load(kr, (unsigned)((c.tok * I + c.g * 8) * 2), ((key + ab * 16) * I + ks * 32) * 2);
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) {
            const int off = (dt * 16 * cap + key) * 2, vo = (c.tok * cap + c.g * 4) * 2;
            const uint2 x = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(vr, vo, off, 0));
            const uint2 y = __builtin_bit_cast(uint2, __builtin_amdgcn_raw_buffer_load_b64(vr, vo + 32, off, 0));
            V[dt] = make_uint4(x.x, x.y, y.x, y.y);
        }
    }
};

// (the attention's results [wave][8][64] take both halves of the sums' memory)
static_assert(2 * kRedBytes >= kPassWaves * 8 * 1024, "room for eight waves' results");

template <int QTV, int FTV, int KDV, int KFV, int QC, int FC, int OC = 8>
struct WideCut {
    static constexpr int QT = QTV, FT = FTV, KD = KDV, KF = KFV;  // as in pass_kernel.hip
    using Qkv = Stream<KD, QT, QC, true>;
    using Out = Stream<KD, 1, OC, false>;
    using In = Stream<KD, FT, FC, true>;
    using Ffn = Stream<KF, 1, OC, false>;
    static constexpr bool EARLY = In::NC <= 2;  // the FFN's first weights all fit the registers
};
// (pieces of the 4096-wide cut: 8 and 6 tiles a request of q, k, v and the FFN 669 and 673 us, 12 and 12 663, 15 and 18 the same)
using Cut2048 = WideCut<3, 4, 8, 24, 4, 4>;
using Cut2048Two = WideCut<2, 4, 8, 24, 4, 4>;
using Cut4096 = WideCut<3, 6, 16, 44, 4, 2>;
using Cut4096Rows = WideCut<3, 6, 16, 44, 2, 1, 4>;  // two row tiles: four loads of activations a tile

__host__ __device__ inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Key ranges of a head: 256 keys each, a power of two, as long as there are workgroups.
__host__ __device__ inline int wide_splits(int nkeys, int heads, int groups) {
    int s = 1;
    while (s < kWideSplits && s * 256 < nkeys && heads * s * 2 <= groups) s *= 2;
    return s;
}

// Who does what: the first workgroups with q, k, v and the FFN's input, and the heads (head0, each in `ranges`).
// Apart, up to 1280 keys: the heads are the first workgroups', in ranges that half of those with features
// of the residual stream hold, q, k, v and the FFN's input the last ones', so that these weights are asked for while the heads work and
// nobody's heads wait behind them.  More keys take more workgroups than that: the heads are the last ones', the rest begins
// with the first (q, k, v: see wide_two).
struct WideParts {
    bool apart;
    int q, i, head0, ranges;
};
template <class Cut>
__host__ __device__ inline WideParts wide_parts(int keys, int d, int heads, int tq, int tf, int groups) {
    WideParts p;
    p.apart = Cut::EARLY && keys <= kWideApart;
    p.q = p.apart ? groups - ceil_div(tq, Cut::QT) : 0;
    p.i = p.apart ? groups - ceil_div(tf, Cut::FT) : 0;
    p.ranges = wide_splits(keys, heads, p.apart ? d >> 5 : groups);
    p.head0 = p.apart ? 0 : groups - heads * p.ranges;
    return p;
}

// Workgroups [0, d / 16) own sixteen features of the residual stream each; the rest: wide_parts.
template <bool GATED, class Cut, int ROOM>
__global__ __launch_bounds__(kPassThreads, 1) void wide_kernel(const PassArgs a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    using Way = WideWalk<ROOM>;
    constexpr int QT = Cut::QT, FT = Cut::FT, DH = kWideHead;
    constexpr bool EARLY = Cut::EARLY, PACK = Way::PACKED;
    constexpr int P = Way::P, NT = Way::NT;
    Way c;
    c.lds = smem;
    c.failed = a.sync + kPassSyncWords - 1;
    c.spins = a.spins;
    c.wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    c.lane = (int)threadIdx.x & 63;
    c.wg = (int)blockIdx.x;
    c.dead = false;
    c.place(a.T, a.room);
    int T = a.T, d = a.d, I = a.I, F = a.F;
    const int len = *a.len_ptr;
    auto tq = [&] { return 3 * (I >> 4); };
    auto tf = [&] { return GATED ? F >> 3 : F >> 4; };
    const WideParts who = wide_parts<Cut>(len + T, d, a.heads * NT, tq(), tf(), a.groups);
    const int uq = c.wg - who.q, uf = c.wg - who.i;
    const int q0 = uq * QT, q1 = min(q0 + QT, tq()), i0 = uf * FT;  // tiles of the projections
    const bool owner = c.wg < d >> 4, qkv = uq >= 0 && q0 < tq(), ffn = uf >= 0 && i0 < tf();
    const bool mine = owner && c.wave < NT;  // (a row tile each)
    const int S = who.ranges, place = c.wg - who.head0;
    const bool att = place >= 0 && place < a.heads * NT * S;
    const int h = att ? place / (S * NT) : 0, rt = NT > 1 && att ? place / S % NT : 0, split = att ? place % S : 0;  // (rt: the row tile)

    float4 next_gain = make_float4(0.f, 0.f, 0.f, 0.f), x = make_float4(0.f, 0.f, 0.f, 0.f);
    auto n0 = [&] { return c.wg * 16 + c.g * 4; };
    auto gain = [&](const float* g) { return ldf4(whole(g), mine ? n0() * 4 : 0); };
    auto publish = [&](const float4& gn, char* planes) {
        if (!mine) return;
        const float w[4] = {x.x * gn.x, x.y * gn.y, x.z * gn.z, x.w * gn.w};
        const float ss = quad_rows_sum(x.x * x.x + x.y * x.y + x.z * x.z + x.w * x.w);
        put_rows<PACK, true>(c, planes, n0(), w, c.wave);
        if (c.g == 0) {
            const int row = NT > 1 ? c.wave * 16 + c.tok : c.tok;
            const int off = (n0() >> 5) * tile_size(c, true) + c.R * 128 + (row * 2 + ((n0() >> 4) & 1)) * 4;
            if (row < T) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(ss), whole(planes), off, 0, Way::kOut);
            if (row < c.R) __builtin_amdgcn_raw_buffer_store_b32(kNotThere, whole(planes + c.clear), off, 0, Way::kOut);
        }
    };
    auto add = [&] {
        const f32x4 s = total<NT, PACK, false>(c, NT > 1 ? c.wave : 0);
        x = make_float4(x.x + s[0], x.y + s[1], x.z + s[2], x.w + s[3]);
    };
    typename Cut::Qkv sq;
    typename Cut::Out so;
    typename Cut::In si;
    typename Cut::Ffn sf;
    const CLayer* L = (const CLayer*)(uintptr_t)a.layers;
    char* z = c.scratch(a);
    if (owner) {
        const int pos = len + (NT > 1 ? c.row(c.wave) : c.t);
        const float4 gn = gain(L->ln1);
        if (mine) {
            if (a.emb) {
                int er = a.tokens[pos] + a.tie_shift;
                er = er >= a.vocab ? er - a.vocab : er;
                const char* p = (const char*)a.emb + ((size_t)(er >> 4) * (d >> 5) + (n0() >> 5)) * kTileBytes + ((er & 15) + 16 * ((n0() & 31) >> 3)) * 16 + (n0() & 7) * 2;
                const uint2 raw = *(const uint2*)p;
                float4 pe = make_float4(0.f, 0.f, 0.f, 0.f);
                if (a.pe) pe = *(const float4*)(a.pe + (size_t)pos * d + n0());
                const float sc = a.embed_scale;
                x = make_float4(__builtin_fmaf(bf2f(raw.x & 0xFFFFu), sc, pe.x), __builtin_fmaf(bf2f(raw.x >> 16), sc, pe.y),
                                __builtin_fmaf(bf2f(raw.y & 0xFFFFu), sc, pe.z), __builtin_fmaf(bf2f(raw.y >> 16), sc, pe.w));
            } else {
                x = *(const float4*)(a.x_in + (size_t)pos * d + n0());
            }
        }
        publish(gn, z + a.at.x1);
    }
    sq.forget();
    if (qkv) sq.open(c, L->wqkv, q0, d >> 5, q1);
    for (int l = 0; l < a.n_layers; ++l) {
        L = (const CLayer*)(uintptr_t)a.layers + l;
        const bool last = l + 1 == a.n_layers;
        asm volatile("" : "+v"(c.lane));
        asm volatile("" : "+s"(T), "+s"(d), "+s"(I), "+s"(F));
        c.place(T, a.room);
        // ---- q, k, v ----
        if (qkv) {
            const int qq = NT > 1 ? c.wave >> 1 : c.wave, qu = NT > 1 ? c.wave & 1 : 0;  // this wave's tile and row tile
            const int nf = min(q0 + qq, q1 - 1) * 16 + c.g * 4;
            double2 turn[2] = {};  // cos and sin of this lane's two pairs
            if (a.rope && qq < QT) {
                const double2* tb = a.rope + ((size_t)(len + (NT > 1 ? c.row(qu) : c.t)) * DH + nf % DH) / 2;
                turn[0] = tb[0];
                turn[1] = tb[1];
            }
            const char* xs = pinned(z + a.at.x1);
            f32x4 acc[QT * NT];
            c.template nap<350>();
            sq.run(c, acc, xs, L->wqkv, q0, d >> 5, q1);
            leave_rows<QT, true>(c, acc);
            if (q0 + qq < q1) {
                const float f = row_factor(c, d, a.eps, qu);
                f32x4 s = total<QT * NT, PACK, false>(c, qq * NT + qu) * f;
                const int row = NT > 1 ? qu * 16 + c.tok : c.tok;
                const int seg = nf / I, nn = nf - seg * I, pos = len + row, hd = nn / DH, f0 = nn % DH;
                if (a.rope && seg < 2) {
#pragma unroll
                    for (int p = 0; p < 2; ++p) {
                        const float x0 = s[2 * p], x1 = s[2 * p + 1];
                        s[2 * p] = (float)((double)x0 * turn[p].x - (double)x1 * turn[p].y);
                        s[2 * p + 1] = (float)((double)x0 * turn[p].y + (double)x1 * turn[p].x);
                    }
                }
                char* out = z + (seg == 0 ? a.at.q : seg == 1 ? a.at.k : a.at.v);
                const Rsrc o = whole(out), n = whole(out + c.clear), kv = whole(seg == 1 ? L->kc : L->vc);
                if (seg == 0) {
                    const int off = ((hd * c.R + row) * DH + f0) * 4;
                    const v4u v = {__float_as_uint(s[0]), __float_as_uint(s[1]), __float_as_uint(s[2]), __float_as_uint(s[3])};
                    if (row < T) __builtin_amdgcn_raw_buffer_store_b128(v, o, off, 0, Way::kOut);
                    if (row < c.R) __builtin_amdgcn_raw_buffer_store_b128(v4u{kNotThere, kNotThere, kNotThere, kNotThere}, n, off, 0, Way::kOut);
                } else if (seg == 1) {
                    const int off = ((hd * c.R + row) * DH + f0) * 2;
                    const unsigned k01 = pack_bf16x2(s[0], s[1]), k23 = pack_bf16x2(s[2], s[3]);
                    if (row < T) {
                        st8<Way::kOut>(o, off, k01, k23);
                        st8<Way::kOut>(kv, (pos * I + nn) * 2, k01, k23);
                    }
                    if (row < c.R) st8<Way::kOut>(n, off, kNotThere, kNotThere);
                } else {
                    const int room = fresh_room(c.R), off = ((hd * DH + f0) * room + row) * 4;
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        const unsigned b = f2bf(s[v]);
                        if (row < room) __builtin_amdgcn_raw_buffer_store_b32(row < T ? b << 16 : 0u, o, off + v * room * 4, 0, Way::kOut);
                        if (row < T) __builtin_amdgcn_raw_buffer_store_b16((unsigned short)b, kv, ((nn + v) * a.vcap + pos) * 2, 0, Way::kOut);
                        if (row < room) __builtin_amdgcn_raw_buffer_store_b32(kNotThere, n, off + v * room * 4, 0, Way::kOut);
                    }
                }
            }
            lds_barrier();  // (stored: see the head of this file)
        }
        // ---- attention ----
        float4 gn = make_float4(0.f, 0.f, 0.f, 0.f);
        if (owner) {
            gn = gain(L->ln2);
            next_gain = gain(last ? L->ln2 : L[1].ln1);
        }
        if (!att) {
            so.forget();
            if (owner) so.open(c, L->wo, c.wg, I >> 5, d >> 4);
            if constexpr (EARLY) {
                c.template nap<1000>();  // (behind the keys and values)
                si.forget();
                if (ffn) si.open(c, L->win, i0, d >> 5, tf());
            }
        } else {
            const int nblk = (len + 31) >> 5;
            Range<Way> r = {whole(L->kc + (size_t)h * DH * 2), whole(L->vc + (size_t)h * DH * a.vcap * 2), I, a.vcap, nblk, {}, {}};
            const int first = split + S * c.wave;
            const bool newest = split == nblk % S && c.wave == nblk / S % kPassWaves, busy = first < nblk;
            if (busy && !newest) r.load(c, first);
            float m_run = -INFINITY, l_run = 0.f;
            f32x4 O[8];
#pragma unroll
            for (int dt = 0; dt < 8; ++dt) O[dt] = f32x4{0.f, 0.f, 0.f, 0.f};
            const bool low = c.tok >= 8;
            if (busy || newest) {
                const int room = fresh_room(c.R);
                const Rsrc fq = whole(z + a.at.q + h * c.R * DH * 4), fk = whole(z + a.at.k + h * c.R * DH * 2), fv = whole(z + a.at.v + h * room * DH * 4);
                float4 qv[4][2];
                uint4 kn[4 * NT];
                float4 vn[8 * NT];
                const int mine_row = NT > 1 ? c.row(rt) : c.row();
                auto fetch = [&](bool fresh) {  // the queries; the new rows' keys and values too
                    int tries = 0;
                    bool missing;
#pragma unroll 1
                    do {
                        asm volatile("" ::: "memory");
                        unsigned m = 0u;
                        auto see = [&](const uint4& v) { m = max(max(m, max(v.x, v.y)), max(v.z, v.w)); };
#pragma unroll
                        for (int i = 0; i < 8; ++i) qv[i >> 1][i & 1] = ldf4<Way::kIn>(fq, mine_row * DH * 4 + (i >> 1) * 128 + c.g * 32 + (i & 1) * 16);
                        if (fresh) {
#pragma unroll
                            for (int ks = 0; ks < 4 * NT; ++ks) kn[ks] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(fk, (NT > 1 ? c.row(ks >> 2) : c.t) * DH * 2 + (ks & 3) * 64 + c.g * 16, 0, Way::kIn));
#pragma unroll
                            for (int dt = 0; dt < 8 * NT; ++dt) vn[dt] = ldf4<Way::kIn>(fv, (((dt & 7) * 16 + c.tok) * room + (NT > 1 ? c.g * 4 + (dt >> 3) * 16 : min(c.g * 4, room - 4))) * 4);
#pragma unroll
                            for (int ks = 0; ks < 4 * NT; ++ks) see(kn[ks]);
#pragma unroll
                            for (int dt = 0; dt < 8 * NT; ++dt) see(__builtin_bit_cast(uint4, vn[dt]));
                        }
#pragma unroll
                        for (int i = 0; i < 8; ++i) see(__builtin_bit_cast(uint4, qv[i >> 1][i & 1]));
                        missing = __builtin_amdgcn_ballot_w64(m == kNotThere) != 0ull && !c.dead;
                    } while (missing && ++tries < c.spins);
                    if (missing) c.give_up();
                };
                auto parts = [&](const float (&v)[8], bf16x8 (&o)[P]) {  // packed: high parts in columns 0 .. 7, low parts in 8 .. 15
                    uint32_t hi[4], lo[4];
#pragma unroll
                    for (int j = 0; j < 4; ++j) split_bf16x2(v[2 * j], v[2 * j + 1], hi[j], lo[j]);
                    if constexpr (PACK) {
                        o[0] = as_bf(make_uint4(low ? lo[0] : hi[0], low ? lo[1] : hi[1], low ? lo[2] : hi[2], low ? lo[3] : hi[3]));
                    } else {
                        o[0] = as_bf(make_uint4(hi[0], hi[1], hi[2], hi[3]));
                        o[P - 1] = as_bf(make_uint4(lo[0], lo[1], lo[2], lo[3]));
                    }
                };
                bf16x8 Q[4][P];
                auto split_query = [&] {
                    const float sc = a.att_scale;
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) {
                        const float v[8] = {qv[ks][0].x * sc, qv[ks][0].y * sc, qv[ks][0].z * sc, qv[ks][0].w * sc,
                                            qv[ks][1].x * sc, qv[ks][1].y * sc, qv[ks][1].z * sc, qv[ks][1].w * sc};
                        parts(v, Q[ks]);
                    }
                };
                auto process = [&](int key, bool edge, int lim) {
                    f32x4 s[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
                        for (int p = 0; p < P; ++p)
#pragma unroll
                            for (int ab = 0; ab < 2; ++ab) s[ab] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf(r.K[ab][ks]), Q[ks][p], s[ab], 0, 0, 0);
                    float p[8], top = m_run;
#pragma unroll
                    for (int v = 0; v < 8; ++v) {
                        p[v] = s[v >> 2][v & 3];
                        if constexpr (PACK) p[v] += dpp_f<0x128, 0xF>(0.f, p[v]);
                        if (edge && key + (v >> 2) * 16 + c.g * 4 + (v & 3) > lim) p[v] = -INFINITY;
                        top = fmaxf(top, p[v]);
                    }
                    const float m_new = quad_rows_max(top), base = m_new == -INFINITY ? 0.f : m_new;
                    float sum = 0.f;
#pragma unroll
                    for (int v = 0; v < 8; ++v) {
                        p[v] = fexp(p[v] - base);
                        sum += p[v];
                    }
                    const float f = fexp(m_run - base);
                    l_run = l_run * f + quad_rows_sum(sum);
                    m_run = m_new;
                    bf16x8 w[P];
                    parts(p, w);
#pragma unroll
                    for (int dt = 0; dt < 8; ++dt) {
                        O[dt] *= f;
#pragma unroll
                        for (int u = 0; u < P; ++u) O[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf(r.V[dt]), w[u], O[dt], 0, 0, 0);
                    }
                };
                if (newest) {
                    fetch(true);
                    split_query();
#pragma unroll
                    for (int ks = 0; ks < 4; ++ks) {
                        r.K[0][ks] = kn[ks];
                        r.K[1][ks] = NT > 1 ? kn[4 * (NT - 1) + ks] : make_uint4(0u, 0u, 0u, 0u);
                    }
#pragma unroll
                    for (int dt = 0; dt < 8; ++dt) {  // (bf16 values in the upper halves)
                        const uint4 v = __builtin_bit_cast(uint4, vn[dt]);
                        const uint4 v2 = __builtin_bit_cast(uint4, vn[8 * (NT - 1) + dt]);
                        r.V[dt] = make_uint4(__builtin_amdgcn_perm(v.y, v.x, 0x07060302u), __builtin_amdgcn_perm(v.w, v.z, 0x07060302u), NT > 1 ? __builtin_amdgcn_perm(v2.y, v2.x, 0x07060302u) : 0u,
                                             NT > 1 ? __builtin_amdgcn_perm(v2.w, v2.z, 0x07060302u) : 0u);
                    }
                    process(len, true, len + mine_row);
                    if (busy) r.load(c, first);
                } else {
                    fetch(false);
                    split_query();
                }
#pragma unroll 1
                for (int blk = first; blk < nblk; blk += S * kPassWaves) {
                    process(blk * 32, blk * 32 + 31 >= len, len - 1);
                    if (blk + S * kPassWaves < nblk) r.load(c, blk + S * kPassWaves);
                }
            } else {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // (its filling of the last layer: other waves have waited for a read since)
            }
            // the waves' results: joined in LDS, a wave per sixteen features
            float* cm = (float*)(c.lds + kMl);
            float* cl = cm + kPassWaves * 16;
            lds_barrier();  // (both halves of the sums' memory are free)
            if (c.g == 0) {
                cm[c.wave * 16 + c.tok] = m_run;
                cl[c.wave * 16 + c.tok] = l_run;
            }
#pragma unroll
            for (int dt = 0; dt < 8; ++dt) *(f32x4*)(c.lds + kRed + ((c.wave * 8 + dt) * 64 + c.lane) * 16) = O[dt];
            lds_barrier();
            float w[kPassWaves], M = -INFINITY, Lsum = 0.f;
            f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int v = 0; v < kPassWaves; ++v) {
                w[v] = cm[v * 16 + c.tok];
                M = fmaxf(M, w[v]);
            }
            const float base = M == -INFINITY ? 0.f : M;
#pragma unroll
            for (int v = 0; v < kPassWaves; ++v) {
                const float f = fexp(w[v] - base);
                Lsum += cl[v * 16 + c.tok] * f;
                o += *(const f32x4*)(c.lds + kRed + ((v * 8 + c.wave) * 64 + c.lane) * 16) * f;
            }
            if constexpr (PACK) {
#pragma unroll
                for (int v = 0; v < 4; ++v) o[v] += dpp_f<0x128, 0xF>(0.f, o[v]);
            }
            lds_barrier();  // (read: the next stage's sums may come)
            char* out = pinned(z + a.at.a1);
            auto give = [&](int dt, const f32x4& v, float sum) {
                const float inv = 1.f / sum;
                const float t4[4] = {v[0] * inv, v[1] * inv, v[2] * inv, v[3] * inv};
                put_rows<PACK, false>(c, out, h * DH + dt * 16 + c.g * 4, t4, rt);
            };
            {
                // parts handed over between its workgroups, each of which joins 128 / S of the features
                char* pp = z + a.at.part + h * kWideSplits * c.R * DH * 4;
                char* pt = z + a.at.top + h * kWideSplits * c.R * 8;
                const Rsrc po = whole(pp), to = whole(pt), pn = whole(pp + c.clear), tn = whole(pt + c.clear);
                const int row = NT > 1 ? rt * 16 + c.tok : c.tok;
                if (S > 1 && row < T) {
                    const v4u v = {__float_as_uint(o[0]), __float_as_uint(o[1]), __float_as_uint(o[2]), __float_as_uint(o[3])};
                    __builtin_amdgcn_raw_buffer_store_b128(v, po, ((split * c.R + row) * DH + c.wave * 16 + c.g * 4) * 4, 0, Way::kOut);
                    if (c.wave == 0 && c.g == 0) st8<Way::kOut>(to, (split * c.R + row) * 8, __float_as_uint(M), __float_as_uint(Lsum));
                }
                for (int s = split; s < kWideSplits; s += S)  // (also the places of ranges that there are not in this pass)
                    if (row < c.R) {
                        __builtin_amdgcn_raw_buffer_store_b128(v4u{kNotThere, kNotThere, kNotThere, kNotThere}, pn, ((s * c.R + row) * DH + c.wave * 16 + c.g * 4) * 4, 0, Way::kOut);
                        if (c.wave == 0 && c.g == 0) st8<Way::kOut>(tn, (s * c.R + row) * 8, kNotThere, kNotThere);
                    }
                const int per = 8 / S, dt = split * per + c.wave;
                if (S == 1) {
                    give(c.wave, o, Lsum);
                } else if (c.wave < per) {
                    float4 v[kWideSplits];
                    v2u ml[kWideSplits];
                    int tries = 0;
                    bool missing;
#pragma unroll 1
                    do {
                        asm volatile("" ::: "memory");
                        unsigned m = 0u;
#pragma unroll
                        for (int s = 0; s < kWideSplits; ++s) {
                            const int e = min(s, S - 1) * c.R + (NT > 1 ? c.row(rt) : c.row());
                            v[s] = ldf4<Way::kIn>(po, (e * DH + dt * 16 + c.g * 4) * 4);
                            ml[s] = __builtin_bit_cast(v2u, __builtin_amdgcn_raw_buffer_load_b64(to, e * 8, 0, Way::kIn));
                        }
#pragma unroll
                        for (int s = 0; s < kWideSplits; ++s) {
                            const uint4 b = __builtin_bit_cast(uint4, v[s]);
                            m = max(max(m, max(max(b.x, b.y), max(b.z, b.w))), max(ml[s].x, ml[s].y));
                        }
                        missing = __builtin_amdgcn_ballot_w64(m == kNotThere) != 0ull && !c.dead;
                    } while (missing && ++tries < c.spins);
                    if (missing) c.give_up();
                    float all = -INFINITY, sum = 0.f;
                    f32x4 j = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int s = 0; s < kWideSplits; ++s) all = fmaxf(all, __uint_as_float(ml[s].x));
#pragma unroll
                    for (int s = 0; s < kWideSplits; ++s) {
                        const float f = s < S ? fexp_full(__uint_as_float(ml[s].x) - all) : 0.f;
                        sum += __uint_as_float(ml[s].y) * f;
                        j += f32x4{v[s].x, v[s].y, v[s].z, v[s].w} * f;
                    }
                    give(dt, j, sum);
                }
            }
            lds_barrier();
            so.forget();
            if (owner) so.open(c, L->wo, c.wg, I >> 5, d >> 4);
            if constexpr (EARLY) {
                si.forget();
                if (ffn) si.open(c, L->win, i0, d >> 5, tf());
            }
        }
        // ---- output projection ----
        if (owner) {
            const char* xs = pinned(z + a.at.a1);
            f32x4 acc[NT];
            so.run(c, acc, xs, L->wo, c.wg, I >> 5, d >> 4);
            leave_rows<1, false>(c, acc);
            if (mine) add();
            publish(gn, z + a.at.x2);
            lds_barrier();
        }
        if constexpr (!EARLY) {
            si.forget();
            if (ffn) si.open(c, L->win, i0, d >> 5, tf());
        }
        // ---- FFN ----
        if (ffn) {
            constexpr int FW = GATED ? FT / 2 : FT;  // waves with results
            const char* xs = pinned(z + a.at.x2);
            f32x4 acc[FT * NT];
            c.template nap<350>();
            si.run(c, acc, xs, L->win, i0, d >> 5, tf());
            leave_rows<FT, true>(c, acc);
            auto hidden = [&](int unit, int u) {
                const int tile = uf * FW + unit;  // of the hidden state
                if (unit >= FW || tile >= F >> 4) return;
                const float rms = row_factor(c, d, a.eps, u);
                float w[4];
                if constexpr (GATED) {
                    const f32x4 s = total<FT * NT, PACK, false>(c, 2 * unit * NT + u) * rms, up = total<FT * NT, PACK, false>(c, (2 * unit + 1) * NT + u) * rms;
#pragma unroll
                    for (int v = 0; v < 4; ++v) w[v] = (a.act == BILD_ACT_GATED_GELU ? gelu_tanh_f(s[v]) : silu_f(s[v])) * up[v];
                } else {
                    const f32x4 s = total<FT * NT, PACK, false>(c, unit * NT + u) * rms;
#pragma unroll
                    for (int v = 0; v < 4; ++v) w[v] = fmaxf(s[v], 0.f);
                }
                put_rows<PACK, false>(c, z + a.at.h, tile * 16 + c.g * 4, w, u);
            };
            if constexpr (NT == 1) {
                hidden(c.wave, 0);
            } else {
                for (int k = c.wave; k < FW * NT; k += kPassWaves) hidden(k >> 1, k & 1);
            }
            lds_barrier();
        }
        sf.forget();
        if (owner) sf.open(c, L->wout, c.wg, F >> 5, d >> 4);
        const char* hidden = z + a.at.h;
        z = c.next(z, a.at.layer);
        c.walk_on(a.at.layer);
        if (owner) {
            const char* xs = pinned(hidden);
            f32x4 acc[NT];
            c.template nap<650>();
            sf.run(c, acc, xs, L->wout, c.wg, F >> 5, d >> 4);
            leave_rows<1, false>(c, acc);
            if (mine) add();
            if (!last) publish(next_gain, z + a.at.x1);
            lds_barrier();
        }
        sq.forget();
        if (qkv && !last) sq.open(c, L[1].wqkv, q0, d >> 5, q1);
    }
    const int row = NT > 1 ? c.wave * 16 + c.tok : c.tok;
    if (mine && row < T) {
        *(float4*)(a.x_out + (size_t)row * d + n0()) = x;
        if (a.x_keep) *(float4*)(a.x_keep + (size_t)(len + row) * d + n0()) = x;
    }
}

// Sizes the kernel is made for: runs of inputs that fit the registers, all of it on the chip at once.
template <class Cut>
static bool wide_fits(int d, int heads, int F, bool gated, int cus) {
    const int I = heads * kWideHead, in = (std::max(d, I) / 32 + kPassWaves - 1) / kPassWaves, tf = gated ? F / 8 : F / 16;
    return in <= Cut::KD && (F / 32 + kPassWaves - 1) / kPassWaves <= Cut::KF && (3 * I / 16 + Cut::QT - 1) / Cut::QT <= cus && (tf + Cut::FT - 1) / Cut::FT <= cus &&
           d / 16 <= cus && heads <= cus;
}

// Most rows there is a kernel for: above eight, which take twice the registers for activations, models of the widest cut alone (its FFN's first
// weights do not wait in registers while others are multiplied); above sixteen, two row tiles and twice the workgroups of heads, 4096-wide ones.
int wide_most(int d, int heads, int F, bool gated, int cus) {
    return wide_fits<Cut2048>(d, heads, F, gated, cus) ? kWideRows : d < kWideRowsFrom || 2 * heads > cus ? 16 : kWideRowsMost;
}

// Passes of nine rows and more: where they are taken.  What they do better than kernels of their own is to read weights on while activations are handed
// over; what they do worse, twice the activations' loads and products, goes with the width and is the same however wide the hidden state is.  So the line
// is one of the hidden state (1.2 times for a gated one) and the heads' width against the model's.  Its time over the kernels' own, 900 shapes drawn at random, layers of 0.7 GB together, three
// lengths from 64 to 7900 tokens, 9, 12 and 16 rows, by F + I / 2 - 2 d / 5 (1.2 F gated) of those 2304 to 4096 wide, the least, middle and most of the shapes' means: below 2560 1.02, 1.09, 1.23, to 3560 0.99, 1.06,
// 1.14, to 4560 0.95, 1.01, 1.08, to 5560 0.92, 0.97, 1.02, to 8560 0.89, 0.94, 1.00, above 0.85, 0.90, 0.95.  Of 2340 times on this side three are over 1.04 (1.05), of 3700 on the other 49 under 0.96 (0.93).
// 4096 wide, 32 heads, hidden states up to 3400, 4096, 5200, 6400, 8192, 11 264: without a gate 1.06, 1.05, 0.97, 0.96, 0.94, 0.90, gated 1.01, 0.99, 0.93, 0.93, 0.92, 0.86.  2048 wide (hidden states above 6144)
// gated up to 8192 0.90 to 0.94, wider 1.01 to 1.07, without a gate 0.98 to 1.06.  Narrower ones, whose separate kernels are others (takes_thin), 0.77 to 0.99.
static bool wide_many(int d, int heads, int F, bool gated) {
    if (d < 2048) return true;
    if (d == 2048) return gated && F <= 8192;
    return (gated ? 12 * F / 10 : F) + heads * kWideHead / 2 - 2 * d / 5 >= 4560;
}

// Most rows it is taken for at some length.
int wide_rows(int d, int heads, int F, bool gated, int cus) {
    const int most = wide_most(d, heads, F, gated, cus);
    if (most <= kWideRows || !wide_many(d, heads, F, gated)) return std::min(most, kWideRows);
    return std::min(most, F > 8192 ? kWideRowsMost : F > 4096 ? 24 : 16);
}

// Most keys of a pass of T rows.  Each of two row tiles goes over a head's keys by itself, and up to 4096 features of the hidden state the kernels of their own are
// better, up to 8192 behind many keys.  4096 wide, 17 and 24 rows over 200, 1000, 2000, 3000, 4000, 5500 tokens, its time over the others', mean of 10 to 40 shapes, without a gate 4320 to 8192
// 0.94, 0.94, 0.99, 1.00, 1.02, 1.06, above 0.86, 0.86, 0.90, 0.91, 0.94, 0.97, gated 0.96, 0.97, 1.01, 1.03, 1.04, 1.08 and 0.90, 0.90, 0.93, 0.94, 0.96, 1.00; 25 and 32 rows without a gate
// 0.99, 1.02, 1.04, 1.06, 1.08, 1.12 and 0.91, 0.93, 0.95, 0.97, 0.99, 1.03, gated 1.01, 1.03, 1.05, 1.07, 1.09, 1.14 and 0.94, 0.95, 0.97, 0.99, 1.01, 1.05.  The 7B shape, 17, 24, 25, 32 rows, us, kernels of
// their own / this, over 64 tokens 3599, 3609, 3628, 3622 / 3270, 3265, 3492, 3496, 2016 3771, 3790, 3811, 3820 / 3429, 3434, 3666, 3674, 3200 3925, 3942 / 3684, 3687, 4072 3967, 3988 / 3856, 3857; 32 rows
// over 3200 and 4097 4118, 4178 / 4087, 4268.
// Below 2048 wide, 9, 12, 16 rows: up to 6500 keys 0.92, 0.87, 0.84, nine rows without a gate below 7680 1.00 (0.92 to 1.12, wider 0.88); 8000 keys 1.07, 0.99, 0.95 below 8192, above 0.99, 0.93, 0.88.
int wide_keys(int T, int d, int F, bool gated) {
    if (T <= kWideRows) return 8192;
    if (T <= 16) return d >= 2048 ? 8192 : T == 9 && !gated && F < 7680 ? 0 : T > 9 && F >= 8192 ? 8192 : 6656;
    return T > 24 ? 2048 : F > 8192 ? 4096 : gated ? 1280 : 2048;
}

int wide_groups(int d, int heads, int d_head, int F, bool gated, int cus) {
    if (d_head != kWideHead || d <= 1024 || d % 256 != 0 || F % 32 != 0) return 0;
    return wide_fits<Cut2048>(d, heads, F, gated, cus) || wide_fits<Cut4096>(d, heads, F, gated, cus) ? cus : 0;
}

// Two tiles of q, k, v a workgroup instead of three, where that many workgroups there are: models up to 2048 wide whose heads and
// projections are not apart, up to 2304 keys or as long as workgroups with heads have no part of q, k, v.  2048-wide, 16 layers, one row, us, two tiles / three /
// apart: 200 keys 451, 471, 412; 700 468, 471, 420; 1000 471, 472, 438; 1100 457, 485, 442; 1250 461, 487, 454; 1350 464, 489, 464; 2000 483, 492,
// 529; 4000 593, 548, 672.  A kernel of its own, chosen by the host: in the one with registers for three, two tiles cost eight rows at 1400 and
// 2000 keys 511, 525 (506, 520 here), with a body for either in one kernel the other lengths lose 1.2 %.  1280-wide, one row, at 1400, 2000, 2400 keys with
// registers for three (three tiles above 2304) 313, 317, 341, here 305, 309, 327.
bool wide_two(int d, int heads, int F, bool gated, int cus, int keys) {
    const int tq = 3 * heads * kWideHead / 16, two = ceil_div(tq, Cut2048Two::QT);
    return wide_fits<Cut2048Two>(d, heads, F, gated, cus) && keys > kWideApart && (keys <= 2304 || two <= cus - heads * wide_splits(keys, heads, cus));
}

bool wide_split(int d, int heads, int F, bool gated, int cus, int keys, int rows, int out[7]) {
    if (!wide_groups(d, heads, kWideHead, F, gated, cus) || rows > wide_rows(d, heads, F, gated, cus) || keys > wide_keys(rows, d, F, gated)) return false;
    const int tq = 3 * heads * kWideHead / 16, tf = gated ? F / 8 : F / 16;
    auto is = [&](auto cut) {
        using Cut = decltype(cut);
        const WideParts p = wide_parts<Cut>(keys, d, heads * (rows > 16 ? 2 : 1), tq, tf, cus);
        out[0] = Cut::QT; out[1] = p.q; out[2] = Cut::FT; out[3] = p.i; out[4] = p.head0; out[5] = p.ranges; out[6] = p.apart;
    };
    if (wide_two(d, heads, F, gated, cus, keys)) is(Cut2048Two());
    else if (wide_fits<Cut2048>(d, heads, F, gated, cus)) is(Cut2048());
    else if (rows > 16) is(Cut4096Rows());
    else is(Cut4096());
    return true;
}

hipError_t wide_init() {
    static hipError_t done = [] {
#define BILD_W(CV, RV) (const void*)wide_kernel<false, CV, RV>, (const void*)wide_kernel<true, CV, RV>
        const void* fns[] = {BILD_W(Cut2048, 0), BILD_W(Cut2048, 1), BILD_W(Cut2048, 2), BILD_W(Cut2048Two, 0), BILD_W(Cut2048Two, 1), BILD_W(Cut2048Two, 2),
                             BILD_W(Cut4096, 0), BILD_W(Cut4096, 1), BILD_W(Cut4096, 2), BILD_W(Cut4096, 16), BILD_W(Cut4096Rows, 32)};
#undef BILD_W
        return raise_lds_limit(fns, 160 * 1024);
    }();
    return done;
}

hipError_t launch_wide(const PassArgs& a, hipStream_t st) {
    if (hipError_t e = wide_init(); e != hipSuccess) return e;
    const bool gated = a.act != BILD_ACT_RELU;
    if (a.groups < 1 || a.groups != wide_groups(a.d, a.heads, a.I / std::max(a.heads, 1), a.F, gated, a.groups) || a.T < 1 || a.T > wide_most(a.d, a.heads, a.F, gated, a.groups) || a.room < a.T || a.cross || a.rel_bias ||
        !a.turn || !a.layers || !a.sync || !a.scratch || !a.x_out || !a.len_ptr)
        return hipErrorInvalidValue;
    const dim3 grid(a.groups), block(kPassThreads);
    const bool small = wide_fits<Cut2048>(a.d, a.heads, a.F, gated, a.groups);
    if (a.two && !wide_fits<Cut2048Two>(a.d, a.heads, a.F, gated, a.groups)) return hipErrorInvalidValue;
#define BILD_WC(CV, RV)                                                                                                \
    do {                                                                                                               \
        if (gated) hipLaunchKernelGGL((wide_kernel<true, CV, RV>), grid, block, kRel, st, a);                          \
        else hipLaunchKernelGGL((wide_kernel<false, CV, RV>), grid, block, kRel, st, a);                               \
    } while (0)
#define BILD_W(RV)                                                                                                     \
    do {                                                                                                               \
        if (a.two) BILD_WC(Cut2048Two, RV);                                                                            \
        else if (small) BILD_WC(Cut2048, RV);                                                                          \
        else BILD_WC(Cut4096, RV);                                                                                     \
    } while (0)
    if (a.room > 16) BILD_WC(Cut4096Rows, 32);
    else if (a.room > 8) BILD_WC(Cut4096, 16);
    else if (a.room == 1) BILD_W(1);
    else if (a.room == 2) BILD_W(2);
    else BILD_W(0);
#undef BILD_W
#undef BILD_WC
    return hipGetLastError();
}

}  // namespace bild
