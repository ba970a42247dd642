// What the kernels that walk all layers of a decoder pass share (pass_kernel.hip, whose head explains it, and pass_wide.hip): where a
// workgroup is in the pass and in the hand-over memory, activations as they are handed over, sums over the waves.
#pragma once
#include "kernel_common.h"

namespace bild {

constexpr int kPassWaves = 8, kPassThreads = 64 * kPassWaves;

typedef __attribute__((address_space(4))) const PassLayer CLayer;  // (read through the scalar cache)
typedef __amdgpu_buffer_rsrc_t Rsrc;
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));
// (an address worked out here, not behind the wait that follows)
template <class P>
__device__ __forceinline__ P* pinned(P* p) {
    asm volatile("" : "+s"(p));
    return p;
}
__device__ __forceinline__ Rsrc whole(const void* p) { return make_rsrc(p, 0xFFFFFFFFu); }
template <int AUX = 0>
__device__ __forceinline__ float4 ldf4(Rsrc r, int off) { return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, AUX)); }
__device__ __forceinline__ bf16x8 as_bf(const uint4& v) { return __builtin_bit_cast(bf16x8, v); }
template <int AUX>
__device__ __forceinline__ void st8(Rsrc r, int off, unsigned a, unsigned b) {
    const v2u v = {a, b};
    __builtin_amdgcn_raw_buffer_store_b64(v, r, off, 0, AUX);
}

constexpr unsigned kNotThere = 0xFFFFFFFFu;  // (two NaNs of a kind no conversion gives, as bf16 parts; one as a sum)

// LDS: sums of the waves (up to six tiles each; attention joins its waves there too), their (max, sum) of either attention, the head's query, the
// waves' sums of squares (twice, like the sums), their weights of one row's keys, the head's relative-position biases
constexpr int kRedBytes = kPassWaves * 6 * 1024;  // twice: a stage's sums are read while the next one's are written
constexpr int kRed = 0, kMl = 2 * kRedBytes, kMlBytes = 2 * kPassWaves * 16 * 4, kQ = kMl + 2 * kMlBytes, kQLd = 68, kSq = kQ + 16 * kQLd * 4, kSqBytes = kPassWaves * 16 * 4, kP = kSq + 2 * kSqBytes, kRel = kP + kPassWaves * 256;

// Rows there is room for in the hand-over memory (the layout's): known to the kernel, or (0) not.
template <int ROOM>
struct Room {
    static constexpr int R = ROOM;
    __device__ __forceinline__ void room(int) {}
};
template <>
struct Room<0> {
    int R;
    __device__ __forceinline__ void room(int r) { R = r; }
};
template <bool DIE, bool FP32, int ROOM>
struct Walk : Room<ROOM> {
    using Room<ROOM>::R;
    static constexpr int KNOWN = ROOM;
    static constexpr bool HEAD = false;    // LM head and policy inside (pass_head.h)
    static constexpr bool F32 = FP32;      // of an fp32 model
    static constexpr bool ONE = FP32 && ROOM == 1;  // ... and one row (see multiply)
    static constexpr bool ROOM1 = !FP32 && ROOM == 1;  // a producer's sum of squares behind its sixteen features, in one line
    // Input tiles beside each other in a load of a projection with N of them per wave (see multiply).  One row fills an eighth of
    // a load, so always.  Two rows where there are more than four tiles: for fewer the sums by row cost more than the loads (T5-large
    // shape 434 us with and 428 without).  Four rows nowhere: the FFN's output alone 455 -> 452 there, but 514 -> 523 at the mT5-large shape.
    template <int N>
    static constexpr int side() { return FP32 ? (ROOM == 1 ? 16 : 1) : ROOM == 1 ? 8 : ROOM == 2 && N > 4 ? 4 : 1; }
    static constexpr int KS = F32 ? 4 : 5;  // inputs of a weight tile, logarithm
    static constexpr int ESZ = F32 ? 4 : 2;
    static constexpr int BK = F32 ? 16 : 32;  // keys a wave takes at a time
    static constexpr int kIn = 16;  // reads of what may not be there yet: past the L1 (sc1)
    // what is handed over goes as far as all readers see it: to the die's L2 (the L1s write through), or past the L2s (sc0 sc1)
    static constexpr int kOut = DIE ? 0 : 17;
    char* lds;
    unsigned* failed;
    int spins;
    int wg, wave, lane, tok, g, t, t8;  // t: this lane's row, clamped to the last one; t8: of the packed order
    bool dead;
    int red = 0, sq = 0;            // halves of the sums' memory in use
    float ss;                       // this wave's part of its lane's row's sum of squares
    int slot, clear;                // clear: from what this layer hands over to where the layer after the next will: filled with "not there yet"

    int T;                          // rows
    __device__ __forceinline__ void place(int rows, int room) {
        T = rows;
        this->room(room);
        tok = lane & 15;
        g = lane >> 4;
        t = min(tok, T - 1);
        t8 = min(tok & 7, T - 1);
    }
    // This layer's hand-over memory, of three that take turns (see the head of this file); next(): of the layer after it.
    __device__ __forceinline__ char* scratch(const PassArgs& a) {
        slot = (int)(*a.turn * (unsigned)a.n_layers % 3u);
        clear = slot == 0 ? 2 * a.at.layer : -a.at.layer;
        return a.scratch + slot * a.at.layer;
    }
    __device__ __forceinline__ char* next(char* z, int layer) const { return z + (slot == 2 ? -2 * layer : layer); }
    __device__ __forceinline__ void walk_on(int layer) {
        slot = slot == 2 ? 0 : slot + 1;
        clear = slot == 0 ? 2 * layer : -layer;
    }
    __device__ __forceinline__ void give_up() {
        dead = true;
        if (lane == 0) asm volatile("global_store_dword %0, %1, off sc0 sc1" ::"v"(failed), "v"(1u) : "memory");
    }
    __device__ __forceinline__ void rest(int turns) const {
#pragma unroll 1
        for (int i = 0; i < turns; ++i) __builtin_amdgcn_s_sleep(3);
    }
    // (about NS nanoseconds; see the head of this file)
    template <int NS>
    __device__ __forceinline__ void nap() const {
        if constexpr (!DIE) __builtin_amdgcn_s_sleep(NS / 27);
    }
};

// fp32: sixteen inputs, component v of a lane group g is input 4 g + v (two sums, so that products do not wait for each other)
__device__ __forceinline__ void products(f32x4& a, f32x4& b, const uint4& w, const uint4& x) {
    a = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w.x), __uint_as_float(x.x), a, 0, 0, 0);
    b = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w.y), __uint_as_float(x.y), b, 0, 0, 0);
    a = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w.z), __uint_as_float(x.z), a, 0, 0, 0);
    b = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(w.w), __uint_as_float(x.w), b, 0, 0, 0);
}

// This wave's run of input tiles of a projection over tk tiles.
struct Run {
    int k0, n;
};
__device__ __forceinline__ Run run_of(int wave, int tk) {
    const int per = (tk + kPassWaves - 1) / kPassWaves;
    return {wave * per, max(0, min(per, tk - wave * per))};
}

// (tiles past the last of the `tiles` there are: the last one again; the wave's input tiles J0 .. J1 - 1)
template <int N, int RW, int J0 = 0, int J1 = N, class Walk>
__device__ __forceinline__ void request(const Walk& c, uint4 (&W)[N * RW], const void* w, int unit, int tk, int tiles) {
    const Run r = run_of(c.wave, tk);
    const Rsrc rs = whole((const char*)w + (size_t)unit * RW * tk * kTileBytes);
    const int most = tiles - 1 - unit * RW;
#pragma unroll
    for (int j = J0; j < J1; ++j)
        if (j < r.n) {
#pragma unroll
            for (int q = 0; q < RW; ++q) W[j * RW + q] = buf_load(rs, (unsigned)c.lane * 16u, ((RW == 1 ? 0 : min(q, most)) * tk + r.k0 + j) * kTileBytes);
        }
}

// A tile of planes that a norm's projection reads has its producers' sums of squares behind it, [row][first, second sixteen
// inputs] (an own line: a producer's part of a row lies where its planes' readers look anyway).
// (fp32 models: tiles of sixteen inputs, a producer each, [four inputs][row] and one sum per row)
__host__ __device__ __forceinline__ int tile_bytes(bool normed, int room, bool f32) { return f32 ? room * 64 + (normed ? 64 : 0) : room * 128 + (normed ? 128 : 0); }
// What lane j of this lane's sixteen has; j is a constant once unrolled.
template <int J>
__device__ __forceinline__ uint4 from_lane(const uint4& v, int j) {
    if constexpr (J < 16) {
        if (j != J) return from_lane<J + 1>(v, j);
        return make_uint4(__builtin_amdgcn_update_dpp(0, v.x, 0x150 + J, 0xF, 0xF, true), __builtin_amdgcn_update_dpp(0, v.y, 0x150 + J, 0xF, 0xF, true),
                          __builtin_amdgcn_update_dpp(0, v.z, 0x150 + J, 0xF, 0xF, true), __builtin_amdgcn_update_dpp(0, v.w, 0x150 + J, 0xF, 0xF, true));
    }
    return v;
}
// 1/rms of this lane's row, behind leave()
template <class Walk>
__device__ __forceinline__ float norm_factor(const Walk& c, int d, float eps) {
    float p[kPassWaves], s = 0.f;
    if constexpr (Walk::ROOM1) {
        const float4 v = *(const float4*)(c.lds + kSq + c.sq + c.tok * 16);
        s = (v.x + v.y) + (v.z + v.w);
        s += dpp_f<0x128, 0xF>(0.f, s);
        s += dpp_f<0x124, 0xF>(0.f, s);
        s += dpp_f<0x122, 0xF>(0.f, s);
        s += dpp_f<0x121, 0xF>(0.f, s);
        return __builtin_amdgcn_rsqf(s * __builtin_amdgcn_rcpf((float)d) + eps);
    }
#pragma unroll
    for (int v = 0; v < kPassWaves; ++v) p[v] = *(const float*)(c.lds + kSq + c.sq + (v * 16 + c.tok) * 4);
#pragma unroll
    for (int v = 0; v < kPassWaves; ++v) s += p[v];
    return __builtin_amdgcn_rsqf(s * __builtin_amdgcn_rcpf((float)d) + eps);
}

// acc = W x over this wave's inputs.  x lies in tiles of 32 inputs in the order in which the operand's lanes want it: quarters of
// eight inputs, in each the rows one after the other, 16 bytes per row; the high parts of a tile and then its low parts.  (A load
// is then one dense piece: with the rows' 64 bytes 128 apart a pass of eight rows took 854 us instead of 737.)
// Up to eight rows (PACK) one operand holds the high parts of the rows in its columns 0 .. 7 and the low parts in 8 .. 15: half
// the loads and products (a compute unit's 64 bytes a cycle are what the FFN output's 256 loads of 1 KiB wait for); the halves
// are added in total().  A quarter then has the rows' high parts and their low parts.
// NORM: the rows' sums of squares as well, to c.ss.
//
// A load takes the compute unit's first cache sixteen cycles however few of its bytes differ, so with one or two rows it brings
// 8 / rows tiles: lane (tile, row; quarter) a piece of its own.  The operands change places (activations first), so that a product's
// rows are the tiles' in their places, of which one is of use: it lies in one register of one pair of lane groups, and what the
// tiles contribute is picked by a register's number and one select instead of masks on the operands (four instructions a tile).
// The sums are then by row: acc[.][t], feature = lane & 15, a part in each lane group (leave() adds those).  One row with the sums
// of squares behind its producers' features gets them by the same load, in columns 4 .. 7.  All-to-all hand-overs of 64 lines in a
// kernel of their own: 1.51 us a stage with eight loads a wave, 0.89 with one; 128 lines 2.24 and 0.93.
//
// One row of an fp32 model (Walk::ONE) has no use for the matrix cores, whose fp32 products of sixteen rows take eight times as long
// as a lane's own four inputs: lane (feature, four inputs) sums those, leave() adds the four lanes of a feature.
template <int N, int RW, bool PACK, bool NORM, class Walk>
__device__ __forceinline__ void multiply(Walk& c, f32x4 (&acc)[RW], const uint4 (&W)[N * RW], const void* planes, int tk) {
    const Run r = run_of(c.wave, tk);
    const Rsrc xs = whole(planes);
    const int S = tile_bytes(NORM, c.R, Walk::F32);
    constexpr int SIDE = Walk::template side<N>();
    constexpr int P = PACK || Walk::F32 ? 1 : 2, NL = (N + SIDE - 1) / SIDE, B = NL * P <= 16 ? NL : 4;  // loads of a piece
    constexpr int IN = Walk::kIn;
    static_assert(NL % B == 0 && (!NORM || N <= 4) && (SIDE == 1 || B == NL), "whole pieces; a lane group per tile");
    const int beside = SIDE == 1 ? 0 : Walk::F32 ? c.tok : (c.tok & (NORM && Walk::ROOM1 ? 3 : 7)) / c.R;  // this lane's tile of a load
    const int row = SIDE == 1 ? (PACK ? c.t8 : c.t) : Walk::F32 ? 0 : min((c.tok & 7) & (c.R - 1), c.T - 1);
    constexpr bool SUMS = NORM && Walk::ROOM1;  // lanes of columns 4 .. 7 get the sums of squares: four tiles' two each
    static_assert(!SUMS || N <= 4, "room for the sums beside the tiles");
    const int at = !SUMS ? (PACK ? (c.g * 2 + (c.tok >> 3)) * c.R + row : c.g * c.R + row) * 16
                         : (c.tok & 4) ? (c.g & 1) * 128 + 64 : (c.g >> 1) * 128 + (c.g & 1) * 32 + (c.tok >> 3) * 16;
    const int k0 = r.k0 * S;
    uint4 X[NL > B ? 2 : 1][P * B];
    v2u sq = {0u, 0u};
    f32x4 low[RW];
#pragma unroll
    for (int q = 0; q < RW; ++q) acc[q] = low[q] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto get = [&](uint4 (&x)[P * B], v2u& sq, int j0) {
#pragma unroll
        for (int j = 0; j < B; ++j)
            if ((j0 + j) * SIDE < r.n) {
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    // (tiles past the wave's last one: that one again)
                    const int off = SIDE == 1 ? at + p * c.R * 64 : at + min((j0 + j) * SIDE + beside, r.n - 1) * S, from = SIDE == 1 ? k0 + (j0 + j) * S : k0;
                    x[P * j + p] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(xs, off, from, IN));
                }
            }
        if constexpr (NORM && !SUMS) {  // (lane group g: tile g)
            const int tile = min(c.g, max(r.n - 1, 0)) * S, from = r.n > 0 ? k0 : 0;
            if constexpr (Walk::F32) {
                const unsigned v = __builtin_amdgcn_raw_buffer_load_b32(xs, tile + c.R * 64 + c.t * 4, from, IN);
                sq = v2u{c.g < r.n ? v : 0u, 0u};
            } else {
                const v2u v = __builtin_bit_cast(v2u, __builtin_amdgcn_raw_buffer_load_b64(xs, tile + c.R * 128 + c.t * 8, from, IN));
                sq = c.g < r.n ? v : v2u{0u, 0u};
            }
        }
    };
    auto lacks = [&](const uint4 (&x)[P * B], const v2u& sums, int j0) {
        unsigned m = max(sums.x, sums.y);
#pragma unroll
        for (int j = 0; j < B; ++j)
            if ((j0 + j) * SIDE < r.n) {
#pragma unroll
                for (int p = 0; p < P; ++p) m = max(max(m, max(x[P * j + p].x, x[P * j + p].y)), max(x[P * j + p].z, x[P * j + p].w));
            }
        return __builtin_amdgcn_ballot_w64(m == kNotThere) != 0ull && !c.dead;
    };
    // all of it again and again until every word is there
    auto wait = [&](uint4 (&x)[P * B], int j0) {
        int n = 0;
        bool missing;
#pragma unroll 1
        do {
            asm volatile("" ::: "memory");
            if (NL == B || n > 0) get(x, sq, j0);
            missing = lacks(x, sq, j0);
        } while (missing && ++n < c.spins);
        if (missing) c.give_up();
    };
    auto mul = [&](const uint4 (&x)[P * B], int j0) {
        if constexpr (SIDE > 1 && !Walk::F32) {
            constexpr int ND = N < SIDE ? N : SIDE;
            f32x4 D[RW][ND];  // of the tiles in one place: rows of the others' places are of no use
#pragma unroll
            for (int q = 0; q < RW; ++q)
#pragma unroll
                for (int j = 0; j < ND; ++j) D[q][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < N; ++j)
                if (j < r.n) {
#pragma unroll
                    for (int q = 0; q < RW; ++q) D[q][j % SIDE] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf(x[j / SIDE]), as_bf(W[j * RW + q]), D[q][j % SIDE], 0, 0, 0);
                }
#pragma unroll
            for (int q = 0; q < RW; ++q)
#pragma unroll
                for (int t = 0; t < Walk::R; ++t) {
                    float even = 0.f, odd = 0.f;
#pragma unroll
                    for (int j = 0; j < ND; ++j) {
                        const int m = j * Walk::R + t;
                        (m < 4 ? even : odd) += D[q][j][m & 3];
                    }
                    acc[q][t] = c.g & 1 ? odd : even;
                }
            return;
        }
#pragma unroll
        for (int j = 0; j < (SIDE == 1 ? B : N); ++j)
            if (j0 + j < r.n) {
                uint4 v = x[SIDE == 1 ? P * j : j / SIDE];
                if constexpr (Walk::ONE) v = from_lane<0>(v, j % SIDE);
#pragma unroll
                for (int q = 0; q < RW; ++q) {
                    const uint4 w = W[(j0 + j) * RW + q];
                    if constexpr (Walk::ONE) {
                        acc[q][0] = __builtin_fmaf(__uint_as_float(w.x), __uint_as_float(v.x), acc[q][0]);
                        acc[q][1] = __builtin_fmaf(__uint_as_float(w.y), __uint_as_float(v.y), acc[q][1]);
                        acc[q][2] = __builtin_fmaf(__uint_as_float(w.z), __uint_as_float(v.z), acc[q][2]);
                        acc[q][3] = __builtin_fmaf(__uint_as_float(w.w), __uint_as_float(v.w), acc[q][3]);
                    } else if constexpr (Walk::F32) {
                        products(acc[q], RW == 1 ? low[q] : acc[q], w, v);
                    } else {
                        f32x4& even = RW == 1 && PACK && (j & 1) ? low[q] : acc[q];
                        even = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf(w), as_bf(v), even, 0, 0, 0);
                        f32x4& lo_acc = RW == 1 ? low[q] : acc[q];
                        if (!PACK) lo_acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf(w), as_bf(x[P * j + P - 1]), lo_acc, 0, 0, 0);
                    }
                }
            }
    };
    if constexpr (NL == B) {
        wait(X[0], 0);
        mul(X[0], 0);
    } else {  // two pieces on their way
        get(X[0], sq, 0);
        get(X[1], sq, B);
#pragma unroll
        for (int j0 = 0; j0 < N; j0 += B) {
            if (j0 >= r.n) break;
            wait(X[(j0 / B) & 1], j0);
            mul(X[(j0 / B) & 1], j0);
            if (j0 + 2 * B < N) get(X[(j0 / B) & 1], sq, j0 + 2 * B);
        }
    }
    if constexpr (RW == 1 && SIDE == 1) acc[0] += low[0];
    if constexpr (SUMS) c.ss = (c.tok & 3) < r.n ? __uint_as_float(X[0][0].x) : 0.f;
    else if constexpr (NORM) c.ss = quad_rows_sum(__uint_as_float(sq.x) + __uint_as_float(sq.y));
}

// The waves' results side by side in LDS; `tile`'s total over the waves, in wave order.
// (ROW: multiply()'s sums of one row, [wave][tile][feature])
template <int RW, bool NORM, bool ROW, class Walk>
__device__ __forceinline__ void leave(Walk& c, const f32x4 (&acc)[RW]) {
    c.red = kRedBytes - c.red;
    if constexpr (NORM) {
        c.sq = kSqBytes - c.sq;
        if constexpr (Walk::ROOM1) {
            if (c.g < 2 && (c.tok & 12) == 4) *(float*)(c.lds + kSq + c.sq + (c.wave * 8 + c.g * 4 + (c.tok & 3)) * 4) = c.ss;
        } else {
            if (c.g == 0) *(float*)(c.lds + kSq + c.sq + (c.wave * 16 + c.tok) * 4) = c.ss;
        }
    }
#pragma unroll
    for (int q = 0; q < RW; ++q) {
        if constexpr (ROW) {
            float s[Walk::R];
#pragma unroll
            for (int t = 0; t < Walk::R; ++t) s[t] = quad_rows_sum(Walk::ONE ? (acc[q][0] + acc[q][1]) + (acc[q][2] + acc[q][3]) : acc[q][t]);
            float v = s[0];  // of row g
#pragma unroll
            for (int t = 1; t < Walk::R; ++t) v = c.g == t ? s[t] : v;
            if (c.g < Walk::R) *(float*)(c.lds + kRed + c.red + (((c.wave * RW + q) * Walk::R + c.g) * 16 + c.tok) * 4) = v;
        } else {
            *(f32x4*)(c.lds + kRed + c.red + ((c.wave * RW + q) * 64 + c.lane) * 16) = acc[q];
        }
    }
    lds_barrier();
}
template <int RW, bool PACK, bool ROW, class Walk>
__device__ __forceinline__ f32x4 total(const Walk& c, int tile) {
    f32x4 p[kPassWaves];
#pragma unroll
    for (int v = 0; v < kPassWaves; ++v)
        p[v] = *(const f32x4*)(c.lds + kRed + c.red + (ROW ? (((v * RW + tile) * c.R + min(c.tok, c.R - 1)) * 16 + c.g * 4) * 4 : ((v * RW + tile) * 64 + c.lane) * 16));
    f32x4 s = p[0];
#pragma unroll
    for (int v = 1; v < kPassWaves; ++v) s += p[v];
    if constexpr (PACK && !ROW) {
#pragma unroll
        for (int v = 0; v < 4; ++v) s[v] += dpp_f<0x128, 0xF>(0.f, s[v]);  // row_ror:8: columns 8 .. 15 to 0 .. 7
    }
    return s;
}

// Sixteen features of a row's activations in that order: this lane's four.
template <bool PACK, bool NORM, class Walk>
__device__ __forceinline__ void put_planes(const Walk& c, void* planes, int n0, const float (&w)[4], float ss = 0.f) {
    if constexpr (Walk::F32) {
        const int off = (n0 >> 4) * tile_bytes(NORM, c.R, true) + (((n0 & 15) >> 2) * c.R + c.tok) * 16;
        const v4u v = {__float_as_uint(w[0]), __float_as_uint(w[1]), __float_as_uint(w[2]), __float_as_uint(w[3])};
        if (c.tok < c.T) __builtin_amdgcn_raw_buffer_store_b128(v, whole(planes), off, 0, Walk::kOut);
        if (c.tok < c.R) __builtin_amdgcn_raw_buffer_store_b128(v4u{kNotThere, kNotThere, kNotThere, kNotThere}, whole((const char*)planes + c.clear), off, 0, Walk::kOut);
        return;
    }
    uint32_t h01, l01, h23, l23;
    split_bf16x2(w[0], w[1], h01, l01);
    split_bf16x2(w[2], w[3], h23, l23);
    // (eight features' high parts to the even lane groups, their low parts to the odd ones: one store, one write of a line)
    const auto p01 = __builtin_amdgcn_permlane16_swap(h01, l01, false, false), p23 = __builtin_amdgcn_permlane16_swap(h23, l23, false, false);
    v4u v = {p01[0], p23[0], p01[1], p23[1]};
    const int tile = (n0 >> 5) * tile_bytes(NORM, c.R, false), half = (n0 >> 4) & 1;
    int off = tile + (half * 2 + (c.g >> 1)) * (PACK ? 32 : 16) * c.R + (c.g & 1) * (PACK ? 16 : 64) * c.R + c.tok * 16;
    bool put = c.tok < c.T, fill = c.tok < c.R;
    if constexpr (NORM && Walk::ROOM1) {
        off = tile + half * 128 + c.g * 16;
        if (c.tok == 1) {
            off = tile + half * 128 + 64;
            v = v4u{__float_as_uint(ss), __float_as_uint(ss), __float_as_uint(ss), __float_as_uint(ss)};
        }
        put = fill = c.tok == 0 || (c.tok == 1 && c.g == 0);
    }
    if (put) __builtin_amdgcn_raw_buffer_store_b128(v, whole(planes), off, 0, Walk::kOut);
    if (fill) __builtin_amdgcn_raw_buffer_store_b128(v4u{kNotThere, kNotThere, kNotThere, kNotThere}, whole((const char*)planes + c.clear), off, 0, Walk::kOut);
}

// What the projections hand over to a head: [row][64] queries (fp32) and keys (bf16), [64][row] values (bf16 in the upper half of a
// word, so that four rows' values are one load; `room` rows, a multiple of four).
struct Fresh {
    Rsrc q, k, v;
    int room;
};
__host__ __device__ inline int fresh_room(int rows) { return (rows + 3) & ~3; }

// A row's scaled query of a head (bf16 models): [sixteen features][eight features][high, low parts], 256 bytes.
// This lane's four features of a row as the 16 bytes it stores there, at [sixteen features] * 64 + g * 16
__device__ __forceinline__ v4u query_parts(const f32x4& q) {
    uint32_t h01, l01, h23, l23;
    split_bf16x2(q[0], q[1], h01, l01);
    split_bf16x2(q[2], q[3], h23, l23);
    const auto p01 = __builtin_amdgcn_permlane16_swap(h01, l01, false, false), p23 = __builtin_amdgcn_permlane16_swap(h23, l23, false, false);
    return v4u{p01[0], p23[0], p01[1], p23[1]};
}
// ... and where lane (row, g) finds features 32 ks + 8 g ..: high parts in columns 0 .. 7 and low ones in 8 .. 15, or part p
template <bool PACK, class Walk>
__device__ __forceinline__ int query_piece(const Walk& c, int ks, int p) {
    return (2 * ks + (c.g >> 1)) * 64 + (c.g & 1) * 32 + (PACK ? c.tok >> 3 : p) * 16;
}

}  // namespace bild
