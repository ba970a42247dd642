// bild_head_stats / bild_head_stats_static: the final norm + LM head + softmax statistics of the decoding path
// (the fused vocabulary sweep of a decoder pass) as a call of its own on hidden rows the caller already holds
// on the device.  Both entry points run the same kernels; they differ only in where the scratch buffer lives
// (per-workgroup partial statistics, the logits of the targets):
//   bild_head_stats         takes it from the model's pool (a few buffers at most, freed with the model) and gives it back
//                           before returning: an allocation and its release cost more than a row of a small vocabulary;
//   bild_head_stats_static  uses a file-scope device array, so the call allocates nothing at all.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstring>

#include "bild_state.h"
#include "gemm_thin.h"
#include "head.h"
#include "kernel_common.h"

using namespace bild;

namespace {

// Scratch layout (bytes): [0, 256) workgroups that have arrived (pool buffers: zero between calls); [256, 512) logits of the targets, one float per row, and the rows' sums of squares; [512, ...) partial statistics,
// StatPart[rows][workgroups].
constexpr size_t kHdrBytes = 512;
constexpr size_t kStaticScratchBytes = (size_t)4 << 20;  // 4 MiB
constexpr int kStaticMaxParts = (int)((kStaticScratchBytes - kHdrBytes) / (sizeof(StatPart) * kMaxRows));

// One copy per GPU the library runs on, kept until the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress: the device address of the array is looked up once per device (scratch_of_device) and that
// pointer is what kernels and every other call receive.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// slot counts the head kernel can be pointed at
static __device__ int counts[kMaxRows + 2] = {0,  1,  2,  3,  4,  5,  6,  7,  8,  9,  10, 11, 12, 13, 14, 15, 16,
                                              17, 18, 19, 20, 21, 22, 23, 24, 25, 26, 27, 28, 29, 30, 31, 32, 33};
static_assert(kMaxRows == 32, "one count per number of rows and one more");

constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices] = {};
void* g_counts_ptr[kMaxDevices] = {};

int of_device(void* (&table)[kMaxDevices], const void* symbol, void** out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return BILD_EHIP;
    void* p = __atomic_load_n(&table[dev], __ATOMIC_ACQUIRE);
    if (!p) {
        if (hipGetSymbolAddress(&p, symbol) != hipSuccess || !p) return BILD_EHIP;
        __atomic_store_n(&table[dev], p, __ATOMIC_RELEASE);
    }
    *out = p;
    return BILD_OK;
}

struct MergeArgs {
    const StatPart* part;
    int nparts;
    const float* zt;
    const int* targets;
    int vocab;
    bild_row_stats* out;
    unsigned* done;  // (see HeadArgs)
    unsigned call;
};

// Merges the per-workgroup partial statistics of one row per workgroup, in a fixed order, and writes the row's result.  One
// workgroup for all rows, a wave for one row after the other, took 72 us at 21 rows of 7 816 partials (250 112 ids).
__global__ __launch_bounds__(1024) void head_stats_merge_kernel(const MergeArgs a) {
    __shared__ StatPart share[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nwv = blockDim.x >> 6, t = blockIdx.x;
    const StatPart* row = a.part + (size_t)t * a.nparts;
    StatPart sp[8];
    const int stride = nwv * 64 * 8;
    Stat r = stat_neutral();
    for (int p0 = wave * 64 * 8; p0 < a.nparts; p0 += stride) {
        load_parts(sp, row, p0 + lane, a.nparts);
        take_parts(r, sp, p0 + lane, a.nparts);
    }
    r = join_parts(r);
    if (lane == 0) share[wave] = StatPart{r.m, r.s, r.idx, 0};
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < nwv; ++w) r = stat_merge<true>(r, Stat{share[w].m, share[w].s, share[w].idx});
        const int tgt = a.targets ? a.targets[t] : -1;
        const bool has = tgt >= 0 && tgt < a.vocab;
        put_row_stats(a.out, t, r.m, r.s, r.idx, has, has ? a.zt[t] : 0.f, a.done, a.call);  // (the head kernel has left it)
    }
}

// The launch shape of the head for `rows` rows; *nparts receives the number of workgroups (partials per row).
GemmArgs head_gemm(const bild_model* m, const float* x, int rows, const int32_t* targets, void* scr, const int* slots) {
    GemmArgs g;
    std::memset((void*)&g, 0, sizeof(g));
    const bild_model_config& c = m->cfg;
    g.W = m->head;
    g.x = x;
    g.ldx = c.d_model;
    g.T = rows;
    g.gain = m->dec_final;
    g.eps = c.norm_eps;
    g.d_head = c.d_head;
    g.i_dim = m->inner();
    g.act = c.act;
    g.vocab = c.vocab;
    g.epi = EPI_LMHEAD;
    g.scale = c.logit_scale;
    // the kernel takes the target of row t from y[t + 1] while t + 1 < *ylen_ptr: y is the caller's array moved down
    // by one slot, and the slot count is rows + 1 (0 without targets, so that y is never read)
    g.y = targets ? targets - 1 : slots;
    g.ylen_ptr = slots + (targets ? rows + 1 : 0);
    g.zt = (float*)((char*)scr + 256);
    g.part = (StatPart*)((char*)scr + kHdrBytes);
    gemm_pick_shape(g, c.dtype);
    g.part_ld = (int)gemm_num_blocks(g);
    return g;
}

int head_stats_run(const bild_model* m, int rows, const int32_t* targets, bild_row_stats* out, hipStream_t st, const GemmArgs& g, unsigned* done, unsigned call) {
    HIPC(launch_gemm(g, m->cfg.dtype, st));
    MergeArgs ma;
    ma.part = g.part;
    ma.nparts = g.part_ld;
    ma.zt = g.zt;
    ma.targets = targets;
    ma.vocab = m->cfg.vocab;
    ma.out = out;
    ma.done = done;
    ma.call = call;
    hipLaunchKernelGGL(head_stats_merge_kernel, dim3(rows), dim3(ma.nparts > 2048 ? 1024 : 256), 0, st, ma);
    HIPC(hipGetLastError());
    return BILD_OK;
}

// The same by the kernel whose workgroups stay for the whole sweep, where it is made for the shape (workgroups > 0).  `joins`: its
// last workgroup writes the results itself, which takes a count that no other call touches; else a launch of its own does.
int head_sweep_run(const bild_model* m, const float* x, int rows, const int32_t* targets, bild_row_stats* out, hipStream_t st, const GemmArgs& g, int groups, bool joins, unsigned* done,
                   unsigned call) {
    HeadArgs h;
    std::memset((void*)&h, 0, sizeof(h));
    h.W = m->head;
    h.x = x;
    h.ldx = m->cfg.d_model;
    h.T = rows;
    h.f32 = m->cfg.dtype == BILD_DT_F32;
    h.gain = g.gain;
    h.eps = g.eps;
    h.scale = g.scale;
    h.vocab = g.vocab;
    h.y = g.y;
    h.ylen_ptr = g.ylen_ptr;
    h.part = g.part;
    h.part_ld = groups;
    h.zt = g.zt;
    if (joins) {
        h.out = out;
        h.arrived = (unsigned*)((char*)g.zt - 256);
        h.done = done;
        h.call = call;
    }
    HIPC(launch_head(h, st));
    if (!joins) {
        const MergeArgs ma = {g.part, groups, g.zt, targets, m->cfg.vocab, out, done, call};
        hipLaunchKernelGGL(head_stats_merge_kernel, dim3(rows), dim3(256), 0, st, ma);
        HIPC(hipGetLastError());
    }
    return BILD_OK;
}
// (behind `parts` workgroups' partial statistics)
size_t planes_at(int rows, int parts) { return (kHdrBytes + (size_t)parts * rows * sizeof(StatPart) + 1023) / 1024 * 1024; }
ThinArgs planes_head(const bild_model* m, int rows, const GemmArgs& g, void* scr) {
    ThinArgs a;
    std::memset((void*)&a, 0, sizeof(a));
    a.W = m->head;
    a.T = rows;
    a.epi = EPI_LMHEAD;
    a.part_ld = thin_shape(m->head, EPI_LMHEAD, 0, rows).groups;
    a.xp = (const char*)scr + planes_at(rows, a.part_ld);
    a.ssq = (const float*)((const char*)scr + 384);
    a.ssq_parts = 1;
    a.eps = g.eps;
    a.scale = g.scale;
    a.vocab = g.vocab;
    a.y = g.y;
    a.ylen_ptr = g.ylen_ptr;
    a.part = g.part;
    a.zt = g.zt;
    return a;
}
size_t planes_scratch(const bild_model* m, int rows, int parts) { return planes_at(rows, parts) + plane_bytes(rows, (size_t)m->head.tk * 32); }
int head_planes_run(const bild_model* m, const float* x, int rows, const int32_t* targets, bild_row_stats* out, hipStream_t st, const ThinArgs& a, unsigned* done, unsigned call) {
    RowCopyArgs r;
    std::memset((void*)&r, 0, sizeof(r));
    r.src = x;
    r.d = m->cfg.d_model;
    r.T = rows;
    HIPC(launch_row_tiles(r, m->dec_final, const_cast<char*>(a.xp), const_cast<float*>(a.ssq), st));
    HIPC(launch_gemm_thin(a, st));
    const MergeArgs ma = {a.part, a.part_ld, a.zt, targets, m->cfg.vocab, out, done, call};
    hipLaunchKernelGGL(head_stats_merge_kernel, dim3(rows), dim3(256), 0, st, ma);
    HIPC(hipGetLastError());
    return BILD_OK;
}
// Whether the short workgroups of the GEMM, which stage all rows, find room for two on a compute unit.
bool two_short(const TMat& W, int dtype, int rows) {
    GemmArgs g;
    std::memset((void*)&g, 0, sizeof(g));
    g.W = W;
    g.T = rows;
    g.epi = EPI_LMHEAD;
    gemm_pick_shape(g, dtype);
    return gemm_lds_bytes(g, dtype) <= (size_t)80 * 1024;
}

}  // namespace

// Which kernels have the head.  One rule for both entry points, whose results are the same bits.  All figures us, short workgroups / the other.
//
// Planes: bf16 rows wider than the sweep's registers hold, as tile planes for the thin GEMM (gemm_thin.hip), which has them on their way beside the weights, where
// every short workgroup stages all of them.  A launch more, so from five rows on.  A call that waits, 5, 9, 16, 20, 32 rows: 4096 x 4000
// 24.9, 28.2, 36.7, 36.5, 52.6 / 22.6, 24.4, 28.7, 28.8, 30.7; x 16 000 49.3, 43.6, 66.5, 80.9, 102 / 43.9, 41.5, 41.7, 45.5, 48.0; x 50 000 121, 104 to 110, 158, 196, 234 / 104, 108, 113, 114,
// 120; 2112 x 50 000, 5, 9, 20 rows 55, 78, 118 / 52, 54, 60; 3072 76, 101, 147 / 72, 73, 83; 5120 143, 155, 236 / 118,
// 122, 131.  Eight rows and less of 8 MB the same, one and four rows of any size 0 to 10 % slower.  Where two short workgroups fit a compute unit they are as fast: nine
// rows of 4096 x 24 000, 32 000, 50 000, 64 000, 100 000 61.6, 60.9, 105, 117, 198 / 54.8, 64.7, 109, 119, 184; five of 7424 x 16 000, 24 000, 32 000, 50 000 57, 91, 106, 165 / 55, 95, 107, 169
// (but twelve of 3072, eleven of 3456, ten of 3712, eight of 4608, seven of 5312, six of 6144 1.00 to 1.6 times as long at all sizes).
//
// Sweep (head.hip), bf16.  Up to eight rows of matrices of 50 MB or so are the short workgroups', of which more are on a compute unit when weights begin to arrive.
// A call that does not wait and one that does (there the sweep joins its results itself), one row: 512 x 16 000 ids
// 9.4 / 9.1, 17.1 / 16.8; x 32 128 9.9 / 10.4, 17.8 / 18.0; x 64 000 17.2 / 18.6, 25.0 / 24.0; 1024 x 4000 8.8 / 8.8, 16.8 / 16.6; x 16 000 9.9 / 10.4, 17.9 / 17.9;
// x 32 128 16.7 / 18.4, 24.6 / 24.1; 2048 x 1000 9.7 / 10.4, 17.3 / 16.2; x 7809 10.3 / 11.4, 18.6 / 19.3; x 16 000 17.0 / 17.9, 24.7 / 24.2; 125 MB 512, 1024,
// 2048 wide 32.7 / 27.7, 25.6 / 26.8, 28.2 / 26.8 and 41.2 / 33.0, 33.6 / 32.7, 35.7 / 32.3.  Two, four, eight rows: 512 x 64 000 20.7, 20.7, 21.2 / 18.3, 18.6,
// 18.7; 1024 x 16 000 10.7, 11.4, 13.0 / 10.3, 10.8, 11.8; x 32 128 16.8, 17.1, 17.8 / 18.0, 18.2, 19.1; 2048 x 7809 11.4, 12.5, 14.7 / 11.5, 12.4, 13.8; x 16 000 17.4,
// 17.4, 20.9 / 18.3, 19.2, 20.6.  From nine rows on the sweep is never slower.
//
// Sweep, fp32, a call that waits, 1, 8, 16, 32 rows: 512 x 50 000 34.5, 36.3, 38.7, 50.1 / 32.0, 32.1, 34.1, 42.0; x 250 112 119, 123, 124, 157 / 102, 102, 104, 116; 1024 x 4000
// 20.7, 20.4, 22.4, 26.1 / 18.4, 19.6, 21.2, 24.1; x 50 000 53.6, 51.4, 58.4, 98.7 / 46.5, 47.7, 51.2, 59.7; up to 1024 wide at any size (0.7 to 1.03 times), but for
// one row up to 256 wide (256 x 32 000, 50 000, 64 000 19.9, 25.4, 27.8 / 21.4, 28.0, 27.6).
// Up to 2048 wide, small and large matrices, and the others from nine rows on: 2048 x 1000 20.1, 22.2, 24.2, 31.7 / 18.3, 19.6, 23.7, 28.8; x 4000
// 20.6, 22.9, 25.4, 32.6 / 21.8, 22.7, 25.9, 30.2; x 16 000 38.6, 40.4, 51.5, 73.7 / 38.2, 40.1, 45.1, 49.9 (four rows 36.4 / 39.4); x 50 000 98, 101, 130, 191 / 86, 87, 89, 106; four rows x 32 000,
// 36 000 57, 73 / 60, 63; 1536 x 50 000, 60 000, 90 000, one row 71, 82, 117 / 73, 84, 109.  Not a little above the last-level cache's 256 MB below 1536 wide (1280 x 40 000, 60 000, 90 000, 1, 9 rows
// 51, 56; 68, 69; 105, 104 / 51, 51; 81, 78; 99, 96), nor large ones with two row tiles below 1792 (1280 x 60 000, 90 000, 17, 32 rows 114, 161; 120, 138 / 101, 103; 137, 140; 1536 x 90 000, 128 000 134, 147; 177, 191 / 142, 144; 194, 196).
// Wider ones spill registers, and win only against short workgroups that do not fit a compute unit twice: 4096 x 12 000, 1, 8, 9, 10, 16 rows 48.6, 68.8, 60.2, 75.3, 88.2 /
// 58, 58, 58.2, 58.2, 60.5; x 26 000 98, 111, 97, 116, 125 / 110, 108, 110, 110, 113; x 46 000 153, 167, 155, 170, 183 / 166, 163, 165, 166, 168; x 60 000 193, 212, 193, 219, 235 / 202, 195, 197, 198, 199;
// 3840 x 20 000 10, 16 rows 94, 102 / 80, 83, x 46 000 151, 159 / 165, 166; 3712 x 12 000 12, 16 rows 68, 75 / 54, 56; 2112 to 3456 x 16 000 to 75 000 0.9 to 1.45 times as long.
int bild::head_route(const TMat& W, int dtype, int rows) {
    const int tk = W.tk;
    const size_t mb = ((size_t)W.tn * tk * kTileBytes) >> 20;
    if (dtype == BILD_DT_BF16) {
        if (tk > 64) {
            if (rows <= 4 || (rows <= 8 && (size_t)W.tn * tk * kTileBytes < (size_t)16 << 20)) return HEAD_SHORT;
            const bool even = (rows > 8 ? tk > 120 && mb < 600 : tk >= 224) && mb >= 200;
            return even && two_short(W, dtype, rows) ? HEAD_SHORT : HEAD_PLANES;
        }
        return rows > 8 || mb >= 96 || (rows > 1 ? mb < 48 || tk <= 16 : mb < (tk > 32 ? 8u : 24u)) ? HEAD_SWEEP : HEAD_SHORT;
    }
    if (tk <= 64) return rows == 1 && tk <= 16 && mb >= 24 && mb < 60 ? HEAD_SHORT : HEAD_SWEEP;
    if (tk <= 128) {
        if (rows > 16) return tk < 112 && mb >= 400 ? HEAD_SHORT : HEAD_SWEEP;
        if (tk < 96 && mb >= 256 && mb < 400) return HEAD_SHORT;
        return rows > 8 || mb < 16 || mb >= (tk < 128 ? 320u : 256u) ? HEAD_SWEEP : HEAD_SHORT;
    }
    if (rows > 16 || tk < 232 || mb < 128 || (tk < 256 && mb >= 320) || (rows <= 9 && (tk < 256 || mb < 600))) return HEAD_SHORT;
    return two_short(W, dtype, rows) ? HEAD_SHORT : HEAD_SWEEP;
}

namespace {

// Workgroups of the sweep; 0: other kernels have the head.
int sweep_groups(const bild_model* m, int rows) {
    return head_route(m->head, m->cfg.dtype, rows) == HEAD_SWEEP ? head_groups(m->head, rows, m->cfg.dtype != BILD_DT_BF16) : 0;
}

bool all_done(const unsigned* done, unsigned call, int rows) {
    for (int r = 0; r < rows; ++r)
        if (__atomic_load_n(done + r, __ATOMIC_ACQUIRE) != call) return false;
    return true;
}
// Whether all rows' results are in memory, seen in the words the kernel leaves in pinned memory: some microseconds before the stream's
// completion reaches the host.  (512 x 32 128 ids, one row, the host waiting for the stream / polling: the call 22.4 / 17.5 us, with a copy of the
// result to the host behind it 37.0 / 31.9, with another launch 27.0 / 23.3; with a device synchronisation alone, which then comes before the
// stream has retired the launch, 25.6 / 29.0.)  Not for long: what else is on the stream is waited for without spinning.
bool rows_done(const unsigned* done, unsigned call, int rows) {
    const auto t0 = std::chrono::steady_clock::now();
    int r = 0;
    for (unsigned spins = 1;; ++spins) {
        while (r < rows && __atomic_load_n(done + r, __ATOMIC_ACQUIRE) == call) ++r;
        if (r == rows) return true;
        if ((spins & 255) == 0 && std::chrono::steady_clock::now() - t0 > std::chrono::milliseconds(2)) return false;
    }
}

int check_args(const bild_model* m, const float* x, int rows, bild_row_stats* out) {
    if (!m || !x || !out || rows < 1 || rows > kMaxRows) return BILD_EINVAL;
    if (((uintptr_t)x & 15) != 0) return BILD_EINVAL;  // rows are read with 16-byte loads
    return BILD_OK;
}

}  // namespace

extern "C" int bild_head_stats(const bild_model* m, const float* x_dev, int rows, const int32_t* targets_dev,
                               bild_row_stats* out_dev, void* hip_stream) {
    if (int rc = check_args(m, x_dev, rows, out_dev)) return rc;
    if (gemm_init() != hipSuccess || head_init() != hipSuccess || gemm_thin_init() != hipSuccess) return BILD_EHIP;
    hipStream_t st = (hipStream_t)hip_stream;
    void* slots = nullptr;
    if (int rc = of_device(g_counts_ptr, HIP_SYMBOL(counts), &slots)) return rc;
    GemmArgs g = head_gemm(m, x_dev, rows, targets_dev, nullptr, (const int*)slots);
    const int groups = sweep_groups(m, rows);
    const bool planes = head_route(m->head, m->cfg.dtype, rows) == HEAD_PLANES;
    const size_t bytes = std::max(kHdrBytes + (size_t)std::max(g.part_ld, groups) * sizeof(StatPart) * rows, planes ? planes_scratch(m, rows, thin_shape(m->head, EPI_LMHEAD, 0, rows).groups) : 0);
    HeadScratch b = m->head_pool.take(bytes, st);
    if (!b.p) return BILD_ENOMEM;
    g.zt = (float*)((char*)b.p + 256);
    g.part = (StatPart*)((char*)b.p + kHdrBytes);
    // (one row per wave of the last workgroup: more are joined sooner by a launch of a workgroup each; 512 x 32 128 ids, 1, 8, 16, 32
    // rows: 22.2, 23.0, 25.0, 29.9 us joined in the sweep, 22.9, 23.3, 23.6, 25.4 by a launch)
    b.calls += 1;
    int rc = planes   ? head_planes_run(m, x_dev, rows, targets_dev, out_dev, st, planes_head(m, rows, g, b.p), b.done_dev, b.calls)
             : groups ? head_sweep_run(m, x_dev, rows, targets_dev, out_dev, st, g, groups, rows <= 8, b.done_dev, b.calls)
                      : head_stats_run(m, rows, targets_dev, out_dev, st, g, b.done_dev, b.calls);
    // the scratch is in use until here
    const bool seen = rc == BILD_OK && b.done && rows_done(b.done, b.calls, rows);
    if (!seen && hipStreamSynchronize(st) != hipSuccess && rc == BILD_OK) rc = BILD_EHIP;
    if (!seen && rc == BILD_OK && b.done && !all_done(b.done, b.calls, rows)) rc = BILD_EHIP;  // (nobody wrote the results)
    if (rc == BILD_OK) m->head_pool.give(b);
    else b.release();  // what it holds is not known
    return rc;
}

extern "C" int bild_head_stats_static(const bild_model* m, const float* x_dev, int rows, const int32_t* targets_dev,
                                      bild_row_stats* out_dev, void* hip_stream) {
    if (int rc = check_args(m, x_dev, rows, out_dev)) return rc;
    if (gemm_init() != hipSuccess || head_init() != hipSuccess || gemm_thin_init() != hipSuccess) return BILD_EHIP;
    void *scr = nullptr, *slots = nullptr;
    if (int rc = of_device(g_scratch_ptr, HIP_SYMBOL(scratch), &scr)) return rc;
    if (int rc = of_device(g_counts_ptr, HIP_SYMBOL(counts), &slots)) return rc;
    const GemmArgs g = head_gemm(m, x_dev, rows, targets_dev, scr, (const int*)slots);
    if (g.part_ld > kStaticMaxParts) return BILD_ECAP;  // more partial statistics than the array holds
    if (head_route(m->head, m->cfg.dtype, rows) == HEAD_PLANES) {
        const ThinArgs a = planes_head(m, rows, g, scr);
        if (planes_scratch(m, rows, a.part_ld) <= kStaticScratchBytes) return head_planes_run(m, x_dev, rows, targets_dev, out_dev, (hipStream_t)hip_stream, a, nullptr, 0);
    }
    // (calls that overlap on a GPU share the scratch: a count left wrong by them would outlast them)
    if (const int groups = sweep_groups(m, rows)) return head_sweep_run(m, x_dev, rows, targets_dev, out_dev, (hipStream_t)hip_stream, g, groups, false, nullptr, 0);
    return head_stats_run(m, rows, targets_dev, out_dev, (hipStream_t)hip_stream, g, nullptr, 0);
}
