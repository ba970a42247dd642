// bild_head_stats / bild_head_stats_static: the final norm + LM head + softmax statistics of the decoding path
// (the fused vocabulary sweep of a decoder pass) as a call of its own on hidden rows the caller already holds
// on the device.  Both entry points run the same kernels; they differ only in where the scratch buffer lives
// (per-workgroup partial statistics, the logits of the targets):
//   bild_head_stats         takes it from the model's pool (a few buffers at most, freed with the model) and gives it back
//                           before returning: an allocation and its release cost more than a row of a small vocabulary;
//   bild_head_stats_static  uses a file-scope device array, so the call allocates nothing at all.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstring>

#include "bild_state.h"
#include "kernel_common.h"

using namespace bild;

namespace {

// Scratch layout (bytes): [256, 512) logits of the targets, one float per row; [512, ...) partial statistics,
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
        bild_row_stats o;
        o.zmax = r.m;
        o.lse = r.m + logf(r.s);
        o.argmax = r.idx;
        o.z_target = __builtin_nanf("");
        if (a.targets) {
            const int tgt = a.targets[t];
            if (tgt >= 0 && tgt < a.vocab) o.z_target = a.zt[t];  // (the head kernel has left it)
        }
        a.out[t] = o;
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

int head_stats_run(const bild_model* m, int rows, const int32_t* targets, bild_row_stats* out, hipStream_t st, const GemmArgs& g) {
    HIPC(launch_gemm(g, m->cfg.dtype, st));
    MergeArgs ma;
    ma.part = g.part;
    ma.nparts = g.part_ld;
    ma.zt = g.zt;
    ma.targets = targets;
    ma.vocab = m->cfg.vocab;
    ma.out = out;
    hipLaunchKernelGGL(head_stats_merge_kernel, dim3(rows), dim3(ma.nparts > 2048 ? 1024 : 256), 0, st, ma);
    HIPC(hipGetLastError());
    return BILD_OK;
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
    if (gemm_init() != hipSuccess) return BILD_EHIP;
    hipStream_t st = (hipStream_t)hip_stream;
    void* slots = nullptr;
    if (int rc = of_device(g_counts_ptr, HIP_SYMBOL(counts), &slots)) return rc;
    GemmArgs g = head_gemm(m, x_dev, rows, targets_dev, nullptr, (const int*)slots);
    const size_t bytes = kHdrBytes + (size_t)g.part_ld * sizeof(StatPart) * rows;
    HeadScratch b = m->head_pool.take(bytes);
    if (!b.p) return BILD_ENOMEM;
    g.zt = (float*)((char*)b.p + 256);
    g.part = (StatPart*)((char*)b.p + kHdrBytes);
    int rc = head_stats_run(m, rows, targets_dev, out_dev, st, g);
    if (hipStreamSynchronize(st) != hipSuccess && rc == BILD_OK) rc = BILD_EHIP;  // the scratch is in use until here
    m->head_pool.give(b);
    return rc;
}

extern "C" int bild_head_stats_static(const bild_model* m, const float* x_dev, int rows, const int32_t* targets_dev,
                                      bild_row_stats* out_dev, void* hip_stream) {
    if (int rc = check_args(m, x_dev, rows, out_dev)) return rc;
    if (gemm_init() != hipSuccess) return BILD_EHIP;
    void *scr = nullptr, *slots = nullptr;
    if (int rc = of_device(g_scratch_ptr, HIP_SYMBOL(scratch), &scr)) return rc;
    if (int rc = of_device(g_counts_ptr, HIP_SYMBOL(counts), &slots)) return rc;
    const GemmArgs g = head_gemm(m, x_dev, rows, targets_dev, scr, (const int*)slots);
    if (g.part_ld > kStaticMaxParts) return BILD_ECAP;  // more partial statistics than the array holds
    return head_stats_run(m, rows, targets_dev, out_dev, (hipStream_t)hip_stream, g);
}
