// GEMM of bf16 models over 2 .. 32 rows whose activations travel as tile planes (gemm_thin.hip).
#pragma once
#include "bild_internal.h"

namespace bild {

struct ThinArgs {
    TMat W;
    const char* xp;         // input: tile planes (plane_offset), W.tk input tiles wide, times the norm's gain where there is one
    int T;                  // rows, at most kMaxRows
    const float* ssq;       // normed input: [ssq_parts][kMaxRows] partial sums of squares per row
    int ssq_parts;
    float eps;
    int epi;                // EPI_STORE, EPI_RESID, EPI_ACT, EPI_QKV or EPI_LMHEAD
    int act;
    // inputs cut into slices, a workgroup each, whose sums the last of them joins (thin_shape)
    float* sums;            // [kThinSums]
    unsigned* arrived;      // [kThinArrivals], zero between launches
    // EPI_STORE: out[t][n] = v; EPI_RESID: out[t][n] += v, and the planes of the result times np_gain
    float* out;
    int ldo;
    char* np;               // output planes, np_tk tiles wide (EPI_RESID, EPI_ACT)
    int np_tk;
    const float* np_gain;
    float* np_ssq;          // EPI_RESID: [W.tn][kMaxRows] sums of squares of sixteen features each
    // EPI_QKV
    int q_dim, i_dim, d_head, vcap;
    float* q_out;
    void *k_cache, *v_cache;
    const int* pos_ptr;     // position of row 0 = *pos_ptr
    const double2* rope;    // null: no rotation
    // EPI_LMHEAD: rows first .. T - 1
    int first;
    float scale;
    int vocab;
    const int *y, *ylen_ptr;  // target of row t is y[*pos_ptr + t + 1] if below *ylen_ptr (pos_ptr null: 0)
    StatPart* part;         // [row - first][part_ld], one per workgroup
    int part_ld;
    float* zt;
    float* dbg;             // nullable: [row - first][vocab] logits
};
struct ThinShape {
    int rw, groups, slices;  // feature tiles per workgroup, workgroups (EPI_LMHEAD: partials per row) and slices of the inputs
};
ThinShape thin_shape(const TMat& W, int epi, int act, int T);
constexpr int kThinArrivals = 256;
constexpr size_t kThinSums = (size_t)256 * 12 * 256;  // floats: a workgroup's units of 64 x 4 for at most 256 workgroups
hipError_t launch_gemm_thin(const ThinArgs& a, hipStream_t st);
hipError_t gemm_thin_init();

}  // namespace bild
