// Attention of bf16 models over a long cache for up to 32 rows, keys split over workgroups and joined by the last (attn_split.hip).
#pragma once
#include "bild_internal.h"

namespace bild {

struct AttnSplitArgs {
    const float* q;      // [T][i_dim]
    const void *k, *v;   // [capacity][i_dim]; transposed: [i_dim][vcap]
    int vcap, i_dim, heads, d_head, T;
    int causal;          // 1: row t sees keys <= *len_ptr + t; 0: *len_ptr keys
    const int* len_ptr;
    float scale;
    int splits;          // workgroups per head
    int waves;           // per workgroup, 4 or 8
    float* part;         // [kAttnSplitFloats]
    unsigned* arrived;   // [kAttnSplitHeads], zero between launches
    float* out;          // [T][i_dim], or
    char* ob_t;          // (non-null) tile planes of it
};
constexpr int kAttnSplitGroups = 512, kAttnSplitHeads = 256;
constexpr size_t kAttnSplitFloats = (size_t)kAttnSplitGroups * (32 * 128 + 64);
// splits and waves for up to `keys` keys of a cache of `vcap`; 0 splits: not a shape the kernel is made for
void attn_split_shape(int heads, int d_head, int i_dim, int vcap, int keys, int* splits, int* waves);
hipError_t launch_attn_split(const AttnSplitArgs& a, hipStream_t st);
hipError_t attn_split_init();

}  // namespace bild
