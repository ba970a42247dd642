// LM head: final norm, vocabulary sweep, softmax statistics (head.hip).
#pragma once
#include "bild_internal.h"

namespace bild {

struct HeadArgs {
    TMat W;
    const float* x;      // [T][ldx]
    int ldx, T;
    bool f32;            // of an fp32 model
    const float* gain;
    float eps, scale;
    int vocab;
    const int *y, *ylen_ptr, *pos_ptr;  // target of row t is y[p + t + 1] if p + t + 1 < *ylen_ptr, p = *pos_ptr (null: 0) + pos_add
    int pos_add;
    StatPart* part;      // [T][part_ld], one per workgroup
    int part_ld;
    float* zt;           // [T] logit of the target
    float* dbg;          // nullable: [T][vocab] logits
    // non-null: the last workgroup joins the partials and writes the rows' results here
    bild_row_stats* out;
    unsigned* arrived;   // zero between launches
    unsigned *done, call;  // (done nullable) pinned host memory: `call` goes to done[row] once the row's result is in memory
};
// workgroups (partials per row); 0: not a shape the kernel is made for
int head_groups(const TMat& W, int T, bool f32);
hipError_t launch_head(const HeadArgs& a, hipStream_t st);
hipError_t head_init();
// which kernels have the head of bild_head_stats (head_stats.hip): the GEMM's short workgroups and a merge, this kernel, the thin GEMM on tile planes
enum { HEAD_SHORT, HEAD_SWEEP, HEAD_PLANES };
int head_route(const TMat& W, int dtype, int rows);

#ifdef __HIPCC__
// One row's result, by one lane: past the caches, and acknowledged before the host is told.
__device__ __forceinline__ void put_row_stats(bild_row_stats* out, int row, float zmax, float s, int argmax, bool has_target, float z_target, unsigned* done, unsigned call) {
    typedef unsigned v4u __attribute__((ext_vector_type(4)));
    static_assert(sizeof(bild_row_stats) == 16, "one store");
    bild_row_stats o;
    o.zmax = zmax;
    o.lse = zmax + logf(s);
    o.argmax = argmax;
    o.z_target = has_target ? z_target : __builtin_nanf("");
    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, o), __builtin_amdgcn_make_buffer_rsrc((void*)(out + row), 0, 16, 0x00027000), 0, 0, 17);
    if (done) {
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_raw_buffer_store_b32(call, __builtin_amdgcn_make_buffer_rsrc((void*)(done + row), 0, 4, 0x00027000), 0, 0, 17);
    }
}
#endif

}  // namespace bild
