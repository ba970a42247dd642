// Partial results of several workgroups that the last of them to arrive joins, in one launch.
#pragma once
#include "kernel_common.h"

namespace bild {

// Called by all threads of a workgroup after its partial results have been stored with kPartAux; true in the last of the `n`
// workgroups that share `counter` (zero before the launch and after it), which then reads all of them with kPartAux.  The
// stores go past the L2s and are waited for, so that the count says that they are in memory; the readers' L2 drops a line that
// another die writes.  `share`: a word of LDS nobody else uses.
constexpr int kPartAux = 17;  // sc0 sc1
__device__ __forceinline__ bool last_in(unsigned* counter, unsigned n, unsigned* share) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    lds_barrier();
    if (threadIdx.x == 0) {
        const unsigned before = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (before == n - 1) __hip_atomic_store(counter, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *share = before;
    }
    lds_barrier();
    return __builtin_amdgcn_readfirstlane((int)*share) == (int)n - 1;
}

}  // namespace bild
