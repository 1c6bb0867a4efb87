// Waits for the kernels whose global loads go straight into LDS (decay_input.hip, key_compress.hip).  Such loads are outside the
// compiler's view of a wave's own LDS accesses, so these kernels count them by hand.
#pragma once
#include <hip/hip_runtime.h>

namespace wkv6 {
namespace {

// At most `kYounger` of the wave's youngest loads may still be on their way behind this, and no LDS access moves across it.
template <int kYounger>
__device__ __forceinline__ void wait_loads() {
    static_assert(kYounger >= 0 && kYounger < 64, "vmcnt");
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt((kYounger & 15) | (kYounger >> 4) << 14 | 7 << 4 | 15 << 8);
    __builtin_amdgcn_sched_barrier(0);
}

}  // namespace
}  // namespace wkv6
