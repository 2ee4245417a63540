// What the projection kernels share: direct global -> LDS copies, the barrier and the waits of
// their LDS rings, and the SwiGLU activation.
#pragma once

#include "common.hpp"

namespace orthrus {

__device__ __forceinline__ float silu(float g) { return g / (1.f + __expf(-g)); }

// 16-byte global -> LDS copy: lane i of the wave writes lds + 16 * i (lds is wave-uniform).
// AUX is the cache policy: 0 default, kNonTemporal for data the launch reads exactly once.
constexpr int kNonTemporal = 2;
template <int AUX = 0>
__device__ __forceinline__ void copy16_to_lds(const void *src, char *lds) {
    __builtin_amdgcn_global_load_lds(src, (__attribute__((address_space(3))) void *)lds, 16, 0, AUX);
}

// s_waitcnt immediate that waits until at most n vector-memory operations are outstanding
// (gfx9 encoding: vmcnt[3:0] in bits 3:0 and vmcnt[5:4] in bits 15:14; expcnt and lgkmcnt at
// their maxima so they impose no wait)
template <int N>
constexpr int vmcnt_imm() {
    static_assert(N >= 0 && N < 64, "vmcnt range");
    return (N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8);
}

// workgroup barrier for the LDS ring: the LDS reads issued before it have completed and no
// memory access moves across it; unlike __syncthreads it does not drain the outstanding
// global->LDS copies of later stages (their completion is awaited explicitly with vmcnt)
__device__ __forceinline__ void ring_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

}  // namespace orthrus
