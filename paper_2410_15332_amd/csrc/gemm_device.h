// Device helpers of the GEMM kernels: buffer->LDS loads and what waits for them.
#pragma once

#include <hip/hip_runtime.h>

namespace epic {

constexpr int kBufWord3 = 0x00020000;                   // gfx9 raw buffer descriptor word 3

typedef __attribute__((address_space(3))) void lds_void;

// One 16-byte-per-lane buffer->LDS load (1 KB per wavefront: lane l's 16 bytes land
// at dst + 16 l).  A plain function, so the call is never a template-dependent
// expression (the host pass cannot check this builtin inside a template).
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t rs, char* dst, int voff, int soff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (lds_void*)dst, 16, voff, soff, 0, 0);
}

// Workgroup barrier ordering LDS accesses only (waits for this wavefront's LDS
// reads, not for its buffer->LDS loads still in flight).
__device__ __forceinline__ void barrier_lds() {
  __asm__ volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// At most N of this wavefront's vector memory operations outstanding (they
// complete in issue order); gfx9 encoding: vmcnt bits [3:0] and [15:14].
template <int N>
__device__ __forceinline__ void wait_vmem() {
  static_assert(N >= 0 && N < 64, "vmcnt field");
  __builtin_amdgcn_s_waitcnt((N & 15) | (0x7 << 4) | (0xF << 8) | ((N >> 4) << 14));
}

}  // namespace epic
