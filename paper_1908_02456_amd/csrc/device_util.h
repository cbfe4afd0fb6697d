// Device helpers shared by the sweeps (fused.hip, kernels_staged.hip).
#pragma once

#include <hip/hip_runtime.h>

namespace abc_dev {

// Workgroup barrier ordering LDS only.  __syncthreads() also waits for every
// outstanding global load (vmcnt(0)), which would drain the next plane's
// prefetch at each barrier; here only LDS traffic (lgkmcnt) is waited for.
// The empty asm statements keep the compiler from moving memory accesses
// across the barrier; loads still in flight are waited for where their
// registers are first used.
__device__ __forceinline__ void sync_lds() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0xC07F);  // gfx9 encoding: vmcnt 63, expcnt 7, lgkmcnt 0
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Raw buffer loads: an offset at or beyond the buffer's size returns zero,
// which is how halo cells outside the box read as zero without a select on
// the loaded value (a select would force the wait right after the load).
// Buffers are limited to below 4 GiB (checked on the host).
constexpr unsigned kOob = 0xFFFFFFF0u;

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* p, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ void bload(__amdgpu_buffer_rsrc_t r, unsigned off, double2& v) {
  v = __builtin_bit_cast(double2, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
__device__ __forceinline__ void bload(__amdgpu_buffer_rsrc_t r, unsigned off, float2& v) {
  v = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
__device__ __forceinline__ void bload(__amdgpu_buffer_rsrc_t r, unsigned off, double& v) {
  v = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
__device__ __forceinline__ void bload(__amdgpu_buffer_rsrc_t r, unsigned off, float& v) {
  v = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}

}  // namespace abc_dev
