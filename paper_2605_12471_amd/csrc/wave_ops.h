// Operations of one wavefront shared by the attention kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#define LDS_PTR(T, p) ((T __attribute__((address_space(3)))*)(uintptr_t)(p))

namespace kvfold {

// Lanes l and l ^ 32 exchange x; both end with the maximum / the sum.
__device__ __forceinline__ float pair_max(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pair_sum(float x) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Lanes l and l ^ 16 exchange x; both end with the maximum / the sum.
__device__ __forceinline__ float row16_max(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float row16_sum(float x) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// One wavefront-wide 1 KiB copy global -> LDS: lane l's 16 bytes, read from base + off, land at
// lds_base + 16*l.  The compiler is not told about the LDS write; ordering is done by hand with
// wait_vm<> + barrier.  The hardware needs one wait state between a write of m0 and a copy to LDS, and the compiler
// adds none inside an asm block.
__device__ __forceinline__ void dma16(const unsigned char* base_uniform, unsigned off, unsigned lds_base_uniform) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base_uniform), "s"(lds_base_uniform)
               : "memory", "m0");
}

// The same from an address of each lane's own.
__device__ __forceinline__ void dma16_at(const unsigned char* from, unsigned lds_base_uniform) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(from), "s"(lds_base_uniform) : "memory", "m0");
}

// Wait until at most N of the wavefront's vector memory operations are outstanding.
template <int N>
__device__ __forceinline__ void wait_vm() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

}  // namespace kvfold
