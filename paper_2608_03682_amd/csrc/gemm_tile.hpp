// Device helpers shared by the GEMM kernels: global loads the compiler can
// count, direct global->LDS copies and the explicit waits that go with them.
#pragma once

#include "kernels.hpp"

namespace phyai {
namespace {

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) u32x4_t gu32x4_t;

// 16-, 8- and 2-byte loads through a global (not generic) pointer, which the
// compiler counts with vmcnt alone
__device__ __forceinline__ u32x4_t gload16(const void* p) { return *(gu32x4_t*)(p); }
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u32x2_t gload8(const void* p) {
  return *(const __attribute__((address_space(1))) u32x2_t*)(p);
}
__device__ __forceinline__ uint32_t gload2(const void* p) {
  return *(const __attribute__((address_space(1))) uint16_t*)(p);
}

typedef __attribute__((address_space(3))) void lds_void_t;

__device__ __forceinline__ void dma16(const void* src, lds_void_t* lds) {
  const uint32_t m = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(m), "v"(src) : "memory", "m0");
}
// A wave-uniform pointer as such: the compiler may keep a uniform value in
// vector registers, which an "s" operand does not accept.
__device__ __forceinline__ const uint8_t* uniform_ptr(const uint8_t* p) {
  const uint64_t v = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return reinterpret_cast<const uint8_t*>((uint64_t)hi << 32 | lo);
}
// the same with a wave-uniform base and a 32-bit byte offset per lane
__device__ __forceinline__ void dma16_off(const uint8_t* base, uint32_t off, lds_void_t* lds) {
  const uint32_t m = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(lds));
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(m), "v"(off), "s"(uniform_ptr(base)) : "memory", "m0");
}
__device__ __forceinline__ u32x4_t gload16_off(const uint8_t* base, uint32_t off) {
  return *(gu32x4_t*)((const __attribute__((address_space(1))) uint8_t*)base + off);
}
#define GEMM_WAIT_VMCNT(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | (((n) >> 4) << 14) | 0x70 | 0xF00)
__device__ __forceinline__ void bare_barrier() {
  __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0)
  __builtin_amdgcn_s_barrier();
}
__device__ __forceinline__ int aswz(int row) { return (row >> 1) & 7; }


}  // namespace
}  // namespace phyai
