// Direct transfers into LDS and addressing that keeps the compiler from forming 64-bit addresses per lane.
#pragma once

#include "common.hpp"

namespace maskkv {

// Direct global -> LDS transfer of 16 (4) bytes per lane from base + off to lds + lane * 16 (4).
__device__ __forceinline__ void dma16(const char* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(off), "s"(base), "s"(lds) : "memory");
}
// The same for what is read once: it passes through the caches without taking the place of what is kept there.
__device__ __forceinline__ void dma16_streamed(const char* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(off), "s"(base), "s"(lds) : "memory");
}
__device__ __forceinline__ void dma4(const char* base, uint32_t off, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" ::"v"(off), "s"(base), "s"(lds) : "memory");
}

// The same from an address of its own per lane.
__device__ __forceinline__ void dma16_from(const char* src, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(lds) : "memory");
}

// Global memory by a uniform base (two scalar registers, hidden from the optimiser, which would otherwise form one 64-bit
// address per lane and keep it) and a 32-bit offset per lane.
typedef __attribute__((address_space(1))) char* Base;
__device__ __forceinline__ Base base_of(const void* p) {
  Base b = (Base)p;
  asm volatile("" : "+s"(b));
  return b;
}
template <typename T>
__device__ __forceinline__ __attribute__((address_space(1))) T* at(Base b, uint32_t off, int imm = 0) {
  return reinterpret_cast<__attribute__((address_space(1))) T*>(b + off + imm);
}
// LDS by its own 32-bit address (the name of the array would be added to every lane's offset again and again).
template <typename T>
__device__ __forceinline__ __attribute__((address_space(3))) T* in_lds(uint32_t addr, int imm = 0) {
  return reinterpret_cast<__attribute__((address_space(3))) T*>((__attribute__((address_space(3))) char*)(uintptr_t)addr + imm);
}

}  // namespace maskkv
