// Copies from global memory straight into LDS (gfx950: 16 bytes per lane, no registers in between).  They count as
// vector loads in order; a kernel that uses them waits by their number.
#pragma once
#include "common.h"

namespace rlx {

// One copy of 64 x 16 bytes: lane i's 16 bytes at `g` -> LDS address lds + 16 i.  The wait state between the write of
// m0 and its use is the assembler's to place, hence the s_nop.  No register is written by the copy.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"   // m0 as a clobber: "reserved register"
__device__ __forceinline__ void copy_to_lds(const void* g, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds), "v"(g) : "memory", "m0");
}
// The same from a uniform address plus a 32-bit lane offset.
__device__ __forceinline__ void copy_to_lds(const void* base, uint32_t offset, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(offset), "s"(base) : "memory", "m0");
}
// ... for data that the launch reads once (load_stream_16)
__device__ __forceinline__ void copy_to_lds_stream(const void* base, uint32_t offset, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds), "v"(offset), "s"(base) : "memory", "m0");
}
#pragma clang diagnostic pop
// Waits until at most N of this wave's copies are in flight and its LDS reads are done, then for the other waves.
template <int N>
__device__ __forceinline__ void wait_copies_and_barrier() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// LDS address of a shared array, as the copies take it
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const unsigned char*)p;
}

}  // namespace rlx
