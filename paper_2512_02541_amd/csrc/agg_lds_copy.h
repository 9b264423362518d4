// Device helpers for tiles that go global -> LDS without passing through registers: the copy
// instruction, the wait for it and the barrier that goes with it.  Used by the attention and the
// projection kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace agg {

typedef __attribute__((address_space(3))) char lds_char;

// Workgroup barrier that orders LDS traffic only: global loads issued for a later tile
// stay in flight across it.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Asynchronous copy global -> LDS without passing through registers: lane i of the wavefront
// lands the 16 bytes at `base + voff(i)` at LDS address m0 + 16 i.  Written as assembly so that
// the compiler's wait-count pass does not serialise later LDS reads of OTHER buffers behind this
// copy; the loop waits for it explicitly before the barrier.  M0 is a register the compiler
// reserves and sets right before each of its own uses; the kernels that use this have none (a build test
// checks that no compiler-emitted instruction of them reads M0).
__device__ __forceinline__ void dma16(const void* base, uint32_t voff, uint32_t m0) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"
               :
               : "v"(voff), "s"(base), "s"(m0)
               : "memory");
}
// a pointer every lane agrees on, as two scalar registers (what the copy's base operand needs)
__device__ __forceinline__ const uint16_t* uniform_ptr(const uint16_t* q) {
  const uint64_t v = (uint64_t)(uintptr_t)q;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (const uint16_t*)(uintptr_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ void wait_vm0() { __builtin_amdgcn_s_waitcnt(0x0F70); }  // vmcnt(0) only
// all but this wavefront's kLeft youngest copies, loads and stores are done
template <int kLeft>
__device__ __forceinline__ void wait_vm() {
  static_assert(kLeft >= 0 && kLeft < 64, "six counter bits: 3..0 and 15..14 of the operand");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (kLeft & 15) | ((kLeft >> 4) << 14));
}

}  // namespace agg
