// Requests that move memory straight into LDS, and the waits and barriers that go with them.
#pragma once
#include "mfma_kernels.h"

namespace alora {

typedef int32_t i32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void wave_barrier() { asm volatile("s_barrier" ::: "memory"); }
template <int N> __device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// 64 lanes x 16 bytes from rsrc[voff + soff] to LDS bytes lds .. lds + 1023, lane after lane; lanes whose offset is out of the
// resource's range write zeros.  Inline assembly: the compiler would make every later LDS read wait for all of these.  (m0 is a
// reserved register, in which the compiler keeps no value from one instruction to another: it takes it for no clobber.)
__device__ __forceinline__ void load_to_lds(i32x4 rsrc, int voff, int soff, int lds) {
  lds = __builtin_amdgcn_readfirstlane(lds);      // (no instruction where the compiler has it in a scalar register already)
  soff = __builtin_amdgcn_readfirstlane(soff);
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(voff), "s"(rsrc), "s"(soff)
               : "memory");
}
__device__ __forceinline__ i32x4 make_rsrc(const void *p, uint64_t bytes) {
  const uint64_t a = (uint64_t)p;
  i32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
  r[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32) & 0xffff);
  r[2] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(bytes > 0xffffffffull ? 0xffffffffull : bytes));
  r[3] = 0x00020000;
  return r;
}

// Requests to LDS want 16-byte addresses (ordinary loads do not care): weights that lie otherwise take the kernels without them.
inline bool lds_aligned(const void *p) { return ((uintptr_t)p & 15) == 0; }

// One rotation pair (u, w) = columns c and c + h/2 of a head (Eq.3's K_t before it is appended), the sums and products in one
// fixed form: the rows that different kernels append are compared bit for bit.
__device__ __forceinline__ float rope_lo(float u, float w, float cs, float sn) { return __builtin_fmaf(u, cs, -(w * sn)); }
__device__ __forceinline__ float rope_hi(float u, float w, float cs, float sn) { return __builtin_fmaf(w, cs, u * sn); }

}  // namespace alora
