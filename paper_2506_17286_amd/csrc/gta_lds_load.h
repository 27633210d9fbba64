// Loads from memory straight into LDS: 16 bytes per lane from rsrc + voff (+ soff) to LDS offset lds + 16 * lane.  vmcnt
// counts them; the compiler does not know that, so every wait for these loads is spelled out.  (M0 holds nothing the
// compiler keeps.)
#pragma once
#include <hip/hip_runtime.h>

namespace gta {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ void load_to_lds(u32x4 rsrc, unsigned voff, unsigned soff, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(voff), "s"(rsrc), "s"(soff));
}
__device__ __forceinline__ void load_to_lds(u32x4 rsrc, unsigned voff, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds), "v"(voff), "s"(rsrc));
}

// Buffer of `bytes` at `base`: reads past its end return 0.  Both have to be wave-uniform.
__device__ __forceinline__ u32x4 buffer_of(const void *base, unsigned bytes) {
  const uint64_t b = (uint64_t)base;
  return u32x4{(unsigned)b, (unsigned)(b >> 32) & 0xffffu, bytes, 0x00020000u};
}
// the same where the compiler does not see that they are
__device__ __forceinline__ u32x4 uniform_buffer_of(const void *base, unsigned bytes) {
  const u32x4 b = buffer_of(base, bytes);
  return u32x4{(unsigned)__builtin_amdgcn_readfirstlane((int)b[0]), (unsigned)__builtin_amdgcn_readfirstlane((int)b[1]),
               (unsigned)__builtin_amdgcn_readfirstlane((int)b[2]), b[3]};
}

}  // namespace gta
