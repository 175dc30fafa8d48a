// What the matrix-core kernels that take any shape share: loads through a bounds-checked buffer descriptor straight
// into LDS.
#pragma once

#include "kernels.h"

namespace po {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));

// Byte address of a pointer into the block's LDS as the hardware counts it (the generic -> LDS conversion and its null
// check happen here, once, instead of at every load).
__device__ __forceinline__ unsigned lds_byte(const void* p) {
  return (unsigned)(size_t)((const void __attribute__((address_space(3)))*)p);
}

// Buffer descriptor of `bytes` bytes at p: a load whose offset reaches past the end returns zero instead of touching
// memory, which is how rows and k-indices beyond the edge of an operand become zeros without a branch.  p and bytes
// must be the same in every lane.
__device__ __forceinline__ i32x4 buffer_of(const void* p, unsigned bytes) {
  uint64_t a = (uint64_t)(size_t)p;
  i32x4 r;
  r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
  r[1] = __builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32) & 0xffff);
  r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
  r[3] = 0x00020000;
  return r;
}
constexpr unsigned kOutOfBuffer = 0xfffffff0u;  // an offset no buffer reaches

// One wave-wide load of 1 KiB: lane L's 16 bytes at `offset` of the buffer land in LDS at lds_base + 16 L.  Inline
// assembly because the compiler would wait for the load before every later LDS read; the caller waits itself.
__device__ __forceinline__ void buffer_to_lds(unsigned lds_base, unsigned offset, i32x4 buffer) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds_base), "v"(offset),
               "s"(buffer)
               : "memory");
}

// Waits until at most N of this wave's loads are outstanding (they complete in issue order).
template <int N>
__device__ __forceinline__ void wait_loads() {
  static_assert(N < 64, "the counter has six bits");
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
__device__ __forceinline__ void wait_lds_reads() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// Whether one of this lane's results is an infinity or NaN.
template <int N>
__device__ __forceinline__ bool not_finite(const f32x16 (&acc)[N]) {
  float z = 0.f;
#pragma unroll
  for (int d = 0; d < N; ++d)
#pragma unroll
    for (int e = 0; e < 16; ++e) z = fmaf(acc[d][e], 0.f, z);
  return !(z == 0.f);
}

}  // namespace po
