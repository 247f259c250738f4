// Device-side pieces shared by the kernels that load tiles straight into LDS: buffer descriptors, the load itself and
// the matrix instructions.
#pragma once
#include <hip/hip_runtime.h>

namespace spc {
namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

// c += a . b over the 64 bytes (4 x 16 per row or column) that the four lane groups hold
template <typename T> __device__ __forceinline__ f32x4 mma(u32x4 a, u32x4 b, f32x4 c);
template <> __device__ __forceinline__ f32x4 mma<_Float16>(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
}
template <> __device__ __forceinline__ f32x4 mma<__bf16>(u32x4 a, u32x4 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
template <> __device__ __forceinline__ f32x4 mma<float>(u32x4 a, u32x4 b, f32x4 c) {
  // 16x16x4: lane group g multiplies its i-th element, reduction channel 4 g + i of the 16
  const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
#pragma unroll
  for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_16x16x4f32(x[i], y[i], c, 0, 0, 0);
  return c;
}

__device__ __forceinline__ u32x4 rsrc_of(const void* base, unsigned bytes) {
  const unsigned long long a = (unsigned long long)base;
  return u32x4{(unsigned)a, (unsigned)(a >> 32), bytes, 0x00020000u};
}
// 64 lanes x 16 bytes from a buffer into LDS: lane l fills lds + 16 l, zeros where its offset is out of range.
// (The five wait states that a vector-memory instruction needs behind a vector instruction that writes one of
// its scalar registers are part of it.  m0 is a reserved register, which clobber lists do not take; no instruction that
// is generated for these kernels uses it: LDS accesses need it up to gfx8 only.)
__device__ __forceinline__ void load_to_lds(u32x4 rsrc, unsigned voff, unsigned soff, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" ::"s"(lds), "v"(voff), "s"(rsrc),
               "s"(soff)
               : "memory");
}
// The same with 4 bytes per lane: lane l fills lds + 4 l.
__device__ __forceinline__ void load_dword_to_lds(u32x4 rsrc, unsigned voff, unsigned lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 4\n\tbuffer_load_dword %1, %2, 0 offen lds" ::"s"(lds), "v"(voff), "s"(rsrc) : "memory");
}
// Own loads have landed and own LDS reads are done.
__device__ __forceinline__ void wait_own_loads() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory"); }
// Own loads but the N youngest have landed and own LDS reads are done; after the barrier everyone's.
template <int N = 0> __device__ __forceinline__ void wait_loads_and_sync() {
  static_assert(N < 64, "vmcnt");
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"i"(N) : "memory");
}
// Own LDS reads are done; after the barrier everyone's.
__device__ __forceinline__ void sync_lds() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

}  // namespace
}  // namespace spc
