// FP32 matrix instructions and buffer accesses of the transform kernels.
//
// Lane l of a wavefront: m = l & 15, q = l >> 4.  An instruction takes A[row m][term q] and
// B[term q][column m] from lane l and adds to D[row 4 q + i][column m], i = 0..3, in lane l.
// The terms of a contraction may be taken in any order as long as A and B agree, so each lane
// loads runs of consecutive terms.  Terms, rows and columns past an axis read 0 (addresses past
// the end of a buffer resource) or meet a 0 on the other side.
#pragma once

#include "bl_internal.h"

namespace bl {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef __amdgpu_buffer_rsrc_t Rsrc;
constexpr uint32_t kPast = 0xFFFFFFF0u;   // past every buffer (all smaller than this)

__device__ __forceinline__ Rsrc rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), (short)0, (int)bytes, 0x00020000);
}
__device__ __forceinline__ f4 ld4(Rsrc r, uint32_t off) {
  return __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}
__device__ __forceinline__ float ld1(Rsrc r, uint32_t off) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)off, 0, 0));
}
__device__ __forceinline__ f2 ld2(Rsrc r, uint32_t off) {
  return __builtin_bit_cast(f2, __builtin_amdgcn_raw_buffer_load_b64(r, (int)off, 0, 0));
}
typedef uint32_t u2 __attribute__((ext_vector_type(2)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ void st1(Rsrc r, uint32_t off, float v) {
  __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, v), r, (int)off, 0, 0);
}
__device__ __forceinline__ void st2(Rsrc r, uint32_t off, f2 v) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2, v), r, (int)off, 0, 0);
}
__device__ __forceinline__ void st4(Rsrc r, uint32_t off, f4 v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, v), r, (int)off, 0, 0);
}
__device__ __forceinline__ f4 mfma(float a, float b, f4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ __forceinline__ int wave_of(int tid) { return __builtin_amdgcn_readfirstlane(tid >> 6); }

}  // namespace
}  // namespace bl
