// bf16 conversions and the vector types of the bf16 MFMA kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace ccut {

typedef float float4v __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// fp32 -> bf16, round to nearest even (NaN kept quiet)
__device__ inline uint16_t f2bf(float x) {
  uint32_t u = __float_as_uint(x);
  if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x7FFFFFu)) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
// two at once, by the hardware's conversion (the same value for every x but NaN)
__device__ inline uint32_t f2bf2(float x0, float x1) {
  typedef float float2v __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((float2v{x0, x1}), bf16x2));
}
__device__ inline float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// D = A B + C, v_mfma_f32_16x16x32_bf16: lane l supplies A[row l % 16]
// [k 8 (l / 16) + i] and B[k 8 (l / 16) + i][col l % 16] for i < 8;
// accumulator register g holds D[row 4 (l / 16) + g][col l % 16].  Its result
// has the bits of two chained 16x16x16 products over k 0..15 and k 16..31
// (compared on gfx950 over 512000 elements of mixed magnitudes), and swapping
// the operands gives the transpose's bits.
__device__ inline float4v mfma_bf16(u32x4 a, u32x4 b, float4v c) {
  typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0,
                                                 0);
}

// Position of element (n, k) of an N x K weight in lane order: per 16 columns
// n and 32 inner indices k one 1 KB block, lane l's 16 bytes its eight k.
__host__ __device__ inline uint32_t lane_order(uint32_t n, uint32_t k, uint32_t K) {
  return (((n >> 4) * (K >> 5) + (k >> 5)) * 64 + ((k >> 3) & 3u) * 16 + (n & 15u)) * 8 + (k & 7u);
}

}  // namespace ccut
