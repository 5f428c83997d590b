// 16 x 16 tiles of the FP64 and FP32 matrix instructions.
//
// Operand layouts (checked on the device): lane l holds A[l%16][l/16] and B[l/16][l%16] in both
// v_mfma_f64_16x16x4f64 and v_mfma_f32_16x16x4f32; the four results of lane l are
// D[4v + l/16][l%16] (FP64) and D[4(l/16) + v][l%16] (FP32), v = 0..3.
#pragma once

#include <hip/hip_runtime.h>

namespace nir {

template <class T>
using dense_v4 = T __attribute__((ext_vector_type(4)));

template <class T>
__device__ __forceinline__ dense_v4<T> dense_mfma(T a, T b, dense_v4<T> c) {
  if constexpr (sizeof(T) == 8)
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
// row of result v of lane group lk (= l / 16) within a 16 x 16 tile
template <class T>
__device__ __forceinline__ int dense_drow(int v, int lk) {
  return sizeof(T) == 8 ? 4 * v + lk : 4 * lk + v;
}

constexpr int dense_ceil(int a, int b) { return (a + b - 1) / b; }

}  // namespace nir
