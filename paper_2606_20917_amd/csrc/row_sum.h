// One row of the scatter-reduce (assembly.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

namespace nir {

constexpr int kScatterEntries = 4;   // entries of a scatter-reduce row read together

// Sum of CSR row g over its entries in ascending (element, mode) order.  A row is a chain of
// dependent reads (offsets, index, value) and holds one to eight entries on a mesh of hexahedra, so
// K entries go through every stage together: three memory latencies for a row of up to K.  Counted
// down from the row's length, as the array may reach the last int32 index.
template <class T>
__device__ __forceinline__ T row_sum(const int32_t* __restrict__ off, const int32_t* __restrict__ idx,
                                     const T* __restrict__ yl, int64_t g) {
  constexpr int K = kScatterEntries;
  const int32_t at = off[g];
  const int32_t* __restrict__ row = idx + at;
  T s = T(0);
  for (int32_t left = off[g + 1] - at; left > 0; left -= K, row += K) {
    int32_t n[K];
    T v[K];
#pragma unroll
    for (int i = 0; i < K; ++i) n[i] = i < left ? row[i] : -1;
#pragma unroll
    for (int i = 0; i < K; ++i) v[i] = n[i] >= 0 ? yl[n[i]] : T(0);
#pragma unroll
    for (int i = 0; i < K; ++i)
      if (n[i] >= 0) s += v[i];
  }
  return s;
}

}  // namespace nir
