// 1-D contractions of the modified basis over the Gauss-Lobatto-Legendre points, folded by even-odd
// symmetry.
//
// The Gauss-Lobatto-Legendre points are symmetric, z_{Q-1-i} = -z_i, and the modified C0
// basis of section 2.2 maps onto itself under the reflection z -> -z: the two vertex modes
// swap, psi_0(-z) = psi_1(z), and an interior mode p >= 2 (a bubble times P^{1,1}_{p-2}) has
// parity (-1)^p; derivatives take the opposite parity.  So a 1-D contraction over a point pair
// (i, Q-1-i) needs only half of the mode sums:
//   modes -> points:  e = (c0+c1, c2, c4, ...),  o = (c0-c1, c3, c5, ...)
//                     S = BE(i).e,  A = BO(i).o:  v_i = S + A,  v_{Q-1-i} = S - A
//                     (derivative: SD = DO(i).o, AD = DE(i).e, d_i = SD + AD, d_{Q-1-i} = SD - AD)
//   points -> modes:  s_i = v_i + v_{Q-1-i},  a_i = v_i - v_{Q-1-i}
//                     E += BE(i) s + DE(i) a_w,  O += BO(i) a + DO(i) s_w
//                     c0 = E0 + O0, c1 = E0 - O0, c_{2k} = E_k, c_{2k+1} = O_k
// with folded table rows (i = 0 .. ceil(Q/2)-1, 2P values each):
//   BE(i) = ((B_i0 + B_i1)/2, B_i2, B_i4, ...),  BO(i) = ((B_i0 - B_i1)/2, B_i3, B_i5, ...)
//   DE(i) = ((D_i0 + D_i1)/2, D_i2, D_i4, ...),  DO(i) = ((D_i0 - D_i1)/2, D_i3, D_i5, ...)
// For odd Q the middle point pairs with itself: its BO and DE entries vanish (stored as exact
// zeros), it takes v = S, d = SD, and contributes once to the transposed sums.
// Each contraction costs ceil(Q/2) * P multiply-adds instead of Q * P.
#pragma once

#include "nir_internal.h"
#include "uniform_table.h"

namespace nir {

template <int P>
struct EoDims {
  static constexpr int Q = P + 1;
  static constexpr int H = (Q + 1) / 2;        // folded rows (point pairs, middle included)
  static constexpr int NE = 1 + (P - 1) / 2;   // even group: c0+c1 and the even interior modes
  static constexpr int NO = P - NE;            // odd group: c0-c1 and the odd interior modes
  static constexpr bool MID = (Q & 1) != 0;    // a middle point z = 0
  static constexpr int ROW = 2 * P;            // values per folded row
};

// one folded row through a fresh pointer (see fresh_table)
template <int P, class T>
struct HexTabEO {
  static constexpr int NE = EoDims<P>::NE;
  const_ptr<T> t;
  __device__ __forceinline__ T BE(int k) const { return t[k]; }
  __device__ __forceinline__ T BO(int k) const { return t[NE + k]; }
  __device__ __forceinline__ T DE(int k) const { return t[P + k]; }
  __device__ __forceinline__ T DO(int k) const { return t[P + NE + k]; }
};

template <int P, class T>
__device__ __forceinline__ void eo_fold(const T* c, T* ev, T* od) {
  ev[0] = c[0] + c[1];
  od[0] = c[0] - c[1];
#pragma unroll
  for (int k = 1; k < EoDims<P>::NE; ++k) ev[k] = c[2 * k];
#pragma unroll
  for (int k = 1; k < EoDims<P>::NO; ++k) od[k] = c[2 * k + 1];
}

template <int P, class T>
__device__ __forceinline__ void eo_unfold(const T* ev, const T* od, T* c) {
  c[0] = ev[0] + od[0];
  c[1] = ev[0] - od[0];
#pragma unroll
  for (int k = 1; k < EoDims<P>::NE; ++k) c[2 * k] = ev[k];
#pragma unroll
  for (int k = 1; k < EoDims<P>::NO; ++k) c[2 * k + 1] = od[k];
}

// modes -> the point pair of one folded row: value (S +- A) and derivative (SD +- AD).  `mid`
// (a constant after unrolling) skips the half that vanishes on the middle row.
template <int P, class T>
__device__ __forceinline__ void eo_val(const HexTabEO<P, T>& tk, const T* ev, const T* od, T& S, T& A,
                                       bool mid = false) {
  S = T(0);
  A = T(0);
#pragma unroll
  for (int k = 0; k < EoDims<P>::NE; ++k) S += tk.BE(k) * ev[k];
  if (!mid) {
#pragma unroll
    for (int k = 0; k < EoDims<P>::NO; ++k) A += tk.BO(k) * od[k];
  }
}

template <int P, class T>
__device__ __forceinline__ void eo_der(const HexTabEO<P, T>& tk, const T* ev, const T* od, T& SD, T& AD,
                                       bool mid = false) {
  SD = T(0);
  AD = T(0);
#pragma unroll
  for (int k = 0; k < EoDims<P>::NO; ++k) SD += tk.DO(k) * od[k];
  if (!mid) {
#pragma unroll
    for (int k = 0; k < EoDims<P>::NE; ++k) AD += tk.DE(k) * ev[k];
  }
}

// points -> modes, one folded row: E += BE s, O += BO a (values) and E += DE a, O += DO s
// (derivative test functions); on the middle row a = 0 and that half is skipped
template <int P, class T>
__device__ __forceinline__ void eo_tval(const HexTabEO<P, T>& tk, T s, T a, T* E, T* O, bool mid = false) {
#pragma unroll
  for (int k = 0; k < EoDims<P>::NE; ++k) E[k] += tk.BE(k) * s;
  if (!mid) {
#pragma unroll
    for (int k = 0; k < EoDims<P>::NO; ++k) O[k] += tk.BO(k) * a;
  }
}

template <int P, class T>
__device__ __forceinline__ void eo_tder(const HexTabEO<P, T>& tk, T s, T a, T* E, T* O, bool mid = false) {
  if (!mid) {
#pragma unroll
    for (int k = 0; k < EoDims<P>::NE; ++k) E[k] += tk.DE(k) * a;
  }
#pragma unroll
  for (int k = 0; k < EoDims<P>::NO; ++k) O[k] += tk.DO(k) * s;
}

// the point pair (h, Q-1-h) of a pencil folded into sum and difference (the middle point alone)
template <int P, class T>
__device__ __forceinline__ void eo_pair(const T* v, int h, bool mid, T& sv, T& av) {
  sv = mid ? v[h] : v[h] + v[P - h];
  av = mid ? T(0) : v[h] - v[P - h];
}

}  // namespace nir
