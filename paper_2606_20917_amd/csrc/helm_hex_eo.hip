// Fused Helmholtz apply on hexahedra with even-odd folded 1-D contractions: the register-pencil
// kernel of helm_hex.hip (sweeps A, B, C, pointwise, C^T, B^T, A^T; paper section 2.2,
// eqs. (16), (20)) with every contraction over point pairs (i, Q-1-i), about half the
// multiply-adds; the point loop runs one pair ahead on its geometric factors.

#include "helm_hex_eo_dev.h"

namespace nir {

// SF: the block's factors staged through LDS, requested all at once (FP32 at P <= 4 on
// per-point factors, where it measured 4-11 % faster; in FP64 it measured slower)
template <int P, class T, bool DEF>
constexpr bool eo_staged_factors() {
  return DEF && sizeof(T) == 4 && P <= 4;
}

template <int P, class T, bool DEF, int E, bool TP, bool MAP, bool SF = eo_staged_factors<P, T, DEF>() && !TP>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(hex_waves_target<P, T, E, TP>())))
k_helm_hex_eo(const T* __restrict__ tabs, const T* __restrict__ x, T* __restrict__ y, const T* __restrict__ helm,
              const T* __restrict__ wq, T lambda, int64_t nelmt, const int32_t* __restrict__ map) {
  using D = HexPencilDims<P, T, E, TP>;
  __shared__ T lds[D::LDS + (SF ? E * 7 * D::NQ + D::BLOCK : 0)];
  helm_hex_eo_group<P, T, DEF, E, TP, true, 1, false, SF, MAP>(
      tabs, x, y, helm, wq, lambda, nelmt, int64_t(blockIdx.x) * E, lds, nullptr, nullptr, nullptr, map);
}

// Elements per block on per-element factors, where the sweeps and their barriers bound the kernel:
// one element at P = 7, whose 64 pencils are one wavefront (32^3 hexes, blocks of 4 -> 1: FP64 121
// -> 100 us, FP32 69 -> 57 us), and at P = 9 and 10 (FP64 P = 10, blocks of 2 -> 1: 478 -> 436 us);
// otherwise near 128 pencils (P = 4, 10 -> 5 elements: FP64 26.7 -> 24.8 us) or all that fit
template <int P>
constexpr int eo_affine_elems() {
  return P == 7 || P >= 9 ? 1 : (P == 3 ? 4 : (P == 4 ? 5 : (P == 5 ? 3 : 256 / ((P + 1) * (P + 1)))));
}

// Counts of affine elements at which all that fit in a block (P = 5: 7 elements, P = 9 and 10: 2) run in
// fewer rounds of the 256 CUs than the blocks above: one block of 2 a CU against two of 1 to 512, three of
// 2 against five of 1 to 1,536 (us, blocks above -> these: FP64 at 400 elements, P = 9, 10: 10.0 -> 9.2,
// 12.1 -> 11.3; at 1,455, P = 10: 25.8 -> 22.1, in FP32 15.1 -> 13.9; at 3,552, P = 9 in FP32 21.1 -> 19.6),
// four of 7 against eight of 3 to 7,168 (6,938 at P = 5 in FP64 12.5 -> 11.5)
template <int P, class T>
constexpr bool eo_affine_wide(int64_t n) {
  constexpr bool F64 = sizeof(T) == 8;
  if (P == 5) return F64 && n > 6144 && n <= 7168;
  if (P == 9) return (n > 256 && n <= 512) || (!F64 && n > 1280 && n <= 5120);
  if (P == 10) return (F64 && n > 256 && n <= 512) || (n > 1280 && n <= 1536);
  return false;
}

template <int P, class T, bool DEF, bool TP, bool WIDE = false>
static void launch_eo_cfg(const T* tb, const T* x, T* y, const T* helm, const T* wq, T lam, int64_t nelmt,
                          const int32_t* map, hipStream_t s) {
  if constexpr (!DEF && !TP && !WIDE && ((P == 5 && sizeof(T) == 8) || P >= 9))
    if (eo_affine_wide<P, T>(nelmt)) return launch_eo_cfg<P, T, DEF, TP, true>(tb, x, y, helm, wq, lam, nelmt, map, s);
  constexpr int E = DEF    ? hex_block_elems<P, T>(TP ? kFamEOS : kFamEO)
                    : WIDE ? 256 / ((P + 1) * (P + 1)) : eo_affine_elems<P>();
  using D = HexPencilDims<P, T, E, TP>;
  const int64_t nb = (nelmt + E - 1) / E;
  const dim3 grid(static_cast<unsigned>(nb)), block(D::BLOCK);
  // a kernel each, as in helm_hex.hip; affine elements always run the one with the branch, the faster
  // code for them (FP32 at P = 4 and 7, 100 to 900 elements 4-7 %, FP64 at P = 3 8 %)
  if (!DEF || map)
    hipLaunchKernelGGL((k_helm_hex_eo<P, T, DEF, E, TP, true>), grid, block, 0, s, tb, x, y, helm, wq, lam, nelmt, map);
  else if constexpr (DEF)
    hipLaunchKernelGGL((k_helm_hex_eo<P, T, DEF, E, TP, false>), grid, block, 0, s, tb, x, y, helm, wq, lam, nelmt, map);
}

template <int P, class T>
static nir_status launch_eo_P(const nir_basis* b, int deformed, bool split, const OpArgs& a, hipStream_t s) {
  const T* tb = sizeof(T) == 8 ? reinterpret_cast<const T*>(b->eo64) : reinterpret_cast<const T*>(b->eo32);
  if (!tb) return fail(NIR_ENOTSUP, "the folded basis rows need a hexahedral basis with Q = P + 1");
  if (a.nelmt > 0x7fffffff) return fail(NIR_EINVAL, "too many elements for one launch");
  const T* wq = sizeof(T) == 8 ? reinterpret_cast<const T*>(b->t64.wq) : reinterpret_cast<const T*>(b->t32.wq);
  const T* x = static_cast<const T*>(a.in0);
  T* y = static_cast<T*>(a.out0);
  const T* helm = static_cast<const T*>(a.helm);
  const T lam = T(a.lambda);
  if (deformed) {
    if (split)
      launch_eo_cfg<P, T, true, true>(tb, x, y, helm, wq, lam, a.nelmt, a.map, s);
    else
      launch_eo_cfg<P, T, true, false>(tb, x, y, helm, wq, lam, a.nelmt, a.map, s);
  } else {
    if (split)
      launch_eo_cfg<P, T, false, true>(tb, x, y, helm, wq, lam, a.nelmt, a.map, s);
    else
      launch_eo_cfg<P, T, false, false>(tb, x, y, helm, wq, lam, a.nelmt, a.map, s);
  }
  return hip_check(hipGetLastError(), "hex even-odd Helmholtz launch");
}

nir_status launch_helm_hex_eo(const nir_basis* b, int dtype, int deformed, const OpArgs& a, hipStream_t s,
                              bool split) {
#define NIR_CASE(PP)                                                                   \
  case PP:                                                                             \
    return dtype == NIR_F64 ? launch_eo_P<PP, double>(b, deformed, split, a, s)         \
                            : launch_eo_P<PP, float>(b, deformed, split, a, s);
  switch (b->P) {
    NIR_CASE(2) NIR_CASE(3) NIR_CASE(4) NIR_CASE(5) NIR_CASE(6)
    NIR_CASE(7) NIR_CASE(8) NIR_CASE(9) NIR_CASE(10)
    default: return fail(NIR_ENOTSUP, "P=%d not compiled", b->P);
  }
#undef NIR_CASE
}

}  // namespace nir
