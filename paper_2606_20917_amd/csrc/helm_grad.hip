// Fused Helmholtz apply of affine tetrahedra through the gradient in an orthonormal basis, on the
// FP64 or FP32 matrix cores.
//
// With per-element factors the operator of eqs. (6), (7) needs no quadrature per element: the
// reference gradient of a mode lies in the polynomials of degree P - 2, so with D_a the
// coefficients of d phi / d xi_a in an orthonormal basis of that space (G = (P-1)P(P+1)/6
// functions, weighted by the rule's weights; the rule integrates the products exactly)
//   y_e = sum_a D_a^T (sum_b g_ab D_b x_e) + lambda g_6 M x_e,   M = B^T W B.
// Elements are the rows of three stacked GEMMs: T = X [D_0^T | D_1^T | D_2^T] and X M (K = M modes),
// then Y = sum_a F_a D_a with F_a = sum_b g_ab T_b (K = 3 G).  That is 6 M G + M^2 multiply-adds an
// element against the 7 M^2 of the seven stacked reference matrices (helm_dense.hip): 0.73 of them
// at P = 8.
//
// What bounds it: the matrix cores (an FP64 tile step of 2048 operations takes 64 cycles), so a block
// keeps all of T of its elements in LDS, in the place of their coefficients, and runs three
// phases without a barrier inside: coefficients -> T and X M in registers, T to LDS, T -> Y.  The A
// operand F is formed from LDS as it is read (nine multiply-adds for the operands of 3 CT2 tile
// steps); B operands come from L2 two steps ahead.  Half of the steps multiply zeros: the basis is
// orthonormal, so D_a is sparse (of its 4 x 16 blocks at P = 8 those with a nonzero are 210 of 480 in the
// first GEMM and 208 of 504 in the third, of the mass matrix 183 of 240), and the K loops run over all.
#include <cmath>
#include <type_traits>
#include <vector>

#include "mfma_tile.h"
#include "nir_internal.h"

namespace nir {

// NW wavefronts a block in a WR x WC grid over row tiles (RTW each) and column tiles
template <int P, class T, int NW_, int WC_, int RTW_>
struct GradDims {
  static constexpr int M = P * (P + 1) * (P + 2) / 6, G = (P - 1) * P * (P + 1) / 6;
  static constexpr int MK = (M + 3) / 4 * 4;              // K of the first two GEMMs
  static constexpr int NG = (G + 3) / 4;                  // groups of 4 gradient functions: K = 12 NG of the third
  static constexpr int NT1 = dense_ceil(3 * G, 16), N1P = NT1 * 16;
  static constexpr int NCT = dense_ceil(M, 16), MP = NCT * 16;
  static constexpr int NW = NW_, WC = WC_, WR = NW / WC, BLOCK = 64 * NW;
  static constexpr int RTW = RTW_, RT = RTW * WR, ROWS = 16 * RT;
  static constexpr int CT1 = dense_ceil(NT1, WC), CT2 = dense_ceil(NCT, WC);
  static constexpr int XSTR = MK + 1, TSTR = (3 * G) | 1; // odd LDS row strides
  static constexpr int LDS = ROWS * (XSTR > TSTR ? XSTR : TSTR);
};

// B1 [MK][N1P]: column a G + g of row m is D_a[g][m]; Mm [MP][MP]: the mass matrix;
// B2 [12 NG][MP]: row (3 k + a) 4 + i is D_a[4 k + i][.]; all zero-padded
template <int P, class T, int NW, int WC_, int RTW_, int PD>
__global__ void __launch_bounds__(64 * NW) k_helm_grad(const T* __restrict__ B1, const T* __restrict__ Mm,
                                                   const T* __restrict__ B2, const T* __restrict__ x,
                                                   T* __restrict__ y, const T* __restrict__ helm, T lambda,
                                                   int64_t nelmt) {
  using D = GradDims<P, T, NW, WC_, RTW_>;
  constexpr int M = D::M, G = D::G, MK = D::MK, MP = D::MP, N1P = D::N1P, NT1 = D::NT1, NCT = D::NCT, RTW = D::RTW,
                CT1 = D::CT1, CT2 = D::CT2, WC = D::WC, XSTR = D::XSTR, TSTR = D::TSTR, ROWS = D::ROWS;
  __shared__ T lds[D::LDS];
  const int64_t e0 = int64_t(blockIdx.x) * ROWS;
  const int ne = int(min(int64_t(ROWS), nelmt - e0));
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
  const int li = l & 15, lk = l >> 4;
  const int wr = w / WC, wc = w - wr * WC;   // row tiles wr RTW ..; column tiles wc + WC u

  // B operands of one K step: this wave's column tiles of row k + lk (tiles past the end repeat the
  // last one; their results are not used)
  auto load_b = [&](const T* __restrict__ B, int stride, int nt, int k, auto& b, auto ctc) {
    constexpr int CT = decltype(ctc)::value;
    const T* __restrict__ r = B + int64_t(k + lk) * stride + li;
#pragma unroll
    for (int u = 0; u < CT; ++u) b[u] = r[min(wc + WC * u, nt - 1) * 16];
  };
  using C1 = std::integral_constant<int, CT1>;
  using C2 = std::integral_constant<int, CT2>;
  // PD (1 or 2) K steps ahead: the operands of step k are copied out before those of step k + PD
  // are requested into their place
  T b1[PD][CT1], b2[PD][CT2];
  auto load_1 = [&](int k, int i) {
    load_b(B1, N1P, NT1, k, b1[i], C1{});
    load_b(Mm, MP, NCT, k, b2[i], C2{});
  };
  load_1(0, 0);
  if constexpr (PD == 2 && MK > 4) load_1(4, 1);
  // the block's coefficients, zero-padded to MK columns and ROWS rows
#pragma unroll 8
  for (int f = threadIdx.x; f < ROWS * MK; f += D::BLOCK) {
    const int r = f / MK, m = f - r * MK;
    lds[r * XSTR + m] = (r < ne && m < M) ? x[(e0 + r) * M + m] : T(0);
  }
  __syncthreads();

  // ---- T = X [D_0^T | D_1^T | D_2^T] and X M
  dense_v4<T> t1[RTW][CT1], acc[RTW][CT2];
#pragma unroll
  for (int t = 0; t < RTW; ++t) {
#pragma unroll
    for (int u = 0; u < CT1; ++u) t1[t][u] = dense_v4<T>{T(0), T(0), T(0), T(0)};
#pragma unroll
    for (int u = 0; u < CT2; ++u) acc[t][u] = dense_v4<T>{T(0), T(0), T(0), T(0)};
  }
  T xn[RTW];
  auto load_x = [&](int k) {
#pragma unroll
    for (int t = 0; t < RTW; ++t) xn[t] = lds[((wr * RTW + t) * 16 + li) * XSTR + k + lk];
  };
  auto step_1 = [&](int k, int i) {
    T xa[RTW], c1[CT1], c2[CT2];
#pragma unroll
    for (int t = 0; t < RTW; ++t) xa[t] = xn[t];
#pragma unroll
    for (int u = 0; u < CT1; ++u) c1[u] = b1[i][u];
#pragma unroll
    for (int u = 0; u < CT2; ++u) c2[u] = b2[i][u];
    if (k + 4 * PD < MK) load_1(k + 4 * PD, i);
    if (k + 4 < MK) load_x(k + 4);
#pragma unroll
    for (int t = 0; t < RTW; ++t) {
#pragma unroll
      for (int u = 0; u < CT1; ++u) t1[t][u] = dense_mfma<T>(xa[t], c1[u], t1[t][u]);
#pragma unroll
      for (int u = 0; u < CT2; ++u) acc[t][u] = dense_mfma<T>(xa[t], c2[u], acc[t][u]);
    }
  };
  load_x(0);
#pragma unroll 1
  for (int m0 = 0; m0 + 4 * (PD - 1) < MK; m0 += 4 * PD) {
    step_1(m0, 0);
    if constexpr (PD == 2) step_1(m0 + 4, 1);
  }
  if constexpr (PD == 2 && MK % 8 == 4) step_1(MK - 4, 0);
  T bn[PD][3][CT2];
  auto load_2 = [&](int k, int i) {
#pragma unroll
    for (int a = 0; a < 3; ++a) load_b(B2, MP, NCT, (3 * k + a) * 4, bn[i][a], C2{});
  };
  load_2(0, 0);
  if constexpr (PD == 2 && D::NG > 1) load_2(1, 1);
  // factors of this lane's A rows, and the mass factor of its result rows (rows past the batch end
  // read element e0's; they are not stored)
  T g[RTW][6];
#pragma unroll
  for (int t = 0; t < RTW; ++t) {
    const int ra = (wr * RTW + t) * 16 + li;
#pragma unroll
    for (int c = 0; c < 6; ++c) g[t][c] = helm[(e0 + (ra < ne ? ra : 0)) * 7 + c];
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int r = (wr * RTW + t) * 16 + dense_drow<T>(v, lk);
      const T gm = lambda * helm[(e0 + (r < ne ? r : 0)) * 7 + 6];
#pragma unroll
      for (int u = 0; u < CT2; ++u) acc[t][u][v] *= gm;
    }
  }
  __syncthreads();   // the coefficients are read
#pragma unroll
  for (int t = 0; t < RTW; ++t)
#pragma unroll
    for (int u = 0; u < CT1; ++u) {
      const int n = (wc + WC * u) * 16 + li;
#pragma unroll
      for (int v = 0; v < 4; ++v)
        if (n < 3 * G) lds[((wr * RTW + t) * 16 + dense_drow<T>(v, lk)) * TSTR + n] = t1[t][u][v];
    }
  __syncthreads();

  // ---- Y += sum_a F_a D_a, F_a = sum_b g_ab T_b
  T dn[RTW][3];
  auto load_t = [&](int k) {
    const bool in = 4 * k + lk < G;
    const int at = in ? 4 * k + lk : 0;
#pragma unroll
    for (int t = 0; t < RTW; ++t) {
      const T* __restrict__ r = lds + ((wr * RTW + t) * 16 + li) * TSTR + at;
#pragma unroll
      for (int a = 0; a < 3; ++a) dn[t][a] = in ? r[a * G] : T(0);
    }
  };
  auto step_2 = [&](int k, int i) {
    T b[3][CT2], f[RTW][3];
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
      for (int u = 0; u < CT2; ++u) b[a][u] = bn[i][a][u];
    if (k + PD < D::NG) load_2(k + PD, i);
#pragma unroll
    for (int t = 0; t < RTW; ++t) {
      f[t][0] = g[t][0] * dn[t][0] + g[t][1] * dn[t][1] + g[t][2] * dn[t][2];
      f[t][1] = g[t][1] * dn[t][0] + g[t][3] * dn[t][1] + g[t][4] * dn[t][2];
      f[t][2] = g[t][2] * dn[t][0] + g[t][4] * dn[t][1] + g[t][5] * dn[t][2];
    }
    if (k + 1 < D::NG) load_t(k + 1);
#pragma unroll
    for (int t = 0; t < RTW; ++t)
#pragma unroll
      for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int u = 0; u < CT2; ++u) acc[t][u] = dense_mfma<T>(f[t][a], b[a][u], acc[t][u]);
  };
  load_t(0);
#pragma unroll 1
  for (int k = 0; k + PD - 1 < D::NG; k += PD) {
    step_2(k, 0);
    if constexpr (PD == 2) step_2(k + 1, 1);
  }
  if constexpr (PD == 2 && D::NG % 2 == 1) step_2(D::NG - 1, 0);
#pragma unroll
  for (int t = 0; t < RTW; ++t)
#pragma unroll
    for (int u = 0; u < CT2; ++u) {
      const int ct = wc + WC * u, col = ct * 16 + li;
      if (ct >= NCT || col >= M) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int r = (wr * RTW + t) * 16 + dense_drow<T>(v, lk);
        if (r < ne) y[(e0 + r) * M + col] = acc[t][u][v];
      }
    }
}

// Block shape by order and type: the fastest of NW in {4, 6, 8, 12, 16}, WC, RTW in 1..4 and PD in
// {1, 2} on 82,944 and 9,001 affine tetrahedra (MI355X, lambda = 1).  At P <= 4 one or two column tiles
// hold everything and the wavefronts split the rows; from P = 5 they split the columns, so that each B
// operand is read by one wavefront only, in a count that the tiles of both GEMMs divide: at P = 7 11
// and 6 tiles by 6 wavefronts (FP64, by 4: 184 -> 156 us; FP32 at 9,001 elements 20.1 -> 16.7), at P = 9
// 23 and 11 by 12 (by 8: 670 -> 584).  From P = 8 a block has 8 wavefronts and more, as T of its rows
// leaves LDS for one or two blocks a CU.  Time in us on 82,944 elements, seven stacked reference
// matrices -> this kernel, P = 4..10:
//   FP64   24.2 -> 17.8   53.9 -> 40.6   97 -> 76   190 -> 156   385 -> 272   955 -> 584  1353 -> 1057
//   FP32   13.7 -> 10.2   37.8 -> 22.8   53 -> 44   125 -> 95    185 -> 148   480 -> 302   651 -> 568
struct GradCfg {
  int NW, WC, RTW, PD;
};
template <int P, class T>
constexpr GradCfg grad_cfg() {
  constexpr GradCfg c64[9] = {{4, 1, 1, 2}, {4, 1, 1, 1}, {4, 2, 1, 2}, {4, 4, 1, 2}, {4, 4, 1, 2},
                              {12, 6, 1, 1}, {8, 8, 2, 2}, {12, 12, 3, 2}, {8, 8, 1, 1}};
  constexpr GradCfg c32[9] = {{4, 1, 1, 2}, {4, 1, 1, 2}, {4, 1, 1, 2}, {4, 4, 2, 2}, {4, 4, 1, 2},
                              {6, 6, 1, 1}, {8, 8, 3, 2}, {4, 4, 3, 1}, {8, 8, 2, 1}};
  return sizeof(T) == 8 ? c64[P - 2] : c32[P - 2];
}

template <int P, class T>
static nir_status launch_grad_P(const nir_basis* b, const OpArgs& a, hipStream_t s) {
  constexpr GradCfg c = grad_cfg<P, T>();
  using D = GradDims<P, T, c.NW, c.WC, c.RTW>;
  static_assert(D::LDS * sizeof(T) <= 160 * 1024, "LDS budget");
  const int64_t nb = (a.nelmt + D::ROWS - 1) / D::ROWS;
  if (nb > 0x7fffffff) return fail(NIR_EINVAL, "too many elements for one launch");
  if (nb == 0) return ok();
  const T *B1, *Mm;
  if constexpr (sizeof(T) == 8) {
    B1 = b->grad64;
    Mm = b->dense64;
  } else {
    B1 = b->grad32;
    Mm = b->dense32;
  }
  hipLaunchKernelGGL((k_helm_grad<P, T, c.NW, c.WC, c.RTW, c.PD>), dim3(unsigned(nb)), dim3(D::BLOCK), 0, s, B1,
                     Mm, B1 + D::MK * D::N1P, static_cast<const T*>(a.in0),
                     static_cast<T*>(a.out0), static_cast<const T*>(a.helm), T(a.lambda), a.nelmt);
  return hip_check(hipGetLastError(), "affine tetrahedron Helmholtz launch");
}

nir_status launch_helm_grad(const nir_basis* b, int dtype, const OpArgs& a, hipStream_t s) {
#define NIR_CASE(PP) \
  case PP: return dtype == NIR_F64 ? launch_grad_P<PP, double>(b, a, s) : launch_grad_P<PP, float>(b, a, s);
  switch (b->P) {
    NIR_CASE(2) NIR_CASE(3) NIR_CASE(4) NIR_CASE(5) NIR_CASE(6)
    NIR_CASE(7) NIR_CASE(8) NIR_CASE(9) NIR_CASE(10)
    default: return fail(NIR_ENOTSUP, "P=%d not compiled", b->P);
  }
#undef NIR_CASE
}

// ---------------------------------------------------------------- tables
// D_a[g][m] = int psi_g (d phi_m / d xi_a) over the reference tetrahedron is a sum of products of three
// 1-D integrals, as psi_g and phi_m are products of a factor each in eta1, eta2, eta3 and so are the
// chain rule (eq. (23)) and the volume element (1-eta2)/2 ((1-eta3)/2)^2, whose powers cancel the
// poles.  They are formed in extended precision with a Gauss-Legendre rule that is exact for them and
// rounded once: entries that vanish come out as noise otherwise, and the apply, whose error against
// 64-bit dense operators is that of its tables, would lose two digits.
using real = long double;

static real jacobi(int n, real a, real b, real x) {   // P_n^{(a,b)}(x), three-term recurrence
  real p = 1, q = 0;
  for (int k = 1; k <= n; ++k) {
    const real c = 2 * k + a + b;
    const real r = k == 1 ? (a - b + (a + b + 2) * x) / 2
                          : (((c - 1) * (a * a - b * b) + (c - 2) * (c - 1) * c * x) * p -
                             2 * (k + a - 1) * (k + b - 1) * c * q) / (2 * k * (k + a + b) * (c - 2));
    q = p;
    p = r;
  }
  return p;
}
static real ipow(real x, int n) {
  real v = 1;
  for (int k = 0; k < n; ++k) v *= x;
  return v;
}
static real djacobi(int n, real a, real b, real x) { return n ? (n + a + b + 1) / 2 * jacobi(n - 1, a + 1, b + 1, x) : 0; }

// the modified basis factor psi^b_pq (psi^a_q for p = 0) and its derivative
static void modified(int p, int q, real z, real* v, real* d) {
  const real h = (1 + z) / 2, l = (1 - z) / 2;
  if (p == 0) {
    if (q < 2) {
      *v = q ? h : l;
      *d = q ? real(0.5) : real(-0.5);
    } else {
      *v = h * l * jacobi(q - 2, 1, 1, z);
      *d = -z / 2 * jacobi(q - 2, 1, 1, z) + h * l * djacobi(q - 2, 1, 1, z);
    }
    return;
  }
  const real da = -real(p) / 2 * ipow(l, p - 1), a = ipow(l, p);
  if (q == 0) {
    *v = a;
    *d = da;
    return;
  }
  const real j = jacobi(q - 1, 2 * p - 1, 1, z), dj = djacobi(q - 1, 2 * p - 1, 1, z);
  *v = a * h * j;
  *d = da * h * j + a * j / 2 + a * h * dj;
}

// Values [n] of one factor at the rule's points; the integrals of two such vectors under a weight
using Vec = std::vector<real>;
static real dot(const Vec& f, const Vec& g) {
  real s = 0;
  for (size_t n = 0; n < f.size(); ++n) s += f[n] * g[n];
  return s;
}
static real integral(const Vec& w, const Vec& f, const Vec& g) {
  real s = 0;
  for (size_t n = 0; n < w.size(); ++n) s += w[n] * f[n] * g[n];
  return s;
}

// The gradient tables of a tetrahedral basis (shape kTet with reference matrices): psi_g the
// orthonormal polynomials of degree P - 2,
//   psi_ijk = c P_i(eta1) ((1-eta2)/2)^i P_j^{(2i+1,0)}(eta2) ((1-eta3)/2)^{i+j} P_k^{(2i+2j+2,0)}(eta3).
// Synchronous; the basis owns grad64 afterwards, which holds grad32 too.
nir_status build_grad_tables(nir_basis* b) {
  if (b->shape != kTet || !b->dense64) return NIR_OK;
  const int P = b->P, M = b->M, G = (P - 1) * P * (P + 1) / 6, N = P + 3;
  const int MK = (M + 3) / 4 * 4, NG = (G + 3) / 4, N1P = (3 * G + 15) / 16 * 16, MP = (M + 15) / 16 * 16;
  // Gauss-Legendre, N points: exact to degree 2 P + 5 (integrands reach 2 P + 1)
  Vec z(N), w(N), one(N, real(1)), zero(N, real(0));
  for (int n = 0; n < N; ++n) {
    real x = -std::cos(std::acos(real(-1)) * (n + real(0.75)) / (N + real(0.5)));
    for (int it = 0; it < 50; ++it) {
      const real step = jacobi(N, 0, 0, x) / djacobi(N, 0, 0, x);
      x -= step;
      if (std::fabs(step) < real(1e-17)) break;   // the error after a step is of its square
    }
    const real d = djacobi(N, 0, 0, x);
    z[n] = x;
    w[n] = 2 / ((1 - x * x) * d * d);
  }
  // weights in eta1: 1 and 1 + eta1; in eta2: 2, (1-eta2)/2, the same times 1 + eta2; in eta3:
  // (1-eta3)/4 and (1-eta3)^2/4
  Vec w1x(N), w2a(N), w2v(N), w2x(N), w3a(N), w3v(N);
  for (int n = 0; n < N; ++n) {
    w1x[n] = w[n] * (1 + z[n]);
    w2a[n] = w[n] * 2;
    w2v[n] = w[n] * (1 - z[n]) / 2;
    w2x[n] = w2v[n] * (1 + z[n]);
    w3a[n] = w[n] * (1 - z[n]) / 4;
    w3v[n] = w3a[n] * (1 - z[n]);
  }
  auto factor = [&](int p, int q, Vec& v, Vec& d) {
    v.resize(N);
    d.resize(N);
    for (int n = 0; n < N; ++n) modified(p, q, z[n], &v[n], &d[n]);
  };
  auto shifted = [&](int power, int deg, int alpha) {   // ((1-z)/2)^power P_deg^{(alpha,0)}
    Vec f(N);
    for (int n = 0; n < N; ++n) f[n] = ipow((1 - z[n]) / 2, power) * jacobi(deg, alpha, 0, z[n]);
    return f;
  };
  // one array: the FP64 tables, then the same in FP32
  const size_t nt = size_t(MK) * N1P + size_t(12) * NG * MP;
  std::vector<double> tabs(nt + nt / 2, 0.0);
  double* B1 = tabs.data();
  double* B2 = B1 + size_t(MK) * N1P;
  // factors of the expansion: eta1 psi^a_p, eta2 psi^b_pq, eta3 psi^b_cr, c = p + q, from the same rule
  std::vector<Vec> a1(P), d1(P), a2(P * P), d2(P * P);
  for (int p = 0; p < P; ++p) {
    factor(0, p, a1[p], d1[p]);
    for (int q = 0; p + q < P; ++q) factor(p, q, a2[p * P + q], d2[p * P + q]);
  }
  // eta3 integrals of psi_ijk: of s = i + j and k alone, the norm's share included
  std::vector<Vec> va(P * P), vd(P * P);
  for (int sl = 0; sl <= P - 2; ++sl)
    for (int k = 0; sl + k <= P - 2; ++k) {
      const Vec f3 = shifted(sl, k, 2 * sl + 2);
      const real c3 = 1 / std::sqrt(integral(w3v, f3, f3));
      Vec fa(N), fv(N), &a = va[sl * P + k], &d = vd[sl * P + k];
      for (int n = 0; n < N; ++n) {
        fa[n] = c3 * f3[n] * w3a[n];
        fv[n] = c3 * f3[n] * w3v[n];
      }
      a.resize(P * P);
      d.resize(P * P);
      for (int t = 0; t < P; ++t)
        for (int r = 0; t + r < P; ++r) {
          a[t * P + r] = dot(fa, a2[t * P + r]);
          d[t * P + r] = dot(fv, d2[t * P + r]);
        }
    }
  int g = 0;
  for (int i = 0; i <= P - 2; ++i) {
    const Vec f1 = shifted(0, i, 0);
    // the integrals with P_i over eta1, for every psi^a_p and the constant (index P: modes (0,1,r) and
    // (0,0,1), whose vertex terms add up to one in eta1)
    Vec v1(P + 1), dd1(P + 1), x1(P + 1);
    for (int p = 0; p <= P; ++p) {
      const Vec& v = p < P ? a1[p] : one;
      const Vec& d = p < P ? d1[p] : zero;
      v1[p] = integral(w, f1, v);
      dd1[p] = integral(w, f1, d);
      x1[p] = integral(w1x, f1, d);
    }
    for (int j = 0; i + j <= P - 2; ++j) {
      const Vec f2 = shifted(i, j, 2 * i + 1);
      const real c12 = 1 / std::sqrt(integral(w, f1, f1) * integral(w2v, f2, f2));
      // the eta1 and eta2 parts of the three derivatives, per (p,q) (index P^2: the apex mode (0,0,1)):
      // D_0 = e0 va, D_1 = e1 va, D_2 = e2 va + ev vd
      Vec e0(P * P + 1), e1(P * P + 1), e2(P * P + 1), ev(P * P + 1), fa(N), fv(N), fx(N);
      for (int n = 0; n < N; ++n) {
        fa[n] = c12 * w2a[n] * f2[n];
        fv[n] = c12 * w2v[n] * f2[n];
        fx[n] = c12 * w2x[n] * f2[n];
      }
      for (int t = 0; t <= P * P; ++t) {
        const bool apex = t == P * P;
        if (!apex && t / P + t % P >= P) continue;
        const Vec& v = apex ? one : a2[t];
        const Vec& d = apex ? zero : d2[t];
        const int k1 = apex || t == 1 ? P : t / P;
        const real c2 = dot(fa, v), A = x1[k1] * c2 / 2;
        e0[t] = dd1[k1] * c2;
        e1[t] = A + 2 * v1[k1] * dot(fv, d);
        e2[t] = A + v1[k1] * dot(fx, d);
        ev[t] = v1[k1] * dot(fv, v);
      }
      for (int k = 0; i + j + k <= P - 2; ++k, ++g) {
        const Vec &a = va[(i + j) * P + k], &d = vd[(i + j) * P + k];
        double* b2 = B2 + size_t(12 * (g / 4) + g % 4) * MP;
        int m = 0;
        for (int p = 0; p < P; ++p)
          for (int q = 0; p + q < P; ++q)
            for (int r = 0; p + q + r < P; ++r, ++m) {
              const int t = p == 0 && q == 0 && r == 1 ? P * P : p * P + q, k3 = (p + q) * P + r;
              const double D[3] = {double(e0[t] * a[k3]), double(e1[t] * a[k3]), double(e2[t] * a[k3] + ev[t] * d[k3])};
              for (int c = 0; c < 3; ++c) B1[size_t(m) * N1P + c * G + g] = b2[size_t(4 * c) * MP + m] = D[c];
            }
      }
    }
  }
  float* t32 = reinterpret_cast<float*>(B1 + nt);
  for (size_t k = 0; k < nt; ++k) t32[k] = float(B1[k]);
  NIR_TRYS(hip_check(hipMalloc(&b->grad64, tabs.size() * 8), "hipMalloc"));
  b->grad32 = reinterpret_cast<float*>(b->grad64 + nt);
  return hip_check(hipMemcpy(b->grad64, tabs.data(), tabs.size() * 8, hipMemcpyHostToDevice), "copy");
}

}  // namespace nir
