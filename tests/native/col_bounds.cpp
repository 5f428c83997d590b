// The collapsed-shape Helmholtz groups on the host, one thread per lane, built under AddressSanitizer (or
// ThreadSanitizer: no two lanes touch a value without a barrier between) by tests/test_native_bounds.py:
// every order, both types, per-element and per-point factors, in the launch shapes of the standalone
// kernels and of the persistent mixed kernel, with every count of elements that a last group can have
// around its ends.  Every buffer and every table has an allocation of its exact size; LDS starts as NaN
// for each block.  A batch of equal factors at all points gives the per-element result.
//
// CHECK_SHAPE: the shape; the tables are those that nir_basis_create makes, with the device's memory calls
// replaced by the host's.
#include "host_lanes.h"

#include "helm_col.h"
#include "mixed_kernels.h"

using namespace nir;

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  *p = std::malloc(n);
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return ""; }
}
namespace nir {
nir_status build_dense_refs(nir_basis*) { return NIR_OK; }
nir_status build_grad_tables(nir_basis*) { return NIR_OK; }
}

static int g_bad = 0;
static int64_t g_runs = 0;

// the tables that the groups read, each in an allocation of its own
template <class T>
struct Tables {
  std::vector<std::unique_ptr<Exact<T>>> own;
  DevTab<T> tb{};
  const T* pen;
  const T* copy(const T* p, size_t n) {
    own.emplace_back(new Exact<T>(n));
    std::copy(p, p + n, own.back()->p);
    return own.back()->p;
  }
  Tables(const nir_basis* b, const DevTab<T>& t, const T* pencil) {
    const int P = b->P, Q = b->Q;
    const size_t na = col_a_off(b->shape, P, P), nb = b->shape == kTet ? col_b_off(b->shape, P, P) : 0;
    for (int d = 0; d < 3; ++d) tb.z[d] = copy(t.z[d], Q);
    tb.T3 = copy(t.T3, size_t(b->M) * Q);
    tb.dT3 = copy(t.dT3, size_t(b->M) * Q);
    tb.wq = copy(t.wq, size_t(Q) * Q * Q);
    tb.eo = copy(t.eo, size_t((Q + 1) / 2) * 2 * P);
    tb.T3t = copy(t.T3t, na);
    tb.dT3t = copy(t.dT3t, na);
    if (nb) {
      tb.T2t = copy(t.T2t, nb);
      tb.dT2t = copy(t.dT2t, nb);
    }
    pen = copy(pencil, size_t(2) * Q * P);
  }
};

template <class T>
struct Batch {
  Exact<T> x, y, affine, point;
  Batch(int64_t ne, int M, int NQ, const T* wq) : x(ne * M), y(ne * M, T(-9)), affine(ne * 7), point(ne * 7 * NQ) {
    for (size_t k = 0; k < x.n; ++k) x.p[k] = T(int(k * 13 % 29) - 14) / 16;
    for (size_t k = 0; k < affine.n; ++k) affine.p[k] = T(int(k * 5 % 17) + 1) / 8;
    for (size_t k = 0; k < point.n; ++k) point.p[k] = affine.p[k / NQ] * wq[k % NQ];
  }
};

// one launch shape: `threads` lanes, `elems` elements a block, `lds` values
template <class T, class F>
static void launch(int P, const char* what, int threads, int elems, int lds, int64_t ne, const Exact<T>& y, F body) {
  Exact<T> l(lds);
  std::fill(y.p, y.p + y.n, T(-9));
  run_blocks(threads, (ne + elems - 1) / elems,
             [&](int64_t) { std::fill(l.p, l.p + l.n, std::numeric_limits<T>::quiet_NaN()); },
             [&](int64_t b) { body(b * elems, l.p); });
  ++g_runs;
  for (size_t k = 0; k < y.n; ++k)
    if (!std::isfinite(y.p[k])) {
      std::printf("%s, P %d, %d bytes a value, %lld elements: value %zu is %g\n", what, P, int(sizeof(T)), (long long)ne, k,
                  double(y.p[k]));
      ++g_bad;
      return;
    }
}

template <class T>
static void compare(int P, const char* what, int64_t ne, const Exact<T>& y, const std::vector<T>& ref) {
  double top = 0, err = 0;
  for (size_t k = 0; k < y.n; ++k) {
    top = std::max(top, std::fabs(double(ref[k])));
    err = std::max(err, std::fabs(double(ref[k]) - double(y.p[k])));
  }
  if (!(err <= (sizeof(T) == 8 ? 1e-12 : 1e-4) * top)) {
    std::printf("%s, P %d, %d bytes a value, %lld elements: off by %g of %g\n", what, P, int(sizeof(T)), (long long)ne, err, top);
    ++g_bad;
  }
}

// counts of elements: a last group of one, of the middle and of all but one of a group's elements
static std::vector<int64_t> counts(std::vector<int64_t> n) {
  n.erase(std::remove_if(n.begin(), n.end(), [](int64_t k) { return k < 1; }), n.end());
  std::sort(n.begin(), n.end());
  n.erase(std::unique(n.begin(), n.end()), n.end());
  return n;
}

template <int P, class T, bool DEF, bool ONE = false>
static void group(const Tables<T>& t, int64_t ne, Batch<T>& b) {
  using D = ColKernelDims<CHECK_SHAPE, P, T, DEF, ONE>;
  launch<T>(P, DEF ? "per-point group" : "per-element group", D::BLOCK, D::E, D::LDS, ne, b.y, [&](int64_t first, T* lds) {
    helm_col_group<CHECK_SHAPE, P, T, DEF, D::E>(t.tb, t.pen, b.x.p, b.y.p, DEF ? b.point.p : b.affine.p, T(0.75), ne, first, lds);
  });
}

template <int P, class T, bool DEF>
static void mixed(const Tables<T>& t, int64_t ne, Batch<T>& b) {
  using C = MixedCol<CHECK_SHAPE, P, T>;
  launch<T>(P, DEF ? "per-point item" : "per-element item", kMixedBlock, C::ELEMS, C::LDS, ne, b.y, [&](int64_t first, T* lds) {
    helm_col_group<CHECK_SHAPE, P, T, DEF, C::E, C::NSUB>(t.tb, t.pen, b.x.p, b.y.p, DEF ? b.point.p : b.affine.p, T(0.75), ne,
                                                    first, lds);
  });
}

template <int P, class T>
static void order(const nir_basis* basis, const DevTab<T>& tab, const T* pen) {
  const Tables<T> t(basis, tab, pen);
  constexpr int NQ = (P + 1) * (P + 1) * (P + 1);
  using D = ColKernelDims<CHECK_SHAPE, P, T, true>;
  using A = ColKernelDims<CHECK_SHAPE, P, T, false>;
  const int e = A::E, d = D::E;
  const std::vector<int64_t> ns = counts({1, e / 2 + 1, e - 1, e + 1, d - 1, d + 1});
  for (int64_t ne : ns) {
    Batch<T> b(ne, basis->M, NQ, t.tb.wq);
    group<P, T, true>(t, ne, b);
    const std::vector<T> ref(b.y.p, b.y.p + b.y.n);
    group<P, T, false>(t, ne, b);
    compare(P, "per-element group", ne, b.y, ref);
    if constexpr (col_has_one<CHECK_SHAPE, P, T, true>) {
      group<P, T, true, true>(t, ne, b);
      compare(P, "group of one a CU", ne, b.y, ref);
    }
  }
  if constexpr (CHECK_SHAPE != kPyr && P <= kMixedMaxP) {
    using C = MixedCol<CHECK_SHAPE, P, T>;
    // the first group alone, not full and just full, one group past the end, the last group short
    for (int64_t ne : counts({1, C::E, C::E + 1, C::ELEMS - 1, C::ELEMS + 1})) {
      Batch<T> b(ne, basis->M, NQ, t.tb.wq);
      mixed<P, T, true>(t, ne, b);
      const std::vector<T> ref(b.y.p, b.y.p + b.y.n);
      mixed<P, T, false>(t, ne, b);
      compare(P, "per-element item", ne, b.y, ref);
    }
  }
}

template <int P>
static void orders() {
  nir_basis* b = nullptr;
  if (nir_basis_create(CHECK_SHAPE, P, P + 1, &b) != NIR_OK) {
    ++g_bad;
    return;
  }
  order<P, double>(b, b->t64, b->pencil64);
  order<P, float>(b, b->t32, b->pencil32);
  nir_basis_destroy(b);
  if constexpr (P < CHECK_PMAX) orders<P + 1>();
}

int main() {
  orders<CHECK_PMIN>();
  std::printf("shape %d, P %d to %d: %lld runs, %d failures\n", CHECK_SHAPE, CHECK_PMIN, CHECK_PMAX, (long long)g_runs, g_bad);
  return g_bad == 0 ? 0 : 1;
}
