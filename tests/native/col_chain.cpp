// Chain-rule factors of the collapsed shapes in FP32 and FP64 at the points of every order, against the
// same factors of the same (rounded) coordinates in long double.  k1 of the tetrahedron rounds four times
// (1 - z3, its reciprocal, 1 - z2, the divide), k1 of the others and k2 twice, e2 once: as many units of
// half an ulp, and a hundredth for their products.
#include "host_lanes.h"

#include "helm_col_dev.h"

using namespace nir;

static int g_bad = 0;

template <int SHAPE, class T>
static void check(int P, T z2, T z3) {
  const ColChain<T> c = col_chain<SHAPE>(z2, z3);
  using L = long double;
  const L one = 1, r = one / (one - L(z3)), u = L(std::numeric_limits<T>::epsilon()) / 2 * 1.01L;
  const L want[3] = {one + L(z2), SHAPE == kTet ? 2 * r / (one - L(z2)) : r, r};
  const T got[3] = {c.e2, c.k1, c.k2};
  const int rounds[3] = {1, SHAPE == kTet ? 4 : 2, 2};
  for (int k = 0; k < 3; ++k) {
    const L err = std::fabs(L(got[k]) - want[k]), bar = rounds[k] * u * std::fabs(want[k]);
    if (!(err <= bar)) {
      std::printf("shape %d, P %d, %d bytes, z2 %g, z3 %g: factor %d off by %Lg of %Lg\n", SHAPE, P, int(sizeof(T)), double(z2),
                  double(z3), k, err, want[k]);
      ++g_bad;
    }
  }
}

template <int SHAPE>
static void orders() {
  for (int P = kMinP; P <= kMaxP; ++P) {
    HostTables t;
    if (!build_tables(SHAPE, P, P + 1, t)) {
      ++g_bad;
      continue;
    }
    for (double z2 : t.z[1])
      for (double z3 : t.z[2]) {
        check<SHAPE, double>(P, z2, z3);
        check<SHAPE, float>(P, float(z2), float(z3));
      }
  }
}

int main() {
  orders<kPrism>();
  orders<kTet>();
  orders<kPyr>();
  std::printf("chain factors: %d failures\n", g_bad);
  return g_bad == 0 ? 0 : 1;
}
