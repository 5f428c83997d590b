// Gathered coefficients (OpArgs::map) only reach kernels that gather.  Linked against libnir.so and run
// without a device, so that a launch that is let through fails with NIR_EHIP and one that is refused
// with NIR_EINVAL: for every hexahedral variant, and for the collapsed shapes, the launch with a map is
// let through exactly where the kernel takes the map.
#include <cstdio>

#include "nir_internal.h"

using namespace nir;

int main() {
  int n = 0;
  if (hipGetDeviceCount(&n) == hipSuccess && n > 0) {
    std::printf("a device is visible\n");
    return 2;
  }
  int bad = 0;
  int32_t map[64] = {};
  double x[64] = {};
  auto basis = [&](int shape, int P) {   // as far as a launch looks at it on the host
    nir_basis b{};
    b.shape = shape;
    b.P = P;
    b.Q = P + 1;
    b.M = int(modes_of(shape, P));
    b.eo64 = x;
    b.eo32 = reinterpret_cast<float*>(x);
    return b;
  };
  OpArgs a{};
  a.in0 = a.out0 = x;
  a.helm = x;
  a.nelmt = 1;
  a.map = map;
  auto launch = [&](int shape, int P, int dtype, int deformed) {
    const nir_basis b = basis(shape, P);
    return launch_helm_auto(&b, dtype, deformed, a, nullptr);
  };
  for (int dtype : {NIR_F64, NIR_F32})
    for (int deformed = 0; deformed < 2; ++deformed) {
      for (int v = NIR_VARIANT_AUTO; v < NIR_VARIANT_DENSE; ++v) {
        if (nir_set_helmholtz_variant(kHex, 4, dtype, v) != NIR_OK) ++bad;
        const int st = launch(kHex, 4, dtype, deformed), want = v == NIR_VARIANT_GENERIC ? NIR_EINVAL : NIR_EHIP;
        if (st != want) {
          std::printf("hexahedra, dtype %d, deformed %d, variant %d: status %d, not %d\n", dtype, deformed, v, st, want);
          ++bad;
        }
      }
      for (int shape : {kPrism, kTet, kPyr})
        for (int v : {NIR_VARIANT_AUTO, NIR_VARIANT_GENERIC, NIR_VARIANT_PENCIL, NIR_VARIANT_DENSE}) {
          if (nir_set_helmholtz_variant(shape, 4, dtype, v) != NIR_OK) ++bad;
          const int st = launch(shape, 4, dtype, deformed);
          if (st != NIR_EINVAL) {
            std::printf("shape %d, dtype %d, deformed %d, variant %d: status %d\n", shape, dtype, deformed, v, st);
            ++bad;
          }
        }
    }
  // a variant asked for once stays the one that runs, whatever is selected in between
  nir_set_helmholtz_variant(kHex, 4, NIR_F64, NIR_VARIANT_AUTO);
  const int v = helm_variant(kHex, 4, NIR_F64, 1, 1);
  nir_set_helmholtz_variant(kHex, 4, NIR_F64, NIR_VARIANT_GENERIC);
  const nir_basis b = basis(kHex, 4);
  if (!helm_gathers(kHex, v) || launch_helm_variant(v, &b, NIR_F64, 1, a, nullptr) != NIR_EHIP) ++bad;
  if (helm_gathers(kHex, helm_variant(kHex, 4, NIR_F64, 1, 1))) ++bad;
  std::printf("map routes checked: %d failures\n", bad);
  return bad == 0 ? 0 : 1;
}
