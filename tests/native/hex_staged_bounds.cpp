// The hexahedral even-odd Helmholtz group with staged factors (FP32, P = 2..4, per-point factors) on the
// host, one thread per lane, built under AddressSanitizer: every count of elements in the last group,
// with the coefficients direct and through a map, all buffers of their exact sizes.  The gathered apply
// equals the direct one.
#include "host_lanes.h"

#include "helm_hex.h"
#include "helm_hex_eo_dev.h"

using namespace nir;

static int g_bad = 0;

template <int P>
static void check() {
  using T = float;
  constexpr int E = hex_block_elems<P, T>(kFamEO);
  using D = HexPencilDims<P, T, E, false>;
  constexpr int NQ = D::NQ, M = D::M, F = EoDims<P>::H * EoDims<P>::ROW;
  Exact<T> tabs(F), wq(NQ, T(1)), lds(D::LDS + E * 7 * NQ + D::BLOCK);
  for (int k = 0; k < F; ++k) tabs.p[k] = T((k * 7) % 11 - 5) / 8;
  for (int ne = 1; ne <= 2 * E; ++ne) {
    Exact<T> x(size_t(ne) * M), xg(size_t(ne) * M), helm(size_t(ne) * 7 * NQ), y(size_t(ne) * M, T(-9)),
        yg(size_t(ne) * M, T(-9));
    Exact<int32_t> map(size_t(ne) * M);
    for (size_t k = 0; k < x.n; ++k) {
      x.p[k] = T(int(k * 13 % 29) - 14) / 16;
      map.p[k] = int32_t(x.n - 1 - k);
      xg.p[x.n - 1 - k] = x.p[k];
    }
    for (size_t k = 0; k < helm.n; ++k) helm.p[k] = T(int(k * 5 % 17) - 8) / 8;
    auto run = [&](auto gather) {
      constexpr bool G = decltype(gather)::value;
      run_blocks(D::BLOCK, (ne + E - 1) / E,
                 [&](int64_t) { std::fill(lds.p, lds.p + lds.n, std::numeric_limits<T>::quiet_NaN()); },
                 [&](int64_t b) {
                   helm_hex_eo_group<P, T, true, E, false, true, 1, false, true, G>(
                       tabs.p, G ? xg.p : x.p, G ? yg.p : y.p, helm.p, wq.p, T(1), ne, b * E, lds.p, nullptr, nullptr,
                       nullptr, G ? map.p : nullptr);
                 });
    };
    run(std::false_type{});
    run(std::true_type{});
    for (size_t k = 0; k < y.n; ++k)
      if (!(y.p[k] == yg.p[k]) || !std::isfinite(y.p[k])) {
        std::printf("P %d, %d elements: value %zu is %g direct and %g gathered\n", P, ne, k, y.p[k], yg.p[k]);
        ++g_bad;
        break;
      }
  }
}

int main() {
  check<2>();
  check<3>();
  check<4>();
  std::printf("staged groups checked: %d failures\n", g_bad);
  return g_bad == 0 ? 0 : 1;
}
