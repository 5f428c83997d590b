// Rows of the scatter-reduce on the host, built under AddressSanitizer and UndefinedBehaviorSanitizer: every
// length around the entries read together, at the start of the index array and at the end of the int32
// range that an assembly may fill, with the row's entries in an allocation of their exact size.
#include "host_lanes.h"

#include "row_sum.h"

using namespace nir;

int main() {
  int bad = 0;
  for (int32_t end : {0, INT32_MAX - 4, INT32_MAX - 1, INT32_MAX})   // 0: the row starts the array
    for (int n = 1; n <= 2 * kScatterEntries + 1; ++n) {
      const int32_t at = end ? end - n : 0;
      Exact<int32_t> idx(n), off(2);
      Exact<double> yl(n);
      off.p[0] = at;
      off.p[1] = at + n;
      double want = 0.0;
      for (int k = 0; k < n; ++k) {
        idx.p[k] = n - 1 - k;
        yl.p[n - 1 - k] = k * k + 1;
        want += k * k + 1;
      }
      const double got = row_sum(off.p, idx.p - at, yl.p, 0);
      if (got != want) {
        std::printf("row of %d entries to %d: %g, not %g\n", n, end, got, want);
        ++bad;
      }
    }
  std::printf("rows checked: %d failures\n", bad);
  return bad == 0 ? 0 : 1;
}
