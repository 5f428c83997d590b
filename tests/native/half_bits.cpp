// half_bits against its definition: the nearest of all finite FP16 values, ties to the even one.  Every
// finite FP16 value, the midpoints between neighbours and the FP32 values next to these, both signs.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <vector>

#include "half_bits.h"

int main() {
  std::vector<float> val(0x7c00);   // value of the bits 0 .. 0x7bff, ascending
  for (int b = 0; b < 0x7c00; ++b)
    val[b] = b < 0x400 ? std::ldexp(float(b), -24) : std::ldexp(float(0x400 + (b & 0x3ff)), (b >> 10) - 25);
  int bad = 0;
  long n = 0;
  auto check = [&](float a) {
    const float m = std::fabs(a);
    if (!(m < 65520.f)) return;
    int hi = int(std::lower_bound(val.begin(), val.end(), m) - val.begin());   // first value >= m
    int want = std::min(hi, 0x7bff);
    if (want > 0 && val[want] != m) {
      const double up = hi > 0x7bff ? 65536.0 : double(val[hi]), dn = val[hi - 1], mid = 0.5 * (up + dn);
      want = m < mid || (m == mid && ((hi - 1) & 1) == 0) ? hi - 1 : hi;
    }
    float v;
    const uint16_t got = nir::half_bits(a, &v);
    const int expect = want | (std::signbit(a) ? 0x8000 : 0);
    const float ev = std::signbit(a) ? -val[want] : val[want];
    ++n;
    if (got != expect || v != ev || std::signbit(v) != std::signbit(ev)) {
      if (bad++ < 10) std::printf("%a: bits %04x, not %04x, value %a\n", double(a), got, expect, double(v));
    }
  };
  for (int b = 0; b < 0x7c00; ++b) {
    const float mid = b + 1 < 0x7c00 ? float(0.5 * (double(val[b]) + double(val[b + 1]))) : 65519.996f;
    for (float c : {val[b], mid})
      for (float a : {c, std::nextafter(c, 0.f), std::nextafter(c, 1e9f)}) {
        check(a);
        check(-a);
      }
  }
  std::printf("%ld values, %d failures\n", n, bad);
  return bad == 0 ? 0 : 1;
}
