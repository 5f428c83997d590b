// Round-to-nearest-even conversion of FP32 to FP16 bits on the host, without the compiler's conversion
// call (5 to 10 ns a value, most of the time of creating a basis with reference matrices).
#pragma once

#include <cstdint>
#include <cstring>

namespace nir {

// The FP16 bits of `a`, |a| < 65520 (what rounds to a finite value), and their value.  From 2^-14 up
// half an ulp of the 13 dropped bits, less one where the kept part is even, carries into it; below, the
// addition to 0.5, whose ulp is the subnormals' step 2^-24, rounds the same way.
inline uint16_t half_bits(float a, float* value) {
  uint32_t u;
  std::memcpy(&u, &a, 4);
  const uint32_t sign = u & 0x80000000u, m = u ^ sign;
  const uint32_t r = m + 0xfffu + (m >> 13 & 1u);
  float f;
  std::memcpy(&f, &m, 4);
  f += 0.5f;
  uint32_t fb, sb;
  std::memcpy(&fb, &f, 4);
  const float sub = f - 0.5f;
  std::memcpy(&sb, &sub, 4);
  const bool normal = m >= 0x38800000u;
  const uint32_t h = normal ? (r >> 13) - 0x1c000u : fb - 0x3f000000u;
  const uint32_t v = (normal ? r & ~0x1fffu : sb) | sign;
  std::memcpy(value, &v, 4);
  return uint16_t(h | sign >> 16);
}

}  // namespace nir
