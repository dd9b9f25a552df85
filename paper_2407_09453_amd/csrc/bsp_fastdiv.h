// x / d by one multiply-high (library private; plain C++, also compiled on the host by the
// tests).  mul = floor(2^32 / d) + 1; the quotient floor(x * mul / 2^32) equals x / d while
// x * d < 2^32, which every launcher checks for the dividends it can produce.
#ifndef BSP_FASTDIV_H
#define BSP_FASTDIV_H

#include <stdint.h>

struct FastDiv {
  uint32_t d, mul;
};
inline FastDiv make_fastdiv(uint32_t d) {
  FastDiv f;
  f.d = d;
  f.mul = d > 1 ? (uint32_t)((0x100000000ull / d) + 1) : 0u;
  return f;
}
// the same arithmetic as the device's __umulhi
inline uint32_t fdiv_host(uint32_t x, FastDiv f) {
  return f.d == 1 ? x : (uint32_t)(((uint64_t)x * f.mul) >> 32);
}

// x / d for what lies in LDS or a workgroup's tile (x < 2^15, 1 <= d <= 2^15): one 24-bit multiplication and a
// shift, both at full rate, where a multiply-high takes four times as long.  mul = floor(2^s / d) + 1 with
// s = 16 + ceil(log2 d): mul <= 2^16 * 2 + 1, so x * mul < 2^32, and x * d < 2^s, so the quotient is exact.
struct SmallDiv {
  uint32_t mul, shift;
};
inline SmallDiv make_smalldiv(uint32_t d) {
  SmallDiv f;
  f.shift = 16;
  while ((1u << (f.shift - 16)) < d) ++f.shift;
  f.mul = (uint32_t)((1ull << f.shift) / d) + 1;
  return f;
}
// the same arithmetic as the device's 24-bit multiplication
inline uint32_t sdiv_host(uint32_t x, SmallDiv f) { return (uint32_t)((uint64_t)(x & 0xFFFFFFu) * (f.mul & 0xFFFFFFu)) >> f.shift; }

#endif
