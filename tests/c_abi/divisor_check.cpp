// divide() against n / d: small divisors, those around powers of two, random ones; quotients around multiples of the divisor.
#include <cstdint>
#include <cstdio>
#include <random>
#include <vector>

#include "divisor.h"

int main() {
  std::mt19937_64 gen(20501);
  const int64_t top = INT32_MAX;
  std::vector<int64_t> divisors;
  for (int64_t d = 1; d <= 3000; d++) divisors.push_back(d);
  for (int k = 11; k <= 31; k++)
    for (int64_t d = ((int64_t)1 << k) - 2; d <= ((int64_t)1 << k) + 2; d++)
      if (d <= top) divisors.push_back(d);
  for (int i = 0; i < 3000; i++) divisors.push_back(1 + (int64_t)(gen() % (uint64_t)(top >> (gen() % 31))));
  for (int64_t d : divisors) {
    const tr::Divisor by = tr::make_divisor((unsigned)d);
    auto same = [&](int64_t n) {
      if (n < 0 || n > top || tr::divide(by, (int)n) == n / d) return true;
      std::printf("%lld / %lld: %d\n", (long long)n, (long long)d, tr::divide(by, (int)n));
      return false;
    };
    for (int64_t n = 0; n < 300; n++)
      if (!same(n) || !same(top - n)) return 1;
    for (int i = 0; i < 300; i++) {
      const int64_t n = (int64_t)(gen() % ((uint64_t)top + 1)), q = n / d * d;
      if (!same(n) || !same(q - 1) || !same(q) || !same(q + 1)) return 1;
    }
  }
  std::printf("divisor ok\n");
}
