// pc_div against the division: every divisor up to 70000, those around powers of two and random ones, at the multiples of
// the divisor where the quotient changes, the ends of the range and random numbers.
#include <stdio.h>
#include <random>
#include "div31.h"

static const long long TOP = 0x7fffffffLL;
static bool same(long long n, int d, PcDiv x) {
  if (n < 0 || n > TOP || pc_div((int)n, x) == (int)n / d) return true;
  printf("%lld / %d: %d\n", n, d, pc_div((int)n, x));
  return false;
}
static bool check(long long d0, std::mt19937& rng) {
  if (d0 < 1 || d0 > TOP) return true;
  const int d = (int)d0;
  const PcDiv x = pc_div_by(d);
  const long long last = TOP / d * d;
  bool ok = same(0, d, x) && same(1, d, x) && same(TOP, d, x) && same(TOP - 1, d, x) && same(last - 1, d, x) && same(last, d, x);
  for (int i = 0; i < 60 && ok; ++i) {
    const long long n = rng() & 0x7fffffff, m = n / d * d;
    ok = same(n, d, x) && same(m - 1, d, x) && same(m, d, x) && same(m + d - 1, d, x);
  }
  return ok;
}
int main() {
  std::mt19937 rng(5);
  for (int d = 1; d <= 70000; ++d)
    if (!check(d, rng)) return 1;
  for (int l = 16; l < 32; ++l)
    for (long long e = -40; e <= 40; ++e)
      if (!check((1LL << l) + e, rng)) return 1;
  for (int i = 0; i < 200000; ++i)
    if (!check(rng() & 0x7fffffff, rng)) return 1;
  return 0;
}
