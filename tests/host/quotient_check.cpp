// Compares pc_quotient_by_reciprocal with the division, bit for bit: every mantissa of the scale (2^23) with every
// mantissa of a bf16 value (2^7).  Exponents do not matter while nothing under- or overflows.
#include "fp8_quotient.h"
#include <atomic>
#include <stdint.h>
#include <stdio.h>
#include <string.h>
#include <thread>
#include <vector>

static float from_bits(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
static uint32_t bits(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }

int main() {
  std::atomic<long long> pairs{0}, wrong{0};
  const uint32_t n = 1u << 23, workers = 8;
  std::vector<std::thread> pool;
  for (uint32_t w = 0; w < workers; ++w)
    pool.emplace_back([&, w] {
      long long bad = 0;
      for (uint32_t m = w * (n / workers); m < (w + 1) * (n / workers); ++m) {
        const float scale = from_bits(0x3f800000u | m), inv = 1.0f / scale;
        for (uint32_t x = 0; x < 128; ++x) {
          const float v = from_bits(0x3f800000u | (x << 16));
          bad += bits(pc_quotient_by_reciprocal(v, scale, inv)) != bits(v / scale);
        }
      }
      wrong += bad; pairs += (long long)(n / workers) * 128;
    });
  for (auto& t : pool) t.join();
  printf("%lld pairs, %lld differ\n", (long long)pairs, (long long)wrong);
  return wrong == 0 && pairs == (1LL << 30) ? 0 : 1;
}
