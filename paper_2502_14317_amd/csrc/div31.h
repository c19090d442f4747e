// Division of whole numbers below 2^31 by a divisor that the host knows: with 2^(l - 1) < d <= 2^l and
// m = ceil(2^(31 + l) / d), m d is at most 2^l above 2^(31 + l), so n / d = (n m) >> (31 + l) exactly (Granlund and
// Montgomery, "Division by invariant integers using multiplication", 1994, theorem 4.2 at N = 31).  Two scalar
// multiplications and a shift, where the compiler's division by a kernel argument is a chain of some 25 instructions
// through a reciprocal.  In front of a workgroup's first load those chains are latency: 8 decoding steps of one
// sequence of 8 x 2048 keys 150.2 -> 146.3 us, the preparation, score passes and selection of a layer of 4 x 512 tokens
// (8 heads of 64 values) 1.1 us, of 12 ragged chunks of 2011 6 us.  Plain C++ so that a host program can compare it with the division
// (tests/host/div31_check.cpp).
#pragma once
#include <stdint.h>
#ifndef __HIPCC__
#define __host__
#define __device__
#endif

struct PcDiv {
  uint32_t mul;
  int shift;
};
// d < 1: whoever divides by it is not launched
__host__ __device__ inline PcDiv pc_div_by(int d) {
  PcDiv x = {0u, 31};
  if (d < 1) return x;
  while ((1LL << (x.shift - 31)) < d) ++x.shift;
  x.mul = (uint32_t)(((1ULL << x.shift) + (uint32_t)d - 1) / (uint32_t)d);
  return x;
}
__host__ __device__ inline int pc_div(int n, PcDiv x) {
  return (int)(((uint64_t)(uint32_t)n * x.mul) >> x.shift);
}
__host__ __device__ inline int pc_mod(int n, int d, PcDiv x) { return n - pc_div(n, x) * d; }
