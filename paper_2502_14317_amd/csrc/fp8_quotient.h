// The correctly rounded quotient x / scale from inv, the rounded reciprocal of scale, and one residual:
// q = x inv, q' = q - (q scale - x) inv.  Plain C++ so that a host program can compare it with the division for every
// pair of mantissas (tests/host/quotient_check.cpp).
#pragma once
#include <math.h>
#ifndef __HIPCC__
#define __host__
#define __device__
#endif

__host__ __device__ inline float pc_quotient_by_reciprocal(float x, float scale, float inv) {
  const float q = x * inv;
  return fmaf(-fmaf(q, scale, -x), inv, q);
}
