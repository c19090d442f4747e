// Rotation of query rows as a workgroup function: a launch of its own (decode_attn.hip) and behind the
// rotation table's workgroups (prep.hip).
#pragma once
#include "pc_common.h"

// Query rows rotated at positions pos0 + t (pos0 < 0: they arrive rotated), times mul, all in fp64 and
// rounded to bf16 once: the tile kernel's operand (mul = softmax scale x log2(e)) and the few-row
// path's where the merge needs it too (mul = 1).  One workgroup per query row: its first threads
// compute the D / 2 angles once for all heads, while the rows, 16 bytes of each half a thread, are
// on their way.  Bound by memory and the fp64 latency in front: 2048 rows of 32 x 128 values (33 MB)
// 9.6 us, 15.4 with every thread computing its own angles.
template <int D>
__device__ __forceinline__ void pc_rope_q_workgroup(const uint16_t* __restrict__ q, uint16_t* __restrict__ q_rot, int row,
                                                    int n_q, int n_heads, int pos0, const PcRope& rope, double mul) {
  constexpr int HALF = D / 2, TPR = HALF / 8;                       // threads per head row
  __shared__ double2 angle[HALF];                                   // (cos, sin)
  const int i0 = (threadIdx.x % TPR) * 8;
  const long long row0 = (long long)row * n_heads;           // (b, t, head 0)
  int h = threadIdx.x / TPR;
  uint4 a = make_uint4(0, 0, 0, 0), b = a;
  if (h < n_heads) {
    a = *(const uint4*)(q + (row0 + h) * D + i0);
    b = *(const uint4*)(q + (row0 + h) * D + i0 + HALF);
  }
  if (threadIdx.x < HALF) {
    double sn = 0.0, cs = 1.0;
    if (pos0 >= 0)
      pc_sincos((double)(pos0 + row % n_q) * pc_rope_theta(rope, (int)threadIdx.x), sn, cs);
    angle[threadIdx.x] = make_double2(cs, sn);
  }
  __syncthreads();
  while (h < n_heads) {
    const uint32_t aw[4] = {a.x, a.y, a.z, a.w}, bw[4] = {b.x, b.y, b.z, b.w};
    uint32_t ra[4], rb[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double2 c0 = angle[i0 + 2 * e], c1 = angle[i0 + 2 * e + 1];
      const double x1l = bf16_lo_to_f32(aw[e]), x1h = bf16_hi_to_f32(aw[e]);
      const double x2l = bf16_lo_to_f32(bw[e]), x2h = bf16_hi_to_f32(bw[e]);
      ra[e] = pack_bf16x2((float)((x1l * c0.x - x2l * c0.y) * mul), (float)((x1h * c1.x - x2h * c1.y) * mul));
      rb[e] = pack_bf16x2((float)((x2l * c0.x + x1l * c0.y) * mul), (float)((x2h * c1.x + x1h * c1.y) * mul));
    }
    const long long at = (row0 + h) * D + i0;
    h += 256 / TPR;
    if (h < n_heads) {
      a = *(const uint4*)(q + (row0 + h) * D + i0);
      b = *(const uint4*)(q + (row0 + h) * D + i0 + HALF);
    }
    *(uint4*)(q_rot + at) = make_uint4(ra[0], ra[1], ra[2], ra[3]);
    *(uint4*)(q_rot + at + HALF) = make_uint4(rb[0], rb[1], rb[2], rb[3]);
  }
}
