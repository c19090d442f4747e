// What a layer's other launches read and nothing of which depends on the keys, in one launch (a launch of
// its own each costs 3 to 6 us):
//   the rotation table        cos / sin of position * theta_i, computed in fp64, stored fp32; for the local
//                             attention's queries a second one, turned (two pairs' positions side by side) and
//                             times scale * log2(e)
//   the query block           rotated for the global attention (pc_rope_q_workgroup)
//   the score passes' queries the voting rows as ready MFMA operands: rotated in fp32, scaled to log2 units,
//                             split into bf16 hi + lo, so that a workgroup of the passes starts with
//                             coalesced loads instead of gathering, rotating and splitting 32 rows a wavefront
//                             (both passes together 4 to 8 us longer at 100 to 500 workgroups; with many voting
//                             rows, 12 chunks of 203 rows x 32 heads, a launch of 20 us)
// Bound by latency and the fp64 angles: 4 x 9 KV heads of 32 columns of 64 values 4 us in all, 16 x 8 of 128 columns
// of 128 values 9.
#include "rope.h"

// One wavefront: k-steps ks and ks + D / 32 of a block of 32 columns.
template <int D>
__device__ __forceinline__ void split_query_columns(const PcScoreQueries& a, const PcRope& rope, long long unit, int lane) {
  constexpr int KS = D / 16, HALF = D / 2;
  // (column blocks of all chunks and KV heads are fewer than 2^31: their keys would not fit in memory)
  const int ks = (int)(unit % (KS / 2)), block = (int)(unit / (KS / 2));
  const int cg = pc_div(block, a.cb_div), cb = block - cg * a.n_cb;
  const int c = pc_div(cg, a.heads_div), g = cg - c * a.n_kv_heads, n_heads = a.G * a.n_kv_heads;
  // a short chunk is [len context rows ; the query rows]: its voting rows end at len + w_q
  const int ctx_len = a.chunk_lens ? min(max(a.chunk_lens[c], 0), a.w) : a.w;
  const int col = min(32 * cb + lane % 32, a.n_cols - 1), head = pc_div(col, a.obs_div);
  const int row = ctx_len + (a.L - a.w) - a.w_obs + (col - head * a.w_obs);
  const int i0 = 16 * ks + 8 * (lane / 32);
  const uint16_t* qrow = a.q + (((long long)c * a.L + row) * n_heads + g * a.G + head) * D;
  const uint4 x1 = *(const uint4*)(qrow + i0), x2 = *(const uint4*)(qrow + HALF + i0);
  const uint32_t aw[4] = {x1.x, x1.y, x1.z, x1.w}, bw[4] = {x2.x, x2.y, x2.z, x2.w};
  u32x4 h1, l1, h2, l2;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    float2 cs[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      double sn, co;
      pc_sincos((double)row * pc_rope_theta(rope, i0 + 2 * e + u), sn, co);
      cs[u] = make_float2((float)co, (float)sn);
    }
    const float x1l = bf16_lo_to_f32(aw[e]), x1h = bf16_hi_to_f32(aw[e]);
    const float x2l = bf16_lo_to_f32(bw[e]), x2h = bf16_hi_to_f32(bw[e]);
    uint32_t hi, lo;
    // logits come out of the matrix cores in log2 units: the scale rides on q
    split_bf16x2((x1l * cs[0].x - x2l * cs[0].y) * a.scale_log2, (x1h * cs[1].x - x2h * cs[1].y) * a.scale_log2, hi, lo);
    h1[e] = hi; l1[e] = lo;
    split_bf16x2((x2l * cs[0].x + x1l * cs[0].y) * a.scale_log2, (x2h * cs[1].x + x1h * cs[1].y) * a.scale_log2, hi, lo);
    h2[e] = hi; l2[e] = lo;
  }
  // [hi, lo][k-step][half][column][8]
  const int cols = min(a.n_cols, 32), n = lane % 32, step = 2 * cols;
  if (n >= cols) return;                                           // a single block of fewer columns holds no others
  u32x4* dst = (u32x4*)a.q_split + ((long long)cg * a.n_cb + cb) * (2 * KS) * step + (lane / 32) * cols + n;
  dst[ks * step] = h1;        dst[(ks + KS / 2) * step] = h2;
  dst[(KS + ks) * step] = l1; dst[(KS + ks + KS / 2) * step] = l2;
}

template <int D>
__global__ __launch_bounds__(256) void layer_prep_kernel(PcPrepArgs a, int table_blocks, long long split_units) {
  // the tables, 16 positions a workgroup; the queries' one with the positions side by side goes through LDS
  constexpr int HALF = D / 2, PER = 16 * HALF / 256;
  __shared__ float2 turned[HALF][17];                               // [pair][position]
  int bid = (int)(blockIdx.y * gridDim.x + blockIdx.x);
  if (bid < table_blocks) {
    const int p0 = 16 * bid, i = threadIdx.x % HALF, rows = (a.n_pos + 127) / 128 * 128;
    const double theta = pc_rope_theta(a.rope, i);
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int p = threadIdx.x / HALF + (256 / HALF) * u;
      double sn, cs;
      pc_sincos((double)(p0 + p) * theta, sn, cs);
      if (p0 + p < a.n_pos) a.table[(long long)(p0 + p) * HALF + i] = make_float2((float)cs, (float)sn);
      turned[i][p] = make_float2((float)(cs * a.q_scale), (float)(sn * a.q_scale));
    }
    if (a.q_table == nullptr) return;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
      const int x = threadIdx.x + 256 * u;
      const int pair = x / 32 * 2 + x % 2, p = x % 32 / 2;
      a.q_table[((long long)(pair / 2) * rows + p0 + p) * 2 + pair % 2] = turned[pair][p];
    }
    return;
  }
  bid -= table_blocks;
  if (bid < a.n_q) {
    pc_rope_q_workgroup<D>(a.q_blk, a.q_rot, bid, a.n_q, a.n_heads, a.pos0, a.rope, a.mul);
    return;
  }
  const long long unit = (bid - a.n_q) * 4LL + __builtin_amdgcn_readfirstlane(threadIdx.x / PC_WAVE);
  if (unit < split_units) split_query_columns<D>(a.scores, a.rope, unit, threadIdx.x % PC_WAVE);
}

int pc_launch_prep(const PcPrepArgs& a, int head_dim, hipStream_t st) {
  const long long table_blocks = a.q_table ? (a.n_pos + 127LL) / 128 * 8 : (a.n_pos + 15LL) / 16;
  const long long units = a.scores.q_split ? (long long)a.scores.n_chunks * a.scores.n_kv_heads * a.scores.n_cb * (head_dim / 32) : 0;
  const long long blocks = table_blocks + a.n_q + (units + 3) / 4;
  if (blocks > 0x7fffffffLL - PC_GRID_X) return PC_ERR_SHAPE;
  PcProfScope prof(PC_KERNEL_LAYER_PREP, st);
  const dim3 grid = pc_grid_2d(blocks), block(256);
  if (head_dim == 128) hipLaunchKernelGGL(layer_prep_kernel<128>, grid, block, 0, st, a, (int)table_blocks, units);
  else hipLaunchKernelGGL(layer_prep_kernel<64>, grid, block, 0, st, a, (int)table_blocks, units);
  PC_LAUNCH_CHECK();
  return PC_OK;
}
