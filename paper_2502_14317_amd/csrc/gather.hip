// KV compaction gather (Eq. 7: K_r = K_x[kept], V_r = V_x[kept]).
//
// HBM-bound byte copy.  One head row is D bf16 = 128 or 256 bytes; a lane moves one 16-byte
// piece of a K row and the matching piece of the V row, so D/8 adjacent lanes read one
// contiguous row and a wavefront writes 1 KiB of contiguous destination per store.  A wavefront
// stays inside one destination segment (b, s, g), so that everything but the token index is a
// scalar; a thread handles UNROLL rows, so that several independent loads are in flight (4; 2 where
// the last of a segment's wavefronts would idle for more than an eighth of its rows; 1 where 4 leave
// CUs without a workgroup).  The source is touched once here, so its loads carry the non-temporal hint.  The
// rows are read next (by the attention or the quantisation), so as many as the last-level cache holds are stored
// without it: 67 MB 25.7 -> 24.8 us, 201 MB 72 -> 65, 268 MB 91.5 -> 81 and up to 2 % off the layers behind it
// (a short one: 250 -> 243); more than that with it: 524 MB 175 us, 198 without.
// Measured with 64 x 16 x 8 segments of k rows, segments packed row by row / a workgroup (64 rows of 128
// values) inside one segment / a wavefront inside one (us): k = 1 7.6 / 9.7 / 6.3, 65 99 / 130 / 94, 100
// 147 / 172 / 147, 128 201 / 198 / 195; rows of 64 values, k = 100 78 / 84 / 73, 129 99 / 147 / 93, 200 148 /
// 189 / 147; with the maxima k = 65 2197 / 136 / 99 (packed, a row updates its segment by itself).  A
// workgroup whose rows end just behind a segment's multiple is all but idle, and packed rows cost four
// divisions each.
#include "pc_common.h"

// largest bf16 magnitude (15-bit pattern) among the 8 values of a 16-byte piece
__device__ __forceinline__ uint32_t pc_piece_amax(uint4 x) {
  const uint32_t w[4] = {x.x, x.y, x.z, x.w};
  uint32_t m = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) m = max(m, max(w[e] & 0x7fffu, (w[e] >> 16) & 0x7fffu));
  return m;
}

// AMAX: also leave, per destination segment (b, s, g), the largest |value| of its K rows and of
// its V rows (as fp32 bit patterns, so an integer maximum orders them): what a later
// quantisation of the compacted cache needs, taken while the rows are in flight.  The maxima
// must start at zero (amax_clear_kernel); an integer maximum does not depend on the order of
// the updates, so the result is deterministic.  Updates of one cache line follow each other at about 10 ns
// (32 segments share one), so a workgroup makes one per segment that it holds: 256 segments of 2048 rows of
// 128 values, an update per wavefront 135 us, now 87 (without maxima 85); a look at the value so far in front
// of the update 153 (asked for with the rows) and 754 (behind them).
template <int LANES_PER_ROW, bool AMAX, int UNROLL>
__global__ __launch_bounds__(256) void gather_kv_kernel(
    const uint4* __restrict__ k_src, const uint4* __restrict__ v_src,
    const int32_t* __restrict__ chunk_idx, const int32_t* __restrict__ tok_idx,
    uint4* __restrict__ k_dst, uint4* __restrict__ v_dst,
    int n_chunks, int rows, int n_sel, int n_kv_heads, int k, unsigned units_per_seg, unsigned n_units,
    uint32_t* __restrict__ k_amax, uint32_t* __restrict__ v_amax, int keep) {
  __shared__ uint32_t red[AMAX ? 4 : 1][3];                     // per wavefront: segment, maxima
  constexpr int ROWS = PC_WAVE / LANES_PER_ROW;                 // rows of a wavefront per step
  const int piece = threadIdx.x % LANES_PER_ROW;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / PC_WAVE);
  const unsigned unit = blockIdx.x * 4 + (unsigned)wave;
  if (!AMAX && unit >= n_units) return;
  const unsigned bsg = min(unit, n_units - 1) / units_per_seg;  // ((b * n_sel + s) * H_kv + g)
  const int first = (int)(unit % units_per_seg) * (ROWS * UNROLL) + (int)(threadIdx.x % PC_WAVE) / LANES_PER_ROW;
  const int g = (int)(bsg % (unsigned)n_kv_heads);
  const unsigned bs = bsg / (unsigned)n_kv_heads;
  const int s = (int)(bs % (unsigned)n_sel), b = (int)(bs / (unsigned)n_sel);
  const int c = chunk_idx ? chunk_idx[bs] : s;
  const bool write = c >= 0 && unit < n_units;                  // c < 0: destination segment without a source chunk
  if (!AMAX && !write) return;
  const bool have = write && c < n_chunks;
  const long long dst0 = (long long)bsg * k;
  const long long src0 = ((long long)b * n_chunks + c) * rows * n_kv_heads + g;

  uint4 kv[UNROLL], vv[UNROLL];
#pragma unroll
  for (int u = 0; u < UNROLL; ++u) {
    const int r = first + u * ROWS;
    kv[u] = make_uint4(0, 0, 0, 0);
    vv[u] = make_uint4(0, 0, 0, 0);
    const int t = have && r < k ? tok_idx[dst0 + r] : -1;
    if (t >= 0 && t < rows) {
      const long long src = (src0 + (long long)t * n_kv_heads) * LANES_PER_ROW + piece;
      kv[u] = pc_load_once(k_src + src);
      vv[u] = pc_load_once(v_src + src);
    }
  }
#pragma unroll
  for (int u = 0; u < UNROLL; ++u) {
    const int r = first + u * ROWS;
    if (write && r < k) {
      uint4* kd = k_dst + (dst0 + r) * LANES_PER_ROW + piece;
      uint4* vd = v_dst + (dst0 + r) * LANES_PER_ROW + piece;
      if (keep) { *kd = kv[u]; *vd = vv[u]; } else { pc_store_once(kd, kv[u]); pc_store_once(vd, vv[u]); }
    }
  }
  if (AMAX) {
    // over the thread's rows (those behind k are zeros), the wavefront, then its neighbours in the same segment
    uint32_t mk = 0, mv = 0;
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) { mk = max(mk, pc_piece_amax(kv[u])); mv = max(mv, pc_piece_amax(vv[u])); }
#pragma unroll
    for (int off = PC_WAVE / 2; off > 0; off >>= 1) {
      mk = max(mk, (uint32_t)__shfl_xor((int)mk, off));
      mv = max(mv, (uint32_t)__shfl_xor((int)mv, off));
    }
    if (threadIdx.x % PC_WAVE == 0) { red[wave][0] = bsg; red[wave][1] = mk; red[wave][2] = mv; }
    __syncthreads();
    if (threadIdx.x % PC_WAVE == 0 && (wave == 0 || red[wave - 1][0] != bsg)) {
      for (int w = wave + 1; w < 4 && red[w][0] == bsg; ++w) { mk = max(mk, red[w][1]); mv = max(mv, red[w][2]); }
      if (mk) atomicMax(k_amax + bsg, mk << 16);
      if (mv) atomicMax(v_amax + bsg, mv << 16);
    }
  }
}

// zero the maxima of the segments the gather is about to fill (those with a source chunk)
__global__ void amax_clear_kernel(const int32_t* __restrict__ chunk_idx, long long n_bs, int n_kv_heads,
                                  uint32_t* __restrict__ k_amax, uint32_t* __restrict__ v_amax) {
  const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;      // (b, s, g)
  if (i >= n_bs * n_kv_heads) return;
  if (chunk_idx && chunk_idx[i / n_kv_heads] < 0) return;
  k_amax[i] = 0u; v_amax[i] = 0u;
}

int pc_launch_gather(const void* k_src, const void* v_src, const int32_t* chunk_idx,
                     const int32_t* tok_idx, int batch, int n_chunks, int rows, int n_sel,
                     int n_kv_heads, int k, int head_dim, void* k_dst, void* v_dst,
                     float* k_amax, float* v_amax, hipStream_t st) {
  const long long n_dst_rows = (long long)batch * n_sel * n_kv_heads * k;
  if (n_dst_rows == 0) return PC_OK;
  const bool amax = k_amax != nullptr;
  if (amax) {
    const long long n = (long long)batch * n_sel * n_kv_heads;
    hipLaunchKernelGGL(amax_clear_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, chunk_idx,
                       (long long)batch * n_sel, n_kv_heads, (uint32_t*)k_amax, (uint32_t*)v_amax);
    PC_LAUNCH_CHECK();
  }
  const int lanes = head_dim / 8;
  const long long n_segs = (long long)batch * n_sel * n_kv_heads;
  const int step = PC_WAVE / lanes;                             // rows of a wavefront per step
  int unroll = n_segs * ((k + 4 * step - 1) / (4 * step)) < 4 * 512 ? 1 : 4;
  if (unroll == 4 && (k + 4LL * step - 1) / (4 * step) * (4 * step) * 8 > k * 9LL) unroll = 2;
  const long long units_per_seg = (k + (long long)unroll * step - 1) / (unroll * step);
  const long long units = n_segs * units_per_seg;               // wavefronts
  if (units > 0xffffffffLL) return PC_ERR_SHAPE;
  dim3 grid((unsigned)((units + 3) / 4)), block(256);
  const int keep = 4LL * head_dim * n_dst_rows <= (256LL << 20);      // bytes of K and V against the last-level cache
  PcProfScope prof(PC_KERNEL_GATHER, st);
#define PC_GATHER_LAUNCH(LANES, AMAX, UNROLL)                                                        \
  hipLaunchKernelGGL((gather_kv_kernel<LANES, AMAX, UNROLL>), grid, block, 0, st, (const uint4*)k_src, \
                     (const uint4*)v_src, chunk_idx, tok_idx, (uint4*)k_dst, (uint4*)v_dst, n_chunks, \
                     rows, n_sel, n_kv_heads, k, (unsigned)units_per_seg, (unsigned)units, (uint32_t*)k_amax, (uint32_t*)v_amax, keep)
#define PC_GATHER_PICK(LANES)                                                                        \
  if (amax) { if (unroll == 4) PC_GATHER_LAUNCH(LANES, true, 4); else if (unroll == 2) PC_GATHER_LAUNCH(LANES, true, 2); else PC_GATHER_LAUNCH(LANES, true, 1); } \
  else { if (unroll == 4) PC_GATHER_LAUNCH(LANES, false, 4); else if (unroll == 2) PC_GATHER_LAUNCH(LANES, false, 2); else PC_GATHER_LAUNCH(LANES, false, 1); }
  if (lanes == 16) { PC_GATHER_PICK(16) } else { PC_GATHER_PICK(8) }
#undef PC_GATHER_PICK
#undef PC_GATHER_LAUNCH
  PC_LAUNCH_CHECK();
  return PC_OK;
}
