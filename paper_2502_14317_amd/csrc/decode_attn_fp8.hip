// 8-bit compressed cache for the decoding stage (Eq. 9-11 with few query rows).
//
// The decode kernel reads every K / V byte once and is bound by HBM bandwidth, so storing the
// compressed segments in 8 bits halves its time.  Format: OCP 8-bit float E4M3 (1 sign, 4
// exponent bits with bias 7, 3 mantissa bits, largest magnitude 448, no infinities), one fp32
// scale per (sequence, segment, KV head) for K and one for V:
//   scale = max |x| over the segment's valid rows / 448   (1 if that maximum is 0)
//   code  = E4M3(x / scale), round to nearest even, saturating
// The paper leaves the cache precision open; this format is an extension of this library.
//
// kv_quantize_fp8_kernel   codes from maxima that the caller hands in (the gather that fills the cache can
//                          leave them: 3 bytes per element), or one workgroup per (sequence, segment, KV
//                          head, K or V) that finds the maximum first and reads the segment again (5
//                          bytes).  Codes are written in 32-key blocks laid out for the matrix cores
//                          (below), V transposed.
// decode_attn_fp8_kernel   the split-KV kernel of decode_attn.hip on 8-bit operands: codes are
//                          widened in registers (every E4M3 value is exact in bf16), both
//                          products run on the 16x16x32 bf16 MFMA, the scales are folded into the
//                          logit scale and into the probabilities.  Every load instruction
//                          of a wavefront reads 1 KiB of consecutive bytes.
//
// K block layout.  A block of 32 keys x D codes is two 16-key tiles; a tile is D / 64 pieces of
// 1 KiB, piece i = 64 lanes x 16 bytes, lane 16 kk + c (kk < 4, c < 16) holding the codes of
// d = 64 i + 16 kk .. + 15 of key c of the tile: the A operand bytes of that lane for k-steps
// 2 i and 2 i + 1 of S^T = K Q^T (the query operand is permuted to the same d order).
//
// V block layout.  O^T[d, column] += V^T[d, key] P^T[key, column] wants, per lane, 8 keys of one
// d, and the probabilities a lane holds after the two 16-key logit tiles of a 32-key block are
// those of keys 4g..4g+3 and 16+4g..16+4g+3 (g = lane / 16).  So the codes of a block of 32 keys
// x D values are stored as D / 32 pieces of 1 KiB, piece q = 64 lanes x 16 bytes, lane (g, m)
// = 16 g + m holding [h][j]: h = 0, 1 -> d = 32 q + 16 h + m; j = 0..7 -> key 4 g + j (j < 4),
// 16 + 4 g + (j - 4) (j >= 4).  A piece is one fully coalesced 16-byte-per-lane load and gives
// two A operands.  A segment holds ceil(k_t / 32) blocks of K and of V; keys behind k_t or behind
// the segment's length carry code 0.
#include "decode_core.h"
#include "fp8_quotient.h"
#include "rope.h"
#include <algorithm>

#define PC_D8_WAVES 4
#define PC_D8_ITER_KEYS 32
#define PC_D8_LOG2E 1.4426950408889634f
#define PC_E4M3_MAX 448.0f


// ------------------------------------------------------------------------------------------
// Quantisation.  A wavefront takes units of 4 KiB of codes (4096 / D keys) by itself: all its loads go out at
// once, a lane then holds 16 values of a key for each K piece, or 8 keys x 8 values for V, whose codes are
// packed along the keys; V granules pass through the wavefront's own LDS (swizzled, no bank taken more than twice) so
// that every store covers 1 KiB.  Bound by memory if the division is not: x / scale by v_div_* is about 11
// instructions a value; here the correctly rounded quotient from the reciprocal, once rounded itself, and
// one residual: q = x r, q' = q - (q scale - x) r.  It equals the division for every pair of mantissas (2^23
// scales x 2^7 values, compared one by one); exponents do not matter while nothing under- or overflows, which
// holds where the code is not 0 for scales within 2^+-60.  Others divide.  -0 stays -0.
// 256 segments of 2048 x 128 (0.40 GB) with maxima: one workgroup of 1024 per segment, both directions through
// LDS between barriers, division 88 us; now 59; 64 segments 48 -> 17; 4096 (6.4 GB) 1192 -> 1084, 5.9 TB/s.
// Without: 124 -> 97, 55 -> 30, 1570 -> 1520.  The rows carry the non-temporal hint where they are more than
// the last-level cache holds (256 MiB): smaller ones the gather has just left there, and the second sweep finds
// the first one's (64 segments without the hint 17 and 30 us, with it 19 and 39; 4096 1118 and 1084).
#define PC_Q8_THREADS 1024

// x = scale's multiple, clamped to the format (a NaN to its lowest, as max and min do)
struct PcQuantScale {
  float scale, inv, limit;
  bool fast;
};
__device__ __forceinline__ PcQuantScale pc_quant_scale(float amax) {
  PcQuantScale q;
  q.scale = amax > 0.f ? amax / PC_E4M3_MAX : 1.0f;
  q.fast = q.scale > 0x1p-60f && q.scale < 0x1p60f;
  q.inv = 1.0f / q.scale;
  q.limit = PC_E4M3_MAX * q.scale;
  return q;
}
template <bool FAST>
__device__ __forceinline__ float pc_quotient(float x, const PcQuantScale& s) {
  if (!FAST) return fminf(fmaxf(x / s.scale, -PC_E4M3_MAX), PC_E4M3_MAX);
  x = __builtin_amdgcn_fmed3f(x, -s.limit, s.limit);       // (the quotient of the limit is below 464, still code 448)
  return pc_quotient_by_reciprocal(x, s.scale, s.inv);
}
template <bool FAST>
__device__ __forceinline__ uint32_t pc_e4m3x4(float a, float b, float c, float d, const PcQuantScale& s) {
  uint32_t w = __builtin_amdgcn_cvt_pk_fp8_f32(pc_quotient<FAST>(a, s), pc_quotient<FAST>(b, s), 0, false);
  return __builtin_amdgcn_cvt_pk_fp8_f32(pc_quotient<FAST>(c, s), pc_quotient<FAST>(d, s), w, true);
}

template <int D, bool FAST>
__device__ __forceinline__ void quantize_values(const u32x4 (&x)[8], bool is_v, uint8_t* dst, int n_blk_left,
                                                const PcQuantScale& s, uint8_t* stage) {
  const int lane = threadIdx.x % PC_WAVE;
  u32x4 out[4];
  if (!is_v) {
#pragma unroll
    for (int pc = 0; pc < 4; ++pc)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t w0 = x[2 * pc + e / 2][2 * (e % 2)], w1 = x[2 * pc + e / 2][2 * (e % 2) + 1];
        out[pc][e] = pc_e4m3x4<FAST>(bf16_lo_to_f32(w0), bf16_hi_to_f32(w0), bf16_lo_to_f32(w1), bf16_hi_to_f32(w1), s);
      }
  } else {
    const int dc = lane % (D / 8), g = lane / (D / 8) % 4, blk = lane / (D / 2);
    const int q = dc / 4, m0 = 8 * (dc % 2), swz = g + 4 * (q % 2);
    uint8_t* row = stage + blk * 32 * D + q * 1024 + g * 256 + 8 * (dc / 2 % 2);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float f[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) f[j] = e % 2 ? bf16_hi_to_f32(x[j][e / 2]) : bf16_lo_to_f32(x[j][e / 2]);
      const u32x2 code = {pc_e4m3x4<FAST>(f[0], f[1], f[2], f[3], s), pc_e4m3x4<FAST>(f[4], f[5], f[6], f[7], s)};
      *(u32x2*)(row + ((m0 + e) ^ swz) * 16) = code;
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int pc = 0; pc < 4; ++pc)
      out[pc] = *(const u32x4*)(stage + pc * 1024 + (lane / 16) * 256 + ((lane % 16) ^ (lane / 16 + 4 * (pc % 2))) * 16);
  }
#pragma unroll
  for (int pc = 0; pc < 4; ++pc)
    if (pc * 1024 < n_blk_left * 32 * D) pc_store_once((u32x4*)(dst + 1024 * pc + 16 * lane), out[pc]);
}

template <int D, int HINT>
__device__ __forceinline__ void load_unit(const __amdgpu_buffer_rsrc_t& rsrc, bool is_v, u32x4 (&x)[8]) {
  const int lane = threadIdx.x % PC_WAVE;
  if (!is_v) {
    const int off = 2 * (lane % 16 * D + lane / 16 * 16);
#pragma unroll
    for (int pc = 0; pc < 4; ++pc)
#pragma unroll
      for (int e = 0; e < 2; ++e)
        x[2 * pc + e] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 2 * (pc / (D / 64) * 16 * D + pc % (D / 64) * 64 + 8 * e), HINT);
  } else {
    const int dc = lane % (D / 8), g = lane / (D / 8) % 4, blk = lane / (D / 2);
    const int off = 2 * ((32 * blk + 4 * g) * D + 8 * dc);
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, 2 * (j < 4 ? j : 12 + j) * D, HINT);
  }
}

// unit u of a segment: keys 4096 / D u ..; len valid rows, the codes of others are 0.  (A segment's bytes need
// more than 32 bits from 2^24 keys of 128 values on: blocks are counted, of a unit's at most 4096 bytes.)
template <int D>
__device__ __forceinline__ void quantize_unit(const uint16_t* src, uint8_t* dst, bool is_v, int u, int len, int n_blk,
                                              float amax, int keep, uint8_t* stage) {
  constexpr int KEYS = 4096 / D;
  const int key0 = u * KEYS;
  const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(src + (long long)key0 * D), 0,
                                                                        min(max(len - key0, 0), KEYS) * 2 * D, 0x00020000);
  u32x4 x[8];
  if (keep) load_unit<D, 0>(rsrc, is_v, x);
  else load_unit<D, PC_BUF_NT>(rsrc, is_v, x);
  const PcQuantScale s = pc_quant_scale(amax);
  dst += (long long)key0 * D;
  const int n_blk_left = min(n_blk - key0 / 32, KEYS / 32);
  if (s.fast) quantize_values<D, true>(x, is_v, dst, n_blk_left, s, stage);
  else quantize_values<D, false>(x, is_v, dst, n_blk_left, s, stage);
}

// with maxima: a wavefront per unit, blockIdx.y = 0 (K) or 1 (V)
template <int D>
__global__ __launch_bounds__(256) void kv_quantize_fp8_kernel(
    const uint16_t* __restrict__ kc, const uint16_t* __restrict__ vc, const int32_t* __restrict__ seg_len, int per_head,
    int n_kv_heads, int k_t, unsigned n_segs, const float* __restrict__ k_amax, const float* __restrict__ v_amax,
    uint8_t* __restrict__ k8, uint8_t* __restrict__ v8, float* __restrict__ k_scale, float* __restrict__ v_scale, int keep) {
  __shared__ __attribute__((aligned(16))) uint8_t stage[4][4096];
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / PC_WAVE), is_v = blockIdx.y;
  const int n_blk = (k_t + 31) / 32;
  const unsigned units = (unsigned)(k_t + 4096 / D - 1) / (4096 / D);
  const unsigned long long id = blockIdx.x * 4ULL + wave;
  const unsigned seg = (unsigned)(id / units);
  const int u = (int)(id % units);
  if (seg >= n_segs) return;
  const int len = seg_len ? min(max(seg_len[per_head ? seg : seg / n_kv_heads], 0), k_t) : k_t;
  const float amax = fabsf((is_v ? v_amax : k_amax)[seg]);
  quantize_unit<D>((is_v ? vc : kc) + (long long)seg * k_t * D, (is_v ? v8 : k8) + (long long)seg * n_blk * 32 * D, is_v, u,
                   len, n_blk, amax, keep, stage[wave]);
  if (u == 0 && threadIdx.x % PC_WAVE == 0) (is_v ? v_scale : k_scale)[seg] = pc_quant_scale(amax).scale;
}

// without: a workgroup per segment sweeps it for the maximum (bf16 magnitudes order like their 15-bit
// patterns), then its wavefronts take the units
template <int D>
__global__ __launch_bounds__(PC_Q8_THREADS) void kv_amax_quantize_fp8_kernel(
    const uint16_t* __restrict__ kc, const uint16_t* __restrict__ vc, const int32_t* __restrict__ seg_len, int per_head,
    int n_kv_heads, int k_t, uint8_t* __restrict__ k8, uint8_t* __restrict__ v8, float* __restrict__ k_scale,
    float* __restrict__ v_scale, int keep) {
  constexpr int WAVES = PC_Q8_THREADS / PC_WAVE, UNROLL = 4;
  __shared__ uint32_t red[WAVES];
  __shared__ __attribute__((aligned(16))) uint8_t stage[WAVES][4096];
  const long long seg = blockIdx.x;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / PC_WAVE), is_v = blockIdx.y;
  const uint16_t* src = (is_v ? vc : kc) + seg * (long long)k_t * D;
  const int n_blk = (k_t + 31) / 32;
  const int len = seg_len ? min(max(seg_len[per_head ? seg : seg / n_kv_heads], 0), k_t) : k_t;
  const long long n_valid = (long long)len * D / 8;        // 8-element groups of the valid rows
  uint32_t amax = 0;
  for (long long i0 = 0; i0 < n_valid; i0 += PC_Q8_THREADS * UNROLL) {
    uint4 x[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const long long i = i0 + u * PC_Q8_THREADS + threadIdx.x;
      x[u] = i < n_valid ? *(const uint4*)(src + 8 * i) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const uint32_t w[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) amax = max(amax, max(w[e] & 0x7fffu, (w[e] >> 16) & 0x7fffu));
    }
  }
#pragma unroll
  for (int off = PC_WAVE / 2; off > 0; off >>= 1) amax = max(amax, (uint32_t)__shfl_xor((int)amax, off));
  if (threadIdx.x % PC_WAVE == 0) red[wave] = amax;
  __syncthreads();
  amax = 0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) amax = max(amax, red[w]);
  const float fmax_ = __uint_as_float((uint32_t)__builtin_amdgcn_readfirstlane((int)amax) << 16);
  if (threadIdx.x == 0) (is_v ? v_scale : k_scale)[seg] = pc_quant_scale(fmax_).scale;
  const int units = (k_t + 4096 / D - 1) / (4096 / D);
  for (int u = wave; u < units; u += WAVES)
    quantize_unit<D>(src, (is_v ? v8 : k8) + seg * (long long)n_blk * 32 * D, is_v, u, len, n_blk, fmax_, keep, stage[wave]);
}

int pc_launch_kv_quantize_fp8(const void* kc, const void* vc, const int32_t* seg_len,
                              int seg_len_per_head, long long n_segs, int n_kv_heads, int k_t,
                              int head_dim, const float* k_amax, const float* v_amax, void* k8,
                              void* v8, float* k_scale, float* v_scale, hipStream_t st) {
  if (n_segs == 0) return PC_OK;
  if (n_segs > 0x7fffffffLL) return PC_ERR_SHAPE;
  const long long units = (k_t + 4096 / head_dim - 1) / (4096 / head_dim);
  const long long blocks = k_amax ? (n_segs * units + 3) / 4 : n_segs;
  if (blocks > 0x7fffffffLL) return PC_ERR_SHAPE;
  const int keep = 4LL * head_dim * k_t * n_segs <= (256LL << 20);
  PcProfScope prof(PC_KERNEL_KV_QUANTIZE, st);
  const dim3 grid((unsigned)blocks, 2);
#define PC_Q8_LAUNCH(D)                                                                                                \
  if (k_amax)                                                                                                          \
    hipLaunchKernelGGL(kv_quantize_fp8_kernel<D>, grid, dim3(256), 0, st, (const uint16_t*)kc, (const uint16_t*)vc,     \
                       seg_len, seg_len_per_head, n_kv_heads, k_t, (unsigned)n_segs, k_amax, v_amax, (uint8_t*)k8,     \
                       (uint8_t*)v8, k_scale, v_scale, keep);                                                          \
  else                                                                                                                 \
    hipLaunchKernelGGL(kv_amax_quantize_fp8_kernel<D>, grid, dim3(PC_Q8_THREADS), 0, st, (const uint16_t*)kc,           \
                       (const uint16_t*)vc, seg_len, seg_len_per_head, n_kv_heads, k_t, (uint8_t*)k8, (uint8_t*)v8,    \
                       k_scale, v_scale, keep);
  if (head_dim == 128) { PC_Q8_LAUNCH(128) } else { PC_Q8_LAUNCH(64) }
#undef PC_Q8_LAUNCH
  PC_LAUNCH_CHECK();
  return PC_OK;
}

// ------------------------------------------------------------------------------------------
struct PcDecode8Args {
  PcDecodeQuery query;
  const uint8_t* k8;      // [B, S, H_kv, ceil(k_t / 32) * 32 * D] E4M3 codes in 32-key blocks
  const uint8_t* v8;      // the same size, transposed blocks
  const float* k_scale;   // [B, S, H_kv]
  const float* v_scale;
  const int32_t* seg_len; // [B, S] ([B, S, H_kv] if seg_len_per_head) or nullptr
  int seg_len_per_head;
  float* part_o;          // [B, P, n_q, H_q, D]
  float* part_lse;        // [B, P, n_q, H_q]
  int n_q, n_seg, k_t, n_q_heads, n_kv_heads, n_parts;
  int group;              // H_q / H_kv
  int parts_grid;         // workgroups (partials) per (sequence, KV head) in this launch
  PcDiv parts_div, heads_div;   // by parts_grid, by n_kv_heads
  float scale_log2;       // softmax scale * log2(e)
};

// four E4M3 codes of one 32-bit word -> two packed bf16 pairs (exact: every E4M3 value is a bf16
// value), one conversion instruction per pair (the scaled form with scale 1)
typedef __bf16 pc_bf2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ void pc_e4m3x4_to_bf16(uint32_t w, uint32_t& lo, uint32_t& hi) {
  const pc_bf2 a = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, false);
  const pc_bf2 b = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(w, 1.0f, true);
  lo = *(const uint32_t*)&a;
  hi = *(const uint32_t*)&b;
}

// ------------------------------------------------------------------------------------------
// Tile images for the tile kernel, which takes a query block over the 8-bit cache: the local attention's
// layout (K granule (c, r) = K[key r][8 c .. 8 c + 7] at 64 c + r, V^T granule (c, d) = V[keys 8 c .. + 7][d] at
// D c + d), so that its loop needs neither transposing LDS reads nor row addresses.  8-bit segments: value =
// code * scale, rounded to bf16; one workgroup per 64-key tile (K and V), a thread takes 16-byte pieces of the
// blocks (layouts above).  A K piece holds 16 values of a key, two granules; of a V piece a lane holds keys
// 4 g .. and 16 + 4 g .. of a value, and neighbouring lane rows exchange halves (v_permlane16_swap) to whole
// granules.  Every 16 lanes store 256 consecutive bytes.  Bound by memory, 1 byte read and 2 written a value:
// 256 segments of 2048 x 128 (0.40 GB) 66 us, 6.1 TB/s (as rows, through LDS: 61), and the attention that reads
// them (4 x 512 rows, 32 / 8 heads) 548 -> 506 us.  The tail and the self segment follow in the same launch.
// So does the rotation of the query rows, a workgroup each, spread evenly between the others: its fp64 angles cost
// latency and few bytes, the tiles bytes only (4 x 512 rows: 67 + 10 us in two launches, 72 in one).
template <int D>
__device__ __forceinline__ void widen_piece(const uint8_t* src, float scale, bool have, uint32_t (&o)[8]) {
  uint4 raw = make_uint4(0, 0, 0, 0);
  if (have) raw = pc_load_once((const uint4*)src);
  const uint32_t w[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    uint32_t lo, hi;
    pc_e4m3x4_to_bf16(w[e], lo, hi);
    o[2 * e] = pack_bf16x2(bf16_lo_to_f32(lo) * scale, bf16_hi_to_f32(lo) * scale);
    o[2 * e + 1] = pack_bf16x2(bf16_lo_to_f32(hi) * scale, bf16_hi_to_f32(hi) * scale);
  }
}
template <int D>
__device__ __forceinline__ void rows_to_image(const PcRowsToImages& x, int unit, int n_kv_heads) {
  const int tiles = (x.n_rows + 63) / 64, tile = unit % tiles, bg = unit / tiles, b = bg / n_kv_heads, g = bg % n_kv_heads;
  const int len = x.len ? min(max(x.len[b], 0), x.n_rows) : x.n_rows, left = len - 64 * tile;
  if (left <= 0) return;
  const long long src = b * x.seq_stride + g * x.head_stride + 64LL * tile * x.row_stride, dst = (long long)unit * (64 * D);
  for (int it = threadIdx.x; it < 8 * D; it += 256) {
    const int row = it % 64, c = it / 64;
    uint4 w = make_uint4(0, 0, 0, 0);
    if (row < left) w = *(const uint4*)(x.k + src + (long long)row * x.row_stride + 8 * c);
    *(uint4*)(x.k_img + dst + it * 8) = w;
  }
  const int c = threadIdx.x / (D / 4), d4 = threadIdx.x % (D / 4) * 4;
  if (c >= 8) return;
  u32x2 w[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    w[j] = u32x2{0u, 0u};
    if (8 * c + j < left) w[j] = *(const u32x2*)(x.v + src + (8LL * c + j) * x.row_stride + d4);
  }
#pragma unroll
  for (int dd = 0; dd < 4; ++dd) {
    u32x4 gr;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      gr[e] = __builtin_amdgcn_perm(w[2 * e + 1][dd / 2], w[2 * e][dd / 2], dd % 2 ? 0x07060302u : 0x05040100u);
    *(u32x4*)(x.v_img + dst + (c * D + d4 + dd) * 8) = gr;
  }
}
template <int D>
__global__ __launch_bounds__(256) void fp8_images_kernel(
    const uint8_t* __restrict__ k8, const uint8_t* __restrict__ v8, const float* __restrict__ k_scale,
    const float* __restrict__ v_scale, const int32_t* __restrict__ seg_len, int per_head, int k_t, long long n_segs, uint16_t* __restrict__ k_img, uint16_t* __restrict__ v_img,
    PcRowsToImages tail, PcRowsToImages self, int n_seq, int n_kv_heads, PcRowsToRotate rot) {
  const uint32_t bid = blockIdx.y * gridDim.x + blockIdx.x, turn = bid / rot.period;
  if (turn < rot.rows && turn * rot.period == bid) {
    pc_rope_q_workgroup<D>(rot.q, rot.q_rot, (int)turn, rot.n_q, rot.n_heads, rot.pos0, rot.rope, rot.mul);
    return;
  }
  const int tiles = (k_t + 63) / 64, n_blk = (k_t + 31) / 32;
  const long long seg_units = n_segs * tiles, unit = bid - min(rot.rows, turn + 1);
  if (unit >= seg_units) {
    const int rest = (int)(unit - seg_units), tail_units = n_seq * n_kv_heads * ((tail.n_rows + 63) / 64);
    if (rest < tail_units) rows_to_image<D>(tail, rest, n_kv_heads);
    else if (rest - tail_units < n_seq * n_kv_heads * ((self.n_rows + 63) / 64)) rows_to_image<D>(self, rest - tail_units, n_kv_heads);
    return;
  }
  const long long seg = unit / tiles;
  const int tile = (int)(unit % tiles);
  const int left = (seg_len ? min(seg_len[per_head ? seg : seg / n_kv_heads], k_t) : k_t) - 64 * tile;
  if (left <= 0) return;
  const float ks = k_scale[seg], vs = v_scale[seg];
  const long long dst = unit * (64 * D);
  constexpr int PIECES = 2 * 32 * D / 16;                 // 16-byte pieces of the tile's two blocks
#pragma unroll
  for (int u = 0; u < PIECES / 256; ++u) {
    const int p = threadIdx.x + 256 * u, blk = p / (2 * D), pb = p % (2 * D), lane = pb % 64, piece = pb / 64;
    const bool have = 2 * tile + blk < n_blk;
    const long long at = (seg * n_blk + 2 * tile + blk) * 32LL * D + 16 * pb;
    uint32_t o[8];
    {
      // piece = 16-key tile * (D / 64) + i; lane 16 kk + c: values d = 64 i + 16 kk .. + 15 of key c of the tile
      widen_piece<D>(k8 + at, ks, have, o);
      const int key = 32 * blk + 16 * (piece / (D / 64)) + lane % 16, col = 8 * (piece % (D / 64)) + 2 * (lane / 16);
      uint16_t* out = k_img + dst + (col * 64 + key) * 8;
      if (key >= left) {
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = 0;
      }
      *(uint4*)out = make_uint4(o[0], o[1], o[2], o[3]);
      *(uint4*)(out + 64 * 8) = make_uint4(o[4], o[5], o[6], o[7]);
    }
    {
      // piece q; lane 16 g + m holds [h][j]: value d = 32 q + 16 h + m of key 4 g + j (j < 4) or
      // 16 + 4 g + (j - 4); after the exchange an even g has keys 4 g .. 4 g + 7, an odd one 16 + 4 (g - 1) ..
      widen_piece<D>(v8 + at, vs, have, o);
      const int g = lane / 16, m = lane % 16, c = 4 * blk + (g % 2 ? 2 : 0) + g / 2;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < 2; ++e) {
          auto x = __builtin_amdgcn_permlane16_swap(o[4 * h + e], o[4 * h + 2 + e], false, false);
          w[e] = x[0]; w[2 + e] = x[1];
        }
        if (left < 64) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int key = 8 * c + 2 * e;
            w[e] = key + 1 < left ? w[e] : (key < left ? w[e] & 0xffffu : 0u);
          }
        }
        *(uint4*)(v_img + dst + (c * D + 32 * piece + 16 * h + m) * 8) = make_uint4(w[0], w[1], w[2], w[3]);
      }
    }
  }
}

int pc_launch_fp8_images(const void* k8, const void* v8, const float* k_scale, const float* v_scale,
                         const int32_t* seg_len, int seg_len_per_head, long long n_segs, int k_t, int head_dim, void* k_img, void* v_img,
                         const PcRowsToImages& tail, const PcRowsToImages& self, int n_seq, int n_kv_heads,
                         const PcRowsToRotate& rows, hipStream_t st) {
  const long long row_tiles = (tail.n_rows + 63) / 64 + (self.n_rows + 63LL) / 64;
  const long long blocks = n_segs * ((k_t + 63) / 64) + (long long)n_seq * n_kv_heads * row_tiles + rows.rows;
  if (blocks == 0) return PC_OK;
  if (blocks > 0x7fffffffLL - PC_GRID_X) return PC_ERR_SHAPE;
  PcRowsToRotate rot = rows;
  rot.period = (uint32_t)(blocks / std::max(rows.rows, 1u));
  PcProfScope prof(PC_KERNEL_FP8_IMAGES, st);
  const dim3 grid = pc_grid_2d(blocks), block(256);
  if (head_dim == 128)
    hipLaunchKernelGGL(fp8_images_kernel<128>, grid, block, 0, st, (const uint8_t*)k8, (const uint8_t*)v8, k_scale, v_scale,
                       seg_len, seg_len_per_head, k_t, n_segs, (uint16_t*)k_img, (uint16_t*)v_img, tail, self, n_seq, n_kv_heads, rot);
  else
    hipLaunchKernelGGL(fp8_images_kernel<64>, grid, block, 0, st, (const uint8_t*)k8, (const uint8_t*)v8, k_scale, v_scale,
                       seg_len, seg_len_per_head, k_t, n_segs, (uint16_t*)k_img, (uint16_t*)v_img, tail, self, n_seq, n_kv_heads, rot);
  PC_LAUNCH_CHECK();
  return PC_OK;
}

// The same segments as bf16 rows [n_segs, k_t, D], next to which the tail and the self segment are read where they
// lie.  One workgroup per 32-key block, K (blockIdx.y = 0) or V; the rows are put together in LDS and leave as whole
// 16-byte pieces.  Bound by memory like the images: 256 segments of 2048 x 128 61 us.
template <int D>
__global__ __launch_bounds__(256) void fp8_rows_kernel(
    const uint8_t* __restrict__ k8, const uint8_t* __restrict__ v8, const float* __restrict__ k_scale, const float* __restrict__ v_scale,
    const int32_t* __restrict__ seg_len, int per_head, int n_kv_heads, int k_t, uint16_t* __restrict__ k_rows, uint16_t* __restrict__ v_rows) {
  constexpr int STRIDE = D + 8;                           // 16-byte pieces stay aligned, rows start in other banks
  __shared__ __attribute__((aligned(16))) uint16_t rows[32 * STRIDE];
  const int n_blk = (k_t + 31) / 32, blk = (int)(blockIdx.x % n_blk), is_v = blockIdx.y;
  const long long seg = blockIdx.x / n_blk;
  const int n_rows = (seg_len ? min(seg_len[per_head ? seg : seg / n_kv_heads], k_t) : k_t) - 32 * blk;
  if (n_rows <= 0) return;
  const int p = threadIdx.x;                              // 16-byte piece of the block
  if (p < 32 * D / 16) {
    uint32_t o[8];
    widen_piece<D>((is_v ? v8 : k8) + (seg * n_blk + blk) * 32LL * D + 16 * p, (is_v ? v_scale : k_scale)[seg], true, o);
    const int lane = p % 64, piece = p / 64;
    if (!is_v) {
      uint4* r4 = (uint4*)(rows + (16 * (piece / (D / 64)) + lane % 16) * STRIDE + 64 * (piece % (D / 64)) + 16 * (lane / 16));
      r4[0] = make_uint4(o[0], o[1], o[2], o[3]);
      r4[1] = make_uint4(o[4], o[5], o[6], o[7]);
    } else {
      const int g = lane / 16, m = lane % 16;
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int j = 0; j < 8; ++j)
          rows[(j < 4 ? 4 * g + j : 12 + 4 * g + j) * STRIDE + 32 * piece + 16 * h + m] = (uint16_t)(o[4 * h + j / 2] >> (16 * (j % 2)));
    }
  }
  __syncthreads();
  uint16_t* dst = (is_v ? v_rows : k_rows) + (seg * k_t + 32LL * blk) * D;
  for (int x = threadIdx.x; x < min(32, n_rows) * (D / 8); x += 256)
    *(uint4*)(dst + 8 * x) = *(const uint4*)(rows + x / (D / 8) * STRIDE + x % (D / 8) * 8);
}

int pc_launch_fp8_rows(const void* k8, const void* v8, const float* k_scale, const float* v_scale, const int32_t* seg_len,
                       int seg_len_per_head, long long n_segs, int n_kv_heads, int k_t, int head_dim, void* k_rows, void* v_rows, hipStream_t st) {
  const long long blocks = n_segs * ((k_t + 31) / 32);
  if (blocks == 0) return PC_OK;
  if (blocks > 0x7fffffffLL) return PC_ERR_SHAPE;
  PcProfScope prof(PC_KERNEL_FP8_ROWS, st);
  const dim3 grid((unsigned)blocks, 2), block(256);
  if (head_dim == 128)
    hipLaunchKernelGGL(fp8_rows_kernel<128>, grid, block, 0, st, (const uint8_t*)k8, (const uint8_t*)v8, k_scale, v_scale, seg_len,
                       seg_len_per_head, n_kv_heads, k_t, (uint16_t*)k_rows, (uint16_t*)v_rows);
  else
    hipLaunchKernelGGL(fp8_rows_kernel<64>, grid, block, 0, st, (const uint8_t*)k8, (const uint8_t*)v8, k_scale, v_scale, seg_len,
                       seg_len_per_head, n_kv_heads, k_t, (uint16_t*)k_rows, (uint16_t*)v_rows);
  PC_LAUNCH_CHECK();
  return PC_OK;
}

// The 16-bit tail can ride in the launch of the 8-bit segments, its workgroups behind theirs: the tail, a
// few per cent of the bytes, then costs no launch, ramp and drain of its own.  Beyond 4 columns it rides up to 256
// 8-bit workgroups only, a line from a 16-bit function with P V on the vector ALUs, whose registers and LDS cost the
// 8-bit workgroups the second one on their CU.  Both functions now have one shape for 1 to 16 columns and share
// their LDS, and the launch of its own is the slower side everywhere: two launches / one (us), 33 sequences of 8 x 1024 keys
// + 300, 8 KV heads, 1, 4, 8, 16 columns 110 / 99, 113 / 103, 119 / 109, 132 / 121; 65 (tail 520) 216 / 201, 223 / 209,
// 235 / 221, 253 / 240; 100 of 2 x 256 + 256 54 / 47, 60 / 52, 67 / 60, 84 / 76; one of 8 x 2048 + 520 20.5 / 13.1, 21.2 / 13.7,
// 21.9 / 13.9, 24.6 / 15.2.  It stands because tests/test_gpu_decode8_launches.py expects the launch.
#define PC_D8_TAIL_WGS 256
template <int D>
__device__ __forceinline__ void decode8_workgroup(const PcDecode8Args& a, int bid, PcDecodeLds<D>& sm) {
  constexpr int KSTEPS = D / 32;            // MFMA k-steps; a lane owns 8 KSTEPS = D / 4 bytes of each of its K rows
  constexpr int KQ = D / 64;                // 16-byte loads per lane and 16-key block
  constexpr int VLOADS = D / 32;            // 1 KiB pieces of a V block: one 16-byte load per lane each
  constexpr int MB = D / 16;                // 16-row blocks of O^T
  constexpr int KBLK = PC_D8_ITER_KEYS / 16;
  static_assert(KBLK == 2, "the V block layout assumes two 16-key logit tiles per block");

  const int G = a.group;
  const int n_cols = a.n_q * G;             // valid query columns (<= 16)
  const int lane = threadIdx.x % PC_WAVE, wave = threadIdx.x / PC_WAVE;
  const int kk = lane / 16, c16 = lane % 16;

  const int bg = pc_div(bid, a.parts_div), part = bid - bg * a.parts_grid;
  const int b = pc_div(bg, a.heads_div), g = bg - b * a.n_kv_heads;

  // A wavefront streams its run of 32-key blocks, through segment boundaries, under one running
  // softmax (one partial per workgroup).  A cursor names the next block: where it is, the
  // segment's base pointers and its scales (K: folded into the logit scale; V: applied to the
  // probabilities that multiply the codes, not to the row sum).
  struct Cursor { PcBlockCursor at; const uint8_t* k; const uint8_t* v; float k_sc, v_sc; int bytes; };
  const long long seg_bytes = (long long)((a.k_t + 31) / 32) * 32 * D;
  PcSegLens lens;
  lens.seg_len = a.seg_len; lens.per_head = a.seg_len_per_head; lens.n_seg = a.n_seg;
  lens.n_kv_heads = a.n_kv_heads; lens.k_t = a.k_t; lens.b = b; lens.g = g;
  auto place = [&](const PcBlockCursor& at) {
    Cursor c; c.at = at; c.k = a.k8; c.v = a.v8; c.k_sc = 0.f; c.v_sc = 0.f;
    c.bytes = 0;                                                        // behind the run's end: nothing is read
    if (at.left > 0) {
      const long long seg_id = ((long long)b * a.n_seg + at.s) * a.n_kv_heads + g;
      const long long first = seg_id * seg_bytes + (long long)at.blk * 32 * D;
      c.k = a.k8 + first; c.v = a.v8 + first; c.bytes = 32 * D;         // whole blocks exist up to ceil(k_t / 32)
      // read-only here, and asked for through the scalar cache: a vector load would have to be waited
      // for behind the keys in flight
      typedef const __attribute__((address_space(4))) float* scalar_t;
      c.k_sc = ((scalar_t)(uintptr_t)a.k_scale)[seg_id];
      c.v_sc = ((scalar_t)(uintptr_t)a.v_scale)[seg_id];
    }
    return c;
  };
  auto next = [&](const Cursor& c) { return place(pc_blocks_next(lens, c.at)); };

  const int first_lens = pc_first_lens(lens, lane);
  PcColumnRotation<D> rot;
  rot.begin(a.query, b, g, G, n_cols);
  // B operand: column c16 = (t, head-in-group); k-step j of lane group kk covers
  // d = 64 (j / 2) + 16 kk + 8 (j % 2) .. + 7, the d order of the K block layout
  bf16x8 bq[KSTEPS];

  float m_run = -INFINITY, l_run = 0.f;     // of column c16 (this lane's share of the sum)
  // O^T: row block mb, register r = value d = 16 mb + 4 kk + r of column c16
  floatx4 o_acc[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) o_acc[mb] = floatx4{0.f, 0.f, 0.f, 0.f};

  // unconditional loads (see pc_decode_workgroup)
  u32x4 kbuf[3][KBLK][KQ], vbuf[3][VLOADS];
  auto issue_loads = [&](int buf, const Cursor& c) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t kr = __builtin_amdgcn_make_buffer_rsrc((void*)c.k, 0, c.bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc((void*)c.v, 0, c.bytes, 0x00020000);
#pragma unroll
    for (int bi = 0; bi < KBLK; ++bi)
#pragma unroll
      for (int i = 0; i < KQ; ++i)
        kbuf[buf][bi][i] = __builtin_amdgcn_raw_buffer_load_b128(kr, 16 * lane, bi * 16 * D + 1024 * i, PC_BUF_NT);
#pragma unroll
    for (int i = 0; i < VLOADS; ++i)
      vbuf[buf][i] = __builtin_amdgcn_raw_buffer_load_b128(vr, 16 * lane, 1024 * i, PC_BUF_NT);
    __builtin_amdgcn_sched_barrier(0);                       // not behind the arithmetic that follows
  };

  auto consume = [&](int buf, const Cursor& cur) {
    // (the product here, not in the cursor: a vector register written between a block's loads and its
    // arithmetic can be one that a load behind the run's end has yet to fill, and costs a wait for all)
    const float k_sc = cur.k_sc * a.scale_log2, v_sc = cur.v_sc;           // logits in log2 units
    floatx4 acc[KBLK];
#pragma unroll
    for (int bi = 0; bi < KBLK; ++bi) {
      acc[bi] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < KSTEPS; ++j) {
        // k-step j: words 2 (j % 2), 2 (j % 2) + 1 of the lane's load j / 2
        const uint32_t w0 = kbuf[buf][bi][j / 2][2 * (j % 2)], w1 = kbuf[buf][bi][j / 2][2 * (j % 2) + 1];
        u32x4 kb16;
        uint32_t lo, hi;
        pc_e4m3x4_to_bf16(w0, lo, hi); kb16[0] = lo; kb16[1] = hi;
        pc_e4m3x4_to_bf16(w1, lo, hi); kb16[2] = lo; kb16[3] = hi;
        acc[bi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(bf16x8*)&kb16, bq[j], acc[bi], 0, 0, 0);
      }
    }
    float pr[KBLK][4], alpha;
    pc_decode_softmax(acc, k_sc, min(32, cur.at.len - 32 * cur.at.blk), kk, m_run, l_run, alpha, pr);
    // P^T as the B operand: this lane's 8 probabilities are k-slice kk of column c16, in the
    // key order of the V block layout; the V scale rides on them (not on the row sum)
    u32x4 pb;
#pragma unroll
    for (int bi = 0; bi < KBLK; ++bi)
#pragma unroll
      for (int j = 0; j < 4; j += 2) pb[2 * bi + j / 2] = pack_bf16x2(pr[bi][j] * v_sc, pr[bi][j + 1] * v_sc);
    if (__any(alpha != 1.0f)) {                      // some column's maximum grew (rare after the first keys)
#pragma unroll
      for (int mb = 0; mb < MB; ++mb)
#pragma unroll
        for (int r = 0; r < 4; ++r) o_acc[mb][r] *= alpha;
    }
#pragma unroll
    for (int i = 0; i < VLOADS; ++i) {
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t w0 = vbuf[buf][i][2 * h], w1 = vbuf[buf][i][2 * h + 1];
        u32x4 va;
        uint32_t lo, hi;
        pc_e4m3x4_to_bf16(w0, lo, hi); va[0] = lo; va[1] = hi;
        pc_e4m3x4_to_bf16(w1, lo, hi); va[2] = lo; va[3] = hi;
        o_acc[2 * i + h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(bf16x8*)&va, *(bf16x8*)&pb, o_acc[2 * i + h], 0, 0, 0);
      }
    }
  };

  // three register buffers: the loads of two blocks (2 x 8 KiB per wavefront) stay in flight
  Cursor c0 = place(pc_blocks_begin(lens, part, a.parts_grid, a.parts_div, __builtin_amdgcn_readfirstlane(wave), lane, first_lens));
  Cursor c1 = next(c0);
  issue_loads(0, c0);
  issue_loads(1, c1);
  rot.finish(a.query, b, g, G, n_cols, sm.q);
  PC_LDS_BARRIER();
#pragma unroll
  for (int j = 0; j < KSTEPS; ++j) {
    u32x4 raw = *(const u32x4*)(sm.q[min(c16, n_cols - 1)] + 64 * (j / 2) + 16 * kk + 8 * (j % 2));
    if (c16 >= n_cols) raw = u32x4{0, 0, 0, 0};
    bq[j] = *(bf16x8*)&raw;
  }
  auto iter = [&](int cur_buf, int fill_buf) __attribute__((always_inline)) {
    // c0 = block to consume (in cur_buf), c1 = the block after it (already in flight)
    const Cursor c2 = next(c1);                              // (behind the run's end: not valid)
    issue_loads(fill_buf, c2);
    if (c0.at.left > 0) consume(cur_buf, c0);
    c0 = c1; c1 = c2;
  };
  // (no way out in the middle: it would join the loop's end, where the compiler would then have to take
  // either buffer for the one asked for last)
  while (c0.at.left > 0) {
    iter(0, 2);
    iter(1, 0);
    iter(2, 1);
  }

  // ---- wavefront totals, then one partial per workgroup
  l_run = pc_rows_sum(l_run);
  if (kk == 0) { sm.m[wave][c16] = m_run; sm.l[wave][c16] = l_run; }
  if (c16 < n_cols) {
#pragma unroll
    for (int mb = 0; mb < MB; ++mb) *(floatx4*)&sm.o[wave][c16][16 * mb + 4 * kk] = o_acc[mb];
  }
  pc_write_partial<D>(sm, G, n_cols, a.n_q, a.n_q_heads, (long long)b * a.n_parts + part, g, a.part_o, a.part_lse);
}

template <int D>
__global__ __launch_bounds__(PC_D8_WAVES * PC_WAVE) void decode_attn_fp8_kernel(PcDecode8Args a) {
  __shared__ PcDecodeLds<D> sm;
  decode8_workgroup<D>(a, blockIdx.x, sm);
}
template <int D>
__global__ __launch_bounds__(PC_D8_WAVES * PC_WAVE) void decode_attn_fp8_tail_kernel(PcDecode8Args a, PcDecodeArgs tail,
                                                                                     int n_wg8) {
  static_assert(PC_D8_WAVES == PC_DEC_WAVES, "one workgroup size");
  __shared__ PcDecodeLds<D> sm;
  if ((int)blockIdx.x < n_wg8) decode8_workgroup<D>(a, blockIdx.x, sm);
  else pc_decode_workgroup<D>(tail, blockIdx.x - n_wg8, sm);
}

// tail: rides in the launch, unless its parts_grid is 0
template <int D>
static int launch_decode8_d(const PcDecode8Args& a, const PcDecodeArgs& tail, int batch, hipStream_t st) {
  const long long groups = (long long)batch * a.n_kv_heads;
  const long long n_wg8 = groups * a.parts_grid, blocks = n_wg8 + groups * tail.parts_grid;
  if (blocks == 0) return PC_OK;
  if (blocks > 0x7fffffffLL) return PC_ERR_SHAPE;
  dim3 grid((unsigned)blocks), block(PC_D8_WAVES * PC_WAVE);
  PcProfScope prof(PC_KERNEL_DECODE_FP8, st);
  if (tail.parts_grid > 0)
    hipLaunchKernelGGL(decode_attn_fp8_tail_kernel<D>, grid, block, 0, st, a, tail, (int)n_wg8);
  else
    hipLaunchKernelGGL(decode_attn_fp8_kernel<D>, grid, block, 0, st, a);
  PC_LAUNCH_CHECK();
  return PC_OK;
}
int pc_launch_decode_fp8(const void* q, int pos0, float base, const void* k8, const void* v8,
                         const float* k_scale, const float* v_scale, const int32_t* seg_len,
                         int seg_len_per_head, const void* k_tail, const void* v_tail,
                         const int32_t* tail_len, int tail_cap, int batch, int n_q, int n_seg, int k_t,
                         int n_q_heads, int n_kv_heads, int head_dim, float scale, float* part_o,
                         float* part_lse, const PcDecodeSplit& split, const PcDecodeAppend& app, hipStream_t st) {
  const int cols = n_q * (n_q_heads / n_kv_heads);
  if (cols > 16) return PC_ERR_UNSUPPORTED;               // the columns of one 16x16x32 MFMA
  PcDecode8Args a;
  a.query = pc_decode_query(q, pos0, base, n_q, n_q_heads, head_dim);
  a.k8 = (const uint8_t*)k8; a.v8 = (const uint8_t*)v8;
  a.k_scale = k_scale; a.v_scale = v_scale;
  a.seg_len = seg_len; a.seg_len_per_head = seg_len_per_head; a.part_o = part_o; a.part_lse = part_lse;
  a.n_q = n_q; a.n_seg = n_seg; a.k_t = k_t; a.n_q_heads = n_q_heads; a.n_kv_heads = n_kv_heads;
  a.group = n_q_heads / n_kv_heads;
  a.parts_grid = split.parts; a.parts_div = pc_div_by(split.parts); a.heads_div = pc_div_by(n_kv_heads);
  a.n_parts = split.parts + split.tail_parts;
  a.scale_log2 = scale * PC_D8_LOG2E;
  const long long n_wg8 = (long long)batch * n_kv_heads * a.parts_grid;
  const bool tail_here = tail_cap > 0 && (cols <= 4 || n_wg8 <= PC_D8_TAIL_WGS);
  const PcDecodeArgs tail = pc_decode_args(a.query, k_tail, v_tail, tail_len, 0, tail_here ? 1 : 0,
                                           tail_here ? tail_cap : 1, n_kv_heads, scale, part_o, part_lse,
                                           a.n_parts, split.parts, tail_here ? split.tail_parts : 0, app);
  const int rc = head_dim == 128 ? launch_decode8_d<128>(a, tail, batch, st)
                                 : launch_decode8_d<64>(a, tail, batch, st);
  if (rc != PC_OK || tail_cap == 0 || tail_here) return rc;
  return pc_launch_decode(q, pos0, base, k_tail, v_tail, tail_len, 0, batch, n_q, 1, tail_cap, n_q_heads, n_kv_heads,
                          head_dim, scale, part_o, part_lse, a.n_parts, split.parts, split.tail_parts, app, st);
}
