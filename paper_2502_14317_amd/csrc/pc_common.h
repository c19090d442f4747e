// Internal helpers shared by the HIP translation units of the ParallelComp library (gfx950).
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>
#include "div31.h"
#include "parallelcomp.h"
#include "parallelcomp_bench.h"

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // 16-byte register quad

#define PC_WAVE 64

// ---------------------------------------------------------------- host-side error plumbing
void pc_set_hip_error(int err);
#define PC_HIP_TRY(expr)                                   \
  do {                                                     \
    hipError_t _e = (expr);                                \
    if (_e != hipSuccess) {                                \
      pc_set_hip_error((int)_e);                           \
      return PC_ERR_HIP;                                   \
    }                                                      \
  } while (0)
#define PC_LAUNCH_CHECK() PC_HIP_TRY(hipGetLastError())

// Brackets the kernel launches of one scope with HIP events when profiling is enabled.
struct PcProfScope {
  int slot;
  hipStream_t st;
  PcProfScope(int kernel_id, hipStream_t stream);
  ~PcProfScope();
};

// hipFuncAttributeMaxDynamicSharedMemorySize, set once per (kernel, device) instead of on every
// launch: `done` holds one bit per device ordinal (ordinals beyond 63 set it every time).
#include <atomic>
static inline int pc_raise_dynamic_lds(const void* kernel, int bytes, std::atomic<uint64_t>& done) {
  int dev = 0;
  PC_HIP_TRY(hipGetDevice(&dev));
  const uint64_t bit = dev < 64 ? (1ull << dev) : 0ull;
  if (bit && (done.load(std::memory_order_acquire) & bit)) return PC_OK;
  PC_HIP_TRY(hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes));
  done.fetch_or(bit, std::memory_order_release);
  return PC_OK;
}

// A grid dimension holds fewer than 2^32 threads, and more are not always refused: some launches then silently
// run the first few of their workgroups only.  `blocks` workgroups of up to 256 threads as (x, y), number
// y * gridDim.x + x; the last row may hold more than there are.
#define PC_GRID_X (1LL << 23)
static inline dim3 pc_grid_2d(long long blocks) {
  if (blocks <= PC_GRID_X) return dim3((unsigned)blocks);
  return dim3((unsigned)PC_GRID_X, (unsigned)((blocks + PC_GRID_X - 1) / PC_GRID_X));
}

static inline size_t pc_align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }
static inline bool pc_aligned(const void* p, size_t a) { return ((uintptr_t)p % a) == 0; }

// ---------------------------------------------------------------- bf16 <-> fp32 (device)
__device__ __forceinline__ float bf16_lo_to_f32(uint32_t pair) { return __uint_as_float(pair << 16); }
__device__ __forceinline__ float bf16_hi_to_f32(uint32_t pair) { return __uint_as_float(pair & 0xffff0000u); }
__device__ __forceinline__ float bf16_bits_to_f32(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }

// round-to-nearest-even; inputs are finite by contract (NaN keeps a NaN pattern)
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
// two fp32 -> packed bf16 pair (round-to-nearest-even) in one v_cvt_pk_bf16_f32
typedef __bf16 pc_bf16x2 __attribute__((ext_vector_type(2)));
typedef float pc_f32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  pc_f32x2 v = {lo, hi};
  pc_bf16x2 r = __builtin_convertvector(v, pc_bf16x2);
  return *(uint32_t*)&r;
}

// ---------------------------------------------------------------- rotation angles
// RoPE angles in 64 bits: theta_i = base^(-2 i / D) for i < D / 2 as the product of the factors of i's
// set bits, f[b] = base^(-2 2^b / D) from the host; angle = position * theta_i.  Written out here because
// the math library's exp and sincos (2 KB of code each, with the branch for huge arguments) were most of
// the time of the small launches and of every decode workgroup's start.  Relative error of theta below 1e-15
// (exp of a rounded product: up to 3e-15), of the reduced sine and cosine below 2e-16 absolute.
struct PcRope { double f[6]; };
static inline PcRope pc_rope_factors(float base, int head_dim) {
  PcRope r;
  for (int b = 0; b < 6; ++b) r.f[b] = pow((double)base, -2.0 * (double)(1 << b) / (double)head_dim);
  return r;
}
__host__ __device__ __forceinline__ double pc_rope_theta(const PcRope& r, int i) {
  double t = 1.0;
#pragma unroll
  for (int b = 0; b < 6; ++b) t *= (i >> b) & 1 ? r.f[b] : 1.0;
  return t;
}
// sine and cosine of x, 0 <= x < 2^31: reduction by multiples of pi / 2 (Cody and Waite: two parts of pi / 2,
// each product exact in the fused multiply-add), then the Taylor polynomials on [-pi / 4, pi / 4]
__host__ __device__ __forceinline__ void pc_sincos(double x, double& sn, double& cs) {
  const double n = rint(x * 0.63661977236758134308);               // 2 / pi
  const double r = fma(-n, 6.123233995736766e-17, fma(-n, 1.5707963267948966, x));
  const int quadrant = (int)(unsigned)n;
  const double z = r * r;
  double s = -1.0 / 1307674368000.0;                               // 1 / 15!
  s = fma(s, z, 1.0 / 6227020800.0);
  s = fma(s, z, -1.0 / 39916800.0);
  s = fma(s, z, 1.0 / 362880.0);
  s = fma(s, z, -1.0 / 5040.0);
  s = fma(s, z, 1.0 / 120.0);
  s = fma(s, z, -1.0 / 6.0);
  s = fma(s * z, r, r);
  double c = 1.0 / 20922789888000.0;                               // 1 / 16!
  c = fma(c, z, -1.0 / 87178291200.0);
  c = fma(c, z, 1.0 / 479001600.0);
  c = fma(c, z, -1.0 / 3628800.0);
  c = fma(c, z, 1.0 / 40320.0);
  c = fma(c, z, -1.0 / 720.0);
  c = fma(c, z, 1.0 / 24.0);
  c = fma(c, z, -0.5);
  c = fma(c, z, 1.0);
  const double a = quadrant & 1 ? c : s, b = quadrant & 1 ? s : c;
  sn = quadrant & 2 ? -a : a;
  cs = (quadrant + 1) & 2 ? -b : b;
}

// (x0, x1) -> packed bf16 pair of the values and packed bf16 pair of the rounding remainders
// (both roundings to nearest-even, in hardware; inputs are finite by contract)
__device__ __forceinline__ void split_bf16x2(float x0, float x1, uint32_t& hi, uint32_t& lo) {
  hi = pack_bf16x2(x0, x1);
  lo = pack_bf16x2(x0 - bf16_lo_to_f32(hi), x1 - bf16_hi_to_f32(hi));
}

// 16-byte global load / store of data that is touched once (streamed): the non-temporal hint
// keeps it from displacing reusable lines in the caches
#define PC_BUF_NT 2        // the same hint on a buffer load
__device__ __forceinline__ uint4 pc_load_once(const uint4* p) {
  const u32x4 v = __builtin_nontemporal_load((const u32x4*)p);
  return make_uint4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void pc_store_once(uint4* p, uint4 x) {
  const u32x4 v = {x.x, x.y, x.z, x.w};
  __builtin_nontemporal_store(v, (u32x4*)p);
}
__device__ __forceinline__ u32x4 pc_load_once(const u32x4* p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ void pc_store_once(u32x4* p, u32x4 x) { __builtin_nontemporal_store(x, p); }

// Exchange between lane l and lane l ^ 32 without going through LDS: v_permlane32_swap leaves
// the low half's values in both halves of the first result and the high half's in the second.
__device__ __forceinline__ float pc_xhalf_max(float x) {
  const unsigned u = __float_as_uint(x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float pc_xhalf_sum(float x) {
  const unsigned u = __float_as_uint(x);
  auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// The same between lane l and lane l ^ 16 (v_permlane16_swap exchanges neighbouring rows of 16 lanes): max and sum
// over the four lanes l % 16 + 16 i, left in all of them.
__device__ __forceinline__ float pc_rows_max(float x) {
  const unsigned u = __float_as_uint(x);
  auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return pc_xhalf_max(fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1])));
}
__device__ __forceinline__ float pc_rows_sum(float x) {
  const unsigned u = __float_as_uint(x);
  auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  return pc_xhalf_sum(__uint_as_float(r[0]) + __uint_as_float(r[1]));
}

// fp32 score -> uint32 key whose unsigned order is the float order; NaN -> 0 (below everything),
// -0.0 and +0.0 map to the same key
__device__ __forceinline__ uint32_t pc_order_key(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return 0u;
  if ((u << 1) == 0u) u = 0u;
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// chunk_score[c] = sum of per_chunk block sums; chunk_score == nullptr: nothing to do
struct PcChunkSum { const float* blk_sum; float* chunk_score; int per_chunk; };
// The sum of chunk c in a fixed order, so that it does not depend on timing or on who computes it: 256
// strided partial sums, added pairwise 128 apart, 64, .. 1.
// By 256 threads; red: 256 floats of LDS.
__device__ __forceinline__ void pc_chunk_sum(const float* blk_sum, float* chunk_score, int per_chunk, int c, float* red) {
  const float* src = blk_sum + (long long)c * per_chunk;
  float x = 0.f;
  for (int i = threadIdx.x; i < per_chunk; i += 256) x += src[i];
  red[threadIdx.x] = x;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
    __syncthreads();
  }
  if (threadIdx.x == 0) chunk_score[c] = red[0];
}

// ---------------------------------------------------------------- kernels' host launchers
// (each defined in its own translation unit; all arguments already validated)
int pc_launch_gather(const void* k_src, const void* v_src, const int32_t* chunk_idx,
                     const int32_t* tok_idx, int batch, int n_chunks, int rows, int n_sel,
                     int n_kv_heads, int k, int head_dim, void* k_dst, void* v_dst,
                     float* k_amax, float* v_amax, hipStream_t st);   // amax: both or neither
int pc_launch_select_chunks(const float* score, int n, int k, int32_t* out_idx, float* out_score,
                            hipStream_t st);
// cls_lo >= cls_hi: plain top-k (Eq. 7); else Eq. 8 first.  out_cnt may be nullptr.
int pc_launch_select_tokens(const float* tok_score, const int32_t* chunk_idx, int n_sel,
                            int n_kv_heads, int chunk_len, int k, float lambda, int cls_lo,
                            int cls_hi, const int32_t* chunk_lens, int32_t* out_idx,
                            int32_t* out_cnt, hipStream_t st);

// Chunks and tokens in one launch: every workgroup adds up and ranks the chunk scores for itself.  sum: the
// pass-2 block sums; also written: sum.chunk_score, chunk_idx, chunk_top (nullable).
// (and the gather of [.., rows, H_kv, D] rows where pc_select_gather_fits)
bool pc_select_gather_fits(int k, int head_dim);
bool pc_select_layer_fits(int n_chunks, int per_chunk, bool gather);
int pc_launch_select_layer(const PcChunkSum& sum, int n_chunks, int n_sel, const float* tok_score, int n_kv_heads, int chunk_len,
                           int k, float lambda, int cls_lo, int cls_hi, const int32_t* chunk_lens, int32_t* chunk_idx,
                           float* chunk_top, int32_t* out_idx, int32_t* out_cnt, const void* k_src, const void* v_src, int rows,
                           int head_dim, void* kc, void* vc, hipStream_t st);
int pc_launch_chunk_sums(const PcChunkSum& sum, int n_chunks, hipStream_t st);

int pc_launch_chunk_queue(const float* batch_score, int n_batch, int chunk_id0, int cap,
                          int32_t* queue_id, float* queue_score, int32_t* queue_slot,
                          int32_t* slot_src, hipStream_t st);

// prep.hip: the rotation table [n_pos, D / 2], n_q query rows as pc_launch_rope_q leaves them (0: none), and the
// score passes' query columns (q_split nullptr: none; filled in by pc_scores_queries)
struct PcScoreQueries {
  const uint16_t* q;       // [C, L, H_q, D] before RoPE
  const int32_t* chunk_lens;
  uint16_t* q_split;       // [C, H_kv, n_cb][hi, lo][D / 16][2][min(n_cols, 32)][8]: rotated, scaled, split query columns as MFMA operands
  int n_chunks, L, w, w_obs, n_kv_heads, G, n_cols, n_cb;
  PcDiv cb_div, heads_div, obs_div;      // by n_cb, n_kv_heads, w_obs
  float scale_log2;        // softmax scale x log2(e)
};
struct PcPrepArgs {
  float2* table;
  int n_pos;
  float2* q_table;         // the local attention's queries: [D / 4][n_pos rounded up to 128][2 pairs], times q_scale; nullptr: none
  double q_scale;
  PcRope rope;
  const uint16_t* q_blk;
  uint16_t* q_rot;
  int n_q, n_heads, pos0;
  double mul;
  PcScoreQueries scores;
};
int pc_launch_prep(const PcPrepArgs& a, int head_dim, hipStream_t st);

// K/V pre-pass of the local attention: K rotated -> k_rope (row-major, optional) and K tile images;
// V -> V^T tile images.  Images: [n_seq][n_kv_heads][Lp / 64][64 * D].
int pc_launch_kv_prepass(const void* k, const void* v, const float2* table, void* k_rope,
                         void* k_img, void* v_img, int n_seq, int L, int Lp, int n_kv_heads,
                         int head_dim, hipStream_t st);

// Flash-style tile kernel.  Local (global == 0): causal attention inside n_seq sequences of n_rows
// rows.  Global: n_rows query rows per sequence over groups of key segments under one softmax.
// A group: segments [n] of up to cap keys each, bf16 rows of D; key j of (sequence, segment, KV
// head) at element seq * seq_stride + segment * seg_stride + head * head_stride + j * row_stride.
struct PcKvGroup {
  const void* k;            // rotated keys
  const void* v;
  const int32_t* len;       // [n_seq, n] (x [n_kv_heads] if len_per_head) valid keys, or nullptr (= cap)
  int len_per_head, n, cap; // n = 0: no such group
  int causal;               // key j visible to query row t iff j <= t (cap = n_rows)
  int row_stride;
  long long seq_stride, seg_stride, head_stride;
};
#define PC_KV_GROUPS 3
struct PcFlashArgs {
  int global;
  int images;               // global: the groups' segments are tile images (row_stride D, a segment whole tiles)
  const void* q;            // [n_seq, n_rows, H_q, D] bf16.  Local: rotated and scaled here by `table`; global:
                            //   rotated, multiplied by scale * log2(e) and rounded beforehand
  const float2* table;      // local: the queries' table [D / 4][table_rows][2 pairs], (cos, sin) x scale x log2(e)
  int table_rows;           //   (n_rows rounded up to 128)
  int wide_heads;           // 64 rows a wavefront: heads of a workgroup (set by the launcher)
  void* o;                  // [n_seq, n_rows, H_q, D] bf16
  float* lse;               // [n_seq, H_q, n_rows] or nullptr
  int n_seq, n_rows, n_q_heads, n_kv_heads, head_dim;
  int group_batch;          // (sequence, KV head) groups an XCD interleaves, >= 1 (set by the launcher)
  // what a workgroup divides its number by (set by the launcher): H_q / H_kv = group, Q tiles, workgroups of a group, of
  // an XCD's batch of groups, groups of a batch and of the last one, KV heads, parts; with 64 rows a wavefront
  // per_group_div is by the groups beyond a multiple of 8, and group = the workgroups of wide_heads heads each that share a Q tile
  int group, n_qt;
  PcDiv group_div, qt_div, per_group_div, per_batch_div, batch_div, last_div, heads_div, parts_div;
  float scale;
  // local
  const void* k_img;        // K tile images (rotated keys), image index = seq * img_seq_stride +
  const void* v_img;        //   head * img_head_stride + tile; V^T likewise
  long long img_seq_stride, img_head_stride;                               // in tile images
  const int32_t* seq_ctx;   // [n_seq] context rows per sequence or nullptr: sequence s has
  int seq_add;              //   min(seq_ctx[s], n_rows - seq_add) + seq_add rows (and keys)
  PcChunkSum sum;           // done by sum_blocks workgroups in front of the attention's (a multiple of
  int sum_blocks;           //   8, so that those keep their XCDs; set by the launcher)
  // global
  PcKvGroup grp[PC_KV_GROUPS];
  float window;             // log2 units a row's maximum may exceed its reference at a tile's first keys
  int n_parts;              // workgroups a Q tile's keys are cut into; 1: o and lse are written
  float* part_o;            // n_parts > 1: [n_seq, n_parts, n_rows, H_q, D] fp32
  float* part_lse;          // [n_seq, n_parts, n_rows, H_q]
};
// How many parts the global attention's keys are cut into (n_tiles: 64-key tiles of a KV head at
// full lengths), 1 to 64
int pc_flash_parts(int n_seq, int n_rows, int n_q_heads, int n_kv_heads, int head_dim, long long n_tiles);
// Partial rows to have room for: at least rows x pc_flash_parts (rows = n_seq x n_rows x n_q_heads) of
// this and of every smaller call, so it never falls where a size grows
size_t pc_flash_part_rows(size_t rows, long long n_tiles, int has_self);
int pc_launch_flash(const PcFlashArgs& a, hipStream_t st);
// Which calls get 64 query rows a wavefront: local ones (heads of a workgroup, or 0), and blocks of rows over tile images
int pc_flash_wide(int n_seq, int n_rows, int n_q_heads, int n_kv_heads, int head_dim);
int pc_flash_wide_images(int n_seq, int n_rows, int n_q_heads, int n_kv_heads, int head_dim, long long n_tiles, int n_parts);
// One launch of both (the chunk sums are not its business), and the parts of the global one in it
int pc_launch_flash_both(const PcFlashArgs& local, const PcFlashArgs& global, hipStream_t st);
int pc_flash_both_parts(int n_seq, int n_rows, int n_q, int n_q_heads, int n_kv_heads, int head_dim, long long n_tiles, int most);

int pc_launch_self_info(const void* logits, const int32_t* targets, int n_chunks, int n_tokens,
                        int vocab, int negate, float* token_nll, float* info, hipStream_t st);

size_t pc_scores_ws_bytes(const pc_shape* s);
PcScoreQueries pc_scores_queries(const pc_shape* s, const void* q, const int32_t* chunk_lens, void* ws);
// Pre-pass duties the first score pass can take over (it reads and rotates every key anyway):
// the rotated keys (k_rope, nullable), the K tile images and the V^T tile images of
// pc_launch_kv_prepass, Lp = L rounded up to 64.
struct PcPrepassOut { const void* v; void* k_rope; void* k_img; void* v_img; int Lp; };
// later: the chunk scores' last addition is left to the caller, who passes it to pc_launch_flash
// (the query columns of pc_scores_queries come first)
int pc_launch_scores(const pc_shape* s, const void* k, const int32_t* chunk_lens, const float2* table,
                     void* ws, float* tok_score, float* chunk_score, const PcPrepassOut* pre,
                     PcChunkSum* later, hipStream_t st);

// q [batch, n_q, n_heads, D] -> rotated at positions pos0 + t (pos0 < 0: it arrives rotated) and
// multiplied by mul in fp64, rounded to bf16 once
int pc_launch_rope_q(const void* q, void* q_rot, int batch, int n_q, int n_heads, int D, int pos0,
                     float base, float mul, hipStream_t st);
// How the split-KV decode kernels cut the keys into workgroups (n_bg = batch * H_kv): the keys of a
// (sequence, KV head) group, all its segments laid end to end in blocks of 32 keys, are cut into `parts`
// equal runs of blocks, one workgroup (and one partial result) each; those of the 16-bit tail of an
// 8-bit cache (elem_bytes 1) into tail_parts.  room, tail_room: partials the workspace has room for, never
// fewer than parts and tail_parts.
struct PcDecodeSplit { int parts, tail_parts, room, tail_room; };
PcDecodeSplit pc_decode_split(int k_t, int n_seg, int elem_bytes, int tail_cap, int head_dim, long long n_bg);

// A wavefront's walk over its run of 32-key blocks.  The group's blocks are numbered through all
// segments (segment s has ceil(len_s / 32) of them); part `part` of n_parts takes blocks
// [NB part / n_parts, NB (part + 1) / n_parts), wavefront w of n_waves the w-th of n_waves equal
// runs of that.  Everything here is wavefront-uniform.
struct PcSegLens {
  const int32_t* seg_len;   // [B, S] ([B, S, H_kv] if per_head) or nullptr (= k_t)
  int per_head, n_seg, n_kv_heads, k_t, b, g;
  __device__ __forceinline__ int at(int s) const { return per_head ? (b * n_seg + s) * n_kv_heads + g : b * n_seg + s; }
  __device__ __forceinline__ int len(int s) const {
    if (!seg_len) return k_t;
    // read-only while a kernel runs: where the index is uniform this is a scalar load, which does not
    // queue behind the keys in flight
    typedef const __attribute__((address_space(4))) int32_t* scalar_t;
    return min(max(((scalar_t)(uintptr_t)seg_len)[at(s)], 0), k_t);
  }
};
struct PcBlockCursor {
  int s, blk, n_blk, len, left;   // segment, block within it, its block count and length, blocks left in the run (0: behind its end)
};
// inclusive prefix sum over the wavefront's lanes (row shifts, then the rows' totals broadcast onwards)
__device__ __forceinline__ int pc_wave_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);    // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);    // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);    // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);    // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);    // row_bcast:15
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);    // row_bcast:31
  return x;
}
// Runs as equal as possible: the first total % n of n runs hold a block more.  32 bits are enough for
// what fits in memory (a block of a group is at least 2 KiB of keys).
// first: pc_first_lens, asked for in front of whatever else a workgroup starts with, so that the first keys wait for it
// alone: as it lies in memory and by every lane, since the limits or a condition beside the load would be waited for there
__device__ __forceinline__ int pc_first_lens(const PcSegLens& L, int lane) {
  return L.seg_len && L.n_seg > 0 ? L.seg_len[L.at(min(lane, L.n_seg - 1))] : 0;
}
__device__ __forceinline__ PcBlockCursor pc_blocks_begin(const PcSegLens& L, int part, int n_parts, PcDiv parts_div, int wave, int lane, int first) {
  constexpr int WAVES = 4;
  PcBlockCursor c; c.s = 0; c.blk = 0; c.n_blk = 0; c.len = 0; c.left = 0;
  const int nb_full = (L.k_t + 31) / 32;
  // lanes take a segment each, 64 segments per round; up to 64 segments the one round is kept
  int total = 0, len = 0, nb = 0, incl = 0;
  asm volatile("" : "+v"(first));                             // not in front of it
  first = lane < L.n_seg ? min(max(first, 0), L.k_t) : 0;
  if (!L.seg_len) {
    total = L.n_seg * nb_full;
  } else {
    for (int s0 = 0; s0 < L.n_seg; s0 += PC_WAVE) {
      len = s0 == 0 ? first : (s0 + lane < L.n_seg ? L.len(s0 + lane) : 0);
      nb = (len + 31) / 32;
      incl = pc_wave_scan(nb);
      total += __builtin_amdgcn_readlane(incl, PC_WAVE - 1);
    }
  }
  const int per = pc_div(total, parts_div), extra = total - per * n_parts;
  const int lo = part * per + min(part, extra), n = per + (part < extra);
  const int w_lo = lo + n * wave / WAVES, w_hi = lo + n * (wave + 1) / WAVES;
  if (w_lo >= w_hi) return c;
  c.left = w_hi - w_lo;
  if (!L.seg_len) {
    c.s = w_lo / nb_full; c.blk = w_lo % nb_full; c.n_blk = nb_full; c.len = L.k_t;
    return c;
  }
  int base = 0;
  for (int s0 = 0; s0 < L.n_seg; s0 += PC_WAVE) {
    if (L.n_seg > PC_WAVE) {
      len = s0 == 0 ? first : (s0 + lane < L.n_seg ? L.len(s0 + lane) : 0);
      nb = (len + 31) / 32;
      incl = pc_wave_scan(nb);
    }
    const int rel = w_lo - base;                              // the run's first block, counted from this round's first segment
    const unsigned long long hit = __ballot(nb > 0 && incl - nb <= rel && rel < incl);
    if (hit) {
      const int src = __ffsll((long long)hit) - 1;
      c.s = s0 + src;
      c.n_blk = __builtin_amdgcn_readlane(nb, src);
      c.blk = rel - (__builtin_amdgcn_readlane(incl, src) - c.n_blk);
      c.len = __builtin_amdgcn_readlane(len, src);
      return c;
    }
    base += __builtin_amdgcn_readlane(incl, PC_WAVE - 1);
  }
  c.left = 0;
  return c;                                                   // not reached: w_lo < total
}
__device__ __forceinline__ PcBlockCursor pc_blocks_next(const PcSegLens& L, PcBlockCursor c) {
  if (c.left <= 1) { c.left = 0; return c; }
  --c.left;
  if (++c.blk < c.n_blk) return c;
  c.blk = 0;
  for (++c.s; c.s < L.n_seg; ++c.s) {                         // the next segment that has keys
    c.len = L.len(c.s);
    c.n_blk = (c.len + 31) / 32;
    if (c.n_blk > 0) return c;
  }
  c.left = 0;                                                 // not reached: left counted real blocks
  return c;
}
int pc_launch_kv_append(const void* k_new, const void* v_new, int batch, int n_new, int n_seg,
                        int seg, int k_t, int n_kv_heads, int head_dim, int pos0, float base,
                        void* kc, void* vc, int32_t* seg_len, int seg_len_per_head,
                        hipStream_t st);
struct PcDecodeAppend;     // decode_core.h
// A decoding step in the merge: the new token's row of the last of n_seg segments [.., H_kv, cap, D] (one more
// key, where self_row >= 0), and the lengths [B, n_seg] ([B, n_seg, H_kv] if len_per_head) that count it
struct PcMergeStep {
  const int32_t* self_row; // [B, H_kv] or nullptr: no step
  const uint16_t* k;
  const uint16_t* v;
  int32_t* seg_len;
  int n_seg, cap, len_per_head;
};
// q: rotated by the kernel at positions pos0 + t (pos0 < 0: it arrives rotated)
int pc_launch_decode(const void* q, int pos0, float base, const void* kc, const void* vc,
                     const int32_t* seg_len, int seg_len_per_head, int batch, int n_q, int n_seg, int k_t, int n_q_heads, int n_kv_heads,
                     int head_dim, float scale, float* part_o, float* part_lse, int n_parts, int part0,
                     int parts_grid, const PcDecodeAppend& app, hipStream_t st);
// k_amax, v_amax [n_segs] (both or neither): the largest |value| of every segment's valid rows,
// known beforehand (the gather leaves it): the kernel then reads the segment once
int pc_launch_kv_quantize_fp8(const void* kc, const void* vc, const int32_t* seg_len,
                              int seg_len_per_head, long long n_segs, int n_kv_heads, int k_t,
                              int head_dim, const float* k_amax, const float* v_amax, void* k8,
                              void* v8, float* k_scale, float* v_scale, hipStream_t st);
// Tile images (the tile kernel's) of the global attention's keys over the 8-bit cache, in one launch: 8-bit
// segments widened to code * scale (rounded to bf16), and 16-bit rows.  Every segment takes whole 64-key
// tiles, [segment][tiles][64 * D]; keys behind its length are zeros in the last tile, later tiles are not written.
struct PcRowsToImages {
  const uint16_t* k;        // bf16 rows; row j of (sequence, head) at seq * seq_stride + head * head_stride + j * row_stride
  const uint16_t* v;
  const int32_t* len;       // [n_seq] valid rows or nullptr (= n_rows)
  int n_rows, row_stride;   // n_rows = 0: none
  long long seq_stride, head_stride;
  uint16_t* k_img;          // [n_seq][n_kv_heads][tiles][64 * D]
  uint16_t* v_img;
};
// ... and the query rows that the same attention takes, rotated (pos0 + t; pos0 < 0: as they are) and scaled by mul
struct PcRowsToRotate {
  const uint16_t* q;        // bf16 [rows = B n_q][n_heads][D]
  uint16_t* q_rot;
  uint32_t rows, period;    // every period-th workgroup takes a row (set by the launch)
  int n_q, n_heads, pos0;
  PcRope rope;
  double mul;
};
int pc_launch_fp8_images(const void* k8, const void* v8, const float* k_scale, const float* v_scale,
                         const int32_t* seg_len, int seg_len_per_head, long long n_segs, int k_t, int head_dim, void* k_img, void* v_img,
                         const PcRowsToImages& tail, const PcRowsToImages& self, int n_seq, int n_kv_heads,
                         const PcRowsToRotate& rows, hipStream_t st);
// The segments alone as bf16 rows [n_segs, k_t, D] (those behind a length are not written)
int pc_launch_fp8_rows(const void* k8, const void* v8, const float* k_scale, const float* v_scale, const int32_t* seg_len,
                       int seg_len_per_head, long long n_segs, int n_kv_heads, int k_t, int head_dim, void* k_rows, void* v_rows, hipStream_t st);
// Partials of the 8-bit segments, then those of the 16-bit tail (tail_cap > 0)
int pc_launch_decode_fp8(const void* q, int pos0, float base, const void* k8, const void* v8,
                         const float* k_scale, const float* v_scale, const int32_t* seg_len,
                         int seg_len_per_head, const void* k_tail, const void* v_tail,
                         const int32_t* tail_len, int tail_cap, int batch, int n_q, int n_seg, int k_t,
                         int n_q_heads, int n_kv_heads, int head_dim, float scale, float* part_o,
                         float* part_lse, const PcDecodeSplit& split, const PcDecodeAppend& app, hipStream_t st);
// Merge of the tile kernel's partials [batch, n_parts, n_q, H_q, D] (no self segment)
int pc_launch_merge_rows(const float* part_o, const float* part_lse, void* out, float* lse_out, int batch,
                         int n_q, int n_q_heads, int head_dim, int n_parts, hipStream_t st);
int pc_launch_merge(const float* part_o, const float* part_lse, const void* q_rot,
                    const void* k_self, const void* v_self, const PcMergeStep& step, void* out, float* lse_out,
                    int batch, int n_q, int n_q_heads, int n_kv_heads, int head_dim, int n_parts, float scale,
                    hipStream_t st);
