// Chunk-batched causal local attention (Eq. 1-2) with chunk-local RoPE, for gfx950.
//
// Two kernels (and the two modes of the second in one launch):
//   kv_prepass_kernel   K -> rotated K (bf16, the KV cache later steps gather from) and K tile
//                       images; V -> V^T tile images (the layouts the tile kernel copies to LDS)
//   flash_fwd_kernel    online-softmax attention on 32x32x16 bf16 MFMA
//
// flash_fwd_kernel computes S^T = K Q^T and O^T = V^T P^T.  In the MFMA result layout a lane
// then owns ONE query (column) and holds many keys (rows) in its registers, so the row max
// and row sum are in-register reductions plus one exchange between lane l and l+32, the
// rescale factor of O is a per-lane scalar, and P^T in registers is already the B operand
// of the second product (after rounding to bf16).  K rows are fed to the first MFMA in a
// permuted order (bits 2 and 3 of the row index swapped) so that the 8 probabilities a lane
// holds for one k-step belong to 8 consecutive keys, i.e. one 16-byte granule of V^T.
//
// Workgroup: 4 wavefronts x 32 query rows = 128 rows of one (sequence, query head), one
// wavefront per SIMD, at most 256 registers and 80 KiB of LDS, so that two workgroups share a
// CU: the second wavefront of every SIMD belongs to an independent workgroup and fills the
// issue slots the first one leaves (a single wavefront cannot keep the matrix pipe busy: its
// own vector-ALU, LDS and barrier time is exposed).  Key tiles of 64 are copied into LDS by
// direct global->LDS loads (K double-, V^T triple-buffered).  Causal structure: a Q tile only
// visits key tiles up to its diagonal and the mask is applied on diagonal tiles only.
// Workgroups are ordered so that one XCD works on one (sequence, KV head) at a time (its K/V
// stay in that XCD's L2) and takes the long (late) Q tiles first.
#include "pc_common.h"
#include <math.h>
#include <algorithm>
#include <type_traits>

#define PC_FA_NB 1                   // 32-row blocks per wavefront
#define PC_FA_WAVES 4                // wavefronts per workgroup (one per SIMD); two workgroups share a CU
#define PC_FA_THREADS (PC_FA_WAVES * PC_WAVE)
#define PC_FA_BM (PC_FA_WAVES * 32 * PC_FA_NB)   // query rows per workgroup
#define PC_FA_BN 64                  // keys per tile
// Largest sum of a lane's 16 probabilities of a step before the reference of its row moves (64 rows a wavefront, behind
// a row's first step).  A probability against a low reference is as exact as any, in fp32 and bf16, which share their
// exponents: the sums stay below 2^110 (2^20 keys) and O^T in fp32 up to values of 2^17 (a few heavy keys: 2^35), beyond
// which a wavefront takes its rows a second time (end of wide_workgroup).  A step taken anew
// costs some two, with 64 rows a wavefront more often than with 32, so on sharp logits a narrow window costs more than the
// maxima that it saves.  16 x 8192 rows, 32 / 8 heads, ms, logits of deviation 1 / 4 / 8 / 16 / 32: 32 rows a wavefront (row
// maxima, 2^8) 7.46 / 7.78 / 7.90 / 8.00 / 7.81, here with 2^48 6.80 / 6.84 / 6.87 / 7.81 / 9.19, 2^64 6.79 / 6.84 / 6.87 / 7.13 /
// 8.47, 2^90 6.81 / 6.83 / 6.87 / 6.89 / 7.79; 12 x 2214 rows, us: 542 / 577 / 602 / 600 / 601, 2^48 487 / 493 / 502 / 562 / 715,
// 2^90 497 / 493 / 501 / 503 / 580.  2^10: 9.7 ms at 8 already.
#define PC_FA_WINDOW 1237940039285380274899124224.f    // 2^90
#define PC_LOG2E 1.4426950408889634f
// orders a wavefront's own LDS writes before its own later LDS reads (no other wavefront involved)
#define PC_FA_WAVE_LDS_SYNC()                                \
  do {                                                       \
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   \
    __builtin_amdgcn_wave_barrier();                         \
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");   \
  } while (0)
#define PC_LN2 0.6931471805599453f

// ------------------------------------------------------------------------------------------
// Tile images.  flash_fwd_kernel copies whole 64-key tiles of K and V^T into LDS with contiguous
// 1 KiB loads, so this pre-pass writes both in the exact byte order the MFMA operand reads want,
// 16-byte granules (8 bf16) stored granule-column by granule-column:
//   K image   [16 * D / 128 .. i.e. D/8 columns][64 keys]:   granule (c, r) = K[key r][8c .. 8c+7]
//   V^T image [8 columns][D rows]:                           granule (c, d) = V[keys 8c .. 8c+7][d]
// The 16 lanes an LDS read serves together then touch 256 consecutive bytes (no bank conflict,
// no swizzle), and every operand address is one per-lane base plus an immediate offset.
// Images of one (sequence, KV head) are consecutive: [n_seq][n_kv_heads][Lp / 64][64 * D].
// Keys past the end of a sequence are zero in both images.
// One workgroup per (sequence, KV head, 64-row tile).
template <int D>
__global__ __launch_bounds__(256) void kv_prepass_kernel(
    const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
    const float2* __restrict__ table, uint16_t* __restrict__ k_rope, uint16_t* __restrict__ k_img,
    uint16_t* __restrict__ v_img, int L, int Lp, int n_kv_heads) {
  constexpr int HALF = D / 2;
  constexpr int VSTRIDE = D + 2;                  // bf16 elements, odd number of dwords
  __shared__ uint16_t v_lds[64 * VSTRIDE];
  const int seq = blockIdx.x, g = blockIdx.y, tile = blockIdx.z;
  const int row0 = tile * 64;
  const long long seq_base = (long long)seq * L;
  const long long img = (((long long)seq * n_kv_heads + g) * (Lp / 64) + tile) * (64 * D);

  // ---- K: rotate pairs (i, i + D/2); a thread handles 8 consecutive i of one row
  constexpr int K_ITEMS = 64 * (HALF / 8);
  for (int it = threadIdx.x; it < K_ITEMS; it += 256) {
    const int r = it / (HALF / 8), i0 = (it % (HALF / 8)) * 8;
    const int row = row0 + r;
    uint4 oa = make_uint4(0, 0, 0, 0), ob = make_uint4(0, 0, 0, 0);
    if (row < L) {
      const long long off = ((seq_base + row) * n_kv_heads + g) * D;
      const uint4 a = pc_load_once((const uint4*)(k + off + i0));
      const uint4 b = pc_load_once((const uint4*)(k + off + HALF + i0));
      const uint32_t aw[4] = {a.x, a.y, a.z, a.w}, bw[4] = {b.x, b.y, b.z, b.w};
      uint32_t ra[4], rb[4];
      const float2* cs = table + (long long)row * HALF + i0;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float2 c0 = cs[2 * e], c1 = cs[2 * e + 1];
        const float x1l = bf16_lo_to_f32(aw[e]), x1h = bf16_hi_to_f32(aw[e]);
        const float x2l = bf16_lo_to_f32(bw[e]), x2h = bf16_hi_to_f32(bw[e]);
        ra[e] = pack_bf16x2(x1l * c0.x - x2l * c0.y, x1h * c1.x - x2h * c1.y);
        rb[e] = pack_bf16x2(x2l * c0.x + x1l * c0.y, x2h * c1.x + x1h * c1.y);
      }
      oa = make_uint4(ra[0], ra[1], ra[2], ra[3]);
      ob = make_uint4(rb[0], rb[1], rb[2], rb[3]);
      if (k_rope != nullptr) {
        pc_store_once((uint4*)(k_rope + off + i0), oa);
        pc_store_once((uint4*)(k_rope + off + HALF + i0), ob);
      }
    }
    pc_store_once((uint4*)(k_img + img + ((i0 / 8) * 64 + r) * 8), oa);
    pc_store_once((uint4*)(k_img + img + (((HALF + i0) / 8) * 64 + r) * 8), ob);
  }

  // ---- V: 64 x D tile -> LDS -> V^T image (zero beyond row L)
  constexpr int V_ITEMS = 64 * (D / 8);
  for (int it = threadIdx.x; it < V_ITEMS; it += 256) {
    const int r = it / (D / 8), c8 = (it % (D / 8)) * 8;
    const int row = row0 + r;
    uint4 x = make_uint4(0, 0, 0, 0);
    if (row < L) x = pc_load_once((const uint4*)(v + ((seq_base + row) * n_kv_heads + g) * D + c8));
    uint32_t* dst = (uint32_t*)(v_lds + r * VSTRIDE + c8);   // 4-byte aligned: VSTRIDE, c8 even
    dst[0] = x.x; dst[1] = x.y; dst[2] = x.z; dst[3] = x.w;
  }
  __syncthreads();
  constexpr int T_ITEMS = 8 * D;                  // (granule column = group of 8 keys, d)
  for (int it = threadIdx.x; it < T_ITEMS; it += 256) {
    const int c = it / D, d = it % D;
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t lo = v_lds[(8 * c + 2 * e) * VSTRIDE + d];
      const uint32_t hi = v_lds[(8 * c + 2 * e + 1) * VSTRIDE + d];
      w[e] = lo | (hi << 16);
    }
    pc_store_once((uint4*)(v_img + img + (c * D + d) * 8), make_uint4(w[0], w[1], w[2], w[3]));
  }
}

int pc_launch_kv_prepass(const void* k, const void* v, const float2* table, void* k_rope,
                         void* k_img, void* v_img, int n_seq, int L, int Lp, int n_kv_heads,
                         int head_dim, hipStream_t st) {
  if (n_kv_heads > 65535 || Lp / 64 > 65535) return PC_ERR_SHAPE;       // grid limits
  dim3 grid(n_seq, n_kv_heads, Lp / 64), block(256);
  PcProfScope prof(PC_KERNEL_KV_PREPASS, st);
  if (head_dim == 128)
    hipLaunchKernelGGL(kv_prepass_kernel<128>, grid, block, 0, st, (const uint16_t*)k,
                       (const uint16_t*)v, table, (uint16_t*)k_rope, (uint16_t*)k_img,
                       (uint16_t*)v_img, L, Lp, n_kv_heads);
  else
    hipLaunchKernelGGL(kv_prepass_kernel<64>, grid, block, 0, st, (const uint16_t*)k,
                       (const uint16_t*)v, table, (uint16_t*)k_rope, (uint16_t*)k_img,
                       (uint16_t*)v_img, L, Lp, n_kv_heads);
  PC_LAUNCH_CHECK();
  return PC_OK;
}

// ------------------------------------------------------------------------------------------
template <int D>
struct FlashSmem {
  static constexpr int KBUF = 2;                   // K tile t lives in buffer t % 2
  static constexpr int VBUF = 3;                   // V^T tile t in buffer t % 3 (read one period early)
  static constexpr int K_ELEMS = PC_FA_BN * D;
  static constexpr int V_ELEMS = D * PC_FA_BN;
  static constexpr int BYTES = (KBUF * K_ELEMS + VBUF * V_ELEMS) * 2;
};

// row index of the first MFMA's A operand -> key within a 32-key block (swap bits 2 and 3)
__device__ __forceinline__ int pc_key_of_row(int m) {
  return (m & ~12) | ((m & 4) << 1) | ((m & 8) >> 1);
}

#define PC_FA_LOCAL 0
#define PC_FA_ROWS 1
#define PC_FA_IMAGES 2

// The global attention's keys as tiles of 64: the tiles that every row of the workgroup sees whole
// come first (no mask), then those that need one (a segment's ragged last tile, the causal
// diagonal), so that the main loop holds no mask.  `full` tiles of a segment of `len` keys:
__device__ __forceinline__ int pc_seg_len(const PcKvGroup& kg, int b, int g, int n_kv_heads, int s) {
  if (!kg.len) return kg.cap;
  return min(max(kg.len[kg.len_per_head ? (b * kg.n + s) * n_kv_heads + g : b * kg.n + s], 0), kg.cap);
}
// t0, t1: first and last query row of the workgroup (a causal segment's keys end at t1)
__device__ __forceinline__ int pc_full_tiles(const PcKvGroup& kg, int len, int t0) {
  return (kg.causal ? min(t0 + 1, len) : len) / 64;
}
__device__ __forceinline__ int pc_seg_tiles(const PcKvGroup& kg, int len, int t0, int t1, bool masked) {
  const int end = kg.causal ? min(t1 + 1, len) : len, full = pc_full_tiles(kg, len, t0);
  return masked ? (end + 63) / 64 - full : full;
}
// Sum over a group's segments, and the segment that holds tile `rel` of it (0 <= rel < sum; all
// wavefront-uniform).  With lengths on the device the lanes take a segment each, 64 per round.
__device__ __forceinline__ int pc_kv_tiles(const PcKvGroup& kg, int b, int g, int n_kv_heads, int t0, int t1,
                                           bool masked, int lane) {
  if (!kg.len) return kg.n * pc_seg_tiles(kg, kg.cap, t0, t1, masked);
  int total = 0;
  for (int s0 = 0; s0 < kg.n; s0 += PC_WAVE) {
    int nt = s0 + lane < kg.n ? pc_seg_tiles(kg, pc_seg_len(kg, b, g, n_kv_heads, s0 + lane), t0, t1, masked) : 0;
#pragma unroll
    for (int off = PC_WAVE / 2; off > 0; off >>= 1) nt += __shfl_xor(nt, off);
    total += __builtin_amdgcn_readfirstlane(nt);
  }
  return total;
}
__device__ __forceinline__ void pc_kv_find(const PcKvGroup& kg, int b, int g, int n_kv_heads, int t0, int t1,
                                           bool masked, int lane, int rel, int& seg, int& tile, int& len) {
  if (!kg.len) {
    const int nt = pc_seg_tiles(kg, kg.cap, t0, t1, masked);
    seg = rel / nt; tile = rel % nt; len = kg.cap;
    return;
  }
  for (int s0 = 0; s0 < kg.n; s0 += PC_WAVE) {
    const int l = s0 + lane < kg.n ? pc_seg_len(kg, b, g, n_kv_heads, s0 + lane) : 0;
    const int nt = pc_seg_tiles(kg, l, t0, t1, masked);
    int incl = nt;                                           // inclusive prefix sum over the lanes
#pragma unroll
    for (int off = 1; off < PC_WAVE; off <<= 1) {
      const int up = __shfl_up(incl, off);
      if (lane >= off) incl += up;
    }
    const unsigned long long hit = __ballot(incl - nt <= rel && rel < incl);
    if (hit) {
      const int src = __ffsll((long long)hit) - 1;
      seg = s0 + src;
      tile = rel - __builtin_amdgcn_readfirstlane(__shfl(incl - nt, src));
      len = __builtin_amdgcn_readfirstlane(__shfl(l, src));
      return;
    }
    rel -= __builtin_amdgcn_readfirstlane(__shfl(incl, PC_WAVE - 1));
  }
}

// MODE PC_FA_LOCAL: causal local attention of whole sequences over tile images of K and V^T.
// MODE PC_FA_ROWS: a block of query rows over groups of row-major segments (compressed segments, a
//   16-bit tail, the causal self segment) under one softmax.  PC_FA_IMAGES: the same over segments that
//   are tile images (the 8-bit cache, which has to be widened anyway).  The rows of a KV head's G query
//   heads are packed into one run of n_rows * G rows (row r = query r / G, head r % G of the
//   group), so a short query block fills its 128-row tiles; all segments' tiles laid end to end
//   are cut into n_parts equal runs, one workgroup each.  With one part the workgroup writes the
//   final output, otherwise a partial result for the merge.
template <int D, int MODE>
__device__ __forceinline__ void flash_workgroup(const PcFlashArgs& a, int bid, uint16_t* smem) {
  constexpr bool GLOBAL = MODE != PC_FA_LOCAL;
  using SM = FlashSmem<D>;
  constexpr int KS = D / 16;        // k-steps of the first product (over head_dim)
  constexpr int DB = D / 32;        // 32-row blocks of O^T (over head_dim)
  constexpr int HALF = D / 2;
  auto k_at = [&](int t) __attribute__((always_inline)) { return (t % SM::KBUF) * SM::K_ELEMS; };
  auto k_lds = [&](int t) __attribute__((always_inline)) { return smem + k_at(t); };
  auto v_lds = [&](int t) __attribute__((always_inline)) {
    return smem + SM::KBUF * SM::K_ELEMS + (t % SM::VBUF) * SM::V_ELEMS;
  };

  // ---- which (sequence, head, Q tile): one XCD (blockIdx % 8) works through whole
  //      (sequence, KV head) groups, heavy Q tiles first, the group's query heads adjacent; the
  //      last groups, when their number is no multiple of 8, are dealt out to all XCDs.  By multiplications (PcDiv): a
  //      run of divisions by arguments stood in front of the first load.  In a layer that is no more than two runs differ
  //      by (us, divisions / now): 4 x 576 rows, 8 heads of 64 values 35.8 / 35.3, 1 x 4096, 32 heads 227.5 / 227.0, 36 of them 6083 / 6051.
  const int G = a.group, n_qt = a.n_qt;
  const int rows_wg = GLOBAL ? a.n_rows * G : a.n_rows;      // rows that the Q tiles of a head (of a group) cover
  const int per_group = GLOBAL ? n_qt * a.n_parts : G * n_qt;
  const int n_groups = a.n_seq * a.n_kv_heads, full_blocks = n_groups / 8 * 8 * per_group;
  int cg, within;
  if (bid < full_blocks) {
    const int xcd = bid % 8, jb = bid / 8;
    const int batch = pc_div(jb, a.per_batch_div), in_batch = jb - batch * (a.group_batch * per_group);
    const int left = n_groups / 8 - batch * a.group_batch, n_batch = min(a.group_batch, left);
    within = pc_div(in_batch, left >= a.group_batch ? a.batch_div : a.last_div);
    cg = (batch * a.group_batch + in_batch - within * n_batch) * 8 + xcd;
  } else {
    const int rest = bid - full_blocks;
    const int at = pc_div(rest, a.per_group_div);
    cg = n_groups / 8 * 8 + at;
    within = rest - at * per_group;
  }
  const int seq = pc_div(cg, a.heads_div), g = cg - seq * a.n_kv_heads;
  const int turn = pc_div(within, GLOBAL ? a.qt_div : a.group_div);
  const int part = GLOBAL ? turn : 0;
  const int qt = GLOBAL ? within - turn * n_qt : n_qt - 1 - turn;
  const int h = GLOBAL ? g * G : g * G + within - turn * G;  // (GLOBAL: the group's first head)

  const int tid = threadIdx.x, lane = tid % PC_WAVE, wave = tid / PC_WAVE;
  const int hf = lane / 32, n = lane % 32;
  const int row0_wg = qt * PC_FA_BM;
  // rows (= keys) of this sequence: a short chunk is [its context rows ; the query rows]
  const int seq_rows = GLOBAL ? rows_wg
                       : (a.seq_ctx ? min(max(a.seq_ctx[seq], 0), a.n_rows - a.seq_add) + a.seq_add : a.n_rows);
  if (row0_wg >= seq_rows) return;                 // a Q tile of padding rows (uniform over the workgroup)
  constexpr int NB = PC_FA_NB;
  const int row0 = row0_wg + 32 * NB * wave;      // first query row of this wavefront
  // query row -> index in [row, head] of its q and output rows, its position
  auto row_at = [&](int r) __attribute__((always_inline)) {
    return GLOBAL ? ((long long)seq * a.n_rows + pc_div(r, a.group_div)) * a.n_q_heads + h + pc_mod(r, G, a.group_div)
                  : ((long long)seq * a.n_rows + r) * a.n_q_heads + h;
  };
  auto pos_of = [&](int r) __attribute__((always_inline)) { return GLOBAL ? pc_div(r, a.group_div) : r; };
  int my_row[NB], my_t[NB], max_key[NB];
  const int wave_s = __builtin_amdgcn_readfirstlane(wave);

  // ---- local: keys [0, key_end) in T 64-key tiles; steps of 32 keys [0, J0) are visible to every
  //      row of the workgroup (no mask)
  const int n_valid = seq_rows;
  int T = (min(n_valid, row0_wg + PC_FA_BM) + 63) / 64;
  const int J0 = (min(row0_wg, n_valid - 1) + 1) / 32;
  const long long img0 = (seq * a.img_seq_stride + g * a.img_head_stride) * (64LL * D);
  const uint16_t* kbase = (const uint16_t*)a.k_img + img0;
  const uint16_t* vbase = (const uint16_t*)a.v_img + img0;

  struct Limit { int cut, c0; };                   // a (global) tile's valid keys, its first key's position if causal
  // ---- global: a cursor over the run's tiles, the unmasked ones of all segments first.  Inside a
  //      segment it moves by scalar additions; the groups' descriptions are read only where a
  //      segment begins.  `cut` is how many keys from the tile's first on are valid, c0 the first
  //      key's position if the segment is causal, else far below every row.
  struct Cursor {
    const uint16_t* k; const uint16_t* v;
    int row_bytes, cut, c0, c0_step;
    int in_seg, in_phase, left;                    // tiles left in the segment, among the unmasked / masked ones, in the run
    int grp, seg;
    bool masked, seg_start;
  };
  Cursor cur = {};
  const int wg_t0 = pc_div(row0_wg, a.group_div), wg_t1 = pc_div(min(row0_wg + PC_FA_BM, rows_wg) - 1, a.group_div);
  int run_full = 0, masked_lo = 0;                           // unmasked tiles of the run; its first masked tile
  auto cur_place = [&](int tile, int len) __attribute__((always_inline)) {   // tile: among the segment's of this phase
    const PcKvGroup& kg = a.grp[cur.grp];
    const int idx = tile + (cur.masked ? pc_full_tiles(kg, len, wg_t0) : 0);
    const long long at = seq * kg.seq_stride + cur.seg * kg.seg_stride + g * kg.head_stride + 64LL * idx * kg.row_stride;
    cur.k = (const uint16_t*)kg.k + at; cur.v = (const uint16_t*)kg.v + at;
    cur.row_bytes = 2 * kg.row_stride;
    cur.cut = len - 64 * idx;
    cur.c0 = kg.causal ? 64 * idx : -(1 << 28);
    cur.c0_step = kg.causal ? 64 : 0;
    cur.in_seg = pc_seg_tiles(kg, len, wg_t0, wg_t1, cur.masked) - tile;
    cur.seg_start = idx == 0;
  };
  auto cur_seek = [&](int rel) __attribute__((always_inline)) {              // to tile `rel` of the phase
    int tile = 0, len = 0;
    cur.grp = 0;
    for (; cur.grp < PC_KV_GROUPS; ++cur.grp) {
      const PcKvGroup& kg = a.grp[cur.grp];
      const int nt = kg.n > 0 ? pc_kv_tiles(kg, seq, g, a.n_kv_heads, wg_t0, wg_t1, cur.masked, lane) : 0;
      if (rel < nt) break;
      rel -= nt;
    }
    pc_kv_find(a.grp[cur.grp], seq, g, a.n_kv_heads, wg_t0, wg_t1, cur.masked, lane, rel, cur.seg, tile, len);
    cur_place(tile, len);
  };
  auto cur_next = [&]() __attribute__((always_inline)) {     // stays on the run's last tile
    if (cur.left <= 1) return;
    --cur.left;
    if (cur.in_phase > 1 && cur.in_seg > 1) {
      --cur.in_phase; --cur.in_seg;
      cur.k += 32 * cur.row_bytes; cur.v += 32 * cur.row_bytes;      // 64 rows
      cur.cut -= 64; cur.c0 += cur.c0_step; cur.seg_start = false;
    } else if (cur.in_phase > 1) {
      --cur.in_phase;
      int len;
      do {                                                   // the next segment that has tiles of this kind
        if (++cur.seg >= a.grp[cur.grp].n) { cur.seg = 0; ++cur.grp; }
        len = a.grp[cur.grp].n > 0 ? pc_seg_len(a.grp[cur.grp], seq, g, a.n_kv_heads, cur.seg) : 0;
        len = __builtin_amdgcn_readfirstlane(len);
      } while (len == 0 || pc_seg_tiles(a.grp[cur.grp], len, wg_t0, wg_t1, cur.masked) == 0);
      cur_place(0, len);
    } else {
      cur.masked = true;
      cur.in_phase = cur.left;
      cur_seek(masked_lo);
    }
  };
  if (GLOBAL) {
    int n_full = 0, n_masked = 0;
    for (int i = 0; i < PC_KV_GROUPS; ++i)
      if (a.grp[i].n > 0) {
        n_full += pc_kv_tiles(a.grp[i], seq, g, a.n_kv_heads, wg_t0, wg_t1, false, lane);
        n_masked += pc_kv_tiles(a.grp[i], seq, g, a.n_kv_heads, wg_t0, wg_t1, true, lane);
      }
    // every part (of 64 at most) takes an equal run of all tiles, [lo, hi) of [full ; masked] (2^25 tiles of a KV head,
    // of at most 2^20 segments, would not fit in memory)
    const int lo = pc_div((n_full + n_masked) * part, a.parts_div);
    const int hi = pc_div((n_full + n_masked) * (part + 1), a.parts_div);
    T = cur.left = hi - lo;
    run_full = max(0, min(hi, n_full) - lo);
    masked_lo = max(0, lo - n_full);
    if (T > 0) {
      cur.masked = run_full == 0;
      cur.in_phase = cur.masked ? T : run_full;
      cur_seek(cur.masked ? masked_lo : lo);
    }
  }

  // ---- cooperative tile loads, straight from global memory into LDS, through buffer descriptors.
  //      Local: a tile image is copied as it is, wavefront w issuing instruction i for its 1 KiB
  //      block WAVES i + w (descriptor base + scalar offset + one constant per-lane offset).
  //      Images of the global mode: the same from the cursor's tile.  Rows: wavefront w takes rows
  //      16 w .. + 15, an instruction 64 bytes of each (the four lanes of a row adjacent), in LDS [16-row group][64-byte column block][row].
  //      Of a K row's four 16-byte granules in a block, granule c lies at place c ^ (row % 16 / 4), so
  //      that the 16 lanes an operand read serves together (one granule column, 16 rows) touch 256
  //      different bytes; V is kept straight: half a wavefront's transposing read takes 4 rows =
  //      256 consecutive bytes.  A tile's descriptor ends behind its last valid row: the rows after
  //      it arrive as zeros.
  constexpr int WAVES = PC_FA_WAVES;
  constexpr int T_LD = D / 8 / WAVES;              // load instructions per wavefront per tile
  constexpr int IMG_BYTES = 64 * D * 2;
  typedef __attribute__((address_space(3))) void* lptr_t;
  const int n_img = (a.n_rows + 63) / 64;
  const __amdgpu_buffer_rsrc_t k_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)kbase, 0, n_img * IMG_BYTES, 0x00020000);
  const __amdgpu_buffer_rsrc_t v_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)vbase, 0, n_img * IMG_BYTES, 0x00020000);
  const int ld_goff = 1024 * wave_s + 16 * lane;
  // what the (global) loads of the cursor's tile need
  struct TileLoad { const uint16_t* k; const uint16_t* v; int bytes, k_off, v_off; };
  auto tile_load = [&]() __attribute__((always_inline)) {
    TileLoad x;
    x.k = cur.k; x.v = cur.v;
    if (MODE == PC_FA_IMAGES) { x.bytes = x.v_off = x.k_off = 0; return x; }
    x.bytes = (min(cur.cut, 64) - 1) * cur.row_bytes + 2 * D;
    int id = tid;                                  // recomputed per tile: the loop has no registers to spare
    asm volatile("" : "+v"(id));
    x.v_off = (id / 4) * cur.row_bytes + 16 * (id % 4);            // row 16 wave + lane / 4
    x.k_off = x.v_off ^ (id & 48);                                 // ^ 16 (lane / 16); rows start at multiples of 64 bytes
    return x;
  };
  auto load_rows_i = [&](const uint16_t* base, int bytes, int off, uint16_t* dst, int i) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lptr_t)(dst + 512 * (T_LD * wave_s + i)), 16, off, 64 * i, 0, 0);
  };
  auto load_image_i = [&](const uint16_t* base, uint16_t* dst, int i) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, IMG_BYTES, 0x00020000);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lptr_t)(dst + 512 * (WAVES * i + wave_s)), 16, ld_goff, 1024 * WAVES * i, 0, 0);
  };
  // (tile t into the buffers of tile `to`)
  auto load_k_i = [&](const TileLoad& x, int t, int to, int i) __attribute__((always_inline)) {
    if (MODE == PC_FA_ROWS)
      load_rows_i(x.k, x.bytes, x.k_off, k_lds(to), i);
    else if (MODE == PC_FA_IMAGES)
      load_image_i(x.k, k_lds(to), i);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(k_rsrc, (lptr_t)(k_lds(to) + 512 * (WAVES * i + wave_s)), 16,
                                               ld_goff, t * IMG_BYTES + 1024 * WAVES * i, 0, 0);
  };
  auto load_v_i = [&](const TileLoad& x, int t, int to, int i) __attribute__((always_inline)) {
    if (MODE == PC_FA_ROWS)
      load_rows_i(x.v, x.bytes, x.v_off, v_lds(to), i);
    else if (MODE == PC_FA_IMAGES)
      load_image_i(x.v, v_lds(to), i);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(v_rsrc, (lptr_t)(v_lds(to) + 512 * (WAVES * i + wave_s)), 16,
                                               ld_goff, t * IMG_BYTES + 1024 * WAVES * i, 0, 0);
  };
  // s_waitcnt vmcnt(N): N newest loads of this wavefront may still be in flight
#define PC_WAIT_VMCNT(N) __builtin_amdgcn_s_waitcnt(0x0F70 | ((N) & 15) | (((N) >> 4) << 14))

  // ---- Q^T as B operand, NB 32-row blocks: lane holds query n of each, d = 16*ks + 8*hf .. +7.
  //      The softmax scale and log2(e) are folded into Q before its rounding to bf16 (local: they ride on
  //      the rotation table), so the first product yields logits in log2 units and the exponent needs
  //      no multiply.  (Global: the rows arrive rotated, scaled and rounded, see rope_q_kernel.)
  //
  // The wavefront's 32 query rows are fetched with coalesced loads (a load instruction covers whole rows,
  // 1 KiB contiguous where the rows are adjacent) and handed to the lanes that own them through a
  // private, XOR-swizzled LDS area in the V buffers of tiles 1 and 2; a gather straight into the operand
  // layout (every lane its own row) would touch 32 to 64 cache lines per instruction.  The table holds two
  // pairs' (cos, sin) of consecutive rows side by side, so the lanes of 32 rows read it straight into
  // registers, 16 bytes each (one pair, 8 bytes: twice the instructions, 2000 cycles more).  The first tiles
  // (K 0, V 0, K 1) are asked for behind the queries: one memory latency in front of the first product
  // instead of two.  Cycles of a workgroup in front of its loop and behind it,
  // 12 x 1550 rows, 32 / 8 heads, with the table through LDS, 64-bit addresses a row, tiles after the rotation ->
  // now: queries 4470 -> 5600, rotation 4300 -> 2690, tiles 1840 -> 510, output 2310 -> 1840 (a tile takes 2400);
  // the launch 331 -> 318 us, 20 x 500 85.8 -> 82, 36 x 4096 of 32 / 32 heads 4434 -> 4367, 8 x 8192 3637 -> 3613.
  bf16x8 bq[NB][KS];
  static_assert(NB == 1, "the staging areas are sized for one row block per wavefront");
  constexpr int PPR = D / 8;                      // 16-byte pieces per row
  constexpr int RPL = PC_WAVE / PPR;              // rows per load instruction
  constexpr int NLD = 32 / RPL;                   // load instructions per 32 rows
  my_row[0] = row0 + n;
  my_t[0] = pos_of(my_row[0]);
  max_key[0] = min(my_row[0], n_valid - 1);
  // local: the wavefront's rows of q and o through descriptors that end behind the sequence's last row
  const int row0_s = row0_wg + 32 * wave_s, rows_left = min(seq_rows - row0_s, 32);
  const int qo_stride = a.n_q_heads * (2 * D);
  const int qo_bytes = rows_left > 0 ? (rows_left - 1) * qo_stride + 2 * D : 0;
  const long long qo_at = (((long long)seq * a.n_rows + (rows_left > 0 ? row0_s : 0)) * a.n_q_heads + h) * D;
  Limit lim0 = {};
  {
    // (global: addresses from an opaque copy of the lane index, so that the epilogue's, which are alike, are
    // not kept in registers across the loop, which has none to spare: 4 spills instead of 24)
    int l = lane;
    if (GLOBAL) asm volatile("" : "+v"(l));
    const int l_row = l / PPR, l_piece = l % PPR, n = l % 32, hf = l / 32;
    uint16_t* st_q = smem + SM::KBUF * SM::K_ELEMS + SM::V_ELEMS + wave * (32 * D);
    u32x4 rq[NLD];
    u32x4 cs[GLOBAL ? 1 : KS / 2][4];              // (cos, sin) x scale of the lane's row, pairs 16 ks + 8 hf + 2 e, + 1
    if (GLOBAL) {
#pragma unroll
      for (int i = 0; i < NLD; ++i)
        rq[i] = pc_load_once((const u32x4*)((const uint16_t*)a.q + row_at(min(row0 + RPL * i + l_row, seq_rows - 1)) * D + 8 * l_piece));
    } else {
      const __amdgpu_buffer_rsrc_t q_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)((const uint16_t*)a.q + qo_at), 0, qo_bytes, 0x00020000);
      const int q_off = l_row * qo_stride + 16 * l_piece;
#pragma unroll
      for (int i = 0; i < NLD; ++i) rq[i] = __builtin_amdgcn_raw_buffer_load_b128(q_rsrc, q_off, RPL * i * qo_stride, PC_BUF_NT);
      const __amdgpu_buffer_rsrc_t t_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)a.table, 0, HALF * a.table_rows * 8, 0x00020000);
      const int t_off = 16 * (4 * hf * a.table_rows + row0 + n);
#pragma unroll
      for (int ks = 0; ks < KS / 2; ++ks)
#pragma unroll
        for (int e = 0; e < 4; ++e) cs[ks][e] = __builtin_amdgcn_raw_buffer_load_b128(t_rsrc, t_off, 16 * (8 * ks + e) * a.table_rows, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    if (!GLOBAL || T > 0) {
      const TileLoad ld = GLOBAL ? tile_load() : TileLoad{};
#pragma unroll
      for (int i = 0; i < T_LD; ++i) load_k_i(ld, 0, 0, i);
#pragma unroll
      for (int i = 0; i < T_LD; ++i) load_v_i(ld, 0, 0, i);
      if (GLOBAL) { lim0 = {cur.cut, cur.c0}; cur_next(); }
      const TileLoad ld1 = GLOBAL ? tile_load() : TileLoad{};
#pragma unroll
      for (int i = 0; i < T_LD; ++i) load_k_i(ld1, min(1, T - 1), 1, i);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int r = RPL * i + l_row;
      *(u32x4*)(st_q + (r * PPR + (l_piece ^ (r % PPR))) * 8) = rq[i];
    }
    PC_FA_WAVE_LDS_SYNC();
    auto piece = [&](int p) __attribute__((always_inline)) { return *(const u32x4*)(st_q + (n * PPR + (p ^ (n % PPR))) * 8); };
#pragma unroll
    for (int ks = 0; ks < (GLOBAL ? KS : KS / 2); ++ks) {
      const u32x4 x1 = piece(2 * ks + hf);
      if (GLOBAL) { bq[0][ks] = *(const bf16x8*)&x1; continue; }
      const u32x4 x2 = piece(2 * ks + hf + PPR / 2);         // the row's second half
      u32x4 ra, rbv;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const u32x4 cw = cs[GLOBAL ? 0 : ks][e];
        const float c0x = __uint_as_float(cw[0]), c0y = __uint_as_float(cw[1]), c1x = __uint_as_float(cw[2]), c1y = __uint_as_float(cw[3]);
        const float x1l = bf16_lo_to_f32(x1[e]), x1h = bf16_hi_to_f32(x1[e]);
        const float x2l = bf16_lo_to_f32(x2[e]), x2h = bf16_hi_to_f32(x2[e]);
        ra[e] = pack_bf16x2(x1l * c0x - x2l * c0y, x1h * c1x - x2h * c1y);
        rbv[e] = pack_bf16x2(x2l * c0x + x1l * c0y, x2h * c1x + x1h * c1y);
      }
      bq[0][ks] = *(bf16x8*)&ra;
      bq[0][ks + KS / 2] = *(bf16x8*)&rbv;
    }
  }

  // A operand of the second product from row-major V, V^T(d = n, 8 keys): two transposing reads of
  // 4 keys each.  16 lanes point at 4 rows x 16 columns (8 bytes a lane) and receive a column's 4 rows.
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  auto read_v_rows = [&](const uint16_t* p) __attribute__((always_inline)) {
    union { s16x4 h[2]; bf16x8 v; } x;
    typedef __attribute__((address_space(3))) s16x4* rptr_t;
    x.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((rptr_t)p);
    x.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((rptr_t)(p + 4 * 32));
    return x.v;
  };
  floatx16 o_acc[NB][DB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int r = 0; r < 16; ++r) o_acc[nb][db][r] = 0.f;
  // Softmax state per row: reference m_run (log2 units), row sum l_run, and -m_run replicated
  // over an accumulator tile: it is the C operand of the first MFMA of every S^T, so S^T comes
  // out of the matrix pipe already relative to the reference.
  float m_run[NB], l_run[NB];
  floatx16 negm[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    m_run[nb] = 0.f; l_run[nb] = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) negm[nb][r] = 0.f;
  }
  const int krow = pc_key_of_row(n);               // LDS row this lane feeds into MFMA row n

  // A step is 32 keys.  Step j reads K rows / V^T columns 32 (j & 1) .. + 31 of tile j >> 1.
  // S^T of step j lives in s_buf[j & 1], its probabilities P^T (bf16) in p_buf[j & 1].
  floatx16 s_buf[2][NB];                           // [step parity][row block]
  u32x4 p_buf[2][NB][2];                            // [step parity][row block][16-key k-step], bf16 pairs

  // Per-lane element offsets of the MFMA A operands inside a tile.  Image: K granule
  // (2 ks + hf, 32 (j & 1) + krow), V^T granule (4 (j & 1) + 2 ts + hf, 32 db + n).  Rows: K
  // granule 2 ks + hf of row 32 (j & 1) + krow, whose place in its block changes by one bit between
  // even and odd ks; V keys 8 hf .. + 3 of the column group (lane / 16) % 2.  Everything but the
  // lane's own part is a compile-time offset of the LDS read.
  int k_base, v_base;
  if (MODE == PC_FA_ROWS) {
    k_base = (krow / 16) * (16 * D) + (krow % 16) * 32 + ((hf ^ (krow % 16 / 4)) * 8);
    v_base = (8 * hf + (lane % 16) / 4) * 32 + 16 * ((lane / 16) % 2) + 4 * (lane % 4);
  } else {
    k_base = (hf * 64 + krow) * 8;
    v_base = (hf * D + n) * 8;
  }
  auto read_k = [&](int tile, int half, int ks) __attribute__((always_inline)) {
    return MODE == PC_FA_ROWS ? *(const bf16x8*)(smem + ((tile + 32 * D * half + k_base) ^ (16 * (ks % 2))) + 512 * (ks / 2))
                  : *(const bf16x8*)(smem + tile + 32 * 8 * half + k_base + 2 * ks * 64 * 8);
  };
  auto read_v = [&](const uint16_t* tile, int half, int ts, int db) __attribute__((always_inline)) {
    return MODE == PC_FA_ROWS ? read_v_rows(tile + 32 * D * half + v_base + 16 * D * ts + 512 * db)
                  : *(const bf16x8*)(tile + 4 * half * D * 8 + v_base + 2 * ts * D * 8 + 32 * db * 8);
  };

  // MFMA A operands, read from LDS one region ahead of their use
  bf16x8 ka[KS], va[2][DB];                        // K rows of a step; V^T [16-key k-step][d block]
  using no_mask = std::integral_constant<bool, false>;
  using with_mask = std::integral_constant<bool, true>;
  using yes = std::integral_constant<bool, true>;
  using no = std::integral_constant<bool, false>;

  // One step of the software pipeline, j = the step whose softmax runs now.  A region is NM
  // slices of [one MFMA, at most one LDS operand read, a few vector-ALU instructions], and the
  // compiler may not move instructions across a slice boundary, so the three pipes are fed
  // evenly by construction instead of by the scheduler's heuristics:
  //   region 1:  MFMA  O^T += V^T(j-1) P^T(j-1)     LDS  K(j+1) operands
  //              VALU  row maxima of S^T(j), reference update, first part of P^T(j)
  //   (rare)     rescale O after the reference of some row moved
  //   region 2:  MFMA  S^T(j+1) = K(j+1) Q^T        LDS  V^T(j) operands
  //              VALU  rest of P^T(j) = exp2(S^T(j) - m)
  // Register r of a row block at lane half hf is key 32 j + 16 (r / 8) + 8 hf + (r % 8).
  // Lazy rescale: the reference m_run of a row only moves when the step maximum exceeds it by
  // more than `window` (log2 units), 8 as a rule; until then p = exp2(s - m_run) <= 256 and O, l keep their scale.  The P V
  // products of step j - 1 (old reference) are all issued in region 1, so O is rescaled after it.
  // has_pv / has_qk are compile-time: the first step has no previous P V, the last no next K Q^T.
  // Steps that lie wholly above a wavefront's rows on the diagonal: those inside the loop are
  // not skipped, their logits are masked to -inf and add exact zeros (straight-line code keeps
  // the register allocation of the loop tight); the ones at the very end (the last period and
  // the last step) are left out per wavefront, see the end of the main loop.
  constexpr int NM = NB * KS;                      // MFMAs per region (= 2 NB DB)
  constexpr int MAX_SL = NM / 4;                   // slices of region 1 that take the row maxima
  constexpr int NG = 16 * NB + 1;                  // probability groups per step
  // groups placed in region 1: the share of its free slices among all slices that take groups
  constexpr int G1 = NG * (NM - MAX_SL - 1) / (2 * NM - MAX_SL - 1);
  // A mask hides the keys behind the row's last visible one; the step's first key counts as key
  // `k0`.  A (global) tile's limits: its valid keys, and its first key's position where the segment
  // is causal.
  auto step = [&](auto mask_tag, auto has_pv, auto has_qk, auto has_ld, const Limit& lim, float window, int j, int k0,
                  int t_ld, const TileLoad& ld, floatx16(&s_cur)[NB],
                  floatx16(&s_next)[NB], u32x4(&p_cur)[NB][2],
                  const u32x4(&p_prev)[NB][2]) __attribute__((always_inline)) {
    constexpr bool MASK = decltype(mask_tag)::value;
    constexpr bool PV = decltype(has_pv)::value, QK = decltype(has_qk)::value, LD = decltype(has_ld)::value;
    const int kt = k_at((j + 1) >> 1);
    const uint16_t* vt = v_lds(j >> 1);
    float t[NB], alpha[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) { t[nb] = 0.f; alpha[nb] = 1.f; }
    bool grow_any = false;
    // probability e (0..31: row block e / 16, register e % 16) of this step
    // The probabilities of a step go through two stages, one stage per group: group g takes
    // the exp2 of element g and the sum / bf16 pack of element g - 1, so no instruction waits on
    // the one issued just before it.  Element e is register e % 16 of row block e / 16.  Opaque
    // uses pin each group to the slice it is written in: without them the compiler sinks this
    // (side-effect-free) arithmetic past slice boundaries.
    float pr[16 * NB];
    auto prob_group = [&](int g) __attribute__((always_inline)) {
      if (g >= 1 && g - 1 < 16 * NB) {
        const int e = g - 1, nb = e / 16, r = e % 16;
        l_run[nb] += pr[e];
        asm volatile("" : "+v"(l_run[nb]));
        if (r % 2 == 1) {
          uint32_t w = pack_bf16x2(pr[e - 1], pr[e]);
          asm volatile("" : "+v"(w));
          p_cur[nb][r / 8][(r % 8) / 2] = w;
        }
      }
      if (g < 16 * NB) {
        pr[g] = __builtin_amdgcn_exp2f(s_cur[g / 16][g % 16]);
        asm volatile("" : "+v"(pr[g]));
      }
    };
    // ---------------- region 1
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      if (PV) {
        const int ts = i / (NB * DB), db = (i / NB) % DB, nb = i % NB;
        o_acc[nb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
            va[ts][db], *(const bf16x8*)&p_prev[nb][ts], o_acc[nb][db], 0, 0, 0);
      }
      if (QK && i < KS) ka[i] = read_k(kt, (j + 1) & 1, i);
      if (LD && i >= NM - 2 * T_LD) {               // one tile-load instruction per slice
        const int li = i - (NM - 2 * T_LD);
        if (li < T_LD) load_k_i(ld, t_ld, t_ld, li);
        else load_v_i(ld, t_ld, t_ld, li - T_LD);
      }
      if (MASK && i == 0) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int key = k0 + 16 * (r / 8) + 8 * hf + (r % 8);
            if (key > (GLOBAL ? min(lim.cut - 1, my_t[nb] - lim.c0) : max_key[nb])) s_cur[nb][r] = -INFINITY;
          }
      }
      if (i < MAX_SL) {
        // the 8 links of each row block's maximum chain, 8 / MAX_SL per slice
#pragma unroll
        for (int q = i * (8 / MAX_SL); q < (i + 1) * (8 / MAX_SL); ++q)
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) {
            if (q == 0) t[nb] = fmaxf(fmaxf(s_cur[nb][0], s_cur[nb][1]), s_cur[nb][2]);
            else if (q < 7) t[nb] = fmaxf(fmaxf(t[nb], s_cur[nb][2 * q + 1]), s_cur[nb][2 * q + 2]);
            else t[nb] = fmaxf(t[nb], s_cur[nb][15]);
          }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) asm volatile("" : "+v"(t[nb]));
      }
      if (i == MAX_SL) {
        // Does any row's maximum leave the window of its reference?  S^T is already relative
        // to the reference, so the test is a compare with a constant; everything else is rare.
        bool grow = !PV;                            // the first step sets the reference exactly
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) grow |= t[nb] > window;
        grow_any = __any(grow);
        if (grow_any) {
#pragma unroll
          for (int nb = 0; nb < NB; ++nb) {
            const float tm = pc_xhalf_max(t[nb]);   // both lane halves hold keys of the same row
            const bool gr = PV ? tm > window : tm != -INFINITY;
            const float delta = gr ? tm : 0.f;
            alpha[nb] = PV ? __builtin_amdgcn_exp2f(-delta) : 1.0f;   // nothing accumulated before the first step
            m_run[nb] += delta;
            l_run[nb] *= alpha[nb];
#pragma unroll
            for (int r = 0; r < 16; ++r) { negm[nb][r] = -m_run[nb]; s_cur[nb][r] -= delta; }
          }
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) asm volatile("" : "+v"(l_run[nb]));
      }
#pragma unroll
      for (int g = 0; g < G1; ++g)
        if (MAX_SL + 1 + g * (NM - MAX_SL - 1) / G1 == i) prob_group(g);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (grow_any) {
      // O sits in the accumulation registers; walk it one 16-register block at a time so this
      // rare path needs only a handful of temporaries
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int db = 0; db < DB; ++db) {
#pragma unroll
          for (int r = 0; r < 16; ++r) o_acc[nb][db][r] *= alpha[nb];
          __builtin_amdgcn_sched_barrier(0);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    // ---------------- region 2
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      if (QK) {
        const int ks = i / NB, nb = i % NB;
        s_next[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[ks], bq[nb][ks], ks == 0 ? negm[nb] : s_next[nb], 0, 0, 0);
      }
      if (i < KS) {
        const int ts = i / DB, db = i % DB;
        va[ts][db] = read_v(vt, j & 1, ts, db);
      }
#pragma unroll
      for (int g = G1; g < NG; ++g)
        if ((g - G1) * NM / (NG - G1) == i) prob_group(g);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // first S^T of a workgroup: operands of step 0, then the product
  auto first_qk = [&](floatx16(&s)[NB]) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) ka[ks] = read_k(k_at(0), 0, ks);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) s[nb][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        s[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[ks], bq[nb][ks], s[nb], 0, 0, 0);
  };
  // trailing O^T += V^T(j) P^T(j) of the last step
  auto last_pv = [&](const u32x4(&p)[NB][2]) __attribute__((always_inline)) {
#pragma unroll
    for (int ts = 0; ts < 2; ++ts)
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          o_acc[nb][db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(va[ts][db], *(const bf16x8*)&p[nb][ts], o_acc[nb][db], 0, 0, 0);
  };

  // Keeps k_base / v_base opaque in a loop: it stops the compiler from hoisting a dozen
  // loop-invariant per-lane addresses out of the loop into registers the loop cannot spare;
  // recomputing them costs a few vector-ALU instructions per period.
  auto opaque_bases = [&]() __attribute__((always_inline)) { asm volatile("" : "+v"(k_base), "+v"(v_base)); };
  // One period = two steps.  Period p runs steps 2p+1 and 2p+2: it reads K tile p + 1 and the
  // V^T tiles p and p + 1 (the latter only its first half, for the next period's first step).
  // After its barrier it issues the loads of K(p + 2) and V(p + 2), one instruction per slice
  // of its first step, into the buffers that held K(p) and V(p - 1), both last read before
  // that barrier; the next period's barrier waits for them.  Past the last tile the loads repeat
  // tile T - 1 into buffers nobody reads again, which keeps the loop free of branches.
  const TileLoad no_ld = {};
  const Limit no_lim = {};
  // K 0, V 0 and K 1 have landed, and every wavefront has left its staging area: V 1 may move in
  if (!GLOBAL || T > 0) {
    PC_WAIT_VMCNT(0);
    __syncthreads();
    const TileLoad ld = GLOBAL ? tile_load() : TileLoad{};   // the cursor is on tile 1
#pragma unroll
    for (int i = 0; i < T_LD; ++i) load_v_i(ld, min(1, T - 1), 1, i);
  }
  if (!GLOBAL) {
    const TileLoad ld = {};                        // (images: addressed by tile number)
    first_qk(s_buf[0]);
    step(with_mask{}, no{}, yes{}, no{}, no_lim, 8.0f, 0, 0, 0, no_ld, s_buf[0], s_buf[1], p_buf[0], p_buf[1]);
    auto period = [&](auto mask_tag, int p) __attribute__((always_inline)) {
      opaque_bases();
      PC_WAIT_VMCNT(0);
      __syncthreads();
      const int t_ld = min(p + 2, T - 1);
      step(mask_tag, yes{}, yes{}, yes{}, no_lim, 8.0f, 2 * p + 1, 32 * (2 * p + 1), t_ld, ld, s_buf[1], s_buf[0], p_buf[1], p_buf[0]);
      step(mask_tag, yes{}, yes{}, no{}, no_lim, 8.0f, 2 * p + 2, 32 * (2 * p + 2), 0, no_ld, s_buf[0], s_buf[1], p_buf[0], p_buf[1]);
    };
    const int n_plain = min(T - 1, max(0, (J0 - 1) / 2));   // periods whose steps need no mask
    // Last step with a key visible to any row of this wavefront.  On the diagonal the steps
    // behind it hold only masked keys: the wavefront keeps the workgroup's barrier count but
    // leaves their arithmetic out (the tile loads of the last period only repeat tile T - 1).
    const int j_need = __builtin_amdgcn_readfirstlane(min(row0 + 32 * NB - 1, n_valid - 1) >> 5);
    const bool skip_last_period = T >= 2 && j_need < 2 * T - 3;
    const int n_periods = skip_last_period ? T - 2 : T - 1;
    int p = 0;
    for (; p < min(n_plain, n_periods); ++p) period(no_mask{}, p);
    for (; p < n_periods; ++p) period(with_mask{}, p);
    if (skip_last_period) {
      PC_WAIT_VMCNT(0);
      __syncthreads();                                       // the barrier of period T - 2
    }
    // ---- last period: step 2T-1 and the trailing P V
    PC_WAIT_VMCNT(0);
    __syncthreads();
    if (j_need >= 2 * T - 1) {
      step(with_mask{}, yes{}, no{}, no{}, no_lim, 8.0f, 2 * T - 1, 32 * (2 * T - 1), 0, no_ld, s_buf[1], s_buf[0], p_buf[1], p_buf[0]);
      last_pv(p_buf[1]);
    } else {
      last_pv(p_buf[0]);                                     // P V of the last step that ran (an even one)
    }
  } else if (T > 0) {
    // The same pipeline over the cursor's tiles; a tile carries its own limits (tile p + 2 is the
    // cursor's, lim0 / lim1 belong to tiles p and p + 1).  Every row that sees a key of the run sees
    // its first one, so the first step sets the row's reference as in the local kernel.
    first_qk(s_buf[0]);
    step(with_mask{}, no{}, yes{}, no{}, lim0, 8.0f, 0, 0, 0, no_ld, s_buf[0], s_buf[1], p_buf[0], p_buf[1]);
    auto period = [&](auto mask_tag, int p) __attribute__((always_inline)) {
      // the cursor is on tile p + 1 here
      const Limit lim1 = {cur.cut, cur.c0};
      // at the start of a segment the reference moves up to the step's maximum, however little it
      // grew, as it does at the start of a run: probability 1 is exact in bf16, so a short
      // segment's heaviest key carries no rounding error
      const float window = cur.seg_start ? 0.0f : a.window;
      cur_next();                                            // tile p + 2 (or the last one again)
      const TileLoad ld = tile_load();
      const int t_ld = min(p + 2, T - 1);
      opaque_bases();
      PC_WAIT_VMCNT(0);
      __syncthreads();
      step(mask_tag, yes{}, yes{}, yes{}, lim0, 8.0f, 2 * p + 1, 32, t_ld, ld, s_buf[1], s_buf[0], p_buf[1], p_buf[0]);
      step(mask_tag, yes{}, yes{}, no{}, lim1, window, 2 * p + 2, 0, 0, no_ld, s_buf[0], s_buf[1], p_buf[0], p_buf[1]);
      lim0 = lim1;
    };
    int p = 0;
    for (; p < run_full - 1; ++p) period(no_mask{}, p);      // tiles p and p + 1 are both unmasked
    for (; p < T - 1; ++p) period(with_mask{}, p);
    PC_WAIT_VMCNT(0);
    __syncthreads();
    // does the last tile's second half hold a key that some row of the wavefront sees?
    if (__builtin_amdgcn_readfirstlane(min(lim0.cut - 1, pc_div(min(row0 + 31, rows_wg - 1), a.group_div) - lim0.c0)) >= 32) {
      step(with_mask{}, yes{}, no{}, no{}, lim0, 8.0f, 2 * T - 1, 32, 0, no_ld, s_buf[1], s_buf[0], p_buf[1], p_buf[0]);
      last_pv(p_buf[1]);
    } else {
      last_pv(p_buf[0]);
    }
  } else {
    __syncthreads();                               // every wavefront has left its staging area
  }

  // ---- epilogue: lane halves hold disjoint key subsets of the same query
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const float l = pc_xhalf_sum(l_run[nb]);
    const float inv_l = l > 0.f ? 1.f / l : 0.f;
    const float lse = l > 0.f ? m_run[nb] * PC_LN2 + logf(l) : -INFINITY;
    if (GLOBAL && a.n_parts > 1) {
      if (my_row[nb] < seq_rows) {
        const long long prow = (((long long)seq * a.n_parts + part) * a.n_rows + pc_div(my_row[nb], a.group_div)) * a.n_q_heads + h + pc_mod(my_row[nb], G, a.group_div);
        float* po = a.part_o + prow * D;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            floatx4 x = {o_acc[nb][db][4 * i] * inv_l, o_acc[nb][db][4 * i + 1] * inv_l,
                         o_acc[nb][db][4 * i + 2] * inv_l, o_acc[nb][db][4 * i + 3] * inv_l};
            *(floatx4*)(po + 32 * db + 8 * i + 4 * hf) = x;
          }
        if (hf == 0) a.part_lse[prow] = lse;
      }
    } else {
      // The lane that owns a query holds its output row in 8-byte pieces; stored from there,
      // an instruction would touch 32 rows.  The rows go through a swizzled staging area in the
      // K buffers (nobody reads K after the last barrier: the last step has no next S^T) and
      // leave as whole 16-byte-per-lane rows, 1 KiB per instruction where rows are adjacent.
      static_assert(NB == 1 && PC_FA_WAVES * 32 * D <= SM::KBUF * SM::K_ELEMS, "staging area is the K buffers");
      uint16_t* st_o = smem + wave * (32 * D);
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          uint2 x;
          x.x = pack_bf16x2(o_acc[nb][db][4 * i] * inv_l, o_acc[nb][db][4 * i + 1] * inv_l);
          x.y = pack_bf16x2(o_acc[nb][db][4 * i + 2] * inv_l, o_acc[nb][db][4 * i + 3] * inv_l);
          const int p = 4 * db + i;                             // 16-byte piece of the row; half hf of it
          *(uint2*)(st_o + (n * PPR + (p ^ (n % PPR))) * 8 + 4 * hf) = x;
        }
      PC_FA_WAVE_LDS_SYNC();
      const int l_row = lane / PPR, l_piece = lane % PPR;
      const __amdgpu_buffer_rsrc_t o_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)((uint16_t*)a.o + qo_at), 0, qo_bytes, 0x00020000);
#pragma unroll
      for (int k = 0; k < NLD; ++k) {
        const int r = RPL * k + l_row;
        const u32x4 x = *(const u32x4*)(st_o + (r * PPR + (l_piece ^ (r % PPR))) * 8);
        if (!GLOBAL) {                                         // (rows behind the sequence: dropped)
          __builtin_amdgcn_raw_buffer_store_b128(x, o_rsrc, l_row * qo_stride + 16 * l_piece, RPL * k * qo_stride, PC_BUF_NT);
          continue;
        }
        const int grow = row0 + 32 * nb + r;
        if (grow < seq_rows)
          pc_store_once((u32x4*)((uint16_t*)a.o + row_at(grow) * D + 8 * l_piece), x);
      }
      if (my_row[nb] < seq_rows && hf == 0 && a.lse)
        a.lse[((long long)seq * a.n_q_heads + h + (GLOBAL ? pc_mod(my_row[nb], G, a.group_div) : 0)) * a.n_rows + pos_of(my_row[nb])] = lse;
    }
  }
}

#include "prefill_wide.h"

template <int D, int MODE>
__global__ __launch_bounds__(PC_FA_THREADS, 2) void flash_fwd_kernel(PcFlashArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  int bid = blockIdx.x;
  if (MODE == PC_FA_LOCAL) {
    static_assert(PC_FA_THREADS == 256, "pc_chunk_sum");
    if (bid < a.sum_blocks) {
      if (bid < a.n_seq) pc_chunk_sum(a.sum.blk_sum, a.sum.chunk_score, a.sum.per_chunk, bid, (float*)smem);
      return;
    }
    bid -= a.sum_blocks;
  }
  flash_workgroup<D, MODE>(a, bid, smem);
}

// Local and global attention in one launch, for a layer whose selections are done before the local
// attention (which nothing of the path reads): the global workgroups stand in front, so that they and their
// latencies hide behind the local ones.  glob_blocks of them, padded to `front`, a multiple of 8, so that
// the local ones keep their XCDs.
template <int D>
__global__ __launch_bounds__(PC_FA_THREADS, 2) void flash_both_kernel(PcFlashArgs local, PcFlashArgs global, int glob_blocks,
                                                                      int front) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  const int bid = blockIdx.x;
  if (bid >= front) flash_workgroup<D, PC_FA_LOCAL>(local, bid - front, smem);
  else if (bid < glob_blocks) flash_workgroup<D, PC_FA_ROWS>(global, bid, smem);
}

template <int MODE>
__global__ __launch_bounds__(PC_FA_THREADS, 1) void flash_wide_kernel(PcFlashArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  int bid = blockIdx.x;
  if (bid < a.sum_blocks) {
    if (bid < a.n_seq) pc_chunk_sum(a.sum.blk_sum, a.sum.chunk_score, a.sum.per_chunk, bid, (float*)smem);
    return;
  }
  wide_workgroup<MODE>(a, bid - a.sum_blocks, smem);
}
template <int MODE>
__global__ __launch_bounds__(PC_FA_THREADS, 1) void flash_both_wide_kernel(PcFlashArgs local, PcFlashArgs global, int glob_blocks,
                                                                           int front) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  const int bid = blockIdx.x;
  if (bid >= front) wide_workgroup<MODE>(local, bid - front, smem);
  else if (bid < glob_blocks) flash_workgroup<FW_D, PC_FA_ROWS>(global, bid, smem);
}

// The global part's reference follows the maximum at every tile there (window 0), as it starts anew in every part of
// a run that is cut: one long run is then at least as exact as the parts it replaces (512 rows over 8 x 2048
// keys, from 64 bits: 4 parts 5.52e-3, one part 5.46e-3, with the lazy window 5.54e-3).  It costs 2 % of a launch
// that holds global workgroups only, and does not show here.

// Workgroups of a call without those of the chunk sums; fills in what the launcher decides
template <bool GLOBAL>
static long long flash_blocks(PcFlashArgs& a) {
  const int G = a.n_q_heads / a.n_kv_heads;
  const long long rows_wg = GLOBAL ? (long long)a.n_rows * G : a.n_rows;
  const long long n_qt = (rows_wg + PC_FA_BM - 1) / PC_FA_BM;
  // Local: a group that cannot fill an XCD's 64 workgroup slots by itself is interleaved with
  // others, up to three rounds of slots, so that the long Q tiles of all of them start first.  A
  // group that can keeps its XCD to itself: its short tiles then overlap the start of the next
  // group's long ones.  Measured (us, 1 group at a time / 4 / 8): 1 x 4096 rows, 32 heads (32 tiles a
  // group) 158 / 142 / 142, 36 of them 4632 / 4532 / 4571, 2 x 3300 200 / 180 / 182; 12 x 2214 ragged,
  // 32 / 8 heads (72 tiles a group) 323 / 385 / 392, 16 x 8192 (256) 7485 / 7490 / 7508.
  const long long per_group = n_qt * (GLOBAL ? a.n_parts : G), groups_xcd = (long long)a.n_seq * a.n_kv_heads / 8;
  a.group_batch = 1;
  if (!GLOBAL && per_group < 64 && groups_xcd > 1) {
    const long long m = (192 + per_group - 1) / per_group, batches = (groups_xcd + m - 1) / m;
    a.group_batch = (int)((groups_xcd + batches - 1) / batches);           // batches of equal size
  }
  const int last = (int)(groups_xcd % a.group_batch);
  a.group = G; a.n_qt = (int)n_qt;
  a.group_div = pc_div_by(G); a.qt_div = pc_div_by(a.n_qt); a.heads_div = pc_div_by(a.n_kv_heads);
  a.per_group_div = pc_div_by((int)per_group); a.per_batch_div = pc_div_by((int)(a.group_batch * per_group));
  a.batch_div = pc_div_by(a.group_batch); a.last_div = pc_div_by(last);
  a.parts_div = pc_div_by(GLOBAL ? a.n_parts : 1);
  return (long long)a.n_seq * a.n_kv_heads * per_group;
}

// ---- 64 rows a wavefront (wide_workgroup)
// Heads of a workgroup: the largest power of two up to 8 that divides the group; 1: rows of one head
static int wide_heads(int G) { return G % 8 == 0 ? 8 : G % 4 == 0 ? 4 : G % 2 == 0 ? 2 : 1; }
// Which local calls take it, and the heads of a workgroup (0: 32 rows a wavefront).  A workgroup costs 12000 cycles around
// its loop that nothing else on its CU hides, and 256 CUs hold one each: long rows, more than 1.25 rounds of them.  Of
// full Q tiles from 1984 rows on, with two heads, whose Q tile is 128 positions too, from 3072, with one head, whose causal
// end is four tiles long, from 7680; where the 32 rows' last Q tile of 128 is half empty and the narrower one here is not,
// from 1280 on.  Calls with the pre-pass (us, 32 rows a wavefront / 64; sequences x rows): 32 / 8 heads, 1 x 2500 68.6 / 71.9, 1 x
// 3000 90.8 / 86.5, 2 x 1300 53.4 / 48.1, 36 x 1300 693 / 653, 4 x 1500 98.5 / 102.0, 36 x 1500 810 / 820, 16 x 1920 1.007 times as long,
// 16 x 1984 0.975, 16 x 2048 0.975, 36 x 3000 2653 / 2501, 4 x 8192 1834 / 1710; 16 / 4, 2 x 2500 70.1 / 72.6, 12 x 1300 124 / 115, 8 x 1500
// 97.5 / 100.4, 1 x 8192 282 / 228; 8 / 1, 8 x 1300 51.6 / 45.7, 24 x 1408 1.017 times as long, 4 x 4096 152 / 126; 4 / 2, 24 x 2000 129 /
// 132, 12 x 2500 101 / 95, 16 x 2500 126 / 127, 36 x 3000 362 / 353, 8 x 4096 154 / 136.  One head: 32 / 32, 8 x 2000 384 / 402, 8 x
// 4096 1199 / 1172, 4 x 6144 1200 / 1222, 8 x 8192 4054 / 3907; 7 / 7, 8 x 6144 1.053 times as long, 8 x 7680 0.986.
int pc_flash_wide(int n_seq, int n_rows, int n_q_heads, int n_kv_heads, int head_dim) {
  if (head_dim != FW_D || n_q_heads > 65536) return 0;       // (64 rows of q or o: 32-bit byte offsets)
  const int heads = wide_heads(n_q_heads / n_kv_heads), P = 256 / heads;
  const bool half_empty = (n_rows + PC_FA_BM - 1) / PC_FA_BM * PC_FA_BM > (n_rows + P - 1) / P * P;
  const int least = heads == 1 ? 7680 : half_empty ? 1280 : heads == 2 ? 3072 : 1984;
  const long long workgroups = (long long)n_seq * (n_q_heads / heads) * ((n_rows + P - 1) / P);
  return n_rows >= least && workgroups > 320 ? heads : 0;
}
// ... and which block attentions over tile images (the 8-bit cache), in the same parts: where 32 rows a wavefront put
// two workgroups on a CU (one alone has its LDS to itself: nothing to gain), no block of 256 packed rows has an empty
// half, and a workgroup's run is 32 tiles or more of 64 or more in all, worth the start.  Whole cache build and attention (us, 32 rows a wavefront /
// 64), sequences x segments x keys, rows (tiles a run): 32 / 8 heads, 4 x 8 x 2048, 512 (264) 691 / 648, 2 x 8 x 2048, 512 (132) 379 /
// 359, 3 x 8 x 2048, 512 (66) 565 / 544, 3 x 8 x 2048, 128 (51) 285 / 277, 2 x 8 x 2048, 128 (32) 205 / 203, 3 x 4 x 1500, 512 (26) 265 /
// 268, 2 x 8 x 700, 256 (23) 118 / 119, 1 x 8 x 2048, 128 (16) 127 / 130, 2 x 8 x 700, 128 (11) 102 / 105; of fewer in all: 4 x 4 x 400, 384 (34) 104 / 106,
// 3 x 4 x 400, 512 (36) 103 / 105; half empty: 3 x 8 x 2048, 24
// (12) 237 / 261, 32 / 32, 2 x 8 x 2048, 128 (32) 607 / 645.
int pc_flash_wide_images(int n_seq, int n_rows, int n_q_heads, int n_kv_heads, int head_dim, long long n_tiles, int n_parts) {
  const long long rows = (long long)n_rows * (n_q_heads / n_kv_heads), blocks = (rows + PC_FA_BM - 1) / PC_FA_BM;
  return head_dim == FW_D && blocks % 2 == 0 && blocks * n_seq * n_kv_heads * n_parts > 256 &&
         n_tiles >= 64 && n_tiles >= 32LL * n_parts;
}
static bool wide_images_fits(const PcFlashArgs& a) {
  long long tiles = 0;
  for (const PcKvGroup& kg : a.grp) tiles += (long long)kg.n * ((kg.cap + 63) / 64);
  return a.images && pc_flash_wide_images(a.n_seq, a.n_rows, a.n_q_heads, a.n_kv_heads, a.head_dim, tiles, a.n_parts);
}
static int wide_fits(const PcFlashArgs& a) { return pc_flash_wide(a.n_seq, a.n_rows, a.n_q_heads, a.n_kv_heads, a.head_dim); }
// As flash_blocks.  Groups of fewer than two rounds of an XCD's 32 slots are interleaved up to two rounds: 16 x
// 2000 rows, 32 / 8 heads, 573 -> 558 us.
static long long wide_blocks(PcFlashArgs& a) {
  const int G = a.n_q_heads / a.n_kv_heads;
  a.wide_heads = a.global ? 1 : wide_heads(G);               // (global: packed rows)
  a.group = G / a.wide_heads;
  const int P = 256 / a.wide_heads;
  a.n_qt = (int)(((a.global ? (long long)a.n_rows * G : a.n_rows) + P - 1) / P);
  if (a.global) {
    a.group_batch = 1;
    a.group_div = pc_div_by(G); a.heads_div = pc_div_by(a.n_kv_heads); a.qt_div = pc_div_by(a.n_qt);
    a.parts_div = pc_div_by(a.n_parts); a.per_batch_div = pc_div_by(a.n_qt * a.n_parts);
    a.batch_div = a.last_div = pc_div_by(1); a.per_group_div = pc_div_by((int)((long long)a.n_seq * a.n_kv_heads % 8));
    return (long long)a.n_seq * a.n_kv_heads * a.n_qt * a.n_parts;
  }
  const long long per_group = (long long)a.n_qt * a.group, n_groups = (long long)a.n_seq * a.n_kv_heads, groups_xcd = n_groups / 8;
  a.group_batch = 1;
  if (per_group < 64 && groups_xcd > 1) {
    const long long m = (64 + per_group - 1) / per_group, batches = (groups_xcd + m - 1) / m;
    a.group_batch = (int)((groups_xcd + batches - 1) / batches);
  }
  a.group_div = pc_div_by(a.group); a.heads_div = pc_div_by(a.n_kv_heads);
  a.per_batch_div = pc_div_by((int)(a.group_batch * per_group));
  a.batch_div = pc_div_by(a.group_batch); a.last_div = pc_div_by((int)(groups_xcd % a.group_batch));
  a.per_group_div = pc_div_by((int)(n_groups % 8));
  return n_groups * per_group;
}

// image loads address one (sequence, head) region with 32-bit byte offsets
static bool images_too_long(const PcFlashArgs& a) {
  return ((long long)a.n_rows + 63) / 64 * 64 * a.head_dim * 2 >= 0x7fffffffLL;
}

template <int D, int MODE>
static int launch_flash_t(const PcFlashArgs& args, hipStream_t st) {
  constexpr bool GLOBAL = MODE != PC_FA_LOCAL;
  PcFlashArgs a = args;
  using SM = FlashSmem<D>;
  auto kern = flash_fwd_kernel<D, MODE>;
  static std::atomic<uint64_t> raised{0};          // one per instantiation of this launcher
  const int lds_rc = pc_raise_dynamic_lds((const void*)kern, SM::BYTES, raised);
  if (lds_rc != PC_OK) return lds_rc;
  a.sum_blocks = !GLOBAL && a.sum.chunk_score ? (a.n_seq + 7) / 8 * 8 : 0;
  const long long blocks = flash_blocks<GLOBAL>(a) + a.sum_blocks;
  if (blocks == 0) return PC_OK;
  if (blocks > 0x7fffffffLL || (!GLOBAL && images_too_long(a))) return PC_ERR_SHAPE;
  PcProfScope prof(PC_KERNEL_FLASH, st);
  hipLaunchKernelGGL(kern, dim3((unsigned)blocks), dim3(PC_FA_THREADS), SM::BYTES, st, a);
  PC_LAUNCH_CHECK();
  return PC_OK;
}

template <int D>
static int launch_flash_both_t(const PcFlashArgs& local, const PcFlashArgs& global, hipStream_t st) {
  PcFlashArgs l = local, g = global;
  using SM = FlashSmem<D>;
  static std::atomic<uint64_t> raised{0};
  const int lds_rc = pc_raise_dynamic_lds((const void*)flash_both_kernel<D>, SM::BYTES, raised);
  if (lds_rc != PC_OK) return lds_rc;
  const long long glob_blocks = flash_blocks<true>(g), front = (glob_blocks + 7) / 8 * 8, blocks = front + flash_blocks<false>(l);
  if (blocks > 0x7fffffffLL || images_too_long(l)) return PC_ERR_SHAPE;
  PcProfScope prof(PC_KERNEL_FLASH, st);
  hipLaunchKernelGGL(flash_both_kernel<D>, dim3((unsigned)blocks), dim3(PC_FA_THREADS), SM::BYTES, st, l, g, (int)glob_blocks, (int)front);
  PC_LAUNCH_CHECK();
  return PC_OK;
}
template <int MODE>
static int launch_wide_t(const PcFlashArgs& args, hipStream_t st) {
  PcFlashArgs a = args;
  static std::atomic<uint64_t> raised{0};
  const int lds_rc = pc_raise_dynamic_lds((const void*)flash_wide_kernel<MODE>, FW_LDS_BYTES, raised);
  if (lds_rc != PC_OK) return lds_rc;
  a.sum_blocks = !a.global && a.sum.chunk_score ? (a.n_seq + 7) / 8 * 8 : 0;
  const long long blocks = wide_blocks(a) + a.sum_blocks;
  if (blocks > 0x7fffffffLL || (!a.global && images_too_long(a))) return PC_ERR_SHAPE;
  PcProfScope prof(PC_KERNEL_FLASH, st);
  hipLaunchKernelGGL(flash_wide_kernel<MODE>, dim3((unsigned)blocks), dim3(PC_FA_THREADS), FW_LDS_BYTES, st, a);
  PC_LAUNCH_CHECK();
  return PC_OK;
}
template <int MODE>
static int launch_both_wide_t(const PcFlashArgs& local, const PcFlashArgs& global, hipStream_t st) {
  PcFlashArgs l = local, g = global;
  static_assert(FlashSmem<FW_D>::BYTES <= FW_LDS_BYTES, "both fit");
  static std::atomic<uint64_t> raised{0};
  const int lds_rc = pc_raise_dynamic_lds((const void*)flash_both_wide_kernel<MODE>, FW_LDS_BYTES, raised);
  if (lds_rc != PC_OK) return lds_rc;
  const long long glob_blocks = flash_blocks<true>(g), front = (glob_blocks + 7) / 8 * 8, blocks = front + wide_blocks(l);
  if (blocks > 0x7fffffffLL || images_too_long(l)) return PC_ERR_SHAPE;
  PcProfScope prof(PC_KERNEL_FLASH, st);
  hipLaunchKernelGGL(flash_both_wide_kernel<MODE>, dim3((unsigned)blocks), dim3(PC_FA_THREADS), FW_LDS_BYTES, st, l, g, (int)glob_blocks, (int)front);
  PC_LAUNCH_CHECK();
  return PC_OK;
}
int pc_launch_flash_both(const PcFlashArgs& local, const PcFlashArgs& global, hipStream_t st) {
  if (const int heads = wide_fits(local))
    return heads > 1 ? launch_both_wide_t<PC_FW_PAIR>(local, global, st) : launch_both_wide_t<PC_FW_HEAD>(local, global, st);
  return local.head_dim == 128 ? launch_flash_both_t<128>(local, global, st) : launch_flash_both_t<64>(local, global, st);
}

// Parts of the global attention's keys next to a local attention of n_seq sequences of n_rows rows, 1 to
// `most`: the least estimated time of both, which share 512 slots.  A slot holds a workgroup for some 10 us +
// 1.54 us a 64-key tile (local; 2.1 global; head_dim 64 1.0 and 1.4), and the launch does not end before the
// longest; cutting costs the merge, 5 us + what it reads.  Whole layers (us), chosen parts / others: 1 x 3584 + 512 rows, 32 /
// 32 heads, 1 x 1792 kept: 1 part 227 / 2 parts 235, 4 244; 12 x 2011 + 203, 32 / 8, 5 x 701: 1 626 / 2 629, 4 634; 4 x 4096 +
// 128, 32 / 8, 4 x 3000: 1 626 / 2 630, 16 639; 2 x 3000 + 64, 32 / 8, 2 x 2500: 2 212 / 1 227, 4 214, 16 226; 8 x 1500 + 512, 16 /
// 4, 8 x 1400: 3 254 / 1 356, 2 257, 8 267; 1 x 1000 + 24, 24 / 8 of 64 values, 1 x 900: 2 49.7 / 1 54.9, 3 48.3, 16 51.9.
// With 64 rows a wavefront 256 slots, 8 us + 1.45 a tile (local), and the global ones have their CU to themselves (1.27).
int pc_flash_both_parts(int n_seq, int n_rows, int n_q, int n_q_heads, int n_kv_heads, int head_dim, long long n_tiles, int most) {
  const int wide = pc_flash_wide(n_seq, n_rows, n_q_heads, n_kv_heads, head_dim);
  const int heads = wide ? wide : 1, rows = wide ? 256 / heads : PC_FA_BM;
  const double loc_us = wide ? 1.45 : head_dim == 128 ? 1.54 : 1.0, glob_us = wide ? 1.27 : head_dim == 128 ? 2.1 : 1.4;
  const double slots = wide ? 256.0 : 512.0, start_us = wide ? 8.0 : 10.0;
  double work = 0.0, longest = 0.0;
  for (int r0 = 0; r0 < n_rows; r0 += rows) {
    const double us = start_us + loc_us * ((std::min(n_rows, r0 + rows) + 63) / 64);
    work += us * n_seq * (n_q_heads / heads);
    longest = us;
  }
  const long long wgs = (long long)n_kv_heads * (((long long)n_q * (n_q_heads / n_kv_heads) + PC_FA_BM - 1) / PC_FA_BM);
  const double merge_us = 0.4 + (double)n_q * n_q_heads * head_dim * 4 / 7e6;
  int best_p = 1;
  double best = 0.0;
  for (int p = 1; p <= most && p <= n_tiles; ++p) {
    const double each = 10.0 + glob_us * (double)((n_tiles + p - 1) / p);
    const double us = std::max((work + each * (double)(wgs * p)) / slots, std::max(longest, each)) + (p > 1 ? 5.0 + merge_us * p : 0.0);
    if (p == 1 || us < best) { best = us; best_p = p; }
  }
  return best_p;
}

int pc_launch_flash(const PcFlashArgs& a, hipStream_t st) {
  if (a.global && wide_images_fits(a)) return launch_wide_t<PC_FW_IMAGES>(a, st);
  if (const int heads = a.global ? 0 : wide_fits(a)) return heads > 1 ? launch_wide_t<PC_FW_PAIR>(a, st) : launch_wide_t<PC_FW_HEAD>(a, st);
  if (a.head_dim == 128)
    return !a.global ? launch_flash_t<128, PC_FA_LOCAL>(a, st)
                     : (a.images ? launch_flash_t<128, PC_FA_IMAGES>(a, st) : launch_flash_t<128, PC_FA_ROWS>(a, st));
  return !a.global ? launch_flash_t<64, PC_FA_LOCAL>(a, st)
                   : (a.images ? launch_flash_t<64, PC_FA_IMAGES>(a, st) : launch_flash_t<64, PC_FA_ROWS>(a, st));
}

#define PC_FA_PARTS_MAX 64
#define PC_FA_PARTS_WGS 2048
#define PC_FA_PARTS_MIN 4
int pc_flash_parts(int n_seq, int n_rows, int n_q_heads, int n_kv_heads, int head_dim, long long n_tiles) {
  // The parts that minimise the estimated time of the tile kernel and the merge together.
  // Measured (parts swept from 1 to 32 over eight shapes; head_dim 128): a workgroup costs about
  // 10 us (query rows, first tiles, output) and 1.27 us a tile alone on its CU, 2.1 us next to
  // another (512 fit at a time); the merge 5 us, and 0.4 us and 7 TB/s for every part.  E.g. 512
  // rows, 32 / 8 heads, 8 x 2048 keys (128 workgroups a part): 342 us with 1 part, 205 with 2, 163
  // with 4, 176 with 8, 208 with 16; four such sequences: 575 with 1 part, 625 with 2.
  const long long G = n_q_heads / n_kv_heads;
  const long long wgs = (long long)n_seq * n_kv_heads * ((n_rows * G + PC_FA_BM - 1) / PC_FA_BM);
  const double pair_us = head_dim == 128 ? 2.1 : 1.4, alone_us = head_dim == 128 ? 1.27 : 0.95;
  const double merge_us = 0.4 + (double)n_seq * n_rows * n_q_heads * head_dim * 4 / 7e6;
  // At most 2048 workgroups (four rounds) or 4 parts, whichever is more: the partials of a call stay
  // within a bound that pc_flash_part_rows can state.  By the estimate above that costs 0.07 % on
  // average and 14 % at worst (just above one round) over 1 to 64 sequences x 17 to 2048 rows.
  const long long p_wgs = wgs * PC_FA_PARTS_MIN < PC_FA_PARTS_WGS ? PC_FA_PARTS_WGS / wgs : PC_FA_PARTS_MIN;
  const long long p_cap = p_wgs < PC_FA_PARTS_MAX ? p_wgs : PC_FA_PARTS_MAX;
  const int p_max = (int)(n_tiles < 1 ? 1 : (n_tiles > p_cap ? p_cap : n_tiles));
  int best_p = 1;
  double best = 0.0;
  for (int p = 1; p <= p_max; ++p) {
    const long long n = wgs * p;
    const double tiles = (double)((n_tiles + p - 1) / p);
    const double run = n <= 256 ? tiles * alone_us + 10.0 : (double)((n + 511) / 512) * (tiles * pair_us + 10.0);
    const double cost = run + (p > 1 ? 5.0 + merge_us * p : 0.0);
    if (p == 1 || cost < best) { best = cost; best_p = p; }
  }
  return best_p;
}

size_t pc_flash_part_rows(size_t rows, long long n_tiles, int has_self) {
  // at most PC_FA_PARTS_MAX parts and one per tile; at most PC_FA_PARTS_WGS workgroups of PC_FA_BM rows or
  // PC_FA_PARTS_MIN parts.  A self segment asks for one part more, so that the room grows with it too.
  const size_t parts = (size_t)(n_tiles < 1 ? 1 : (n_tiles > PC_FA_PARTS_MAX ? PC_FA_PARTS_MAX : n_tiles)) + (has_self ? 1 : 0);
  const size_t by_wgs = (size_t)PC_FA_PARTS_WGS * PC_FA_BM, by_parts = rows * PC_FA_PARTS_MIN;
  const size_t bound = by_wgs > by_parts ? by_wgs : by_parts;
  return rows * parts < bound ? rows * parts : bound;
}
