// Cumulative query->key attention scores (Eq. 5-6):
//   tok_score[c, g, j] = sum over the query heads h of KV group g and over the voting rows r
//                        (the last w_obs rows of the chunk sequence) of P[c, h, r, j],  j < w,
// where P[c, h, r, :] is the causal softmax row of Eq. 1 over ALL keys of the sequence.
// The probability block [H_q, w_obs, L] is never written to memory: it is recomputed.
//
// Accuracy.  The scores decide which tokens are kept, so logits are computed to about fp32
// accuracy although they run on the bf16 matrix cores: q and k are rotated in fp32 and split
// into bf16 hi + lo parts, and q.k = hi.hi + hi.lo + lo.hi (three MFMAs; the lo.lo term is
// below 2^-16 relative).
//
// Two passes over the keys, both fully parallel over key blocks of 128 to 1024 keys (the largest
// block that still leaves every CU several workgroups: a workgroup's start-up is then spread over
// more keys); the query columns come rotated, scaled and split as MFMA operands (prep.hip):
//   pass 1  (S^T = K Q^T, a lane owns a voting row)  per-block running max / sum of every
//           voting row -> workspace [c, g, key block, column] (m, l)
//   the blocks' (m, l) are combined into the row logsumexp by pass 2 itself while they are few, by a
//   small kernel in between otherwise
//   pass 2  (S = Q K^T, a lane owns a key)           recompute the logits, p = exp2(s - lse)
//           and sum p over the columns (voting rows x heads of the group) for each key
//           -> tok_score
// Pass 2 also leaves the sum of its tok_score block; those are added per chunk in a fixed order
// (deterministic) -> chunk_score, by a last kernel in the standalone call and by workgroups of the
// attention launch that follows in the prefill call.
//
// Fused K/V pre-pass.  Inside pc_chunk_prefill_attn pass 1 takes over the work of
// kv_prepass_kernel (switched on by its output pointers): it already reads every key row once and rotates it in
// fp32, and the bf16 "hi" half of the split IS the rotated key rounded to bf16, so in its first
// round over the columns it also writes the rotated keys (row-major cache) and the K tile images,
// and moves V through LDS into the V^T tile images.  The keys are then read from HBM once for
// both jobs, and rotated once.
//
// Any number of voting rows: up to 128 (row, head) columns of a KV group (4 blocks of 32) are kept in
// registers while the keys stream by (scores_kernel).  More columns turn the loops round
// (scores_many_kernel): 128 keys are staged once and stay in LDS, the columns stream by.
#include "pc_common.h"
#include <math.h>
#include <type_traits>

#define PC_SC_THREADS 256
#define PC_SC_WAVES 4
#define PC_SC_KB 256        // keys per workgroup
#define PC_SC_KB_SMALL 128  // where 256 leave CUs idle
#define PC_SC_SMALL_WGS 350
#define PC_SC_KB_MAX 1024   // the largest
#define PC_SC_TILE 64       // keys staged in LDS at a time
#define PC_SC_KB_MANY 128   // keys per workgroup with more than 4 column blocks; half where that leaves CUs idle
#define PC_SC_LSE_BLOCKS 64 // up to this many blocks of pass 1, pass 2 combines their (max, sum) itself
#define PC_SC_LOG2E 1.4426950408889634f
// orders a wavefront's own LDS writes and reads (no other wavefront involved)
#define PC_SC_WAVE_LDS_SYNC()                                \
  do {                                                       \
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   \
    __builtin_amdgcn_wave_barrier();                         \
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");   \
  } while (0)

struct PcScoreArgs {
  const uint16_t* k;       // [C, L, H_kv, D] before RoPE
  const int32_t* chunk_lens; // [C] context rows per chunk or nullptr (= w)
  const float2* table;     // [L, D/2] (cos, sin)
  float2* ml;              // workspace [C, H_kv, n_kb, n_cols] (max in log2 units, sum)
  float* lse2;             // workspace [C, H_kv, 32 n_cb] row logsumexp in log2 units (+inf behind n_cols)
  const uint16_t* q_split; // workspace: the query columns as MFMA operands (PcScoreQueries)
  float* tok_score;        // [C, H_kv, w]
  int L, w, w_obs, n_q_heads, n_kv_heads, n_kb, n_cols, n_cb;
  PcDiv heads_div, obs_div;  // by n_kv_heads, w_obs
  int kb_keys;             // keys per workgroup: 64 to 1024 (pass 1 at most 512 when WPC == 4)
  float* blk_sum;          // workspace [C, H_kv, n_kb]: sum of each pass-2 block's tok_score
  // pre-pass duties of pass 1 (all nullptr: off): V rows in, rotated keys / K images / V^T images out
  const uint16_t* v;       // [C, L, H_kv, D]
  uint16_t* k_rope;        // [C, L, H_kv, D] or nullptr
  uint16_t* k_img;         // tile images [C][H_kv][Lp / 64][64 * D]
  uint16_t* v_img;
  int Lp;                  // L rounded up to 64
};

// K tile staging, split in two so that the loads of the next tile are in flight while the matrix
// cores work on this one: fetch (global -> registers), stage (rotate in fp32, split hi / lo,
// registers -> LDS).  A thread always handles the same 8 rotation pairs, of rows RP apart, so it
// reads (cos, sin) from the table once, for its first row, and turns them by the constant angle of
// RP rows from item to item (one complex multiplication per pair in fp32, at most kb_keys / RP - 1
// <= 31 in a chain: ~1e-7 relative per link).
// PRE: pass 1, which also carries the pre-pass duties where they are wanted (`pre`).
// OWN (tiles of 128): a wavefront's 32 rows of the tile lie side by side in LDS, 32 wave .. + 31, where it alone reads them:
// local row m is row RP (m / RW) + RW wave + m % RW of the tile.  Otherwise a row lies at its place.
template <int D, int TILE, bool PRE, bool OWN = false>
struct PcKeyStage {
  static constexpr int HALF = D / 2, KSTRIDE = D + 8;
  static constexpr int ITEMS = TILE * (HALF / 8) / PC_SC_THREADS;      // per thread and tile
  static constexpr int RP = PC_SC_THREADS / (HALF / 8);                // rows between a thread's items
  static constexpr int RW = PC_WAVE / (HALF / 8);                      // rows of a wavefront's item
  static_assert(ITEMS >= 1 && TILE * (HALF / 8) % PC_SC_THREADS == 0, "tile / thread mismatch");
  static_assert(!OWN || RW * ITEMS == 32, "32 rows a wavefront");
  // V: a thread takes 8 consecutive keys x 4 values (eight 8-byte loads), transposes them in
  // registers and stores four 16-byte granules of the V^T image, (8 keys, d) each
  static constexpr int V_ALL = (TILE / 8) * (D / 4);                   // such items per tile
  static constexpr int V_ITEMS = (V_ALL + PC_SC_THREADS - 1) / PC_SC_THREADS;
  int tid, st_r0, st_i0;
  bool pre;
  uint4 pf_x1[ITEMS], pf_x2[ITEMS];
  float2 cs_cur[8], cs_step[8];
  u32x2 pf_v[PRE ? V_ITEMS : 1][8];

  __device__ __forceinline__ void begin(const PcScoreArgs& a, int thread, int first_key, bool with_pre) {
    tid = thread; pre = with_pre;
    st_r0 = tid / (HALF / 8); st_i0 = (tid % (HALF / 8)) * 8;
    const float4* c4 = (const float4*)(a.table + (long long)min(first_key + st_r0, a.L - 1) * HALF + st_i0);
    const float4* s4 = (const float4*)(a.table + (long long)min(RP, a.L - 1) * HALF + st_i0);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float4 cv = c4[e], sv4 = s4[e];
      cs_cur[2 * e] = make_float2(cv.x, cv.y); cs_cur[2 * e + 1] = make_float2(cv.z, cv.w);
      cs_step[2 * e] = make_float2(sv4.x, sv4.y); cs_step[2 * e + 1] = make_float2(sv4.z, sv4.w);
    }
  }
  __device__ __forceinline__ void fetch(const PcScoreArgs& a, int c, int g, int key0) {
#pragma unroll
    for (int u = 0; u < ITEMS; ++u) {
      const int row = min(key0 + st_r0 + u * RP, a.L - 1);
      const uint16_t* krow = a.k + (((long long)c * a.L + row) * a.n_kv_heads + g) * D;
      pf_x1[u] = pc_load_once((const uint4*)(krow + st_i0));
      pf_x2[u] = pc_load_once((const uint4*)(krow + HALF + st_i0));
    }
    if (pre) {
#pragma unroll
      for (int u = 0; u < V_ITEMS; ++u) {
        const int it = tid + u * PC_SC_THREADS;
        const int row0 = key0 + 8 * (it / (D / 4)), d4 = (it % (D / 4)) * 4;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          pf_v[u][j] = u32x2{0u, 0u};                                // rows past the sequence: zeros in the image
          if (it < V_ALL && row0 + j < a.L)
            pf_v[u][j] = __builtin_nontemporal_load(
                (const u32x2*)(a.v + (((long long)c * a.L + row0 + j) * a.n_kv_heads + g) * D + d4));
        }
      }
    }
  }
  __device__ __forceinline__ void stage(const PcScoreArgs& a, int c, int g, int key0, uint16_t* k_hi, uint16_t* k_lo) {
    const long long img_cg = ((long long)c * a.n_kv_heads + g) * (a.Lp / 64);   // first tile image of (c, g)
    if (pre) {
      // V^T tile images: granule (c8, d) = V[keys 8 c8 .. 8 c8 + 7][d]; word e of a granule pairs
      // the values of keys 2 e and 2 e + 1 (one byte permute per word)
#pragma unroll
      for (int u = 0; u < V_ITEMS; ++u) {
        const int it = tid + u * PC_SC_THREADS;
        const int row0 = key0 + 8 * (it / (D / 4)), d4 = (it % (D / 4)) * 4;
        if (it < V_ALL && row0 < a.Lp) {
          uint16_t* img = a.v_img + (img_cg + row0 / 64) * (64LL * D) + (((row0 % 64) / 8) * D + d4) * 8;
          uint4 gr[4];
          uint32_t* gw = (uint32_t*)gr;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const u32x2 r0 = pf_v[u][2 * e], r1 = pf_v[u][2 * e + 1];
            gw[0 * 4 + e] = __builtin_amdgcn_perm(r1.x, r0.x, 0x05040100u);   // d4 + 0: low halves
            gw[1 * 4 + e] = __builtin_amdgcn_perm(r1.x, r0.x, 0x07060302u);   // d4 + 1: high halves
            gw[2 * 4 + e] = __builtin_amdgcn_perm(r1.y, r0.y, 0x05040100u);   // d4 + 2
            gw[3 * 4 + e] = __builtin_amdgcn_perm(r1.y, r0.y, 0x07060302u);   // d4 + 3
          }
          // ordinary stores: an instruction writes 16 bytes of every 64 a lane owns, and the
          // last-level cache merges the four pieces of a line (with the streaming hint they
          // reached memory as partial lines: 2.4 times slower)
#pragma unroll
          for (int dd = 0; dd < 4; ++dd) *(uint4*)(img + dd * 8) = gr[dd];
        }
      }
    }
#pragma unroll
    for (int u = 0; u < ITEMS; ++u) {
      const int r = st_r0 + u * RP, i0 = st_i0;
      const uint32_t aw[4] = {pf_x1[u].x, pf_x1[u].y, pf_x1[u].z, pf_x1[u].w};
      const uint32_t bw[4] = {pf_x2[u].x, pf_x2[u].y, pf_x2[u].z, pf_x2[u].w};
      uint32_t h1[4], l1[4], h2[4], l2[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float2 c0 = cs_cur[2 * e], c1 = cs_cur[2 * e + 1];
        const float x1l = bf16_lo_to_f32(aw[e]), x1h = bf16_hi_to_f32(aw[e]);
        const float x2l = bf16_lo_to_f32(bw[e]), x2h = bf16_hi_to_f32(bw[e]);
        split_bf16x2(x1l * c0.x - x2l * c0.y, x1h * c1.x - x2h * c1.y, h1[e], l1[e]);
        split_bf16x2(x2l * c0.x + x1l * c0.y, x2h * c1.x + x1h * c1.y, h2[e], l2[e]);
      }
      const int at = (OWN ? 32 * (tid / PC_WAVE) + RW * u + tid % PC_WAVE / (HALF / 8) : r) * KSTRIDE + i0;
      *(uint4*)(k_hi + at) = make_uint4(h1[0], h1[1], h1[2], h1[3]);
      *(uint4*)(k_lo + at) = make_uint4(l1[0], l1[1], l1[2], l1[3]);
      *(uint4*)(k_hi + at + HALF) = make_uint4(h2[0], h2[1], h2[2], h2[3]);
      *(uint4*)(k_lo + at + HALF) = make_uint4(l2[0], l2[1], l2[2], l2[3]);
      if (pre) {
        // the hi halves are the rotated key rounded to bf16: the cache row and its K image granules
        const int row = key0 + r;
        const bool in_seq = row < a.L;
        const uint4 oa = in_seq ? make_uint4(h1[0], h1[1], h1[2], h1[3]) : make_uint4(0, 0, 0, 0);
        const uint4 ob = in_seq ? make_uint4(h2[0], h2[1], h2[2], h2[3]) : make_uint4(0, 0, 0, 0);
        if (in_seq && a.k_rope != nullptr) {
          uint16_t* dst = a.k_rope + (((long long)c * a.L + row) * a.n_kv_heads + g) * D;
          pc_store_once((uint4*)(dst + i0), oa);
          pc_store_once((uint4*)(dst + HALF + i0), ob);
        }
        if (row < a.Lp) {
          uint16_t* img = a.k_img + (img_cg + row / 64) * (64LL * D);
          pc_store_once((uint4*)(img + ((i0 / 8) * 64 + row % 64) * 8), oa);
          pc_store_once((uint4*)(img + (((HALF + i0) / 8) * 64 + row % 64) * 8), ob);
        }
      }
      // (cos, sin) of the thread's next row: angle + RP theta
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float cn = cs_cur[e].x * cs_step[e].x - cs_cur[e].y * cs_step[e].y;
        const float sn = cs_cur[e].y * cs_step[e].x + cs_cur[e].x * cs_step[e].y;
        cs_cur[e] = make_float2(cn, sn);
      }
    }
  }
};

// (chunk, KV head) of a workgroup: heads fastest in the grid's first dimension or, where that would pass its
// 2^32 threads, in the third
__device__ __forceinline__ int score_chunk(const PcScoreArgs& a) {
  return gridDim.z > 1 ? blockIdx.x : pc_div(blockIdx.x, a.heads_div);
}
__device__ __forceinline__ int score_head(const PcScoreArgs& a) {
  return gridDim.z > 1 ? blockIdx.z : blockIdx.x - pc_div(blockIdx.x, a.heads_div) * a.n_kv_heads;
}

// WPC = wavefronts per block of 32 columns.  With 4 or more column blocks (a GQA group of 4
// heads x 32 voting rows) a wavefront owns a column block and takes both 32-key halves of every
// 64-key tile (WPC = 1).  With fewer column blocks the wavefronts of a block share its keys
// instead of idling: WPC = 2 splits the halves of a 64-key tile, WPC = 4 (one column block, e.g.
// MHA with 32 voting rows) the four 32-key quarters of a 128-key tile.  Pass 2 is bound by its vector instructions at two
// wavefronts a SIMD (one wavefront issues one about every 5 cycles): without a barrier between staging and products,
// with the voting rows' positions computed for masked tiles only and twice the keys a workgroup, WPC = 4 takes 330 ->
// 277 us at 36 x 3584 keys of 32 heads, 19.5 -> 16.7 at 1 x 3584, 6.8 -> 6.0 at 4 x 512 keys of 8 heads of 64 values.
// (The staging of the next tile between the MFMAs of this one: 283, 17.6 and 5.3.  Pass 1 without the barriers 1189 ->
// 1203.)
template <int D, int PASS, int WPC>
__global__ __launch_bounds__(PC_SC_THREADS, 2) void scores_kernel(PcScoreArgs a) {
  // The pre-pass duties ride on pass 1 and are switched at run time (a.v_img != nullptr), so the
  // standalone score call and the fused one execute the same code and give the same bits.
  constexpr int KS = D / 16, KSTRIDE = D + 8;
  constexpr int TILE = WPC == 4 ? 2 * PC_SC_TILE : PC_SC_TILE;   // keys staged in LDS at a time
  constexpr int NSUB = TILE / 32;                                // 32-key sub-blocks per tile
  __shared__ __attribute__((aligned(16))) uint16_t k_hi[TILE * KSTRIDE];
  __shared__ __attribute__((aligned(16))) uint16_t k_lo[TILE * KSTRIDE];
  // pass 2 with four wavefronts a column block: each stages the 32 keys that it takes itself, so that none waits for
  // another, and a key's sum has one owner
  constexpr bool OWN = WPC == 4 && PASS == 2;
  constexpr int TOK_ROWS = OWN ? 1 : PC_SC_WAVES;
  __shared__ float tok_part[TOK_ROWS][PASS == 2 ? PC_SC_KB_MAX : 1];
  __shared__ float2 ml_part[PC_SC_WAVES][32];

  const int c = score_chunk(a), g = score_head(a), kblock = blockIdx.y;
  const int tid = threadIdx.x, lane = tid % PC_WAVE, wave = tid / PC_WAVE;
  const int hf = lane / 32, n = lane % 32;
  // a short chunk is [len context rows ; the query rows]: its voting rows end at len + w_q
  const int ctx_len = a.chunk_lens ? min(max(a.chunk_lens[c], 0), a.w) : a.w;
  const int first_obs = ctx_len + (a.L - a.w) - a.w_obs;
  const long long ml_base = (((long long)c * a.n_kv_heads + g) * a.n_kb) * a.n_cols;

  const float* lse2 = a.lse2 + ((long long)c * a.n_kv_heads + g) * (32 * a.n_cb);

  // pass 2: every wavefront accumulates its columns' share of the keys' sums in its own LDS row
  if (PASS == 2 && !OWN)
    for (int i = lane; i < a.kb_keys; i += PC_WAVE) tok_part[wave][i] = 0.f;

  const int kb0 = wave % WPC;                      // this wavefront's first sub-block of a tile
  const int cb = wave / WPC;                       // its column block
  const bool active = cb < a.n_cb;
  // ---- this lane's column as an MFMA operand
  const int col = min(32 * cb + n, a.n_cols - 1);
  bf16x8 qhi[KS], qlo[KS];
  {
    const int cols = min(a.n_cols, 32);            // a single block of fewer columns holds no others
    const uint16_t* src = a.q_split + ((((long long)c * a.n_kv_heads + g) * a.n_cb + min(cb, a.n_cb - 1)) * (4 * KS * cols) + hf * cols + min(n, cols - 1)) * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      qhi[ks] = *(const bf16x8*)(src + ks * cols * 16);
      qlo[ks] = *(const bf16x8*)(src + (KS + ks) * cols * 16);
    }
  }
  // pass 1: this lane's voting row (column) and its running statistics
  const int my_qrow = first_obs + pc_mod(col, a.w_obs, a.obs_div);
  float m_run = -INFINITY, l_run = 0.f;
  // keys that count: pass 1 the sequence's, pass 2 its context rows; the pre-pass wants all rows
  const bool pre = PASS == 1 && a.v_img != nullptr;
  const int key_end = PASS == 1 ? ctx_len + (a.L - a.w) : ctx_len;
  const int stage_end = pre ? a.L : key_end;
  typedef PcKeyStage<D, TILE, PASS == 1, OWN> Stage;
  Stage keys;
  keys.begin(a, tid, kblock * a.kb_keys, pre);
  if (kblock * a.kb_keys < stage_end) keys.fetch(a, c, g, kblock * a.kb_keys);

  // pass 2: the voting rows / logsumexp of the 16 result registers (rows of S).  Where pass 1 left few
  // blocks, every wavefront combines its columns' (max, sum) itself, while its first keys are on
  // their way: a lane half takes every other block.
  float lse_r[16];
  if (PASS == 2) {
    float lse = INFINITY;                                  // column 32 cb + n; exp2(-inf) = 0 for padding columns
    const int my_col = 32 * cb + n;
    if (active && my_col < a.n_cols && a.n_kb <= PC_SC_LSE_BLOCKS) {
      const float2* src = a.ml + ml_base + my_col;
      float M = -INFINITY, sum = 0.f;
      for (int kb = hf; kb < a.n_kb; kb += 8) {
        float2 v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = src[(long long)min(kb + 2 * i, a.n_kb - 1) * a.n_cols];
        float m_new = M;
#pragma unroll
        for (int i = 0; i < 4; ++i) m_new = fmaxf(m_new, v[i].x);
        if (sum > 0.f) sum *= exp2f(M - m_new);
        M = m_new;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (kb + 2 * i < a.n_kb && v[i].y > 0.f) sum += v[i].y * exp2f(v[i].x - M);
      }
      const float m_o = __shfl_xor(M, 32), s_o = __shfl_xor(sum, 32);
      const float top = fmaxf(M, m_o);
      float tot = 0.f;
      // the lower half's share first, on both sides: both halves hold the same bits
      const float m0 = hf ? m_o : M, s0 = hf ? s_o : sum, m1 = hf ? M : m_o, s1 = hf ? sum : s_o;
      if (s0 > 0.f) tot += s0 * exp2f(m0 - top);
      if (s1 > 0.f) tot += s1 * exp2f(m1 - top);
      lse = top + log2f(tot);
    } else if (active && my_col < a.n_cols) {
      lse = lse2[my_col];
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int in_cb = 8 * (r / 4) + 4 * hf + (r % 4);
      lse_r[r] = __shfl(lse, in_cb);
    }
  }

  // one loop body (not unrolled): leaves room for the prefetch registers
  const int n_tiles = a.kb_keys / TILE;
#pragma unroll 1
  for (int t = 0; t < n_tiles; ++t) {
    const int key0 = kblock * a.kb_keys + t * TILE;
    if (key0 >= stage_end) break;                         // uniform over the workgroup
    // (a thread's angles go on for 512 keys, 4 tiles: 16 items at 128 values, 15 links of a chain, 8 at 64; then they are read anew)
    if (OWN && t > 0 && t % (PC_SC_KB_MAX / 2 / TILE) == 0) keys.begin(a, tid, key0, pre);
    if (OWN) PC_SC_WAVE_LDS_SYNC(); else __syncthreads(); // previous tile fully consumed
    keys.stage(a, c, g, key0, k_hi, k_lo);
    if (OWN) PC_SC_WAVE_LDS_SYNC(); else __syncthreads();
    if (t + 1 < n_tiles && key0 + TILE < stage_end) keys.fetch(a, c, g, key0 + TILE);
    if (!active || key0 >= key_end) continue;
    // every key of the tile is visible to every voting row: no causal mask (all but the last
    // tiles of a sequence; the voting rows sit at its end)
    const bool unmasked = key0 + TILE - 1 <= first_obs;

#pragma unroll
    for (int kq = 0; kq < NSUB / WPC; ++kq) {
      const int kb = kb0 + kq * WPC;
      floatx16 s;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = 0.f;
      const uint16_t* ph = k_hi + (32 * kb + n) * KSTRIDE + 8 * hf;
      const uint16_t* pl = k_lo + (32 * kb + n) * KSTRIDE + 8 * hf;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8 kh = *(const bf16x8*)(ph + 16 * ks);
        const bf16x8 kl = *(const bf16x8*)(pl + 16 * ks);
        if (PASS == 1) {     // rows = keys, columns = voting rows
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kl, qhi[ks], s, 0, 0, 0);
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kh, qlo[ks], s, 0, 0, 0);
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kh, qhi[ks], s, 0, 0, 0);
        } else {             // rows = voting rows, columns = keys
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qhi[ks], kl, s, 0, 0, 0);
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qlo[ks], kh, s, 0, 0, 0);
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qhi[ks], kh, s, 0, 0, 0);
        }
      }
      if (PASS == 1) {
        float sv[16], tmax = -INFINITY;
        if (unmasked) {
#pragma unroll
          for (int r = 0; r < 16; ++r) { sv[r] = s[r]; tmax = fmaxf(tmax, sv[r]); }
        } else {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int key = key0 + 32 * kb + 8 * (r / 4) + 4 * hf + (r % 4);
            sv[r] = (key <= my_qrow) ? s[r] : -INFINITY;
            tmax = fmaxf(tmax, sv[r]);
          }
        }
        const float m_new = fmaxf(m_run, tmax);
        if (m_new > -INFINITY) {
          float sum = 0.f;
#pragma unroll
          for (int r = 0; r < 16; ++r) sum += __builtin_amdgcn_exp2f(sv[r] - m_new);
          l_run = l_run * __builtin_amdgcn_exp2f(m_run - m_new) + sum;
          m_run = m_new;
        }
      } else {
        const int in_tile = OWN ? Stage::RP * (n / Stage::RW) + Stage::RW * wave + n % Stage::RW : 32 * kb + n, key = key0 + in_tile;
        float sum = 0.f;
        if (unmasked) {       // padding columns carry lse = +inf: their p is 0 without a mask
#pragma unroll
          for (int r = 0; r < 16; ++r) sum += __builtin_amdgcn_exp2f(s[r] - lse_r[r]);
        } else {
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            const int cc = 32 * cb + 8 * (r / 4) + 4 * hf + (r % 4);
            const float p = __builtin_amdgcn_exp2f(s[r] - lse_r[r]);
            sum += (cc < a.n_cols && key <= first_obs + pc_mod(cc, a.w_obs, a.obs_div)) ? p : 0.f;
          }
        }
        sum += __shfl_xor(sum, 32);
        if (hf == 0) {
          if (OWN) tok_part[0][t * TILE + in_tile] = sum; else tok_part[wave][t * TILE + in_tile] += sum;
        }
      }
    }
  }

  if (PASS == 1) {
    // the lane halves hold disjoint keys of the same column; then the WPC wavefronts of the
    // column block (disjoint keys again) are combined in wavefront order
    const float m_o = __shfl_xor(m_run, 32), l_o = __shfl_xor(l_run, 32);
    float M = fmaxf(m_run, m_o);
    float l = 0.f;
    if (l_run > 0.f) l += l_run * exp2f(m_run - M);
    if (l_o > 0.f) l += l_o * exp2f(m_o - M);
    if (WPC > 1) {
      if (hf == 0) ml_part[wave][n] = make_float2(M, l);
      __syncthreads();
      if (kb0 == 0) {
        M = -INFINITY;
#pragma unroll
        for (int i = 0; i < WPC; ++i) M = fmaxf(M, ml_part[wave + i][n].x);
        l = 0.f;
#pragma unroll
        for (int i = 0; i < WPC; ++i) {
          const float2 v = ml_part[wave + i][n];
          if (v.y > 0.f) l += v.y * exp2f(v.x - M);
        }
      }
    }
    const int cc = 32 * cb + n;
    if (active && kb0 == 0 && hf == 0 && cc < a.n_cols)
      a.ml[ml_base + (long long)kblock * a.n_cols + cc] = make_float2(M, l);
  }

  if (PASS == 2) {
    __syncthreads();
    float blk = 0.f;                                         // this thread's share of the block's sum
    for (int i = tid; i < a.kb_keys; i += PC_SC_THREADS) {
      const int key = kblock * a.kb_keys + i;
      if (key < a.w) {
        float x = 0.f;
#pragma unroll
        for (int wv = 0; wv < TOK_ROWS; ++wv) x += tok_part[wv][i];
        x = key < ctx_len ? x : 0.f;
        a.tok_score[((long long)c * a.n_kv_heads + g) * a.w + key] = x;
        blk += x;
      }
    }
    // block sum in a fixed order: lanes (xor tree), then the wavefronts in order
#pragma unroll
    for (int off = PC_WAVE / 2; off > 0; off >>= 1) blk += __shfl_xor(blk, off);
    __syncthreads();                                         // tok_part is read no more: reuse its first floats
    if (lane == 0) tok_part[0][wave] = blk;
    __syncthreads();
    if (tid == 0) {
      float tot = 0.f;
#pragma unroll
      for (int wv = 0; wv < PC_SC_WAVES; ++wv) tot += tok_part[0][wv];
      a.blk_sum[((long long)c * a.n_kv_heads + g) * gridDim.y + kblock] = tot;
    }
  }
}

// ------------------------------------------------------------------------------------------
// More than 4 column blocks (many voting rows, e.g. every query row as Eq. 6 prints it).  Keeping
// columns in registers and streaming the keys would rotate, split and stage every key once per
// 128 columns.  Here a workgroup stages its 128 keys (hi and lo, 68 KiB) once and the columns
// stream by: a wavefront takes every fourth column block and reads it as ready MFMA operands
// (split once, in prep.hip) while the block before is multiplied.  No barrier and no
// conversion in the loop: bound by the matrix cores (96 MFMAs a block, 1.25 PFLOP/s where the chip is full) and, next
// to them, 64 exponentials a lane.  A product (32 keys x 32 columns) is a run of slices that the compiler may not mix:
// a k-step's three MFMAs, the LDS reads for three k-steps later, a share of the exponentials of the product before.
// Left to itself it waited for every operand read in front of its MFMA and put the exponentials behind the product.
// Compiler's order -> slices, the passes alone (us): 4 chunks of 2011 rows, 203 voting, 32 / 8 heads 77 + 57 -> 67 + 46,
// 12 138 + 125 -> 128 + 110, 16 x 7680, 512 voting 1460 + 1371 -> 1397 + 1293.  Minus the logsumexp as the products'
// C operand (no subtraction in front of the exponentials) was 7 % faster in pass 2, at 0.2 % more error: not taken.
// Every query row voting, pass 1 with the pre-pass + pass 2 (us), rounds of 128 columns over re-staged keys / the compiler's
// order / now: 12 ragged chunks of 2011 rows, 203 rows voting, 32 / 8 heads 324 + 305 / 215 + 154 / 135 + 91; 16 x 7680, 512
// voting 2052 + 2081 / 1487 + 1281 / 1335 + 1163; 36 x 3584, 32 / 32 heads 2805 + 2369 / 3019 + 1834 / 2807 + 1652 (the pre-pass,
// 1.25 ms of memory traffic, does not overlap the products).
template <int D, int PASS, int TILE>
__global__ __launch_bounds__(PC_SC_THREADS, D == 64 ? 3 : 2) void scores_many_kernel(PcScoreArgs a) {
  constexpr int KS = D / 16, KSTRIDE = D + 8, NSUB = TILE / 32;
  __shared__ __attribute__((aligned(16))) uint16_t k_hi[TILE * KSTRIDE];
  __shared__ __attribute__((aligned(16))) uint16_t k_lo[TILE * KSTRIDE];
  __shared__ float tok_part[PC_SC_WAVES][PASS == 2 ? TILE : 1];

  const int c = score_chunk(a), g = score_head(a), kblock = blockIdx.y, key0 = kblock * TILE;
  const int tid = threadIdx.x, lane = tid % PC_WAVE, wave = __builtin_amdgcn_readfirstlane(tid / PC_WAVE);
  const int hf = lane / 32, n = lane % 32;
  const int ctx_len = a.chunk_lens ? min(max(a.chunk_lens[c], 0), a.w) : a.w;
  const int first_obs = ctx_len + (a.L - a.w) - a.w_obs;
  const int key_end = PASS == 1 ? ctx_len + (a.L - a.w) : ctx_len;
  const bool pre = PASS == 1 && a.v_img != nullptr;
  const long long cg = (long long)c * a.n_kv_heads + g;
  // every key that counts here is visible to every voting row (pass 2 drops what lies behind the context rows)
  const bool unmasked = (PASS == 1 ? key0 + TILE : min(key0 + TILE, ctx_len)) - 1 <= first_obs;
  const int n_keys = key_end - key0;                       // keys that count (<= 0: nobody looks at this tile)
  float tok[NSUB];
#pragma unroll
  for (int kq = 0; kq < NSUB; ++kq) tok[kq] = 0.f;

  bf16x8 q[2 * KS];                                        // a column block: hi, lo
  auto q_of = [&](int cb) __attribute__((always_inline)) { return a.q_split + ((cg * a.n_cb + cb) * (2 * KS) * PC_WAVE + lane) * 8; };
  auto load_q = [&](const uint16_t* src) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < 2 * KS; ++i) q[i] = *(const bf16x8*)(src + i * PC_WAVE * 8);
  };
  // pass 2: the logsumexp of the rows of the column block that the arithmetic is at, and of the next one
  floatx16 lse, lse_next;
  auto load_lse = [&](floatx16& x, int cb) __attribute__((always_inline)) {
    const float* src = a.lse2 + cg * (32 * a.n_cb) + 32 * cb + 4 * hf;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float4 v = *(const float4*)(src + 8 * i);
      x[4 * i] = v.x; x[4 * i + 1] = v.y; x[4 * i + 2] = v.z; x[4 * i + 3] = v.w;
    }
  };
  if (wave < a.n_cb) load_q(q_of(wave));                   // in flight while the keys are staged
  if (key0 < (pre ? a.L : key_end)) {
    PcKeyStage<D, TILE, PASS == 1> keys;
    keys.begin(a, tid, key0, pre);
    keys.fetch(a, c, g, key0);
    keys.stage(a, c, g, key0, k_hi, k_lo);
  }
  __syncthreads();

  // The products of a wavefront, NSUB of them a column block, one after the other; the K operands go round a ring that
  // is read AHEAD k-steps before its use (behind a product's last ones the next product's)
  constexpr int RING = 4, AHEAD = 3;
  static_assert(KS % RING == 0, "k-steps go round the operand ring");
  bf16x8 ring[RING][2];                                    // hi, lo
  floatx16 s_buf[2];
  int k_at = n * KSTRIDE + 8 * hf;                         // opaque in the loops: the reads stay where they are written
  auto opaque_at = [&]() __attribute__((always_inline)) { asm volatile("" : "+v"(k_at)); };
  auto read_k = [&](int kq, int ks) __attribute__((always_inline)) {
    ring[ks % RING][0] = *(const bf16x8*)(k_hi + k_at + 32 * kq * KSTRIDE + 16 * ks);
    ring[ks % RING][1] = *(const bf16x8*)(k_lo + k_at + 32 * kq * KSTRIDE + 16 * ks);
  };
  constexpr int MAX_SL = KS / 4;                           // slices of pass 1 that take the maxima
  float m_run = -INFINITY, l_run = 0.f;                    // pass 1: of the column block that the arithmetic is at
  // What a mask starts from.  Pass 1: the last key that the voting row of the lane's column sees, counted as the lane's
  // registers are.  Pass 2: the first voting row of the column block (the same one for all lanes).
  auto limit_of = [&](int cb) __attribute__((always_inline)) {
    return PASS == 1 ? first_obs + pc_mod(min(32 * cb + n, a.n_cols - 1), a.w_obs, a.obs_div) - key0 - 4 * hf
                     : pc_mod(32 * cb, a.w_obs, a.obs_div);
  };
  // pass 2: the rows of a column block from voting row row0 on that see the lane's key of product kq, a bit each, moved to
  // where the lane's registers count from.  The rows of every head of the block are a run that ends at the head's last.
  // In the slices like everything else: a loop of its own, product after product, had cost more than the slices won.  That
  // loop -> now (both passes, us): 12 chunks of 2011 + 203 rows, 32 / 8 heads, 512 voting 603 -> 548, all 2214 3114 -> 2529; 1 of
  // 1000 + 64, 8 heads, 600 voting 40.2 -> 30.5; 16 of 1000 + 64, 24 / 8 heads of 64 values, 300 voting 144 -> 122.
  auto rows_that_see = [&](int row0, int kq) __attribute__((always_inline)) {
    const int first = min(max(key0 + 32 * kq + n - first_obs, 0), a.w_obs);
    auto below = [](int x) __attribute__((always_inline)) { return x <= 0 ? 0u : ~0u >> (32 - min(x, 32)); };
    uint32_t rows = 0;
    for (int head = -row0; head < 32; head += a.w_obs) rows |= below(head + a.w_obs) & ~below(head + first);
    return rows >> (4 * hf);
  };
  // A product's arithmetic in KS shares: s holds product kq of a column block (MASK: keys that a row does not see are
  // left out; pass 2 asks once a product which rows do).
  auto arith = [&](auto mask_tag, int share, floatx16& s, int kq, int limit, float& top, float& sum, uint32_t& seen) __attribute__((always_inline)) {
    constexpr bool MASK = decltype(mask_tag)::value;
    if (PASS == 1) {
      if (share < MAX_SL) {
        if (share == 0) {
          top = m_run;
          if (MASK) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
              if (32 * kq + 8 * (r / 4) + (r % 4) > limit) s[r] = -INFINITY;
          }
        }
#pragma unroll
        for (int i = 0; i < 16 / MAX_SL; ++i) top = fmaxf(top, s[share * (16 / MAX_SL) + i]);
        asm volatile("" : "+v"(top));
        if (share == MAX_SL - 1) {                         // (no key seen yet: any finite reference does)
          const float ref = top > -INFINITY ? top : 0.f;
          l_run *= __builtin_amdgcn_exp2f(m_run - ref);
          m_run = top; top = ref;
          asm volatile("" : "+v"(l_run));
        }
      } else {
        constexpr int SL = KS - MAX_SL;
        const int i = share - MAX_SL;
        if (i == 0) sum = 0.f;
#pragma unroll
        for (int r = 16 * i / SL; r < 16 * (i + 1) / SL; ++r) sum += __builtin_amdgcn_exp2f(s[r] - top);
        asm volatile("" : "+v"(sum));
        if (share == KS - 1) l_run += sum;
      }
    } else {
      if (share == 0) {
        sum = 0.f;
        if (MASK) seen = rows_that_see(limit, kq);
      }
#pragma unroll
      for (int r = share * (16 / KS); r < (share + 1) * (16 / KS); ++r) {
        const float p = __builtin_amdgcn_exp2f(s[r] - lse[r]);
        sum += MASK ? __uint_as_float(__float_as_uint(p) & (uint32_t)__builtin_amdgcn_sbfe((int)seen, 8 * (r / 4) + r % 4, 1)) : p;
      }
      asm volatile("" : "+v"(sum));
      if (share == KS - 1) tok[kq] += sum;
    }
  };
  // pass 1: a column block's (max, sum) over this block of keys; the lane halves hold disjoint keys of the same column
  auto leave = [&](int cb) __attribute__((always_inline)) {
    const float M = pc_xhalf_max(m_run);
    const float l = pc_xhalf_sum(l_run != 0.f ? l_run * __builtin_amdgcn_exp2f(m_run - M) : 0.f);
    if (hf == 0 && 32 * cb + n < a.n_cols)
      a.ml[(cg * a.n_kb + kblock) * a.n_cols + 32 * cb + n] = make_float2(M, l);
    m_run = -INFINITY; l_run = 0.f;
  };
  auto product = [&](const bf16x8& cols, const bf16x8& keys, const floatx16& c) __attribute__((always_inline)) {
    return PASS == 1 ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(keys, cols, c, 0, 0, 0)     // rows = keys, columns = voting rows
                     : __builtin_amdgcn_mfma_f32_32x32x16_bf16(cols, keys, c, 0, 0, 0);    // rows = voting rows, columns = keys
  };
  // Column block cb, and the last product's arithmetic of the block before it.  Behind its last use in the block an
  // operand makes room for the next block's: KS - 1 k-steps before that needs it.
  auto block = [&](auto mask_tag, auto products_tag, int cb) __attribute__((always_inline)) {
    constexpr bool MASK = decltype(mask_tag)::value;
    constexpr int PRODUCTS = decltype(products_tag)::value;
    int limit = MASK ? limit_of(max(cb - PC_SC_WAVES, 0)) : 0;
    const int next = min(cb + PC_SC_WAVES, a.n_cb - 1);
    const uint16_t* src = q_of(next);
    opaque_at();
    static_assert(PRODUCTS % 2 == 0, "products take turns in s_buf");
#pragma unroll
    for (int kq = 0; kq < PRODUCTS; ++kq) {
      floatx16& s = s_buf[kq % 2];
      float top = 0.f, sum = 0.f;
      uint32_t seen = 0;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8 kh = ring[ks % RING][0], kl = ring[ks % RING][1];
        if (ks == 0) {
          floatx16 zero;
#pragma unroll
          for (int r = 0; r < 16; ++r) zero[r] = 0.f;
          s = product(q[ks], kl, zero);
        } else {
          s = product(q[ks], kl, s);
        }
        if (PASS == 2 && kq == 0 && ks == 0) load_lse(lse_next, cb);
        const int to = ks + AHEAD;
        if (to < KS) read_k(kq, to); else read_k((kq + 1) % PRODUCTS, to - KS);
        s = product(q[KS + ks], kh, s);
        if (ks > 0) arith(mask_tag, ks, s_buf[1 - kq % 2], (kq + PRODUCTS - 1) % PRODUCTS, limit, top, sum, seen);
        s = product(q[ks], kh, s);
        if (ks == 0) {                                     // (the product before is through by then)
          __builtin_amdgcn_sched_barrier(0);
          arith(mask_tag, ks, s_buf[1 - kq % 2], (kq + PRODUCTS - 1) % PRODUCTS, limit, top, sum, seen);
        }
        if (kq == PRODUCTS - 1) {
          q[ks] = *(const bf16x8*)(src + ks * PC_WAVE * 8);
          q[KS + ks] = *(const bf16x8*)(src + (KS + ks) * PC_WAVE * 8);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      if (PASS == 2 && kq == 0) lse = lse_next;
      if (PASS == 1 && kq == 0) {
        if (cb >= PC_SC_WAVES) leave(cb - PC_SC_WAVES);
        m_run = -INFINITY; l_run = 0.f;
      }
      if (MASK && kq == 0) limit = limit_of(cb);
    }
  };
  auto blocks = [&](auto mask_tag, auto products_tag) __attribute__((always_inline)) {
    // (an address of the branch's own: operand reads merged in front of the branches were in registers for all of them)
    asm volatile("; operands of branch %1" : "+v"(k_at) : "n"(2 * decltype(products_tag)::value + decltype(mask_tag)::value));
#pragma unroll
    for (int ks = 0; ks < AHEAD; ++ks) read_k(0, ks);
    // nothing before the first block: exponents that add nothing (pass 1: a sum that is dropped)
#pragma unroll
    for (int r = 0; r < 16; ++r) { s_buf[1][r] = 0.f; lse[r] = INFINITY; }
    int cb = wave;
#pragma unroll 1
    for (; cb < a.n_cb; cb += PC_SC_WAVES) block(mask_tag, products_tag, cb);
    float top = 0.f, sum = 0.f;
    uint32_t seen = 0;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) arith(mask_tag, ks, s_buf[1], decltype(products_tag)::value - 1, limit_of(cb - PC_SC_WAVES), top, sum, seen);
    if (PASS == 1) leave(cb - PC_SC_WAVES);
  };
  // A tile with up to 64 keys that count (the last one of the context or of the sequence) takes two products a column
  // block instead of four, with the same bits.  Four always / two (both passes, us): 300 chunks of 24 + 8 rows, 64 heads on one
  // KV head, 8 voting 76.1 / 64.9; 200 of 100 + 33, 32 / 8 heads, 33 voting 167.7 / 157.2; 60 ragged of 700 + 60, 60 voting
  // 154.7 / 147.1; no such tile in 12 of 2011 + 203, 2214 voting 2623 / 2598.
  if (wave < a.n_cb && n_keys > 0) {
    // Columns in registers for several branches at once cost the third wavefront a SIMD at 64 values (prefill of 11 chunks of
    // 2470 + 179 rows, 8 heads, all query rows voting: 186.7 -> 189.9 us).  So the short tiles' branch stands first, and pass 2
    // loads a masked tile's columns anew, at 64 values a short one's too.  At 128 values LDS allows two wavefronts: there a
    // short tile keeps the columns that are on their way (first call above: 65.4 us, anew 67.8).
    if (NSUB > 2 && n_keys <= 64) {
      if (PASS == 2 && D == 64) load_q(q_of(wave));
      // (pass 1: such a tile ends the sequence, some row does not see all of it)
      if (PASS == 2 && unmasked) blocks(std::false_type{}, std::integral_constant<int, 2>{});
      else blocks(std::true_type{}, std::integral_constant<int, 2>{});
    } else if (unmasked) {
      blocks(std::false_type{}, std::integral_constant<int, NSUB>{});
    } else {
      if (PASS == 2) load_q(q_of(wave));
      blocks(std::true_type{}, std::integral_constant<int, NSUB>{});
    }
  } else if (PASS == 1) {
    for (int cb = wave; cb < a.n_cb; cb += PC_SC_WAVES) leave(cb);     // nobody looks at these keys
  }

  if (PASS == 2) {
#pragma unroll
    for (int kq = 0; kq < NSUB; ++kq) {
      const float x = tok[kq] + __shfl_xor(tok[kq], 32);
      if (hf == 0) tok_part[wave][32 * kq + n] = x;
    }
    __syncthreads();
    float blk = 0.f;
    if (tid < TILE && key0 + tid < a.w) {
      float x = 0.f;
#pragma unroll
      for (int wv = 0; wv < PC_SC_WAVES; ++wv) x += tok_part[wv][tid];
      x = key0 + tid < ctx_len ? x : 0.f;
      a.tok_score[cg * a.w + key0 + tid] = x;
      blk = x;
    }
    // block sum in a fixed order: lanes (xor tree), then the wavefronts in order
#pragma unroll
    for (int off = PC_WAVE / 2; off > 0; off >>= 1) blk += __shfl_xor(blk, off);
    __syncthreads();
    if (lane == 0) tok_part[0][wave] = blk;
    __syncthreads();
    if (tid == 0) {
      float tot = 0.f;
#pragma unroll
      for (int wv = 0; wv < PC_SC_WAVES; ++wv) tot += tok_part[0][wv];
      a.blk_sum[cg * gridDim.y + kblock] = tot;
    }
  }
}

// Row logsumexp (log2 units) of every voting row from the per-key-block (max, sum) of pass 1,
// combined in block order.  One thread per column, the blocks read once, in batches of 8
// independent loads.
__global__ __launch_bounds__(128) void scores_lse_kernel(const float2* __restrict__ ml,
                                                         float* __restrict__ lse2, int n_kb,
                                                         int n_cols, int n_pad) {
  const int col = blockIdx.y * 128 + threadIdx.x;
  if (col >= n_pad) return;
  if (col >= n_cols) {                                       // padding of the last column block: p = 0
    lse2[(long long)blockIdx.x * n_pad + col] = INFINITY;
    return;
  }
  const float2* src = ml + (long long)blockIdx.x * n_kb * n_cols + col;
  float M = -INFINITY, sum = 0.f;
  for (int kb0 = 0; kb0 < n_kb; kb0 += 8) {
    float2 v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = src[(long long)min(kb0 + i, n_kb - 1) * n_cols];
    float m_new = M;
#pragma unroll
    for (int i = 0; i < 8; ++i) m_new = fmaxf(m_new, v[i].x);
    if (sum > 0.f) sum *= exp2f(M - m_new);
    M = m_new;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      if (kb0 + i < n_kb && v[i].y > 0.f) sum += v[i].y * exp2f(v[i].x - M);
  }
  lse2[(long long)blockIdx.x * n_pad + col] = M + log2f(sum);
}

// chunk_score[c] = sum of tok_score[c, :, :] = sum of the chunk's pass-2 block sums (the standalone
// score call; inside the prefill call the attention launch that follows does it).
__global__ __launch_bounds__(256) void chunk_score_kernel(const float* __restrict__ blk_sum,
                                                          float* __restrict__ chunk_score,
                                                          int per_chunk) {
  __shared__ float red[256];
  pc_chunk_sum(blk_sum, chunk_score, per_chunk, blockIdx.x, red);
}

int pc_launch_chunk_sums(const PcChunkSum& sum, int n_chunks, hipStream_t st) {
  PcProfScope prof(PC_KERNEL_CHUNK_SCORE, st);
  hipLaunchKernelGGL(chunk_score_kernel, dim3(n_chunks), dim3(256), 0, st, sum.blk_sum, sum.chunk_score, sum.per_chunk);
  PC_LAUNCH_CHECK();
  return PC_OK;
}

template <int D, int PASS>
static void launch_scores_pass(int wpc, dim3 grid, dim3 block, hipStream_t st, const PcScoreArgs& a) {
  if (wpc == 0 && a.kb_keys == PC_SC_KB_MANY)
    hipLaunchKernelGGL((scores_many_kernel<D, PASS, PC_SC_KB_MANY>), grid, block, 0, st, a);
  else if (wpc == 0) hipLaunchKernelGGL((scores_many_kernel<D, PASS, PC_SC_KB_MANY / 2>), grid, block, 0, st, a);
  else if (wpc == 4) hipLaunchKernelGGL((scores_kernel<D, PASS, 4>), grid, block, 0, st, a);
  else if (wpc == 2) hipLaunchKernelGGL((scores_kernel<D, PASS, 2>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((scores_kernel<D, PASS, 1>), grid, block, 0, st, a);
}

// Keys per workgroup of scores_many_kernel: 128, or 64 where that is less than one workgroup per CU
#define PC_SC_MANY_WGS 256
static size_t key_blocks(const pc_shape* s, int kb) {
  const size_t L = (size_t)s->chunk_len + s->query_len;
  return (size_t)s->n_chunks * s->n_kv_heads * ((L + kb - 1) / kb);
}
static int many_kb_keys(const pc_shape* s) {
  return key_blocks(s, PC_SC_KB_MANY) < PC_SC_MANY_WGS ? PC_SC_KB_MANY / 2 : PC_SC_KB_MANY;
}
// Key blocks of all chunks and KV heads that the workspace has room for.  A workspace serves every call
// with no more chunks or rows than the one it was sized for (a short last batch is an example), so
// this must not fall where the larger block takes over: blocks of half the keys, of which there are
// never as many as 2 x PC_SC_MANY_WGS (PC_SC_SMALL_WGS), have room behind that point too.
static size_t key_blocks_room(const pc_shape* s, size_t n_cb) {
  const bool many = n_cb > PC_SC_WAVES;
  const size_t large = key_blocks(s, many ? PC_SC_KB_MANY : PC_SC_KB), small = key_blocks(s, many ? PC_SC_KB_MANY / 2 : PC_SC_KB_SMALL);
  const size_t most = 2 * (many ? PC_SC_MANY_WGS : PC_SC_SMALL_WGS), small_max = small < most ? small : most;
  return large > small_max ? large : small_max;
}

// Workspace of the score passes: per-block (max, sum) of pass 1, the combined row logsumexp, the
// block sums of pass 2 and the split query columns.
struct PcScoreWs { size_t ml, lse2, blk_sum, q_split, total; };
static PcScoreWs scores_ws_layout(const pc_shape* s) {
  const size_t n_cols = (size_t)(s->n_q_heads / s->n_kv_heads) * s->obs_window;
  const size_t n_cb = (n_cols + 31) / 32, cg = (size_t)s->n_chunks * s->n_kv_heads, blocks = key_blocks_room(s, n_cb);
  PcScoreWs w;
  size_t off = 0;
  w.ml = off;      off = pc_align_up(off + blocks * n_cols * sizeof(float2), 256);
  w.lse2 = off;    off = pc_align_up(off + cg * n_cb * 32 * sizeof(float), 256);
  w.blk_sum = off; off = pc_align_up(off + blocks * sizeof(float), 256);
  w.q_split = off; off += cg * n_cb * (n_cols < 32 ? n_cols : 32) * (size_t)s->head_dim * 2 * 2;
  w.total = off;
  return w;
}

size_t pc_scores_ws_bytes(const pc_shape* s) { return scores_ws_layout(s).total; }

PcScoreQueries pc_scores_queries(const pc_shape* s, const void* q, const int32_t* chunk_lens, void* ws) {
  PcScoreQueries a = {};
  a.q = (const uint16_t*)q; a.chunk_lens = chunk_lens;
  a.q_split = (uint16_t*)((char*)ws + scores_ws_layout(s).q_split);
  a.n_chunks = s->n_chunks; a.L = s->chunk_len + s->query_len; a.w = s->chunk_len; a.w_obs = s->obs_window;
  a.n_kv_heads = s->n_kv_heads; a.G = s->n_q_heads / s->n_kv_heads;
  a.n_cols = a.G * s->obs_window; a.n_cb = (a.n_cols + 31) / 32;
  a.cb_div = pc_div_by(a.n_cb); a.heads_div = pc_div_by(a.n_kv_heads); a.obs_div = pc_div_by(a.w_obs);
  const float scale = s->softmax_scale > 0.f ? s->softmax_scale : 1.0f / sqrtf((float)s->head_dim);
  a.scale_log2 = scale * PC_SC_LOG2E;
  return a;
}

int pc_launch_scores(const pc_shape* s, const void* k, const int32_t* chunk_lens, const float2* table,
                     void* ws, float* tok_score, float* chunk_score, const PcPrepassOut* pre,
                     PcChunkSum* later, hipStream_t st) {
  const PcScoreWs w = scores_ws_layout(s);
  PcScoreArgs a = {};
  a.q_split = (const uint16_t*)((char*)ws + w.q_split); a.k = (const uint16_t*)k; a.table = table; a.chunk_lens = chunk_lens;
  a.ml = (float2*)((char*)ws + w.ml); a.lse2 = (float*)((char*)ws + w.lse2);
  a.blk_sum = (float*)((char*)ws + w.blk_sum);
  a.tok_score = tok_score;
  a.L = s->chunk_len + s->query_len; a.w = s->chunk_len; a.w_obs = s->obs_window;
  a.n_q_heads = s->n_q_heads; a.n_kv_heads = s->n_kv_heads;
  a.heads_div = pc_div_by(a.n_kv_heads); a.obs_div = pc_div_by(a.w_obs);
  a.n_cols = (s->n_q_heads / s->n_kv_heads) * s->obs_window;
  a.n_cb = (a.n_cols + 31) / 32;
  const bool many = a.n_cb > PC_SC_WAVES;
  const int wpc = many ? 0 : (a.n_cb == 1 ? 4 : (a.n_cb == 2 ? 2 : 1));
  // keys per workgroup: double while at least 512 workgroups (one full round of two per CU)
  // remain: fewer, longer workgroups spread their start-up over more keys (measured: 4 and 8
  // chunks of 8192 rows 10 % faster than with twice as many workgroups of half the keys); half where 256
  // leave CUs idle (and pass 2 still combines the blocks itself).  Both passes, 256 / 128 keys (us): 1 x 1174 rows,
  // 8 KV heads (40 workgroups of 256) 26.8 / 20.7, 2 x 2800, 4 (88) 37.8 / 28.5, 20 x 500, 8 (320) 55.0 / 52.1, 12 x 900 of
  // 64 values, 8 (384) 37.6 / 35.7, 3 x 860, 32 (384) 50.7 / 51.5, 1 x 4096, 32 (512) 55.7 / 67.5.
  a.kb_keys = many ? many_kb_keys(s) : PC_SC_KB;
  if (!many && key_blocks(s, PC_SC_KB) < PC_SC_SMALL_WGS && a.L <= PC_SC_LSE_BLOCKS * PC_SC_KB_SMALL) a.kb_keys = PC_SC_KB_SMALL;
  const int kb_cap = wpc == 4 ? PC_SC_KB_MAX / 2 : PC_SC_KB_MAX;
  while (!many && a.kb_keys >= PC_SC_KB && a.kb_keys < kb_cap && key_blocks(s, 2 * a.kb_keys) >= 512) a.kb_keys *= 2;
  a.n_kb = (a.L + a.kb_keys - 1) / a.kb_keys;
  // pass 2 looks at context keys only.  A key's sum has one owner where four wavefronts share a column block: its blocks
  // have room for twice as many keys (36 x 3584 keys of 32 KV heads, 512 / 1024 keys: 300 / 277 us).  Blocks start at
  // multiples of pass 1's and the angles are read anew there, so blocks of 512 and of 1024 keys give the same bits (blocks
  // of equal size move the places where the angles' chains begin, and of two nearly equal scores the other is then kept).
  // Smaller blocks, which calls of fewer or shorter chunks take in both passes, begin their chains elsewhere and cut pass 1's
  // sums elsewhere: there the last bits differ.
  int kb2 = a.kb_keys;
  if (wpc == 4 && kb2 == kb_cap && key_blocks(s, 2 * kb2) >= 512) kb2 *= 2;
  const int n_kb2 = (a.w + kb2 - 1) / kb2;
  if (a.n_kb > 65535 || s->n_kv_heads > 65535) return PC_ERR_SHAPE;   // grid limits
  // heads fastest: neighbouring workgroups read neighbouring rows of a token, and an XCD (workgroups go round the
  // eight) gets every chunk, whatever the chunks' lengths.  Chunks fastest -> heads fastest (us): pass 1 of
  // 36 x 4096 rows, 32 KV heads 1292 -> 1200; pass 2 of 12 ragged chunks of 2011 rows, 203 voting 120 -> 107; 8 heads of
  // chunks of one length: 64 x 8704 1165 -> 1184 and 474 -> 478, 16 x 8192 262 -> 263 and 135 -> 139.
  const long long cg = (long long)s->n_chunks * s->n_kv_heads;
  const unsigned gx = (unsigned)(cg <= PC_GRID_X ? cg : s->n_chunks), gz = (unsigned)(cg <= PC_GRID_X ? 1 : s->n_kv_heads);
  const dim3 grid(gx, a.n_kb, gz), grid2(gx, n_kb2, gz), block(PC_SC_THREADS);
  if (pre) {
    a.v = (const uint16_t*)pre->v; a.k_rope = (uint16_t*)pre->k_rope; a.k_img = (uint16_t*)pre->k_img;
    a.v_img = (uint16_t*)pre->v_img; a.Lp = pre->Lp;
  }
  {
    PcProfScope prof(pre ? PC_KERNEL_PREPASS_SCORES : PC_KERNEL_SCORES_P1, st);
    if (s->head_dim == 128) launch_scores_pass<128, 1>(wpc, grid, block, st, a);
    else launch_scores_pass<64, 1>(wpc, grid, block, st, a);
  }
  PC_LAUNCH_CHECK();
  if (many || a.n_kb > PC_SC_LSE_BLOCKS) {
    PcProfScope prof(PC_KERNEL_SCORES_LSE, st);
    hipLaunchKernelGGL(scores_lse_kernel, dim3(s->n_chunks * s->n_kv_heads, (32 * a.n_cb + 127) / 128),
                       dim3(128), 0, st, a.ml, a.lse2, a.n_kb, a.n_cols, 32 * a.n_cb);
  }
  a.kb_keys = kb2;
  {
    PcProfScope prof(PC_KERNEL_SCORES_P2, st);
    if (s->head_dim == 128) launch_scores_pass<128, 2>(wpc, grid2, block, st, a);
    else launch_scores_pass<64, 2>(wpc, grid2, block, st, a);
  }
  PC_LAUNCH_CHECK();
  if (later) {
    *later = PcChunkSum{a.blk_sum, chunk_score, s->n_kv_heads * n_kb2};
  } else if (chunk_score) {
    return pc_launch_chunk_sums(PcChunkSum{a.blk_sum, chunk_score, s->n_kv_heads * n_kb2}, s->n_chunks, st);
  }
  return PC_OK;
}
