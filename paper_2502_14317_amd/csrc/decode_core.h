// The split-KV attention for few query rows over bf16 segments, as a workgroup function: launched by
// itself (decode_attn.hip) and next to the 8-bit segments' workgroups (decode_attn_fp8.hip).
#pragma once
#include "pc_common.h"
#include <math.h>

#define PC_DEC_WAVES 4
#define PC_DEC_ITER_KEYS 32
#define PC_DEC_LOG2E 1.4426950408889634f

#define PC_WAVE_LDS_SYNC()                                   \
  do {                                                       \
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");   \
    __builtin_amdgcn_wave_barrier();                         \
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");   \
  } while (0)

// The query rows of the few-row kernels: bf16 [B, n_q, H_q, D], rotated by the kernel at positions
// pos0 + t (fp64 angles, rounded to bf16 once); pos0 < 0: they arrive rotated.
struct PcDecodeQuery {
  const uint16_t* q;
  int pos0, n_q, n_q_heads;
  PcRope rope;
};

// The columns (query t, head) of KV head g, rotated, into LDS: column n = t * G + head in group.  In two
// steps, so that the first keys can be asked for in between: `begin` asks for the query values (they are
// the older loads, so waiting for them leaves the keys in flight), `finish` rotates and writes.
template <int D>
struct PcColumnRotation {
  static constexpr int HALF = D / 2;
  int i, n0;                                                // the thread's rotation pair, its first column
  uint32_t a, b;
  __device__ __forceinline__ const uint16_t* row(const PcDecodeQuery& x, int seq, int g, int G, int n) const {
    return x.q + (((long long)seq * x.n_q + n / G) * x.n_q_heads + g * G + n % G) * D;
  }
  __device__ __forceinline__ void begin(const PcDecodeQuery& x, int seq, int g, int G, int n_cols) {
    i = threadIdx.x % HALF; n0 = threadIdx.x / HALF;
    const uint16_t* r = row(x, seq, g, G, min(n0, n_cols - 1));
    a = r[i]; b = r[i + HALF];
  }
  __device__ __forceinline__ void finish(const PcDecodeQuery& x, int seq, int g, int G, int n_cols, uint16_t (*cols)[D]) {
    const double theta = pc_rope_theta(x.rope, i);
    int at = -1;
    double sn = 0.0, cs = 1.0;
    for (int n = n0; n < n_cols; n += blockDim.x / HALF) {
      if (n != n0) { const uint16_t* r = row(x, seq, g, G, n); a = r[i]; b = r[i + HALF]; }
      uint32_t ra = a, rb = b;                              // pos0 < 0: as they are
      if (x.pos0 >= 0) {
        if (n / G != at) { at = n / G; pc_sincos((double)(x.pos0 + at) * theta, sn, cs); }
        const double x1 = bf16_bits_to_f32((uint16_t)a), x2 = bf16_bits_to_f32((uint16_t)b);
        ra = f32_to_bf16_bits((float)(x1 * cs - x2 * sn));
        rb = f32_to_bf16_bits((float)(x2 * cs + x1 * sn));
      }
      cols[n][i] = (uint16_t)ra;
      cols[n][i + HALF] = (uint16_t)rb;
    }
  }
};
// A decoding step's new token (one query row): its key, rotated at `pos` (pos < 0: it arrives rotated), and
// value are stored behind the rows of the last segment, unless that is full; the merge takes the token as
// one more key and counts the row.  In two steps like the columns.
struct PcDecodeAppend {
  const uint16_t* k_new;   // [B, H_kv, D] or nullptr: no step
  const uint16_t* v_new;
  int pos;
  uint16_t* q_rot;         // [B, H_q, D] out: the rotated query for the merge; nullptr: the merge has it already
  int32_t* self_row;       // [B, H_kv] out: the row written, -1 if there was no room
};
template <int D>
struct PcRowAppend {
  uint32_t a, b, v;
  __device__ __forceinline__ void begin(const PcDecodeAppend& x, int bg) {
    const int i = threadIdx.x % (D / 2);
    const uint16_t* k = x.k_new + (long long)bg * D;
    a = k[i]; b = k[i + D / 2];
    v = x.v_new[(long long)bg * D + threadIdx.x % D];
  }
  __device__ __forceinline__ void finish(const PcDecodeAppend& x, const PcRope& rope, int bg, int len, int cap,
                                         uint16_t* k_seg, uint16_t* v_seg) {
    const int tid = threadIdx.x;
    if (tid == 0) x.self_row[bg] = len < cap ? len : -1;
    if (len >= cap) return;
    const long long at = (long long)len * D;
    if (tid < D / 2) {
      uint32_t ra = a, rb = b;
      if (x.pos >= 0) {
        double sn, cs;
        pc_sincos((double)x.pos * pc_rope_theta(rope, tid), sn, cs);
        const double x1 = bf16_bits_to_f32((uint16_t)a), x2 = bf16_bits_to_f32((uint16_t)b);
        ra = f32_to_bf16_bits((float)(x1 * cs - x2 * sn));
        rb = f32_to_bf16_bits((float)(x2 * cs + x1 * sn));
      }
      k_seg[at + tid] = (uint16_t)ra;
      k_seg[at + tid + D / 2] = (uint16_t)rb;
    }
    if (tid < D) v_seg[at + tid] = (uint16_t)v;
  }
};
// Barrier over what the wavefronts wrote to LDS; loads from memory stay in flight
#define PC_LDS_BARRIER()                                     \
  do {                                                       \
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");  \
    __builtin_amdgcn_s_barrier();                            \
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");  \
  } while (0)

struct PcDecodeArgs {
  PcDecodeQuery query;
  PcDecodeAppend app;
  const uint16_t* kc;     // [B, S, H_kv, k_t, D]
  const uint16_t* vc;
  const int32_t* seg_len; // [B, S] ([B, S, H_kv] if seg_len_per_head) or nullptr
  int seg_len_per_head;
  float* part_o;          // [B, P, n_q, H_q, D]
  float* part_lse;        // [B, P, n_q, H_q]
  int n_q, n_seg, k_t, n_q_heads, n_kv_heads, n_parts;
  int parts_grid;         // workgroups (partials) per (sequence, KV head) in this launch
  int part0;              // index of this launch's first partial among the n_parts
  float scale_log2;       // softmax scale * log2(e)
};

// One workgroup (PC_DEC_WAVES wavefronts) of the split-KV attention, number `bid` of batch * H_kv *
// parts_grid.
template <int D, int NQ>
__device__ __forceinline__ void pc_decode_workgroup(const PcDecodeArgs& a, int bid) {
  constexpr int KSTEPS = D / 32;            // MFMA k-steps over the head dimension
  constexpr int LPR = D / 8;                // lanes per V row (16-byte pieces)
  constexpr int RPI = PC_WAVE / LPR;        // V rows per load instruction
  constexpr int VLOADS = PC_DEC_ITER_KEYS / RPI;
  constexpr int KBLK = PC_DEC_ITER_KEYS / 16;

  __shared__ float p_lds[PC_DEC_WAVES][PC_DEC_ITER_KEYS][NQ];
  __shared__ float alpha_lds[PC_DEC_WAVES][NQ];
  __shared__ float red_o[PC_DEC_WAVES][NQ][D];
  __shared__ float red_m[PC_DEC_WAVES][NQ], red_l[PC_DEC_WAVES][NQ];
  __shared__ __attribute__((aligned(16))) uint16_t q_lds[NQ][D];

  const int G = a.n_q_heads / a.n_kv_heads;
  const int n_cols = a.n_q * G;             // valid query columns (<= NQ)
  const int lane = threadIdx.x % PC_WAVE, wave = threadIdx.x / PC_WAVE;
  const int kk = lane / 16, c16 = lane % 16;

  const int part = bid % a.parts_grid; bid /= a.parts_grid;
  const int g = bid % a.n_kv_heads;    bid /= a.n_kv_heads;
  const int b = bid;

  // A wavefront streams its run of 32-key blocks, through segment boundaries; the running
  // softmax carries over (same query columns, same KV head), so a workgroup leaves one partial.
  // A cursor names the next block: where it is, plus the segment's base pointers.
  struct Cursor { PcBlockCursor at; const uint16_t* k; const uint16_t* v; int bytes; };
  PcSegLens lens;
  lens.seg_len = a.seg_len; lens.per_head = a.seg_len_per_head; lens.n_seg = a.n_seg;
  lens.n_kv_heads = a.n_kv_heads; lens.k_t = a.k_t; lens.b = b; lens.g = g;
  auto place = [&](const PcBlockCursor& at) {
    Cursor c; c.at = at; c.k = a.kc; c.v = a.vc; c.bytes = 0;       // behind the run's end: nothing is read
    if (at.left > 0) {
      const long long first = ((((long long)b * a.n_seg + at.s) * a.n_kv_heads + g) * a.k_t + 32LL * at.blk) * D;
      c.k = a.kc + first; c.v = a.vc + first;
      c.bytes = min(32, at.len - 32 * at.blk) * (2 * D);
    }
    return c;
  };
  auto next = [&](const Cursor& c) { return place(pc_blocks_next(lens, c.at)); };

  PcColumnRotation<D> rot;
  rot.begin(a.query, b, g, G, n_cols);
  // the group's last workgroup also stores the new token: nobody reads its row in this launch (the
  // lengths still exclude it)
  const bool append = a.app.k_new != nullptr && part == a.parts_grid - 1;
  PcRowAppend<D> row;
  if (append) row.begin(a.app, b * a.n_kv_heads + g);
  bf16x8 bq[KSTEPS];                        // B operand: column c16 = (t, head-in-group); lane holds d = 32*ks + 8*kk .. +7

  float m_run = -INFINITY, l_run = 0.f;     // of column c16 (this lane's share of the sum)
  float o_acc[NQ][8];
#pragma unroll
  for (int n = 0; n < NQ; ++n)
#pragma unroll
    for (int e = 0; e < 8; ++e) o_acc[n][e] = 0.f;

  const int v_row = lane / LPR, v_piece = lane % LPR;

  // A block's rows through buffer descriptors that end behind its last valid row: the rows after it arrive
  // as zeros, and behind the run's end nothing is read.  So the loads are unconditional, and the waits in
  // front of a block's arithmetic count the next block's loads as what they are, in flight (with loads
  // under a condition the compiler must assume that they were not issued and waits for all).
  u32x4 kbuf[2][KBLK][KSTEPS], vbuf[2][VLOADS];
  const int k_off = 2 * (c16 * D + 8 * kk), v_off = 2 * (v_row * D + 8 * v_piece);
  auto issue_loads = [&](int buf, const Cursor& c) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t kr = __builtin_amdgcn_make_buffer_rsrc((void*)c.k, 0, c.bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc((void*)c.v, 0, c.bytes, 0x00020000);
#pragma unroll
    for (int bi = 0; bi < KBLK; ++bi)
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks)
        kbuf[buf][bi][ks] = __builtin_amdgcn_raw_buffer_load_b128(kr, k_off, 2 * (16 * bi * D + 32 * ks), PC_BUF_NT);
#pragma unroll
    for (int i = 0; i < VLOADS; ++i)
      vbuf[buf][i] = __builtin_amdgcn_raw_buffer_load_b128(vr, v_off, 2 * RPI * i * D, PC_BUF_NT);
    __builtin_amdgcn_sched_barrier(0);                       // not behind the arithmetic that follows
  };

  auto consume = [&](int buf, const Cursor& cur) {
    const int key0 = 32 * cur.at.blk, w_end = cur.at.len;
    // S^T block: keys x columns
    floatx4 acc[KBLK];
#pragma unroll
    for (int bi = 0; bi < KBLK; ++bi) {
      acc[bi] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks)
        acc[bi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(bf16x8*)&kbuf[buf][bi][ks], bq[ks],
                                                          acc[bi], 0, 0, 0);
    }
    float sv[KBLK][4];
    float bmax = -INFINITY;
#pragma unroll
    for (int bi = 0; bi < KBLK; ++bi)
#pragma unroll
      for (int j = 0; j < 4; ++j) sv[bi][j] = acc[bi][j] * a.scale_log2;
    if (key0 + 32 > w_end) {                         // a segment's last block
#pragma unroll
      for (int bi = 0; bi < KBLK; ++bi)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (key0 + 16 * bi + 4 * kk + j >= w_end) sv[bi][j] = -INFINITY;
    }
#pragma unroll
    for (int bi = 0; bi < KBLK; ++bi)
#pragma unroll
      for (int j = 0; j < 4; ++j) bmax = fmaxf(bmax, sv[bi][j]);
    bmax = pc_rows_max(bmax);
    const float m_new = fmaxf(m_run, bmax);          // finite: every block holds a valid key
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);   // arguments <= 0: the bare instruction
    m_run = m_new;
    float psum = 0.f;
#pragma unroll
    for (int bi = 0; bi < KBLK; ++bi)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float p = __builtin_amdgcn_exp2f(sv[bi][j] - m_new);
        psum += p;
        if (c16 < NQ) p_lds[wave][16 * bi + 4 * kk + j][c16] = p;
      }
    l_run = l_run * alpha + psum;
    const bool moved = __any(alpha != 1.0f);         // some column's maximum grew (rare after the first keys)
    if (moved && kk == 0 && c16 < NQ) alpha_lds[wave][c16] = alpha;
    PC_WAVE_LDS_SYNC();
    // rescale (only when a maximum moved), then o[n][:] += p[key][n] * v[key][:]
    if (moved) {
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        const float al = alpha_lds[wave][n];
#pragma unroll
        for (int e = 0; e < 8; ++e) o_acc[n][e] *= al;
      }
    }
#pragma unroll
    for (int i = 0; i < VLOADS; ++i) {
      const int key_local = RPI * i + v_row;
      float vf[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        vf[2 * e] = bf16_lo_to_f32(vbuf[buf][i][e]); vf[2 * e + 1] = bf16_hi_to_f32(vbuf[buf][i][e]);
      }
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        const float p = p_lds[wave][key_local][n];    // 0 for masked keys
#pragma unroll
        for (int e = 0; e < 8; ++e) o_acc[n][e] = fmaf(p, vf[e], o_acc[n][e]);
      }
    }
    PC_WAVE_LDS_SYNC();
  };

  Cursor cur = place(pc_blocks_begin(lens, part, a.parts_grid, __builtin_amdgcn_readfirstlane(wave), lane));
  issue_loads(0, cur);

  rot.finish(a.query, b, g, G, n_cols, q_lds);
  PC_LDS_BARRIER();
  if (append) {
    const long long seg0 = (((long long)b * a.n_seg + a.n_seg - 1) * a.n_kv_heads + g) * a.k_t * D;
    row.finish(a.app, a.query.rope, b * a.n_kv_heads + g, lens.len(a.n_seg - 1), a.k_t, const_cast<uint16_t*>(a.kc) + seg0,
               const_cast<uint16_t*>(a.vc) + seg0);
    if (a.app.q_rot)
      for (int x = threadIdx.x; x < n_cols * D; x += blockDim.x)     // one query row: heads g G .. are adjacent
        a.app.q_rot[((long long)b * a.n_q_heads + g * G) * D + x] = q_lds[x / D][x % D];
  }
#pragma unroll
  for (int ks = 0; ks < KSTEPS; ++ks) {
    u32x4 raw = *(const u32x4*)(q_lds[min(c16, n_cols - 1)] + 32 * ks + 8 * kk);
    if (c16 >= n_cols) raw = u32x4{0, 0, 0, 0};
    bq[ks] = *(bf16x8*)&raw;
  }

  while (cur.at.left > 0) {
    Cursor nx = next(cur);
    issue_loads(1, nx);
    consume(0, cur);
    if (nx.at.left == 0) break;
    cur = next(nx);
    issue_loads(0, cur);
    consume(1, nx);
  }

  // ---- wavefront totals: sum the per-lane shares
  l_run = pc_rows_sum(l_run);
#pragma unroll
  for (int n = 0; n < NQ; ++n)
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float x = o_acc[n][e];
#pragma unroll
      for (int off = LPR; off < PC_WAVE; off <<= 1) x += __shfl_xor(x, off);
      o_acc[n][e] = x;
    }
  if (kk == 0 && c16 < NQ) { red_m[wave][c16] = m_run; red_l[wave][c16] = l_run; }
  if (v_row == 0) {
#pragma unroll
    for (int n = 0; n < NQ; ++n)
#pragma unroll
      for (int e = 0; e < 8; ++e) red_o[wave][n][8 * v_piece + e] = o_acc[n][e];
  }
  __syncthreads();

  // ---- merge the 4 wavefronts, write one partial per workgroup
  const int part_out = a.part0 + part;
  for (int idx = threadIdx.x; idx < n_cols * D; idx += blockDim.x) {
    const int n = idx / D, d = idx % D;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < PC_DEC_WAVES; ++w) M = fmaxf(M, red_m[w][n]);
    float num = 0.f, den = 0.f;
    if (M > -INFINITY) {
#pragma unroll
      for (int w = 0; w < PC_DEC_WAVES; ++w) {
        const float sc = exp2f(red_m[w][n] - M);
        num += sc * red_o[w][n][d];
        den += sc * red_l[w][n];
      }
    }
    const int t = n / G, hg = n % G;
    const long long row = (((long long)b * a.n_parts + part_out) * a.n_q + t) * a.n_q_heads + g * G + hg;
    a.part_o[row * D + d] = (den > 0.f) ? num / den : 0.f;
    if (d == 0) a.part_lse[row] = (den > 0.f) ? (M + log2f(den)) * 0.6931471805599453f : -INFINITY;
  }
}

static inline PcDecodeQuery pc_decode_query(const void* q, int pos0, float base, int n_q, int n_q_heads, int head_dim) {
  PcDecodeQuery x;
  x.q = (const uint16_t*)q; x.pos0 = pos0; x.n_q = n_q; x.n_q_heads = n_q_heads;
  x.rope = pc_rope_factors(base > 1.0f ? base : 2.0f, head_dim);        // (not looked at where nothing is rotated)
  return x;
}
static inline PcDecodeArgs pc_decode_args(const PcDecodeQuery& query, const void* kc, const void* vc,
                                          const int32_t* seg_len, int seg_len_per_head, int batch, int n_seg,
                                          int k_t, int n_kv_heads, float scale, float* part_o, float* part_lse,
                                          int n_parts, int part0, const PcDecodeAppend& app) {
  PcDecodeArgs a;
  a.query = query; a.part0 = part0; a.app = app;
  a.kc = (const uint16_t*)kc; a.vc = (const uint16_t*)vc;
  a.seg_len = seg_len; a.seg_len_per_head = seg_len_per_head; a.part_o = part_o; a.part_lse = part_lse;
  a.n_q = query.n_q; a.n_seg = n_seg; a.k_t = k_t; a.n_q_heads = query.n_q_heads; a.n_kv_heads = n_kv_heads;
  a.parts_grid = pc_decode_split(k_t, n_seg, (long long)batch * n_kv_heads).n_parts;
  a.n_parts = n_parts;
  a.scale_log2 = scale * PC_DEC_LOG2E;
  return a;
}
