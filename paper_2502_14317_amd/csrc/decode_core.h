// The split-KV attention for few query rows over bf16 segments, as a workgroup function: launched by
// itself (decode_attn.hip) and next to the 8-bit segments' workgroups (decode_attn_fp8.hip).
#pragma once
#include "pc_common.h"
#include <math.h>

#define PC_DEC_WAVES 4
#define PC_DEC_ITER_KEYS 32
#define PC_DEC_LOG2E 1.4426950408889634f

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
    if (x.n_q == 1) return x.q + ((long long)seq * x.n_q_heads + g * G + n) * D;
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
  int group;              // H_q / H_kv
  int parts_grid;         // workgroups (partials) per (sequence, KV head) in this launch
  PcDiv parts_div, heads_div;   // by parts_grid, by n_kv_heads
  int part0;              // index of this launch's first partial among the n_parts
  float scale_log2;       // softmax scale * log2(e)
};

// LDS of a split-KV workgroup (the 16-bit and the 8-bit function of one launch use the same)
template <int D>
struct PcDecodeLds {
  float o[PC_DEC_WAVES][16][D];
  float m[PC_DEC_WAVES][16], l[PC_DEC_WAVES][16];
  __attribute__((aligned(16))) uint16_t q[16][D];
};
// The 4 wavefronts' (o, max in log2 units, sum) in LDS -> the workgroup's partial
template <int D>
__device__ __forceinline__ void pc_write_partial(const PcDecodeLds<D>& sm, int G, int n_cols, int n_q, int n_q_heads,
                                                 long long part_row, int g, float* part_o, float* part_lse) {
  __syncthreads();
  for (int idx = threadIdx.x; idx < n_cols * (D / 4); idx += PC_DEC_WAVES * PC_WAVE) {
    const int n = idx / (D / 4), d4 = idx % (D / 4) * 4;
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < PC_DEC_WAVES; ++w) M = fmaxf(M, sm.m[w][n]);
    floatx4 num = {0.f, 0.f, 0.f, 0.f};
    float den = 0.f;
    if (M > -INFINITY) {
#pragma unroll
      for (int w = 0; w < PC_DEC_WAVES; ++w) {
        const float sc = exp2f(sm.m[w][n] - M);
        const floatx4 x = *(const floatx4*)&sm.o[w][n][d4];
#pragma unroll
        for (int e = 0; e < 4; ++e) num[e] += sc * x[e];
        den += sc * sm.l[w][n];
      }
    }
    const long long row = (part_row * n_q + n / G) * n_q_heads + g * G + n % G;
    floatx4 y;
#pragma unroll
    for (int e = 0; e < 4; ++e) y[e] = den > 0.f ? num[e] / den : 0.f;
    *(floatx4*)(part_o + row * D + d4) = y;
    if (d4 == 0) part_lse[row] = (den > 0.f) ? (M + log2f(den)) * 0.6931471805599453f : -INFINITY;
  }
}
// A block's logits (lane: column lane % 16, keys 16 bi + 4 (lane / 16) + j) -> probabilities relative to the
// running maximum of the column, which moves (alpha: what everything before is worth now); keys behind
// the segment's end are masked in its last block.
__device__ __forceinline__ void pc_decode_softmax(const floatx4 (&acc)[2], float scale, int keys, int kk, float& m_run,
                                                  float& l_run, float& alpha, float (&pr)[2][4]) {
  float top = -INFINITY;
#pragma unroll
  for (int bi = 0; bi < 2; ++bi)
#pragma unroll
    for (int j = 0; j < 4; ++j) pr[bi][j] = acc[bi][j] * scale;
  if (keys < 32) {
#pragma unroll
    for (int bi = 0; bi < 2; ++bi)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (16 * bi + 4 * kk + j >= keys) pr[bi][j] = -INFINITY;
  }
#pragma unroll
  for (int bi = 0; bi < 2; ++bi)
#pragma unroll
    for (int j = 0; j < 4; ++j) top = fmaxf(top, pr[bi][j]);
  const float m_new = fmaxf(m_run, pc_rows_max(top));          // finite: every block holds a valid key
  alpha = __builtin_amdgcn_exp2f(m_run - m_new);               // arguments <= 0: the bare instruction
  m_run = m_new;
  float sum = 0.f;
#pragma unroll
  for (int bi = 0; bi < 2; ++bi)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      pr[bi][j] = __builtin_amdgcn_exp2f(pr[bi][j] - m_new);
      sum += pr[bi][j];
    }
  l_run = l_run * alpha + sum;
}

// One workgroup (PC_DEC_WAVES wavefronts) of the split-KV attention, number `bid` of batch * H_kv *
// parts_grid.  Both products on the 16x16x32 MFMA, S^T = K Q^T and O^T += V^T P^T, with the query columns on
// the N side, so that a lane owns one column throughout.  V arrives row-major, D / 16 values of a key a lane, 16
// lanes a row, four whole rows an instruction: eight keys of a lane, transposed by byte permutes, are D / 16 operands,
// operand e of the values D / 16 m + e.  A workgroup of few blocks spends a sixth of its time issuing its first loads, so
// there are as few as the bytes allow (16 of V in 8-byte pieces, two half rows each, now 8), and the segments' lengths,
// which the first key's place needs, are asked for in front of the query: one sequence of 8 x 2048 keys and a tail of
// 520, 8 KV heads, 15.0 -> 14.2 us; 16 sequences are bound by memory, 603 and 602.  A third and a fourth block in
// flight 16.5 and 17.0, K in contiguous KiB an instruction 13.6 but 637 for the 16.
// The lane's keys are those whose probabilities it holds, so P goes from the logit registers into the
// operand, as two bf16 halves (hi + lo), two MFMAs a block of V: 2^-17 relative where an fp32 operand had 2^-24.  The
// sum of the row takes P in fp32.  Outputs are rounded to bf16 (2^-9), so theirs is the error that shows: 3.3e-3 to
// 4.0e-3 of their norm from 64 bits over 14 sizes (1 to 16 sequences of 1 to 32 segments of 725 to 2048 keys, two inputs
// each), with fp32 operands the same to 1e-6, above and below.
// P V on the vector ALUs (32 multiply-adds per loaded piece and column, P through LDS, a kernel each for 4, 8
// and 16 columns) took 21.3 us a step of 8 x 2048 keys, 4 columns, this 20.1.
template <int D>
__device__ __forceinline__ void pc_decode_workgroup(const PcDecodeArgs& a, int bid, PcDecodeLds<D>& sm) {
  constexpr int KSTEPS = D / 32;            // MFMA k-steps over the head dimension
  constexpr int VE = D / 16;                // values a lane takes of a V row, VE m .. of lane m: 16 (8) bytes
  typedef uint32_t vpiece __attribute__((ext_vector_type(VE / 2)));
  constexpr int KBLK = PC_DEC_ITER_KEYS / 16;

  const int G = a.group;
  const int n_cols = a.n_q * G;             // valid query columns (<= 16)
  const int lane = threadIdx.x % PC_WAVE, wave = threadIdx.x / PC_WAVE;
  const int kk = lane / 16, c16 = lane % 16;

  const int bg = pc_div(bid, a.parts_div), part = bid - bg * a.parts_grid;
  const int b = pc_div(bg, a.heads_div), g = bg - b * a.n_kv_heads;

  // A wavefront streams its run of 32-key blocks, through segment boundaries; the running
  // softmax carries over (same query columns, same KV head), so a workgroup leaves one partial.
  // A cursor names the next block: where it is, plus its rows.
  struct Cursor { PcBlockCursor at; const uint16_t* k; const uint16_t* v; int keys; };
  PcSegLens lens;
  lens.seg_len = a.seg_len; lens.per_head = a.seg_len_per_head; lens.n_seg = a.n_seg;
  lens.n_kv_heads = a.n_kv_heads; lens.k_t = a.k_t; lens.b = b; lens.g = g;
  auto place = [&](const PcBlockCursor& at) {
    Cursor c; c.at = at; c.k = a.kc; c.v = a.vc; c.keys = 0;        // behind the run's end: nothing is read
    if (at.left > 0) {
      const long long first = ((((long long)b * a.n_seg + at.s) * a.n_kv_heads + g) * a.k_t + 32LL * at.blk) * D;
      c.k = a.kc + first; c.v = a.vc + first;
      c.keys = min(32, at.len - 32 * at.blk);
    }
    return c;
  };
  auto next = [&](const Cursor& c) { return place(pc_blocks_next(lens, c.at)); };

  const int first_lens = pc_first_lens(lens, lane);
  PcColumnRotation<D> rot;
  rot.begin(a.query, b, g, G, n_cols);
  // the group's last workgroup also stores the new token: nobody reads its row in this launch (the
  // lengths still exclude it)
  const bool append = a.app.k_new != nullptr && part == a.parts_grid - 1;
  PcRowAppend<D> row;
  if (append) row.begin(a.app, b * a.n_kv_heads + g);

  // A block's rows through buffer descriptors that end behind its last valid row: the rows after it arrive
  // as zeros, and behind the run's end nothing is read.  So the loads are unconditional, and the waits in
  // front of a block's arithmetic count the next block's loads as what they are, in flight (with loads
  // under a condition the compiler must assume that they were not issued and waits for all).
  // V: key i of the lane is 4 kk + i (i < 4) or 16 + 4 kk + i - 4, its values VE c16 .. + VE - 1: whole rows an instruction.
  u32x4 kbuf[2][KBLK][KSTEPS];
  vpiece vbuf[2][8];
  const int k_off = 2 * (c16 * D + 8 * kk), v_off = 2 * (4 * kk * D + VE * c16);
  auto issue_loads = [&](int buf, const Cursor& c) __attribute__((always_inline)) {
    const __amdgpu_buffer_rsrc_t kr = __builtin_amdgcn_make_buffer_rsrc((void*)c.k, 0, c.keys * (2 * D), 0x00020000);
    const __amdgpu_buffer_rsrc_t vr = __builtin_amdgcn_make_buffer_rsrc((void*)c.v, 0, c.keys * (2 * D), 0x00020000);
#pragma unroll
    for (int bi = 0; bi < KBLK; ++bi)
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks)
        kbuf[buf][bi][ks] = __builtin_amdgcn_raw_buffer_load_b128(kr, k_off, 2 * (16 * bi * D + 32 * ks), PC_BUF_NT);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if constexpr (VE == 8) vbuf[buf][i] = __builtin_amdgcn_raw_buffer_load_b128(vr, v_off, 2 * (i < 4 ? i : i + 12) * D, PC_BUF_NT);
      else vbuf[buf][i] = __builtin_amdgcn_raw_buffer_load_b64(vr, v_off, 2 * (i < 4 ? i : i + 12) * D, PC_BUF_NT);
    }
    __builtin_amdgcn_sched_barrier(0);                       // not behind the arithmetic that follows
  };

  bf16x8 bq[KSTEPS];                        // B operand: column c16 = (t, head-in-group); lane holds d = 32*ks + 8*kk .. +7
  float m_run = -INFINITY, l_run = 0.f;     // of column c16 (this lane's share of the sum)
  // O^T: o_acc[e], register i = value d = VE (4 kk + i) + e of column c16
  floatx4 o_acc[VE];
#pragma unroll
  for (int e = 0; e < VE; ++e) o_acc[e] = floatx4{0.f, 0.f, 0.f, 0.f};

  auto consume = [&](int buf, const Cursor& cur) __attribute__((always_inline)) {
    floatx4 acc[KBLK];
#pragma unroll
    for (int bi = 0; bi < KBLK; ++bi) {
      acc[bi] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks)
        acc[bi] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(bf16x8*)&kbuf[buf][bi][ks], bq[ks], acc[bi], 0, 0, 0);
    }
    float pr[KBLK][4], alpha;
    pc_decode_softmax(acc, a.scale_log2, cur.keys, kk, m_run, l_run, alpha, pr);
    u32x4 p_hi, p_lo;
#pragma unroll
    for (int bi = 0; bi < KBLK; ++bi)
#pragma unroll
      for (int j = 0; j < 4; j += 2) {
        const uint32_t h = pack_bf16x2(pr[bi][j], pr[bi][j + 1]);
        p_hi[2 * bi + j / 2] = h;
        p_lo[2 * bi + j / 2] = pack_bf16x2(pr[bi][j] - bf16_lo_to_f32(h), pr[bi][j + 1] - bf16_hi_to_f32(h));
      }
    if (__any(alpha != 1.0f)) {                      // some column's maximum grew (rare after the first keys)
#pragma unroll
      for (int e = 0; e < VE; ++e)
#pragma unroll
        for (int i = 0; i < 4; ++i) o_acc[e][i] *= alpha;
    }
#pragma unroll
    for (int e = 0; e < VE; ++e) {
      u32x4 va;                                      // value VE c16 + e of the lane's 8 keys
#pragma unroll
      for (int i = 0; i < 4; ++i)
        va[i] = __builtin_amdgcn_perm(vbuf[buf][2 * i + 1][e / 2], vbuf[buf][2 * i][e / 2], e % 2 ? 0x07060302u : 0x05040100u);
      o_acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(bf16x8*)&va, *(bf16x8*)&p_lo, o_acc[e], 0, 0, 0);
      o_acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(*(bf16x8*)&va, *(bf16x8*)&p_hi, o_acc[e], 0, 0, 0);
    }
  };

  Cursor cur = place(pc_blocks_begin(lens, part, a.parts_grid, a.parts_div, __builtin_amdgcn_readfirstlane(wave), lane, first_lens));
  issue_loads(0, cur);

  rot.finish(a.query, b, g, G, n_cols, sm.q);
  PC_LDS_BARRIER();
  if (append) {
    const long long seg0 = (((long long)b * a.n_seg + a.n_seg - 1) * a.n_kv_heads + g) * a.k_t * D;
    row.finish(a.app, a.query.rope, b * a.n_kv_heads + g, lens.len(a.n_seg - 1), a.k_t, const_cast<uint16_t*>(a.kc) + seg0,
               const_cast<uint16_t*>(a.vc) + seg0);
    if (a.app.q_rot)
      for (int x = threadIdx.x; x < n_cols * D; x += blockDim.x)     // one query row: heads g G .. are adjacent
        a.app.q_rot[((long long)b * a.n_q_heads + g * G) * D + x] = sm.q[x / D][x % D];
  }
#pragma unroll
  for (int ks = 0; ks < KSTEPS; ++ks) {
    u32x4 raw = *(const u32x4*)(sm.q[min(c16, n_cols - 1)] + 32 * ks + 8 * kk);
    if (c16 >= n_cols) raw = u32x4{0, 0, 0, 0};
    bq[ks] = *(bf16x8*)&raw;
  }

  // (no way out in the middle: it would join the loop's end, where the compiler would then have to take
  // either buffer for the one asked for last)
  while (cur.at.left > 0) {
    const Cursor nx = next(cur);
    issue_loads(1, nx);
    consume(0, cur);
    cur = next(nx);
    issue_loads(0, cur);
    if (nx.at.left > 0) consume(1, nx);
  }

  // ---- wavefront totals, then one partial per workgroup
  l_run = pc_rows_sum(l_run);
  if (kk == 0) { sm.m[wave][c16] = m_run; sm.l[wave][c16] = l_run; }
  if (c16 < n_cols) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int e = 0; e < VE; e += 4)
        *(floatx4*)&sm.o[wave][c16][VE * (4 * kk + i) + e] = floatx4{o_acc[e][i], o_acc[e + 1][i], o_acc[e + 2][i], o_acc[e + 3][i]};
  }
  pc_write_partial<D>(sm, G, n_cols, a.n_q, a.n_q_heads, (long long)b * a.n_parts + a.part0 + part, g, a.part_o, a.part_lse);
}

static inline PcDecodeQuery pc_decode_query(const void* q, int pos0, float base, int n_q, int n_q_heads, int head_dim) {
  PcDecodeQuery x;
  x.q = (const uint16_t*)q; x.pos0 = pos0; x.n_q = n_q; x.n_q_heads = n_q_heads;
  x.rope = pc_rope_factors(base > 1.0f ? base : 2.0f, head_dim);        // (not looked at where nothing is rotated)
  return x;
}
static inline PcDecodeArgs pc_decode_args(const PcDecodeQuery& query, const void* kc, const void* vc,
                                          const int32_t* seg_len, int seg_len_per_head, int n_seg,
                                          int k_t, int n_kv_heads, float scale, float* part_o, float* part_lse,
                                          int n_parts, int part0, int parts_grid, const PcDecodeAppend& app) {
  PcDecodeArgs a;
  a.query = query; a.part0 = part0; a.app = app;
  a.kc = (const uint16_t*)kc; a.vc = (const uint16_t*)vc;
  a.seg_len = seg_len; a.seg_len_per_head = seg_len_per_head; a.part_o = part_o; a.part_lse = part_lse;
  a.n_q = query.n_q; a.n_seg = n_seg; a.k_t = k_t; a.n_q_heads = query.n_q_heads; a.n_kv_heads = n_kv_heads;
  a.group = query.n_q_heads / n_kv_heads;
  a.parts_grid = parts_grid; a.parts_div = pc_div_by(parts_grid); a.heads_div = pc_div_by(n_kv_heads);
  a.n_parts = n_parts;
  a.scale_log2 = scale * PC_DEC_LOG2E;
  return a;
}
