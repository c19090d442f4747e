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
  double log_base;
};

// The columns (query t, head) of KV head g, rotated, into LDS: column n = t * G + head in group.
template <int D>
__device__ __forceinline__ void pc_rotate_columns(const PcDecodeQuery& x, int b, int g, int G, int n_cols,
                                                  uint16_t (*cols)[D]) {
  constexpr int HALF = D / 2;
  const int i = threadIdx.x % HALF;                         // a thread keeps its rotation pair
  const double theta = exp(-2.0 * (double)i / (double)D * x.log_base);
  int at = -1;
  double sn = 0.0, cs = 1.0;
  for (int n = threadIdx.x / HALF; n < n_cols; n += blockDim.x / HALF) {
    const int t = n / G;
    if (t != at) { sincos((double)(x.pos0 + t) * theta, &sn, &cs); at = t; }
    const uint16_t* row = x.q + (((long long)b * x.n_q + t) * x.n_q_heads + g * G + n % G) * D;
    const double x1 = bf16_bits_to_f32(row[i]), x2 = bf16_bits_to_f32(row[i + HALF]);
    cols[n][i] = (uint16_t)f32_to_bf16_bits((float)(x1 * cs - x2 * sn));
    cols[n][i + HALF] = (uint16_t)f32_to_bf16_bits((float)(x2 * cs + x1 * sn));
  }
}

struct PcDecodeArgs {
  PcDecodeQuery query;
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
  struct Cursor { PcBlockCursor at; int key0; const uint16_t* k; const uint16_t* v; bool valid; };
  PcSegLens lens;
  lens.seg_len = a.seg_len; lens.per_head = a.seg_len_per_head; lens.n_seg = a.n_seg;
  lens.n_kv_heads = a.n_kv_heads; lens.k_t = a.k_t; lens.b = b; lens.g = g;
  auto place = [&](const PcBlockCursor& at) {
    Cursor c; c.at = at; c.valid = at.valid; c.key0 = 32 * at.blk; c.k = nullptr; c.v = nullptr;
    if (at.valid) {
      const long long seg_base = ((((long long)b * a.n_seg + at.s) * a.n_kv_heads + g) * a.k_t) * D;
      c.k = a.kc + seg_base; c.v = a.vc + seg_base;
    }
    return c;
  };
  auto next = [&](const Cursor& c) { return place(pc_blocks_next(lens, c.at)); };

  // B operand: column c16 = (t, head-in-group); lane holds d = 32*ks + 8*kk .. +7
  bf16x8 bq[KSTEPS];
  {
    const bool valid = c16 < n_cols;
    const int n = valid ? c16 : 0;
    if (a.query.pos0 >= 0) {
      pc_rotate_columns<D>(a.query, b, g, G, n_cols, q_lds);
      __syncthreads();
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks) {
        uint4 raw = valid ? *(const uint4*)(q_lds[n] + 32 * ks + 8 * kk) : make_uint4(0, 0, 0, 0);
        bq[ks] = *(bf16x8*)&raw;
      }
    } else {
      const uint16_t* qrow = a.query.q + (((long long)b * a.n_q + n / G) * a.n_q_heads + g * G + n % G) * D;
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks) {
        uint4 raw = valid ? *(const uint4*)(qrow + 32 * ks + 8 * kk) : make_uint4(0, 0, 0, 0);
        bq[ks] = *(bf16x8*)&raw;
      }
    }
  }

  float m_run = -INFINITY, l_run = 0.f;     // of column c16 (this lane's share of the sum)
  float o_acc[NQ][8];
#pragma unroll
  for (int n = 0; n < NQ; ++n)
#pragma unroll
    for (int e = 0; e < 8; ++e) o_acc[n][e] = 0.f;

  const int v_row = lane / LPR, v_piece = lane % LPR;

  uint4 kbuf[2][KBLK][KSTEPS], vbuf[2][VLOADS];
  auto issue_loads = [&](int buf, const Cursor& c) {
#pragma unroll
    for (int bi = 0; bi < KBLK; ++bi) {
      const int row = min(c.key0 + 16 * bi + c16, c.at.len - 1);
#pragma unroll
      for (int ks = 0; ks < KSTEPS; ++ks)
        kbuf[buf][bi][ks] = pc_load_once((const uint4*)(c.k + (long long)row * D + 32 * ks + 8 * kk));
    }
#pragma unroll
    for (int i = 0; i < VLOADS; ++i) {
      const int row = min(c.key0 + RPI * i + v_row, c.at.len - 1);
      vbuf[buf][i] = pc_load_once((const uint4*)(c.v + (long long)row * D + 8 * v_piece));
    }
  };

  auto consume = [&](int buf, const Cursor& cur) {
    const int key0 = cur.key0, w_end = cur.at.len;
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
      for (int j = 0; j < 4; ++j) {
        const int key = key0 + 16 * bi + 4 * kk + j;
        sv[bi][j] = (key < w_end) ? acc[bi][j] * a.scale_log2 : -INFINITY;
        bmax = fmaxf(bmax, sv[bi][j]);
      }
    bmax = fmaxf(bmax, __shfl_xor(bmax, 16));
    bmax = fmaxf(bmax, __shfl_xor(bmax, 32));
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
      const uint4 raw = vbuf[buf][i];
      float vf[8];
      vf[0] = bf16_lo_to_f32(raw.x); vf[1] = bf16_hi_to_f32(raw.x);
      vf[2] = bf16_lo_to_f32(raw.y); vf[3] = bf16_hi_to_f32(raw.y);
      vf[4] = bf16_lo_to_f32(raw.z); vf[5] = bf16_hi_to_f32(raw.z);
      vf[6] = bf16_lo_to_f32(raw.w); vf[7] = bf16_hi_to_f32(raw.w);
#pragma unroll
      for (int n = 0; n < NQ; ++n) {
        const float p = p_lds[wave][key_local][n];    // 0 for masked keys
#pragma unroll
        for (int e = 0; e < 8; ++e) o_acc[n][e] = fmaf(p, vf[e], o_acc[n][e]);
      }
    }
    PC_WAVE_LDS_SYNC();
  };

  Cursor cur = place(pc_blocks_begin(lens, part, a.parts_grid, __builtin_amdgcn_readfirstlane(wave),
                                     PC_DEC_WAVES, lane));
  if (cur.valid) {
    issue_loads(0, cur);
    while (true) {
      Cursor nx = next(cur);
      if (nx.valid) issue_loads(1, nx);
      consume(0, cur);
      if (!nx.valid) break;
      cur = nx;
      nx = next(cur);
      if (nx.valid) issue_loads(0, nx);
      consume(1, cur);
      if (!nx.valid) break;
      cur = nx;
    }
  }

  // ---- wavefront totals: sum the per-lane shares
  l_run += __shfl_xor(l_run, 16);
  l_run += __shfl_xor(l_run, 32);
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

static inline PcDecodeQuery pc_decode_query(const void* q, int pos0, float base, int n_q, int n_q_heads) {
  PcDecodeQuery x;
  x.q = (const uint16_t*)q; x.pos0 = pos0; x.n_q = n_q; x.n_q_heads = n_q_heads;
  x.log_base = log((double)(pos0 >= 0 ? base : 2.0f));
  return x;
}
static inline PcDecodeArgs pc_decode_args(const PcDecodeQuery& query, const void* kc, const void* vc,
                                          const int32_t* seg_len, int seg_len_per_head, int batch, int n_seg,
                                          int k_t, int n_kv_heads, float scale, float* part_o, float* part_lse,
                                          int n_parts, int part0) {
  PcDecodeArgs a;
  a.query = query; a.part0 = part0;
  a.kc = (const uint16_t*)kc; a.vc = (const uint16_t*)vc;
  a.seg_len = seg_len; a.seg_len_per_head = seg_len_per_head; a.part_o = part_o; a.part_lse = part_lse;
  a.n_q = query.n_q; a.n_seg = n_seg; a.k_t = k_t; a.n_q_heads = query.n_q_heads; a.n_kv_heads = n_kv_heads;
  a.parts_grid = pc_decode_split(k_t, n_seg, (long long)batch * n_kv_heads).n_parts;
  a.n_parts = n_parts;
  a.scale_log2 = scale * PC_DEC_LOG2E;
  return a;
}
