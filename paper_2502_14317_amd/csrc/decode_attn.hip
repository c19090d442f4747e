// Parallel (global) attention for few query rows: the HBM-bound split-KV kernel and the exact
// logsumexp merge (Eq. 9-11: one softmax over [K^1 .. K^S, K^q], evaluated as independent
// per-piece softmaxes that are merged by LSE = log sum exp(lse_p), o = sum exp(lse_p - LSE) o_p).
//
// Every K/V byte is read exactly once, so the kernel is bound by HBM bandwidth.  Design:
//   * the keys of a (sequence, KV head) group, all its segments end to end in blocks of 32, are
//     cut into equal runs, one workgroup (4 wavefronts) each, so that the launch has one
//     workgroup per CU where the shapes allow (long runs, equal work, no ragged last round);
//     a wavefront owns a contiguous quarter of the run and streams it 32 keys at a time with
//     16-byte loads, the next 32 keys already in flight while the current ones are used;
//   * the query columns of one KV group (n_q * G <= 16) form the N side of a 16x16x32 bf16
//     MFMA: S^T = K Q^T, so the lane that owns a column owns its running max and sum;
//   * P V runs on the same MFMA, V transposed in registers, P as two bf16 halves (hi + lo);
//   * partial (o, lse) per workgroup go to the workspace; a second kernel merges them.
#include "decode_core.h"
#include "rope.h"

template <int D>
__global__ __launch_bounds__(PC_DEC_WAVES * PC_WAVE) void decode_attn_kernel(PcDecodeArgs a) {
  __shared__ PcDecodeLds<D> sm;
  pc_decode_workgroup<D>(a, blockIdx.x, sm);
}

// ------------------------------------------------------------------------------------------
// Merge of partials (+ the causal self segment of the few-row path, or a decoding step's new token).  One
// workgroup of 256 threads per (b, t, h): D / 4 threads take a partial, 4 values each, 8 (16) partials at a
// time, under a running maximum of their own, and are put together at the end in a fixed order, so that
// nothing waits for the logsumexps of all partials first.  lse values are natural logarithms.
// Latency: one sequence's 32 partials 4.8 us with D threads a row and the weights in a pass of their own, 4.2 with the
// own key and the length to count asked for behind the partials' arithmetic, now 3.9 (8 steps 157.6 -> 154 us).
struct PcMergeArgs {
  const float* part_o;     // [B, P, n_q, H_q, D]
  const float* part_lse;   // [B, P, n_q, H_q]
  const uint16_t* q;       // rotated q, used only with a self segment or a step
  const uint16_t* k_self;  // [B, n_q, H_kv, D] or nullptr: row t sees keys 0 .. t
  const uint16_t* v_self;
  PcMergeStep step;
  uint16_t* out;           // [B, n_q, H_q, D]
  float* lse_out;          // [B, H_q, n_q] or nullptr
  int n_rows;              // B n_q H_q
  int n_q, n_q_heads, n_kv_heads, n_parts;
  PcDiv q_div, heads_div, group_div;    // by n_q, n_q_heads, H_q / H_kv
  float scale;
};

// PARTS: there are partials (without a condition on their loads the waits behind them count those as in flight)
template <int D, bool PARTS>
__global__ __launch_bounds__(256) void merge_kernel(PcMergeArgs a) {
  constexpr int TPR = D / 4, GROUPS = 256 / TPR, U = 4;
  __shared__ floatx4 num_lds[GROUPS][TPR];
  __shared__ float2 ml_lds[GROUPS];
  const int grp = threadIdx.x / TPR, d4 = threadIdx.x % TPR * 4;
  // (a workgroup behind the last row goes along and writes nothing: a way out here would part the arguments' loads)
  const uint32_t at = blockIdx.y * gridDim.x + blockIdx.x, bid = min(at, (uint32_t)a.n_rows - 1u);
  const bool own_row = at < (uint32_t)a.n_rows;
  const int bt = pc_div((int)bid, a.heads_div), h = (int)bid - bt * a.n_q_heads;
  const int b = pc_div(bt, a.q_div), t = bt - b * a.n_q;
  const int g = pc_div(h, a.group_div);
  // partial p of this (b, t, h): row = row0 + p * row_stride
  const long long row0 = ((long long)b * a.n_parts * a.n_q + t) * a.n_q_heads + h;
  const long long row_stride = (long long)a.n_q * a.n_q_heads;
  const long long orow = ((long long)b * a.n_q + t) * a.n_q_heads + h;

  // All that comes from memory is asked for in front of the arithmetic: the first round of partials, the
  // group's first own key (from the last group on: it has the fewest partials), the length to count up.
  float l[U];
  floatx4 x[U];
  auto load = [&](int p0) __attribute__((always_inline)) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const long long row = row0 + min(p0 + u * GROUPS, a.n_parts - 1) * row_stride;
      l[u] = a.part_lse[row];
      x[u] = *(const floatx4*)(a.part_o + row * D + d4);
    }
  };
  const bool counts = a.step.seg_len && h == 0 && own_row;
  const int n_len = a.step.len_per_head ? a.n_kv_heads : 1;
  int32_t* len_at = a.step.seg_len + ((long long)b * a.step.n_seg + a.step.n_seg - 1) * n_len;
  int own_len = 0;
  // (by a vector load, so that the partials follow it at once: a scalar one would be waited for with the arguments)
  int step_row = 0, lane0 = 0;
  asm volatile("" : "+v"(lane0));
  if (a.step.self_row) step_row = a.step.self_row[b * a.n_kv_heads + g + lane0];
  if (PARTS) load(grp);
  step_row = __builtin_amdgcn_readfirstlane(step_row);
  // keys of the launch's own: the self segment's first t + 1, or a step's one
  const uint16_t* k_self = a.step.self_row ? a.step.k : a.k_self;
  const uint16_t* v_self = a.step.self_row ? a.step.v : a.v_self;
  const int n_self = a.step.self_row ? step_row >= 0 : (a.k_self ? t + 1 : 0);
  const long long self0 =
      a.step.self_row ? ((((long long)b * a.step.n_seg + a.step.n_seg - 1) * a.n_kv_heads + g) * a.step.cap + max(step_row, 0)) * D
                      : ((long long)b * a.n_q * a.n_kv_heads + g) * D;
  uint2 kw = make_uint2(0, 0), vw = kw, qw = kw;
  auto load_self = [&](int j) __attribute__((always_inline)) {
    const long long from = self0 + (long long)j * a.n_kv_heads * D + d4;
    kw = *(const uint2*)(k_self + from); vw = *(const uint2*)(v_self + from);
  };
  if (k_self) {
    qw = *(const uint2*)(a.q + orow * D + d4);
    load_self(max(min(GROUPS - 1 - grp, n_self - 1), 0));
  }
  if (counts) own_len = len_at[min((int)threadIdx.x, n_len - 1)];
  __builtin_amdgcn_sched_barrier(0);

  float m = -INFINITY, den = 0.f;
  floatx4 num = {0.f, 0.f, 0.f, 0.f};
  for (int p0 = grp; PARTS && p0 < a.n_parts; p0 += GROUPS * U) {
    if (p0 != grp) load(p0);
    float top = m;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (p0 + u * GROUPS >= a.n_parts) l[u] = -INFINITY;
      top = fmaxf(top, l[u]);
    }
    if (top > -INFINITY) {
      const float w0 = expf(m - top);
      m = top; den *= w0;
#pragma unroll
      for (int e = 0; e < 4; ++e) num[e] *= w0;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const float w = expf(l[u] - top);
        den += w;
#pragma unroll
        for (int e = 0; e < 4; ++e) num[e] += w * x[u][e];
      }
    }
  }
  for (int j = GROUPS - 1 - grp; j < n_self; j += GROUPS) {
    if (j >= GROUPS) load_self(j);
    float s = bf16_lo_to_f32(kw.x) * bf16_lo_to_f32(qw.x) + bf16_hi_to_f32(kw.x) * bf16_hi_to_f32(qw.x) +
              bf16_lo_to_f32(kw.y) * bf16_lo_to_f32(qw.y) + bf16_hi_to_f32(kw.y) * bf16_hi_to_f32(qw.y);
#pragma unroll
    for (int off = TPR / 2; off > 0; off >>= 1) s += __shfl_xor(s, off);
    s *= a.scale;
    const float top = fmaxf(m, s);
    const float w0 = m > -INFINITY ? expf(m - top) : 0.f, w = expf(s - top);
    m = top;
    den = den * w0 + w;
    num[0] = num[0] * w0 + w * bf16_lo_to_f32(vw.x); num[1] = num[1] * w0 + w * bf16_hi_to_f32(vw.x);
    num[2] = num[2] * w0 + w * bf16_lo_to_f32(vw.y); num[3] = num[3] * w0 + w * bf16_hi_to_f32(vw.y);
  }
  num_lds[grp][d4 / 4] = num;
  if (d4 == 0) ml_lds[grp] = make_float2(m, den);
  __syncthreads();
  if (threadIdx.x < TPR && own_row) {
    float M = -INFINITY;
#pragma unroll
    for (int i = 0; i < GROUPS; ++i) M = fmaxf(M, ml_lds[i].x);
    float tot = 0.f;
    floatx4 y = {0.f, 0.f, 0.f, 0.f};
    if (M > -INFINITY) {
#pragma unroll
      for (int i = 0; i < GROUPS; ++i) {
        const float w = expf(ml_lds[i].x - M);
        const floatx4 x = num_lds[i][d4 / 4];
        tot += w * ml_lds[i].y;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] += w * x[e];
      }
    }
    const float inv = tot > 0.f ? 1.f / tot : 0.f;
    *(uint2*)(a.out + orow * D + d4) = make_uint2(pack_bf16x2(y[0] * inv, y[1] * inv), pack_bf16x2(y[2] * inv, y[3] * inv));
    if (a.lse_out && d4 == 0)
      a.lse_out[((long long)b * a.n_q_heads + h) * a.n_q + t] = tot > 0.f ? M + logf(tot) : -INFINITY;
  }
  // count the step's row (nothing else in this launch looks at the lengths)
  if (counts) {
    for (int i = threadIdx.x; i < n_len; i += 256) {
      const int len = min(max(i < 256 ? own_len : len_at[i], 0), a.step.cap);
      len_at[i] = min(len + 1, a.step.cap);
    }
  }
}

// Merge for a block of query rows: bound by reading the fp32 partials once.  A thread owns 4
// values of one output row (D / 4 threads a row, 16-byte loads, whole rows per wavefront) and
// computes the row's weights for itself: the partials' logsumexps are the same address for all
// threads of a row.
template <int D>
__global__ __launch_bounds__(256) void merge_rows_kernel(const float* __restrict__ part_o,
                                                         const float* __restrict__ part_lse,
                                                         uint16_t* __restrict__ out,
                                                         float* __restrict__ lse_out, long long n_rows,
                                                         int n_q, int n_q_heads, int n_parts) {
  constexpr int TPR = D / 4;
  const long long row = ((long long)blockIdx.x * 256 + threadIdx.x) / TPR;      // (b, t, h)
  const int d4 = (threadIdx.x % TPR) * 4;
  if (row >= n_rows) return;
  const long long th = (long long)n_q * n_q_heads, b = row / th, in_b = row % th;
  const float* lse = part_lse + b * n_parts * th + in_b;
  const float* po = part_o + (b * n_parts * th + in_b) * D + d4;
  float M = -INFINITY;
  for (int p = 0; p < n_parts; ++p) M = fmaxf(M, lse[p * th]);
  floatx4 num = {0.f, 0.f, 0.f, 0.f};
  float den = 0.f;
  if (M > -INFINITY) {
#pragma unroll 4
    for (int p = 0; p < n_parts; ++p) {
      const float w = expf(lse[p * th] - M);
      const floatx4 x = __builtin_nontemporal_load((const floatx4*)(po + p * th * D));
      den += w;
#pragma unroll
      for (int e = 0; e < 4; ++e) num[e] += w * x[e];
    }
  }
  float y[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) y[e] = den > 0.f ? num[e] / den : 0.f;
  *(uint2*)(out + row * D + d4) = make_uint2(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]));
  if (lse_out && d4 == 0)
    lse_out[(b * n_q_heads + in_b % n_q_heads) * n_q + in_b / n_q_heads] = den > 0.f ? M + logf(den) : -INFINITY;
}

int pc_launch_merge_rows(const float* part_o, const float* part_lse, void* out, float* lse_out, int batch,
                         int n_q, int n_q_heads, int head_dim, int n_parts, hipStream_t st) {
  const long long n_rows = (long long)batch * n_q * n_q_heads;
  const long long blocks = (n_rows * (head_dim / 4) + 255) / 256;
  if (blocks == 0) return PC_OK;
  if (blocks > 0x7fffffffLL) return PC_ERR_SHAPE;
  PcProfScope prof(PC_KERNEL_MERGE, st);
  const dim3 grid((unsigned)blocks), block(256);
  if (head_dim == 128)
    hipLaunchKernelGGL(merge_rows_kernel<128>, grid, block, 0, st, part_o, part_lse, (uint16_t*)out, lse_out,
                       n_rows, n_q, n_q_heads, n_parts);
  else
    hipLaunchKernelGGL(merge_rows_kernel<64>, grid, block, 0, st, part_o, part_lse, (uint16_t*)out, lse_out,
                       n_rows, n_q, n_q_heads, n_parts);
  PC_LAUNCH_CHECK();
  return PC_OK;
}

// ------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) void rope_q_kernel(const uint16_t* __restrict__ q, uint16_t* __restrict__ q_rot,
                                                     int n_rows, int n_q, int n_heads, int pos0, PcRope rope, double mul) {
  const uint32_t row = blockIdx.y * gridDim.x + blockIdx.x;
  if (row < (uint32_t)n_rows) pc_rope_q_workgroup<D>(q, q_rot, (int)row, n_q, n_heads, pos0, rope, mul);
}

int pc_launch_rope_q(const void* q, void* q_rot, int batch, int n_q, int n_heads, int D, int pos0,
                     float base, float mul, hipStream_t st) {
  const long long blocks = (long long)batch * n_q;
  if (blocks == 0) return PC_OK;
  if (blocks > 0x7fffffffLL - PC_GRID_X) return PC_ERR_SHAPE;
  PcProfScope prof(PC_KERNEL_ROPE_Q, st);
  const dim3 grid = pc_grid_2d(blocks), block(256);
  const PcRope rope = pc_rope_factors(pos0 >= 0 ? base : 2.0f, D);
  if (D == 128)
    hipLaunchKernelGGL(rope_q_kernel<128>, grid, block, 0, st, (const uint16_t*)q, (uint16_t*)q_rot, (int)blocks, n_q,
                       n_heads, pos0, rope, (double)mul);
  else
    hipLaunchKernelGGL(rope_q_kernel<64>, grid, block, 0, st, (const uint16_t*)q, (uint16_t*)q_rot, (int)blocks, n_q,
                       n_heads, pos0, rope, (double)mul);
  PC_LAUNCH_CHECK();
  return PC_OK;
}

// ------------------------------------------------------------------------------------------
// Decoding stage: append the K / V rows of newly generated tokens to one segment of the
// compacted cache (the growing tail behind the query block).  One workgroup per sequence: it
// reads the segment's length(s), writes the rows behind them (K rotated at pos0 + t when
// pos0 >= 0, fp64 angles) and, after a barrier that orders every read of a length before its
// update, stores the new length(s), all on the device, so a decode loop needs no host round
// trip.  Rows that would not fit the segment's capacity are dropped.
// A thread keeps its rotation pair i, so its angle is computed once per new row, not once per head.
#define PC_APPEND_THREADS 1024
__global__ __launch_bounds__(PC_APPEND_THREADS) void kv_append_kernel(
    const uint16_t* __restrict__ k_new, const uint16_t* __restrict__ v_new, int n_new, int n_seg,
    int seg, int k_t, int n_kv_heads, int D, int pos0, PcRope rope, uint16_t* __restrict__ kc,
    uint16_t* __restrict__ vc, int32_t* __restrict__ seg_len, int per_head) {
  const int b = blockIdx.x;
  const int half = D / 2;
  const long long len_base = per_head ? ((long long)b * n_seg + seg) * n_kv_heads
                                      : (long long)b * n_seg + seg;
  const int i = threadIdx.x % half;
  const double theta = pc_rope_theta(rope, i);
  int at = -1;
  double sn = 0.0, cs = 1.0;
  const long long rows = (long long)n_new * n_kv_heads;
  for (long long it = threadIdx.x / half; it < rows; it += PC_APPEND_THREADS / half) {
    const int g = (int)(it % n_kv_heads), t = (int)(it / n_kv_heads);
    const int len = min(max(seg_len[len_base + (per_head ? g : 0)], 0), k_t);
    if (len + t >= k_t) continue;                          // no room left in this head's segment
    const long long src = (((long long)b * n_new + t) * n_kv_heads + g) * D;
    const long long dst = ((((long long)b * n_seg + seg) * n_kv_heads + g) * k_t + len + t) * D;
    const uint16_t a1 = k_new[src + i], a2 = k_new[src + i + half];
    if (pos0 >= 0) {
      if (t != at) { pc_sincos((double)(pos0 + t) * theta, sn, cs); at = t; }
      const float x1 = bf16_bits_to_f32(a1), x2 = bf16_bits_to_f32(a2);
      kc[dst + i] = (uint16_t)f32_to_bf16_bits((float)(x1 * cs - x2 * sn));
      kc[dst + i + half] = (uint16_t)f32_to_bf16_bits((float)(x2 * cs + x1 * sn));
    } else {
      kc[dst + i] = a1; kc[dst + i + half] = a2;
    }
    vc[dst + i] = v_new[src + i]; vc[dst + i + half] = v_new[src + i + half];
  }
  __syncthreads();                                         // every length has been read
  const int n_len = per_head ? n_kv_heads : 1;
  for (int g = threadIdx.x; g < n_len; g += blockDim.x) {
    const int len = min(max(seg_len[len_base + g], 0), k_t);
    seg_len[len_base + g] = len + min(n_new, k_t - len);
  }
}

int pc_launch_kv_append(const void* k_new, const void* v_new, int batch, int n_new, int n_seg,
                        int seg, int k_t, int n_kv_heads, int head_dim, int pos0, float base,
                        void* kc, void* vc, int32_t* seg_len, int seg_len_per_head, hipStream_t st) {
  PcProfScope prof(PC_KERNEL_KV_APPEND, st);
  hipLaunchKernelGGL(kv_append_kernel, dim3(batch), dim3(PC_APPEND_THREADS), 0, st, (const uint16_t*)k_new,
                     (const uint16_t*)v_new, n_new, n_seg, seg, k_t, n_kv_heads, head_dim, pos0,
                     pc_rope_factors(pos0 >= 0 ? base : 2.0f, head_dim), (uint16_t*)kc, (uint16_t*)vc, seg_len,
                     seg_len_per_head);
  PC_LAUNCH_CHECK();
  return PC_OK;
}

template <int D>
static int launch_decode_d(const PcDecodeArgs& a, int batch, hipStream_t st) {
  const long long blocks = (long long)batch * a.n_kv_heads * a.parts_grid;
  if (blocks == 0) return PC_OK;
  if (blocks > 0x7fffffffLL) return PC_ERR_SHAPE;
  dim3 grid((unsigned)blocks), block(PC_DEC_WAVES * PC_WAVE);
  PcProfScope prof(PC_KERNEL_DECODE, st);
  hipLaunchKernelGGL(decode_attn_kernel<D>, grid, block, 0, st, a);
  PC_LAUNCH_CHECK();
  return PC_OK;
}

// Partials of a group that the workspace has room for: the parts that minimise rounds / parts, rounds of
// one workgroup a CU, at least one block a wavefront at full lengths, at most 64.
static int split_room(int k_t, int n_seg, long long n_bg) {
  const int n_cu = 256;                                    // MI355X
  const long long blocks_full = (long long)n_seg * ((k_t + 31) / 32);
  const long long p_cap = blocks_full / PC_DEC_WAVES;
  const int p_max = (int)(p_cap < 1 ? 1 : (p_cap > 64 ? 64 : p_cap));
  if (n_seg <= 0) return 0;                                // no segments: no launch, no partial
  int room = 1;
  double best = 0.0;
  for (int p = 1; p <= p_max; ++p) {
    const long long rounds = (n_bg * p + n_cu - 1) / n_cu;
    const double cost = (double)rounds / p / (rounds == 1 ? 0.89 : 0.81);
    if (p == 1 || cost < best * (1.0 - 1e-9)) { best = cost; room = p; }
  }
  return room;
}

PcDecodeSplit pc_decode_split(int k_t, int n_seg, int elem_bytes, int tail_cap, int head_dim, long long n_bg) {
  // The parts, within the room, of the least estimated time.  Measured over 17 shapes x 10 numbers of parts a
  // cache precision (1 to 65 sequences, 4 to 256 KV heads in all, 3 MB to 2.2 GB, data out of the caches): a
  // launch and its merge cost some 10.5 us; a workgroup alone on its CU reads 38 GB/s (8-bit, in whole KiB
  // and with two blocks ahead, 57), less as the others load the memory; 256 CUs together 6.9 (6.6) TB/s; a
  // further round of workgroups on a CU costs 3.5 us.  E.g. 16-bit, 33 sequences of 8 x 1024 keys, 8 KV heads:
  // 1 part 291 us, 4 218, 8 222, 31 (whole rounds) 268; 65: 4 parts 391, 63 499; 8-bit, one sequence of 8 x 2048:
  // 16 parts + 4 of the tail 15.5 us, 32 + 4 (a second round for 32 CUs) 19.9; 65 sequences 2 parts 192, 63 274.
  PcDecodeSplit d = {};
  d.room = split_room(k_t, n_seg, n_bg);
  d.tail_room = tail_cap > 0 ? split_room(tail_cap, 1, n_bg) : 0;
  const double seg_bytes = (double)n_seg * k_t * head_dim * 2 * elem_bytes, tail_bytes = (double)tail_cap * head_dim * 4;
  const double mem = elem_bytes == 1 ? 6.6e6 : 6.9e6, alone = elem_bytes == 1 ? 57e3 : 38e3, slower = elem_bytes == 1 ? 110.0 : 33.0;
  const int p_max = d.room > 0 ? d.room : d.tail_room;
  double best = 0.0;
  for (int p = 1; p <= p_max; ++p) {
    int parts = d.room > 0 ? p : 0, tail = d.room > 0 ? d.tail_room : p;
    if (parts > 0 && tail > 0) {                           // tail workgroups of about the others' size
      const int even = (int)(p * tail_bytes / seg_bytes + 0.5);
      tail = even < 1 ? 1 : (even < tail ? even : tail);
    }
    const long long wgs = n_bg * (parts + tail), rounds = (wgs + 255) / 256;
    double us = 10.5 + 3.5 * (double)(rounds - 1);
    if (rounds == 1) {                                     // the longest workgroup
      const double rate = alone - slower * (double)wgs, fair = mem / (double)wgs;
      const double most = (parts > 0 ? seg_bytes / parts : 0.0) > (tail > 0 ? tail_bytes / tail : 0.0) ? seg_bytes / parts : tail_bytes / tail;
      us += most / (rate < fair ? rate : fair);
    } else {
      us += (double)rounds * (seg_bytes + tail_bytes) / (parts + tail) / (mem / 256.0);
    }
    // on a par within one round: more of the CUs
    if (p == 1 || us < best * (rounds == 1 ? 1.005 : 1.0)) { best = us; d.parts = parts; d.tail_parts = tail; }
  }
  return d;
}

int pc_launch_decode(const void* q, int pos0, float base, const void* kc, const void* vc,
                     const int32_t* seg_len, int seg_len_per_head, int batch, int n_q, int n_seg, int k_t, int n_q_heads, int n_kv_heads,
                     int head_dim, float scale, float* part_o, float* part_lse, int n_parts,
                     int part0, int parts_grid, const PcDecodeAppend& app, hipStream_t st) {
  const PcDecodeArgs a = pc_decode_args(pc_decode_query(q, pos0, base, n_q, n_q_heads, head_dim), kc, vc, seg_len,
                                        seg_len_per_head, n_seg, k_t, n_kv_heads, scale, part_o,
                                        part_lse, n_parts, part0, parts_grid, app);
  return head_dim == 128 ? launch_decode_d<128>(a, batch, st) : launch_decode_d<64>(a, batch, st);
}

int pc_launch_merge(const float* part_o, const float* part_lse, const void* q_rot,
                    const void* k_self, const void* v_self, const PcMergeStep& step, void* out, float* lse_out,
                    int batch, int n_q, int n_q_heads, int n_kv_heads, int head_dim, int n_parts, float scale,
                    hipStream_t st) {
  PcMergeArgs a;
  a.part_o = part_o; a.part_lse = part_lse; a.q = (const uint16_t*)q_rot;
  a.k_self = (const uint16_t*)k_self; a.v_self = (const uint16_t*)v_self; a.step = step;
  a.out = (uint16_t*)out; a.lse_out = lse_out;
  a.n_q = n_q; a.n_q_heads = n_q_heads; a.n_kv_heads = n_kv_heads; a.n_parts = n_parts;
  a.q_div = pc_div_by(n_q); a.heads_div = pc_div_by(n_q_heads); a.group_div = pc_div_by(n_q_heads / n_kv_heads);
  a.scale = scale;
  const long long blocks = (long long)batch * n_q * n_q_heads;
  if (blocks == 0) return PC_OK;
  if (blocks > 0x7fffffffLL - PC_GRID_X) return PC_ERR_SHAPE;
  a.n_rows = (int)blocks;
  PcProfScope prof(PC_KERNEL_MERGE, st);
  const dim3 grid = pc_grid_2d(blocks);
  if (n_parts > 0) {
    if (head_dim == 128) hipLaunchKernelGGL((merge_kernel<128, true>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((merge_kernel<64, true>), grid, dim3(256), 0, st, a);
  } else {
    if (head_dim == 128) hipLaunchKernelGGL((merge_kernel<128, false>), grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL((merge_kernel<64, false>), grid, dim3(256), 0, st, a);
  }
  PC_LAUNCH_CHECK();
  return PC_OK;
}
