// Top-k selection of chunks (Eq. 3-4: a fixed number of best chunks) and of tokens per KV
// head (Eq. 7), under the total order (score descending, index ascending): of equal scores
// the lower index wins.  Scores are mapped to unsigned keys whose integer order is the float
// order, so every comparison is exact integer work.
#include "pc_common.h"

// ------------------------------------------------------------------------------------------
// Chunks: n <= 4096.  One workgroup; rank by counting.  rank(i) = #{j : key_j > key_i or
// (key_j == key_i and j < i)}; item i is kept iff rank(i) < k and lands at out[rank(i)].
__global__ __launch_bounds__(256) void select_chunks_kernel(const float* __restrict__ score, int n,
                                                            int k, int32_t* __restrict__ out_idx,
                                                            float* __restrict__ out_score) {
  __shared__ uint32_t keys[4096];
  for (int i = threadIdx.x; i < n; i += blockDim.x) keys[i] = pc_order_key(score[i]);
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    const uint32_t ki = keys[i];
    int rank = 0;
    for (int j = 0; j < n; ++j) {
      const uint32_t kj = keys[j];
      rank += (kj > ki) || (kj == ki && j < i);
    }
    if (rank < k) {
      out_idx[rank] = i;
      if (out_score) out_score[rank] = score[i];
    }
  }
}

int pc_launch_select_chunks(const float* score, int n, int k, int32_t* out_idx, float* out_score,
                            hipStream_t st) {
  PcProfScope prof(PC_KERNEL_SELECT_CHUNKS, st);
  hipLaunchKernelGGL(select_chunks_kernel, dim3(1), dim3(256), 0, st, score, n, k, out_idx,
                     out_score);
  PC_LAUNCH_CHECK();
  return PC_OK;
}

// ------------------------------------------------------------------------------------------
// The fixed-size priority queue of chunks (sec. 3.1 "Chunk eviction"), updated with one batch
// of newly encoded chunks.  The queue lives on the device: ids in rank order (-1 = empty
// entry), their scores, and the KV slot each entry owns.  One workgroup ranks the resident
// entries and the batch together by counting, under (score descending, earlier chunk first;
// NaN lowest, empty entries last); the best `cap` stay.  A chunk that stays keeps its slot; the
// entrants, in rank order, take the free slots in ascending order.  slot_src[s] names, for the
// later selection / gather launches, the batch-local index of the chunk that enters slot s, or
// -1 where the slot keeps its content.
#define PC_QUEUE_MAX 1024              // capacity and batch size limit (each)
__global__ __launch_bounds__(256) void chunk_queue_kernel(
    const float* __restrict__ batch_score, int n_batch, int chunk_id0, int cap,
    int32_t* __restrict__ queue_id, float* __restrict__ queue_score,
    int32_t* __restrict__ queue_slot, int32_t* __restrict__ slot_src) {
  __shared__ uint32_t key[2 * PC_QUEUE_MAX];
  __shared__ int32_t id[2 * PC_QUEUE_MAX], slot[2 * PC_QUEUE_MAX];
  __shared__ float val[2 * PC_QUEUE_MAX];
  __shared__ int32_t new_id[PC_QUEUE_MAX], new_slot[PC_QUEUE_MAX];
  __shared__ float new_val[PC_QUEUE_MAX];
  __shared__ uint8_t used[PC_QUEUE_MAX];
  const int n = cap + n_batch;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    if (i < cap) {
      id[i] = queue_id[i]; val[i] = queue_score[i]; slot[i] = queue_slot[i];
    } else {
      id[i] = chunk_id0 + (i - cap); val[i] = batch_score[i - cap]; slot[i] = -1;
    }
    key[i] = pc_order_key(val[i]);
  }
  for (int i = threadIdx.x; i < cap; i += blockDim.x) { new_id[i] = -1; new_slot[i] = -1; new_val[i] = 0.f; used[i] = 0; slot_src[i] = -1; }
  __syncthreads();
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    if (id[i] < 0) continue;                                   // an empty entry ranks behind every chunk
    const uint32_t ki = key[i];
    const int ii = id[i];
    int rank = 0;
    for (int j = 0; j < n; ++j) {
      const uint32_t kj = key[j];
      rank += (id[j] >= 0) && ((kj > ki) || (kj == ki && id[j] < ii));
    }
    if (rank < cap) {
      new_id[rank] = ii; new_val[rank] = val[i]; new_slot[rank] = slot[i];
      if (slot[i] >= 0 && slot[i] < cap) used[slot[i]] = 1;
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int f = 0;                                                  // next candidate free slot
    for (int r = 0; r < cap; ++r) {
      if (new_id[r] < 0 || new_slot[r] >= 0) continue;          // empty, or a resident chunk
      while (f < cap && used[f]) ++f;
      if (f >= cap) break;                                      // cannot happen: at most cap entries hold slots
      new_slot[r] = f; used[f] = 1;
      slot_src[f] = new_id[r] - chunk_id0;
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < cap; i += blockDim.x) {
    queue_id[i] = new_id[i]; queue_score[i] = new_val[i]; queue_slot[i] = new_slot[i];
  }
}

int pc_launch_chunk_queue(const float* batch_score, int n_batch, int chunk_id0, int cap,
                          int32_t* queue_id, float* queue_score, int32_t* queue_slot,
                          int32_t* slot_src, hipStream_t st) {
  PcProfScope prof(PC_KERNEL_CHUNK_QUEUE, st);
  hipLaunchKernelGGL(chunk_queue_kernel, dim3(1), dim3(256), 0, st, batch_score, n_batch, chunk_id0,
                     cap, queue_id, queue_score, queue_slot, slot_src);
  PC_LAUNCH_CHECK();
  return PC_OK;
}

// ------------------------------------------------------------------------------------------
// Tokens: one workgroup per (selected chunk, KV head), the n keys in registers: wavefront w owns a
// contiguous index range, KPT slots of 64 consecutive indices.
//  1. The k-th largest key T by counting keys into 2048 equal bins between the smallest and the
//     largest key left, finding the bin that holds it and going on inside that bin (at most three
//     rounds, 11 bits each; as a rule two).  The bins cover the range that the keys really have, so
//     neighbouring scores fall into different bins and the LDS counters do not collide.
//  2. Ordered compaction: every wavefront counts its keys above T and equal to T, the counts are
//     prefix-summed over wavefronts, and a second sweep emits index i iff key_i > T, or key_i == T
//     and fewer than need_eq equal keys precede it.  Output is ascending by construction and ties
//     go to the lower index.
// Attention calibration (Eq. 8) is a predicate on the keys: a token of the position class
// [cls_lo, cls_hi) whose score is above lambda gets key 0, below every candidate (a NaN score
// is a candidate with key 1), and k shrinks to the number of candidates when fewer are left;
// the unused tail of the output is filled with -1 and the kept count is reported.
// Measured, before (keys in LDS, four 8-bit radix passes) and now: 512 tokens x
// 16 workgroups 7.0 -> 5.8 us, 3584 x 32 13.8 -> 9.2, 7680 x 64 27 -> 15.  (Two bits a round counted with
// ballots, no histogram: 8.5, 14.6 and 23.8.)  A bin of up to PC_SEL_FEW keys is ranked by counting instead of
// another round: in a layer's launch 2011 tokens x 40 11.6 -> 10.3, 7680 x 64 17.1 -> 14.9, 3584 x 32 12.
// The bins are cleared while the scores are on their way, and where a layer has few chunks the scores of all of them
// are asked for before the chunk is known (one memory latency less): 1 chunk of 3584 tokens x 32 12.0 -> 9.8 us (8.2 with its block sums asked for at once), 4 of
// 512 x 16 7.1 -> 7.0; 12 chunks of 3584 x 32, their chunks known, 12.0 -> 10.5.
// The layer's gather in the same launch where a segment is small (PC_SEL_GATHER bytes of K and V): the workgroup
// copies the rows that it has just selected (16 segments of 128 rows of 64 values: 6.7 + 3.7 us -> 7.7).  One CU
// moves about 50 bytes a nanosecond, so larger segments are left to the gather's own launch.
#define PC_SEL_BINS 2048
#define PC_SEL_FEW 256        // so many keys of a bin are ranked by counting: one pass over them instead of a round
#define PC_SEL_GATHER 65536
#define PC_SEL_AHEAD 8        // so many scores a thread are asked for before the chunk is known, where that is all chunks'

// A layer's chunk selection in the same launch: every workgroup adds up the chunks' block sums (the order
// of pc_chunk_sum, a wavefront a chunk, its 4 x 64 strided sums asked for at once), ranks them as
// select_chunks_kernel does and takes the chunk of its rank; the first workgroup writes scores and ranks.
// Every workgroup reads all the sums, so it pays for few of them only: a chunk costs about 0.1 us, 1000 sums 0.2,
// against two launches (three with the gather, where the rows of small segments are copied here too).  This / apart
// (us), chunks x sums, 2048 tokens x 64: 4 x 128 7.1 / 9.7, 16 x 128 8.3 / 10.1, 24 x 320 10.2 / 10.5, 32 x 256 10.8 / 10.5,
// 64 x 32 13.1 / 11.3, 64 x 2048 39 / 12; with the gather of 128 rows of 64 values 4 x 128 6.7 / 13.3, 32 x 256 10.5 / 12.0,
// 48 x 256 12.6 / 12.4, 64 x 64 12.8 / 13.0, 64 x 2048 39 / 13.
#define PC_SEL_CHUNKS 64
#define PC_SEL_BLOCKS 2048
#define PC_SEL_CHUNK_COST 400          // a chunk, in sums
#define PC_SEL_COST 18000              // most that all chunks may cost, in sums
#define PC_SEL_COST_GATHER 30000       // with the gather
struct PcSelectChunks {
  PcChunkSum sum;
  int n_chunks;
  int32_t* idx;            // [n_sel] out
  float* top;              // [n_sel] out, nullable
};
struct PcSelectGather {
  const uint4* k_src;      // [C, rows, H_kv, D], nullptr: no gather
  const uint4* v_src;
  uint4* k_dst;            // [n_sel, H_kv, k, D]
  uint4* v_dst;
  int rows, pieces;        // pieces = D / 8
};
// rows list[0 .. k) (k_eff valid ones, zeros behind) of chunk c, KV head g to segment seg
template <int THREADS>
__device__ __forceinline__ void select_gather(const PcSelectGather& x, const uint32_t* list, int k, int k_eff, int c, int g,
                                              int n_kv_heads, long long seg) {
  constexpr int UNROLL = 4;
  const int piece = threadIdx.x % x.pieces, per_step = THREADS / x.pieces;
  const long long src0 = ((long long)c * x.rows * n_kv_heads + g) * x.pieces + piece, dst0 = seg * k * x.pieces + piece;
  for (int r0 = threadIdx.x / x.pieces; r0 < k; r0 += UNROLL * per_step) {
    uint4 kv[UNROLL], vv[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int r = r0 + u * per_step;
      kv[u] = vv[u] = make_uint4(0, 0, 0, 0);
      if (r < k_eff) {
        const long long src = src0 + (long long)list[r] * n_kv_heads * x.pieces;
        kv[u] = x.k_src[src]; vv[u] = x.v_src[src];
      }
    }
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int r = r0 + u * per_step;
      if (r < k) { x.k_dst[dst0 + (long long)r * x.pieces] = kv[u]; x.v_dst[dst0 + (long long)r * x.pieces] = vv[u]; }
    }
  }
}
template <int THREADS>
__device__ __forceinline__ int select_own_chunk(const PcSelectChunks& x, int n_sel, int s, bool writer) {
  __shared__ float score[PC_SEL_CHUNKS];
  __shared__ int own;
  const int wave = threadIdx.x / PC_WAVE, lane = threadIdx.x % PC_WAVE;
  for (int c = wave; c < x.n_chunks; c += THREADS / PC_WAVE) {
    const float* src = x.sum.blk_sum + (long long)c * x.sum.per_chunk;
    float part[4] = {0.f, 0.f, 0.f, 0.f};
    for (int i0 = 0; i0 < x.sum.per_chunk; i0 += 256) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = i0 + 64 * j + lane;
        const float v = src[min(i, x.sum.per_chunk - 1)];          // (under a condition each would be waited for)
        part[j] += i < x.sum.per_chunk ? v : 0.f;
      }
    }
    float v = (part[0] + part[2]) + (part[1] + part[3]);
#pragma unroll
    for (int off = PC_WAVE / 2; off > 0; off >>= 1) v += __shfl_xor(v, off);
    if (lane == 0) score[c] = v;
  }
  __syncthreads();
  const int i = threadIdx.x;
  if (i < x.n_chunks) {
    const uint32_t ki = pc_order_key(score[i]);
    int rank = 0;
    for (int j = 0; j < x.n_chunks; ++j) {
      const uint32_t kj = pc_order_key(score[j]);
      rank += (kj > ki) || (kj == ki && j < i);
    }
    if (rank == s) own = i;
    if (writer) {
      x.sum.chunk_score[i] = score[i];
      if (rank < n_sel) {
        x.idx[rank] = i;
        if (x.top) x.top[rank] = score[i];
      }
    }
  }
  __syncthreads();
  return own;
}

// CHUNKS: the chunk is found here (chunk_idx is not read), otherwise it is chunk_idx[s]
template <int KPT, int THREADS, bool CHUNKS>
__global__ __launch_bounds__(THREADS) void select_tokens_kernel(
    const float* __restrict__ tok_score, const int32_t* __restrict__ chunk_idx, int n_kv_heads, PcDiv heads_div,
    int n, int k, float lambda, int cls_lo, int cls_hi, const int32_t* __restrict__ chunk_lens,
    int32_t* __restrict__ out_idx, int32_t* __restrict__ out_cnt, PcSelectChunks chunks, PcSelectGather gather) {
  constexpr int WAVES = THREADS / PC_WAVE, BPT = PC_SEL_BINS / THREADS;      // bins per thread
  __shared__ uint32_t hist[PC_SEL_BINS];
  __shared__ uint32_t sh_cand, sh_min, sh_max, sh_bin, sh_need, sh_in_bin, sh_few;
  __shared__ uint32_t wave_tot[WAVES], wave_gt[WAVES], wave_eq[WAVES];

  const int s = pc_div(blockIdx.x, heads_div), g = blockIdx.x - s * n_kv_heads;
  const int wave = threadIdx.x / PC_WAVE, lane = threadIdx.x % PC_WAVE;
  const int first = wave * (KPT * PC_WAVE) + lane; // index of the thread's slot 0; slot j: + 64 j
  // The scores of chunk c0 + AHEAD - 1 at most, slot j of chunk c0 + a in x[a KPT + j]
  constexpr int AHEAD = KPT <= PC_SEL_AHEAD ? PC_SEL_AHEAD / KPT : 1;
  float x[AHEAD * KPT];
  auto load = [&](int c0, int n_chunks) __attribute__((always_inline)) {
#pragma unroll
    for (int a = 0; a < AHEAD; ++a)
      if (a < n_chunks) {
        const float* src = tok_score + ((long long)(c0 + a) * n_kv_heads + g) * n;
#pragma unroll
        for (int j = 0; j < KPT; ++j) x[a * KPT + j] = src[min(first + PC_WAVE * j, n - 1)];
      }
  };
  int c;
  const bool ahead = CHUNKS && chunks.n_chunks <= AHEAD;     // few chunks: all their scores, while the chunk is found
  if (CHUNKS) {
    if (ahead) load(0, chunks.n_chunks);
    c = select_own_chunk<THREADS>(chunks, pc_div(gridDim.x, heads_div), s, blockIdx.x == 0);
  } else {
    c = chunk_idx ? chunk_idx[s] : s;
  }
  if (c < 0) return;                               // no chunk for this entry: its outputs stay as they are
  int32_t* dst = out_idx + (long long)blockIdx.x * k;
  if (ahead) {
#pragma unroll
    for (int a = 1; a < AHEAD; ++a)
      if (a == c) {
#pragma unroll
        for (int j = 0; j < KPT; ++j) x[j] = x[a * KPT + j];
      }
  } else {
    load(c, 1);
  }

  const int n_valid = chunk_lens ? min(max(chunk_lens[c], 0), n) : n;   // a short chunk has fewer tokens
  if (threadIdx.x == 0) { sh_cand = 0u; sh_min = 0xffffffffu; sh_max = 0u; sh_few = 0u; }
#pragma unroll
  for (int u = 0; u < BPT; ++u) hist[threadIdx.x + THREADS * u] = 0u;
  uint32_t key[KPT];
#pragma unroll
  for (int j = 0; j < KPT; ++j) {
    const int i = first + PC_WAVE * j;
    key[j] = max(pc_order_key(x[j]), 1u);
    if (i >= n_valid || (i >= cls_lo && i < cls_hi && x[j] > lambda)) key[j] = 0u;
  }
  __syncthreads();
  // number of candidates, their smallest and largest key
  uint32_t cand = 0, lo = 0xffffffffu, hi = 0u;
#pragma unroll
  for (int j = 0; j < KPT; ++j) {
    cand += (uint32_t)__popcll(__ballot(key[j] != 0u));
    if (key[j] != 0u) { lo = min(lo, key[j]); hi = max(hi, key[j]); }
  }
#pragma unroll
  for (int off = PC_WAVE / 2; off > 0; off >>= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, off));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, off));
  }
  if (lane == 0 && cand) { atomicAdd(&sh_cand, cand); atomicMin(&sh_min, lo); atomicMax(&sh_max, hi); }
  __syncthreads();
  const int k_eff = min(k, (int)sh_cand);
  for (int i = k_eff + threadIdx.x; i < k; i += THREADS) dst[i] = -1;
  if (threadIdx.x == 0 && out_cnt) out_cnt[blockIdx.x] = k_eff;
  if (k_eff == 0) {                                // uniform over the workgroup
    if (CHUNKS && gather.k_src) select_gather<THREADS>(gather, hist, k, 0, c, g, n_kv_heads, blockIdx.x);
    return;
  }

  // The need-th largest of the keys in [lo, hi].  T ends as the k-th largest key, or one below the
  // smallest admitted key where a bin is taken whole (then no key equal to T is admitted).
  lo = sh_min; hi = sh_max;
  uint32_t need = (uint32_t)k_eff, T = lo;
  while (lo != hi) {                                 // (the bins are empty here)
    const int shift = max(0, 32 - __clz((int)(hi - lo)) - 11);
#pragma unroll
    for (int j = 0; j < KPT; ++j)
      if (key[j] >= lo && key[j] <= hi) atomicAdd(&hist[(key[j] - lo) >> shift], 1u);
    __syncthreads();
    // keys in higher bins, by a suffix sum: a thread's BPT bins, the wavefront, the wavefronts above
    uint32_t h[BPT], sum = 0;
#pragma unroll
    for (int u = 0; u < BPT; ++u) { h[u] = hist[BPT * threadIdx.x + u]; sum += h[u]; }
    uint32_t suf = sum;
#pragma unroll
    for (int off = 1; off < PC_WAVE; off <<= 1) {
      const uint32_t up = (uint32_t)__shfl_down((int)suf, off);
      if (lane + off < PC_WAVE) suf += up;
    }
    if (lane == 0) wave_tot[wave] = suf;
    __syncthreads();
    uint32_t above = suf - sum;
#pragma unroll
    for (int w = 0; w < WAVES; ++w) above += w > wave ? wave_tot[w] : 0u;
#pragma unroll
    for (int u = BPT - 1; u >= 0; --u) {
      if (h[u] > 0 && above < need && above + h[u] >= need) {
        sh_bin = (uint32_t)(BPT * threadIdx.x + u); sh_need = need - above; sh_in_bin = h[u];
      }
      above += h[u];
    }
    __syncthreads();
    need = sh_need;
    lo += sh_bin << shift;
    T = lo;
    if (need == sh_in_bin) { T = lo - 1u; break; }             // every key of the bin is admitted
    if (shift == 0) break;                                     // the bin is one key value
    hi = min(hi, lo + ((1u << shift) - 1u));
    if (sh_in_bin <= PC_SEL_FEW) {                             // the bin's keys by counting (hist is read no more)
      const uint32_t m = sh_in_bin;
#pragma unroll
      for (int j = 0; j < KPT; ++j)
        if (key[j] >= lo && key[j] <= hi) hist[atomicAdd(&sh_few, 1u)] = key[j];
      __syncthreads();
      if (threadIdx.x < m) {
        const uint32_t mine = hist[threadIdx.x];
        uint32_t gt = 0, ge = 0;
#pragma unroll 8
        for (uint32_t i = 0; i < m; ++i) { gt += hist[i] > mine; ge += hist[i] >= mine; }
        if (gt < need && ge >= need) sh_bin = mine;            // one key value: every writer has the same
      }
      __syncthreads();
      T = sh_bin;
      break;
    }
#pragma unroll
    for (int u = 0; u < BPT; ++u) hist[threadIdx.x + THREADS * u] = 0u;
    __syncthreads();
  }

  uint32_t cnt_gt = 0, cnt_eq = 0;
#pragma unroll
  for (int j = 0; j < KPT; ++j) {
    cnt_gt += (uint32_t)__popcll(__ballot(key[j] > T));
    cnt_eq += (uint32_t)__popcll(__ballot(key[j] == T));
  }
  if (lane == 0) { wave_gt[wave] = cnt_gt; wave_eq[wave] = cnt_eq; }
  __syncthreads();
  uint32_t base_gt = 0, base_eq = 0, total_gt = 0;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    const uint32_t x = wave_gt[w];
    total_gt += x;
    if (w < wave) { base_gt += x; base_eq += wave_eq[w]; }
  }
  // (behind the barrier above hist is free: the selected indices for the gather)
  const uint32_t need_eq = (uint32_t)k_eff - total_gt;      // how many keys equal to T are admitted

  const unsigned long long below = (lane == 0) ? 0ull : (~0ull >> (64 - lane));
#pragma unroll
  for (int j = 0; j < KPT; ++j) {
    const bool gt = key[j] > T, eq = key[j] == T;
    const unsigned long long bg = __ballot(gt), be = __ballot(eq);
    const uint32_t gt_before = base_gt + (uint32_t)__popcll(bg & below);
    const uint32_t eq_before = base_eq + (uint32_t)__popcll(be & below);
    if (gt || (eq && eq_before < need_eq)) {
      const uint32_t at = gt_before + min(eq_before, need_eq);
      dst[at] = first + PC_WAVE * j;
      if (CHUNKS && gather.k_src) hist[at] = (uint32_t)(first + PC_WAVE * j);
    }
    base_gt += (uint32_t)__popcll(bg);
    base_eq += (uint32_t)__popcll(be);
  }
  if (CHUNKS && gather.k_src) {
    __syncthreads();
    select_gather<THREADS>(gather, hist, k, k_eff, c, g, n_kv_heads, blockIdx.x);
  }
}

template <bool CHUNKS>
static int launch_tokens(const float* tok_score, const int32_t* chunk_idx, int n_sel, int n_kv_heads, int chunk_len,
                         int k, float lambda, int cls_lo, int cls_hi, const int32_t* chunk_lens, int32_t* out_idx,
                         int32_t* out_cnt, const PcSelectChunks& chunks, const PcSelectGather& gather, hipStream_t st) {
  PcProfScope prof(PC_KERNEL_SELECT_TOKENS, st);
  // key slots per thread: the smallest power of two that holds the chunk (at most 32768 tokens), up
  // to 8 with 512 threads, whose barriers are cheaper
#define PC_SEL_LAUNCH(KPT, THREADS)                                                                             \
  hipLaunchKernelGGL((select_tokens_kernel<KPT, THREADS, CHUNKS>), dim3(n_sel * n_kv_heads), dim3(THREADS), 0,   \
                     st, tok_score, chunk_idx, n_kv_heads, pc_div_by(n_kv_heads), chunk_len, k, lambda, cls_lo, cls_hi,                \
                     chunk_lens, out_idx, out_cnt, chunks, gather)
  if (chunk_len <= 512) PC_SEL_LAUNCH(1, 512);
  else if (chunk_len <= 1024) PC_SEL_LAUNCH(2, 512);
  else if (chunk_len <= 2048) PC_SEL_LAUNCH(4, 512);
  else if (chunk_len <= 4096) PC_SEL_LAUNCH(8, 512);
  else if (chunk_len <= 8192) PC_SEL_LAUNCH(8, 1024);
  else if (chunk_len <= 16384) PC_SEL_LAUNCH(16, 1024);
  else PC_SEL_LAUNCH(32, 1024);
#undef PC_SEL_LAUNCH
  PC_LAUNCH_CHECK();
  return PC_OK;
}

int pc_launch_select_tokens(const float* tok_score, const int32_t* chunk_idx, int n_sel,
                            int n_kv_heads, int chunk_len, int k, float lambda, int cls_lo,
                            int cls_hi, const int32_t* chunk_lens, int32_t* out_idx,
                            int32_t* out_cnt, hipStream_t st) {
  return launch_tokens<false>(tok_score, chunk_idx, n_sel, n_kv_heads, chunk_len, k, lambda, cls_lo, cls_hi, chunk_lens,
                              out_idx, out_cnt, PcSelectChunks{}, PcSelectGather{}, st);
}

bool pc_select_gather_fits(int k, int head_dim) { return 4LL * head_dim * k <= PC_SEL_GATHER; }
bool pc_select_layer_fits(int n_chunks, int per_chunk, bool gather) {
  return n_chunks <= PC_SEL_CHUNKS && per_chunk <= PC_SEL_BLOCKS &&
         n_chunks * (per_chunk + PC_SEL_CHUNK_COST) <= (gather ? PC_SEL_COST_GATHER : PC_SEL_COST);
}
int pc_launch_select_layer(const PcChunkSum& sum, int n_chunks, int n_sel, const float* tok_score, int n_kv_heads, int chunk_len,
                           int k, float lambda, int cls_lo, int cls_hi, const int32_t* chunk_lens, int32_t* chunk_idx,
                           float* chunk_top, int32_t* out_idx, int32_t* out_cnt, const void* k_src, const void* v_src, int rows,
                           int head_dim, void* kc, void* vc, hipStream_t st) {
  PcSelectGather gather = {};
  if (pc_select_gather_fits(k, head_dim))
    gather = PcSelectGather{(const uint4*)k_src, (const uint4*)v_src, (uint4*)kc, (uint4*)vc, rows, head_dim / 8};
  return launch_tokens<true>(tok_score, nullptr, n_sel, n_kv_heads, chunk_len, k, lambda, cls_lo, cls_hi, chunk_lens, out_idx,
                             out_cnt, PcSelectChunks{sum, n_chunks, chunk_idx, chunk_top}, gather, st);
}
