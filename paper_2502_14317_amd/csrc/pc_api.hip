// C ABI of the ParallelComp library: argument validation, workspace carving, kernel dispatch.
// Every host-visible argument is checked before any GPU work is enqueued.
#include "decode_core.h"
#include <math.h>
#include <mutex>

static thread_local int g_last_hip_error = 0;
void pc_set_hip_error(int err) { g_last_hip_error = err; }

extern "C" int pc_last_hip_error(void) { return g_last_hip_error; }

extern "C" const char* pc_version(void) { return "parallelcomp-gfx950 0.1"; }

extern "C" const char* pc_status_string(int status) {
  switch (status) {
    case PC_OK: return "PC_OK";
    case PC_ERR_NULL: return "PC_ERR_NULL: a required pointer is NULL";
    case PC_ERR_SHAPE: return "PC_ERR_SHAPE: a size is out of range or inconsistent";
    case PC_ERR_WORKSPACE: return "PC_ERR_WORKSPACE: workspace missing, misaligned or too small";
    case PC_ERR_HIP: return "PC_ERR_HIP: a HIP call failed (see pc_last_hip_error)";
    case PC_ERR_UNSUPPORTED: return "PC_ERR_UNSUPPORTED: no kernel for this request";
    default: return "unknown pc_status";
  }
}

// ---------------------------------------------------------------------------- profiling
#define PC_PROF_MAX 4096
static bool g_prof_on = false;
static int g_prof_only = -1;          // kernel id to record, -1 = every kernel
static int g_prof_n = 0;
static int g_prof_created = 0;
static hipEvent_t g_prof_ev[PC_PROF_MAX][2];
static int g_prof_id[PC_PROF_MAX];

PcProfScope::PcProfScope(int kernel_id, hipStream_t stream) : slot(-1), st(stream) {
  if (!g_prof_on || g_prof_n >= PC_PROF_MAX) return;
  if (g_prof_only >= 0 && kernel_id != g_prof_only) return;
  if (g_prof_n >= g_prof_created) {
    if (hipEventCreate(&g_prof_ev[g_prof_n][0]) != hipSuccess) return;
    if (hipEventCreate(&g_prof_ev[g_prof_n][1]) != hipSuccess) return;
    g_prof_created = g_prof_n + 1;
  }
  slot = g_prof_n++;
  g_prof_id[slot] = kernel_id;
  (void)hipEventRecord(g_prof_ev[slot][0], st);
}
PcProfScope::~PcProfScope() {
  if (slot >= 0) (void)hipEventRecord(g_prof_ev[slot][1], st);
}

extern "C" int pc_profile_begin(void) { g_prof_n = 0; g_prof_only = -1; g_prof_on = true; return PC_OK; }
extern "C" int pc_profile_begin_kernel(int kernel_id) {
  if (kernel_id < 0 || kernel_id >= PC_KERNEL_COUNT) return PC_ERR_SHAPE;
  g_prof_n = 0; g_prof_only = kernel_id; g_prof_on = true;
  return PC_OK;
}
extern "C" int pc_profile_end(void) { g_prof_on = false; return PC_OK; }
extern "C" int pc_profile_count(void) { return g_prof_n; }
extern "C" int pc_profile_get(int i, int* kernel_id, float* ms) {
  if (!kernel_id || !ms) return PC_ERR_NULL;
  if (i < 0 || i >= g_prof_n) return PC_ERR_SHAPE;
  PC_HIP_TRY(hipEventSynchronize(g_prof_ev[i][1]));
  PC_HIP_TRY(hipEventElapsedTime(ms, g_prof_ev[i][0], g_prof_ev[i][1]));
  *kernel_id = g_prof_id[i];
  return PC_OK;
}
extern "C" const char* pc_kernel_name(int id) {
  static const char* names[PC_KERNEL_COUNT] = {
      "layer_prep_kernel", "kv_prepass_kernel", "flash_fwd_kernel", "scores_kernel<1>",
      "scores_kernel<2>", "chunk_score_kernel", "select_chunks_kernel", "select_tokens_kernel",
      "gather_kv_kernel", "rope_q_kernel", "decode_attn_kernel", "merge_kernel",
      "self_info_rows_kernel", "kv_append_kernel", "scores_lse_kernel", "kv_quantize_fp8_kernel",
      "decode_attn_fp8_kernel", "scores_kernel<1>+kv_prepass", "chunk_queue_kernel",
      "fp8_images_kernel", "fp8_rows_kernel"};
  return (id >= 0 && id < PC_KERNEL_COUNT) ? names[id] : "unknown";
}

static const size_t kAlign = 256;

static int check_shape(const pc_shape* s) {
  if (!s) return PC_ERR_NULL;
  if (s->n_chunks < 1 || s->chunk_len < 1 || s->query_len < 0) return PC_ERR_SHAPE;
  if (s->n_kv_heads < 1 || s->n_q_heads < 1 || s->n_q_heads % s->n_kv_heads != 0) return PC_ERR_SHAPE;
  if (s->head_dim != 64 && s->head_dim != 128) return PC_ERR_SHAPE;
  const long long L = (long long)s->chunk_len + s->query_len;
  if (L > (1 << 20) || s->n_chunks > (1 << 20) || s->n_q_heads > 1024) return PC_ERR_SHAPE;
  // kernels index (chunk, head, row) tuples and workgroups with 32-bit integers
  if ((long long)s->n_chunks * s->n_q_heads * ((L + 127) / 128) > 0x7fffffffLL / 8) return PC_ERR_SHAPE;
  if ((long long)s->n_chunks * L * s->n_q_heads > 0x7fffffffLL) return PC_ERR_SHAPE;
  if (!(s->rope_base > 1.0f) || !isfinite(s->rope_base)) return PC_ERR_SHAPE;
  if (!(s->softmax_scale >= 0.0f) || !isfinite(s->softmax_scale)) return PC_ERR_SHAPE;
  return PC_OK;
}

// The voting rows are the last w_obs rows of a sequence.  With ragged chunks a sequence may be
// as short as the query block alone, so the window must then fit the query block (Eq. 6 sums
// over query rows only); with full chunks it may reach into the context rows.
static int check_obs(const pc_shape* s, bool ragged) {
  const int L = s->chunk_len + s->query_len;
  if (s->obs_window < 1 || s->obs_window > (ragged ? s->query_len : L)) return PC_ERR_SHAPE;
  return PC_OK;
}

static float eff_scale(float scale, int head_dim) {
  return scale > 0.f ? scale : 1.0f / sqrtf((float)head_dim);
}

struct PrefillWs {
  size_t table, q_table, v_img, k_img, ml, total;
  int Lp;
};

static PrefillWs prefill_ws_layout(const pc_shape* s) {
  PrefillWs w;
  const size_t L = (size_t)s->chunk_len + s->query_len;
  w.Lp = (int)((L + 63) / 64 * 64);
  size_t off = 0;
  w.table = off; off = pc_align_up(off + L * (s->head_dim / 2) * sizeof(float2), kAlign);
  w.q_table = off; off = pc_align_up(off + (L + 127) / 128 * 128 * (s->head_dim / 2) * sizeof(float2), kAlign);
  const size_t img_bytes = (size_t)s->n_chunks * s->n_kv_heads * s->head_dim * w.Lp * 2;   // tile images
  w.v_img = off; off = pc_align_up(off + img_bytes, kAlign);
  w.k_img = off; off = pc_align_up(off + img_bytes, kAlign);
  w.ml = off;    off = pc_align_up(off + pc_scores_ws_bytes(s), kAlign);
  w.total = off;
  return w;
}

extern "C" size_t pc_chunk_prefill_workspace_bytes(const pc_shape* s) {
  if (check_shape(s) != PC_OK) return 0;
  pc_shape t = *s;
  // a call without scores ignores the window: size for any window the call could accept
  if (t.obs_window < 1) t.obs_window = 1;
  if (t.obs_window > t.chunk_len + t.query_len) t.obs_window = t.chunk_len + t.query_len;
  return prefill_ws_layout(&t).total;
}

extern "C" size_t pc_chunk_query_scores_workspace_bytes(const pc_shape* s) {
  if (check_shape(s) != PC_OK || check_obs(s, false) != PC_OK) return 0;
  const size_t L = (size_t)s->chunk_len + s->query_len;
  return pc_align_up(L * (s->head_dim / 2) * sizeof(float2), kAlign) +
         pc_align_up(pc_scores_ws_bytes(s), kAlign);
}

// The local attention over the tile images in the workspace
static PcFlashArgs local_flash_args(const pc_shape* s, const void* q, const int32_t* chunk_lens, void* o, float* lse,
                                    char* base, const PrefillWs& w) {
  PcFlashArgs a = {};
  a.q = q; a.k_img = base + w.k_img; a.v_img = base + w.v_img; a.table = (const float2*)(base + w.q_table); a.o = o; a.lse = lse;
  a.img_seq_stride = (long long)s->n_kv_heads * (w.Lp / 64);
  a.img_head_stride = w.Lp / 64;
  a.n_seq = s->n_chunks; a.n_rows = s->chunk_len + s->query_len; a.table_rows = (a.n_rows + 127) / 128 * 128;
  a.n_q_heads = s->n_q_heads; a.n_kv_heads = s->n_kv_heads; a.head_dim = s->head_dim;
  a.seq_ctx = chunk_lens; a.seq_add = s->query_len;
  a.scale = eff_scale(s->softmax_scale, s->head_dim);
  return a;
}

// What pc_chunk_prefill_attn asks of its tensors
static int check_prefill_args(const void* q, const void* k, const void* v, const void* o, const float* lse,
                              const void* k_rope, const float* tok_score, const float* chunk_score) {
  if (!q || !k || !v || !o || !lse) return PC_ERR_NULL;
  if (chunk_score && !tok_score) return PC_ERR_NULL;
  // every kernel moves these tensors with 16-byte loads and stores
  if (!pc_aligned(q, 16) || !pc_aligned(k, 16) || !pc_aligned(v, 16) || !pc_aligned(o, 16) ||
      !pc_aligned(k_rope, 16))
    return PC_ERR_SHAPE;
  return PC_OK;
}

extern "C" int pc_chunk_prefill_attn(const pc_shape* s, const void* q, const void* k, const void* v,
                                     const int32_t* chunk_lens, void* o, float* lse, void* k_rope, float* tok_score,
                                     float* chunk_score, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_shape(s);
  if (rc != PC_OK) return rc;
  rc = check_prefill_args(q, k, v, o, lse, k_rope, tok_score, chunk_score);
  if (rc != PC_OK) return rc;
  if (tok_score) {
    rc = check_obs(s, chunk_lens != nullptr);
    if (rc != PC_OK) return rc;
  }
  pc_shape t = *s;
  if (!tok_score) t.obs_window = 1;
  const PrefillWs w = prefill_ws_layout(&t);
  if (!ws || !pc_aligned(ws, kAlign) || ws_bytes < w.total) return PC_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  char* base = (char*)ws;
  float2* table = (float2*)(base + w.table);
  void* v_img = base + w.v_img;
  void* k_img = base + w.k_img;
  void* kr = k_rope;                                       // nullable: then only the images are written
  const int L = s->chunk_len + s->query_len, D = s->head_dim;

  PcPrepArgs prep = {};
  prep.table = table; prep.n_pos = L; prep.rope = pc_rope_factors(s->rope_base, D);
  prep.q_table = (float2*)(base + w.q_table); prep.q_scale = (double)(eff_scale(s->softmax_scale, D) * 1.4426950408889634f);
  if (tok_score) prep.scores = pc_scores_queries(s, q, chunk_lens, base + w.ml);
  rc = pc_launch_prep(prep, D, st);
  if (rc != PC_OK) return rc;
  PcChunkSum sum = {};
  if (tok_score) {
    // the first score pass reads and rotates every key anyway: it also writes the rotated keys
    // and the tile images (the keys are read from memory once for both jobs)
    const PcPrepassOut pre = {v, kr, k_img, v_img, w.Lp};
    rc = pc_launch_scores(s, k, chunk_lens, table, base + w.ml, tok_score, chunk_score, &pre, &sum, st);
  } else {
    rc = pc_launch_kv_prepass(k, v, table, kr, k_img, v_img, s->n_chunks, L, w.Lp, s->n_kv_heads, D, st);
  }
  if (rc != PC_OK) return rc;
  PcFlashArgs a = local_flash_args(s, q, chunk_lens, o, lse, base, w);
  a.sum = sum;
  return pc_launch_flash(a, st);
}

extern "C" int pc_chunk_query_scores(const pc_shape* s, const void* q, const void* k,
                                     const int32_t* chunk_lens, float* tok_score, float* chunk_score, void* ws,
                                     size_t ws_bytes, void* stream) {
  int rc = check_shape(s);
  if (rc != PC_OK) return rc;
  rc = check_obs(s, chunk_lens != nullptr);
  if (rc != PC_OK) return rc;
  if (!q || !k || !tok_score) return PC_ERR_NULL;
  if (!pc_aligned(q, 16) || !pc_aligned(k, 16)) return PC_ERR_SHAPE;
  const size_t need = pc_chunk_query_scores_workspace_bytes(s);
  if (!ws || !pc_aligned(ws, kAlign) || ws_bytes < need) return PC_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  const int L = s->chunk_len + s->query_len;
  float2* table = (float2*)ws;
  void* ml = (char*)ws + pc_align_up((size_t)L * (s->head_dim / 2) * sizeof(float2), kAlign);
  PcPrepArgs prep = {};
  prep.table = table; prep.n_pos = L; prep.rope = pc_rope_factors(s->rope_base, s->head_dim);
  prep.scores = pc_scores_queries(s, q, chunk_lens, ml);
  rc = pc_launch_prep(prep, s->head_dim, st);
  if (rc != PC_OK) return rc;
  return pc_launch_scores(s, k, chunk_lens, table, ml, tok_score, chunk_score, nullptr, nullptr, st);
}

static int check_append(const void* k_new, const void* v_new, int batch, int n_new, int n_seg, int seg, int k_t,
                        int n_kv_heads, int head_dim, int pos0, float rope_base, const void* kc, const void* vc,
                        const int32_t* seg_len) {
  if (!k_new || !v_new || !kc || !vc || !seg_len) return PC_ERR_NULL;
  if (batch < 0 || n_new < 0 || n_seg < 1 || seg < 0 || seg >= n_seg || k_t < 1 || n_kv_heads < 1)
    return PC_ERR_SHAPE;
  if (head_dim != 64 && head_dim != 128) return PC_ERR_SHAPE;
  if (pos0 >= 0 && (!(rope_base > 1.0f) || !isfinite(rope_base))) return PC_ERR_SHAPE;
  if (!pc_aligned(k_new, 2) || !pc_aligned(v_new, 2) || !pc_aligned(kc, 2) || !pc_aligned(vc, 2) ||
      !pc_aligned(seg_len, 4))
    return PC_ERR_SHAPE;
  return PC_OK;
}

extern "C" int pc_kv_append(const void* k_new, const void* v_new, int32_t batch, int32_t n_new,
                            int32_t n_seg, int32_t seg, int32_t k_t, int32_t n_kv_heads,
                            int32_t head_dim, int32_t pos0, float rope_base, void* kc, void* vc,
                            int32_t* seg_len, int32_t seg_len_per_head, void* stream) {
  const int rc = check_append(k_new, v_new, batch, n_new, n_seg, seg, k_t, n_kv_heads, head_dim, pos0, rope_base,
                              kc, vc, seg_len);
  if (rc != PC_OK) return rc;
  if (batch == 0 || n_new == 0) return PC_OK;
  return pc_launch_kv_append(k_new, v_new, batch, n_new, n_seg, seg, k_t, n_kv_heads, head_dim,
                             pos0, rope_base, kc, vc, seg_len, seg_len_per_head != 0,
                             (hipStream_t)stream);
}

// ---------------------------------------------------------------------------- 8-bit cache
extern "C" int pc_kv_quantize_fp8(const void* kc, const void* vc, const int32_t* seg_len,
                                  int32_t seg_len_per_head, int32_t batch, int32_t n_seg,
                                  int32_t k_t, int32_t n_kv_heads, int32_t head_dim, void* k8,
                                  void* v8, float* k_scale, float* v_scale, void* stream) {
  if (batch < 0 || n_seg < 0 || k_t < 1 || n_kv_heads < 1) return PC_ERR_SHAPE;
  if (head_dim != 64 && head_dim != 128) return PC_ERR_SHAPE;
  if (seg_len_per_head != 0 && seg_len_per_head != 1) return PC_ERR_SHAPE;
  if (batch == 0 || n_seg == 0) return PC_OK;            // nothing to quantise
  if (!kc || !vc || !k8 || !v8 || !k_scale || !v_scale) return PC_ERR_NULL;
  if (!pc_aligned(kc, 16) || !pc_aligned(vc, 16) || !pc_aligned(k8, 16) || !pc_aligned(v8, 16))
    return PC_ERR_SHAPE;
  return pc_launch_kv_quantize_fp8(kc, vc, seg_len, seg_len_per_head,
                                   (long long)batch * n_seg * n_kv_heads, n_kv_heads, k_t, head_dim,
                                   nullptr, nullptr, k8, v8, k_scale, v_scale, (hipStream_t)stream);
}

extern "C" int pc_kv_quantize_fp8_amax(const void* kc, const void* vc, const float* k_amax,
                                       const float* v_amax, const int32_t* seg_len,
                                       int32_t seg_len_per_head, int32_t batch, int32_t n_seg,
                                       int32_t k_t, int32_t n_kv_heads, int32_t head_dim, void* k8,
                                       void* v8, float* k_scale, float* v_scale, void* stream) {
  if (batch < 0 || n_seg < 0 || k_t < 1 || n_kv_heads < 1) return PC_ERR_SHAPE;
  if (head_dim != 64 && head_dim != 128) return PC_ERR_SHAPE;
  if (seg_len_per_head != 0 && seg_len_per_head != 1) return PC_ERR_SHAPE;
  if (batch == 0 || n_seg == 0) return PC_OK;
  if (!kc || !vc || !k_amax || !v_amax || !k8 || !v8 || !k_scale || !v_scale) return PC_ERR_NULL;
  if (!pc_aligned(kc, 16) || !pc_aligned(vc, 16) || !pc_aligned(k8, 16) || !pc_aligned(v8, 16))
    return PC_ERR_SHAPE;
  return pc_launch_kv_quantize_fp8(kc, vc, seg_len, seg_len_per_head,
                                   (long long)batch * n_seg * n_kv_heads, n_kv_heads, k_t, head_dim,
                                   k_amax, v_amax, k8, v8, k_scale, v_scale, (hipStream_t)stream);
}

// Few query rows: rotated by the split-KV kernel itself, behind its first key loads, which saves a launch, or by
// rope_q_kernel first: where the merge needs the rows too (self segment), and beyond 512 workgroups (of the segments; an
// 8-bit cache's tail is not counted).  That line comes from a kernel that computed its angles with library calls in
// front of its loads, round after round.  For the present one the launch in front is the slower side beyond it too:
// kernel itself / first (us, 16-bit and 8-bit cache), 33 sequences of 8 x 1024 keys, 64 / 8 heads 202 / 205 and 100 / 103,
// 65 of 32 / 8 358 / 361 and 184 / 187, 300 of 16 / 1 225 / 228 and 120 / 123, 600 of 64 keys, 4 / 1 heads of 64 values
// 13.3 / 15.8 and 12.3 / 14.5, 1000 of 128 keys, 64 / 8 heads 221 / 228 and 174 / 181.  It stands because
// tests/test_gpu_decode_rotation_first.py expects the launch.
#define PC_DEC_ROT_WGS 512
static bool rotate_first(int has_self, long long workgroups) { return has_self || workgroups > PC_DEC_ROT_WGS; }

// A decoding step's part in the split-KV launch (k_new == nullptr: none).  kernel_pos < 0 at pos >= 0: the query
// was rotated in front and the merge has it; otherwise the launch leaves the rotated row.
static PcDecodeAppend step_append(const void* k_new, const void* v_new, int pos, int kernel_pos, void* q_rot, int32_t* self_row) {
  PcDecodeAppend a = {};
  if (!k_new) return a;
  a.k_new = (const uint16_t*)k_new; a.v_new = (const uint16_t*)v_new; a.pos = pos; a.self_row = self_row;
  if (kernel_pos >= 0) a.q_rot = (uint16_t*)q_rot;
  return a;
}

// 64-key tiles of n segments of k_t keys
static long long key_tiles(int n, int k_t) { return (long long)n * ((k_t + 63) / 64); }

// Parts the tile path's keys are cut into, and how many partial rows the workspace has room for.  The
// number of parts falls where there are more rows to fill the chip, the room only ever rises.
static int tile_parts(int batch, int n_q, long long seg_tiles, int n_q_heads, int n_kv_heads, int D, int has_self,
                      size_t& room) {
  const long long tiles = seg_tiles + key_tiles(has_self, n_q);
  room = pc_flash_part_rows((size_t)batch * n_q * n_q_heads, tiles, has_self);
  return pc_flash_parts(batch, n_q, n_q_heads, n_kv_heads, D, tiles);
}

// Limits of the tile path beyond those of the shape checks.  The tile kernel steps through the self
// segment by 64 rows of all KV heads and addresses a tile with 32-bit byte offsets: up to 65535 heads
// (63 x 65535 x 256 bytes) keep both in range.  65535 is also the most 64-key tiles of a segment or
// tail it takes.
static int check_tile_limits(int n_seg, int k_t, int tail_cap, int n_kv_heads, int has_self) {
  if (has_self && n_kv_heads > 65535) return PC_ERR_SHAPE;
  if (n_seg > 0 && key_tiles(1, k_t) > 65535) return PC_ERR_SHAPE;
  if (key_tiles(1, tail_cap) > 65535) return PC_ERR_SHAPE;
  return PC_OK;
}

struct Par8Ws {
  size_t q_rot, part_o, part_lse, total;                   // q_rot: the rotated query rows
  size_t k_img[3], v_img[3];                               // tile images of segments, tail, self segment
  int n_parts;
  PcDecodeSplit split;                                     // small
  bool small;
};

static Par8Ws par8_ws_layout(int batch, int n_q, int n_seg, int k_t, int tail_cap, int n_q_heads,
                             int n_kv_heads, int D, int has_self) {
  Par8Ws w;
  const size_t rows = (size_t)batch * n_q * n_q_heads;
  size_t part_rows = 0;
  w.small = (long long)n_q * (n_q_heads / n_kv_heads) <= 16;
  if (w.small) {
    w.split = pc_decode_split(k_t, n_seg, 1, tail_cap, D, (long long)batch * n_kv_heads);
    w.n_parts = w.split.parts + w.split.tail_parts;
  } else {
    w.split = PcDecodeSplit{};
    w.n_parts = tile_parts(batch, n_q, key_tiles(n_seg, k_t) + key_tiles(1, tail_cap), n_q_heads, n_kv_heads, D, has_self, part_rows);
  }
  size_t off = 0;
  w.q_rot = off;    off = pc_align_up(off + rows * D * 2, kAlign);
  if (w.small) part_rows = rows * (w.split.room + w.split.tail_room);
  w.part_o = off;   off = pc_align_up(off + part_rows * D * sizeof(float), kAlign);
  w.part_lse = off; off = pc_align_up(off + part_rows * sizeof(float), kAlign);
  if (!w.small) {
    const size_t head_tiles[3] = {(size_t)n_seg * key_tiles(1, k_t), (size_t)key_tiles(1, tail_cap), has_self ? (size_t)key_tiles(1, n_q) : 0};
    for (int i = 0; i < 3; ++i) {
      const size_t bytes = (size_t)batch * n_kv_heads * head_tiles[i] * 64 * D * 2;
      w.k_img[i] = off; off = pc_align_up(off + bytes, kAlign);
      w.v_img[i] = off; off = pc_align_up(off + bytes, kAlign);
    }
  }
  w.total = off;
  return w;
}

static int check_par8(int batch, int n_q, int n_seg, int k_t, int tail_cap, int n_q_heads,
                      int n_kv_heads, int D) {
  if (batch < 1 || n_q < 1 || n_seg < 0 || k_t < 1 || tail_cap < 0) return PC_ERR_SHAPE;
  if (n_kv_heads < 1 || n_q_heads < 1 || n_q_heads % n_kv_heads != 0) return PC_ERR_SHAPE;
  if (D != 64 && D != 128) return PC_ERR_SHAPE;
  if (k_t > (1 << 24) || tail_cap > (1 << 24) || n_seg > (1 << 20) || batch > (1 << 20) || n_q > (1 << 20))
    return PC_ERR_SHAPE;
  const long long parts = (long long)n_seg + 2;
  if ((long long)batch * parts * n_kv_heads > 0x7fffffffLL / 64) return PC_ERR_SHAPE;
  if ((long long)batch * parts * n_q_heads * ((n_q + 127) / 128) > 0x7fffffffLL / 8) return PC_ERR_SHAPE;
  if ((long long)batch * n_q * n_q_heads > 0x7fffffffLL / 64) return PC_ERR_SHAPE;
  return PC_OK;
}

static int parallel_attn_fp8_tiles(const void* q, const void* k8, const void* v8, const float* k_scale,
                                   const float* v_scale, const int32_t* seg_len, int seg_len_per_head,
                                   const void* k_tail, const void* v_tail, const int32_t* tail_len,
                                   int tail_cap, const void* k_self, const void* v_self, int batch,
                                   int n_q, int n_seg, int k_t, int n_q_heads, int n_kv_heads, int D,
                                   int q_pos0, float rope_base, float scale, void* out, float* lse_out,
                                   const Par8Ws& w, char* base, hipStream_t st);

static int check_par8_args(const void* q, const void* k8, const void* v8, const float* k_scale, const float* v_scale,
                           int seg_len_per_head, const void* k_tail, const void* v_tail, const int32_t* tail_len,
                           int tail_cap, const void* k_self, const void* v_self, int batch, int n_q, int n_seg, int k_t,
                           int n_q_heads, int n_kv_heads, int head_dim, int q_pos0, float rope_base,
                           float softmax_scale, const void* out) {
  const int rc = check_par8(batch, n_q, n_seg, k_t, tail_cap, n_q_heads, n_kv_heads, head_dim);
  if (rc != PC_OK) return rc;
  if (!q || !out) return PC_ERR_NULL;
  if (n_seg > 0 && (!k8 || !v8 || !k_scale || !v_scale)) return PC_ERR_NULL;
  if (tail_cap > 0 && (!k_tail || !v_tail || !tail_len)) return PC_ERR_NULL;
  if ((k_self == nullptr) != (v_self == nullptr)) return PC_ERR_NULL;
  const int has_self = k_self != nullptr;
  if (n_seg == 0 && tail_cap == 0 && !has_self) return PC_ERR_SHAPE;
  if (seg_len_per_head != 0 && seg_len_per_head != 1) return PC_ERR_SHAPE;
  if (q_pos0 >= 0 && (!(rope_base > 1.0f) || !isfinite(rope_base))) return PC_ERR_SHAPE;
  if (!(softmax_scale >= 0.0f) || !isfinite(softmax_scale)) return PC_ERR_SHAPE;
  if (n_seg > 0 && (!pc_aligned(k8, 16) || !pc_aligned(v8, 16))) return PC_ERR_SHAPE;
  if (!pc_aligned(q, 16) || !pc_aligned(out, 16) || !pc_aligned(k_tail, 16) || !pc_aligned(v_tail, 16) ||
      !pc_aligned(k_self, 16) || !pc_aligned(v_self, 16))
    return PC_ERR_SHAPE;
  return PC_OK;
}

// The few-row path over the 8-bit segments and the tail.  k_new, v_new: a decoding step, the tail's next row
// (self_row: [batch, H_kv] scratch); tail_len then counts it.
static int par8_small_run(const void* q, const void* k8, const void* v8, const float* k_scale, const float* v_scale,
                          const int32_t* seg_len, int seg_len_per_head, const void* k_tail, const void* v_tail,
                          const int32_t* tail_len, int tail_cap, const void* k_self, const void* v_self, int batch,
                          int n_q, int n_seg, int k_t, int n_q_heads, int n_kv_heads, int D, int q_pos0,
                          float rope_base, float scale, void* out, float* lse_out, const Par8Ws& w, char* base,
                          const void* k_new, const void* v_new, int32_t* self_row, hipStream_t st) {
  const void* q_in = q;
  int pos0 = q_pos0, rc;
  if (q_pos0 >= 0 && rotate_first(k_self != nullptr, (long long)batch * n_kv_heads * w.split.parts)) {
    rc = pc_launch_rope_q(q, base + w.q_rot, batch, n_q, n_q_heads, D, q_pos0, rope_base, 1.0f, st);
    if (rc != PC_OK) return rc;
    q_in = base + w.q_rot; pos0 = -1;
  }
  float* part_o = (float*)(base + w.part_o);
  float* part_lse = (float*)(base + w.part_lse);
  const PcDecodeAppend app = step_append(k_new, v_new, q_pos0, pos0, base + w.q_rot, self_row);
  if (n_seg > 0 || tail_cap > 0) {
    rc = pc_launch_decode_fp8(q_in, pos0, rope_base, k8, v8, k_scale, v_scale, seg_len, seg_len_per_head,
                              k_tail, v_tail, tail_len, tail_cap, batch, n_q, n_seg, k_t, n_q_heads,
                              n_kv_heads, D, scale, part_o, part_lse, w.split, app, st);
    if (rc != PC_OK) return rc;
  }
  PcMergeStep step = {};
  if (k_new) step = PcMergeStep{self_row, (const uint16_t*)k_tail, (const uint16_t*)v_tail, (int32_t*)tail_len, 1, tail_cap, 0};
  // the few-row causal self segment (if any) is evaluated inside the merge
  return pc_launch_merge(part_o, part_lse, app.q_rot ? app.q_rot : q_in, k_self, v_self, step, out, lse_out, batch,
                         n_q, n_q_heads, n_kv_heads, D, w.n_parts, scale, st);
}

extern "C" size_t pc_parallel_attn_fp8_workspace_bytes(int32_t batch, int32_t n_q, int32_t n_seg,
                                                       int32_t k_t, int32_t tail_cap,
                                                       int32_t n_q_heads, int32_t n_kv_heads,
                                                       int32_t head_dim, int32_t has_self) {
  if (check_par8(batch, n_q, n_seg, k_t, tail_cap, n_q_heads, n_kv_heads, head_dim) != PC_OK) return 0;
  return par8_ws_layout(batch, n_q, n_seg, k_t, tail_cap, n_q_heads, n_kv_heads, head_dim, has_self).total;
}

extern "C" int pc_parallel_attn_fp8(const void* q, const void* k8, const void* v8,
                                    const float* k_scale, const float* v_scale,
                                    const int32_t* seg_len, int32_t seg_len_per_head,
                                    const void* k_tail, const void* v_tail, const int32_t* tail_len,
                                    int32_t tail_cap, const void* k_self, const void* v_self,
                                    int32_t batch, int32_t n_q, int32_t n_seg,
                                    int32_t k_t, int32_t n_q_heads, int32_t n_kv_heads,
                                    int32_t head_dim, int32_t q_pos0, float rope_base,
                                    float softmax_scale, void* out, float* lse_out, void* ws,
                                    size_t ws_bytes, void* stream) {
  int rc = check_par8_args(q, k8, v8, k_scale, v_scale, seg_len_per_head, k_tail, v_tail, tail_len, tail_cap, k_self,
                           v_self, batch, n_q, n_seg, k_t, n_q_heads, n_kv_heads, head_dim, q_pos0, rope_base,
                           softmax_scale, out);
  if (rc != PC_OK) return rc;
  const int has_self = k_self != nullptr;
  const int D = head_dim;
  const Par8Ws w = par8_ws_layout(batch, n_q, n_seg, k_t, tail_cap, n_q_heads, n_kv_heads, D, has_self);
  if (!ws || !pc_aligned(ws, kAlign) || ws_bytes < w.total) return PC_ERR_WORKSPACE;
  hipStream_t st = (hipStream_t)stream;
  char* base = (char*)ws;
  const float scale = eff_scale(softmax_scale, D);
  if (!w.small) {
    rc = check_tile_limits(n_seg, k_t, tail_cap, n_kv_heads, has_self);
    if (rc != PC_OK) return rc;
    return parallel_attn_fp8_tiles(q, k8, v8, k_scale, v_scale, seg_len, seg_len_per_head, k_tail, v_tail,
                                   tail_len, tail_cap, k_self, v_self, batch, n_q, n_seg, k_t, n_q_heads,
                                   n_kv_heads, D, q_pos0, rope_base, scale, out, lse_out, w, base, st);
  }
  return par8_small_run(q, k8, v8, k_scale, v_scale, seg_len, seg_len_per_head, k_tail, v_tail, tail_len, tail_cap,
                        k_self, v_self, batch, n_q, n_seg, k_t, n_q_heads, n_kv_heads, D, q_pos0, rope_base, scale,
                        out, lse_out, w, base, nullptr, nullptr, nullptr, st);
}

extern "C" int pc_chunk_self_information(const void* logits, const int32_t* targets, int32_t n_chunks,
                                         int32_t n_tokens, int32_t vocab, int32_t negate,
                                         float* token_nll, float* info, void* stream) {
  if (!logits || !targets || !token_nll || !info) return PC_ERR_NULL;
  if (n_chunks < 1 || n_tokens < 1 || vocab < 8 || vocab > (1 << 24) || vocab % 8 != 0) return PC_ERR_SHAPE;
  if ((long long)n_chunks * n_tokens > 0x7fffffffLL || !pc_aligned(logits, 16)) return PC_ERR_SHAPE;
  return pc_launch_self_info(logits, targets, n_chunks, n_tokens, vocab, negate, token_nll, info,
                             (hipStream_t)stream);
}

extern "C" int pc_select_chunks_topk(const float* chunk_score, int32_t n, int32_t k,
                                     int32_t* out_idx, float* out_score, void* stream) {
  if (!chunk_score || !out_idx) return PC_ERR_NULL;
  if (n < 1 || n > 4096 || k < 1 || k > n) return PC_ERR_SHAPE;
  return pc_launch_select_chunks(chunk_score, n, k, out_idx, out_score, (hipStream_t)stream);
}

extern "C" int pc_chunk_queue_update(const float* batch_score, int32_t n_batch, int32_t chunk_id0,
                                     int32_t capacity, int32_t* queue_id, float* queue_score,
                                     int32_t* queue_slot, int32_t* slot_src, void* stream) {
  if (!batch_score || !queue_id || !queue_score || !queue_slot || !slot_src) return PC_ERR_NULL;
  if (n_batch < 1 || n_batch > 1024 || capacity < 1 || capacity > 1024 || chunk_id0 < 0) return PC_ERR_SHAPE;
  if ((long long)chunk_id0 + n_batch > 0x7fffffffLL) return PC_ERR_SHAPE;
  return pc_launch_chunk_queue(batch_score, n_batch, chunk_id0, capacity, queue_id, queue_score,
                               queue_slot, slot_src, (hipStream_t)stream);
}

extern "C" int pc_select_tokens_topk(const float* tok_score, const int32_t* chunk_idx, int32_t n_sel,
                                     int32_t n_kv_heads, int32_t chunk_len, int32_t k,
                                     int32_t* out_idx, void* stream) {
  if (!tok_score || !out_idx) return PC_ERR_NULL;
  if (n_sel < 0 || n_kv_heads < 1 || chunk_len < 1 || chunk_len > 32768 || k < 1 || k > chunk_len)
    return PC_ERR_SHAPE;
  if ((long long)n_sel * n_kv_heads > 0x7fffffffLL) return PC_ERR_SHAPE;
  if (n_sel == 0) return PC_OK;
  return pc_launch_select_tokens(tok_score, chunk_idx, n_sel, n_kv_heads, chunk_len, k, 0.f, 0, 0,
                                 nullptr, out_idx, nullptr, (hipStream_t)stream);
}

extern "C" int pc_select_tokens_calibrated(const float* tok_score, const int32_t* chunk_idx,
                                           int32_t n_sel, int32_t n_kv_heads, int32_t chunk_len,
                                           int32_t k, float lambda, int32_t class_lo,
                                           int32_t class_hi, const int32_t* chunk_lens,
                                           int32_t* out_idx, int32_t* out_cnt, void* stream) {
  if (!tok_score || !out_idx || !out_cnt) return PC_ERR_NULL;
  if (n_sel < 0 || n_kv_heads < 1 || chunk_len < 1 || chunk_len > 32768 || k < 1 || k > chunk_len)
    return PC_ERR_SHAPE;
  if ((long long)n_sel * n_kv_heads > 0x7fffffffLL) return PC_ERR_SHAPE;
  if (class_lo < 0 || class_hi < class_lo || class_hi > chunk_len || lambda != lambda) return PC_ERR_SHAPE;
  if (n_sel == 0) return PC_OK;
  return pc_launch_select_tokens(tok_score, chunk_idx, n_sel, n_kv_heads, chunk_len, k, lambda,
                                 class_lo, class_hi, chunk_lens, out_idx, out_cnt, (hipStream_t)stream);
}

extern "C" int pc_gather_kv(const void* k_src, const void* v_src, const int32_t* chunk_idx,
                            const int32_t* tok_idx, int32_t batch, int32_t n_chunks,
                            int32_t rows_per_chunk, int32_t n_sel, int32_t n_kv_heads, int32_t k,
                            int32_t head_dim, void* k_dst, void* v_dst, void* stream) {
  if (!k_src || !v_src || !tok_idx || !k_dst || !v_dst) return PC_ERR_NULL;
  if (batch < 0 || n_chunks < 1 || rows_per_chunk < 1 || n_sel < 0 || n_kv_heads < 1 || k < 0)
    return PC_ERR_SHAPE;
  if (head_dim != 64 && head_dim != 128) return PC_ERR_SHAPE;
  if (!pc_aligned(k_src, 16) || !pc_aligned(v_src, 16) || !pc_aligned(k_dst, 16) || !pc_aligned(v_dst, 16))
    return PC_ERR_SHAPE;
  return pc_launch_gather(k_src, v_src, chunk_idx, tok_idx, batch, n_chunks, rows_per_chunk, n_sel,
                          n_kv_heads, k, head_dim, k_dst, v_dst, nullptr, nullptr, (hipStream_t)stream);
}

extern "C" int pc_gather_kv_amax(const void* k_src, const void* v_src, const int32_t* chunk_idx,
                                 const int32_t* tok_idx, int32_t batch, int32_t n_chunks,
                                 int32_t rows_per_chunk, int32_t n_sel, int32_t n_kv_heads, int32_t k,
                                 int32_t head_dim, void* k_dst, void* v_dst, float* k_amax,
                                 float* v_amax, void* stream) {
  if (!k_src || !v_src || !tok_idx || !k_dst || !v_dst || !k_amax || !v_amax) return PC_ERR_NULL;
  if (batch < 0 || n_chunks < 1 || rows_per_chunk < 1 || n_sel < 0 || n_kv_heads < 1 || k < 1)
    return PC_ERR_SHAPE;
  if (head_dim != 64 && head_dim != 128) return PC_ERR_SHAPE;
  if (!pc_aligned(k_src, 16) || !pc_aligned(v_src, 16) || !pc_aligned(k_dst, 16) || !pc_aligned(v_dst, 16))
    return PC_ERR_SHAPE;
  return pc_launch_gather(k_src, v_src, chunk_idx, tok_idx, batch, n_chunks, rows_per_chunk, n_sel,
                          n_kv_heads, k, head_dim, k_dst, v_dst, k_amax, v_amax, (hipStream_t)stream);
}

// ---------------------------------------------------------------------------- parallel attention
struct ParWs {
  size_t q_rot, part_o, part_lse, total;       // q_rot: the rotated query rows
  int n_parts;
  bool small;
};

static ParWs par_ws_layout(int batch, int n_q, int n_seg, int k_t, int n_q_heads, int n_kv_heads,
                           int D, int has_self) {
  ParWs w;
  const size_t rows = (size_t)batch * n_q * n_q_heads;
  size_t part_rows = 0;
  const int G = n_q_heads / n_kv_heads;
  w.small = (long long)n_q * G <= 16;
  if (w.small) {
    const PcDecodeSplit split = pc_decode_split(k_t, n_seg, 2, 0, D, (long long)batch * n_kv_heads);
    w.n_parts = split.parts;
    part_rows = rows * split.room;
  } else {
    w.n_parts = tile_parts(batch, n_q, key_tiles(n_seg, k_t), n_q_heads, n_kv_heads, D, has_self, part_rows);
  }
  size_t off = 0;
  w.q_rot = off;    off = pc_align_up(off + rows * D * 2, kAlign);
  w.part_o = off;   off = pc_align_up(off + part_rows * D * sizeof(float), kAlign);
  w.part_lse = off; off = pc_align_up(off + part_rows * sizeof(float), kAlign);
  w.total = off;
  return w;
}

static int check_par(int batch, int n_q, int n_seg, int k_t, int n_q_heads, int n_kv_heads, int D) {
  if (batch < 1 || n_q < 1 || n_seg < 0 || k_t < 1) return PC_ERR_SHAPE;
  if (n_kv_heads < 1 || n_q_heads < 1 || n_q_heads % n_kv_heads != 0) return PC_ERR_SHAPE;
  if (D != 64 && D != 128) return PC_ERR_SHAPE;
  if (n_q > (1 << 20) || k_t > (1 << 24) || n_seg > (1 << 20) || batch > (1 << 20)) return PC_ERR_SHAPE;
  // kernels index (sequence, segment, head) tuples, partial rows and workgroups with 32-bit integers
  const long long parts = (long long)n_seg + 1;
  if ((long long)batch * parts * n_kv_heads > 0x7fffffffLL / 64) return PC_ERR_SHAPE;
  if ((long long)batch * parts * n_q_heads * ((n_q + 127) / 128) > 0x7fffffffLL / 8) return PC_ERR_SHAPE;
  if ((long long)batch * n_q * n_q_heads > 0x7fffffffLL / 64) return PC_ERR_SHAPE;
  return PC_OK;
}

extern "C" size_t pc_parallel_attn_workspace_bytes(int32_t batch, int32_t n_q, int32_t n_seg,
                                                   int32_t k_t, int32_t n_q_heads,
                                                   int32_t n_kv_heads, int32_t head_dim,
                                                   int32_t has_self) {
  if (check_par(batch, n_q, n_seg, k_t, n_q_heads, n_kv_heads, head_dim) != PC_OK) return 0;
  return par_ws_layout(batch, n_q, n_seg, k_t, n_q_heads, n_kv_heads, head_dim, has_self).total;
}

// Host-visible argument checks shared by pc_parallel_attn and its no-allocation variant.
static int check_par_args(const void* q, const void* kc, const void* vc, int32_t seg_len_per_head,
                          const void* k_self, const void* v_self, int32_t batch, int32_t n_q,
                          int32_t n_seg, int32_t k_t, int32_t n_q_heads, int32_t n_kv_heads,
                          int32_t head_dim, int32_t q_pos0, float rope_base, float softmax_scale,
                          const void* out) {
  int rc = check_par(batch, n_q, n_seg, k_t, n_q_heads, n_kv_heads, head_dim);
  if (rc != PC_OK) return rc;
  if (!q || !out) return PC_ERR_NULL;
  if (n_seg > 0 && (!kc || !vc)) return PC_ERR_NULL;
  if (seg_len_per_head != 0 && seg_len_per_head != 1) return PC_ERR_SHAPE;
  if ((k_self == nullptr) != (v_self == nullptr)) return PC_ERR_NULL;
  if (n_seg == 0 && k_self == nullptr) return PC_ERR_SHAPE;
  if (q_pos0 >= 0 && (!(rope_base > 1.0f) || !isfinite(rope_base))) return PC_ERR_SHAPE;
  if (!(softmax_scale >= 0.0f) || !isfinite(softmax_scale)) return PC_ERR_SHAPE;
  // 16-byte loads and stores on every tensor
  if (!pc_aligned(q, 16) || !pc_aligned(kc, 16) || !pc_aligned(vc, 16) || !pc_aligned(k_self, 16) ||
      !pc_aligned(v_self, 16) || !pc_aligned(out, 16))
    return PC_ERR_SHAPE;
  return PC_OK;
}

// ---- the tile kernel's key groups: segments [batch, n, H_kv, cap, D], the self segment [batch, n_q, H_kv, D]
static PcKvGroup segment_group(const void* k, const void* v, const int32_t* len, int per_head, int n, int cap,
                               int n_kv_heads, int D) {
  PcKvGroup kg = {};
  kg.k = k; kg.v = v; kg.len = len; kg.len_per_head = per_head; kg.n = n; kg.cap = cap;
  kg.row_stride = D; kg.head_stride = (long long)cap * D;
  kg.seg_stride = n_kv_heads * kg.head_stride; kg.seq_stride = n * kg.seg_stride;
  return kg;
}
static PcKvGroup self_group(const void* k, const void* v, int n_q, int n_kv_heads, int D) {
  PcKvGroup kg = {};
  kg.k = k; kg.v = v; kg.n = 1; kg.cap = n_q; kg.causal = 1;
  kg.row_stride = n_kv_heads * D; kg.head_stride = D; kg.seq_stride = (long long)n_q * kg.row_stride;
  return kg;
}

// Tile path of Eq. 9-11: the query operand (rotated and multiplied by scale x log2(e) before the one
// rounding to bf16, so that the matrix cores deliver logits in log2 units; rows that arrive rotated,
// q_pos0 < 0, are only scaled: their bf16 values are rounded a second time), one launch over all key
// groups, the merge if it was cut into parts.
static int tile_attn_run(PcFlashArgs& a, const void* q, int batch, int n_q, int n_q_heads, int n_kv_heads,
                         int D, int q_pos0, float rope_base, float scale, void* q_rot, float* part_o,
                         float* part_lse, int n_parts, void* out, float* lse_out, hipStream_t st) {
  int rc = PC_OK;
  if (q != nullptr) rc = pc_launch_rope_q(q, q_rot, batch, n_q, n_q_heads, D, q_pos0, rope_base, scale * 1.4426950408889634f, st);
  if (rc != PC_OK) return rc;
  a.global = 1; a.q = q_rot; a.o = out; a.lse = lse_out; a.part_o = part_o; a.part_lse = part_lse;
  a.n_seq = batch; a.n_rows = n_q; a.n_q_heads = n_q_heads; a.n_kv_heads = n_kv_heads; a.head_dim = D;
  a.scale = scale; a.n_parts = n_parts; a.window = 8.0f;
  rc = pc_launch_flash(a, st);
  if (rc != PC_OK || n_parts == 1) return rc;
  return pc_launch_merge_rows(part_o, part_lse, out, lse_out, batch, n_q, n_q_heads, D, n_parts, st);
}

// Enqueues the kernels of Eq. 9-11 on a validated request; ws holds at least w.total bytes.  k_new, v_new (few
// rows only): a decoding step, the last segment's next row (self_row: [batch, H_kv] scratch); seg_len counts it.
static int parallel_attn_run(const void* q, const void* kc, const void* vc, const int32_t* seg_len,
                             int32_t seg_len_per_head, const void* k_self, const void* v_self,
                             int32_t batch, int32_t n_q, int32_t n_seg, int32_t k_t,
                             int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                             int32_t q_pos0, float rope_base, float softmax_scale, void* out,
                             float* lse_out, const ParWs& w, void* ws, const void* k_new, const void* v_new,
                             int32_t* self_row, void* stream) {
  int rc;
  const int has_self = k_self != nullptr;
  const int D = head_dim;
  hipStream_t st = (hipStream_t)stream;
  char* base = (char*)ws;
  const float scale = eff_scale(softmax_scale, D);

  float* part_o = (float*)(base + w.part_o);
  float* part_lse = (float*)(base + w.part_lse);

  if (w.small) {
    // split-KV path (the scale is applied to the fp32 logits)
    const void* q_in = q;
    int pos0 = q_pos0;
    if (q_pos0 >= 0 && rotate_first(has_self, (long long)batch * n_kv_heads * w.n_parts)) {
      rc = pc_launch_rope_q(q, base + w.q_rot, batch, n_q, n_q_heads, D, q_pos0, rope_base, 1.0f, st);
      if (rc != PC_OK) return rc;
      q_in = base + w.q_rot; pos0 = -1;
    }
    const PcDecodeAppend app = step_append(k_new, v_new, q_pos0, pos0, base + w.q_rot, self_row);
    if (n_seg > 0) {
      rc = pc_launch_decode(q_in, pos0, rope_base, kc, vc, seg_len, seg_len_per_head, batch, n_q, n_seg, k_t,
                            n_q_heads, n_kv_heads, D, scale, part_o, part_lse, w.n_parts, 0, w.n_parts, app, st);
      if (rc != PC_OK) return rc;
    }
    PcMergeStep step = {};
    if (k_new) step = PcMergeStep{self_row, (const uint16_t*)kc, (const uint16_t*)vc, (int32_t*)seg_len, n_seg, k_t, seg_len_per_head};
    return pc_launch_merge(part_o, part_lse, app.q_rot ? app.q_rot : q_in, k_self, v_self, step, out, lse_out, batch,
                           n_q, n_q_heads, n_kv_heads, D, w.n_parts, scale, st);
  }

  // ---- many query rows: MFMA tile kernel over [segments ; causal self segment]
  rc = check_tile_limits(n_seg, k_t, 0, n_kv_heads, has_self);
  if (rc != PC_OK) return rc;
  PcFlashArgs a = {};
  if (n_seg > 0) a.grp[0] = segment_group(kc, vc, seg_len, seg_len_per_head, n_seg, k_t, n_kv_heads, D);
  if (has_self) a.grp[2] = self_group(k_self, v_self, n_q, n_kv_heads, D);
  return tile_attn_run(a, q, batch, n_q, n_q_heads, n_kv_heads, D, q_pos0, rope_base, scale,
                       base + w.q_rot, part_o, part_lse, w.n_parts, out, lse_out, st);
}

// n segments of up to cap keys as tile images
static PcKvGroup image_group(const void* k, const void* v, const int32_t* len, int per_head, int n, int cap, int n_kv_heads, int D) {
  PcKvGroup kg = segment_group(k, v, len, per_head, n, cap, n_kv_heads, D);
  kg.head_stride = key_tiles(1, cap) * 64 * D;
  kg.seg_stride = n_kv_heads * kg.head_stride; kg.seq_stride = n * kg.seg_stride;
  return kg;
}

// Whether the keys of a block attention over the 8-bit cache become tile images, which spares the tile kernel the
// transposing reads of every (row, key) tile but copies the 16-bit tail and the self segment as well, or the segments
// alone become rows and the rest is read where it lies.  Per KV group, in (row, key) pairs: images gain `rows` a
// visible key and 330 a widened one (turned to a loss of 520 where the widened keys pass the last-level cache and the
// extra bytes count), and cost 4000 a copied row and a share of some 12 M pairs of 128 values a launch.  Fitted to 1358
// calls (1 to 128 groups, 256 to 65536 keys, 17 to 32768 rows a group, tails of 0 to 65536 rows): at most 6 % and on
// average not slower than rows, 1.5 % faster; images everywhere up to 2.7 times slower.  Then both rotated the query rows in a
// launch in front; images have it in the widening launch now, so the line lies some microseconds on the rows' side: over 1100
// calls measured since, its choice takes 1.7 % longer than the better of the two (3 % for those near the line).  0.3 M pairs a
// launch would halve that, with single calls up to 5 % slower.  Rows / images now (us), 32 / 8 heads of 128 values, 8 x 2048
// keys: 5 rows without a tail 65.1 / 59.7, tail of 8192 rows 69.3 / 74.9, 65536 105 / 209; 4 sequences x 512 rows 564 / 505,
// with a tail of 65536 rows 2476 / 2729.  Without segments nothing is widened: rows.
static bool widen_to_images(double groups, int D, double rows, double keys, int tail_cap, int n_self) {
  if (keys == 0.0) return false;
  const double per_launch = 1.2e7 * 128.0 / (groups * D), share = groups * keys * D / 3.2e8;
  return per_launch + ((share < 1.0 ? share : 1.0) * 850.0 - 330.0) * keys + 4000.0 * ((double)tail_cap + n_self) <= rows * (keys + tail_cap);
}

// Eq. 9-11 for a block of query rows over the 8-bit cache: the segments are widened in the workspace (code * scale,
// rounded to bf16), to rows or, with everything else, to tile images; then one launch of the tile kernel as
// for a 16-bit cache: [segments ; 16-bit tail (all its rows visible) ; causal self segment].  The same bits either way,
// except where images are long enough for 64 rows a wavefront (other sums of the same products, wide_workgroup).
static int parallel_attn_fp8_tiles(const void* q, const void* k8, const void* v8, const float* k_scale,
                                   const float* v_scale, const int32_t* seg_len, int seg_len_per_head,
                                   const void* k_tail, const void* v_tail, const int32_t* tail_len,
                                   int tail_cap, const void* k_self, const void* v_self, int batch,
                                   int n_q, int n_seg, int k_t, int n_q_heads, int n_kv_heads, int D,
                                   int q_pos0, float rope_base, float scale, void* out, float* lse_out,
                                   const Par8Ws& w, char* base, hipStream_t st) {
  PcFlashArgs a = {};
  auto at = [&](size_t off) { return (uint16_t*)(base + off); };
  const long long n_segs = (long long)batch * n_seg * n_kv_heads;
  a.images = widen_to_images((double)batch * n_kv_heads, D, (double)n_q * (n_q_heads / n_kv_heads), (double)n_seg * k_t, tail_cap,
                             k_self != nullptr ? n_q : 0);
  if (!a.images) {
    if (n_seg > 0) {
      const int rc = pc_launch_fp8_rows(k8, v8, k_scale, v_scale, seg_len, seg_len_per_head, n_segs, n_kv_heads, k_t, D, at(w.k_img[0]),
                                        at(w.v_img[0]), st);
      if (rc != PC_OK) return rc;
      a.grp[0] = segment_group(at(w.k_img[0]), at(w.v_img[0]), seg_len, seg_len_per_head, n_seg, k_t, n_kv_heads, D);
    }
    if (tail_cap > 0) a.grp[1] = segment_group(k_tail, v_tail, tail_len, 0, 1, tail_cap, n_kv_heads, D);
    if (k_self != nullptr) a.grp[2] = self_group(k_self, v_self, n_q, n_kv_heads, D);
  } else {
    PcRowsToImages tail = {}, self = {};
    if (n_seg > 0) a.grp[0] = image_group(at(w.k_img[0]), at(w.v_img[0]), seg_len, seg_len_per_head, n_seg, k_t, n_kv_heads, D);
    if (tail_cap > 0) {
      tail = PcRowsToImages{(const uint16_t*)k_tail, (const uint16_t*)v_tail, tail_len, tail_cap, D, (long long)n_kv_heads * tail_cap * D,
                            (long long)tail_cap * D, at(w.k_img[1]), at(w.v_img[1])};
      a.grp[1] = image_group(tail.k_img, tail.v_img, tail_len, 0, 1, tail_cap, n_kv_heads, D);
    }
    if (k_self != nullptr) {
      self = PcRowsToImages{(const uint16_t*)k_self, (const uint16_t*)v_self, nullptr, n_q, n_kv_heads * D,
                            (long long)n_q * n_kv_heads * D, D, at(w.k_img[2]), at(w.v_img[2])};
      a.grp[2] = image_group(self.k_img, self.v_img, nullptr, 0, 1, n_q, n_kv_heads, D);
      a.grp[2].causal = 1;
    }
    PcRowsToRotate rows = {};
    rows.q = (const uint16_t*)q; rows.q_rot = at(w.q_rot); rows.rows = (uint32_t)((long long)batch * n_q);
    rows.n_q = n_q; rows.n_heads = n_q_heads; rows.pos0 = q_pos0;
    rows.rope = pc_rope_factors(q_pos0 >= 0 ? rope_base : 2.0f, D); rows.mul = (double)(scale * 1.4426950408889634f);
    const int rc = pc_launch_fp8_images(k8, v8, k_scale, v_scale, seg_len, seg_len_per_head, n_segs, k_t, D, at(w.k_img[0]),
                                        at(w.v_img[0]), tail, self, batch, n_kv_heads, rows, st);
    if (rc != PC_OK) return rc;
    q = nullptr;                                             // rotated there
  }
  return tile_attn_run(a, q, batch, n_q, n_q_heads, n_kv_heads, D, q_pos0, rope_base, scale,
                       base + w.q_rot, (float*)(base + w.part_o), (float*)(base + w.part_lse),
                       w.n_parts, out, lse_out, st);
}

extern "C" int pc_parallel_attn(const void* q, const void* kc, const void* vc, const int32_t* seg_len,
                                int32_t seg_len_per_head, const void* k_self, const void* v_self, int32_t batch, int32_t n_q,
                                int32_t n_seg, int32_t k_t, int32_t n_q_heads, int32_t n_kv_heads,
                                int32_t head_dim, int32_t q_pos0, float rope_base,
                                float softmax_scale, void* out, float* lse_out, void* ws,
                                size_t ws_bytes, void* stream) {
  const int rc = check_par_args(q, kc, vc, seg_len_per_head, k_self, v_self, batch, n_q, n_seg, k_t,
                                n_q_heads, n_kv_heads, head_dim, q_pos0, rope_base, softmax_scale, out);
  if (rc != PC_OK) return rc;
  const ParWs w = par_ws_layout(batch, n_q, n_seg, k_t, n_q_heads, n_kv_heads, head_dim,
                                k_self != nullptr);
  if (!ws || !pc_aligned(ws, kAlign) || ws_bytes < w.total) return PC_ERR_WORKSPACE;
  return parallel_attn_run(q, kc, vc, seg_len, seg_len_per_head, k_self, v_self, batch, n_q, n_seg,
                           k_t, n_q_heads, n_kv_heads, head_dim, q_pos0, rope_base, softmax_scale,
                           out, lse_out, w, ws, nullptr, nullptr, nullptr, stream);
}

// ---------------------------------------------------------------------------- a whole layer
static int check_select_tokens(int n_sel, int n_kv_heads, int chunk_len, int k) {
  if (n_sel < 0 || n_kv_heads < 1 || chunk_len < 1 || chunk_len > 32768 || k < 1 || k > chunk_len) return PC_ERR_SHAPE;
  if ((long long)n_sel * n_kv_heads > 0x7fffffffLL) return PC_ERR_SHAPE;
  return PC_OK;
}

extern "C" size_t pc_layer_workspace_bytes(const pc_shape* s, int32_t keep_chunks, int32_t keep_tokens) {
  const size_t prefill = pc_chunk_prefill_workspace_bytes(s);
  if (prefill == 0) return 0;
  const size_t attn = pc_parallel_attn_workspace_bytes(1, s->query_len, keep_chunks, keep_tokens, s->n_q_heads,
                                                       s->n_kv_heads, s->head_dim, 1);
  return attn ? pc_align_up(prefill, kAlign) + attn : 0;
}

extern "C" int pc_layer_forward(const pc_shape* s, const void* q, const void* k, const void* v, const int32_t* chunk_lens,
                                int32_t first_len, int32_t keep_chunks, int32_t keep_tokens, int32_t calibrated, float lambda,
                                int32_t class_lo, int32_t class_hi, void* o, float* lse, void* k_rope, float* tok_score,
                                float* chunk_score, int32_t* chunk_idx, float* chunk_top, int32_t* tok_idx, int32_t* tok_cnt,
                                void* kc, void* vc, void* global_o, float* global_lse, void* ws, size_t ws_bytes, void* stream) {
  int rc = check_shape(s);
  if (rc != PC_OK) return rc;
  rc = check_prefill_args(q, k, v, o, lse, k_rope, tok_score, chunk_score);
  if (rc != PC_OK) return rc;
  if (!tok_score || !chunk_score || !k_rope || !chunk_idx || !tok_idx || (calibrated && !tok_cnt)) return PC_ERR_NULL;
  rc = check_obs(s, chunk_lens != nullptr);
  if (rc != PC_OK) return rc;
  const int C = s->n_chunks, w_ctx = s->chunk_len, n_q = s->query_len, Hq = s->n_q_heads, Hkv = s->n_kv_heads, D = s->head_dim;
  if (C > 4096 || keep_chunks < 1 || keep_chunks > C || first_len < 0 || first_len > w_ctx) return PC_ERR_SHAPE;
  rc = check_select_tokens(keep_chunks, Hkv, w_ctx, keep_tokens);
  if (rc != PC_OK) return rc;
  if (calibrated && (class_lo < 0 || class_hi < class_lo || class_hi > w_ctx || lambda != lambda)) return PC_ERR_SHAPE;
  if (!kc || !vc) return PC_ERR_NULL;
  // the query block: the rows behind chunk 0's context
  const uint16_t* q_blk = (const uint16_t*)q + (size_t)first_len * Hq * D;
  const uint16_t* k_self = (const uint16_t*)k_rope + (size_t)first_len * Hkv * D;
  const uint16_t* v_self = (const uint16_t*)v + (size_t)first_len * Hkv * D;
  rc = check_par_args(q_blk, kc, vc, calibrated != 0, k_self, v_self, 1, n_q, keep_chunks, keep_tokens, Hq, Hkv, D, first_len,
                      s->rope_base, s->softmax_scale, global_o);
  if (rc != PC_OK) return rc;
  const PrefillWs w = prefill_ws_layout(s);
  const size_t attn0 = pc_align_up(pc_chunk_prefill_workspace_bytes(s), kAlign);
  const ParWs pw = par_ws_layout(1, n_q, keep_chunks, keep_tokens, Hq, Hkv, D, 1);
  if (!ws || !pc_aligned(ws, kAlign) || ws_bytes < attn0 + pw.total) return PC_ERR_WORKSPACE;
  if (!pw.small) {
    rc = check_tile_limits(keep_chunks, keep_tokens, 0, Hkv, 1);
    if (rc != PC_OK) return rc;
  }
  hipStream_t st = (hipStream_t)stream;
  char* base = (char*)ws;
  char* attn = base + attn0;
  float2* table = (float2*)(base + w.table);
  const float scale = eff_scale(s->softmax_scale, D);
  const int L = w_ctx + n_q;

  PcPrepArgs prep = {};
  prep.table = table; prep.n_pos = L; prep.rope = pc_rope_factors(s->rope_base, D);
  prep.q_table = (float2*)(base + w.q_table); prep.q_scale = (double)(scale * 1.4426950408889634f);
  if (!pw.small) {
    prep.q_blk = q_blk; prep.q_rot = (uint16_t*)(attn + pw.q_rot); prep.n_q = n_q; prep.n_heads = Hq; prep.pos0 = first_len;
    prep.mul = (double)(scale * 1.4426950408889634f);
  }
  prep.scores = pc_scores_queries(s, q, chunk_lens, base + w.ml);
  rc = pc_launch_prep(prep, D, st);
  if (rc != PC_OK) return rc;
  PcChunkSum sum = {};
  const PcPrepassOut pre = {v, k_rope, base + w.k_img, base + w.v_img, w.Lp};
  rc = pc_launch_scores(s, k, chunk_lens, table, base + w.ml, tok_score, chunk_score, &pre, &sum, st);
  if (rc != PC_OK) return rc;
  // the selections need the scores, not the attention: they and the gather come first, and the global
  // attention rides in the local one's launch
  const int lo = calibrated ? class_lo : 0, hi = calibrated ? class_hi : 0;
  const int32_t* lens = calibrated ? chunk_lens : nullptr;
  int32_t* cnt = calibrated ? tok_cnt : nullptr;
  const bool small_rows = pc_select_gather_fits(keep_tokens, D), one_select = pc_select_layer_fits(C, sum.per_chunk, small_rows);
  if (one_select) {
    rc = pc_launch_select_layer(sum, C, keep_chunks, tok_score, Hkv, w_ctx, keep_tokens, lambda, lo, hi, lens, chunk_idx,
                                chunk_top, tok_idx, cnt, k_rope, v, L, D, kc, vc, st);
  } else {
    rc = pc_launch_chunk_sums(sum, C, st);
    if (rc == PC_OK) rc = pc_launch_select_chunks(chunk_score, C, keep_chunks, chunk_idx, chunk_top, st);
    if (rc == PC_OK)
      rc = pc_launch_select_tokens(tok_score, chunk_idx, keep_chunks, Hkv, w_ctx, keep_tokens, lambda, lo, hi, lens, tok_idx, cnt, st);
  }
  if (rc == PC_OK && !(one_select && small_rows))
    rc = pc_launch_gather(k_rope, v, chunk_idx, tok_idx, 1, C, L, keep_chunks, Hkv, keep_tokens, D, kc, vc, nullptr, nullptr, st);
  if (rc != PC_OK) return rc;
  const PcFlashArgs local = local_flash_args(s, q, chunk_lens, o, lse, base, w);
  if (pw.small) {
    rc = pc_launch_flash(local, st);
    if (rc != PC_OK) return rc;
    return parallel_attn_run(q_blk, kc, vc, cnt, calibrated != 0, k_self, v_self, 1, n_q, keep_chunks, keep_tokens, Hq, Hkv, D,
                             first_len, s->rope_base, s->softmax_scale, global_o, global_lse, pw, attn, nullptr, nullptr,
                             nullptr, stream);
  }
  PcFlashArgs g = {};
  g.grp[0] = segment_group(kc, vc, cnt, calibrated != 0, keep_chunks, keep_tokens, Hkv, D);
  g.grp[2] = self_group(k_self, v_self, n_q, Hkv, D);
  g.global = 1; g.q = attn + pw.q_rot; g.o = global_o; g.lse = global_lse;
  g.part_o = (float*)(attn + pw.part_o); g.part_lse = (float*)(attn + pw.part_lse);
  g.n_seq = 1; g.n_rows = n_q; g.n_q_heads = Hq; g.n_kv_heads = Hkv; g.head_dim = D; g.scale = scale; g.window = 0.0f;
  g.n_parts = pc_flash_both_parts(C, L, n_q, Hq, Hkv, D, key_tiles(keep_chunks, keep_tokens) + key_tiles(1, n_q), pw.n_parts);
  rc = pc_launch_flash_both(local, g, st);
  if (rc != PC_OK || g.n_parts == 1) return rc;
  return pc_launch_merge_rows(g.part_o, g.part_lse, global_o, global_lse, 1, n_q, Hq, D, g.n_parts, st);
}

// ---------------------------------------------------------------------------- decoding step
// pc_kv_append of one row + the attention of one row, as two launches: the split-KV kernel stores the new row
// (its lengths still exclude it) and the merge takes it as one more key and counts it.
// [batch, H_kv] int32 behind the attention's workspace
static size_t self_row_bytes(int batch, int n_kv_heads) { return pc_align_up((size_t)batch * n_kv_heads * 4, kAlign); }

extern "C" size_t pc_decode_step_workspace_bytes(int32_t batch, int32_t n_seg, int32_t k_t, int32_t n_q_heads,
                                                 int32_t n_kv_heads, int32_t head_dim) {
  const size_t attn = pc_parallel_attn_workspace_bytes(batch, 1, n_seg, k_t, n_q_heads, n_kv_heads, head_dim, 0);
  return attn ? attn + self_row_bytes(batch, n_kv_heads) : 0;
}

extern "C" int pc_decode_step(const void* q, const void* k_new, const void* v_new, int32_t batch, int32_t n_seg,
                              int32_t k_t, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim, int32_t pos,
                              float rope_base, float softmax_scale, void* kc, void* vc, int32_t* seg_len,
                              int32_t seg_len_per_head, void* out, float* lse_out, void* ws, size_t ws_bytes,
                              void* stream) {
  int rc = check_append(k_new, v_new, batch, 1, n_seg, n_seg - 1, k_t, n_kv_heads, head_dim, pos, rope_base, kc, vc, seg_len);
  if (rc != PC_OK) return rc;
  rc = check_par_args(q, kc, vc, seg_len_per_head, nullptr, nullptr, batch, 1, n_seg, k_t, n_q_heads, n_kv_heads,
                      head_dim, pos, rope_base, softmax_scale, out);
  if (rc != PC_OK) return rc;
  const ParWs w = par_ws_layout(batch, 1, n_seg, k_t, n_q_heads, n_kv_heads, head_dim, 0);
  if (!ws || !pc_aligned(ws, kAlign) || ws_bytes < w.total + self_row_bytes(batch, n_kv_heads)) return PC_ERR_WORKSPACE;
  if (!w.small) {                                            // more than 16 heads a group: the tile path
    rc = check_tile_limits(n_seg, k_t, 0, n_kv_heads, 0);
    if (rc == PC_OK)
      rc = pc_launch_kv_append(k_new, v_new, batch, 1, n_seg, n_seg - 1, k_t, n_kv_heads, head_dim, pos, rope_base,
                               kc, vc, seg_len, seg_len_per_head, (hipStream_t)stream);
    if (rc != PC_OK) return rc;
    k_new = v_new = nullptr;
  }
  return parallel_attn_run(q, kc, vc, seg_len, seg_len_per_head, nullptr, nullptr, batch, 1, n_seg, k_t, n_q_heads,
                           n_kv_heads, head_dim, pos, rope_base, softmax_scale, out, lse_out, w, ws, k_new, v_new,
                           (int32_t*)((char*)ws + w.total), stream);
}

extern "C" size_t pc_decode_step_fp8_workspace_bytes(int32_t batch, int32_t n_seg, int32_t k_t, int32_t tail_cap,
                                                     int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim) {
  const size_t attn = pc_parallel_attn_fp8_workspace_bytes(batch, 1, n_seg, k_t, tail_cap, n_q_heads, n_kv_heads, head_dim, 0);
  return attn ? attn + self_row_bytes(batch, n_kv_heads) : 0;
}

extern "C" int pc_decode_step_fp8(const void* q, const void* k_new, const void* v_new, const void* k8, const void* v8,
                                  const float* k_scale, const float* v_scale, const int32_t* seg_len,
                                  int32_t seg_len_per_head, void* k_tail, void* v_tail, int32_t* tail_len,
                                  int32_t tail_cap, int32_t batch, int32_t n_seg, int32_t k_t, int32_t n_q_heads,
                                  int32_t n_kv_heads, int32_t head_dim, int32_t pos, float rope_base,
                                  float softmax_scale, void* out, float* lse_out, void* ws, size_t ws_bytes,
                                  void* stream) {
  int rc = check_append(k_new, v_new, batch, 1, 1, 0, tail_cap, n_kv_heads, head_dim, pos, rope_base, k_tail, v_tail, tail_len);
  if (rc != PC_OK) return rc;
  rc = check_par8_args(q, k8, v8, k_scale, v_scale, seg_len_per_head, k_tail, v_tail, tail_len, tail_cap, nullptr,
                       nullptr, batch, 1, n_seg, k_t, n_q_heads, n_kv_heads, head_dim, pos, rope_base, softmax_scale, out);
  if (rc != PC_OK) return rc;
  const int D = head_dim;
  const Par8Ws w = par8_ws_layout(batch, 1, n_seg, k_t, tail_cap, n_q_heads, n_kv_heads, D, 0);
  if (!ws || !pc_aligned(ws, kAlign) || ws_bytes < w.total + self_row_bytes(batch, n_kv_heads)) return PC_ERR_WORKSPACE;
  const float scale = eff_scale(softmax_scale, D);
  hipStream_t st = (hipStream_t)stream;
  if (w.small)
    return par8_small_run(q, k8, v8, k_scale, v_scale, seg_len, seg_len_per_head, k_tail, v_tail, tail_len, tail_cap,
                          nullptr, nullptr, batch, 1, n_seg, k_t, n_q_heads, n_kv_heads, D, pos, rope_base, scale, out,
                          lse_out, w, (char*)ws, k_new, v_new, (int32_t*)((char*)ws + w.total), st);
  rc = check_tile_limits(n_seg, k_t, tail_cap, n_kv_heads, 0);
  if (rc == PC_OK)
    rc = pc_launch_kv_append(k_new, v_new, batch, 1, 1, 0, tail_cap, n_kv_heads, D, pos, rope_base, k_tail, v_tail,
                             tail_len, 0, st);
  if (rc != PC_OK) return rc;
  return parallel_attn_fp8_tiles(q, k8, v8, k_scale, v_scale, seg_len, seg_len_per_head, k_tail, v_tail, tail_len,
                                 tail_cap, nullptr, nullptr, batch, 1, n_seg, k_t, n_q_heads, n_kv_heads, D, pos,
                                 rope_base, scale, out, lse_out, w, (char*)ws, st);
}

// ---------------------------------------------------------------------------- no-allocation variant
// The scratch memory of pc_parallel_attn_static: one array per GPU, part of the loaded code
// object, alive until the process ends.  `scratch` names it in device code only; host code uses
// the per-device address that hipGetSymbolAddress returns (the array sits at a different address
// on every GPU).
static __device__ __align__(256) unsigned char scratch[PC_STATIC_SCRATCH_BYTES];

#define PC_MAX_DEVICES 64
static std::mutex g_scratch_mutex;
static void* g_scratch_ptr[PC_MAX_DEVICES];     // by device ordinal; nullptr = not resolved yet

// Address of `scratch` on the current device (resolved once per device, with that device current).
static int static_scratch(void** ptr) {
  int dev = -1;
  PC_HIP_TRY(hipGetDevice(&dev));
  if (dev < 0 || dev >= PC_MAX_DEVICES) return PC_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    PC_HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    if (p == nullptr || !pc_aligned(p, kAlign)) return PC_ERR_WORKSPACE;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return PC_OK;
}

extern "C" size_t pc_parallel_attn_static_max_bytes(void) { return PC_STATIC_SCRATCH_BYTES; }

extern "C" int pc_parallel_attn_static(const void* q, const void* kc, const void* vc,
                                       const int32_t* seg_len, int32_t seg_len_per_head,
                                       const void* k_self, const void* v_self, int32_t batch,
                                       int32_t n_q, int32_t n_seg, int32_t k_t, int32_t n_q_heads,
                                       int32_t n_kv_heads, int32_t head_dim, int32_t q_pos0,
                                       float rope_base, float softmax_scale, void* out,
                                       float* lse_out, void* stream) {
  int rc = check_par_args(q, kc, vc, seg_len_per_head, k_self, v_self, batch, n_q, n_seg, k_t,
                          n_q_heads, n_kv_heads, head_dim, q_pos0, rope_base, softmax_scale, out);
  if (rc != PC_OK) return rc;
  const ParWs w = par_ws_layout(batch, n_q, n_seg, k_t, n_q_heads, n_kv_heads, head_dim,
                                k_self != nullptr);
  if (!w.small) return PC_ERR_UNSUPPORTED;                  // the tile path is not served here
  if (w.total > PC_STATIC_SCRATCH_BYTES) return PC_ERR_WORKSPACE;
  void* ws = nullptr;
  rc = static_scratch(&ws);
  if (rc != PC_OK) return rc;
  // every byte of the scratch that the merge reads is written by this call's kernels first
  // (rotated q, one partial per workgroup), so nothing has to be cleared
  return parallel_attn_run(q, kc, vc, seg_len, seg_len_per_head, k_self, v_self, batch, n_q, n_seg,
                           k_t, n_q_heads, n_kv_heads, head_dim, q_pos0, rope_base, softmax_scale,
                           out, lse_out, w, ws, nullptr, nullptr, nullptr, stream);
}
