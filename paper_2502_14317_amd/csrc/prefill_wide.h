// Attention with 64 query rows a wavefront for head_dim 128: flash_workgroup's local mode for calls of many long rows
// (pc_flash_wide) and its mode of tile images for long runs (pc_flash_wide_images).  Included by prefill_attn.hip.
//
// What bounds flash_workgroup: at 32 rows a wavefront every MFMA has an LDS operand read of its own, so the
// CU's LDS reads take as long as its MFMAs, and on real data the clock falls to 1.5 GHz under the power limit.
// Two 32-row blocks share every K and V^T operand here: half the LDS reads, half the tile copies.  That takes
// 461 registers (over tile images, with the walk, 491 and 76 scalar ones spilled; next to the global attention 29), so one wavefront a SIMD and one workgroup of 256 rows a CU; what the second wavefront used to
// hide has to fit between the MFMAs of the one.  It does: a step is 32 slices of one MFMA (32 cycles), a
// softmax element for each lane (exp2 8, add 4, half a pack 8 cycles) and every other slice an LDS read.
// Cycles a 64-key tile (2048 of MFMAs), before the second row sum (round_part): 2350; without the loads 2320, without the
// barrier 2300, without either and without the LDS reads 2150.  16 x 8192 rows, 32 / 8 heads, with the pre-pass: 7430 us in
// flash_workgroup, 6800 here (4950 and 5010 on all-zero inputs: what is saved is power); 64 x 8704 33.6 and 30.8 ms.
//
// Registers: O^T and Q^T lie in accumulation registers, S^T, P^T and the operands in the others.  The compiler
// would put O^T into the others too and move Q^T back and forth, so P V products are written as assembly text;
// so are the exponentials, sums and packs, which it otherwise moves across the slices (2700 cycles a tile).
// What the compiler then no longer sees to: two issue states between a write of a product's operand and the
// product (P^T is packed a region ahead, and each step's first product waits by itself, as a copy of O^T may
// stand in front of it), twelve between a product and a use of its result (o_settle; S^T is used two
// products after its last one), seven before its addend is written, one between an exponential and the use of its result
// (the group after it).  spacing.py looks for all of them in the compiled code of every build.
//
// PC_FW_PAIR: the workgroup takes `wide_heads` query heads of a KV head (2, 4 or 8) at 256 / wide_heads positions,
// a wavefront two heads at 32 positions: one rotation table row, one mask and one causal end for both blocks.
// PC_FW_HEAD: 256 positions of one head, 64 a wavefront.
// PC_FW_IMAGES: flash_workgroup's mode of that name, rows of a KV group packed, parts and all: 4 x 512 rows of 32 / 8
// heads over 8 x 2048 keys of the 8-bit cache 691 -> 648 us with everything else of the call, 3 sequences (four parts)
// 565 -> 544, 2 x 512 of 32 / 32 722 -> 702.  Loads follow a walk over the segments' tiles that runs three ahead.
#define PC_FW_FAR 262144.f           // a lane's row sum above it shows a reference behind the row's maximum (2^18: 2^10 keys, 2^8 behind)
#define PC_FW_RING 4                 // tiles of K and of V^T in LDS, 128 KiB
constexpr int FW_D = 128, FW_TILE = 64 * FW_D;               // elements of a tile image
constexpr int FW_LDS_BYTES = 2 * PC_FW_RING * FW_TILE * 2;

#define PC_FW_PAIR 0
#define PC_FW_HEAD 1
#define PC_FW_IMAGES 2
template <int MODE>
__device__ __forceinline__ void wide_workgroup(const PcFlashArgs& a, int bid, uint16_t* smem) {
  constexpr bool PAIR = MODE == PC_FW_PAIR, IMAGES = MODE == PC_FW_IMAGES;
  constexpr int D = FW_D, KS = D / 16, DB = D / 32, HALF = D / 2, NB = 2, NM = NB * KS;
  // ---- which (sequence, KV head), Q tile and heads: as flash_workgroup; a.group workgroups share a Q tile.  The
  //      groups that share an XCD change places every other turn: an XCD hands every fourth workgroup to the same
  //      shader engine, in order, and with a short sequence always in the same place two engines got all the
  //      padding (12 ragged chunks of 2214 rows 332 -> 309 us; changed every turn, a group of a batch of 2, 6 or 10 would
  //      keep to two engines too, changed every other one each engine gets a quarter to within 6 %).  The groups beyond a multiple of 8 are dealt to
  //      all XCDs in the same way, long Q tiles of all of them first.
  const int n_qt = a.n_qt, per_group = (IMAGES ? a.n_parts : a.group) * n_qt;
  const int n_groups = a.n_seq * a.n_kv_heads, full_blocks = n_groups / 8 * 8 * per_group;
  int cg, within;
  if (bid < full_blocks) {
    const int xcd = bid % 8, jb = bid / 8;
    const int batch = pc_div(jb, a.per_batch_div), in_batch = jb - batch * (a.group_batch * per_group);
    const int left = n_groups / 8 - batch * a.group_batch, n_batch = min(a.group_batch, left);
    const PcDiv by = left >= a.group_batch ? a.batch_div : a.last_div;
    within = pc_div(in_batch, by);
    const int place = in_batch - within * n_batch + (within >> 1);
    cg = (batch * a.group_batch + pc_mod(place, n_batch, by)) * 8 + xcd;
  } else {
    const int rest = bid - full_blocks, n_rest = n_groups % 8;
    within = pc_div(rest, a.per_group_div);
    cg = n_groups / 8 * 8 + pc_mod(rest - within * n_rest + within, n_rest, a.per_group_div);
  }
  const int seq = pc_div(cg, a.heads_div), g = cg - seq * a.n_kv_heads;
  const int turn = pc_div(within, IMAGES ? a.qt_div : a.group_div);        // (IMAGES: the part)
  const int HW = PAIR ? a.wide_heads : 1, P_WG = 256 / HW;
  constexpr int POS_W = PAIR ? 32 : 64;                      // positions of a wavefront
  const int tid = threadIdx.x, lane = tid % PC_WAVE, wave = __builtin_amdgcn_readfirstlane(tid / PC_WAVE);
  const int hf = lane / 32, n = lane % 32;
  const int pos0_wg = (IMAGES ? within - turn * n_qt : n_qt - 1 - turn) * P_WG;
  const int seq_rows = IMAGES ? a.n_rows * a.group
                              : (a.seq_ctx ? min(max(a.seq_ctx[seq], 0), a.n_rows - a.seq_add) + a.seq_add : a.n_rows);
  if (pos0_wg >= seq_rows) return;                           // padding rows (uniform over the workgroup)
  const int pos0 = pos0_wg + 32 * (2 * wave / HW);           // the wavefront's first position (IMAGES: packed row) and head
  const int h = IMAGES ? g * a.group : (g * a.group + within - turn * a.group) * HW + (PAIR ? 2 * wave % HW : 0);
  int T = (min(seq_rows, pos0_wg + P_WG) + 63) / 64;         // key tiles
  const int J0 = (min(pos0_wg, seq_rows - 1) + 1) / 32;      // steps of 32 keys that every row sees whole
  int max_key[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    max_key[nb] = min(pos0 + (PAIR ? 0 : 32 * nb) + n, seq_rows - 1);
    if (IMAGES) max_key[nb] = pc_div(max_key[nb], a.group_div);        // the row's query
  }
  // IMAGES: a walk over the segments' tiles, those that every row sees whole first (as flash_workgroup's cursor).
  // A tile's limits: valid keys from its first one, that key's position where the segment is causal.
  struct Limit { int cut, c0; bool seg_start; };
  struct Walk { const uint16_t* k; const uint16_t* v; Limit lim; int c0_step, in_seg, in_phase, left, grp, seg; bool masked; };
  Walk cur = {};
  int run_full = 0, masked_lo = 0;                           // unmasked tiles of the run; its first masked tile
  const int wg_t0 = pc_div(pos0_wg, a.group_div), wg_t1 = pc_div(min(pos0_wg + 256, seq_rows) - 1, a.group_div);
  auto walk_place = [&](int tile, int len) __attribute__((always_inline)) {  // tile: among the segment's of this kind
    const PcKvGroup& kg = a.grp[cur.grp];
    const int idx = tile + (cur.masked ? pc_full_tiles(kg, len, wg_t0) : 0);
    const long long at = seq * kg.seq_stride + cur.seg * kg.seg_stride + g * kg.head_stride + (long long)FW_TILE * idx;
    cur.k = (const uint16_t*)kg.k + at; cur.v = (const uint16_t*)kg.v + at;
    cur.lim = {len - 64 * idx, kg.causal ? 64 * idx : -(1 << 28), idx == 0};
    cur.c0_step = kg.causal ? 64 : 0;
    cur.in_seg = pc_seg_tiles(kg, len, wg_t0, wg_t1, cur.masked) - tile;
  };
  auto walk_seek = [&](int rel) __attribute__((always_inline)) {             // to tile `rel` of this kind
    int tile = 0, len = 0;
    for (cur.grp = 0; cur.grp < PC_KV_GROUPS; ++cur.grp) {
      const int nt = a.grp[cur.grp].n > 0 ? pc_kv_tiles(a.grp[cur.grp], seq, g, a.n_kv_heads, wg_t0, wg_t1, cur.masked, lane) : 0;
      if (rel < nt) break;
      rel -= nt;
    }
    pc_kv_find(a.grp[cur.grp], seq, g, a.n_kv_heads, wg_t0, wg_t1, cur.masked, lane, rel, cur.seg, tile, len);
    walk_place(tile, len);
  };
  auto walk_next = [&]() __attribute__((always_inline)) {    // stays on the run's last tile
    if (cur.left <= 1) return;
    --cur.left; --cur.in_phase;
    if (cur.in_phase > 0 && --cur.in_seg > 0) {
      cur.k += FW_TILE; cur.v += FW_TILE;
      cur.lim.cut -= 64; cur.lim.c0 += cur.c0_step; cur.lim.seg_start = false;
    } else if (cur.in_phase > 0) {
      int len;
      do {                                                   // the next segment that has tiles of this kind
        if (++cur.seg >= a.grp[cur.grp].n) { cur.seg = 0; ++cur.grp; }
        len = a.grp[cur.grp].n > 0 ? __builtin_amdgcn_readfirstlane(pc_seg_len(a.grp[cur.grp], seq, g, a.n_kv_heads, cur.seg)) : 0;
      } while (len == 0 || pc_seg_tiles(a.grp[cur.grp], len, wg_t0, wg_t1, cur.masked) == 0);
      walk_place(0, len);
    } else {
      cur.masked = true;
      cur.in_phase = cur.left;
      walk_seek(masked_lo);
    }
  };
  auto walk_begin = [&]() __attribute__((always_inline)) {
    int n_full = 0, n_masked = 0;
    for (int i = 0; i < PC_KV_GROUPS; ++i)
      if (a.grp[i].n > 0) {
        n_full += pc_kv_tiles(a.grp[i], seq, g, a.n_kv_heads, wg_t0, wg_t1, false, lane);
        n_masked += pc_kv_tiles(a.grp[i], seq, g, a.n_kv_heads, wg_t0, wg_t1, true, lane);
      }
    // every part takes an equal run of all tiles, as in flash_workgroup
    const int lo = pc_div((n_full + n_masked) * turn, a.parts_div), hi = pc_div((n_full + n_masked) * (turn + 1), a.parts_div);
    T = cur.left = hi - lo;
    run_full = max(0, min(hi, n_full) - lo);
    masked_lo = max(0, lo - n_full);
    if (T > 0) {
      cur.masked = run_full == 0;
      cur.in_phase = cur.masked ? T : run_full;
      walk_seek(cur.masked ? masked_lo : lo);
    }
  };
  if (IMAGES) walk_begin();
  Limit lim0 = cur.lim, lim1 = {}, lim2 = {};                // of tiles p, p + 1, p + 2

  // ---- tile loads: wavefront w copies bytes 4096 w .. of a tile image, 1 KiB an instruction (the immediate
  //      offset counts on both sides).  Tile t lives in slot t % 4; images behind the last one read as zeros.
  typedef __attribute__((address_space(3))) void* lptr_t;
  constexpr int IMG_BYTES = FW_TILE * 2, T_LD = 4;
  const int n_img = (a.n_rows + 63) / 64;
  const long long img0 = (seq * a.img_seq_stride + g * a.img_head_stride) * (64LL * D);
  const __amdgpu_buffer_rsrc_t k_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)((const uint16_t*)a.k_img + img0), 0, n_img * IMG_BYTES, 0x00020000);
  const __amdgpu_buffer_rsrc_t v_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)((const uint16_t*)a.v_img + img0), 0, n_img * IMG_BYTES, 0x00020000);
  const int ld_goff = 4096 * wave + 16 * lane;
  uint16_t* const v_area = smem + PC_FW_RING * FW_TILE;
  // (IMAGES: tile t is the one that the walk is on)
#define FW_LOAD_K(t, i) __builtin_amdgcn_raw_ptr_buffer_load_lds(IMAGES ? __builtin_amdgcn_make_buffer_rsrc((void*)cur.k, 0, IMG_BYTES, 0x00020000) : k_rsrc, (lptr_t)(smem + ((t) & 3) * FW_TILE + 2048 * wave), 16, ld_goff, IMAGES ? 0 : (t) * IMG_BYTES, 1024 * (i), 0)
#define FW_LOAD_V(t, i) __builtin_amdgcn_raw_ptr_buffer_load_lds(IMAGES ? __builtin_amdgcn_make_buffer_rsrc((void*)cur.v, 0, IMG_BYTES, 0x00020000) : v_rsrc, (lptr_t)(v_area + ((t) & 3) * FW_TILE + 2048 * wave), 16, ld_goff, IMAGES ? 0 : (t) * IMG_BYTES, 1024 * (i), 0)
#define FW_LOAD4(M, t) do { M(t, 0); M(t, 1); M(t, 2); M(t, 3); } while (0)

  // ---- queries, as flash_workgroup fetches, stages (slots 2 and 3 of V) and rotates them, a block after the other.
  //      Of the tiles only K 0 and V 0 are asked for in front of the queries' arrival: 40 loads a
  //      wavefront are 2500 cycles of the CU's path already (5800 -> 4900 cycles until all are out).
  bf16x8 bq[NB][KS];
  floatx16 o_acc[NB][DB];
  constexpr int PPR = D / 8, RPL = PC_WAVE / PPR, NLD = 32 / RPL;
  const int rows_left = min(seq_rows - pos0, POS_W);
  const int qo_stride = a.n_q_heads * (2 * D);
  auto row_at = [&](int r) __attribute__((always_inline)) {  // (IMAGES) a packed row in [row, head] of q and output
    return ((long long)seq * a.n_rows + pc_div(r, a.group_div)) * a.n_q_heads + h + pc_mod(r, a.group, a.group_div);
  };
  const int qo_bytes = rows_left > 0 ? (rows_left - 1) * qo_stride + (PAIR ? 2 * D * NB : 2 * D) : 0;
  const int nb_step = PAIR ? 2 * D : 32 * qo_stride;         // bytes from a row of block 0 to block 1's
  const long long qo_at = (((long long)seq * a.n_rows + (rows_left > 0 ? pos0 : 0)) * a.n_q_heads + h) * D;
  const int l_row = lane / PPR, l_piece = lane % PPR, qo_off = l_row * qo_stride + 16 * l_piece;
  {
    uint16_t* st_q = v_area + 2 * FW_TILE + wave * (32 * D);
    u32x4 rq[NB][NLD], cs[PAIR || IMAGES ? 1 : NB][IMAGES ? 1 : KS / 2][4];
    const __amdgpu_buffer_rsrc_t q_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)((const uint16_t*)a.q + qo_at), 0, qo_bytes, 0x00020000);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int i = 0; i < NLD; ++i)
        rq[nb][i] = IMAGES ? pc_load_once((const u32x4*)((const uint16_t*)a.q + row_at(min(pos0 + 32 * nb + RPL * i + l_row, seq_rows - 1)) * D + 8 * l_piece))
                           : __builtin_amdgcn_raw_buffer_load_b128(q_rsrc, qo_off, RPL * i * qo_stride + nb * nb_step, PC_BUF_NT);
    const __amdgpu_buffer_rsrc_t t_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)a.table, 0, HALF * a.table_rows * 8, 0x00020000);
    const int t_off = 16 * (4 * hf * a.table_rows + pos0 + n);
#pragma unroll
    for (int nb = 0; nb < (IMAGES ? 0 : PAIR ? 1 : NB); ++nb)
#pragma unroll
      for (int ks = 0; ks < (IMAGES ? 0 : KS / 2); ++ks)
#pragma unroll
        for (int e = 0; e < 4; ++e) cs[nb][ks][e] = __builtin_amdgcn_raw_buffer_load_b128(t_rsrc, t_off, 16 * (8 * ks + e) * a.table_rows + 512 * nb, 0);
    __builtin_amdgcn_sched_barrier(0);
    if (!IMAGES || T > 0) { FW_LOAD4(FW_LOAD_K, 0); FW_LOAD4(FW_LOAD_V, 0); }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)                          // (O is cleared while they are on their way)
#pragma unroll
      for (int db = 0; db < DB; ++db) {
#pragma unroll
        for (int r = 0; r < 16; ++r) o_acc[nb][db][r] = 0.f;
        asm volatile("" : "+a"(o_acc[nb][db]));
      }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      if (nb) PC_FA_WAVE_LDS_SYNC();
#pragma unroll
      for (int i = 0; i < NLD; ++i) {
        const int r = RPL * i + l_row;
        *(u32x4*)(st_q + (r * PPR + (l_piece ^ (r % PPR))) * 8) = rq[nb][i];
      }
      PC_FA_WAVE_LDS_SYNC();
      if (nb == 0) {
        __builtin_amdgcn_sched_barrier(0);
        if (!IMAGES || T > 0) {
          if (IMAGES) { walk_next(); lim1 = cur.lim; }
          FW_LOAD4(FW_LOAD_K, 1); FW_LOAD4(FW_LOAD_V, 1);
          if (IMAGES) { walk_next(); lim2 = cur.lim; }
          FW_LOAD4(FW_LOAD_K, 2);
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      auto piece = [&](int p) __attribute__((always_inline)) { return *(const u32x4*)(st_q + (n * PPR + (p ^ (n % PPR))) * 8); };
#pragma unroll
      for (int ks = 0; ks < (IMAGES ? KS : 0); ++ks) {
        const u32x4 x = piece(2 * ks + hf);
        bq[nb][ks] = *(const bf16x8*)&x;
      }
#pragma unroll
      for (int ks = 0; ks < (IMAGES ? 0 : KS / 2); ++ks) {
        const u32x4 x1 = piece(2 * ks + hf), x2 = piece(2 * ks + hf + PPR / 2);
        u32x4 ra, rbv;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const u32x4 cw = cs[PAIR ? 0 : nb][ks][e];
          const float c0x = __uint_as_float(cw[0]), c0y = __uint_as_float(cw[1]), c1x = __uint_as_float(cw[2]), c1y = __uint_as_float(cw[3]);
          const float x1l = bf16_lo_to_f32(x1[e]), x1h = bf16_hi_to_f32(x1[e]);
          const float x2l = bf16_lo_to_f32(x2[e]), x2h = bf16_hi_to_f32(x2[e]);
          ra[e] = pack_bf16x2(x1l * c0x - x2l * c0y, x1h * c1x - x2h * c1y);
          rbv[e] = pack_bf16x2(x2l * c0x + x1l * c0y, x2h * c1x + x1h * c1y);
        }
        bq[nb][ks] = *(bf16x8*)&ra;
        bq[nb][ks + KS / 2] = *(bf16x8*)&rbv;
      }
    }
  }
  floatx16 negm[NB], s_buf[2][NB];                           // -reference, the C operand of every S^T; [step parity] S^T
  u32x4 p_buf[2][NB][2];                                     // [step parity] P^T
  bf16x8 ka[KS], va[2][DB];
  float m_run[NB] = {0.f, 0.f}, l_run[NB] = {0.f, 0.f}, dl_run[NB] = {0.f, 0.f};
  bool far = false;                                          // a sum beyond PC_FW_FAR was scaled down
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
#pragma unroll
    for (int r = 0; r < 16; ++r) negm[nb][r] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(bq[nb][ks]));
  }
  auto o_settle = [&]() __attribute__((always_inline)) {     // O^T may be read by others than the matrix pipe
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      asm volatile("s_nop 15" : "+a"(o_acc[nb][0]), "+a"(o_acc[nb][1]), "+a"(o_acc[nb][2]), "+a"(o_acc[nb][3]));
  };
  auto pv = [&](int i, const u32x4(&p)[NB][2]) __attribute__((always_inline)) {
    const int ts = i / (NB * DB), db = (i / NB) % DB, nb = i % NB;
    if (i == 0) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(o_acc[nb][db]) : "v"(va[ts][db]), "v"(p[nb][ts]));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(o_acc[nb][db]) : "v"(va[ts][db]), "v"(p[nb][ts]));
  };
  const int krow = pc_key_of_row(n);
  int k_base = (hf * 64 + krow) * 8, v_base = (hf * D + n) * 8;
  auto read_k = [&](int t, int half, int ks) __attribute__((always_inline)) {
    return *(const bf16x8*)(smem + (t & 3) * FW_TILE + 32 * 8 * half + k_base + 2 * ks * 64 * 8);
  };
  auto read_v = [&](int t, int half, int i) __attribute__((always_inline)) {
    return *(const bf16x8*)(v_area + (t & 3) * FW_TILE + 4 * half * D * 8 + v_base + 2 * (i / DB) * D * 8 + 32 * (i % DB) * 8);
  };
  using yes = std::integral_constant<bool, true>;
  using no = std::integral_constant<bool, false>;

  // The probabilities of a step in NG groups: exp2 of element gr, sum, maximum and pack of the one before (element e:
  // register e % 16 of block e / 16)
  constexpr int NG = 16 * NB + 1;
  auto prob_group = [&](int gr, const floatx16(&s)[NB], float(&pr)[16 * NB], float(&t)[NB], float(&mx)[NB], u32x4(&p)[NB][2]) __attribute__((always_inline)) {
    if (gr < 16 * NB) asm volatile("v_exp_f32 %0, %1" : "=v"(pr[gr]) : "v"(s[gr / 16][gr % 16]));
    if (gr >= 1) {
      const int e = gr - 1, nb = e / 16, r = e % 16;
      if (r == 1) asm volatile("v_add_f32 %0, %1, %2" : "=v"(t[nb]) : "v"(pr[e - 1]), "v"(pr[e]));
      if (r > 1) asm volatile("v_add_f32 %0, %0, %1" : "+v"(t[nb]) : "v"(pr[e]));
      if (r == 2) asm volatile("v_max3_f32 %0, %1, %2, %3" : "=v"(mx[nb]) : "v"(pr[e - 2]), "v"(pr[e - 1]), "v"(pr[e]));
      if (r > 2 && r % 2 == 0) asm volatile("v_max3_f32 %0, %0, %1, %2" : "+v"(mx[nb]) : "v"(pr[e - 1]), "v"(pr[e]));
      if (r == 15) asm volatile("v_max_f32 %0, %0, %1" : "+v"(mx[nb]) : "v"(pr[e]));
      if (r % 2 == 1) {
        uint32_t w;
        asm volatile("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(w) : "v"(pr[e - 1]), "v"(pr[e]));
        p[nb][r / 8][(r % 8) / 2] = w;
      }
    }
  };
  // What rounding to bf16 added to the heaviest probability of every lane's 16 goes into the output's row sum (dl_run), a
  // step later, in seven parts.  The products take probabilities rounded, t sums them as they are (the
  // logsumexp needs that), and a reference that stays behind leaves the heaviest one no power of two: its rounding would be an
  // error of the weights' sum.  Error against 64 bits on the same operands, as a multiple of what the roundings of
  // probabilities and outputs cost, deviation of the logits 1 / 4 / 8 / 16: flash_workgroup 1.00 / 1.10 / 1.11 / 1.00, without
  // this 1.00 / 1.23 / 1.29 / 1.22, with it 0.99 / 0.99 / 0.98 / 0.88, with all rounded probabilities summed
  // 1.00 / 1.00 / 0.98 / 0.88.  16 x 8192 rows, 32 / 8 heads, with the pre-pass 7000 -> 7180 us; all of them
  // by v_dot2_f32_bf16 8030 (it waits for the matrix pipe), the parts in one slice of the step 7250.
  float heavy[NB] = {0.f, 0.f}, was[NB];
  uint32_t heavy_w;
  auto round_part = [&](int i) __attribute__((always_inline)) {
    if (i == 0) asm volatile("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(heavy_w) : "v"(heavy[0]), "v"(heavy[1]));
    if (i == 1) asm volatile("v_lshlrev_b32 %0, 16, %1" : "=v"(was[0]) : "v"(heavy_w));
    if (i == 2) asm volatile("v_and_b32 %0, 0xffff0000, %1" : "=v"(was[1]) : "v"(heavy_w));
    if (i == 3 || i == 4) asm volatile("v_sub_f32 %0, %0, %1" : "+v"(was[i - 3]) : "v"(heavy[i - 3]));
    if (i == 5 || i == 6) asm volatile("v_add_f32 %0, %0, %1" : "+v"(dl_run[i - 5]) : "v"(was[i - 5]));
  };
  // k0: the step's first key (IMAGES: counted from the tile's first)
  auto mask_step = [&](int k0, const Limit& lim, floatx16(&s)[NB]) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int key = k0 + 16 * (r / 8) + 8 * hf + (r % 8);
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        if (key > (IMAGES ? min(lim.cut - 1, max_key[nb] - lim.c0) : max_key[nb])) s[nb][r] = -INFINITY;
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  // Step j: the products and reads of flash_workgroup's step without its row maxima.  The probabilities are taken against
  // the reference as it stands; whether one left its window shows in the step's sums.  Slices 0 to 15 are the P V products of step j - 1 with the reads of
  // the next keys, 16 to 31 the S^T products of step j + 1 with the reads of V^T(j), reads in the odd ones, where
  // the groups are light; the tile loads in even ones.  The last groups are doubled up so that the test of the sums
  // has its answer at the end.  BAR: the first step of a period waits for the tiles of the period behind
  // its first product.  LD: tile t_ld is asked for, 1 K, 2 V.
  // A rescale holds up all four wavefronts (200 cycles a tile on average with a window of 2^8 and logits of deviation
  // 2): PC_FA_WINDOW is wide.
  auto step = [&](auto mask_tag, auto has_qk, auto bar_tag, auto ld_tag, const Limit& lim, int j, int t_ld, floatx16(&s_cur)[NB],
                  floatx16(&s_next)[NB], u32x4(&p_cur)[NB][2], const u32x4(&p_prev)[NB][2]) __attribute__((always_inline)) {
    constexpr bool MASK = decltype(mask_tag)::value, QK = decltype(has_qk)::value, BAR = decltype(bar_tag)::value;
    constexpr int LD = decltype(ld_tag)::value;
    float t[NB], mx[NB], pr[16 * NB], most = 0.f;            // the step's sums, maxima and probabilities
    if (MASK) mask_step(IMAGES ? 32 * (j & 1) : 32 * j, lim, s_cur);
#pragma unroll
    for (int i = 0; i < 2 * NM; ++i) {
      if (i < NM) {
        pv(i, p_prev);
        if (BAR && i == 0) {
          PC_WAIT_VMCNT(2 * T_LD);
          __builtin_amdgcn_s_barrier();
        }
        if (QK && i % 2 == 1) ka[i / 2] = read_k((j + 1) >> 1, (j + 1) & 1, i / 2);
        if (LD == 1) {
          if (i == 4) FW_LOAD_K(t_ld, 0);
          if (i == 6) FW_LOAD_K(t_ld, 1);
          if (i == 8) FW_LOAD_K(t_ld, 2);
          if (i == 10) FW_LOAD_K(t_ld, 3);
        } else if (LD == 2) {
          if (i == 4) FW_LOAD_V(t_ld, 0);
          if (i == 6) FW_LOAD_V(t_ld, 1);
          if (i == 8) FW_LOAD_V(t_ld, 2);
          if (i == 10) FW_LOAD_V(t_ld, 3);
        }
      } else {
        const int i2 = i - NM, ks = i2 / NB, nb = i2 % NB;
        if (QK) {                                            // (the first as text too: its C operand, -reference, stays where it is)
          if (ks == 0) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" : "=&v"(s_next[nb]) : "v"(ka[0]), "a"(bq[nb][0]), "v"(negm[nb]));
          else s_next[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[ks], bq[nb][ks], s_next[nb], 0, 0, 0);
        }
        if (i2 % 2 == 1) va[i2 / 2 / DB][i2 / 2 % DB] = read_v(j >> 1, j & 1, i2 / 2);
      }
      if (i < 2 * NM - 1) prob_group(i <= 28 ? i : i == 29 ? 30 : 31, s_cur, pr, t, mx, p_cur);
      if (i == 28 || i == 30) prob_group(i == 28 ? 29 : 32, s_cur, pr, t, mx, p_cur);
      if (i == 2 * NM - 1) {
        asm volatile("v_max_f32 %0, %1, %2" : "=v"(most) : "v"(t[0]), "v"(t[1]));
      }
      if (i < 14 && i % 2 == 0) round_part(i / 2);           // of the step before
      __builtin_amdgcn_sched_barrier(0);
    }
    // some row's maximum exceeds its reference by more than 86, or a segment begins (see flash_workgroup): every row whose
    // maximum exceeds its reference moves (only those beyond 6: the same time at deviations from 1 to 32)
    if (__any(most > PC_FA_WINDOW) || (IMAGES && lim.seg_start)) {
      far |= !IMAGES || __any(fmaxf(most, fmaxf(l_run[0], l_run[1])) > PC_FW_FAR);
      o_settle();
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        float tm = s_cur[nb][0];
#pragma unroll
        for (int r = 1; r < 16; ++r) tm = fmaxf(tm, s_cur[nb][r]);
        mx[nb] = tm;
        tm = pc_xhalf_max(tm);
        const float delta = fmaxf(tm, 0.f), alpha = __builtin_amdgcn_exp2f(-delta);
        m_run[nb] += delta;
        l_run[nb] *= alpha;
        dl_run[nb] *= alpha;
        mx[nb] = __builtin_amdgcn_exp2f(mx[nb] - delta);
        t[nb] = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          negm[nb][r] -= delta;
          if (QK) s_next[nb][r] -= delta;
          pr[16 * nb + r] = __builtin_amdgcn_exp2f(s_cur[nb][r] - delta);
          t[nb] += pr[16 * nb + r];
          if (r % 2 == 1) p_cur[nb][r / 8][(r % 8) / 2] = pack_bf16x2(pr[16 * nb + r - 1], pr[16 * nb + r]);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int db = 0; db < DB; ++db) {
#pragma unroll
          for (int r = 0; r < 16; ++r) o_acc[nb][db][r] *= alpha;
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) { l_run[nb] += t[nb]; heavy[nb] = mx[nb]; }
    __builtin_amdgcn_sched_barrier(0);
  };

  if (!IMAGES || T > 0) {                                    // (IMAGES: a part, or rows, without any key)
  // K 0 and V 0 have landed, and every wavefront has left its staging area: V 2 may move in
  PC_WAIT_VMCNT(3 * T_LD);
  __builtin_amdgcn_s_waitcnt(0xC07F);                        // (LDS)
  __builtin_amdgcn_s_barrier();
  FW_LOAD4(FW_LOAD_V, 2);
  // ---- step 0: its row maxima are the first reference
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) ka[ks] = read_k(0, 0, ks);
#pragma unroll
  for (int ks = 0; ks < KS; ++ks)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      s_buf[0][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[ks], bq[nb][ks], ks == 0 ? negm[nb] : s_buf[0][nb], 0, 0, 0);
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) ka[ks] = read_k(0, 1, ks);
  mask_step(0, lim0, s_buf[0]);
  {
    float t[NB], mx[NB], pr[16 * NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      float tm = s_buf[0][nb][0];
#pragma unroll
      for (int r = 1; r < 16; ++r) tm = fmaxf(tm, s_buf[0][nb][r]);
      tm = pc_xhalf_max(tm);
      m_run[nb] = tm != -INFINITY ? tm : 0.f;
#pragma unroll
      for (int r = 0; r < 16; ++r) { negm[nb][r] = -m_run[nb]; s_buf[0][nb][r] -= m_run[nb]; }
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NM; ++i) {
      const int ks = i / NB, nb = i % NB;
      s_buf[1][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[ks], bq[nb][ks], ks == 0 ? negm[nb] : s_buf[1][nb], 0, 0, 0);
      if (i < KS) va[i / DB][i % DB] = read_v(0, 0, i);
#pragma unroll
      for (int gr = (i * NG + NM - 1) / NM; gr < ((i + 1) * NG + NM - 1) / NM; ++gr) prob_group(gr, s_buf[0], pr, t, mx, p_buf[0]);
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) { l_run[nb] = t[nb]; heavy[nb] = mx[nb]; }
  }
  // Period p: steps 2p + 1 and 2p + 2 over K tile p + 1 and V^T tiles p and p + 1.  Tile p + 3 moves into the slots
  // of tile p - 1, last read in front of the period's barrier; two periods of loads (8 instructions) may be in flight
  // there (one: 2560 cycles a tile instead of 2500, in an earlier build).
  auto period = [&](auto mask_tag, int p) __attribute__((always_inline)) {
    asm volatile("" : "+v"(k_base), "+v"(v_base));
    if (IMAGES) { walk_next(); lim0.seg_start = false; }     // the walk is on tile p + 3
    step(mask_tag, yes{}, yes{}, std::integral_constant<int, 1>{}, lim0, 2 * p + 1, p + 3, s_buf[1], s_buf[0], p_buf[1], p_buf[0]);
    step(mask_tag, yes{}, no{}, std::integral_constant<int, 2>{}, lim1, 2 * p + 2, p + 3, s_buf[0], s_buf[1], p_buf[0], p_buf[1]);
    lim0 = lim1; lim1 = lim2; lim2 = cur.lim;
  };
  const int n_plain = IMAGES ? run_full - 1 : min(T - 1, max(0, (J0 - 1) / 2));       // periods whose steps need no mask
  // Last step with a key visible to any row of this wavefront; periods behind it keep up loads and barriers only
  const int j_need = IMAGES ? 2 * T - 1 : min(pos0 + POS_W - 1, seq_rows - 1) >> 5;
  const int n_periods = min(T - 1, (j_need + 1) / 2);
  int p = 0;
  for (; p < min(n_plain, n_periods); ++p) period(no{}, p);
  for (; p < n_periods; ++p) period(yes{}, p);
  for (; p < T - 1; ++p) {
    PC_WAIT_VMCNT(2 * T_LD);
    __builtin_amdgcn_s_barrier();
    FW_LOAD4(FW_LOAD_K, p + 3);
    FW_LOAD4(FW_LOAD_V, p + 3);
  }
  PC_WAIT_VMCNT(0);
  __syncthreads();
  // does the last tile's second half hold a key that some row of the wavefront sees?
  lim0.seg_start = false;
  if (IMAGES ? __builtin_amdgcn_readfirstlane(min(lim0.cut - 1, pc_div(min(pos0 + 63, seq_rows - 1), a.group_div) - lim0.c0)) >= 32 : j_need >= 2 * T - 1) {
    step(yes{}, no{}, no{}, std::integral_constant<int, 0>{}, lim0, 2 * T - 1, 0, s_buf[1], s_buf[0], p_buf[1], p_buf[0]);
#pragma unroll
    for (int i = 0; i < NB * 2; ++i) p_buf[0][i / 2][i % 2] = p_buf[1][i / 2][i % 2];
  }
  // P V of the last step that ran (one place for both: with two the compiler copies O^T in front of the products)
#pragma unroll
  for (int i = 0; i < NM; ++i) pv(i, p_buf[0]);
  o_settle();
#pragma unroll
  for (int i = 0; i < 7; ++i) round_part(i);

  // ---- O^T beyond fp32, which a reference far behind a row's maximum allows for large values: the
  //      wavefront takes its rows once more, straight from the tile images, with references that follow the maxima.  Then
  //      probabilities are at most 1, and values up to 2^107 (2^20 keys) have finite sums.
  if (far || __any(fmaxf(l_run[0], l_run[1]) > PC_FW_FAR)) {
    float z = 0.f;                                           // NaN if some element is no number
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) z = fmaf(o_acc[nb][db][r], 0.f, z);
    if (__any(z != z)) {
      if (IMAGES) walk_begin();
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) {
        m_run[nb] = l_run[nb] = dl_run[nb] = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) negm[nb][r] = 0.f;
#pragma unroll
        for (int db = 0; db < DB; ++db) {
#pragma unroll
          for (int r = 0; r < 16; ++r) o_acc[nb][db][r] = 0.f;
          asm volatile("" : "+a"(o_acc[nb][db]));
        }
      }
#pragma unroll 1
      for (int j = 0; j < (IMAGES ? 2 * T : j_need + 1); ++j) {
        if (IMAGES && j > 0 && j % 2 == 0) walk_next();
        const long long at = img0 + (long long)(j >> 1) * FW_TILE;
        const uint16_t* kt = (IMAGES ? cur.k : (const uint16_t*)a.k_img + at) + 32 * 8 * (j & 1) + k_base;
        const uint16_t* vt = (IMAGES ? cur.v : (const uint16_t*)a.v_img + at) + 4 * (j & 1) * D * 8 + v_base;
#pragma unroll
        for (int i = 0; i < KS; ++i) {
          ka[i] = *(const bf16x8*)(kt + 2 * i * 64 * 8);
          va[i / DB][i % DB] = *(const bf16x8*)(vt + 2 * (i / DB) * D * 8 + 32 * (i % DB) * 8);
        }
#pragma unroll
        for (int i = 0; i < NM; ++i)
          s_buf[0][i % NB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ka[i / NB], bq[i % NB][i / NB], i < NB ? negm[i % NB] : s_buf[0][i % NB], 0, 0, 0);
        mask_step(IMAGES ? 32 * (j & 1) : 32 * j, cur.lim, s_buf[0]);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
          float tm = s_buf[0][nb][0];
#pragma unroll
          for (int r = 1; r < 16; ++r) tm = fmaxf(tm, s_buf[0][nb][r]);
          tm = pc_xhalf_max(tm);
          const float delta = j > 0 ? fmaxf(tm, 0.f) : tm != -INFINITY ? tm : 0.f, alpha = j > 0 ? __builtin_amdgcn_exp2f(-delta) : 1.f;
          m_run[nb] += delta;
          l_run[nb] *= alpha;
          dl_run[nb] *= alpha;
#pragma unroll
          for (int r = 0; r < 16; r += 2) {
            negm[nb][r] = negm[nb][r + 1] = -m_run[nb];
            const float p0 = __builtin_amdgcn_exp2f(s_buf[0][nb][r] - delta), p1 = __builtin_amdgcn_exp2f(s_buf[0][nb][r + 1] - delta);
            const uint32_t w = pack_bf16x2(p0, p1);
            p_buf[0][nb][r / 8][r % 8 / 2] = w;
            l_run[nb] += p0 + p1;
            dl_run[nb] += (bf16_lo_to_f32(w) - p0) + (bf16_hi_to_f32(w) - p1);
          }
#pragma unroll
          for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) o_acc[nb][db][r] *= alpha;
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < NM; ++i) pv(i, p_buf[0]);
        o_settle();
      }
    }
  }
  }
  // ---- epilogue, as flash_workgroup's: whole rows through the K slots (nobody reads K any more)
  static_assert(4 * 32 * D <= PC_FW_RING * FW_TILE, "staging area is the K slots");
  uint16_t* st_o = smem + wave * (32 * D);
  int l_out = lane;                                          // (IMAGES: no addresses kept across the loop)
  if (IMAGES) asm volatile("" : "+v"(l_out));
  const int n_out = l_out % 32, hf_out = l_out / 32, row_out = l_out / PPR, piece_out = l_out % PPR;
  const __amdgpu_buffer_rsrc_t o_rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)((uint16_t*)a.o + qo_at), 0, qo_bytes, 0x00020000);
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const float l = pc_xhalf_sum(l_run[nb]);
    const float inv_l = l > 0.f ? 1.f / (l + pc_xhalf_sum(dl_run[nb])) : 0.f;
    const float lse = l > 0.f ? m_run[nb] * PC_LN2 + logf(l) : -INFINITY;
    if (IMAGES && a.n_parts > 1) {                           // a partial result for the merge
      const int row = pos0 + 32 * nb + n_out;
      if (row < seq_rows) {
        const int query = pc_div(row, a.group_div);
        const long long prow = (((long long)seq * a.n_parts + turn) * a.n_rows + query) * a.n_q_heads + h + row - query * a.group;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            floatx4 x = {o_acc[nb][db][4 * i] * inv_l, o_acc[nb][db][4 * i + 1] * inv_l, o_acc[nb][db][4 * i + 2] * inv_l, o_acc[nb][db][4 * i + 3] * inv_l};
            *(floatx4*)(a.part_o + prow * D + 32 * db + 8 * i + 4 * hf_out) = x;
          }
        if (hf_out == 0) a.part_lse[prow] = lse;
      }
      continue;
    }
    if (nb) PC_FA_WAVE_LDS_SYNC();
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        uint2 x;
        x.x = pack_bf16x2(o_acc[nb][db][4 * i] * inv_l, o_acc[nb][db][4 * i + 1] * inv_l);
        x.y = pack_bf16x2(o_acc[nb][db][4 * i + 2] * inv_l, o_acc[nb][db][4 * i + 3] * inv_l);
        const int q = 4 * db + i;
        *(uint2*)(st_o + (n_out * PPR + (q ^ (n_out % PPR))) * 8 + 4 * hf_out) = x;
      }
    PC_FA_WAVE_LDS_SYNC();
#pragma unroll
    for (int k = 0; k < NLD; ++k) {
      const int r = RPL * k + row_out;
      const u32x4 x = *(const u32x4*)(st_o + (r * PPR + (piece_out ^ (r % PPR))) * 8);
      if (!IMAGES) {
        __builtin_amdgcn_raw_buffer_store_b128(x, o_rsrc, qo_off, RPL * k * qo_stride + nb * nb_step, PC_BUF_NT);
        continue;
      }
      const int row = pos0 + 32 * nb + r;
      if (row < seq_rows) pc_store_once((u32x4*)((uint16_t*)a.o + row_at(row) * D + 8 * piece_out), x);
    }
    const int row = pos0 + (PAIR ? 0 : 32 * nb) + n_out;
    if (row < seq_rows && hf_out == 0 && a.lse) {
      if (IMAGES) a.lse[((long long)seq * a.n_q_heads + h + pc_mod(row, a.group, a.group_div)) * a.n_rows + pc_div(row, a.group_div)] = lse;
      else a.lse[((long long)seq * a.n_q_heads + h + (PAIR ? nb : 0)) * a.n_rows + row] = lse;
    }
  }
#undef FW_LOAD_K
#undef FW_LOAD_V
#undef FW_LOAD4
}
