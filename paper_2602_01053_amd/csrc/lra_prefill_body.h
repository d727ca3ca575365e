// Body of the tile-walking prefill kernels, included inside each of them (lra_prefill_mfma.hip) with the template
// parameters and POOL in scope.  Text rather than a function: the register allocation of the rank-64 forms, which fill
// the register file, comes out without scratch memory for prefill_mfma_kernel on contiguous caches only when the body
// stands in the kernel itself (12 to 16 bytes for far paged pools), for prefill_pool_kernel only when it comes through
// a function.
  static_assert(!(ROPE_K && HAS_BK), "the rotary key side replaces the Qt term");
  // Completed keys K_base + RoPE(L B_K) are held as fp16, whether the key pre-pass left them in the workspace
  // (KC16) or this kernel completes the tiles in LDS (ROPE_K): rounding the sum to bf16 a second time costs
  // 2.5e-3 to 4e-3 of relative error in the output on its own, fp16 (three more bits) a quarter of that.
  // The scores are then an fp16 product, with Q converted once in the prologue (exact for a bf16 Q of
  // ordinary magnitudes); V, L and the probabilities stay bf16.
  constexpr bool KF16 = ROPE_K || KC16;
  static_assert(!(KC16 && (HAS_BK || ROPE_K)), "pre-pass keys: nothing left to add");
  constexpr int BM = 128, BN = 64;
  constexpr int KS = D / 16;   // k-steps of S^T over the head dimension
  constexpr int RKS = RP / 16; // k-steps over the padded rank
  constexpr int DB = D / 32;   // 32-row blocks of O^T
  constexpr int RB = (RP + 31) / 32;  // 32-row blocks of Olr^T
  constexpr int KCH = D / 8;          // 16-byte chunks per K/V row
  constexpr int LCH = RP / 8;         // 16-byte chunks per L row (2, 4 or 8)
  constexpr int K_BYTES = BN * D * 2;
  constexpr int L_BYTES = BN * RP * 2;
  constexpr int STAGE = 2 * K_BYTES + L_BYTES;
  // With a half-empty last 32-row block of Olr^T (rank 16 or 48 after padding), its idle
  // upper lanes read a constant [1, 0, 0, 0] instead of L, so the matrix core also
  // accumulates the softmax row sums.
  constexpr bool ONES_ROW = (RP % 32) != 0;
  constexpr int ONES_AT = 2 * STAGE;

  __shared__ __align__(16) unsigned char smem[2 * STAGE + (ONES_ROW ? 16 : 0)];
  // rotary key side: revolutions per position of every rotary pair (double, and rounded to float for
  // the offsets inside a tile), and the angle of the first key of a tile (fraction of a revolution),
  // double-buffered like the stages
  __shared__ double rope_rate[ROPE_K ? D / 2 : 1];
  __shared__ __align__(16) float rope_rate_f[ROPE_K ? D / 2 : 4];
  __shared__ __align__(16) float rope_fr0[2][ROPE_K ? D / 2 : 4];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, g2 = lane >> 5;
  const int Hq = p.n_q_heads, Hkv = p.n_kv_heads, r = p.rank;
  const int G = p.tile_group;  // q heads whose rows share a q tile: all of a kv head's, or one

  // workgroup -> (kv head, first of the tile's q heads, q tile); consecutive ids go to consecutive XCDs
  const int lin = blockIdx.x;
  const int rest = lin / Hkv, hk = lin - rest * Hkv;
  int qt = rest;
  int head_first = hk * p.group;
  if (p.tile_heads > 1) {  // (the quotient by one is not worth its instructions in a call of one tile per workgroup)
    qt = rest / p.tile_heads;
    head_first += (rest - qt * p.tile_heads) * G;
  }
  const int n_rows = p.n_new * G;                  // query rows of these heads: (new token, q head), the q head fastest
  {
    // Causal q tiles differ in length (tile i walks the keys up to its diagonal).  The 256 compute units take
    // workgroups in rounds of 256; a unit that holds two workgroups holds number k and number k + 256.  Every other
    // round walks its q tiles backwards, so the long tiles of one round sit next to the short tiles of the next
    // and the units finish together.
    const int q_tiles = (n_rows + BM - 1) / BM;
    const int tpr = p.tiles_per_round;
    if (q_tiles > tpr) {
      const int round = qt / tpr, pos = qt - round * tpr;
      const int cnt = min(tpr, q_tiles - round * tpr);
      if ((round & 1)) qt = round * tpr + (cnt - 1 - pos);
    }
  }
  const int t = p.seq_index;
  const int a_idx = p.adapter_index;
  const int n_t = min(PF_CONST_I32(p.seq_lens)[t], p.max_seq_len);
  const int n_new = p.n_new;
  const int q0 = qt * BM;
  if (q0 >= n_rows) return;
  const int base_vis = n_t - n_new;  // new token i sees keys 0 .. base_vis + i
  // First new token of the tile, how many of its q heads lie in the tile before, and the live rows of the tile.  A
  // lane's row is in_tile = 32 wave + l32 rows further: token tok0 + (head0 + in_tile) / G, the quotient (of at most
  // 143 by at most 16) taken exactly by a multiplication, so that it is cheap to form again wherever it is needed:
  // kept in registers through the loop it sent the rank-64 kernels to scratch memory (the three small numbers
  // travel in one scalar register for the same reason).
  const int tok0 = G > 1 ? __builtin_amdgcn_readfirstlane(q0 / G) : q0;
  const int row_map = (q0 - tok0 * G) | (min(BM, n_rows - q0) << 4) | (p.row_mul << 12);
  // (token - tok0, q head of the group) of a row of the tile; false (and the last live row) for one past the end
  auto map_row = [&](int in_tile, int& tok, int& gq) __attribute__((always_inline)) -> bool {
    int m = row_map;
    // (not at d = 64, rank 64 with a Qt term, where the kernel has registers left and, with this barrier to its
    // scheduling, walked a tile alone on its unit in 1.25 times the time)
    if constexpr (!(D == 64 && RP == 64 && HAS_BK)) asm volatile("" : "+s"(m), "+v"(in_tile));
    const int at = (m & 15) + min(in_tile, ((m >> 4) & 255) - 1);
    tok = (at * (m >> 12)) >> 16;
    gq = at - tok * G;
    return in_tile < ((m >> 4) & 255);
  };
  // index of this lane's row in q, out and the workspace; -1: a row past the end, never stored
  auto global_row = [&](bool clamped) __attribute__((always_inline)) -> int {
    int tok, gq;
    const bool live = map_row(wave * 32 + (static_cast<int>(threadIdx.x) & 31), tok, gq);
    return live || clamped ? (tok0 + tok) * Hq + head_first + gq : -1;
  };
  auto token_of = [&](int in_tile) __attribute__((always_inline)) -> int {
    int tok, gq;
    map_row(in_tile, tok, gq);
    return tok0 + tok;
  };
  const int wave_first = __builtin_amdgcn_readfirstlane(base_vis + token_of(wave * 32));  // the smallest limit of this wave
  const int wg_last = __builtin_amdgcn_readfirstlane(base_vis + token_of(BM - 1));       // last key any row of the workgroup sees
  const int n_tiles = wg_last / BN + 1;
  // this workgroup's share of the q tile's key tiles: [tile_begin, tile_end)
  const int split = SPLIT ? blockIdx.y : 0;
  const int tile_begin = SPLIT ? static_cast<int>(static_cast<int64_t>(n_tiles) * split / p.n_splits) : 0;
  const int tile_end = SPLIT ? static_cast<int>(static_cast<int64_t>(n_tiles) * (split + 1) / p.n_splits) : n_tiles;
  if (SPLIT && tile_begin >= tile_end) {
    // more workgroups than key tiles: leave an empty state (zero row sum), all the merge
    // kernel looks at
    const int out_row = global_row(false);
    if (out_row >= 0 && g2 == 0) {
      const int64_t slot = static_cast<int64_t>(out_row) * p.n_splits + split;
      p.part_ml[slot * 2 + 0] = -INFINITY;
      p.part_ml[slot * 2 + 1] = 0.f;
      if (split == 0) p.part_adapter[out_row] = a_idx;
    }
    return;
  }

  // ---------------- tile traffic: HBM -> LDS, no registers in between ----------------
  const PfTileLoader<D, RP, PAGED, POOL> loader(p, smem, wave, lane, hk, t, n_t);
  auto issue_tile = [&](int j, int st) { loader.issue_tile(j, st * STAGE); };

  if (PAGED) loader.fetch_ids(tile_begin * (BN / 16));
  issue_tile(tile_begin * BN, 0);
  if (ONES_ROW && tid == 0) *reinterpret_cast<pf_u32x4*>(smem + ONES_AT) = pf_u32x4{0x00003f80u, 0u, 0u, 0u};

  // ---------------- rotary key side: B_K^T operands of E^T, rotation rates ----------------
  // Wave (pair set ps = wave / 2, key half kt_e = wave % 2); d = 128: feature blocks ps and ps + 2,
  // d = 64: blocks 0 and 1 (waves 2, 3 have nothing to do).  A operand of E^T = B_K^T . L^T: lane
  // (feature l32 of the block, half g2), element e <-> rho = 16ks + 8(e/4) + 4g2 + e%4, the order in
  // which the L operand is read below.
  constexpr int E_WAVES = ROPE_K ? 2 * (D / 64) : 0;
  const int fb_lo = D == 128 ? (wave >> 1) : 0, fb_hi = D == 128 ? (wave >> 1) + 2 : 1;
  const int kt_e = wave & 1;
  pf_bf16x8 bkt[2][ROPE_K ? RKS : 1];
  if (ROPE_K) {
    if (tid < D / 2) {  // read after the barrier that precedes the loop
      const double rate = rope_rate_rev(tid, D, p.key_rope_theta);
      rope_rate[tid] = rate;
      rope_rate_f[tid] = static_cast<float>(rate);
      double rev = static_cast<double>(tile_begin * BN) * rate;
      rev -= floor(rev);
      rope_fr0[0][tid] = static_cast<float>(rev);
    }
    if (wave < E_WAVES) {
      const int64_t ldb = static_cast<int64_t>(Hkv) * D;
      const bf16_t* bkg = static_cast<const bf16_t*>(p.b_k) + static_cast<int64_t>(a_idx) * r * ldb + hk * D;
      const bool has_b = p.b_k != nullptr;  // (a decode call may come without key-side adapters: nothing to add)
#pragma unroll
      for (int sel = 0; sel < 2; ++sel)
#pragma unroll
        for (int ks = 0; ks < RKS; ++ks) {
          uint32_t w4[4];
#pragma unroll
          for (int e2 = 0; e2 < 4; ++e2) {
            uint32_t pair = 0;
#pragma unroll
            for (int x = 0; x < 2; ++x) {
              const int e = 2 * e2 + x;
              const int rho = 16 * ks + 8 * (e >> 2) + 4 * g2 + (e & 3);
              const uint32_t v = (has_b && rho < r) ? bkg[rho * ldb + 32 * (sel == 0 ? fb_lo : fb_hi) + l32] : 0u;
              pair |= v << (16 * x);
            }
            w4[e2] = pair;
          }
          bkt[sel][ks] = pf_as_bf16x8(make_uint4(w4[0], w4[1], w4[2], w4[3]));
        }
    }
  }

  // ---------------- prologue: Q operands, Qt = Q B_K^T ----------------
  // qb[ks]: B operand of S^T: lane (row l32, k = 16ks + 8g2 + e)
  pf_bf16x8 qb[KS];
  {
    const bf16_t* qrow = static_cast<const bf16_t*>(p.q) + static_cast<int64_t>(global_row(true)) * D + g2 * 8;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qb[ks] = pf_as_bf16x8(*reinterpret_cast<const uint4*>(qrow + ks * 16));
  }
  pf_f16x8 qh[KF16 ? KS : 1];  // the same operands as fp16, for scores against fp16 keys
  if constexpr (KF16) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qh[ks] = pf_bf16x8_to_f16x8(qb[ks]);
  }
  // Qt^T[rho][row] = B_K[rho][:] . Q[row][:]: C layout lane (row l32; reg i <-> rho = 32b + 8(i/4) + 4g2 + i%4).
  // As B operand of the rank k-steps of S^T, k-step ks' takes registers 8ks'..8ks'+7 of
  // block b = ks'/2, i.e. element e <-> rho = 16ks' + 8(e/4) + 4g2 + e%4; the L operand
  // below is read in the same order.
  pf_bf16x8 qtb[RKS];
  if (HAS_BK) {
    const int64_t ldb = static_cast<int64_t>(Hkv) * D;
    const bf16_t* bkg = static_cast<const bf16_t*>(p.b_k);
    // rows of this adapter's B_K for kv head hk; rows past the rank (and everything when
    // there is no B_K) lie outside the resource and read as zero
    const __amdgpu_buffer_rsrc_t rs_b = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<bf16_t*>(bkg) + (bkg != nullptr ? static_cast<int64_t>(a_idx) * r * ldb + hk * D : 0), 0,
        bkg != nullptr ? static_cast<int>((static_cast<int64_t>(r - 1) * ldb + D) * 2) : 0, 0x00020000);
#pragma unroll
    for (int b = 0; b < RB; ++b) {
      pf_f32x16 acc;
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[i] = 0.f;
      const int rho = b * 32 + l32;
      const uint32_t boff = rho < r ? static_cast<uint32_t>(rho * ldb * 2 + g2 * 16) : kPfOob;
      pf_u32x4 bk[KS];
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) bk[ks] = __builtin_amdgcn_raw_buffer_load_b128(rs_b, boff, ks * 32, 0);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(pf_bf16x8, bk[ks]), qb[ks], acc, 0, 0, 0);
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const int ks2 = b * 2 + half;
        if (ks2 < RKS) {
          const int o = half * 8;
          qtb[ks2] = pf_as_bf16x8(make_uint4(pf_pack2(acc[o + 0], acc[o + 1]), pf_pack2(acc[o + 2], acc[o + 3]),
                                             pf_pack2(acc[o + 4], acc[o + 5]), pf_pack2(acc[o + 6], acc[o + 7])));
        }
      }
    }
  }

  // ---------------- per-lane LDS read offsets (stage 0; stage 1 is STAGE further) ----------------
  // K rows as A operand of S^T (ds_read_b128): key = 32kt + l32, logical chunk c = 2ks + g2
  // lives at chunk c ^ swizzle(key); row offset and swizzle occupy disjoint address bits,
  // so the address is k_pre ^ (c << 4) (+ kt * 32 rows)
  const int k_pre = l32 * (D * 2) + (pf_swz_k<D>(l32) << 4);
  // V^T as A operand of O^T (ds_read_b64_tr_b16): lane a of a 16-lane group addresses
  // row 4*g2 + a/4 (+ 8 for the second read) of the 16-key k-step, 8 bytes at
  // d = 32b + 16dsel + 4(a%4): chunk 4b + 2dsel + c0, half sub; the swizzle flips chunk
  // bits 2..3, so the address is v_pre ^ (b << 6) (+ row offsets)
  const int a16 = lane & 15;
  const int dsel = (lane >> 4) & 1;   // which 16 of the 32 output rows this 16-lane group produces
  const int vrow = 4 * g2 + (a16 >> 2);
  const int v_pre = K_BYTES + vrow * (D * 2) + ((((a16 & 3) >> 1) + 2 * dsel + pf_swz_v<D>(vrow)) << 4) + (a16 & 1) * 8;
  // L rows as A operand of S^T: two 8-byte pieces per k-step (chunks 2ks' and 2ks' + 1, half
  // g2); the swizzle of row 32kt + l32 does not depend on kt
  int l_rd[RKS][2];
#pragma unroll
  for (int ks = 0; ks < RKS; ++ks)
#pragma unroll
    for (int pc = 0; pc < 2; ++pc)
      l_rd[ks][pc] = 2 * K_BYTES + l32 * (RP * 2) + (((2 * ks + pc) ^ pf_swz_l<LCH>(l32)) << 4) + g2 * 8;
  // L^T as A operand of Olr^T: rows rho = 32b + 16dsel + 4(a%4) .. +3 of key vrow (+8 for the
  // second read; +16 per k-step does not change the swizzle).  In a half-empty last block
  // the upper 16 lanes read the constant [1, 0, 0, 0] instead: output row 32b + 16 then
  // accumulates the row sums; the rows after it are never used.
  int lt_rd[RB][2];
#pragma unroll
  for (int b = 0; b < RB; ++b)
#pragma unroll
    for (int hh = 0; hh < 2; ++hh) {
      const int key = vrow + 8 * hh;
      const int ch = 4 * b + 2 * dsel + ((a16 & 3) >> 1);
      lt_rd[b][hh] = 2 * K_BYTES + key * (RP * 2) + (((ch & (LCH - 1)) ^ pf_swz_l<LCH>(key)) << 4) + (a16 & 1) * 8;
    }
  const bool ones_lane = ONES_ROW && dsel == 1;  // in block RB - 1

  // ---------------- main loop ----------------
  pf_f32x16 o_acc[DB], lr_acc[RB];
#pragma unroll
  for (int b = 0; b < DB; ++b)
#pragma unroll
    for (int i = 0; i < 16; ++i) o_acc[b][i] = 0.f;
#pragma unroll
  for (int b = 0; b < RB; ++b)
#pragma unroll
    for (int i = 0; i < 16; ++i) lr_acc[b][i] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  const float sc = p.scale * 1.44269504088896340736f;
  // The running maximum is only raised when some row's tile maximum exceeds it by more than
  // kSlack (base-2 units): until then probabilities up to 2^kSlack are accumulated, which
  // fp32 sums and bf16 probabilities hold without loss, and the final division by the row
  // sum (taken with the same reference) cancels the factor exactly.
  constexpr float kSlack = 8.0f;
  constexpr int kReadAheadS = 8, kReadAheadPV = 6;

  pf_wait_vm0();
  __syncthreads();

  auto tile_step = [&](int tile, auto st_c) {
    constexpr int ST = decltype(st_c)::value;
    const int j = tile * BN;
    const unsigned char* ks_l = smem + ST * STAGE;  // K region; the V and L offsets are part of v_pre, l_rd, lt_rd
    const bool more = tile + 1 < tile_end;
    // the other stage was last read before the barrier that ended the previous tile; where
    // in the tile the requests are placed makes no measurable difference
    if (more) issue_tile(j + BN, ST ^ 1);

    if (ROPE_K) {
      if (wave < E_WAVES) {
        pf_f32x16 e_lo, e_hi;
#pragma unroll
        for (int i = 0; i < 16; ++i) e_lo[i] = e_hi[i] = 0.f;
#pragma unroll
        for (int ks = 0; ks < RKS; ++ks) {
          const uint2 lo = *reinterpret_cast<const uint2*>(ks_l + l_rd[ks][0] + kt_e * 32 * RP * 2);
          const uint2 hi = *reinterpret_cast<const uint2*>(ks_l + l_rd[ks][1] + kt_e * 32 * RP * 2);
          const pf_bf16x8 lop = pf_as_bf16x8(make_uint4(lo.x, lo.y, hi.x, hi.y));
          e_lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bkt[0][ks], lop, e_lo, 0, 0, 0);
          e_hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bkt[1][ks], lop, e_hi, 0, 0, 0);
        }
        // register i of this lane: key 32 kt_e + l32 of the tile (position j + that), features
        // 32 fb + 8 (i/4) + 4 g2 + i%4 of blocks fb_lo, fb_hi: pair index = the fb_lo feature
        // Angle of (key, pair) in revolutions: that of the tile's first key, kept in double precision
        // by the table threads, plus the key's offset in the tile times the rate (at most 63 x 0.16
        // revolutions: single precision holds it to 1e-6).
        const int key = 32 * kt_e + l32;
        const float key_f = static_cast<float>(key);
        unsigned char* krow = smem + ST * STAGE + key * (D * 2) + 8 * g2;
        const int swz = pf_swz_k<D>(key);
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int dd0 = 32 * fb_lo + 8 * q4 + 4 * g2;
          const pf_f32x4 fr0 = *reinterpret_cast<const pf_f32x4*>(&rope_fr0[ST][dd0]);
          const pf_f32x4 rt = *reinterpret_cast<const pf_f32x4*>(&rope_rate_f[dd0]);
          float lo4[4], hi4[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int i = 4 * q4 + e;
            const float fr = fmaf(key_f, rt[e], fr0[e]);
            const float sn = __builtin_amdgcn_sinf(fr), cs = __builtin_amdgcn_cosf(fr);
            lo4[e] = e_lo[i] * cs - e_hi[i] * sn;
            hi4[e] = e_hi[i] * cs + e_lo[i] * sn;
          }
#pragma unroll
          for (int sel = 0; sel < 2; ++sel) {
            const float* add = sel == 0 ? lo4 : hi4;
            uint2* at = reinterpret_cast<uint2*>(krow + (((4 * (sel == 0 ? fb_lo : fb_hi) + q4) ^ swz) << 4));
            const uint2 old = *at;
            *at = make_uint2(pf_pack2_f16(__uint_as_float(old.x << 16) + add[0], __uint_as_float(old.x & 0xffff0000u) + add[1]),
                             pf_pack2_f16(__uint_as_float(old.y << 16) + add[2], __uint_as_float(old.y & 0xffff0000u) + add[3]));
          }
        }
      }
      __syncthreads();  // the completed keys are visible to the score loop of every wave
      if (more && tid < D / 2) {  // the next tile's first angle, for the expansion after the barrier that ends this tile
        double rev = static_cast<double>(j + BN) * rope_rate[tid];
        rev -= floor(rev);
        rope_fr0[ST ^ 1][tid] = static_cast<float>(rev);
      }
    }

    // S^T for the two 32-key halves of the tile.  The halves alternate, so consecutive
    // matrix instructions never wait for each other's result, and the LDS reads run
    // kReadAheadS operands ahead of the products that consume them.
    pf_f32x16 s[2];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int i = 0; i < 16; ++i) s[kt][i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        const uint4 a4 = *reinterpret_cast<const uint4*>(ks_l + (k_pre ^ ((2 * ks + g2) << 4)) + kt * 32 * D * 2);
        if constexpr (KF16)
          s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(pf_f16x8, a4), qh[ks], s[kt], 0, 0, 0);
        else
          s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pf_as_bf16x8(a4), qb[ks], s[kt], 0, 0, 0);
      }
    if (HAS_BK) {
#pragma unroll
      for (int ks = 0; ks < RKS; ++ks)
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
          const uint2 lo = *reinterpret_cast<const uint2*>(ks_l + l_rd[ks][0] + kt * 32 * RP * 2);
          const uint2 hi = *reinterpret_cast<const uint2*>(ks_l + l_rd[ks][1] + kt * 32 * RP * 2);
          s[kt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pf_as_bf16x8(make_uint4(lo.x, lo.y, hi.x, hi.y)), qtb[ks],
                                                          s[kt], 0, 0, 0);
        }
    }
    // instruction order for the scheduler: kReadAheadS LDS reads, then one product per read
    __builtin_amdgcn_sched_group_barrier(0x100, kReadAheadS, 0);
#pragma unroll
    for (int i = 0; i < 2 * KS; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    if (HAS_BK) {
#pragma unroll
      for (int i = 0; i < 2 * RKS; ++i) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      }
    }
    // causal mask + online softmax.  Element (kt, i) of this lane is key
    // j + 32kt + 8(i/4) + 4g2 + i%4 of row l32.
    if (j + BN - 1 > wave_first) {  // some row of this wave does not see the whole tile
      const int limit = base_vis + token_of(wave * 32 + (static_cast<int>(threadIdx.x) & 31));  // last visible key of this lane's row
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int key = j + 32 * kt + 8 * (i >> 2) + 4 * g2 + (i & 3);
          if (key > limit) s[kt][i] = -INFINITY;
        }
    }
    float mx = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s[kt][i]);
    mx = fmaxf(mx, pf_partner32(mx)) * sc;
    if (__builtin_amdgcn_ballot_w64(mx > m_run + kSlack) != 0) {  // always on the first tile (m_run = -inf)
      const float m_new = fmaxf(m_run, mx);
      // a share that does not start at key 0 may hold rows that have seen nothing yet
      const float alpha = (SPLIT && m_new == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int b = 0; b < DB; ++b) o_acc[b] *= alpha;
#pragma unroll
      for (int b = 0; b < RB; ++b) lr_acc[b] *= alpha;
    }
    // finite from the first tile on (key 0 is visible to every row) unless the share starts later
    const float nm = (SPLIT && m_run == -INFINITY) ? 0.f : -m_run;
    pf_bf16x8 pb[2][2];       // [kt][16-key k-step]
    auto exp_half = [&](int kt) __attribute__((always_inline)) {
      float e[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        e[i] = __builtin_amdgcn_exp2f(fmaf(s[kt][i], sc, nm));
        if (!ONES_ROW) l_run += e[i];
      }
#pragma unroll
      for (int h2 = 0; h2 < 2; ++h2)
        pb[kt][h2] = pf_as_bf16x8(make_uint4(pf_pack2(e[8 * h2 + 0], e[8 * h2 + 1]), pf_pack2(e[8 * h2 + 2], e[8 * h2 + 3]),
                                             pf_pack2(e[8 * h2 + 4], e[8 * h2 + 5]), pf_pack2(e[8 * h2 + 6], e[8 * h2 + 7])));
    };
    // The exponentials of the second 32-key half run under the products of the first: a matrix instruction
    // occupies its pipe for 32 cycles, and the wave is free to issue vector work meanwhile.
    exp_half(0);
    __builtin_amdgcn_sched_barrier(0);
    exp_half(1);
    // O^T += V^T P^T ; Olr^T += L^T P^T, one 16-key k-step at a time.
    // k-step (kt, h2), element e <-> key 32kt + 16h2 + 8(e/4) + 4g2 + e%4.
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int h2 = 0; h2 < 2; ++h2) {
        const int rowoff = (32 * kt + 16 * h2) * (D * 2);
#pragma unroll
        for (int b = 0; b < DB; ++b) {
          const unsigned char* src = ks_l + (v_pre ^ (b << 6)) + rowoff;
          const pf_bf16x8 a = pf_join(pf_read_tr16(src), pf_read_tr16(src + 8 * (D * 2)));
          o_acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[kt][h2], o_acc[b], 0, 0, 0);
        }
#pragma unroll
        for (int b = 0; b < RB; ++b) {
          const int koff = (32 * kt + 16 * h2) * (RP * 2);
          const unsigned char* src0 = ks_l + lt_rd[b][0] + koff;
          const unsigned char* src1 = ks_l + lt_rd[b][1] + koff;
          if (ONES_ROW && b == RB - 1) {
            src0 = ones_lane ? smem + ONES_AT : src0;
            src1 = ones_lane ? smem + ONES_AT : src1;
          }
          const pf_bf16x8 a = pf_join(pf_read_tr16(src0), pf_read_tr16(src1));
          lr_acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[kt][h2], lr_acc[b], 0, 0, 0);
        }
      }
    // the transposed reads (two per operand) run kReadAheadPV operands ahead
    __builtin_amdgcn_sched_group_barrier(0x100, 2 * kReadAheadPV, 0);
#pragma unroll
    for (int i = 0; i < 2 * (DB + RB); ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
      __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, ONES_ROW ? 3 : 5, 0);
    }
#pragma unroll
    for (int i = 0; i < 2 * (DB + RB); ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
    }
    // the next tile has landed (this wave's share) and everybody is done reading this one
    pf_wait_vm0();
    __syncthreads();
  };
  for (int tile = tile_begin; tile < tile_end; tile += 2) {
    tile_step(tile, std::integral_constant<int, 0>{});
    if (tile + 1 < tile_end) tile_step(tile + 1, std::integral_constant<int, 1>{});
  }

  // ---------------- epilogue: O^T += B_V^T Olr^T, O /= l, store ----------------
  const int out_row = global_row(false);
  if (ONES_ROW) {
    // row sums sit in register 8 (rho = 32(RB-1) + 16) of the lanes with g2 == 0
    const float mine = lr_acc[RB - 1][8];
    const float other = pf_partner32(mine);
    l_run = g2 == 0 ? mine : other;
  } else {
    l_run += pf_partner32(l_run);
  }
  if (SPLIT) {
    // this share's state for the merge kernel: m in natural-log units, l, O^T and Olr^T as
    // fp32 rows [slot][d] and [slot][rank]; registers 4q..4q+3 are d (rho) = 32b + 8q + 4g2 + 0..3
    if (out_row >= 0) {
      const int64_t slot = static_cast<int64_t>(out_row) * p.n_splits + split;
      if (g2 == 0) {
        p.part_ml[slot * 2 + 0] = m_run * 0.69314718055994530942f;
        p.part_ml[slot * 2 + 1] = l_run;
        if (split == 0) p.part_adapter[out_row] = a_idx;
      }
#pragma unroll
      for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<pf_f32x4*>(p.part_o + slot * D + 32 * b + 8 * q + 4 * g2) =
              pf_f32x4{o_acc[b][4 * q + 0], o_acc[b][4 * q + 1], o_acc[b][4 * q + 2], o_acc[b][4 * q + 3]};
#pragma unroll
      for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int rho = 32 * b + 8 * q + 4 * g2;  // the rank is a multiple of 8: all four or none
          if (rho < r)
            *reinterpret_cast<pf_f32x4*>(p.part_lr + slot * r + rho) =
                pf_f32x4{lr_acc[b][4 * q + 0], lr_acc[b][4 * q + 1], lr_acc[b][4 * q + 2], lr_acc[b][4 * q + 3]};
        }
    }
    return;
  }
  if (p.b_v != nullptr) {
    const int64_t ldb = static_cast<int64_t>(Hkv) * D;
    const bf16_t* bv = static_cast<const bf16_t*>(p.b_v) + static_cast<int64_t>(a_idx) * r * ldb + hk * D;
#pragma unroll
    for (int ks = 0; ks < RKS; ++ks) {
      // B operand: Olr^T registers 8(ks&1)..+7 of block ks/2: element e <-> rho = 16ks + 8(e/4) + 4g2 + e%4
      const int o = (ks & 1) * 8;
      const pf_f32x16& src = lr_acc[ks >> 1];
      // O_lr as two bf16 terms, the second what the first left over: to 17 bits, against the 8 of the output's own
      // rounding.  (One term cost up to 2^-9 of |O_lr| |B_V|, which calls with several shares, whose merge holds
      // O_lr in fp32, do not pay; 32 to 64 cycles of matrix pipe per 16 ranks and 32 columns, once per q tile.)
      pf_bf16x8 bop[2];
      {
        uint32_t w[2][4];
#pragma unroll
        for (int e2 = 0; e2 < 4; ++e2) {
          const float x0 = src[o + 2 * e2], x1 = src[o + 2 * e2 + 1];
          w[0][e2] = pf_pack2(x0, x1);
          const float r0 = x0 - __uint_as_float(w[0][e2] << 16), r1 = x1 - __uint_as_float(w[0][e2] & 0xffff0000u);
          w[1][e2] = pf_pack2(__builtin_isfinite(r0) ? r0 : 0.f, __builtin_isfinite(r1) ? r1 : 0.f);
        }
#pragma unroll
        for (int term = 0; term < 2; ++term) bop[term] = pf_as_bf16x8(make_uint4(w[term][0], w[term][1], w[term][2], w[term][3]));
      }
      pf_bf16x8 bvt[DB];
#pragma unroll
      for (int b = 0; b < DB; ++b) {
        // A operand: B_V^T: lane (d = 32b + l32, element e <-> rho as above)
        uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int rho = 16 * ks + 8 * (e >> 2) + 4 * g2 + (e & 3);
          const uint32_t val = rho < r ? static_cast<uint32_t>(bv[rho * ldb + 32 * b + l32]) : 0u;
          w[e >> 1] |= val << ((e & 1) * 16);
        }
        bvt[b] = pf_as_bf16x8(make_uint4(w[0], w[1], w[2], w[3]));
      }
#pragma unroll
      for (int term = 1; term >= 0; --term)
#pragma unroll
        for (int b = 0; b < DB; ++b) o_acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bvt[b], bop[term], o_acc[b], 0, 0, 0);
    }
  }
  if (out_row >= 0) {
    const float inv = 1.0f / l_run;
    bf16_t* orow = static_cast<bf16_t*>(p.out) + static_cast<int64_t>(out_row) * D;
#pragma unroll
    for (int b = 0; b < DB; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        // registers 4q..4q+3 are d = 32b + 8q + 4g2 + 0..3
        const uint2 pk = make_uint2(pf_pack2(o_acc[b][4 * q + 0] * inv, o_acc[b][4 * q + 1] * inv),
                                    pf_pack2(o_acc[b][4 * q + 2] * inv, o_acc[b][4 * q + 3] * inv));
        *reinterpret_cast<uint2*>(orow + 32 * b + 8 * q + 4 * g2) = pk;
      }
  }
