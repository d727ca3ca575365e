// Body of the split-KV MFMA decode kernels, included inside each of them (lra_decode_mfma.hip, lra_decode_batch.hip) with
// the template parameters in scope, and with
//   lane, wave    of the thread, the wave uniform
//   h, t, rg      kv head, sequence, row group of the workgroup
//   split         place of its partial state among the p.n_splits of each row
//   j0, keys      its first key and their number, a multiple of 128 of which a wave takes a quarter
//   LAST          true for the shares of a batch in one row: the sequence's queries are first_query .. end_query - 1, and
//                 where last_of_seq is set the slots behind this one are left as empty states.
// Text, so that each kernel has it where its registers come out best: in the kernel itself or in a function (see
// kDecodeByFunction).
  constexpr int NW = 4;
  static_assert(!PA || (!CAUSAL && RT == 1), "per-adapter low-rank caches: decode form, one row tile");
  constexpr int KS = D / 32;       // MFMA k-steps over the head dimension
  constexpr int RKS = RP / 32;     // MFMA k-steps over the (padded) rank
  constexpr int DB = D / 16;       // 16-wide output blocks over d
  constexpr int RB = RP / 16;      // 16-wide output blocks over the rank
  constexpr int KCH = D / 8;       // 16-byte chunks per K/V row
  constexpr int RCH = RP / 8;      // 16-byte chunks per L row in LDS
  constexpr int KROWS = 64 / KCH;  // K/V rows one wave-wide load moves
  constexpr int KVL = 32 / KROWS;  // wave-wide loads per 32-key K (or V) tile
  constexpr int LROWS = 64 / RCH;
  constexpr int LL = 32 / LROWS;
  constexpr int KV_BYTES = 32 * D * 2;
  constexpr int L_BYTES = 32 * RP * 2;
  constexpr int WAVE_BYTES = 2 * KV_BYTES + L_BYTES;
  constexpr int NACC = RT * (DB + RB) * 4 + RT;
  constexpr int MERGE_SLOT = NACC * 64 * 4;
  constexpr int STAGE_TOTAL = NW * WAVE_BYTES;
  constexpr int MERGE_TOTAL = (NW / 2) * MERGE_SLOT;
  constexpr int SMEM = STAGE_TOTAL > MERGE_TOTAL ? STAGE_TOTAL : MERGE_TOTAL;
  constexpr int LSW_SHIFT = (RP == 32) ? 1 : 0;
  constexpr int QT_BYTES = RT * RKS * 1024;
  constexpr int M_BYTES = NW * RT * 16 * 4;
  // Two workgroups per CU need 2 * LDS <= 160 KB.  Where the tile regions alone
  // leave no room, the Qt exchange area and the per-wave maxima live inside the
  // tile regions and the first tile is requested only after the prologue.
  constexpr bool ALIAS = 2 * (SMEM + QT_BYTES + M_BYTES) > 160 * 1024;
  constexpr int EXTRA = ALIAS ? 16 : QT_BYTES + M_BYTES;
  static_assert(QT_BYTES <= WAVE_BYTES && RT * 64 <= WAVE_BYTES, "aliased areas must fit one wave's region");

  __shared__ __align__(16) unsigned char smem[SMEM];
  __shared__ __align__(16) unsigned char extra_lds[EXTRA];
  unsigned char* qt_lds = ALIAS ? smem : extra_lds;

  const int ln = lane & 15, lg = lane >> 4;
  LRA_STAMP_DECL;
  LRA_STAMP(0);
  // The first and the last entry of seq_query_start are fixed by the contract (0 and
  // n_queries): a single sequence needs no table read at all, and the adapter ids can be
  // requested at once instead of one memory round trip later.
  const int32_t len_t = CONST_I32(p.seq_lens)[t];
  int q_begin = 0, q_end = CAUSAL ? p.n_new : p.n_queries;
  if (LAST) {
    q_begin = first_query;
    q_end = end_query;
  } else if (!CAUSAL) {
    if (t > 0) q_begin = CONST_I32(p.seq_query_start)[t];
    if (t + 1 < p.n_seqs) q_end = CONST_I32(p.seq_query_start)[t + 1];
  }
  const int n_t = min(len_t, p.max_seq_len);
  const int n_q = q_end - q_begin;
  const int GP = p.group_pad, G = p.group, r = p.rank;
  const int row0 = rg * RT * 16;
  if (row0 >= n_q * GP) return;
  asm volatile("" ::"s"(n_t));
  LRA_STAMP(1);
  // workspace slot of the row this lane stands for in row tile rt (-1: padding row)
  auto row_slot = [&](int rt) -> int64_t {
    const int R = row0 + rt * 16 + ln;
    const int slot_q = R / GP, gg = R - slot_q * GP;
    if (!(slot_q < n_q && gg < G)) return -1;
    return (static_cast<int64_t>(q_begin + slot_q) * p.n_q_heads + h * G + gg) * p.n_splits + split;
  };
  if constexpr (LAST) {
    if (last_of_seq && wave == 0) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const int64_t slot = row_slot(rt);
        if (slot >= 0)
          for (int s = split + 1 + lg; s < p.n_splits; s += 4) {
            p.part_ml[(slot - split + s) * 2 + 0] = -INFINITY;
            p.part_ml[(slot - split + s) * 2 + 1] = 0.f;
          }
      }
    }
  }
  if (j0 >= n_t) {
    // a split past the end of this sequence: leave an empty state (zero row sum), which is
    // all the merge kernel looks at; the O and O_lr rows of the slot stay unwritten
    if (wave == 0 && lg == 0) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
        const int64_t slot = row_slot(rt);
        if (slot >= 0) {
          p.part_ml[slot * 2 + 0] = -INFINITY;
          p.part_ml[slot * 2 + 1] = 0.f;
        }
      }
    }
    return;
  }
  // The merge kernel takes each row's adapter from the workspace: the workgroups of split 0
  // copy it there (requested now, stored with the state at the end).
  int my_adapter[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    const int R = row0 + rt * 16 + ln;
    const int slot_q = min(R / GP, n_q - 1);
    my_adapter[rt] = CAUSAL ? p.adapter_index : (split == 0 ? p.query_adapter[q_begin + slot_q] : 0);
  }
  // last key each of this lane's rows may see (causal form only)
  int lim[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) lim[rt] = n_t - n_q + min((row0 + rt * 16 + ln) / GP, n_q - 1);
  const int lim_first = n_t - n_q + row0 / GP;  // the smallest of them in this workgroup

  // adapter of every agent slot of every row tile: wave-uniform loads, requested before
  // anything else so that the B_K rows they select can follow one round trip earlier
  // (only in the one-row-tile kernels: in the two-tile ones the extra registers and the wait
  // cost the streaming kernel more than the merge kernel gains)
  const bool warm_bv = RT == 1 && p.b_v != nullptr && split == min(1, p.n_splits - 1);
  int a_slot[RT][4];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt)
#pragma unroll
    for (int si = 0; si < 4; ++si) {
      const int slot = (row0 + rt * 16) / GP + si;
      if (CAUSAL)
        a_slot[rt][si] = (si < 16 / GP && slot < n_q) ? p.adapter_index : -1;
      else
        a_slot[rt][si] = ((HAS_BK || warm_bv || p.l_adapter_stride > 0) && si < 16 / GP && slot < n_q)
                             ? min(max(CONST_I32(p.query_adapter)[q_begin + slot], 0), p.n_adapters - 1)  // device data: kept inside the table
                             : -1;
    }
  const int j1 = min(j0 + keys, n_t);
  const int kpw = keys / NW;  // multiple of 32
  const int jw0 = j0 + wave * kpw;
  const int jw1 = max(jw0, min(jw0 + kpw, j1));  // == jw0 for a wave without keys

  unsigned char* ks_lds = smem + wave * WAVE_BYTES;
  unsigned char* vs_lds = ks_lds + KV_BYTES;
  unsigned char* ls_lds = vs_lds + KV_BYTES;

  const bf16_t* kb = static_cast<const bf16_t*>(p.k_base);
  const bf16_t* vb = static_cast<const bf16_t*>(p.v_base);
  // Low-rank rows: dense, or with a pitch of their own; with one low-rank cache per adapter the host gives every
  // agent a row tile (and this kernel one row tile per workgroup), so the tile's first slot names the cache
  const int64_t lp = p.l_row_stride;
  const bf16_t* lr = static_cast<const bf16_t*>(p.l) +
                     (!PA && p.l_adapter_stride > 0 ? static_cast<int64_t>(max(a_slot[0][0], 0)) * p.l_adapter_stride : 0);
  // PA: ranks per column block (16, 32 or 64), 16-byte chunks per row of a block, bytes per row of a block; the
  // XOR swizzle of the chunk index inside a block row (none for 32-byte rows: 16 rows fill two clocks densely).
  // Without PA the tile is one block of RP ranks and all of this folds to the constants of that layout.
  const int lb = PA ? p.l_block : RP;
  const int lcpr = lb >> 3, lcs = __builtin_ctz(lcpr), lb2 = lb * 2;
  auto swz_l = [&](int row) { return lcpr == 8 ? (row & 7) : (lcpr == 4 ? ((row >> 1) & 3) : 0); };
  const int gps = __builtin_ctz(GP);  // GP is 4, 8 or 16
  const uint32_t ts2 = static_cast<uint32_t>(p.kv_token_stride) * 2u;  // token stride in bytes
  const uint32_t r2 = static_cast<uint32_t>(r) * 2u;                     // L row in bytes
  const uint32_t lp2 = static_cast<uint32_t>(lp) * 2u;                   // bytes between L rows

  // ===================== per-lane constants of the tile traffic =====================
  // The LDS of this chip serves 256 bytes per clock (64 banks): a ds_read_b128 is free of
  // conflicts when 16 consecutive lanes hit 16 different 16-byte positions of that window,
  // a ds_read_b64_tr_b16 when the eight 32-byte pieces of 32 consecutive lanes do.  Rows of
  // 256 bytes (d = 128) all start at position 0, rows of 128 bytes alternate halves; the XOR
  // swizzles below (on the 16-byte chunk index of a row) spread them accordingly:
  //   K (b128, 16 rows per clock)      chunk ^ (row & 15)            | chunk ^ ((row >> 1) & 7)
  //   V (tr_b64, 8 rows per clock)     chunk ^ ((row & 7) << 1)      | chunk ^ (((row >> 1) & 3) << 1)
  auto swz_k = [](int row) { return D == 128 ? (row & 15) : ((row >> 1) & 7); };
  auto swz_v = [](int row) { return D == 128 ? ((row & 7) << 1) : (((row >> 1) & 3) << 1); };
  // global -> LDS: lane l of load i lands at LDS row i*ROWS + l/CH, physical chunk l%CH,
  // and therefore fetches logical chunk (l%CH) ^ swizzle(row).  The swizzle of row
  // i*ROWS + l/CH repeats with period 16/KROWS (K) and 8/KROWS (V) in i.
  constexpr int KPER = KROWS == 4 ? 4 : 2, VPER = KROWS == 4 ? 2 : 1;
  uint32_t k_voff[KPER], v_voff[VPER], l_voff;
  uint32_t l_in_row = 0;  // PA: byte offset of the lane's chunk inside an L row
  bool l_ok = true;       // PA: that chunk lies inside the rank
  {
    const int rr = lane / KCH, pc = lane % KCH;
#pragma unroll
    for (int q = 0; q < KPER; ++q) k_voff[q] = static_cast<uint32_t>(rr) * ts2 + ((pc ^ swz_k(q * KROWS + rr)) << 4);
#pragma unroll
    for (int q = 0; q < VPER; ++q) v_voff[q] = static_cast<uint32_t>(rr) * ts2 + ((pc ^ swz_v(q * KROWS + rr)) << 4);
    if constexpr (PA) {
      // lane -> (row inside a request, chunk of the block row): the swizzle repeats from request to request
      const int lrow = lane >> lcs, lpc = lane & (lcpr - 1);
      const int lch = lpc ^ swz_l(lrow);
      l_ok = lch * 8 < r;
      l_in_row = static_cast<uint32_t>(lch) << 4;
      l_voff = l_ok ? static_cast<uint32_t>(lrow) * lp2 + l_in_row : kOob;
    } else {
      const int lrow = lane / RCH, lpc = lane % RCH;
      const int lch = lpc ^ ((lrow >> LSW_SHIFT) & (RCH - 1));
      l_voff = (lch * 8 < r) ? static_cast<uint32_t>(lrow) * lp2 + (lch << 4) : kOob;
    }
  }
  // LDS -> MFMA operands (byte offsets inside the tile regions).
  // K rows as A operand of S^T: key = 16tt + ln, logical chunk 4ks + lg at chunk ^ swz_k(key):
  // row offset, swizzle and lg sit in disjoint address bits, so the address is
  // k_pre ^ (ks << 6) + tt * 16 rows.
  const int k_pre = ln * (2 * D) + ((swz_k(ln) ^ lg) << 4);
  // V^T as A operand of O^T: this lane addresses row ka (+16tt) of the tile, logical chunk
  // 2b + c0 (+ half sub): address v_pre ^ (b << 5) + tt * 16 rows.
  const int ka = 4 * lg + (ln >> 2);  // row (within a 16-key tile) this lane addresses in transpose reads
  const int v_pre = ka * (2 * D) + ((swz_v(ka) + ((ln & 3) >> 1)) << 4) + (ln & 1) * 8;
  int l_rd[RKS][2];  // L rows as A operand of S^T: two 8-byte pieces per k-step
  int lt_rd[RB];     // L^T as A operand of Olr^T
  if constexpr (PA) {
    // column chunk ch of the tile (8 ranks) lies in block ch / lcpr, chunk ch % lcpr of a row there
    auto chunk_addr = [&](int ch, int row) {
      const int blk = ch >> lcs, cc = ch & (lcpr - 1);
      return blk * (32 * lb2) + row * lb2 + ((cc ^ swz_l(row)) << 4);
    };
#pragma unroll
    for (int ks = 0; ks < RKS; ++ks)
#pragma unroll
      for (int pc = 0; pc < 2; ++pc) l_rd[ks][pc] = chunk_addr(4 * ks + 2 * pc + (lg >> 1), ln) + (lg & 1) * 8;
#pragma unroll
    for (int b = 0; b < RB; ++b) lt_rd[b] = chunk_addr(2 * b + ((ln & 3) >> 1), ka) + (ln & 1) * 8;
  } else {
    const int swz_s = (ln >> LSW_SHIFT) & (RCH - 1);
#pragma unroll
    for (int ks = 0; ks < RKS; ++ks)
#pragma unroll
      for (int pc = 0; pc < 2; ++pc) {
        const int ch = 4 * ks + 2 * pc + (lg >> 1);
        l_rd[ks][pc] = ln * (2 * RP) + ((ch ^ swz_s) << 4) + (lg & 1) * 8;
      }
    const int swz_t = (ka >> LSW_SHIFT) & (RCH - 1);
#pragma unroll
    for (int b = 0; b < RB; ++b) {
      const int ch = 2 * b + ((ln & 3) >> 1);
      lt_rd[b] = ka * (2 * RP) + ((ch ^ swz_t) << 4) + (ln & 1) * 8;
    }
  }

  // Contiguous cache: one resource per wave covering exactly its keys [jw0, jw1).
  u32x4 rs_k = {0u, 0u, 0u, 0u}, rs_v = rs_k, rs_l = rs_k;
  if (!PAGED) {
    const int nk = jw1 - jw0;
    const int64_t base = static_cast<int64_t>(h) * p.kv_head_stride + static_cast<int64_t>(jw0) * p.kv_token_stride;
    const uint32_t bytes = nk > 0 ? static_cast<uint32_t>(nk - 1) * ts2 + D * 2 : 0u;
    rs_k = make_rsrc_words(kb + base, bytes);
    rs_v = make_rsrc_words(vb + base, bytes);
    rs_l = make_rsrc_words(lr + static_cast<int64_t>(jw0) * lp, nk > 0 ? static_cast<uint32_t>(nk - 1) * lp2 + r2 : 0u);
  }
  // PA: one L resource per request of 1 KB - the requests of a column block read the cache of that block's agent
  // slot (a block beyond the tile's slots, or of an empty slot, reads nothing).  Contiguous cache: the rows of the
  // wave's keys, as above.  Paged cache: the adapter's whole pool (the host has checked that it fits 32-bit byte
  // offsets); a lane then addresses its row through the physical block and masks the keys past the wave's range itself.
  constexpr int LREQ = PA ? LL : 1;
  u32x4 rs_la[LREQ];
  uint32_t l_row0[LREQ];  // first tile row of the request
  if constexpr (PA) {
    const int rows_per_req = 64 >> lcs;  // 1 KB of rows of lb ranks
    const int rpb_shift = lcs - 1;       // lb/16 requests per block
    const int nk = jw1 - jw0;
    const uint32_t bytes = PAGED ? (static_cast<uint32_t>(p.num_blocks) * 16u - 1u) * lp2 + r2
                                 : (nk > 0 ? static_cast<uint32_t>(nk - 1) * lp2 + r2 : 0u);
#pragma unroll
    for (int i = 0; i < LL; ++i) {
      const int blk = i >> rpb_shift, qq = i - (blk << rpb_shift);
      const int a = blk == 0 ? a_slot[0][0] : (blk == 1 ? a_slot[0][1] : (blk == 2 ? a_slot[0][2] : a_slot[0][3]));
      const bool live = blk < (16 >> gps) && a >= 0;
      rs_la[i] = make_rsrc_words(static_cast<const bf16_t*>(p.l) + static_cast<int64_t>(live ? a : 0) * p.l_adapter_stride +
                                     (PAGED ? 0 : static_cast<int64_t>(jw0) * lp),
                                 live ? bytes : 0u);
      l_row0[i] = static_cast<uint32_t>(qq * rows_per_req);
    }
  }
  const const_i32_ptr bt = CONST_I32(p.block_table) + static_cast<int64_t>(t) * p.max_blocks_per_seq;

  // Paged cache: the two physical block ids of a step are fetched one step ahead (scalar
  // loads), so the table lookup is off the path that requests the tile.
  int blk_next[2] = {0, 0};
  auto fetch_block_ids = [&](int j) {
    if (PAGED) {
      const int nb_last = (n_t - 1) >> 4;
      blk_next[0] = bt[min(j >> 4, nb_last)];
      blk_next[1] = bt[min((j >> 4) + 1, nb_last)];
    }
  };
  fetch_block_ids(jw0);

  // K_base / V_base requests: non-temporal when this workgroup is the only reader of its keys; with
  // several row groups per (sequence, kv head) the others find the tiles in L2
  const bool stream_kv = p.row_groups == 1;
  auto kv_load = [&](u32x4 rs, unsigned char* lds, uint32_t voff, uint32_t soff) __attribute__((always_inline)) {
    if (stream_kv) buf_load16_to_lds<true>(rs, lds, voff, soff);
    else buf_load16_to_lds<false>(rs, lds, voff, soff);
  };
  // ---- HBM -> LDS for the 32-key step starting at token j ----
  auto issue_tile = [&](int j) {
    if (PAGED) {
      const int64_t hoff = static_cast<int64_t>(h) * p.kv_head_stride;
      const int blk_cur[2] = {blk_next[0], blk_next[1]};
      fetch_block_ids(j + 32);
#pragma unroll
      for (int half = 0; half < 2; ++half) {
        const int jb = j + 16 * half;
        const int blk = blk_cur[half];
        const int nv = max(0, min(16, jw1 - jb));  // slots of this block inside the wave's range
        const uint32_t kv_bytes = nv > 0 ? static_cast<uint32_t>(nv - 1) * ts2 + D * 2 : 0u;
        const u32x4 pk = make_rsrc_words(kb + static_cast<int64_t>(blk) * p.kv_block_stride + hoff, kv_bytes);
        const u32x4 pv = make_rsrc_words(vb + static_cast<int64_t>(blk) * p.kv_block_stride + hoff, kv_bytes);
        const u32x4 pl = make_rsrc_words(lr + static_cast<int64_t>(blk) * 16 * lp, nv > 0 ? static_cast<uint32_t>(nv - 1) * lp2 + r2 : 0u);
#pragma unroll
        for (int i = 0; i < KVL / 2; ++i) {
          const int ii = half * (KVL / 2) + i;
          kv_load(pk, ks_lds + ii * 1024, k_voff[ii % KPER], i * KROWS * ts2);
          kv_load(pv, vs_lds + ii * 1024, v_voff[ii % VPER], i * KROWS * ts2);
        }
        if constexpr (!PA) {
#pragma unroll
          for (int i = 0; i < LL / 2; ++i) {
            const int ii = half * (LL / 2) + i;
            buf_load16_to_lds(pl, ls_lds + ii * 1024, l_voff, i * LROWS * lp2);
          }
        }
      }
      if constexpr (PA) {
        // tile row of this lane in request i: l_row0[i] + lane / lcpr; its physical block is the first or the
        // second of the step; rows at or past the end of the wave's range read nothing (zeros)
        const uint32_t lrow = static_cast<uint32_t>(lane >> lcs);
        const uint32_t pg0 = static_cast<uint32_t>(blk_cur[0]) * 16u * lp2, pg1 = static_cast<uint32_t>(blk_cur[1]) * 16u * lp2;
#pragma unroll
        for (int i = 0; i < LL; ++i) {
          const uint32_t row = l_row0[i] + lrow;
          const bool ok = l_ok && j + static_cast<int>(row) < jw1;
          const uint32_t voff = ok ? (row < 16u ? pg0 : pg1) + (row & 15u) * lp2 + l_in_row : kOob;
          buf_load16_to_lds(rs_la[i], ls_lds + i * 1024, voff, 0u);
        }
      }
    } else {
      const uint32_t s0 = static_cast<uint32_t>(j - jw0);
#pragma unroll
      for (int i = 0; i < KVL; ++i) {
        kv_load(rs_k, ks_lds + i * 1024, k_voff[i % KPER], (s0 + i * KROWS) * ts2);
        kv_load(rs_v, vs_lds + i * 1024, v_voff[i % VPER], (s0 + i * KROWS) * ts2);
      }
      if constexpr (PA) {
#pragma unroll
        for (int i = 0; i < LL; ++i) buf_load16_to_lds(rs_la[i], ls_lds + i * 1024, l_voff, (s0 + l_row0[i]) * lp2);
      } else {
#pragma unroll
        for (int i = 0; i < LL; ++i) buf_load16_to_lds(rs_l, ls_lds + i * 1024, l_voff, (s0 + i * LROWS) * lp2);
      }
    }
  };

  // The first tile is on its way before the prologue touches Q and B_K.
  if ((!ALIAS || !HAS_BK) && jw0 < jw1) issue_tile(jw0);
  LRA_STAMP(2);

  // ===================== prologue: Q operands and Qt = Q B_K^T =====================
  // qb[rt][ks]: lane (row ln of tile rt, k = 32ks + 8lg + e), e = 0..7.  Used as the
  // B operand of S^T and as the B operand of Qt^T = B_K Q^T below.
  bf16x8 qb[RT][KS];
  {
    const __amdgpu_buffer_rsrc_t rs_q =
        make_rsrc(static_cast<const bf16_t*>(p.q) + static_cast<int64_t>(q_begin) * p.n_q_heads * D,
                  static_cast<uint32_t>(n_q) * p.n_q_heads * D * 2);
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int R = row0 + rt * 16 + ln;
      const int slot = R / GP, gg = R - slot * GP;
      const bool valid = slot < n_q && gg < G;
      const uint32_t off = valid ? static_cast<uint32_t>((slot * p.n_q_heads + h * G + gg) * D * 2 + lg * 16) : kOob;
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) qb[rt][ks] = as_bf16x8(buf_load16(rs_q, off, ks * 64));
    }
  }
  // Qt^T block (rho block cb, tile rt) = B_K^a[16cb..16cb+15][:] . Q_tile^T : C layout
  // lane (rho = 16cb + 4lg + j, row ln).  Rows of a tile belong to 16/GP agents; each
  // agent's product is kept only in its own rows (lanes).  The items are spread over
  // the waves and exchanged through LDS in operand-ready form: operand (rt, ks') of
  // lane l is the 16 bytes at ((rt*RKS + ks')*64 + l)*16, elements
  // e -> rho = 32ks' + 16(e/4) + 4lg + e%4.  The L operand below uses the same order.
  bf16x8 qtb[RT][RKS];
  if (HAS_BK) {
    if constexpr (PA) {
      // every piece of the exchange area starts as zero: blocks beyond a slot's rank, the other slots' blocks
      if (wave < RT * RKS) *reinterpret_cast<uint4*>(qt_lds + (wave * 64 + lane) * 16) = make_uint4(0u, 0u, 0u, 0u);
      static_assert(!PA || RT * RKS <= NW, "one piece per wave");
      __syncthreads();
    }
    // Items of a row tile: agent slots (a prefill has one adapter: one B_K for all rows) x rho blocks (1 .. RP/16)
    const int S = CAUSAL ? 1 : 16 / GP;
    const int ncb = (r + 15) >> 4;
    const int inv_ncb = ncb == 1 ? 257 : (ncb == 2 ? 129 : (ncb == 3 ? 86 : 65));  // idx / ncb = idx * inv_ncb / 256 (idx < 16, ncb <= 4)
    const int64_t ldb = static_cast<int64_t>(p.n_kv_heads) * D;
    const bf16_t* bkg = static_cast<const bf16_t*>(p.b_k);
    constexpr int MAXIT = CAUSAL ? 1 : RP / 16;  // items per wave and row tile: at most 4 slots x RP/16 rho blocks over 4 waves
    constexpr int BT = CAUSAL ? 1 : RT;          // row tiles with B_K rows of their own
    const int n_items = S * ncb;
    // Every B_K row of this wave's items is requested before the first product starts, and none that no item is for: a load of sixteen
    // rows takes the memory path of the unit sixteen cycles and more, in front of the tiles of its two workgroups.  (Sixteen or thirty-two
    // per wave before, four of them for an item at rank 16: 5 sequences of 2.4 to 4.6 thousand tokens 20.1 -> 19.0 us, 9 of 3.9 to 4.7 with
    // three agents of 7 heads 27.5 -> 25.2, 2 of 7.7 to 13 22.9 -> 20.4; 55 calls 1.02 in the mean.)
    bf16x8 bt4[BT][MAXIT][KS];
#pragma unroll
    for (int rt = 0; rt < BT; ++rt)
#pragma unroll
      for (int it = 0; it < MAXIT; ++it) {
        const int idx = wave + it * NW;
        if (idx < n_items) {
          const int si = (idx * inv_ncb) >> 8, cb = idx - si * ncb;
          const int a = si == 0 ? a_slot[rt][0] : (si == 1 ? a_slot[rt][1] : (si == 2 ? a_slot[rt][2] : a_slot[rt][3]));
          const uint32_t bytes = a >= 0 ? static_cast<uint32_t>((r - 1) * ldb + D) * 2u : 0u;
          const __amdgpu_buffer_rsrc_t rs_b = make_rsrc(bkg + static_cast<int64_t>(max(a, 0)) * r * ldb + h * D, bytes);
          const uint32_t off = static_cast<uint32_t>((cb * 16 + ln) * ldb * 2 + lg * 16);
#pragma unroll
          for (int ks = 0; ks < KS; ++ks) bt4[rt][it][ks] = as_bf16x8(buf_load16(rs_b, off, ks * 64));
        }
      }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int it = 0; it < MAXIT; ++it) {
        const int idx = wave + it * NW;
        if (idx < n_items) {
          const int si = (idx * inv_ncb) >> 8, cb = idx - si * ncb;
          f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int ks = 0; ks < KS; ++ks)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bt4[CAUSAL ? 0 : rt][it][ks], qb[rt][ks], acc, 0, 0, 0);
          if (CAUSAL || ln / GP == si) {
            const int kb = PA ? si * (lb >> 4) + cb : cb;  // 16-rank block along the L tile's columns
            unsigned char* dst = qt_lds + ((rt * RKS + (kb >> 1)) * 64 + lane) * 16;
            const uint2 pk = make_uint2(pack_bf16x2(acc[0], acc[1]), pack_bf16x2(acc[2], acc[3]));
            if constexpr (PA)
              *reinterpret_cast<uint2*>(dst + (kb & 1) * 8) = pk;
            else if (!(cb & 1) && cb + 1 >= ncb)  // the odd block next to it lies beyond the rank: zeros
              *reinterpret_cast<uint4*>(dst) = make_uint4(pk.x, pk.y, 0u, 0u);
            else
              *reinterpret_cast<uint2*>(dst + (cb & 1) * 8) = pk;
          }
        }
      }
    __syncthreads();
#pragma unroll
    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
      for (int ks = 0; ks < RKS; ++ks) {
        uint4 v = make_uint4(0u, 0u, 0u, 0u);  // k-steps entirely beyond the rank were never written
        if (PA || ks * 32 < r) v = lds_read16(qt_lds + ((rt * RKS + ks) * 64 + lane) * 16);
        qtb[rt][ks] = as_bf16x8(v);
      }
  }
  if (ALIAS && HAS_BK) {
    __syncthreads();  // the exchange area is about to be overwritten by tiles
    if (jw0 < jw1) issue_tile(jw0);
  }

  LRA_STAMP(3);
  // ===================== main loop =====================
  f32x4 o_acc[RT][DB], lr_acc[RT][RB];
  float m_run[RT], l_run[RT];  // m_run in base-2 units of the scaled score
  [[maybe_unused]] float m_top[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    m_run[rt] = -INFINITY;
    m_top[rt] = -INFINITY;
    l_run[rt] = 0.f;
#pragma unroll
    for (int b = 0; b < DB; ++b) o_acc[rt][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < RB; ++b) lr_acc[rt][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const float sc = p.scale * 1.44269504088896340736f;

  for (int j = jw0; j < jw1; j += 32) {
    // the tile requested one step earlier (or before the prologue) has landed
    wait_vm0();
    lds_fence();
    if (j == jw0) LRA_STAMP(4);
    f32x4 s[2][RT];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) {
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) s[tt][rt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        const bf16x8 a = as_bf16x8(lds_read16(ks_lds + (k_pre ^ (ks << 6)) + tt * 32 * D));
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
          s[tt][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qb[rt][ks], s[tt][rt], 0, 0, 0);
      }
      if (HAS_BK) {
#pragma unroll
        for (int ks = 0; ks < RKS; ++ks) {
          const uint2 lo = lds_read8(ls_lds + l_rd[ks][0] + tt * 16 * lb2);  // (16 rows of a block further)
          const uint2 hi = lds_read8(ls_lds + l_rd[ks][1] + tt * 16 * lb2);
          const bf16x8 a = as_bf16x8(make_uint4(lo.x, lo.y, hi.x, hi.y));
#pragma unroll
          for (int rt = 0; rt < RT; ++rt)
            s[tt][rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, qtb[rt][ks], s[tt][rt], 0, 0, 0);
        }
      }
    }
    // online softmax; element (tt, jj) of this lane is key j + 16tt + 4lg + jj of row ln
    const bool tail = j + 32 > jw1 || (CAUSAL && j + 31 > lim_first);
    bf16x8 pb[RT];
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      if (tail) {
#pragma unroll
        for (int tt = 0; tt < 2; ++tt)
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) {
            const int key = j + tt * 16 + lg * 4 + jj;
            if (key >= jw1 || (CAUSAL && key > lim[rt])) s[tt][rt][jj] = -INFINITY;
          }
      }
      float mx = fmaxf(fmaxf(fmaxf(s[0][rt][0], s[0][rt][1]), fmaxf(s[0][rt][2], s[0][rt][3])),
                       fmaxf(fmaxf(s[1][rt][0], s[1][rt][1]), fmaxf(s[1][rt][2], s[1][rt][3])));
      mx = max_over_lane_groups(mx) * sc;  // sc > 0
      // LAST: every 32 keys against their own maximum (at most 2^16 below the largest so far, which keeps the sums in range),
      // so that their largest probability is exact.  The shares of a row are longer than those of the grid, and against the
      // running maximum their error against float64 was 1.2 to 1.8 % above it (16 sequences of 4 k to 64 k tokens 2.187e-3 and
      // 2.214e-3); so 2.033e-3, in the same time.
      if (LAST || __builtin_amdgcn_ballot_w64(mx > m_run[rt]) != 0) {
        if (LAST) m_top[rt] = fmaxf(m_top[rt], mx);
        const float m_new = LAST ? fmaxf(mx, m_top[rt] - 16.f) : fmaxf(m_run[rt], mx);
        // causal form: a row may have seen no key yet (both maxima -inf)
        const float alpha = (CAUSAL && m_new == -INFINITY) ? 1.f : fast_exp2(m_run[rt] - m_new);
        m_run[rt] = m_new;
        l_run[rt] *= alpha;
#pragma unroll
        for (int b = 0; b < DB; ++b) o_acc[rt][b] *= alpha;
#pragma unroll
        for (int b = 0; b < RB; ++b) lr_acc[rt][b] *= alpha;
      }
      const float nm = (CAUSAL && m_run[rt] == -INFINITY) ? 0.f : -m_run[rt];
      float pe[8];
      float sum = 0.f;
#pragma unroll
      for (int tt = 0; tt < 2; ++tt)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const float e = fast_exp2(fmaf(s[tt][rt][jj], sc, nm));
          pe[tt * 4 + jj] = e;
          sum += e;
        }
      l_run[rt] += sum;
      pb[rt] = as_bf16x8(make_uint4(pack_bf16x2(pe[0], pe[1]), pack_bf16x2(pe[2], pe[3]), pack_bf16x2(pe[4], pe[5]),
                                    pack_bf16x2(pe[6], pe[7])));
    }
    // O^T += V^T P^T ; Olr^T += L^T P^T
#pragma unroll
    for (int b = 0; b < DB; ++b) {
      const unsigned char* src = vs_lds + (v_pre ^ (b << 5));
      const bf16x8 a = join_tr(lds_read_tr16(src), lds_read_tr16(src + 32 * D));
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
        o_acc[rt][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, pb[rt], o_acc[rt][b], 0, 0, 0);
    }
#pragma unroll
    for (int b = 0; b < RB; ++b) {
      const unsigned char* src = ls_lds + lt_rd[b];
      const bf16x8 a = join_tr(lds_read_tr16(src), lds_read_tr16(src + 16 * lb2));
#pragma unroll
      for (int rt = 0; rt < RT; ++rt)
        lr_acc[rt][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, pb[rt], lr_acc[rt][b], 0, 0, 0);
    }
    // the next tile overwrites this one: every LDS read above must have returned
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
    lds_fence();
    if (j == jw0) LRA_STAMP(5);
    if (j + 32 < jw1) issue_tile(j + 32);
  }
  LRA_STAMP(6);

  // One workgroup per (sequence, kv head, row group) touches the B_V rows the merge kernel
  // will need (one 4-byte read per 128-byte line) once its keys are done, so that they wait
  // in this XCD's L2 instead of in HBM: wave w takes agent slot w of every row tile.  The
  // values are only looked at by an empty statement at the very end.
  int warm[RT][2];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    warm[rt][0] = warm[rt][1] = 0;
    const int a = wave == 0 ? a_slot[rt][0] : (wave == 1 ? a_slot[rt][1] : (wave == 2 ? a_slot[rt][2] : a_slot[rt][3]));
    if (warm_bv && a >= 0) {
      constexpr int LPR = D * 2 / 128;  // 128-byte lines per B_V row of one kv head
      const int n_lines = r * LPR;      // <= 128
      const char* bv = static_cast<const char*>(p.b_v) +
                       (static_cast<int64_t>(a) * r * p.n_kv_heads * D + static_cast<int64_t>(h) * D) * 2;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int li = i * 64 + lane;
        if (li < n_lines)
          warm[rt][i] = *reinterpret_cast<const int*>(bv + static_cast<int64_t>(li / LPR) * p.n_kv_heads * D * 2 + (li % LPR) * 128);
      }
    }
  }

  // ===================== merge the waves of this workgroup =====================
  // per-wave maxima: in a wave's own tile region when aliased (nobody else touches it
  // before the barrier), else in their own area
  float* m_mine = reinterpret_cast<float*>(ALIAS ? smem + wave * WAVE_BYTES : extra_lds + QT_BYTES + wave * RT * 64);
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    l_run[rt] = sum_over_lane_groups(l_run[rt]);
    if (lg == 0) m_mine[rt * 16 + ln] = m_run[rt];
  }
  __syncthreads();
  float m_all[RT];
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) {
    float mm = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float* m_w = reinterpret_cast<const float*>(ALIAS ? smem + w * WAVE_BYTES : extra_lds + QT_BYTES + w * RT * 64);
      mm = fmaxf(mm, m_w[rt * 16 + ln]);
    }
    m_all[rt] = mm;  // finite (wave 0 always owns a key) unless a causal row sees none of this split
    const float wgt = (CAUSAL && mm == -INFINITY) ? 0.f : fast_exp2(m_run[rt] - mm);
    l_run[rt] *= wgt;
#pragma unroll
    for (int b = 0; b < DB; ++b) o_acc[rt][b] *= wgt;
#pragma unroll
    for (int b = 0; b < RB; ++b) lr_acc[rt][b] *= wgt;
  }
  if (ALIAS) __syncthreads();  // the maxima are about to be overwritten by merge slots
  float* mslots = reinterpret_cast<float*>(smem);
  constexpr int PER_RT = (DB + RB) * 4 + 1;  // floats per lane and row tile: O^T, Olr^T, l
  // Where four slots fit, every wave deposits its state once and then sums and stores a
  // quarter of it (one barrier, four waves writing); otherwise a two-level tree through two
  // slots with wave 0 writing.
  constexpr bool FLAT = NW * MERGE_SLOT <= SMEM;
  if (FLAT) {
    float* dst = mslots + wave * (NACC * 64) + lane;
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
      for (int b = 0; b < DB; ++b)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) dst[(rt * PER_RT + b * 4 + jj) * 64] = o_acc[rt][b][jj];
#pragma unroll
      for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) dst[(rt * PER_RT + (DB + b) * 4 + jj) * 64] = lr_acc[rt][b][jj];
      dst[(rt * PER_RT + (DB + RB) * 4) * 64] = l_run[rt];
    }
    __syncthreads();
    LRA_STAMP(7);
    auto total = [&](int x) {
      float v = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) v += mslots[w * (NACC * 64) + x * 64 + lane];
      return v;
    };
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int64_t slot = row_slot(rt);
      if (slot < 0) continue;
      // blocks are dealt round robin: O^T block b to wave b % 4, Olr^T block b to wave
      // (DB + b) % 4, the row sum to wave 3 (wave-uniform branches)
#pragma unroll
      for (int b = 0; b < DB; ++b)
        if ((b & (NW - 1)) == wave) {
          f32x4 v;
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) v[jj] = total(rt * PER_RT + b * 4 + jj);
          *reinterpret_cast<f32x4*>(p.part_o + slot * D + b * 16 + lg * 4) = v;
        }
#pragma unroll
      for (int b = 0; b < RB; ++b)
        if (((DB + b) & (NW - 1)) == wave) {
          // PA: a row keeps the column block of its own agent slot only, as ranks 0 .. r-1 of its state
          const int cblk = PA ? b >> (lcs - 1) : 0;
          const bool mine = !PA || cblk == (ln >> gps);
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) {
            const int rho = b * 16 + lg * 4 + jj - cblk * lb;
            const float v = total(rt * PER_RT + (DB + b) * 4 + jj);
            if (mine && rho < r) p.part_lr[slot * r + rho] = v;
          }
        }
      if (wave == NW - 1 && lg == 0) {
        p.part_ml[slot * 2 + 0] = m_all[rt] * 0.69314718055994530942f;  // natural-log units
        p.part_ml[slot * 2 + 1] = total(rt * PER_RT + (DB + RB) * 4);
        if (split == 0) p.part_adapter[slot / p.n_splits] = my_adapter[rt];
      }
    }
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) asm volatile("" ::"v"(warm[rt][0]), "v"(warm[rt][1]));
    LRA_STAMP(8);
#ifdef LRA_TIMING
    asm volatile("s_waitcnt vmcnt(0)");
#endif
    LRA_STAMP(9);
    LRA_STAMP_FLUSH();
    return;
  }
#pragma unroll
  for (int stride = NW / 2; stride >= 1; stride >>= 1) {
    if (wave >= stride && wave < 2 * stride) {
      float* dst = mslots + (wave - stride) * (NACC * 64) + lane;
      int x = 0;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
        for (int b = 0; b < DB; ++b)
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) dst[(x++) * 64] = o_acc[rt][b][jj];
#pragma unroll
        for (int b = 0; b < RB; ++b)
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) dst[(x++) * 64] = lr_acc[rt][b][jj];
        dst[(x++) * 64] = l_run[rt];
      }
    }
    __syncthreads();
    if (wave < stride) {
      const float* src = mslots + wave * (NACC * 64) + lane;
      int x = 0;
#pragma unroll
      for (int rt = 0; rt < RT; ++rt) {
#pragma unroll
        for (int b = 0; b < DB; ++b)
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) o_acc[rt][b][jj] += src[(x++) * 64];
#pragma unroll
        for (int b = 0; b < RB; ++b)
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) lr_acc[rt][b][jj] += src[(x++) * 64];
        l_run[rt] += src[(x++) * 64];
      }
    }
    __syncthreads();
  }

  LRA_STAMP(7);
  // ===================== wave 0 writes the workgroup's partial state =====================
  if (wave == 0) {
#pragma unroll
    for (int rt = 0; rt < RT; ++rt) {
      const int64_t slot = row_slot(rt);
      if (slot < 0) continue;
      if (lg == 0) {
        p.part_ml[slot * 2 + 0] = m_all[rt] * 0.69314718055994530942f;  // natural-log units
        p.part_ml[slot * 2 + 1] = l_run[rt];
        if (split == 0) p.part_adapter[slot / p.n_splits] = my_adapter[rt];
      }
#pragma unroll
      for (int b = 0; b < DB; ++b)
        *reinterpret_cast<f32x4*>(p.part_o + slot * D + b * 16 + lg * 4) = o_acc[rt][b];
#pragma unroll
      for (int b = 0; b < RB; ++b) {
        const int cblk = PA ? b >> (lcs - 1) : 0;
        const bool mine = !PA || cblk == (ln >> gps);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const int rho = b * 16 + lg * 4 + jj - cblk * lb;
          if (mine && rho < r) p.part_lr[slot * r + rho] = lr_acc[rt][b][jj];
        }
      }
    }
  }
#pragma unroll
  for (int rt = 0; rt < RT; ++rt) asm volatile("" ::"v"(warm[rt][0]), "v"(warm[rt][1]));
  LRA_STAMP(8);
  LRA_STAMP_FLUSH();
