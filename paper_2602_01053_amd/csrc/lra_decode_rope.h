// The rotary form of the split-KV decode kernels (bf16, gfx950): one share of the keys of one (sequence, kv head) where the
// key side carries an adapter that is rotated, K_j = K_base,j + RoPE_j(L_j B_K) (what App. D.1 leaves to the key cache
// because the rotation stands between L_j and B_K).  decode_mfma_kernel and decode_batch_kernel call it.
//
// The L.Qt term of the plain form is replaced, per 32 keys and agent slot of the 16-row tile, by
//   E^T[f][key]   = B_K^T[f][:] . L^T[:][key]      (v_mfma_f32_32x32x16_bf16; C layout: lane = key, register = feature)
//   rotate the pairs (f, f + D/2) of E^T            (registers; both halves of a pair in one lane, sine and cosine of a
//                                                    (key, pair) shared by the slots)
//   S^T[key][row] += rot(E)[key][f] . Q[row][f]     (v_mfma_f32_32x32x16_bf16; the C layout of E^T is the A layout of this
//                                                    product, Q stands in that order of features in LDS)
// with Q read as zeros in the rows of the other slots (their lanes read a zero piece: no masking instructions).  The B_K^T
// operands of the slots stay in registers for the whole share.
//
// What bounds it on long shares is the vector unit: per 32 keys and slot 128 multiply-adds and 32 conversions a lane, 64 sines and
// cosines for all slots; the products run beside it (4 agents on 60000 keys: vector instructions issue in 64 % of a SIMD's time, the
// matrix pipes are busy for 24 %, LDS for 26 %; on 8192, two steps per wave, it is the round trips before the first: 28 % and 10 %, waiting 53 %).  A wave has 100 to 400 keys, so everything before its first step counts as
// much as the steps: the workgroup fetches the B_K slices and the rows of Q once (the waves share them), the K and L rows
// of the first tile follow at once and its V rows when the operands are picked up; in the loop the next K rows are requested
// as soon as the scores have read this tile's, so the rotation covers their way.
//
// The rows of a 32 x 32 product are 32 keys by 32 columns, of which 16 are rows of Q: the columns repeat them, so that every
// lane has scores, and the 16 x 16 products around it (K_base Q^T, P V) take their keys in the order that makes the sums
// meet in a lane: row 4 g + i of a 16-key tile is key 8 (g % 2) + 4 (g / 2) + i.
#pragma once

#include "lra_common.h"
#include "lra_decode_util.h"
#include "lra_plan.h"
#include "lra_prefill_util.h"

namespace lra {

// h, t, rg: kv head, sequence, row group of the workgroup; split: place of its state among the p.n_splits of each row;
// j0, keys: its first key and their number, a multiple of 128 of which a wave takes a quarter.  LAST: the shares of a batch
// in one row, whose sequence has the queries first_query .. end_query - 1; where last_of_seq is set the slots behind this
// one are left as empty states.
template <int D, int RPE, bool PAGED, bool CAUSAL, bool LAST>
__device__ __forceinline__ void decode_rope_share(const Params& p, const int h, const int t, const int rg, const int split, const int j0,
                                                  const int keys, const bool last_of_seq, const int first_query, const int end_query) {
  constexpr int NW = 4;
  constexpr int RP = RPE;                                                  // ranks of an L row in LDS
  constexpr int NS = RPE == 16 ? 4 : (RPE == 32 ? 2 : kRopeSlots64);        // agent slots with operands in registers
  constexpr int NSL = CAUSAL ? 1 : NS;                                     // (causal: one adapter for all rows)
  // (causal: no slots to choose between, and registers to spare for Q; 24 kv heads of group 1, 23 tokens after 13163, rank 8, 103 us
  // with Q read from LDS each step, 98.7 so; 300 calls 1.01 in the mean)
  constexpr bool HOLD_Q = CAUSAL;
  // (the non-temporal hint chosen once per sixteen rows: decodes 1.017, batches 1.021, prefills of a few tokens 1.025 in the mean against
  // a choice per request, which spreads them; contiguous decode at ranks up to 16 has calls either way, 4 agents on 20011 keys, rank 8,
  // 26.0 us with a choice per request and 26.8 with one per sixteen rows, 2 agents of 7 heads on 53104 29.4 and 27.5, and keeps the first)
  constexpr bool ONE_CHOICE = CAUSAL || LAST || PAGED || RPE != 16;
  constexpr int EK = RPE / 16;     // 16-wide k-steps of the E product
  constexpr int KS = D / 32;       // k-steps of K_base Q^T
  constexpr int DB = D / 16;       // 16-wide output blocks over d; 16-wide k-steps of rot(E) Q
  constexpr int RB = RP / 16;      // 16-wide output blocks over the rank
  constexpr int PB = D / 64;       // blocks of 32 rotary pairs
  constexpr int KCH = D / 8;       // 16-byte chunks per K/V row
  constexpr int RCH = RP / 8;      // 16-byte chunks per L row
  constexpr int KROWS = 64 / KCH;  // K/V rows one wave-wide load moves
  constexpr int KVL = 32 / KROWS;  // wave-wide loads per 32-key K (or V) tile
  constexpr int LROWS = 64 / RCH;
  constexpr int LL = PAGED && LROWS == 32 ? 2 : 32 / LROWS;  // (a request of 32 rows would span two blocks: half a wave each)
  constexpr int ROW_BYTES = 2 * D;
  constexpr int KV_BYTES = 32 * ROW_BYTES;
  constexpr int L_BYTES = 32 * RP * 2;
  // Ranks up to 16 have two stages for the L rows: the next tile's are requested with its K rows.  Above, the one stage is
  // refilled behind P L.
  constexpr bool TWO_L = RPE == 16;
  constexpr int WAVE_BYTES = 2 * KV_BYTES + (TWO_L ? 2 : 1) * L_BYTES;
  // The B_K slice of slot s passes through the V region of wave s (its K and V regions where it does not fit), the rows of
  // Q through a free half of wave 2's.
  constexpr int SLICE_BYTES = RPE * ROW_BYTES;
  constexpr bool TILE_FIRST = SLICE_BYTES <= KV_BYTES;  // the K and L regions are free from the start
  static_assert(SLICE_BYTES <= 2 * KV_BYTES && NS <= NW, "a slice per wave");
  constexpr int QRAW_BYTES = 16 * ROW_BYTES;
  constexpr int QRAW_AT = 2 * WAVE_BYTES + KV_BYTES + (SLICE_BYTES <= KV_BYTES / 2 ? KV_BYTES / 2 : 0);
  static_assert(!TILE_FIRST || NS <= 2 || 2 * SLICE_BYTES <= KV_BYTES, "Q beside, or instead of, a slice");
  // Q in the order of rot(E): entry (row, half of the lanes) holds its DB pieces of 16 bytes and one of padding, which
  // spreads the entries over the banks; the last entry is zero.
  constexpr int QOP_STRIDE = DB * 16 + 16;
  constexpr int NBLK = DB + RB;
  constexpr int MERGE_SLOT = NBLK * 1024 + 512;  // a wave's state: f32x4 blocks, then (m, l) pairs
  static_assert(MERGE_SLOT <= WAVE_BYTES, "a wave's state lives in its own region");

  // [Q in operand order][rates of the pairs, then their phases at each wave's step][the rates in double][tile regions]: what every slot reads lies
  // within the immediate offset of an LDS instruction
  constexpr int TAB_AT = 33 * QOP_STRIDE, RATE_AT = TAB_AT + (64 + NW * 64) * 4, TILES_AT = (RATE_AT + 64 * 8 + 255) / 256 * 256;
  __shared__ __align__(256) unsigned char lds[TILES_AT + NW * WAVE_BYTES + (TILE_FIRST ? 0 : QRAW_BYTES)];
  unsigned char* const q_op = lds;
  float* const rope_tab = reinterpret_cast<float*>(lds + TAB_AT);
  double* const rate_tab = reinterpret_cast<double*>(lds + RATE_AT);
  unsigned char* const smem = lds + TILES_AT;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int ln = lane & 15, lg = lane >> 4, l32 = lane & 31, g2 = lane >> 5;
  LRA_STAMP_DECL;
  LRA_STAMP(0);
  const int32_t len_t = CONST_I32(p.seq_lens)[t];
  int q_begin = 0, q_end = CAUSAL ? p.n_new : p.n_queries;
  if (LAST) {
    q_begin = first_query;
    q_end = end_query;
  } else if (!CAUSAL) {  // (the first and the last entry of seq_query_start are fixed by the contract)
    if (t > 0) q_begin = CONST_I32(p.seq_query_start)[t];
    if (t + 1 < p.n_seqs) q_end = CONST_I32(p.seq_query_start)[t + 1];
  }
  const int n_t = min(len_t, p.max_seq_len);
  const int n_q = q_end - q_begin;
  const int G = p.group, r = p.rank;
  const int gps = __builtin_ctz(p.group_pad);  // rows per agent: 4, 8 or 16
  const int row0 = rg * 16;
  if (row0 >= (n_q << gps)) return;
  asm volatile("" ::"s"(n_t));
  LRA_STAMP(1);
  // workspace slot of the row this lane stands for (-1: padding row)
  auto row_slot = [&]() -> int64_t {
    const int slot_q = (row0 + ln) >> gps, gg = (row0 + ln) & ((1 << gps) - 1);
    if (!(slot_q < n_q && gg < G)) return -1;
    return (static_cast<int64_t>(q_begin + slot_q) * p.n_q_heads + h * G + gg) * p.n_splits + split;
  };
  if constexpr (LAST) {
    if (last_of_seq && wave == 0) {
      const int64_t slot = row_slot();
      if (slot >= 0)
        for (int s = split + 1 + lg; s < p.n_splits; s += 4) {
          p.part_ml[(slot - split + s) * 2 + 0] = -INFINITY;
          p.part_ml[(slot - split + s) * 2 + 1] = 0.f;
        }
    }
  }
  if (j0 >= n_t) {
    // a share past the end of this sequence: an empty state (zero row sum) is all the merge kernel looks at
    if (wave == 0 && lg == 0) {
      const int64_t slot = row_slot();
      if (slot >= 0) {
        p.part_ml[slot * 2 + 0] = -INFINITY;
        p.part_ml[slot * 2 + 1] = 0.f;
      }
    }
    return;
  }
  // adapters of the tile's agent slots (wave-uniform; device data: kept inside the table), -1 for an empty slot
  const int slot0 = row0 >> gps;
  const int n_live = CAUSAL ? 1 : min(16 >> gps, n_q - slot0);
  int a_slot[4];
#pragma unroll
  for (int si = 0; si < 4; ++si)
    a_slot[si] = si >= n_live ? -1
                 : CAUSAL     ? p.adapter_index
                              : min(max(CONST_I32(p.query_adapter)[q_begin + slot0 + si], 0), p.n_adapters - 1);
  // last key this lane's row may see (causal form only), and the smallest of them in this workgroup
  const int lim = n_t - n_q + min((row0 + ln) >> gps, n_q - 1);
  const int lim_first = n_t - n_q + slot0;

  const int j1 = min(j0 + keys, n_t);
  const int kpw = keys / NW;  // multiple of 32
  const int jw0 = j0 + wave * kpw;
  const int jw1 = max(jw0, min(jw0 + kpw, j1));  // == jw0 for a wave without keys

  unsigned char* ks_lds = smem + wave * WAVE_BYTES;
  unsigned char* vs_lds = ks_lds + KV_BYTES;
  unsigned char* ls_lds = vs_lds + KV_BYTES;
  unsigned char* q_raw = TILE_FIRST ? smem + QRAW_AT : smem + NW * WAVE_BYTES;

  const bf16_t* kb = static_cast<const bf16_t*>(p.k_base);
  const bf16_t* vb = static_cast<const bf16_t*>(p.v_base);
  // (one low-rank cache per adapter: the host gives every agent a row tile, the tile's first slot names the cache)
  const int64_t lp = p.l_row_stride;
  const bf16_t* lr = static_cast<const bf16_t*>(p.l) + (p.l_adapter_stride > 0 ? static_cast<int64_t>(max(a_slot[0], 0)) * p.l_adapter_stride : 0);
  const uint32_t ts2 = static_cast<uint32_t>(p.kv_token_stride) * 2u;  // token stride in bytes
  const uint32_t r2 = static_cast<uint32_t>(r) * 2u;                   // L row in bytes
  const uint32_t lp2 = static_cast<uint32_t>(lp) * 2u;                 // bytes between L rows

  // ===================== tile traffic (layouts and swizzles of decode_mfma_kernel) =====================
  auto swz_k = [](int row) { return D == 128 ? (row & 15) : ((row >> 1) & 7); };
  auto swz_v = [](int row) { return D == 128 ? ((row & 7) << 1) : (((row >> 1) & 3) << 1); };
  auto swz_l = [](int row) { return RP == 16 ? 0 : ((row >> (RP == 32 ? 1 : 0)) & (RCH - 1)); };
  constexpr int KPER = KROWS == 4 ? 4 : 2, VPER = KROWS == 4 ? 2 : 1;
  uint32_t k_voff[KPER], v_voff[VPER], l_voff;
  const int rr = lane / KCH, pc = lane % KCH;
#pragma unroll
  for (int q = 0; q < KPER; ++q) k_voff[q] = static_cast<uint32_t>(rr) * ts2 + ((pc ^ swz_k(q * KROWS + rr)) << 4);
#pragma unroll
  for (int q = 0; q < VPER; ++q) v_voff[q] = static_cast<uint32_t>(rr) * ts2 + ((pc ^ swz_v(q * KROWS + rr)) << 4);
  {
    const int lrow = lane / RCH, lch = (lane % RCH) ^ swz_l(lane / RCH);
    l_voff = (lch * 8 < r) ? static_cast<uint32_t>(PAGED ? lrow & 15 : lrow) * lp2 + (lch << 4) : kOob;
  }
  u32x4 rs_k = {0u, 0u, 0u, 0u}, rs_v = rs_k, rs_l = rs_k;  // contiguous cache: the keys [jw0, jw1) of the wave
  if (!PAGED) {
    const int nk = jw1 - jw0;
    const int64_t base = static_cast<int64_t>(h) * p.kv_head_stride + static_cast<int64_t>(jw0) * p.kv_token_stride;
    const uint32_t bytes = nk > 0 ? static_cast<uint32_t>(nk - 1) * ts2 + D * 2 : 0u;
    rs_k = make_rsrc_words(kb + base, bytes);
    rs_v = make_rsrc_words(vb + base, bytes);
    rs_l = make_rsrc_words(lr + static_cast<int64_t>(jw0) * lp, nk > 0 ? static_cast<uint32_t>(nk - 1) * lp2 + r2 : 0u);
  }
  // paged cache: the two blocks of the tile that is requested next, fetched a tile ahead
  const const_i32_ptr bt = CONST_I32(p.block_table) + static_cast<int64_t>(t) * p.max_blocks_per_seq;
  int blk[2] = {0, 0};
  auto fetch_block_ids = [&](int j) {
    if (PAGED) {
      const int nb_last = (n_t - 1) >> 4;
      blk[0] = bt[min(j >> 4, nb_last)];
      blk[1] = bt[min((j >> 4) + 1, nb_last)];
    }
  };
  fetch_block_ids(jw0);
  // K_base / V_base requests: non-temporal when this workgroup is the only reader of its keys
  const bool stream_kv = p.row_groups == 1;
  // rows of one 32-key tile (from token j) of K_base or V_base into LDS
  auto issue_kv = [&](const bf16_t* base, u32x4 rs, unsigned char* lds, const uint32_t* voff, int per, int j) __attribute__((always_inline)) {
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      uint32_t s0 = static_cast<uint32_t>(j - jw0) + 16 * half;
      if (PAGED) {
        const int nv = max(0, min(16, jw1 - j - 16 * half));  // rows of this block inside the wave's range
        rs = make_rsrc_words(base + static_cast<int64_t>(blk[half]) * p.kv_block_stride + static_cast<int64_t>(h) * p.kv_head_stride,
                             nv > 0 ? static_cast<uint32_t>(nv - 1) * ts2 + D * 2 : 0u);
        s0 = 0;
      }
      constexpr int N = KVL / 2;
      if constexpr (!ONE_CHOICE) {
#pragma unroll
        for (int i = 0; i < N; ++i) {
          if (stream_kv) buf_load16_to_lds<true>(rs, lds + (half * N + i) * 1024, voff[(half * N + i) % per], (s0 + i * KROWS) * ts2);
          else buf_load16_to_lds<false>(rs, lds + (half * N + i) * 1024, voff[(half * N + i) % per], (s0 + i * KROWS) * ts2);
        }
      } else if (stream_kv) {
#pragma unroll
        for (int i = 0; i < N; ++i) buf_load16_to_lds<true>(rs, lds + (half * N + i) * 1024, voff[(half * N + i) % per], (s0 + i * KROWS) * ts2);
      } else {
#pragma unroll
        for (int i = 0; i < N; ++i) buf_load16_to_lds<false>(rs, lds + (half * N + i) * 1024, voff[(half * N + i) % per], (s0 + i * KROWS) * ts2);
      }
    }
  };
  auto issue_l = [&](int j, int stage) __attribute__((always_inline)) {
    unsigned char* dst = ls_lds + stage * L_BYTES;
#pragma unroll
    for (int i = 0; i < LL; ++i) {
      if (PAGED) {
        constexpr int PER_BLOCK = LL / 2;
        const int half = i / PER_BLOCK, nv = max(0, min(16, jw1 - j - 16 * half));
        const u32x4 pl = make_rsrc_words(lr + static_cast<int64_t>(blk[half]) * 16 * lp, nv > 0 ? static_cast<uint32_t>(nv - 1) * lp2 + r2 : 0u);
        if (LROWS < 32) buf_load16_to_lds(pl, dst + i * 1024, l_voff, (i % PER_BLOCK) * LROWS * lp2);
        else if (g2 == half) buf_load16_to_lds(pl, dst, l_voff, 0u);
      } else {
        buf_load16_to_lds(rs_l, dst + i * 1024, l_voff, (static_cast<uint32_t>(j - jw0) + i * LROWS) * lp2);
      }
    }
  };
  auto issue_k = [&](int j) __attribute__((always_inline)) { issue_kv(kb, rs_k, ks_lds, k_voff, KPER, j); };
  auto issue_v = [&](int j) __attribute__((always_inline)) { issue_kv(vb, rs_v, vs_lds, v_voff, VPER, j); };

  // ===================== prologue: Q, B_K^T operands, rotation rates =====================
  // Raw rows of Q (the K swizzle; padding rows read as zeros) and the slices B_K[a][:, h*D .. h*D+D) of the live slots (rows
  // = ranks, the V swizzle; ranks beyond r lie outside the resource: zeros), each by one wave, then this wave's first K and L
  // rows where their regions are free.
  const int64_t ldb = static_cast<int64_t>(p.n_kv_heads) * D;
  if (wave < 16 / KROWS) {
    const u32x4 rs_q = make_rsrc_words(static_cast<const bf16_t*>(p.q) + static_cast<int64_t>(q_begin) * p.n_q_heads * D,
                                       static_cast<uint32_t>(n_q) * p.n_q_heads * D * 2);
    const int R = wave * KROWS + rr;
    const int slot_q = (row0 + R) >> gps, gg = (row0 + R) & ((1 << gps) - 1);
    const uint32_t off = slot_q < n_q && gg < G ? static_cast<uint32_t>((slot_q * p.n_q_heads + h * G + gg) * ROW_BYTES + ((pc ^ swz_k(R)) << 4)) : kOob;
    buf_load16_to_lds(rs_q, q_raw + wave * 1024, off, 0u);
  }
  if (wave < n_live && wave < NSL) {
    const uint32_t ldb2 = static_cast<uint32_t>(ldb) * 2u;
    const int a = wave == 0 ? a_slot[0] : (wave == 1 ? a_slot[1] : (wave == 2 ? a_slot[2] : a_slot[3]));
    const u32x4 rs_b = make_rsrc_words(static_cast<const bf16_t*>(p.b_k) + static_cast<int64_t>(a) * r * ldb + h * D,
                                       static_cast<uint32_t>((r - 1) * ldb + D) * 2u);
    uint32_t bk_voff[VPER];
#pragma unroll
    for (int q = 0; q < VPER; ++q) bk_voff[q] = static_cast<uint32_t>(rr) * ldb2 + ((pc ^ swz_v(q * KROWS + rr)) << 4);
#pragma unroll
    for (int i = 0; i < RPE / KROWS; ++i)
      buf_load16_to_lds(rs_b, (TILE_FIRST ? vs_lds : ks_lds) + i * 1024, bk_voff[i % VPER], i * KROWS * ldb2);
  }
  if (TILE_FIRST && jw0 < jw1) {
    issue_k(jw0);
    issue_l(jw0, 0);
  }
  LRA_STAMP(2);
  // (under the requests) phases are formed in double precision, lane = pair, so that positions in the tens of thousands
  // lose nothing; a lane adds its key's own offset in single precision
  if (wave == 0) {
    const double rate = rope_rate_rev(lane & (D / 2 - 1), D, p.key_rope_theta);
    rate_tab[lane] = rate;
    rope_tab[lane] = static_cast<float>(rate);
  }
  float* phase_w = rope_tab + 64 + wave * 64;
  if (wave == 0 && lane < DB) *reinterpret_cast<uint4*>(q_op + 32 * QOP_STRIDE + lane * 16) = make_uint4(0u, 0u, 0u, 0u);
  // requests retire in order: with at most the tile's outstanding, this wave's Q rows and slice have landed
  if (TILE_FIRST && jw0 < jw1) wait_vm<KVL + LL>();
  else wait_vm0();
  lds_fence();
  __syncthreads();
  // Q in the order rot(E) comes out of its product: piece kk = (32-pair block, half of the head, 16-feature half q) of entry
  // (row, g2) holds features 32 block + 16 q + 4 g2 + {0..3, 8..11} (+ D/2)
#pragma unroll
  for (int i = 0; i < DB / NW; ++i) {
    const int kk = wave + i * NW, ch = 4 * (kk >> 2) + 2 * (kk & 1) + (D / 16) * ((kk >> 1) & 1);
    const unsigned char* row = q_raw + ln * ROW_BYTES + 8 * g2;
    const uint2 a = lds_read8(row + ((ch ^ swz_k(ln)) << 4)), b = lds_read8(row + (((ch + 1) ^ swz_k(ln)) << 4));
    *reinterpret_cast<uint4*>(q_op + (ln + 16 * g2) * QOP_STRIDE + kk * 16) = make_uint4(a.x, a.y, b.x, b.y);
  }
  // bkt[slot][block][ek]: lane (feature 32 block + l32, rank 16ek + 8g2 + e), the A operand of E^T
  bf16x8 bkt[NSL][2 * PB][EK];
#pragma unroll
  for (int si = 0; si < NSL; ++si) {
    const unsigned char* slice = smem + si * WAVE_BYTES + (TILE_FIRST ? KV_BYTES : 0);
#pragma unroll
    for (int b = 0; b < 2 * PB; ++b)
#pragma unroll
      for (int ek = 0; ek < EK; ++ek) {
        s16x4 half[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int rank = 16 * ek + 8 * g2 + 4 * q + (ln >> 2), ch = 4 * b + 2 * (lg & 1) + ((ln & 3) >> 1);
          half[q] = lds_read_tr16(slice + rank * ROW_BYTES + ((ch ^ swz_v(rank)) << 4) + (ln & 1) * 8);
        }
        bkt[si][b][ek] = join_tr(half[0], half[1]);
      }
  }
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the regions are about to be written again
  lds_fence();
  __syncthreads();
  if (jw0 < jw1) {
    if (!TILE_FIRST) {
      issue_k(jw0);
      issue_l(jw0, 0);
    }
    issue_v(jw0);
    fetch_block_ids(jw0 + 32);
  }
  LRA_STAMP(3);

  // ===================== main loop =====================
  const int kg = 8 * (lg & 1) + 4 * (lg >> 1);  // first key of this lane's four in a 16-key tile (see the top)
  const int krow = (ln & 3) | ((ln & 4) << 1) | ((ln & 8) >> 1);
  // (K_base Q^T takes its features in the order of q_op too: lane group lg the pieces q = lg / 2 of entry g2 = lg % 2, two
  // 8-byte reads of a K row for every 32 features; Q in operand order of its own would take 16 registers more)
  int k_pre = krow * ROW_BYTES + ((swz_k(krow) ^ (2 * (lg >> 1))) << 4) + 8 * (lg & 1);
  const int q_pre = (ln + 16 * (lg & 1)) * QOP_STRIDE + (lg >> 1) * 16;
  const int ka = kg + (ln >> 2);  // row (within a 16-key tile) this lane addresses in transpose reads
  int v_pre = ka * ROW_BYTES + ((swz_v(ka) + ((ln & 3) >> 1)) << 4) + (ln & 1) * 8;
  int lt_rd[RB];  // L^T as A operand of Olr^T
#pragma unroll
  for (int b = 0; b < RB; ++b) lt_rd[b] = ka * (2 * RP) + (((2 * b + ((ln & 3) >> 1)) ^ swz_l(ka)) << 4) + (ln & 1) * 8;
  const int q_mine = (ln + 16 * g2) * QOP_STRIDE;
  bf16x8 q_held[HOLD_Q ? DB : 1];
  if constexpr (HOLD_Q) {
#pragma unroll
    for (int kk = 0; kk < DB; ++kk) q_held[kk] = as_bf16x8(lds_read16(q_op + q_mine + kk * 16));
  }
  f32x4 o_acc[DB], lr_acc[RB];
  float m_run = -INFINITY, l_run = 0.f;  // m_run in base-2 units of the scaled score
  [[maybe_unused]] float m_top = -INFINITY;
#pragma unroll
  for (int b = 0; b < DB; ++b) o_acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int b = 0; b < RB; ++b) lr_acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float sc = p.scale * 1.44269504088896340736f;

  int l_at = 0;  // stage of the step's L rows, in bytes
  for (int j = jw0; j < jw1; j += 32) {
    const bool more = j + 32 < jw1;
    const unsigned char* lt = ls_lds + l_at;
    // (above rank 16: the addresses derived from these are formed in the loop, not held in sixteen registers around it)
    if constexpr (RPE > 16) asm volatile("" : "+v"(k_pre), "+v"(v_pre));
    wait_vm<KVL>();  // all but the V rows, the youngest requests, have landed
    lds_fence();
    if (j == jw0) LRA_STAMP(4);
    {
      double rev = static_cast<double>(j) * rate_tab[lane];
      rev -= floor(rev);
      phase_w[lane] = static_cast<float>(rev);
    }
    // L^T as B operand of E^T: lane (key l32, rank 16ek + 8g2 + e); held for all slots only where that is four registers
    auto l_operand = [&](int ek) __attribute__((always_inline)) {
      return as_bf16x8(lds_read16(lt + l32 * (2 * RP) + (((2 * ek + g2) ^ swz_l(l32)) << 4)));
    };
    bf16x8 lop;
    if constexpr (EK == 1) lop = l_operand(0);
    f32x4 s[2];
#pragma unroll
    for (int tt = 0; tt < 2; ++tt) s[tt] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {  // 32 features: block ks % PB of half ks / PB of the head
      const bf16x8 q8 = as_bf16x8(lds_read16(q_op + q_pre + (4 * (ks % PB) + 2 * (ks / PB)) * 16));
#pragma unroll
      for (int tt = 0; tt < 2; ++tt) {
        const uint2 a = lds_read8(ks_lds + (k_pre ^ (ks << 6)) + tt * 16 * ROW_BYTES), b = lds_read8(ks_lds + (k_pre ^ (ks << 6) ^ 16) + tt * 16 * ROW_BYTES);
        s[tt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(make_uint4(a.x, a.y, b.x, b.y)), q8, s[tt], 0, 0, 0);
      }
    }
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the K rows have been read
    lds_fence();
    if (more) {
      issue_k(j + 32);
      if (TWO_L) issue_l(j + 32, l_at == 0 ? 1 : 0);
    }
    // scores of the rotated part: lane (row l32 % 16, keys 8(i/4) + 4g2 + i%4 of register i)
    pf_f32x16 s_rot;
#pragma unroll
    for (int i = 0; i < 16; ++i) s_rot[i] = 0.f;
    const float keyf = static_cast<float>(l32);
#pragma unroll
    for (int pb = 0; pb < PB; ++pb) {
      float cs[16], sn[16];  // of pair 32 pb + 8(i/4) + 4g2 + i%4 at key l32
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4 rate4 = *reinterpret_cast<const f32x4*>(rope_tab + 32 * pb + 8 * q + 4 * g2);
        const f32x4 phase4 = *reinterpret_cast<const f32x4*>(phase_w + 32 * pb + 8 * q + 4 * g2);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const float fr = fmaf(keyf, rate4[jj], phase4[jj]);
          sn[4 * q + jj] = __builtin_amdgcn_sinf(fr);
          cs[4 * q + jj] = __builtin_amdgcn_cosf(fr);
        }
      }
#pragma unroll
      for (int si = 0; si < NSL; ++si) {
        if (si > 0 && si >= n_live) continue;
        [[maybe_unused]] const int q_at = (ln >> gps) == si ? q_mine : 32 * QOP_STRIDE;
        pf_f32x16 e_lo, e_hi;
#pragma unroll
        for (int i = 0; i < 16; ++i) e_lo[i] = e_hi[i] = 0.f;
#pragma unroll
        for (int ek = 0; ek < EK; ++ek) {
          if constexpr (EK > 1) lop = l_operand(ek);
          e_lo = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bkt[si][pb][ek], lop, e_lo, 0, 0, 0);
          e_hi = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bkt[si][pb + PB][ek], lop, e_hi, 0, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          uint32_t lo[4], hi[4];
#pragma unroll
          for (int x = 0; x < 4; ++x) {
            const int i = 8 * q + 2 * x;
            lo[x] = pack_bf16x2(e_lo[i] * cs[i] - e_hi[i] * sn[i], e_lo[i + 1] * cs[i + 1] - e_hi[i + 1] * sn[i + 1]);
            hi[x] = pack_bf16x2(e_hi[i] * cs[i] + e_lo[i] * sn[i], e_hi[i + 1] * cs[i + 1] + e_lo[i + 1] * sn[i + 1]);
          }
          bf16x8 q_lo, q_hi;
          if constexpr (HOLD_Q) {
            q_lo = q_held[pb * 4 + q];
            q_hi = q_held[pb * 4 + 2 + q];
          } else {
            q_lo = as_bf16x8(lds_read16(q_op + q_at + (pb * 4 + q) * 16));
            q_hi = as_bf16x8(lds_read16(q_op + q_at + (pb * 4 + 2 + q) * 16));
          }
          s_rot = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(make_uint4(lo[0], lo[1], lo[2], lo[3])), q_lo, s_rot, 0, 0, 0);
          s_rot = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(make_uint4(hi[0], hi[1], hi[2], hi[3])), q_hi, s_rot, 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        float even = s_rot[8 * tt + jj], odd = s_rot[8 * tt + 4 + jj];
        asm("" : "+v"(even), "+v"(odd));  // (two registers: a choice of index would become a search through all sixteen)
        s[tt][jj] += (lg & 1) ? odd : even;
      }

    // online softmax; element (tt, jj) of this lane is key j + 16tt + kg + jj of row ln
    if (j + 32 > jw1 || (CAUSAL && j + 31 > lim_first)) {
#pragma unroll
      for (int tt = 0; tt < 2; ++tt)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const int key = j + tt * 16 + kg + jj;
          if (key >= jw1 || (CAUSAL && key > lim)) s[tt][jj] = -INFINITY;
        }
    }
    float mx = fmaxf(fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3])), fmaxf(fmaxf(s[1][0], s[1][1]), fmaxf(s[1][2], s[1][3])));
    mx = max_over_lane_groups(mx) * sc;  // sc > 0
    // (LAST: every 32 keys against their own maximum, see decode_mfma_kernel)
    if (LAST || __builtin_amdgcn_ballot_w64(mx > m_run) != 0) {
      if (LAST) m_top = fmaxf(m_top, mx);
      const float m_new = LAST ? fmaxf(mx, m_top - 16.f) : fmaxf(m_run, mx);
      // causal form: a row may have seen no key yet (both maxima -inf)
      const float alpha = (CAUSAL && m_new == -INFINITY) ? 1.f : fast_exp2(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int b = 0; b < DB; ++b) o_acc[b] *= alpha;
#pragma unroll
      for (int b = 0; b < RB; ++b) lr_acc[b] *= alpha;
    }
    const float nm = (CAUSAL && m_run == -INFINITY) ? 0.f : -m_run;
    float pe[8], sum = 0.f;
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int jj = 0; jj < 4; ++jj) {
        pe[tt * 4 + jj] = fast_exp2(fmaf(s[tt][jj], sc, nm));
        sum += pe[tt * 4 + jj];
      }
    l_run += sum;
    const bf16x8 pb8 = as_bf16x8(make_uint4(pack_bf16x2(pe[0], pe[1]), pack_bf16x2(pe[2], pe[3]), pack_bf16x2(pe[4], pe[5]), pack_bf16x2(pe[6], pe[7])));
    // Olr^T += L^T P^T, then the V rows: O^T += V^T P^T
#pragma unroll
    for (int b = 0; b < RB; ++b) {
      const bf16x8 a = join_tr(lds_read_tr16(lt + lt_rd[b]), lds_read_tr16(lt + lt_rd[b] + 16 * 2 * RP));
      lr_acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, pb8, lr_acc[b], 0, 0, 0);
    }
    if (!TWO_L) {
      __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the L rows have been read
      lds_fence();
      if (more) issue_l(j + 32, 0);
    }
    if (more) wait_vm<KVL + LL>();  // (the next K and L rows are younger)
    else wait_vm0();
    lds_fence();
#pragma unroll
    for (int b = 0; b < DB; ++b) {
      const unsigned char* src = vs_lds + (v_pre ^ (b << 5));
      o_acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(join_tr(lds_read_tr16(src), lds_read_tr16(src + 16 * ROW_BYTES)), pb8, o_acc[b], 0, 0, 0);
    }
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the V rows have been read
    lds_fence();
    if (j == jw0) LRA_STAMP(5);
    if (more) {
      issue_v(j + 32);
      fetch_block_ids(j + 64);
    }
    if (TWO_L) l_at ^= L_BYTES;
  }
  LRA_STAMP(6);

  // One workgroup per (sequence, kv head, row group) touches the B_V rows the merge kernel will need (one 4-byte read per
  // 128-byte line), so that they wait in this XCD's L2: wave w takes agent slot w.
  int warm[2] = {0, 0};
  {
    const int a = wave == 0 ? a_slot[0] : (wave == 1 ? a_slot[1] : (wave == 2 ? a_slot[2] : a_slot[3]));
    if (p.b_v != nullptr && split == min(1, p.n_splits - 1) && a >= 0) {
      constexpr int LPR = ROW_BYTES / 128;  // 128-byte lines per B_V row of one kv head
      const char* bv = static_cast<const char*>(p.b_v) + (static_cast<int64_t>(a) * r * ldb + static_cast<int64_t>(h) * D) * 2;
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int li = i * 64 + lane;
        if (li < r * LPR) warm[i] = *reinterpret_cast<const int*>(bv + static_cast<int64_t>(li / LPR) * ldb * 2 + (li % LPR) * 128);
      }
    }
  }

  // ===================== merge the waves of this workgroup =====================
  // Every wave deposits its state as it stands in its own region; after one barrier wave w sums blocks w, w + 4, ... of all
  // four with the weights 2^(m_w' - max m), in wave order, and stores them.
  {
    unsigned char* mine = smem + wave * WAVE_BYTES;
#pragma unroll
    for (int b = 0; b < DB; ++b) *reinterpret_cast<f32x4*>(mine + b * 1024 + lane * 16) = o_acc[b];
#pragma unroll
    for (int b = 0; b < RB; ++b) *reinterpret_cast<f32x4*>(mine + (DB + b) * 1024 + lane * 16) = lr_acc[b];
    *reinterpret_cast<f32x2*>(mine + NBLK * 1024 + lane * 8) = f32x2{m_run, sum_over_lane_groups(l_run)};
  }
  __syncthreads();
  LRA_STAMP(7);
  const int64_t slot = row_slot();
  if (slot >= 0) {
    float wgt[NW], m_all = -INFINITY, l_all = 0.f;
    f32x2 ml[NW];
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      ml[w] = *reinterpret_cast<const f32x2*>(smem + w * WAVE_BYTES + NBLK * 1024 + lane * 8);
      m_all = fmaxf(m_all, ml[w][0]);
    }
    // m_all is finite (wave 0 always owns a key) unless a causal row sees none of this share
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      wgt[w] = ml[w][0] == -INFINITY ? 0.f : fast_exp2(ml[w][0] - m_all);
      l_all = fmaf(wgt[w], ml[w][1], l_all);
    }
#pragma unroll
    for (int x = 0; x < NBLK; ++x) {
      if ((x & (NW - 1)) != wave) continue;  // wave-uniform
      f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const f32x4 part = *reinterpret_cast<const f32x4*>(smem + w * WAVE_BYTES + x * 1024 + lane * 16);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) v[jj] = fmaf(wgt[w], part[jj], v[jj]);
      }
      const int rho = (x - DB) * 16 + lg * 4;  // (the rank is a multiple of 8: four entries are inside or outside together)
      if (x < DB) *reinterpret_cast<f32x4*>(p.part_o + slot * D + x * 16 + lg * 4) = v;
      else if (rho < r) *reinterpret_cast<f32x4*>(p.part_lr + slot * r + rho) = v;
    }
    if (wave == NW - 1 && lg == 0) {
      p.part_ml[slot * 2 + 0] = m_all * 0.69314718055994530942f;  // natural-log units
      p.part_ml[slot * 2 + 1] = l_all;
      if (split == 0) {  // (the merge kernel takes each row's adapter from the workspace)
        const int si = ln >> gps;
        p.part_adapter[slot / p.n_splits] = CAUSAL ? p.adapter_index : (si == 0 ? a_slot[0] : (si == 1 ? a_slot[1] : (si == 2 ? a_slot[2] : a_slot[3])));
      }
    }
  }
  asm volatile("" ::"v"(warm[0]), "v"(warm[1]));
  LRA_STAMP(8);
#ifdef LRA_TIMING
  asm volatile("s_waitcnt vmcnt(0)");
#endif
  LRA_STAMP(9);
  LRA_STAMP_FLUSH();
}

}  // namespace lra
