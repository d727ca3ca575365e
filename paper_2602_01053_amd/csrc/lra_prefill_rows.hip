// Causal prefill of a few rows per workgroup (bf16, gfx950): the waves of a workgroup share its 32 query rows and
// divide its KEYS.
//
// The arithmetic is that of prefill_mfma_kernel (scores transposed, App. D.1 key-side reordering,
// v_mfma_f32_32x32x16_bf16, lazily raised softmax reference, row sums on the matrix core at rank 16).  There a
// workgroup owns 128 rows and its four waves walk all keys together, which leaves most of the chip idle in a call of
// some tens or hundreds of new tokens; what is idle can only be filled by dividing the keys among workgroups, at the
// price of a second kernel and of partial states in memory.  Here eight waves share 32 rows, wave w takes the 32-key
// tiles w, w + 8, ..., and the eight states meet in LDS: four times the workgroups, an eighth of the steps, one kernel.
// 62 new tokens on 525 keys, 8 kv heads of group 4: 17.2 -> 9.9 us; 198 on 2199, rank 32: 31.4 -> 20.4 us.
//
// SHARED: p.n_splits workgroups divide the keys of the 32 rows as well (even stretches of 32-key tiles), each leaves one
// state per live row in the workspace and the merge kernel finishes.  For calls of about ten to a hundred tokens on long
// contexts, where one workgroup per 32 rows leaves units idle: 40 after 9000 21.9 -> 17.9 us (see plan_wave_shares).
//
// The softmax reference is raised lazily (kSlack), which leaves the largest probability of a tile anywhere in eight octaves
// and rounds it to bf16; over many tiles, and in the walk of 128 rows, that is no loss.  Calls of the split-KV path's sizes come
// from kernels that took the maximum of about every 32 keys, so that it is exact; where a wave sees a few tiles their
// error against float64 was 1.02 to 1.17 times as large (31 tokens on 846 2.15e-3 -> 2.40e-3).  They take every tile's own
// maximum here (kPrOwn, at most 2^kReach below the largest so far, which keeps the sums in range): 0.93 to 1.0 times, at
// 0.1 us per 256 keys.  (As an argument of the call rather than a form of its own it cost the other calls 0.8 %.)
//
// A wave owns its tiles, so nothing in its loop waits for another wave.  K, L and V have one place each per wave: the
// next K rows are requested when the scores have been taken, the next L and V rows behind the second product, and the
// other wave of the SIMD computes meanwhile.  What bounds the loop is the way from L2 into LDS: 136 KB per 256 keys at
// about 100 GB/s per compute unit, 1.35 us (a wave with 64 rows, which halves that, holds 2 x 80 accumulators and has
// to read Q from LDS in every step: 2.3 us).  Outside the loop 6.5 us: launch, two round trips to memory, the exchange.
#include "lra_prefill_util.h"

namespace lra {

template <int N>
__device__ __forceinline__ void pr_wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N)); }
// every LDS read of this wave has returned, and none moves across (the requests that follow overwrite what was read)
__device__ __forceinline__ void pr_reads_done() {
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
}
__device__ __forceinline__ void pr_fence() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront"); }

enum PrKind { kPrQt = 0, kPrValueOnly = 1, kPrKeysF16 = 2 };  // key-side adapter on Qt; none; completed fp16 keys of the pre-pass
enum PrMode { kPrWhole = 0, kPrShared = 1, kPrOwn = 2 };  // all keys of the 32 rows; a share of them; all, and own references

template <int D, int RP, bool PAGED, int KIND, int MODE>
__global__ __launch_bounds__(512, 2) void prefill_rows_kernel(Params p) {
  static_assert(RP == 16 || RP == 32, "one 32-row block of Olr^T");
  constexpr bool HAS_BK = KIND == kPrQt, KF16 = KIND == kPrKeysF16, SHARED = MODE == kPrShared, OWN = MODE == kPrOwn;
  constexpr int NW = 8, BK = 32, BM = 32;
  constexpr int KS = D / 16, RKS = RP / 16, DB = D / 32;
  constexpr int KCH = D / 8, LCH = RP / 8;
  constexpr int KROWS = 64 / KCH, LROWS = 64 / LCH;
  constexpr int KVL = BK / KROWS, LL = BK / LROWS;  // requests per K (or V) tile and per L tile
  constexpr int TL = 2 * KVL + LL;
  constexpr int KV_BYTES = BK * D * 2, L_BYTES = BK * RP * 2, WT = 2 * KV_BYTES + L_BYTES;
  constexpr bool ONES_ROW = RP == 16;  // idle rows of Olr^T take the softmax row sums
  constexpr int Q_AT = NW * WT, Q_BYTES = BM * D * 2;
  // merging: per wave the state of the 32 rows, [half O block][row][16 columns] (waves below 2 DB keep the one they finish in
  // registers), [row][rho], then (m, l) per row; behind the states the sum of Olr
  constexpr int HALF = 32 * 16 * 4, LR_BYTES = 32 * RP * 4;
  constexpr int SLOT = 2 * DB * HALF + LR_BYTES + 256, SLOT_SHORT = SLOT - HALF;
  constexpr int STATES = 2 * DB * SLOT_SHORT + (NW - 2 * DB) * SLOT;
  constexpr int LR_SUM_AT = STATES;
  constexpr int B_AT = Q_AT + Q_BYTES > STATES + LR_BYTES ? Q_AT + Q_BYTES : STATES + LR_BYTES, B_BYTES = RP * D * 2;  // rows of B_K, then of B_V
  constexpr int ONES_AT = B_AT + B_BYTES;
  constexpr int SMEM = ONES_AT + (ONES_ROW ? 16 : 0);
  static_assert(SMEM <= 160 * 1024, "LDS of one compute unit");
  constexpr float kSlack = 8.0f, kReach = 16.0f;  // (powers of two)

  __shared__ __align__(16) unsigned char smem[SMEM];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, g2 = lane >> 5;
  const int Hq = p.n_q_heads, Hkv = p.n_kv_heads, r = p.rank, G = p.tile_group;
  // Consecutive ids go to consecutive XCDs: a kv head stays on one, or the workgroups that read a key share of it do
  const int n_shares = SHARED ? p.n_splits : 1;
  const int lin = blockIdx.x;
  const int qt = lin / (Hkv * n_shares), in_qt = lin - qt * (Hkv * n_shares);
  const int share = SHARED ? in_qt / Hkv : 0, hk = in_qt - share * Hkv;
  const int t = p.seq_index, a_idx = p.adapter_index, n_new = p.n_new;
  const int32_t len_t = PF_CONST_I32(p.seq_lens)[t];  // (on its way while Q and B_K are asked for)
  const int n_rows = n_new * G, q0 = qt * BM;
  const int tok0 = q0 / G, head0 = q0 - tok0 * G;
  const int live_rows = min(BM, n_rows - q0);
  // (token - tok0, q head) of a row of the tile, the last live row's for one past the end; the quotient of at most
  // 47 by at most 16 is exact by the multiplication
  auto map_row = [&](int in_tile, int& tok, int& gq) __attribute__((always_inline)) {
    const int at = head0 + min(in_tile, live_rows - 1);
    tok = (at * p.row_mul) >> 16;
    gq = at - tok * G;
  };
  const int64_t row_base = static_cast<int64_t>(tok0) * Hq + hk * p.group;
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(PF_LDS_AS(unsigned char, smem)));
  const int rr = lane / KCH, pc = lane % KCH;
  // wave w asks for KROWS rows of Q, in the layout of K rows, and of B_K, then of its first tile
  const int row_w = wave * KROWS + rr;
  const uint32_t chunk_w = static_cast<uint32_t>(pc ^ pf_swz_k<D>(row_w)) << 4;
  if (wave * KROWS < BM) {
    const pf_u32x4 rs_q = pf_rsrc(static_cast<const bf16_t*>(p.q) + row_base * D, kPfPoolBytes);  // (rows of at most 33 tokens)
    int tok, gq;
    map_row(row_w, tok, gq);
    pf_load16_to_lds(rs_q, lds0 + Q_AT + wave * 1024, static_cast<uint32_t>(tok * Hq + gq) * (D * 2) + chunk_w, 0);
  }
  // KROWS rows of an adapter's B_K or B_V for the kv head; rows past the rank lie outside the resource and read as zero
  const uint32_t ldb2 = static_cast<uint32_t>(Hkv) * (D * 2);
  auto issue_b = [&](const void* b, uint32_t lds_at, uint32_t chunk) __attribute__((always_inline)) {
    if (wave * KROWS >= RP) return;
    const pf_u32x4 rs_b = pf_rsrc(static_cast<const bf16_t*>(b) + (static_cast<int64_t>(a_idx) * r * Hkv + hk) * D,
                                  static_cast<uint32_t>(r - 1) * ldb2 + D * 2);
    pf_load16_to_lds(rs_b, lds0 + lds_at + wave * 1024, static_cast<uint32_t>(row_w) * ldb2 + chunk, 0);
  };
  static_assert(RP / KROWS <= NW && BM / KROWS <= NW, "one request per wave");
  if constexpr (HAS_BK) issue_b(p.b_k, B_AT, chunk_w);

  const int n_t = min(len_t, p.max_seq_len);
  const int base_vis = n_t - n_new;  // new token i sees keys 0 .. base_vis + i
  int tok_mine, gq_mine, tok_last, gq_last;
  map_row(l32, tok_mine, gq_mine);
  map_row(BM - 1, tok_last, gq_last);
  const int limit = base_vis + tok0 + tok_mine;  // last key the lane's row sees
  const int first_limit = base_vis + tok0;
  const int all_tiles = (base_vis + tok0 + tok_last) / BK + 1;  // that the workgroup's rows see
  const int tile0 = SHARED ? static_cast<int>(static_cast<int64_t>(all_tiles) * share / n_shares) : 0;
  const int n_tiles = SHARED ? static_cast<int>(static_cast<int64_t>(all_tiles) * (share + 1) / n_shares) : all_tiles;
  const int64_t out_row = row_base + static_cast<int64_t>(tok_mine) * Hq + gq_mine;
  const int64_t slot = SHARED ? out_row * n_shares + share : 0;
  if (SHARED && tile0 >= n_tiles) {  // fewer tiles than shares: no key, which the merge kernel reads off the row sum
    pf_wait_vm0();
    if (tid < BM && tid < live_rows) {
      *reinterpret_cast<pf_f32x2*>(p.part_ml + slot * 2) = pf_f32x2{-INFINITY, 0.f};
      if (share == 0) p.part_adapter[out_row] = a_idx;
    }
    return;
  }

  // ---------------- requests: HBM -> LDS, no registers in between ----------------
  const uint32_t lds_w = lds0 + wave * WT;
  const uint32_t ts2 = static_cast<uint32_t>(p.kv_token_stride) * 2u, bs2 = static_cast<uint32_t>(p.kv_block_stride) * 2u;
  const uint32_t r2 = static_cast<uint32_t>(r) * 2u, lp2 = static_cast<uint32_t>(p.l_row_stride) * 2u;
  const bf16_t* lr_base = static_cast<const bf16_t*>(p.l) + static_cast<int64_t>(a_idx) * p.l_adapter_stride;
  // the swizzle of row i * KROWS + rr repeats with period 16 rows (K) and 4 rows (V) or less in i
  constexpr int KPER = 16 / KROWS, VPER = 4 / KROWS > 0 ? 4 / KROWS : 1;
  uint32_t k_voff[KPER], v_voff[VPER], l_voff;
#pragma unroll
  for (int i = 0; i < KPER; ++i) k_voff[i] = static_cast<uint32_t>(rr) * ts2 + ((pc ^ pf_swz_k<D>(i * KROWS + rr)) << 4);
#pragma unroll
  for (int i = 0; i < VPER; ++i) v_voff[i] = static_cast<uint32_t>(rr) * ts2 + ((pc ^ pf_swz_v<D>(i * KROWS + rr)) << 4);
  const int lrow = lane / LCH, lch = (lane % LCH) ^ pf_swz_l<LCH>(lrow);  // (the swizzle repeats from request to request)
  const bool l_ok = lch * 8 < r;
  l_voff = l_ok ? static_cast<uint32_t>(lrow) * lp2 + (lch << 4) : kPfOob;
  pf_u32x4 rs_k, rs_v, rs_l;
  {
    const int64_t hoff = static_cast<int64_t>(hk) * p.kv_head_stride;
    const uint32_t kv_bytes = PAGED ? kPfPoolBytes : static_cast<uint32_t>(n_t - 1) * ts2 + D * 2;
    rs_k = pf_rsrc(static_cast<const bf16_t*>(p.k_base) + hoff, kv_bytes);
    rs_v = pf_rsrc(static_cast<const bf16_t*>(p.v_base) + hoff, kv_bytes);
    rs_l = pf_rsrc(lr_base, (PAGED ? static_cast<uint32_t>(p.num_blocks) * 16u - 1u : static_cast<uint32_t>(n_t - 1)) * lp2 + r2);
  }
  // Paged: lane l holds the id of block (l & 1) of this wave's tile number (l >> 1), all the tiles it can have
  const int nb_last = (n_t - 1) >> 4;
  int ids = 0;
  if (PAGED) ids = p.block_table[static_cast<int64_t>(t) * p.max_blocks_per_seq + min(2 * (tile0 + wave + NW * (lane >> 1)) + (lane & 1), nb_last)];
  // the wave's tile number `step`, which starts at key j
  auto issue_k = [&](int j, int step) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < KVL; ++i) {
      if constexpr (PAGED) {
        const int tok = j + i * KROWS;
        const uint32_t in_blk = static_cast<uint32_t>(tok & 15) * ts2;
        // (completed keys left by the pre-pass lie at the block's logical index)
        const uint32_t blk = KF16 ? static_cast<uint32_t>(min(tok >> 4, nb_last))
                                  : static_cast<uint32_t>(__builtin_amdgcn_readlane(ids, 2 * step + (i * KROWS >= 16)));
        pf_load16_to_lds(rs_k, lds_w + i * 1024, tok + rr < n_t ? k_voff[i % KPER] : kPfOob, blk * bs2 + in_blk);
      } else {
        pf_load16_to_lds(rs_k, lds_w + i * 1024, k_voff[i % KPER], static_cast<uint32_t>(j + i * KROWS) * ts2);
      }
    }
  };
  auto issue_lv = [&](int j, int step) __attribute__((always_inline)) {
    uint32_t blk[2] = {0u, 0u};
    if constexpr (PAGED) {
      blk[0] = static_cast<uint32_t>(__builtin_amdgcn_readlane(ids, 2 * step));
      blk[1] = static_cast<uint32_t>(__builtin_amdgcn_readlane(ids, 2 * step + 1));
    }
#pragma unroll
    for (int i = 0; i < LL; ++i) {
      const uint32_t dst = lds_w + 2 * KV_BYTES + i * 1024;
      if constexpr (PAGED) {
        const int in_tile = i * LROWS + lrow;
        const uint32_t b = in_tile < 16 ? blk[0] : blk[1];
        const uint32_t voff = l_ok && j + in_tile < n_t ? (b * 16u + static_cast<uint32_t>(in_tile & 15)) * lp2 + (lch << 4) : kPfOob;
        pf_load16_to_lds(rs_l, dst, voff, 0);
      } else {
        pf_load16_to_lds(rs_l, dst, l_voff, static_cast<uint32_t>(j + i * LROWS) * lp2);
      }
    }
#pragma unroll
    for (int i = 0; i < KVL; ++i) {
      const uint32_t dst = lds_w + KV_BYTES + i * 1024;
      if constexpr (PAGED) {
        const int tok = j + i * KROWS;
        pf_load16_to_lds(rs_v, dst, tok + rr < n_t ? v_voff[i % VPER] : kPfOob,
                         blk[i * KROWS >= 16] * bs2 + static_cast<uint32_t>(tok & 15) * ts2);
      } else {
        pf_load16_to_lds(rs_v, dst, v_voff[i % VPER], static_cast<uint32_t>(j + i * KROWS) * ts2);
      }
    }
  };

  const bool has_tile = tile0 + wave < n_tiles;
  if (ONES_ROW && tid == 0) *reinterpret_cast<pf_u32x4*>(smem + ONES_AT) = pf_u32x4{0x00003f80u, 0u, 0u, 0u};
  if (has_tile) {
    issue_k((tile0 + wave) * BK, 0);
    issue_lv((tile0 + wave) * BK, 0);
    pr_wait_vm<TL>();  // only the tile is outstanding: the Q and B_K rows have landed
  } else {
    pf_wait_vm0();
  }
  __syncthreads();

  // ---------------- Q operands, Qt = Q B_K^T ----------------
  // K (and Q, B_K) rows as operands: row l32, logical chunk 2ks + g2 at chunk ^ swizzle
  const int k_pre = l32 * (D * 2) + (pf_swz_k<D>(l32) << 4);
  pf_bf16x8 qb[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    const pf_bf16x8 v = pf_as_bf16x8(*reinterpret_cast<const uint4*>(smem + Q_AT + (k_pre ^ ((2 * ks + g2) << 4))));
    qb[ks] = KF16 ? __builtin_bit_cast(pf_bf16x8, pf_bf16x8_to_f16x8(v)) : v;
  }
  pf_bf16x8 qtb[RKS];
  if constexpr (HAS_BK) {
    const int rho = l32 & (RP - 1);  // (RP = 16: the upper half of the product is not used)
    const int b_pre = B_AT + rho * (D * 2) + (pf_swz_k<D>(rho) << 4);
    pf_f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks)
      acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pf_as_bf16x8(*reinterpret_cast<const uint4*>(smem + (b_pre ^ ((2 * ks + g2) << 4)))), qb[ks], acc, 0, 0, 0);
#pragma unroll
    for (int ks = 0; ks < RKS; ++ks) {
      const int o = ks * 8;
      qtb[ks] = pf_as_bf16x8(make_uint4(pf_pack2(acc[o + 0], acc[o + 1]), pf_pack2(acc[o + 2], acc[o + 3]),
                                        pf_pack2(acc[o + 4], acc[o + 5]), pf_pack2(acc[o + 6], acc[o + 7])));
    }
  }

  const bool has_bv = !SHARED && p.b_v != nullptr;  // (with shares the merge kernel applies B_V)
  if (has_bv) {
    if constexpr (HAS_BK) {
      pr_reads_done();
      __syncthreads();  // everybody has read B_K
    }
    issue_b(p.b_v, B_AT, static_cast<uint32_t>(pc ^ pf_swz_v<D>(row_w)) << 4);  // in the layout of V rows
  }

  // ---------------- per-lane LDS read offsets (as in prefill_mfma_kernel) ----------------
  const unsigned char* tile_lds = smem + wave * WT;
  const int a16 = lane & 15, dsel = (lane >> 4) & 1, vrow = 4 * g2 + (a16 >> 2);
  const int v_pre = KV_BYTES + vrow * (D * 2) + ((((a16 & 3) >> 1) + 2 * dsel + pf_swz_v<D>(vrow)) << 4) + (a16 & 1) * 8;
  int l_rd[RKS][2], lt_rd[2];
#pragma unroll
  for (int ks = 0; ks < RKS; ++ks)
#pragma unroll
    for (int c = 0; c < 2; ++c) l_rd[ks][c] = 2 * KV_BYTES + l32 * (RP * 2) + (((2 * ks + c) ^ pf_swz_l<LCH>(l32)) << 4) + g2 * 8;
#pragma unroll
  for (int hh = 0; hh < 2; ++hh) {
    const int key = vrow + 8 * hh, ch = 2 * dsel + ((a16 & 3) >> 1);
    lt_rd[hh] = 2 * KV_BYTES + key * (RP * 2) + (((ch & (LCH - 1)) ^ pf_swz_l<LCH>(key)) << 4) + (a16 & 1) * 8;
  }
  const bool ones_lane = ONES_ROW && dsel == 1;

  // ---------------- main loop ----------------
  pf_f32x16 o_acc[DB], lr_acc;
  float m_run = -INFINITY, l_run = 0.f;
  [[maybe_unused]] float m_top = -INFINITY;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    lr_acc[i] = 0.f;
#pragma unroll
    for (int b = 0; b < DB; ++b) o_acc[b][i] = 0.f;
  }
  const float sc = p.scale * 1.44269504088896340736f;

  int step = 0;
  for (int tile = tile0 + wave; tile < n_tiles; tile += NW, ++step) {
    const int j = tile * BK;
    const bool more = tile + NW < n_tiles;
    pr_wait_vm<KVL>();  // K and L rows have landed
    pr_fence();
    pf_f32x16 s;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uint4 a4 = *reinterpret_cast<const uint4*>(tile_lds + (k_pre ^ ((2 * ks + g2) << 4)));
      if constexpr (KF16)
        s = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(pf_f16x8, a4), __builtin_bit_cast(pf_f16x8, qb[ks]), s, 0, 0, 0);
      else
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(pf_as_bf16x8(a4), qb[ks], s, 0, 0, 0);
    }
    if constexpr (HAS_BK) {
#pragma unroll
      for (int ks = 0; ks < RKS; ++ks) {
        const uint2 lo = *reinterpret_cast<const uint2*>(tile_lds + l_rd[ks][0]);
        const uint2 hi = *reinterpret_cast<const uint2*>(tile_lds + l_rd[ks][1]);
        const pf_bf16x8 a = pf_as_bf16x8(make_uint4(lo.x, lo.y, hi.x, hi.y));
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qtb[ks], s, 0, 0, 0);
      }
    }
    pr_reads_done();
    if (more) issue_k(j + NW * BK, step + 1);

    pf_bf16x8 pb[2];
    {
      if (j + BK - 1 > first_limit) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (j + 8 * (i >> 2) + 4 * g2 + (i & 3) > limit) s[i] = -INFINITY;
      }
      float mx = s[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
      mx = fmaxf(mx, pf_partner32(mx)) * sc;
      if (OWN || __builtin_amdgcn_ballot_w64(mx > m_run + kSlack) != 0) {
        if (OWN) m_top = fmaxf(m_top, mx);
        const float m_new = OWN ? fmaxf(mx, m_top - kReach) : fmaxf(m_run, mx);
        const float alpha = m_new == -INFINITY ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);  // (a row that has seen nothing yet)
        m_run = m_new;
        l_run *= alpha;
#pragma unroll
        for (int b = 0; b < DB; ++b) o_acc[b] *= alpha;
        lr_acc *= alpha;
      }
      const float nm = m_run == -INFINITY ? 0.f : -m_run;
#pragma unroll
      for (int h2 = 0; h2 < 2; ++h2) {
        float e[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          e[i] = __builtin_amdgcn_exp2f(fmaf(s[8 * h2 + i], sc, nm));
          if (!ONES_ROW) l_run += e[i];
        }
        pb[h2] = pf_as_bf16x8(make_uint4(pf_pack2(e[0], e[1]), pf_pack2(e[2], e[3]), pf_pack2(e[4], e[5]), pf_pack2(e[6], e[7])));
      }
    }
    // O^T += V^T P^T ; Olr^T += L^T P^T
    if (more) pr_wait_vm<KVL>();
    else pf_wait_vm0();
    pr_fence();
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2) {
#pragma unroll
      for (int b = 0; b < DB; ++b) {
        const unsigned char* src = tile_lds + (v_pre ^ (b << 6)) + 16 * h2 * (D * 2);
        const pf_bf16x8 a = pf_join(pf_read_tr16(src), pf_read_tr16(src + 8 * (D * 2)));
        o_acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[h2], o_acc[b], 0, 0, 0);
      }
      const unsigned char* src0 = tile_lds + lt_rd[0] + 16 * h2 * (RP * 2);
      const unsigned char* src1 = tile_lds + lt_rd[1] + 16 * h2 * (RP * 2);
      if (ONES_ROW) {
        src0 = ones_lane ? smem + ONES_AT : src0;
        src1 = ones_lane ? smem + ONES_AT : src1;
      }
      const pf_bf16x8 a = pf_join(pf_read_tr16(src0), pf_read_tr16(src1));
      lr_acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[h2], lr_acc, 0, 0, 0);
    }
    pr_reads_done();
    if (more) issue_lv(j + NW * BK, step + 1);
  }

  // ---------------- the eight states become one ----------------
  pf_wait_vm0();  // (a wave without a tile may have asked for rows of B_V)
  if (ONES_ROW) {
    const float mine = lr_acc[8], other = pf_partner32(mine);
    l_run = g2 == 0 ? mine : other;
  } else {
    l_run += pf_partner32(l_run);
  }
  const int n_active = min(NW, n_tiles - tile0);  // waves that have seen keys
  auto quad = [](const pf_f32x16& v, int q) __attribute__((always_inline)) { return pf_f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]}; };
  auto slot_of = [&](int w) __attribute__((always_inline)) { return smem + (w < 2 * DB ? w * SLOT_SHORT : 2 * DB * SLOT_SHORT + (w - 2 * DB) * SLOT); };
  // half block b of wave w's state, columns 16b .. 16b + 15: registers 4q..4q+3 of a lane, q = 2 (b & 1) + i, are columns
  // 16b + 8i + 4 g2 .. + 3 of row l32 (sixteen lanes of a write or read cover 256 bytes)
  auto o_at = [&](int w, int b, int i) __attribute__((always_inline)) {
    return reinterpret_cast<pf_f32x4*>(slot_of(w) + (b - (w < 2 * DB && b > w)) * HALF + l32 * 64 + (((2 * i + g2) ^ ((l32 >> 2) & 3)) << 4));
  };
  auto lr_at = [&](int w, int q) __attribute__((always_inline)) {
    return reinterpret_cast<pf_f32x4*>(slot_of(w) + (w < 2 * DB ? 2 * DB - 1 : 2 * DB) * HALF + l32 * (RP * 4) + (((2 * q + g2) ^ (RP == 16 ? (l32 >> 2) & 3 : (l32 >> 1) & 7)) << 4));
  };
  auto ml_at = [&](int w) __attribute__((always_inline)) {
    return reinterpret_cast<pf_f32x2*>(slot_of(w) + (w < 2 * DB ? 2 * DB - 1 : 2 * DB) * HALF + LR_BYTES + l32 * 8);
  };
  __syncthreads();  // every wave is done with its tiles
  if (wave < n_active) {
#pragma unroll
    for (int b = 0; b < 2 * DB; ++b)
      if (b != wave) {
#pragma unroll
        for (int i = 0; i < 2; ++i) *o_at(wave, b, i) = quad(o_acc[b >> 1], 2 * (b & 1) + i);
      }
#pragma unroll
    for (int q = 0; q < RP / 8; ++q) *lr_at(wave, q) = quad(lr_acc, q);
    if (g2 == 0) *ml_at(wave) = pf_f32x2{m_run, l_run};
  }
  __syncthreads();
  // Wave w finishes columns 16w .. 16w + 15.  Olr is summed by the last waves, a part each, and handed round behind another
  // barrier; at up to 16 ranks with all keys every wave sums it for itself (that is shorter than the barrier).  All reads leave
  // before the first is used.  The time is that of the bytes through LDS, whose rows have to be spread over all banks.  (With four
  // waves, each with a whole block and all of Olr, and lanes of the same bank: 1.65 us of a call's 9.7 here.  Now rank 24, 106 tokens
  // on 1106 keys 12.7 -> 12.4 us, 24 on 6905 in shares 15.5 -> 14.7; rank 16, 45 on 478 keys 9.47 -> 9.40, 10 on 506 paged 9.64 -> 9.45.)
  const bool finishes = wave < 2 * DB;
  constexpr bool EACH_LR = RP == 16 && !SHARED;
  constexpr int LQ = EACH_LR ? RP / 8 : 1;  // parts of Olr, 8 ranks each, that a wave sums, from lr_q on
  const int lr_q = EACH_LR ? 0 : NW - 1 - wave;
  const bool sums_lr = EACH_LR ? finishes && has_bv : lr_q < RP / 8 && (SHARED || has_bv);
  float m_all = -INFINITY, l_all = 0.f;
  pf_f32x2 ml[NW];
  pf_f32x4 v_o[NW][2], v_lr[NW][LQ];
#pragma unroll
  for (int w = 0; w < NW; ++w) ml[w] = *ml_at(w);
  if (finishes) {
#pragma unroll
    for (int w = 0; w < NW; ++w)
#pragma unroll
      for (int i = 0; i < 2; ++i) v_o[w][i] = *o_at(w, wave, i);  // (its own, and those beyond n_active, are not used)
  }
  if (sums_lr) {
#pragma unroll
    for (int w = 0; w < NW; ++w)
#pragma unroll
      for (int q = 0; q < LQ; ++q) v_lr[w][q] = *lr_at(w, lr_q + q);
  }
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    if (w >= n_active) ml[w] = pf_f32x2{-INFINITY, 0.f};
    m_all = fmaxf(m_all, ml[w][0]);
  }
  pf_f32x4 o[2], lr[LQ];
#pragma unroll
  for (int q = 0; q < LQ; ++q) lr[q] = pf_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    o[i] = pf_f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int b = 0; b < 2 * DB; ++b)
      if (b == wave) o[i] = quad(o_acc[b >> 1], 2 * (b & 1) + i);
  }
  {
    const float own = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m_all);
    o[0] *= own;
    o[1] *= own;
  }
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    if (w >= n_active) break;
    const float wgt = ml[w][0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[w][0] - m_all);
    l_all = fmaf(wgt, ml[w][1], l_all);
    if (finishes && w != wave) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[i][e] = fmaf(wgt, v_o[w][i][e], o[i][e]);
    }
    if (sums_lr) {
#pragma unroll
      for (int q = 0; q < LQ; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) lr[q][e] = fmaf(wgt, v_lr[w][q][e], lr[q][e]);
    }
  }
  const bool live = l32 < live_rows;
  const int col = 16 * wave + 4 * g2;
  if constexpr (SHARED) {
    // the share's state for the merge kernel: m in natural-log units, l, O and Olr as fp32 rows
    if (!live) return;
    if (finishes) {
#pragma unroll
      for (int i = 0; i < 2; ++i) *reinterpret_cast<pf_f32x4*>(p.part_o + slot * D + col + 8 * i) = o[i];
    }
    if (sums_lr && 8 * lr_q < r) *reinterpret_cast<pf_f32x4*>(p.part_lr + slot * r + 8 * lr_q + 4 * g2) = lr[0];
    if (wave == 0 && g2 == 0) {
      *reinterpret_cast<pf_f32x2*>(p.part_ml + slot * 2) = pf_f32x2{m_all * 0.69314718055994530942f, l_all};
      if (share == 0) p.part_adapter[out_row] = a_idx;
    }
    return;
  }
  if (has_bv) {
    auto sum_at = [&](int q) __attribute__((always_inline)) { return reinterpret_cast<pf_f32x4*>(smem + LR_SUM_AT + q * 1024 + lane * 16); };
    if constexpr (!EACH_LR) {
      if (sums_lr) *sum_at(lr_q) = lr[0];
      __syncthreads();
    }
    if (!finishes) return;
    // O^T += B_V^T Olr^T, Olr as two bf16 terms (see prefill_mfma_kernel); the product is that of the 32 columns that the half
    // block lies in
    pf_f32x16 acc;
    const bool upper = (wave & 1) != 0;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      acc[i] = upper ? 0.f : o[i >> 2][i & 3];
      acc[8 + i] = upper ? o[i >> 2][i & 3] : 0.f;
    }
#pragma unroll
    for (int ks = 0; ks < RKS; ++ks) {
      pf_f32x4 x[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        if constexpr (EACH_LR) x[i] = lr[2 * ks + i];
        else x[i] = *sum_at(2 * ks + i);
      }
      uint32_t w2[2][4];
#pragma unroll
      for (int e2 = 0; e2 < 4; ++e2) {
        const float x0 = x[e2 >> 1][2 * (e2 & 1)], x1 = x[e2 >> 1][2 * (e2 & 1) + 1];
        w2[0][e2] = pf_pack2(x0, x1);
        const float r0 = x0 - __uint_as_float(w2[0][e2] << 16), r1 = x1 - __uint_as_float(w2[0][e2] & 0xffff0000u);
        w2[1][e2] = pf_pack2(__builtin_isfinite(r0) ? r0 : 0.f, __builtin_isfinite(r1) ? r1 : 0.f);
      }
      const unsigned char* src = smem + B_AT - KV_BYTES + (v_pre ^ ((wave >> 1) << 6)) + 16 * ks * (D * 2);
      const pf_bf16x8 a = pf_join(pf_read_tr16(src), pf_read_tr16(src + 8 * (D * 2)));
#pragma unroll
      for (int term = 1; term >= 0; --term)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pf_as_bf16x8(make_uint4(w2[term][0], w2[term][1], w2[term][2], w2[term][3])), acc, 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) o[i >> 2][i & 3] = upper ? acc[8 + i] : acc[i];
  } else if (!finishes) {
    return;
  }
  if (!live) return;
  const float inv = 1.0f / l_all;
  bf16_t* dst = static_cast<bf16_t*>(p.out) + out_row * D + col;
#pragma unroll
  for (int i = 0; i < 2; ++i)
    *reinterpret_cast<uint2*>(dst + 8 * i) = make_uint2(pf_pack2(o[i][0] * inv, o[i][1] * inv), pf_pack2(o[i][2] * inv, o[i][3] * inv));
}

template <int D, int RP, bool PAGED, int MODE>
static hipError_t launch_rows3(const Params& p, dim3 grid, hipStream_t s) {
  if (p.keys_f16) {  // (rotary calls of the split-KV path's sizes do not come here)
    if constexpr (MODE == kPrOwn) return hipErrorInvalidValue;
    else hipLaunchKernelGGL((prefill_rows_kernel<D, RP, PAGED, kPrKeysF16, MODE>), grid, dim3(512), 0, s, p);
  } else if (p.b_k != nullptr) {
    hipLaunchKernelGGL((prefill_rows_kernel<D, RP, PAGED, kPrQt, MODE>), grid, dim3(512), 0, s, p);
  } else {
    hipLaunchKernelGGL((prefill_rows_kernel<D, RP, PAGED, kPrValueOnly, MODE>), grid, dim3(512), 0, s, p);
  }
  return hipGetLastError();
}

template <int D, int RP, int MODE>
static hipError_t launch_rows2(const Params& p, dim3 grid, hipStream_t s) {
  return p.block_size != 0 ? launch_rows3<D, RP, true, MODE>(p, grid, s) : launch_rows3<D, RP, false, MODE>(p, grid, s);
}

template <int D, int RP>
static hipError_t launch_rows1(const Params& p, bool own_references, dim3 grid, hipStream_t s) {
  if (p.n_splits > 1) return launch_rows2<D, RP, kPrShared>(p, grid, s);
  return own_references ? launch_rows2<D, RP, kPrOwn>(p, grid, s) : launch_rows2<D, RP, kPrWhole>(p, grid, s);
}

// p.n_splits workgroups divide the keys of 32 rows (1: none of the partial-state fields is used)
hipError_t launch_prefill_rows(const Params& p, bool own_references, hipStream_t s) {
  // (a wave's block ids lie in one register: 32 tiles per wave, 256 per share)
  if ((p.max_seq_len + 31) / 32 > 256 * p.n_splits && p.block_size != 0) return hipErrorInvalidValue;
  if (p.n_splits < 1 || p.n_splits > 64 || p.rank > 32 || (p.block_size != 0 && !prefill_pool_fits(p))) return hipErrorInvalidValue;
  const dim3 grid((p.n_new * p.tile_group + 31) / 32 * p.n_kv_heads * p.n_splits);
  if (p.head_dim == 128) return p.rank <= 16 ? launch_rows1<128, 16>(p, own_references, grid, s) : launch_rows1<128, 32>(p, own_references, grid, s);
  return p.rank <= 16 ? launch_rows1<64, 16>(p, own_references, grid, s) : launch_rows1<64, 32>(p, own_references, grid, s);
}

}  // namespace lra
