// Cache-append producer of the Flash-LoRA-Attention library (bf16, gfx950): the step before
// the attention path.  For the new tokens of one sequence it forms
//     [K' | V | L] = X . [W_K | W_V | A]          (LRAgent Sec. 3.2: base cache from the
//                                                  pretrained projections, LR cache from the
//                                                  shared LoRA down-projection)
// rotates the keys by the model's rotary position embedding (the cached keys are the rotated
// ones, App. D.1) and writes the rows into K_base, V_base and L, contiguous or paged.
//
// Five kernels, chosen by the number of new tokens (launch_append at the end of the file): a
// matrix-vector kernel (1 token), a weight-streaming MFMA kernel (up to 64), and three tiled
// GEMM kernels (128 features x 128 or 64 tokens per workgroup; 256 x 256 for large chunks,
// see wide_tiles_pay; 64 x 64 where those fill the chip once, see append_quarter_tiles).
//
// The tiled GEMM takes the weights one output feature per row (the usual layout of a linear
// layer) and computes transposed, Y^T[feature][token] = W[feature][:] . X[token][:], so
// that both operands are rows of 16-byte chunks along d_model (ds_read_b128, no transposed
// reads) and every lane ends up with four consecutive features of one token: an 8-byte
// store into a cache row.  A workgroup walks d_model in steps of 64; the W and X tiles go
// from HBM straight into a ring of 2 to 4 LDS stages (buffer_load ... lds, swizzled by
// choosing which chunk a lane fetches).  The four waves form a 2 x 2 grid; a wave's two
// 32-feature blocks are chosen d/2 apart, so the two halves of every rotary pair sit in the
// same lane and register of its two accumulators and the rotation needs no data movement.
// The rotation rate of every pair is tabulated once per workgroup in double precision
// (revolutions per position); angle = fractional part of position * rate, so positions in
// the tens of thousands lose nothing.
#include "lra_prefill_util.h"

namespace lra {

// Length of the sequence the new rows are appended to.  max_seq_len is exact for this call: it
// sizes the caches, so a device-side length beyond it cannot be honoured - such a call writes
// nothing (every row index comes out negative and is skipped) rather than overwrite live rows.
__device__ __forceinline__ int append_length(int len, int max_seq_len) { return len <= max_seq_len ? len : 0; }


// BT = 64 halves the token side of the tile (a wave then owns 64 features x 32 tokens): twice the
// workgroups and three quarters of the bytes per step for chunks too small to fill the chip.
// SPLITK: a workgroup takes one of p.k_splits equal parts of d_model and leaves its fp32 sums in the
// workspace, [part][token][feature] (feature = row of w); append_finish_kernel adds the parts,
// rotates, casts and stores.  For chunks whose output tiles would occupy a fraction of the chip
// and walk all of d_model one step after the other.
template <int D, bool PAGED, int NS, int BT = 128, bool SPLITK = false>
__global__ __launch_bounds__(NS == 2 ? 256 : 512, NS == 2 ? 2 : 1) void append_kernel(AppendParams p) {
  constexpr int BF = 128, BK = 64;  // features, d_model step (BT tokens)
  constexpr bool ONE_TB = BT == 64;  // one 32-token block per wave
  constexpr int REQ = ONE_TB ? 6 : 8;  // requests per step and wave
  constexpr int TILE_BYTES = BF * BK * 2;      // the W tile: 128 rows of 128 bytes
  constexpr int STAGE = TILE_BYTES + BT * BK * 2;  // [W tile][X tile]
  constexpr int HALF = D / 2;

  __shared__ __align__(16) unsigned char smem[NS * STAGE];
  __shared__ double rope_rate[D / 2];  // revolutions per position of every rotary pair

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  // waves 4-7 (deeper rings only) request the tiles and do nothing else
  const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool requester = NS != 2 && wave8 >= 4;
  const int wave = wave8 & 3;
  const int l32 = lane & 31, g2 = lane >> 5;
  const int wr = wave >> 1, wc = wave & 1;  // position in the 2 x 2 grid of waves: features, tokens
  const int HD = p.n_kv_heads * D;
  const int n_ct_kv = (HD + BF - 1) / BF;   // feature tiles of the K (and of the V) region
  // Workgroup -> (part of d_model, feature tile, token tile).  Workgroups go to the 8 XCDs in turn.  Each takes a
  // stretch of the L tiles (little matrix work, first) and a stretch of the list of K and V tiles with the smaller
  // operand's index running fastest: the tiles an XCD works on at a time share rows of the larger operand in its L2
  // instead of every XCD reading all of it.  (With the L tiles part of one list an XCD had them all, and the others one
  // more K or V tile than compute units just above a round: 272 tiles 52.5 against 49.3 us.)
  // Where two workgroups share a unit (NS == 2) and the token tiles are a multiple of the XCDs, the plain order
  // (token tiles fastest) also gives an XCD the same token tiles all along; up to two rounds, and if the tokens
  // outnumber the features, it was faster: 4096 new tokens on 4 kv heads 43.7 against 47 us, 5000 on 8 103 against 110
  // (32768 on 2, 1280 tiles: 95 against 86; 8300 on 2, 65 token tiles: 34 against 29).
  const int n_tt = (p.n_new + BT - 1) / BT, n_ft = 2 * n_ct_kv, n_parts = SPLITK ? p.k_splits : 1;
  const int n_l = n_tt * n_parts, n_kv = n_l * n_ft;
  const bool in_order = NS == 2 && p.n_new > HD && n_l + n_kv <= 1024 && (n_tt & (n_l + n_kv <= 512 ? 3 : 7)) == 0;
  bool is_l;
  int item;
  if (in_order) {
    is_l = static_cast<int>(blockIdx.x) < n_l;
    item = is_l ? static_cast<int>(blockIdx.x) : static_cast<int>(blockIdx.x) - n_l;
  } else {
    const int xcd = static_cast<int>(blockIdx.x) & 7, nth = static_cast<int>(blockIdx.x) >> 3;  // this XCD's nth tile
    const int per_xcd = (n_l + n_kv + 7) >> 3;
    const int l_here = (n_l >> 3) + (xcd < (n_l & 7) ? 1 : 0), l_before = xcd * (n_l >> 3) + min(xcd, n_l & 7);
    if (nth >= per_xcd) return;
    is_l = nth < l_here;
    item = is_l ? l_before + nth : xcd * per_xcd - l_before + (nth - l_here);
  }
  if (!is_l && item >= n_kv) return;
  const int per_part = is_l ? n_tt : n_tt * n_ft;
  const int part_z = SPLITK ? item / per_part : 0;
  const int tile = item - part_z * per_part;
  const bool tokens_fast = is_l || in_order || p.n_new <= 2 * HD;
  const int tile_hi = tile / (tokens_fast ? n_tt : n_ft), tile_lo = tile - tile_hi * (tokens_fast ? n_tt : n_ft);
  const int ct = is_l ? -1 : (tokens_fast ? tile_hi : tile_lo), tt = tokens_fast ? tile_lo : tile_hi;
  const int kind = ct < 0 ? 2 : (ct < n_ct_kv ? 0 : 1);  // 0 K, 1 V, 2 L
  const int ct_in = kind == 0 ? ct : (kind == 1 ? ct - n_ct_kv : 0);
  const int feat0 = ct_in * BF;                                 // first feature of the tile inside its region
  const int w_row0 = (kind == 0 ? 0 : (kind == 1 ? HD : 2 * HD)) + feat0;  // its row of w
  const int tok0 = tt * BT;
  const int n_new = p.n_new;
  const int n_t = append_length(PF_CONST_I32(p.seq_lens)[p.seq_index], p.max_seq_len);
  const int pos0 = n_t - n_new;  // cache row (= position) of new token 0

  // ---------------- tile traffic ----------------
  // A wave-wide load moves 8 rows of 128 bytes.  Load i fills rows 8i ..; lane l lands at row
  // 8i + l/8, physical chunk l%8, and fetches logical chunk (l%8) ^ ((row >> 1) & 7).  Wave w
  // issues loads i = w, w+4, w+8, w+12 of either tile: the swizzle of its rows does not
  // depend on the load, so one offset per lane serves all of them.  Rows past the end of w
  // (the L tile holds fewer than 128 features) or of x read as zero.
  const uint32_t ldw2 = static_cast<uint32_t>(p.d_model) * 2u;
  const uint32_t n_w_rows = static_cast<uint32_t>(2 * HD + p.rank);
  const pf_u32x4 rs_w = pf_rsrc(p.w, (n_w_rows - 1) * ldw2 + ldw2);
  const pf_u32x4 rs_x = pf_rsrc(p.x, static_cast<uint32_t>(n_new - 1) * ldw2 + ldw2);
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(PF_LDS_AS(unsigned char, smem)));
  const uint32_t voff = static_cast<uint32_t>(lane >> 3) * ldw2 +
                        (((lane & 7) ^ ((4 * wave + (lane >> 4)) & 7)) << 4);
  // request number part (0..7) of this wave for the step at k0: W and X alternate
  auto issue_part = [&](int k0, int st, int part) __attribute__((always_inline)) {
    const int i = wave + 4 * (part >> 1);
    const uint32_t dst = lds0 + st * STAGE + i * 1024;
    if ((part & 1) == 0) pf_load16_to_lds(rs_w, dst, voff, static_cast<uint32_t>(w_row0 + 8 * i) * ldw2 + k0 * 2);
    else if (8 * i < BT) pf_load16_to_lds(rs_x, dst + TILE_BYTES, voff, static_cast<uint32_t>(tok0 + 8 * i) * ldw2 + k0 * 2);
  };
  auto issue_step = [&](int k0, int st) __attribute__((always_inline)) {
#pragma unroll
    for (int part = 0; part < 8; ++part) issue_part(k0, st, part);
  };
  const int n_steps = SPLITK ? p.d_model / BK / p.k_splits : p.d_model / BK;
  const int k_first = SPLITK ? part_z * n_steps * BK : 0;  // first d_model index of this part
  if (NS == 2 || requester) {
#pragma unroll
    for (int st = 0; st < NS - 1; ++st)
      if (st < n_steps) issue_step(k_first + st * BK, st);
  }
  if constexpr (!SPLITK)  // (the finishing kernel rotates)
    if (tid < D / 2 && p.rope_theta > 0.f) rope_rate[tid] = rope_rate_rev(tid, D, p.rope_theta);  // read after the loop's barriers

  // ---------------- operands ----------------
  // A operand: W rows (features), B operand: X rows (tokens); lane (row l32 of a 32-row block,
  // k = 16ks + 8g2 + e): the 16-byte chunk 2ks + g2 of its row, at chunk ^ ((row >> 1) & 7).
  const int pre = l32 * (BK * 2) + (((l32 >> 1) & 7) << 4);
  // the wave's two feature blocks are half a head apart: rotary pairs meet in one lane
  // The L tile holds at most 64 features (blocks 0 and 1): there every wave takes both and
  // one token block, half the matrix work of a K or V tile.
  const bool lr_tile = kind == 2;
  const int fb0 = lr_tile ? 0 : (D == 128 ? wr : 2 * wr);
  const int fb1 = lr_tile ? 1 : (D == 128 ? wr + 2 : 2 * wr + 1);
  // (BT = 64: one token block per wave, wc or, in the L tile, wave % 2 with waves 2 and 3 repeating 0 and 1)
  const int tb0 = ONE_TB ? (lr_tile ? (wave & 1) : wc) : (lr_tile ? wave : 2 * wc);
  const int tb1 = 2 * wc + 1;  // unused by the L tile and with BT = 64
  const bool stores = !(ONE_TB && lr_tile && wave >= 2);

  pf_f32x16 acc[2][2];  // [feature block fb0 / fb1][token block tb0 / tb1]
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[a][b][i] = 0.f;

  // Step s computes on stage s % NS while the tiles of the next NS - 2 steps are in flight and
  // the one after them is requested: a wave waits until only the loads younger than step s
  // (8 per step and wave) are outstanding, the barrier makes every wave's share visible and
  // retires stage (s - 1) % NS, which the new requests then overwrite.
  // A wave issues in order and a wave-wide request holds it for as long as the memory pipe of
  // the compute unit needs to take it: the requests of a step and its products add up in a wave that
  // issues both.  Two workgroups per compute unit (NS == 2) cover each other; with one (the deeper
  // rings) four waves of their own issue the requests, and the other four only read and multiply:
  // 0.36 -> 0.29 us per step at 64 tokens, 0.54 -> 0.38 at 128.
  if (requester) {
    for (int step = 0; step < n_steps; ++step) {
      if (step + NS - 2 < n_steps) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(REQ * (NS - 2)));
      else pf_wait_vm0();
      __syncthreads();
      if (step + NS - 1 < n_steps) issue_step(k_first + (step + NS - 1) * BK, (step + NS - 1) % NS);
    }
    return;
  }
  auto k_step = [&](int step, auto st_c, auto lr_c) __attribute__((always_inline)) {
    constexpr int ST = decltype(st_c)::value;
    constexpr bool LR = decltype(lr_c)::value;
    constexpr int KS = BK / 16;
    if (NS == 2) pf_wait_vm0();
    __syncthreads();
    const unsigned char* wt = smem + ST * STAGE;
    const unsigned char* xt = wt + TILE_BYTES;
    if (NS == 2 && step + 1 < n_steps) issue_step(k_first + (step + 1) * BK, ST ^ 1);
    // the sixteen operand reads of the step ordered against its sixteen MFMAs: two k-slices of reads, one read per
    // MFMA from then on
    pf_bf16x8 a0[KS], a1[KS], b0[KS], b1[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int off = pre ^ ((2 * ks + g2) << 4);
      a0[ks] = pf_as_bf16x8(*reinterpret_cast<const uint4*>(wt + off + fb0 * 32 * (BK * 2)));
      b0[ks] = pf_as_bf16x8(*reinterpret_cast<const uint4*>(xt + off + tb0 * 32 * (BK * 2)));
      a1[ks] = pf_as_bf16x8(*reinterpret_cast<const uint4*>(wt + off + fb1 * 32 * (BK * 2)));
      if (!LR) b1[ks] = pf_as_bf16x8(*reinterpret_cast<const uint4*>(xt + off + tb1 * 32 * (BK * 2)));
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      acc[0][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[ks], b0[ks], acc[0][0], 0, 0, 0);
      acc[1][0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[ks], b0[ks], acc[1][0], 0, 0, 0);
      if (!LR) {
        acc[0][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[ks], b1[ks], acc[0][1], 0, 0, 0);
        acc[1][1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[ks], b1[ks], acc[1][1], 0, 0, 0);
      }
    }
    constexpr int READS = LR ? 12 : 16, MFMAS = LR ? 8 : 16, AHEAD = READS / 2;
    __builtin_amdgcn_sched_group_barrier(0x100, AHEAD, 0);
#pragma unroll
    for (int i = 0; i < READS - AHEAD; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, MFMAS - (READS - AHEAD), 0);
  };
  auto k_loop = [&](auto lr_c) __attribute__((always_inline)) {
    for (int step = 0; step < n_steps; step += NS) {
      k_step(step, std::integral_constant<int, 0>{}, lr_c);
      if (step + 1 < n_steps) k_step(step + 1, std::integral_constant<int, 1>{}, lr_c);
      if (NS > 2 && step + 2 < n_steps) k_step(step + 2, std::integral_constant<int, 2 % NS>{}, lr_c);
      if (NS > 3 && step + 3 < n_steps) k_step(step + 3, std::integral_constant<int, 3 % NS>{}, lr_c);
    }
  };
  if (lr_tile || ONE_TB) k_loop(std::true_type{});  // one token block per wave
  else k_loop(std::false_type{});

  // ---------------- epilogue: rotate the keys, cast, store into the cache rows ----------------
  // acc[a][b], register i, lane (l32, g2): feature 32*fb_a + 8(i/4) + 4g2 + i%4 of the tile,
  // token 32*tb_b + l32 of the tile.
  if constexpr (SPLITK) {
    // the sums of this part of d_model as they are, four consecutive features per 16-byte store
    const int n_feat = 2 * HD + p.rank;
    const int region = kind == 2 ? p.rank : HD;   // features of this tile's region
    float* part = p.split_ws + static_cast<int64_t>(part_z) * p.n_new * n_feat;
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      if ((b == 1 && (lr_tile || ONE_TB)) || !stores) continue;
      const int tok = tok0 + 32 * (b == 0 ? tb0 : tb1) + l32;
      if (tok >= n_new) continue;
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int f = feat0 + 32 * (a == 0 ? fb0 : fb1) + 8 * q + 4 * g2;  // inside the region: all four or none
          if (f < region)
            *reinterpret_cast<float4*>(part + static_cast<int64_t>(tok) * n_feat + (w_row0 - feat0) + f) =
                make_float4(acc[a][b][4 * q + 0], acc[a][b][4 * q + 1], acc[a][b][4 * q + 2], acc[a][b][4 * q + 3]);
        }
    }
    return;
  }
  bf16_t* kcache = static_cast<bf16_t*>(kind == 0 ? p.k_base : p.v_base);
#pragma unroll
  for (int b = 0; b < 2; ++b) {
    if ((b == 1 && (lr_tile || ONE_TB)) || !stores) continue;
    const int tok = tok0 + 32 * (b == 0 ? tb0 : tb1) + l32;
    const int j = pos0 + tok;  // cache row of this token, and its position
    if (tok >= n_new || j < 0) continue;  // (a sequence length below n_new breaks the contract: nothing is written)
    int64_t row_off;           // element offset of (token j, kv head 0) in K_base / V_base, or of row j in L
    if (PAGED) {
      const int blk = p.block_table[static_cast<int64_t>(p.seq_index) * p.max_blocks_per_seq + (j >> 4)];
      row_off = kind == 2 ? (static_cast<int64_t>(blk) * 16 + (j & 15)) * p.l_row_stride
                          : static_cast<int64_t>(blk) * p.kv_block_stride + static_cast<int64_t>(j & 15) * p.kv_token_stride;
    } else {
      row_off = kind == 2 ? static_cast<int64_t>(j) * p.l_row_stride : static_cast<int64_t>(j) * p.kv_token_stride;
    }
    if (kind == 2) {
      bf16_t* lrow = static_cast<bf16_t*>(p.l) + row_off;
#pragma unroll
      for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int f = 32 * (a == 0 ? fb0 : fb1) + 8 * q + 4 * g2;  // the rank is a multiple of 8: all four or none
          if (f < p.rank)
            *reinterpret_cast<uint2*>(lrow + f) =
                make_uint2(pf_pack2(acc[a][b][4 * q + 0], acc[a][b][4 * q + 1]), pf_pack2(acc[a][b][4 * q + 2], acc[a][b][4 * q + 3]));
        }
      continue;
    }
    if (kind == 0 && p.rope_theta > 0.f) {
      // pair (feature dd, dd + d/2) of a head: acc[0] holds the first half, acc[1] the second
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int dd = (32 * fb0 + 8 * (i >> 2) + 4 * g2 + (i & 3)) % D;  // < d/2 by construction
        float sn, cs;
        rope_sincos(rope_rate[dd], j, sn, cs);
        const float lo = acc[0][b][i], hi = acc[1][b][i];
        acc[0][b][i] = lo * cs - hi * sn;
        acc[1][b][i] = hi * cs + lo * sn;
      }
    }
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int f = feat0 + 32 * (a == 0 ? fb0 : fb1) + 8 * q + 4 * g2;  // feature inside the K (V) region
        if (f < HD) {
          const int head = f / D, dd = f - head * D;
          *reinterpret_cast<uint2*>(kcache + row_off + static_cast<int64_t>(head) * p.kv_head_stride + dd) =
              make_uint2(pf_pack2(acc[a][b][4 * q + 0], acc[a][b][4 * q + 1]), pf_pack2(acc[a][b][4 * q + 2], acc[a][b][4 * q + 3]));
        }
      }
  }
  (void)HALF;
}

// ---------------------------------------------------------------------------------------
// 64 features x 64 tokens per workgroup, for chunks whose tiles of that size fill the chip about once.  What bounds such
// a chunk is what one compute unit pulls from L2, 80 to 95 GB/s: tiles of 128 x 64 occupy half of the units and move 24 KB
// per 64-wide step, these all of them and 16 KB.  Llama-3-8B projection, 509 new tokens: 19.5 -> 16.3 us, of which 0.35 us
// per step of 128.
//
// A tile holds both halves of its rotary pairs: 32 features of a head and the 32 half a head on (d = 64: the head).  Steps
// of 128 along d_model, a ring of four stages; waves 4-7 request, waves 0-3 multiply: wave w takes all 64 features of the
// 32-token block w % 2 and the k half w / 2 of every step.  The two halves are added through LDS at the end, each
// wave finishing half of the features.
//
// The L features have no tiles of their own (they would be a second round of the chip): blocks of 16 features x 16 tokens
// ride on the first feature tiles of the token tile, one per tile: an eighth more bytes there and two small products a step.
// ---------------------------------------------------------------------------------------
template <int D, bool PAGED>
__global__ __launch_bounds__(512, 2) void append_quarter_kernel(AppendParams p) {
  constexpr int BF = 64, BT = 64, BK = 128, NS = 4, KS = BK / 32;  // KS: 16-wide k slices of a wave's half step
  constexpr int ROW = BK * 2, TILE_BYTES = 64 * ROW, LT_BYTES = 16 * ROW;
  constexpr int STAGE = 2 * TILE_BYTES + LT_BYTES;  // [W tile][X tile][W rows of L]
  constexpr int PAIR = D / 2;                       // distance of the tile's two feature blocks
  __shared__ __align__(16) unsigned char smem[NS * STAGE];
  __shared__ double rope_rate[D / 2];  // revolutions per position of every rotary pair

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave8 = __builtin_amdgcn_readfirstlane(tid >> 6);
  const bool requester = wave8 >= 4;
  const int wave = wave8 & 3;
  const int l32 = lane & 31, g2 = lane >> 5;
  const int HD = p.n_kv_heads * D;
  // An XCD takes a stretch of the feature tiles with all their token tiles: its rows of w and all of x.  With more tokens than
  // features the other way round, so that what every XCD reads stays in its L2 of 4 MB (4 kv heads of 64 on a width of 1792, 1720
  // tokens, x of 6.2 MB: 11.1 -> 8.3 us; 2 of 128 on 3584, 1577 tokens 17.3 -> 14.7; level where both fit).
  const int n_tt = (p.n_new + BT - 1) / BT, n_region = HD / BF, n_ft = 2 * n_region, n_items = n_ft * n_tt;
  const int item = (static_cast<int>(blockIdx.x) & 7) * ((n_items + 7) >> 3) + (static_cast<int>(blockIdx.x) >> 3);
  if ((static_cast<int>(blockIdx.x) >> 3) >= ((n_items + 7) >> 3) || item >= n_items) return;
  const bool by_tokens = p.n_new > 2 * HD;
  const int major = item / (by_tokens ? n_ft : n_tt), minor = item - major * (by_tokens ? n_ft : n_tt);
  const int ct = by_tokens ? minor : major, tt = by_tokens ? major : minor;
  const int kind = ct < n_region ? 0 : 1;  // 0 K, 1 V
  const int ct_in = ct - kind * n_region;
  // first feature of the tile inside its region; rows 32..63 of the tile lie PAIR features on
  const int feat0 = D == 128 ? (ct_in >> 1) * 128 + (ct_in & 1) * 32 : ct_in * 64;
  const int w_row0 = kind * HD + feat0, tok0 = tt * BT, n_new = p.n_new;
  const bool rides = ct < 4 * ((p.rank + 15) >> 4);  // carries L features 16 (ct / 4) .. + 15 of the 16 tokens ct % 4
  const int l_feat0 = (ct >> 2) * 16, l_tok0 = (ct & 3) * 16;
  const int n_t = append_length(PF_CONST_I32(p.seq_lens)[p.seq_index], p.max_seq_len);

  // tile traffic: a wave-wide load moves 4 rows of 256 bytes, lane l to row l / 16, physical chunk l % 16 of logical
  // chunk (l % 16) ^ (row % 16); wave w loads rows 16 q + 4 w .. + 3 of every tile
  const uint32_t ldw2 = static_cast<uint32_t>(p.d_model) * 2u;
  const uint32_t n_w_rows = static_cast<uint32_t>(2 * HD + p.rank);
  const pf_u32x4 rs_w = pf_rsrc(p.w, n_w_rows * ldw2);
  const pf_u32x4 rs_x = pf_rsrc(p.x, static_cast<uint32_t>(n_new) * ldw2);
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(PF_LDS_AS(unsigned char, smem)));
  const int lrow = 4 * wave + (lane >> 4);
  const uint32_t voff = static_cast<uint32_t>(lrow) * ldw2 + (((lane & 15) ^ lrow) << 4);
  auto issue_step = [&](int step) __attribute__((always_inline)) {
    const uint32_t dst = lds0 + (step & (NS - 1)) * STAGE + wave * 1024, k2 = static_cast<uint32_t>(step) * ROW;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      pf_load16_to_lds(rs_w, dst + q * 4096, voff, static_cast<uint32_t>(w_row0 + 16 * (q & 1) + (q >> 1) * PAIR) * ldw2 + k2);
      pf_load16_to_lds(rs_x, dst + TILE_BYTES + q * 4096, voff, static_cast<uint32_t>(tok0 + 16 * q) * ldw2 + k2);
    }
    if (rides) pf_load16_to_lds(rs_w, dst + 2 * TILE_BYTES, voff, static_cast<uint32_t>(2 * HD + l_feat0) * ldw2 + k2);
  };
  const int n_steps = p.d_model / BK;
  if (requester) {
#pragma unroll
    for (int st = 0; st < NS - 1; ++st)
      if (st < n_steps) issue_step(st);
    for (int step = 0; step < n_steps; ++step) {
      if (step + NS - 2 >= n_steps) pf_wait_vm0();
      else if (rides) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(9 * (NS - 2)));
      else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(8 * (NS - 2)));
      __syncthreads();
      if (step + NS - 1 < n_steps) issue_step(step + NS - 1);
    }
    __syncthreads();
    __syncthreads();
    return;
  }
  if (tid < D / 2 && p.rope_theta > 0.f) rope_rate[tid] = rope_rate_rev(tid, D, p.rope_theta);  // read after the loop's barriers

  const int tb = wave & 1, kh = wave >> 1;
  const int tok = tok0 + 32 * tb + l32, j = n_t - n_new + tok;  // the lane's token, its cache row and position
  const bool live = tok < n_new && j >= 0;  // (a sequence length below n_new breaks the contract: nothing is written)
  int blk = 0;
  if (PAGED && live) blk = p.block_table[static_cast<int64_t>(p.seq_index) * p.max_blocks_per_seq + (j >> 4)];

  // operands: row l32 of a 32-row block, k = 16 slice + 8 g2 + e: logical chunk 8 kh + 2 slice + g2
  const int pre = l32 * ROW + (((l32 & 15) ^ (8 * kh + g2)) << 4);
  const int pre16 = (lane & 15) * ROW + (((lane & 15) ^ (8 * kh + (lane >> 4))) << 4);  // (16 x 16 x 32: k = 8 (lane / 16) + e)
  const bool l_wave = rides && (l_tok0 >> 5) == tb;
  pf_f32x16 acc[2];
  pf_f32x4 acc_l = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[0][i] = acc[1][i] = 0.f;
  // (Reading a step's operands under the products of the step before changed nothing: 16.3 and 16.2 us at 509 tokens.)
  for (int step = 0; step < n_steps; ++step) {
    __syncthreads();
    const unsigned char* wt = smem + (step & (NS - 1)) * STAGE;
    const unsigned char* xt = wt + TILE_BYTES + tb * 32 * ROW;
    pf_bf16x8 a0[KS], a1[KS], b[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int off = pre ^ (ks << 5);
      b[ks] = pf_as_bf16x8(*reinterpret_cast<const uint4*>(xt + off));
      a0[ks] = pf_as_bf16x8(*reinterpret_cast<const uint4*>(wt + off));
      a1[ks] = pf_as_bf16x8(*reinterpret_cast<const uint4*>(wt + off + 32 * ROW));
    }
    if (l_wave) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        const int off = pre16 ^ (kb << 6);
        const pf_bf16x8 la = pf_as_bf16x8(*reinterpret_cast<const uint4*>(wt + 2 * TILE_BYTES + off));
        const pf_bf16x8 lb = pf_as_bf16x8(*reinterpret_cast<const uint4*>(xt + (l_tok0 & 31) * ROW + off));
        acc_l = __builtin_amdgcn_mfma_f32_16x16x32_bf16(la, lb, acc_l, 0, 0, 0);
      }
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a0[ks], b[ks], acc[0], 0, 0, 0);
      acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a1[ks], b[ks], acc[1], 0, 0, 0);
    }
  }

  // ---------------- the k halves meet: a wave hands over the eight registers of either block the other one finishes --------
  __syncthreads();  // everybody is done with the stages
  float* box = reinterpret_cast<float*>(smem);
  constexpr int PART = 16 * 64;  // floats of one wave's half
  {
    float* mine = box + wave * PART + lane;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      mine[i * 64] = kh == 0 ? acc[0][8 + i] : acc[0][i];
      mine[(8 + i) * 64] = kh == 0 ? acc[1][8 + i] : acc[1][i];
    }
    if (l_wave && kh == 1)
#pragma unroll
      for (int i = 0; i < 4; ++i) box[4 * PART + i * 64 + lane] = acc_l[i];
  }
  __syncthreads();
  float v[2][8];
  {
    const float* other = box + (wave ^ 2) * PART + lane;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      v[0][i] = (kh == 0 ? acc[0][i] : acc[0][8 + i]) + other[i * 64];
      v[1][i] = (kh == 0 ? acc[1][i] : acc[1][8 + i]) + other[(8 + i) * 64];
    }
  }
  if (l_wave && kh == 0) {
    // register i of a lane: L feature l_feat0 + 4 (lane / 16) + i of token l_tok0 + lane % 16
    const int lt = tok0 + l_tok0 + (lane & 15), lj = n_t - n_new + lt, f = l_feat0 + 4 * (lane >> 4);
    if (lt < n_new && lj >= 0 && f < p.rank) {  // (the rank is a multiple of 8: all four or none)
      float x[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = acc_l[i] + box[4 * PART + i * 64 + lane];
      int64_t row = lj;
      if (PAGED) row = static_cast<int64_t>(p.block_table[static_cast<int64_t>(p.seq_index) * p.max_blocks_per_seq + (lj >> 4)]) * 16 + (lj & 15);
      *reinterpret_cast<uint2*>(static_cast<bf16_t*>(p.l) + row * p.l_row_stride + f) = make_uint2(pf_pack2(x[0], x[1]), pf_pack2(x[2], x[3]));
    }
  }
  if (!live) return;
  // v[a][i]: feature 32 a + 16 kh + 8 (i / 4) + 4 g2 + i % 4 of the tile, token 32 tb + l32
  const int head = feat0 / D, dd0 = feat0 - head * D + 16 * kh + 4 * g2;
  if (kind == 0 && p.rope_theta > 0.f) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      float sn, cs;
      rope_sincos(rope_rate[dd0 + 8 * (i >> 2) + (i & 3)], j, sn, cs);
      const float lo = v[0][i], hi = v[1][i];
      v[0][i] = lo * cs - hi * sn;
      v[1][i] = hi * cs + lo * sn;
    }
  }
  const int64_t row_off = PAGED ? static_cast<int64_t>(blk) * p.kv_block_stride + static_cast<int64_t>(j & 15) * p.kv_token_stride
                                : static_cast<int64_t>(j) * p.kv_token_stride;
  bf16_t* dst = static_cast<bf16_t*>(kind == 0 ? p.k_base : p.v_base) + row_off + static_cast<int64_t>(head) * p.kv_head_stride + dd0;
#pragma unroll
  for (int a = 0; a < 2; ++a)
#pragma unroll
    for (int q = 0; q < 2; ++q)
      *reinterpret_cast<uint2*>(dst + a * PAIR + 8 * q) =
          make_uint2(pf_pack2(v[a][4 * q + 0], v[a][4 * q + 1]), pf_pack2(v[a][4 * q + 2], v[a][4 * q + 3]));
}

// ---------------------------------------------------------------------------------------
// 256 features x 256 tokens per workgroup of eight waves (for chunks it is faster on, see
// wide_tiles_pay).  At 128 x 128 a step moves 32 KB into LDS for 2.1 MFLOP and every MFMA costs one 1 KB LDS read: with
// two workgroups per compute unit the LDS is busier than the matrix pipes.  Here a wave owns 128
// features x 64 tokens (eight 32 x 32 accumulators), reads six operands for eight MFMAs, and a step
// moves 64 KB for 8.4 MFLOP; the two waves of a SIMD cover each other's reads and requests.  (Four
// waves of 128 x 128 left a SIMD one wave, which had to interleave its requests with its products by
// hand and had no registers left for the L features.)  Same LDS layout, DMA and epilogue as
// append_kernel; two stages, one workgroup per compute unit.  The wave's four feature blocks are one
// head (d = 128: pairs (0,2), (1,3)) or two (d = 64: pairs (0,1), (2,3)).
//
// The L features (at most 64) have no tiles of their own: as a column of tiles they cost a call a
// place on every compute unit they touched (8192 tokens are 256 K/V tiles, one round of the chip,
// and became two).  The feature tiles of a token tile share its eight 32-token blocks among them
// (tile f takes blocks f and f + F: two at most with the host's F >= 4) and stage the L rows of w
// beside their own; waves 0-3 take one k-slice of a step each for the first block, waves 4-7 for the
// second, one or two MFMAs beside thirty-two.  The four slices are added through LDS at the end.
//
// Workgroup -> tile: an XCD takes every eighth token tile and all feature tiles of it, one after
// the other, so that the 32 tiles it works on at a time are 4 token tiles x 8 feature tiles.
// Llama-3-8B projection, us with the L tiles in the grid and four waves, and as it is: 6000 new
// tokens 130 and 101, 8192 185 and 120, 16384 301 and 239 (1.16 PFLOP/s).
// ---------------------------------------------------------------------------------------
template <int D, bool PAGED, int NLB>  // NLB: 32-row blocks the L features take (1: ranks up to 32, 2)
__global__ __launch_bounds__(512, 2) void append_wide_kernel(AppendParams p) {
  constexpr int BF = 256, BT = 256, BK = 64;
  constexpr int TILE_BYTES = BF * BK * 2;  // 256 rows of 128 bytes
  constexpr int LT_BYTES = NLB * 32 * BK * 2;
  constexpr int STAGE = 2 * TILE_BYTES + LT_BYTES;  // [W tile][X tile][W rows of L]
  __shared__ __align__(16) unsigned char smem[2 * STAGE];
  __shared__ double rope_rate[D / 2];  // revolutions per position of every rotary pair

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, g2 = lane >> 5;
  const int wr = wave >> 2, wc = wave & 3;  // position in the 2 x 4 grid of waves: features, tokens
  const int HD = p.n_kv_heads * D;
  const int n_ct_kv = (HD + BF - 1) / BF;
  const int n_ct = 2 * n_ct_kv;            // feature tiles F
  const int idx = static_cast<int>(blockIdx.x) >> 3;
  const int tt = (idx / n_ct) * 8 + (static_cast<int>(blockIdx.x) & 7), ct = idx % n_ct;
  const int tok0 = tt * BT;
  const int n_new = p.n_new;
  if (tok0 >= n_new) return;
  const int kind = ct < n_ct_kv ? 0 : 1;  // 0 K, 1 V
  const int feat0 = (kind == 0 ? ct : ct - n_ct_kv) * BF;
  const int w_row0 = (kind == 0 ? 0 : HD) + feat0;
  const int lb_mine = ct + (wave >> 2) * n_ct;   // token block whose L features this wave works on, below 8
  const bool l_any = ct < 8, l_wave = lb_mine < 8;
  const int n_t = append_length(PF_CONST_I32(p.seq_lens)[p.seq_index], p.max_seq_len);
  const int pos0 = n_t - n_new;

  // tile traffic: as in append_kernel, 32 wave-wide loads per tile, wave w issues i = w + 8q
  const uint32_t ldw2 = static_cast<uint32_t>(p.d_model) * 2u;
  const uint32_t n_w_rows = static_cast<uint32_t>(2 * HD + p.rank);
  const pf_u32x4 rs_w = pf_rsrc(p.w, (n_w_rows - 1) * ldw2 + ldw2);
  const pf_u32x4 rs_x = pf_rsrc(p.x, static_cast<uint32_t>(n_new - 1) * ldw2 + ldw2);
  const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(PF_LDS_AS(unsigned char, smem)));
  const uint32_t voff = static_cast<uint32_t>(lane >> 3) * ldw2 +
                        (((lane & 7) ^ ((4 * wave + (lane >> 4)) & 7)) << 4);
  // request number part (0..3) of this wave for the step at k0: a W and an X load; the L rows (past the end of w
  // they read as zero) go with the first
  auto issue_part = [&](int k0, int st, int part) __attribute__((always_inline)) {
    const int i = wave + 8 * part;
    const uint32_t dst = lds0 + st * STAGE + i * 1024;
    pf_load16_to_lds(rs_w, dst, voff, static_cast<uint32_t>(w_row0 + 8 * i) * ldw2 + k0 * 2);
    pf_load16_to_lds(rs_x, dst + TILE_BYTES, voff, static_cast<uint32_t>(tok0 + 8 * i) * ldw2 + k0 * 2);
    if (part == 0 && l_any && wave < 4 * NLB)
      pf_load16_to_lds(rs_w, dst + 2 * TILE_BYTES, voff, static_cast<uint32_t>(2 * HD + 8 * i) * ldw2 + k0 * 2);
  };
  const int n_steps = p.d_model / BK;
#pragma unroll
  for (int part = 0; part < 4; ++part) issue_part(0, 0, part);
  if (tid < D / 2 && p.rope_theta > 0.f) rope_rate[tid] = rope_rate_rev(tid, D, p.rope_theta);  // read after the loop's barriers

  const int pre = l32 * (BK * 2) + (((l32 >> 1) & 7) << 4);
  // feature blocks 4 wr + i (i < 4), token blocks 2 wc + j (j < 2)
  const int fbase = 4 * wr, tbase = 2 * wc;
  pf_f32x16 acc[4][2];      // [feature block][token block]
  pf_f32x16 acc_l[NLB];     // [32 L features], token block lb_mine, k-slice wave % 4 of every step
#pragma unroll
  for (int i = 0; i < 16; ++i) {
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 2; ++b) acc[a][b][i] = 0.f;
#pragma unroll
    for (int a = 0; a < NLB; ++a) acc_l[a][i] = 0.f;
  }

  // One step: the tiles have landed, everybody is done with the other stage; the requests of the next step go out
  // beside the products of the first two k-slices, the operands of a k-slice are read under the products of the one
  // before.
  auto k_step = [&](int step, auto st_c, bool more) __attribute__((always_inline)) {
    constexpr int ST = decltype(st_c)::value;
    constexpr int KS = BK / 16;
    pf_wait_vm0();
    __syncthreads();
    const unsigned char* wt = smem + ST * STAGE + fbase * 32 * (BK * 2);
    const unsigned char* xt = smem + ST * STAGE + TILE_BYTES + tbase * 32 * (BK * 2);
    pf_bf16x8 a[2][4], b[2][2];
    auto read_slice = [&](int ks, int buf) __attribute__((always_inline)) {
      const int off = pre ^ ((2 * ks + g2) << 4);
#pragma unroll
      for (int j = 0; j < 2; ++j) b[buf][j] = pf_as_bf16x8(*reinterpret_cast<const uint4*>(xt + off + j * 32 * (BK * 2)));
#pragma unroll
      for (int i = 0; i < 4; ++i) a[buf][i] = pf_as_bf16x8(*reinterpret_cast<const uint4*>(wt + off + i * 32 * (BK * 2)));
    };
    read_slice(0, 0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const int cur = ks & 1;
      __builtin_amdgcn_sched_barrier(0);
      if (more && ks < 2) {
        issue_part((step + 1) * BK, ST ^ 1, 2 * ks);
        issue_part((step + 1) * BK, ST ^ 1, 2 * ks + 1);
      }
      if (ks + 1 < KS) read_slice(ks + 1, cur ^ 1);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[cur][i], b[cur][j], acc[i][j], 0, 0, 0);
    }
    if (l_wave) {  // (uniform)
      const int off = pre ^ ((2 * wc + g2) << 4);
      const pf_bf16x8 bl = pf_as_bf16x8(*reinterpret_cast<const uint4*>(smem + ST * STAGE + TILE_BYTES + lb_mine * 32 * (BK * 2) + off));
#pragma unroll
      for (int i = 0; i < NLB; ++i) {
        const pf_bf16x8 al = pf_as_bf16x8(*reinterpret_cast<const uint4*>(smem + ST * STAGE + 2 * TILE_BYTES + i * 32 * (BK * 2) + off));
        acc_l[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al, bl, acc_l[i], 0, 0, 0);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  for (int step = 0; step < n_steps; step += 2) {
    k_step(step, std::integral_constant<int, 0>{}, step + 1 < n_steps);
    if (step + 1 < n_steps) k_step(step + 1, std::integral_constant<int, 1>{}, step + 2 < n_steps);
  }

  auto cache_row = [&](int j, bool l_row) __attribute__((always_inline)) -> int64_t {  // element offset of (token j, kv head 0), or of row j of L
    if (PAGED) {
      const int blk = p.block_table[static_cast<int64_t>(p.seq_index) * p.max_blocks_per_seq + (j >> 4)];
      return l_row ? (static_cast<int64_t>(blk) * 16 + (j & 15)) * p.l_row_stride
                   : static_cast<int64_t>(blk) * p.kv_block_stride + static_cast<int64_t>(j & 15) * p.kv_token_stride;
    }
    return l_row ? static_cast<int64_t>(j) * p.l_row_stride : static_cast<int64_t>(j) * p.kv_token_stride;
  };
  // epilogue of L: the slices meet in LDS, [wave][feature block][register][lane]; a wave then stores registers
  // 4 wc .. 4 wc + 3 of its token block, features 8 wc + 4 g2 + 0..3
  if (l_any) {
    float* red = reinterpret_cast<float*>(smem);
    static_assert(8 * NLB * 16 * 64 * 4 <= 2 * STAGE, "the slices fit the stages");
    __syncthreads();  // everybody is done with the tiles
    if (l_wave) {
#pragma unroll
      for (int i = 0; i < NLB; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) red[((wave * NLB + i) * 16 + e) * 64 + lane] = acc_l[i][e];
    }
    __syncthreads();
    const int tok = tok0 + 32 * lb_mine + l32, row = pos0 + tok;
    if (l_wave && tok < n_new && row >= 0) {  // (a sequence length below n_new breaks the contract: nothing is written)
      bf16_t* lrow = static_cast<bf16_t*>(p.l) + cache_row(row, true);
#pragma unroll
      for (int i = 0; i < NLB; ++i) {
        float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; ++w)
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] += red[((((wave & 4) + w) * NLB + i) * 16 + 4 * wc + e) * 64 + lane];
        const int f = 32 * i + 8 * wc + 4 * g2;  // the rank is a multiple of 8: all four or none
        if (f < p.rank) *reinterpret_cast<uint2*>(lrow + f) = make_uint2(pf_pack2(v[0], v[1]), pf_pack2(v[2], v[3]));
      }
    }
  }

  // epilogue of K and V.  acc[a][b], register i, lane (l32, g2): feature 32 (fbase + a) + 8 (i/4) + 4 g2 + i%4
  // of the tile, token 32 (tbase + b) + l32 of the tile.
  bf16_t* kcache = static_cast<bf16_t*>(kind == 0 ? p.k_base : p.v_base);
  auto store_block = [&](auto b_c) __attribute__((always_inline)) {
    constexpr int b = decltype(b_c)::value;
    const int tok = tok0 + 32 * (tbase + b) + l32;
    const int j = pos0 + tok;
    if (tok >= n_new || j < 0) return;
    const int64_t row_off = cache_row(j, false);
    if (kind == 0 && p.rope_theta > 0.f) {
      // rotates the pair of blocks (lo, hi); block_lo = position of lo among the wave's four
      auto rotate = [&](pf_f32x16& lo_v, pf_f32x16& hi_v, int block_lo) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const int dd = (32 * block_lo + 8 * (i >> 2) + 4 * g2 + (i & 3)) % D;  // < d/2 by construction
          float sn, cs;
          rope_sincos(rope_rate[dd], j, sn, cs);
          const float lo = lo_v[i], hi = hi_v[i];
          lo_v[i] = lo * cs - hi * sn;
          hi_v[i] = hi * cs + lo * sn;
        }
      };
      if (D == 128) {
        rotate(acc[0][b], acc[2][b], 0);
        rotate(acc[1][b], acc[3][b], 1);
      } else {
        rotate(acc[0][b], acc[1][b], 0);
        rotate(acc[2][b], acc[3][b], 2);
      }
    }
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int f = feat0 + 32 * (fbase + a) + 8 * q + 4 * g2;
        if (f < HD) {
          const int head = f / D, dd = f - head * D;
          *reinterpret_cast<uint2*>(kcache + row_off + static_cast<int64_t>(head) * p.kv_head_stride + dd) =
              make_uint2(pf_pack2(acc[a][b][4 * q + 0], acc[a][b][4 * q + 1]), pf_pack2(acc[a][b][4 * q + 2], acc[a][b][4 * q + 3]));
        }
      }
  };
  store_block(std::integral_constant<int, 0>{});
  store_block(std::integral_constant<int, 1>{});
}

// ---------------------------------------------------------------------------------------
// Few new tokens: one pass over the weights with every compute unit on it.  A workgroup owns PP rotary pairs of features
// (of K, then of V, numbered through) and, the first `rank` workgroups, one L feature; its 8 waves take every eighth 64-wide piece
// of d_model.  Each copies its pieces of the rows and of the tokens into a ring of its own in LDS, eight rows of 128 bytes
// per request, and reads the MFMA operands from there: no barrier before the partial tiles meet.
// What bounds it: up to 16 tokens HBM and the latency of one round (llama-3-8B projection, 17 MB: 6.0 us, 2.8 TB/s), beyond
// that x, which every workgroup reads through its compute unit's one path to L2 (0.1 us per token at d_model 4096).  Operands
// straight from global memory, sixteen features per workgroup, as it was before: sixteen rows per request of 16 lanes pass that
// path at a quarter of its width, and half of the units had no workgroup.  us before and now at 3, 16 and 32 tokens:
// 8.5 / 10.4 / 14.2 and 6.0 / 7.3 / 9.0; 4 kv heads on 3584 8.6 / 9.6 / 12.2 and 4.4 / 4.6 / 5.9; 32 kv heads
// 19.0 / 25.5 / 35.0 and 14.1 / 18.5 / 26.0; 4 of 64 on 256, where all of it is latency, 8 tokens 2.7 and 2.85.
// Up to five requests of eight rows per piece (up to 32 tokens with three pairs, 24 with more) the ring takes half of a unit's LDS or
// less (two workgroups, and the next call's can begin: with all of it 3 tokens 6.4).  Above, a wave keeps two pieces, 96 to 160 KB:
// one workgroup per unit.
// ---------------------------------------------------------------------------------------
template <int D, int WI, int XI, bool PAGED>  // requests of eight rows per piece: weights (2 PP + 1 <= 8 WI), tokens
__global__ __launch_bounds__(512, 2) void append_skinny_kernel(AppendParams p, int pp) {
  constexpr int NW = 8, NT = (XI + 1) / 2, INS = WI + XI, DEPTH = INS <= 5 ? 10 / INS : 2;
  constexpr int SLOT = INS * 1024, RING = DEPTH * SLOT;
  static_assert(RING >= NT * 1024, "a wave's partial tiles fit into its ring");
  __shared__ __align__(16) unsigned char smem[NW * RING];

  // (the parameter block in one round trip, the sequence length first and by hand: only the last step needs it)
  asm volatile("" ::"s"(p.w), "s"(p.x), "s"(p.seq_lens), "s"(p.k_base), "s"(p.v_base), "s"(p.l));
  asm volatile("" ::"s"(p.d_model), "s"(p.n_kv_heads), "s"(p.rank), "s"(p.n_new), "s"(p.seq_index), "s"(p.max_seq_len),
               "s"(p.rope_theta), "s"(p.kv_token_stride), "s"(p.kv_head_stride), "s"(p.l_row_stride));
  int len_raw;
  asm volatile("s_load_dword %0, %1, 0x0" : "=s"(len_raw) : "s"(p.seq_lens + p.seq_index));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, g4 = lane >> 4;
  const int HD = p.n_kv_heads * D, n_new = p.n_new, bx = blockIdx.x;
  const int tok0 = blockIdx.y * (8 * XI);
  // first feature of pair P (its partner lies D / 2 on), counted through K and V
  auto feature = [&](int pair) __attribute__((always_inline)) { return pair / (D / 2) * D + pair % (D / 2); };

  const uint32_t ld2 = static_cast<uint32_t>(p.d_model) * 2u;
  const pf_u32x4 rs_w = pf_rsrc(p.w, static_cast<uint32_t>(2 * HD + p.rank) * ld2);
  const pf_u32x4 rs_x = pf_rsrc(p.x, static_cast<uint32_t>(n_new) * ld2);
  const uint32_t ring = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(PF_LDS_AS(unsigned char, smem))) + wave * RING;
  // A piece's row is 128 bytes, 16-byte chunk c of row R at place c ^ (R / 2) % 8: sixteen lanes that read one chunk of
  // sixteen rows then meet every bank once.
  const int dma_row = lane >> 3;
  uint32_t w_off[WI], x_off[XI];
#pragma unroll
  for (int i = 0; i < WI; ++i) {
    const int R = 8 * i + dma_row;  // rows: first features, partners, the L feature; rows behind them are fetched again
    const int pair = min(bx * pp + (R < pp ? R : (R < 2 * pp ? R - pp : 0)), HD - 1);
    int row = feature(pair) + (R >= pp && R < 2 * pp ? D / 2 : 0);
    if (R == 2 * pp && bx < p.rank) row = 2 * HD + bx;
    w_off[i] = static_cast<uint32_t>(row) * ld2 + (((lane & 7) ^ ((R >> 1) & 7)) << 4);
  }
#pragma unroll
  for (int i = 0; i < XI; ++i) {
    const int R = 8 * i + dma_row;
    x_off[i] = static_cast<uint32_t>(min(tok0 + R, n_new - 1)) * ld2 + (((lane & 7) ^ ((R >> 1) & 7)) << 4);
  }
  // (The workgroups of an XCD, which run together, start on different pieces, so that x comes from different channels of its L2:
  // 4 kv heads on 3584, 64 tokens 8.7 -> 8.4 us.  With fewer than eight pieces the first waves go without, to work out the rates.)
  const int n_pieces = p.d_model / 64;
  const int first = n_pieces >= NW ? (wave + (bx >> 3)) & (NW - 1) : NW - 1 - wave, n = (n_pieces - first + NW - 1) / NW;
  auto request = [&](int i, int slot) __attribute__((always_inline)) {
    const uint32_t k2 = static_cast<uint32_t>(first + NW * i) * 128u, dst = ring + slot * SLOT;
#pragma unroll
    for (int q = 0; q < WI; ++q) pf_load16_to_lds(rs_w, dst + q * 1024, w_off[q], k2);
#pragma unroll
    for (int q = 0; q < XI; ++q) pf_load16_to_lds(rs_x, dst + (WI + q) * 1024, x_off[q], k2);
  };
#pragma unroll
  for (int i = 0; i < DEPTH; ++i)
    if (i < n) request(i, i);

  // thread (pair q or, behind the pairs, the L feature; token): its rotation rate, worked out under the requests
  const int item = tid >> 4, q = item / NT, t_sum = item % NT, tk = l16;
  const int pair = bx * pp + q;
  double rate = 0.0;
  if (q < pp && pair < HD / 2 && p.rope_theta > 0.f) {
    rate = rope_rate_rev(pair % (D / 2), D, p.rope_theta);
    asm volatile("" ::"v"(rate));
  }
  asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(len_raw));

  pf_f32x4 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = pf_f32x4{0.f, 0.f, 0.f, 0.f};
  // operand rows: weights, tokens (16 t on); of eight rows the upper lanes take the same again, for products nobody reads
  auto chunk = [&](int row) __attribute__((always_inline)) { return row * 128 + ((g4 ^ ((row >> 1) & 7)) << 4); };
  const int a_off = chunk(WI == 1 ? l16 & 7 : l16);
  int b_off[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) b_off[t] = WI * 1024 + t * 2048 + chunk(2 * t + 2 > XI ? l16 & 7 : l16);
  int slot = 0;
  for (int i = 0; i < n; ++i) {
    // piece i is there: at most the pieces behind it are under way
    const int behind = min(DEPTH, n - i) - 1;
    static_assert(DEPTH >= 2 && DEPTH <= 10, "the waits below");
#define LRA_WAIT(B) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(DEPTH > B ? B * INS : 0) : "memory")
    if (behind >= 9) LRA_WAIT(9);
    else if (behind == 8) LRA_WAIT(8);
    else if (behind == 7) LRA_WAIT(7);
    else if (behind == 6) LRA_WAIT(6);
    else if (behind == 5) LRA_WAIT(5);
    else if (behind == 4) LRA_WAIT(4);
    else if (behind == 3) LRA_WAIT(3);
    else if (behind == 2) LRA_WAIT(2);
    else if (behind == 1) LRA_WAIT(1);
    else LRA_WAIT(0);
#undef LRA_WAIT
    const unsigned char* st = smem + wave * RING + slot * SLOT;
    pf_bf16x8 a[2], b[NT][2];
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      a[m] = pf_as_bf16x8(*reinterpret_cast<const uint4*>(st + (a_off ^ (m << 6))));
#pragma unroll
      for (int t = 0; t < NT; ++t) b[t][m] = pf_as_bf16x8(*reinterpret_cast<const uint4*>(st + (b_off[t] ^ (m << 6))));
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // (read, before the slot is filled again)
    if (i + DEPTH < n) request(i + DEPTH, slot);
    slot = slot + 1 == DEPTH ? 0 : slot + 1;
#pragma unroll
    for (int m = 0; m < 2; ++m)
#pragma unroll
      for (int t = 0; t < NT; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[m], b[t][m], acc[t], 0, 0, 0);
  }
  // acc[t], register e, lane (l16, g4): row 4 g4 + e, token 16 t + l16; every wave's partial tiles to the start of its ring
#pragma unroll
  for (int t = 0; t < NT; ++t) *reinterpret_cast<pf_f32x4*>(smem + wave * RING + (t * 256 + lane * 4) * 4) = acc[t];
  __syncthreads();

  const bool is_l = q == pp;
  if (q > pp || (is_l ? bx >= p.rank : pair >= HD)) return;
  const int tok = tok0 + 16 * t_sum + tk, j = append_length(len_raw, p.max_seq_len) - n_new + tok;
  if (16 * t_sum + tk >= 8 * XI || tok >= n_new || j < 0) return;
  const int r_lo = is_l ? 2 * pp : q, r_hi = is_l ? 2 * pp : pp + q;  // tile row -> lane tk + 16 (row / 4), register row % 4
  const float* from = reinterpret_cast<const float*>(smem) + t_sum * 256 + 4 * tk;
  float lo = 0.f, hi = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    lo += from[w * (RING / 4) + 64 * (r_lo >> 2) + (r_lo & 3)];
    hi += from[w * (RING / 4) + 64 * (r_hi >> 2) + (r_hi & 3)];
  }
  int64_t blk = 0;
  if (PAGED) blk = p.block_table[static_cast<int64_t>(p.seq_index) * p.max_blocks_per_seq + (j >> 4)];
  if (is_l) {
    const int64_t row = PAGED ? blk * 16 + (j & 15) : j;
    static_cast<bf16_t*>(p.l)[row * p.l_row_stride + bx] = f32_to_bf16(lo);
    return;
  }
  const bool is_k = pair < HD / 2;
  if (is_k && p.rope_theta > 0.f) {
    float sn, cs;
    rope_sincos(rate, j, sn, cs);
    const float x = lo, y = hi;
    lo = x * cs - y * sn;
    hi = y * cs + x * sn;
  }
  const int f = feature(is_k ? pair : pair - HD / 2), head = f / D;
  const int64_t row_off = PAGED ? blk * p.kv_block_stride + static_cast<int64_t>(j & 15) * p.kv_token_stride : static_cast<int64_t>(j) * p.kv_token_stride;
  bf16_t* dst = static_cast<bf16_t*>(is_k ? p.k_base : p.v_base) + row_off + static_cast<int64_t>(head) * p.kv_head_stride + (f - head * D);
  dst[0] = f32_to_bf16(lo);
  dst[D / 2] = f32_to_bf16(hi);
}

// ---------------------------------------------------------------------------------------
// One new token (every decode step appends one): a matrix-vector product.  One wave
// per weight row reads it in fully coalesced 1 KB pieces, all in flight at once, and forms
// the dot products with v_dot2c_f32_bf16; the 2 * Hkv * d + r rows make several hundred
// workgroups, enough outstanding loads to run at HBM speed.  A workgroup's four rows are two
// rotary pairs (features f, f+1 and f + d/2, f+1 + d/2).
// ---------------------------------------------------------------------------------------
typedef __bf16 ap_bf16x2 __attribute__((ext_vector_type(2)));

template <int D, bool PAGED>
__global__ __launch_bounds__(256) void append_gemv_kernel(AppendParams p) {
  __shared__ float red[4];
  // A call of this kernel is one round of requests and a handful of dependent latencies; each is
  // kept off the others' path: the parameter block comes in one round trip, the sequence length
  // (needed only by the last step) is requested first and by hand, the weight requests (the bytes
  // that take long) leave before the activations and unconditionally (pieces beyond the row are
  // fetched from its last piece and multiplied by zero: a load under a condition makes the
  // compiler wait for earlier loads on the spot), and the rotation rate of the pair (double
  // precision exp2 and log2) is worked out while the requests are in flight.
  asm volatile("" ::"s"(p.w), "s"(p.x), "s"(p.seq_lens), "s"(p.k_base), "s"(p.v_base), "s"(p.l));
  asm volatile("" ::"s"(p.d_model), "s"(p.n_kv_heads), "s"(p.rank), "s"(p.seq_index), "s"(p.max_seq_len),
               "s"(p.rope_theta), "s"(p.kv_token_stride), "s"(p.kv_head_stride), "s"(p.l_row_stride));
  int len_raw;
  asm volatile("s_load_dword %0, %1, 0x0" : "=s"(len_raw) : "s"(p.seq_lens + p.seq_index));
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int HD = p.n_kv_heads * D;
  const int groups_kv = HD / 4;
  const int fg = blockIdx.x;
  const int kind = fg < groups_kv ? 0 : (fg < 2 * groups_kv ? 1 : 2);
  const int fg_in = kind == 0 ? fg : (kind == 1 ? fg - groups_kv : fg - 2 * groups_kv);
  const int head = fg_in / (D / 4), sub = fg_in - head * (D / 4);  // K, V: pairs 2 sub, 2 sub + 1 of this head
  const int pr = wave & 1, half = wave >> 1;
  // row of this wave: K/V  head*D + 2 sub + pr (+ d/2 for the second half);  L  4 fg_in + pr + 2 half
  const int feat = kind == 2 ? 4 * fg_in + pr + 2 * half : head * D + 2 * sub + pr + half * (D / 2);
  const int w_row = kind == 2 ? 2 * HD + min(feat, p.rank - 1) : (kind == 1 ? HD : 0) + feat;
  const int64_t ld = p.d_model;
  const uint4* wp = reinterpret_cast<const uint4*>(static_cast<const bf16_t*>(p.w) + static_cast<int64_t>(w_row) * ld);
  const uint4* xp = static_cast<const uint4*>(p.x);

  float acc = 0.f;
  const int n_chunks = p.d_model / 8;  // 16-byte pieces of a row; lane l takes l, l + 64, ...
  constexpr int U = 8;
  double rate = 0.0;  // revolutions per position of this thread's rotary pair (threads of the last step)
  for (int c0 = lane; c0 < n_chunks; c0 += 64 * U) {
    uint4 wv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      // (non-temporal: a weight row is read once per call, by this wave)
      const pf_u32x4 t4 = __builtin_nontemporal_load(reinterpret_cast<const pf_u32x4*>(wp + min(c0 + 64 * u, n_chunks - 1)));
      wv[u] = make_uint4(t4[0], t4[1], t4[2], t4[3]);
    }
    // all weight requests out before anything else.  (The operands stay HIP's uint4 structs on purpose:
    // with native 4-vectors this compiler selected element 0 for all four dot products.)
    __builtin_amdgcn_sched_barrier(0);
    uint4 xv[U];
#pragma unroll
    for (int u = 0; u < U; ++u) xv[u] = xp[min(c0 + 64 * u, n_chunks - 1)];
    __builtin_amdgcn_sched_barrier(0);
    if (c0 == lane && tid < 2 && kind == 0 && p.rope_theta > 0.f) {
      rate = rope_rate_rev(2 * sub + (tid & 1), D, p.rope_theta);
      asm volatile("" ::"v"(rate));  // (here, under the requests, not after the reduction)
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      uint4 x4 = xv[u];
      if (c0 + 64 * u >= n_chunks) x4 = make_uint4(0u, 0u, 0u, 0u);  // (a piece beyond the row)
      acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(ap_bf16x2, wv[u].x), __builtin_bit_cast(ap_bf16x2, x4.x), acc, false);
      acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(ap_bf16x2, wv[u].y), __builtin_bit_cast(ap_bf16x2, x4.y), acc, false);
      acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(ap_bf16x2, wv[u].z), __builtin_bit_cast(ap_bf16x2, x4.z), acc, false);
      acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(ap_bf16x2, wv[u].w), __builtin_bit_cast(ap_bf16x2, x4.w), acc, false);
    }
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
  if (lane == 0) red[wave] = acc;
  __syncthreads();

  // thread = pair: both halves of a rotary pair (K), two independent features (V, L)
  if (tid >= 2) return;
  const int q = tid;
  asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(len_raw));
  const int j = append_length(len_raw, p.max_seq_len) - 1;
  if (j < 0) return;
  float lo = red[q], hi = red[2 + q];
  if (kind == 2) {
    int64_t row_off;
    if (PAGED) {
      const int blk = p.block_table[static_cast<int64_t>(p.seq_index) * p.max_blocks_per_seq + (j >> 4)];
      row_off = (static_cast<int64_t>(blk) * 16 + (j & 15)) * p.l_row_stride;
    } else {
      row_off = static_cast<int64_t>(j) * p.l_row_stride;
    }
    bf16_t* lrow = static_cast<bf16_t*>(p.l) + row_off;
    const int f = 4 * fg_in + q;
    if (f < p.rank) lrow[f] = f32_to_bf16(lo);
    if (f + 2 < p.rank) lrow[f + 2] = f32_to_bf16(hi);
    return;
  }
  const int dd = 2 * sub + q;  // < d/2
  if (kind == 0 && p.rope_theta > 0.f) {
    float sn, cs;
    rope_sincos(rate, j, sn, cs);
    const float a = lo, b = hi;
    lo = a * cs - b * sn;
    hi = b * cs + a * sn;
  }
  int64_t row_off;
  if (PAGED) {
    const int blk = p.block_table[static_cast<int64_t>(p.seq_index) * p.max_blocks_per_seq + (j >> 4)];
    row_off = static_cast<int64_t>(blk) * p.kv_block_stride + static_cast<int64_t>(j & 15) * p.kv_token_stride;
  } else {
    row_off = static_cast<int64_t>(j) * p.kv_token_stride;
  }
  bf16_t* dst = static_cast<bf16_t*>(kind == 0 ? p.k_base : p.v_base) + row_off + static_cast<int64_t>(head) * p.kv_head_stride + dd;
  dst[0] = f32_to_bf16(lo);
  dst[D / 2] = f32_to_bf16(hi);
}

// Second half of the split over d_model: adds the parts append_kernel<..., SPLITK> left in the
// workspace, rotates the keys, casts and writes the cache rows.  Grid (new token, chunk of 256
// items); a thread takes one item, four consecutive features: of V or L as they are, of K together with their
// rotary partners half a head further on.
template <int D, bool PAGED, int MAXP>  // MAXP: 2, 4, 8 or 16, at least the number of parts
__global__ __launch_bounds__(256) void append_finish_kernel(AppendParams p) {
  // A chain of latencies like the other small kernels here: the parameter block in one round trip,
  // the sequence length requested first and by hand, the loads of ALL parts issued at once (from
  // clamped part indices: a part beyond the count is fetched again and not added), and the rotation
  // rates of the pairs worked out while they are in flight.
  asm volatile("" ::"s"(p.split_ws), "s"(p.seq_lens), "s"(p.k_base), "s"(p.v_base), "s"(p.l), "s"(p.block_table));
  asm volatile("" ::"s"(p.n_kv_heads), "s"(p.rank), "s"(p.n_new), "s"(p.seq_index), "s"(p.max_seq_len), "s"(p.k_splits),
               "s"(p.rope_theta), "s"(p.kv_token_stride), "s"(p.kv_head_stride), "s"(p.l_row_stride));
  int len_raw;
  asm volatile("s_load_dword %0, %1, 0x0" : "=s"(len_raw) : "s"(p.seq_lens + p.seq_index));
  const int tid = threadIdx.x;
  const int tok = blockIdx.x;
  const int HD = p.n_kv_heads * D;
  const int n_feat = 2 * HD + p.rank;
  const int k_items = HD / 8, v_items = HD / 4, l_items = p.rank / 4;
  const int it_raw = blockIdx.y * 256 + tid;
  const bool has_item = it_raw < k_items + v_items + l_items;
  const int it = has_item ? it_raw : 0;  // (threads beyond the items repeat item 0 and store nothing)
  const int ks = p.k_splits;
  const float* row = p.split_ws + static_cast<int64_t>(tok) * n_feat;
  const int64_t part_stride = static_cast<int64_t>(p.n_new) * n_feat;
  // first feature of the item's four, and of their rotary partners (key items only)
  const bool is_k = it < k_items, is_v = !is_k && it < k_items + v_items;
  const int head = is_k ? it / (D / 8) : 0, dd = is_k ? (it - head * (D / 8)) * 4 : 0;
  const int f0 = is_k ? head * D + dd : (is_v ? HD + (it - k_items) * 4 : 2 * HD + (it - k_items - v_items) * 4);
  const int f1 = is_k ? f0 + D / 2 : f0;
  float4 x0[MAXP], x1[MAXP];
#pragma unroll
  for (int z = 0; z < MAXP; ++z) {
    const int64_t off = min(z, ks - 1) * part_stride;
    x0[z] = *reinterpret_cast<const float4*>(row + off + f0);
    x1[z] = *reinterpret_cast<const float4*>(row + off + f1);
  }
  __builtin_amdgcn_sched_barrier(0);
  // rotation rates of the pairs, for the workgroups that hold key items (under the loads)
  __shared__ double rope_rate[D / 2];
  if (static_cast<int>(blockIdx.y) * 256 < k_items && p.rope_theta > 0.f) {
    if (tid < D / 2) rope_rate[tid] = rope_rate_rev(tid, D, p.rope_theta);
    __syncthreads();
  }
  if (!has_item) return;
  asm volatile("s_waitcnt lgkmcnt(0)" : "+s"(len_raw));
  const int n_t = append_length(len_raw, p.max_seq_len);
  const int j = n_t - p.n_new + tok;  // cache row of this token, and its position
  if (j < 0) return;
  int64_t kv_off, l_off;  // element offsets of (token j, kv head 0) in K_base / V_base and of row j in L
  if (PAGED) {
    const int blk = p.block_table[static_cast<int64_t>(p.seq_index) * p.max_blocks_per_seq + (j >> 4)];
    kv_off = static_cast<int64_t>(blk) * p.kv_block_stride + static_cast<int64_t>(j & 15) * p.kv_token_stride;
    l_off = (static_cast<int64_t>(blk) * 16 + (j & 15)) * p.l_row_stride;
  } else {
    kv_off = static_cast<int64_t>(j) * p.kv_token_stride;
    l_off = static_cast<int64_t>(j) * p.l_row_stride;
  }
  // the parts in order: the same sum every run
  float4 lo = make_float4(0.f, 0.f, 0.f, 0.f), hi = lo;
#pragma unroll
  for (int z = 0; z < MAXP; ++z)
    if (z < ks) {
      lo.x += x0[z].x; lo.y += x0[z].y; lo.z += x0[z].z; lo.w += x0[z].w;
      hi.x += x1[z].x; hi.y += x1[z].y; hi.z += x1[z].z; hi.w += x1[z].w;
    }
  auto store4 = [&](bf16_t* dst, float4 v) {
    *reinterpret_cast<uint2*>(dst) = make_uint2(pf_pack2(v.x, v.y), pf_pack2(v.z, v.w));
  };
  if (is_k) {
    if (p.rope_theta > 0.f) {
      float l4[4] = {lo.x, lo.y, lo.z, lo.w}, h4[4] = {hi.x, hi.y, hi.z, hi.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float sn, cs;
        rope_sincos(rope_rate[dd + e], j, sn, cs);
        const float a = l4[e], b = h4[e];
        l4[e] = a * cs - b * sn;
        h4[e] = b * cs + a * sn;
      }
      lo = make_float4(l4[0], l4[1], l4[2], l4[3]);
      hi = make_float4(h4[0], h4[1], h4[2], h4[3]);
    }
    bf16_t* dst = static_cast<bf16_t*>(p.k_base) + kv_off + static_cast<int64_t>(head) * p.kv_head_stride + dd;
    store4(dst, lo);
    store4(dst + D / 2, hi);
  } else if (is_v) {
    const int f = f0 - HD, vh = f / D, vd = f - vh * D;
    store4(static_cast<bf16_t*>(p.v_base) + kv_off + static_cast<int64_t>(vh) * p.kv_head_stride + vd, lo);
  } else {
    store4(static_cast<bf16_t*>(p.l) + l_off + (f0 - 2 * HD), lo);
  }
}

template <int D>
static void launch_gemv(const AppendParams& p, hipStream_t s) {
  const int hd = p.n_kv_heads * p.head_dim;
  dim3 grid(2 * (hd / 4) + (p.rank + 3) / 4);
  if (p.block_size != 0) hipLaunchKernelGGL((append_gemv_kernel<D, true>), grid, dim3(256), 0, s, p);
  else hipLaunchKernelGGL((append_gemv_kernel<D, false>), grid, dim3(256), 0, s, p);
}

template <int D, int WI, int XI>
static void launch_skinny(const AppendParams& p, int pp, hipStream_t s) {
  const dim3 grid((p.n_kv_heads * D + pp - 1) / pp, (p.n_new + 8 * XI - 1) / (8 * XI));
  if (p.block_size != 0) hipLaunchKernelGGL((append_skinny_kernel<D, WI, XI, true>), grid, dim3(512), 0, s, p, pp);
  else hipLaunchKernelGGL((append_skinny_kernel<D, WI, XI, false>), grid, dim3(512), 0, s, p, pp);
}

// Pairs per workgroup: one workgroup per compute unit while its rows fit the 16 of a product (up to 1792 K features), else two (16
// kv heads on 4096, 8 tokens: 9.9 us with 4 pairs, 11.2 with 7), and beyond 3072 six pairs (32 kv heads: 15.3 with 6, 15.7 with
// 7, 16.2 with 4).  Two per unit on smaller layers read x twice as often (8 kv heads on 4096, 3 tokens: 6.0 and 7.3).  (From 25
// tokens on their rings leave room for one at a time, and these workgroups run one after the other: with seven pairs, the most a
// product's rows hold, there would still be more than one per unit.)
// Layers of 256 features and less on a width of up to 256 take 0.1 to 0.25 us more at 5 to 16 tokens than with operands straight
// from memory and sixteen features per workgroup (3.1 / 2.85), and neither operands from memory here (3.15), nor a ring of two
// pieces (3.05), nor the rate worked out behind the sums (3.3) brings that back.
// There are 64 workgroups or more, a workgroup for every L feature.
template <int D>
static void launch_skinny_tokens(const AppendParams& p, hipStream_t s) {
  const int hd = p.n_kv_heads * D;
  const int pp = hd <= 1792 ? (hd + 255) / 256 : (hd <= 3072 ? (hd + 511) / 512 : 6);
#define LRA_SKINNY(XI)                                                    \
  (pp <= 3 ? launch_skinny<D, 1, XI>(p, pp, s) : launch_skinny<D, 2, XI>(p, pp, s))
  switch ((p.n_new + 7) / 8) {
    case 1: return LRA_SKINNY(1);
    case 2: return LRA_SKINNY(2);
    case 3: return LRA_SKINNY(3);
    case 4: return LRA_SKINNY(4);
    case 5: return LRA_SKINNY(5);
    case 6: return LRA_SKINNY(6);
    case 7: return LRA_SKINNY(7);
    default: return LRA_SKINNY(8);
  }
#undef LRA_SKINNY
}

// Whether the 256 x 256 tiles, one workgroup per compute unit, are faster than the 128 x 128 tiles with two.  An XCD
// takes every eighth token tile with all its feature tiles, 32 tiles at a time.  Estimated times of rounds, in units
// of 1 / 64 of d_model = 4096: 64 for 512 tiles of 128, three more for every round before it, 31 for a rest of up to
// 256 of them and 54 to 70 beyond; 110 for a full round of an XCD, 74 to 118 for a partial one, 6 % more with two
// blocks of L rows to stage.  Fitted to 650 calls of thirteen layers.  us with 128 and with 256: Llama-3-8B projection
// 3500 new tokens 64 and 96, 6000 127 and 101, 8192 171 and 117, 8700 161 and 192 (two of the XCDs go a second round),
// 12000 252 and 201; 12 kv heads on d_model 2048, 4500 71 and 104; 32 kv heads, 2500 175 and 211, 7000 526 and 445.
// A K and V region that is no multiple of 256 features fills its last feature tile in part and never gains.
static bool wide_tiles_pay(const AppendParams& p, int hd, int64_t tiles128) {
  if (hd % 256 != 0 || tiles128 <= 256) return false;
  const int64_t per_xcd = static_cast<int64_t>(((p.n_new + 255) / 256 + 7) / 8) * 2 * (hd / 256);
  const double rounds = static_cast<double>(tiles128 / 512), rest = static_cast<double>(tiles128 % 512);
  const double part = static_cast<double>(per_xcd % 32) / 32;
  const double t128 = 64.0 * rounds + 1.5 * rounds * (rounds - 1.0) + (rest == 0 ? 0.0 : (rest <= 256 ? 31.0 : 54.0 + 16.0 * (rest - 256) / 256));
  const double t256 = 110.5 * static_cast<double>(per_xcd / 32) + (part == 0 ? 0.0 : 74.0 + 44.0 * part);
  return t256 * (p.rank > 32 ? 1.06 : 1.0) < 0.95 * t128;
}

hipError_t launch_append(const AppendParams& p, bool quarter_tiles, hipStream_t s) {
  const int hd = p.n_kv_heads * p.head_dim;
  const bool paged = p.block_size != 0;
  if (p.k_splits > 1) {
    // Split over d_model (chosen by the host from the sizes, with a workspace): tiles of 128 features
    // x 64 or 128 tokens, four LDS stages, p.k_splits parts, then the finishing kernel.
    const int bt = p.split_bt;
    const int64_t tiles = static_cast<int64_t>((p.n_new + bt - 1) / bt) * (2 * ((hd + 127) / 128) + 1) * p.k_splits;
    const dim3 grid(static_cast<unsigned>((tiles + 7) / 8 * 8));  // (see append_kernel)
#define LRA_APPEND_SPLIT(DD, PG)                                                                                        \
  do {                                                                                                                  \
    if (bt == 64) hipLaunchKernelGGL((append_kernel<DD, PG, 4, 64, true>), grid, dim3(512), 0, s, p);                   \
    else hipLaunchKernelGGL((append_kernel<DD, PG, 4, 128, true>), grid, dim3(512), 0, s, p);                           \
    if (hipGetLastError() != hipSuccess) return hipErrorLaunchFailure;                                                   \
    const dim3 fgrid(p.n_new, (hd / 8 + hd / 4 + p.rank / 4 + 255) / 256);                                              \
    if (p.k_splits <= 2) hipLaunchKernelGGL((append_finish_kernel<DD, PG, 2>), fgrid, dim3(256), 0, s, p);              \
    else if (p.k_splits <= 4) hipLaunchKernelGGL((append_finish_kernel<DD, PG, 4>), fgrid, dim3(256), 0, s, p);         \
    else if (p.k_splits <= 8) hipLaunchKernelGGL((append_finish_kernel<DD, PG, 8>), fgrid, dim3(256), 0, s, p);         \
    else hipLaunchKernelGGL((append_finish_kernel<DD, PG, 16>), fgrid, dim3(256), 0, s, p);                             \
  } while (0)
    if (p.head_dim == 128) {
      if (paged) LRA_APPEND_SPLIT(128, true);
      else LRA_APPEND_SPLIT(128, false);
    } else {
      if (paged) LRA_APPEND_SPLIT(64, true);
      else LRA_APPEND_SPLIT(64, false);
    }
#undef LRA_APPEND_SPLIT
    return hipGetLastError();
  }
  if (p.n_new <= p.skinny_max) {
    if (p.head_dim == 128) p.n_new == 1 ? launch_gemv<128>(p, s) : launch_skinny_tokens<128>(p, s);
    else p.n_new == 1 ? launch_gemv<64>(p, s) : launch_skinny_tokens<64>(p, s);
    return hipGetLastError();
  }
  if (quarter_tiles) {
    const int items = (p.n_new + 63) / 64 * (2 * hd / 64);
    const dim3 qgrid((items + 7) / 8 * 8);  // (see the kernel)
    if (p.head_dim == 128) {
      if (paged) hipLaunchKernelGGL((append_quarter_kernel<128, true>), qgrid, dim3(512), 0, s, p);
      else hipLaunchKernelGGL((append_quarter_kernel<128, false>), qgrid, dim3(512), 0, s, p);
    } else {
      if (paged) hipLaunchKernelGGL((append_quarter_kernel<64, true>), qgrid, dim3(512), 0, s, p);
      else hipLaunchKernelGGL((append_quarter_kernel<64, false>), qgrid, dim3(512), 0, s, p);
    }
    return hipGetLastError();
  }
  const int n_ft = 2 * ((hd + 127) / 128) + 1;
  const int64_t tiles128 = static_cast<int64_t>((p.n_new + 127) / 128) * n_ft;
  // (four feature tiles and more: what the kernel's division of the L features assumes)
  if (hd > 256 && (p.tile == 256 || (p.tile == 0 && p.stages == 0 && wide_tiles_pay(p, hd, tiles128)))) {
    const int n_ct = 2 * ((hd + 255) / 256), t8 = ((p.n_new + 255) / 256 + 7) / 8;
    const dim3 wgrid(8 * t8 * n_ct);  // (see the kernel: XCD, feature tile, token tile)
#define LRA_APPEND_WIDE(DD, PG)                                                                          \
  do {                                                                                                   \
    if (p.rank <= 32) hipLaunchKernelGGL((append_wide_kernel<DD, PG, 1>), wgrid, dim3(512), 0, s, p);    \
    else hipLaunchKernelGGL((append_wide_kernel<DD, PG, 2>), wgrid, dim3(512), 0, s, p);                 \
  } while (0)
    if (p.head_dim == 128) {
      if (paged) LRA_APPEND_WIDE(128, true);
      else LRA_APPEND_WIDE(128, false);
    } else {
      if (paged) LRA_APPEND_WIDE(64, true);
      else LRA_APPEND_WIDE(64, false);
    }
#undef LRA_APPEND_WIDE
    return hipGetLastError();
  }
  const dim3 grid(static_cast<unsigned>((tiles128 + 7) / 8 * 8));
  // One workgroup per compute unit or fewer: nothing shares the LDS, so a deeper ring of
  // stages (more requests in flight per workgroup) is free; beyond that two workgroups per
  // unit with two stages each hide each other's waits.  Not where those would be one round and a little
  // (up to 700 tiles): three rounds of one workgroup per unit then take less than two of two (us with two
  // and with three stages: 576 tiles 87 and 78, 612 105 and 95, 680 110 and 101, 700 62.5 and 62).
  const int stages = p.stages != 0 ? p.stages : (tiles128 <= 256 ? 4 : (tiles128 > 512 && tiles128 <= 700 ? 3 : 2));
  // half-size token tiles while one round of one workgroup per unit holds them, or when asked for (us with 64-token
  // and with 128-token tiles: Llama-3-8B projection 512 new tokens 23 and 28, 700 22 and 28; 8 kv heads of 64 on
  // 2048, 1500 new tokens 13 and 17)
  const int64_t tiles64 = static_cast<int64_t>((p.n_new + 63) / 64) * n_ft;
  if (p.tile == 64 || (p.tile == 0 && p.stages == 0 && tiles64 <= 256)) {
    const dim3 g64(static_cast<unsigned>((tiles64 + 7) / 8 * 8));
    if (p.head_dim == 128) {
      if (paged) hipLaunchKernelGGL((append_kernel<128, true, 4, 64>), g64, dim3(512), 0, s, p);
      else hipLaunchKernelGGL((append_kernel<128, false, 4, 64>), g64, dim3(512), 0, s, p);
    } else {
      if (paged) hipLaunchKernelGGL((append_kernel<64, true, 4, 64>), g64, dim3(512), 0, s, p);
      else hipLaunchKernelGGL((append_kernel<64, false, 4, 64>), g64, dim3(512), 0, s, p);
    }
    return hipGetLastError();
  }
#define LRA_APPEND_LAUNCH(DD, PG, NS_) hipLaunchKernelGGL((append_kernel<DD, PG, NS_>), grid, dim3(NS_ == 2 ? 256 : 512), 0, s, p)
#define LRA_APPEND_STAGES(DD, PG)            \
  do {                                       \
    if (stages == 2) LRA_APPEND_LAUNCH(DD, PG, 2);      \
    else if (stages == 3) LRA_APPEND_LAUNCH(DD, PG, 3); \
    else LRA_APPEND_LAUNCH(DD, PG, 4);                  \
  } while (0)
  if (p.head_dim == 128) {
    if (paged) LRA_APPEND_STAGES(128, true);
    else LRA_APPEND_STAGES(128, false);
  } else {
    if (paged) LRA_APPEND_STAGES(64, true);
    else LRA_APPEND_STAGES(64, false);
  }
#undef LRA_APPEND_STAGES
#undef LRA_APPEND_LAUNCH
  return hipGetLastError();
}

}  // namespace lra
