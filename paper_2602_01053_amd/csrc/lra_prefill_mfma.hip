// MFMA causal prefill kernel of the Flash-LoRA-Attention library (bf16, gfx950).
//
// Alg. 1 of LRAgent (Sec. 3.3) for L_c new tokens of one agent after L_p cached
// ones, with the key side reordered as in App. D.1: per 64-key tile
//   S^T[key][row]  = K_base[key][:] . Q[row][:] + L[key][:] . Qt[row][:]   (MFMA, k = d + r)
//   online softmax along keys, causal mask aligned to the end of the sequence
//   O^T[d][row]   += V_base^T[d][key] . P^T[key][row]                      (MFMA)
//   Olr^T[p][row] += L^T[p][key]      . P^T[key][row]                      (MFMA)
// and after the last tile O^T += B_V^T . Olr^T (two more MFMA k-steps per 16 ranks: Olr, an
// fp32 sum over all keys, enters as two bf16 terms), O /= l.  Qt = Q B_K^T is formed once per
// wave before the loop (MFMA).
//
// A workgroup owns a q tile of 128 query rows (4 waves x 32 rows) and walks the key tiles up to
// its causal limit.  A row is a new token of one of tile_group q heads of a kv head, the q head
// fastest: of all that share the kv head where keys are the larger part of a call (a tile of 128
// tokens of one q head is a quarter full at 32 new tokens, and four workgroups walk every key;
// 333 tokens on 5333, group 4: 76 us with tiles of one head, 57 with tiles of the group), of one
// where a few tokens meet few keys (see plan_prefill_tiles).  v_mfma_f32_32x32x16_bf16
// throughout; the transposed score tile leaves P^T in the lanes that need it as the B operand
// of the second product.  K_base / V_base / L tiles are shared by the four waves:
// every wave requests its quarter of the next tile straight from HBM into the
// other LDS stage (buffer_load ... lds, swizzled by choosing which chunk each lane
// fetches) at the top of the current tile; one wait and one barrier per tile.
// ds_read_b128 feeds the K operand, ds_read_b64_tr_b16 the transposed V and L
// operands, both scheduled several products ahead.  Two workgroups share a CU, so
// the softmax arithmetic of one overlaps the matrix work of the other.
// Workgroups are numbered so that all q tiles of a kv head run on the same XCD and
// share its L2.
#include "lra_prefill_util.h"

namespace lra {

// HAS_BK = false is the value-only setting (b_k == NULL, keys fully shared): no Qt and no
// L term in the scores; L is still staged for P.L.
// SPLIT = true: the key tiles of a q tile are shared by gridDim.y workgroups; each leaves its
// softmax state (m, l, O, O_lr per row) in the workspace and the merge kernel combines
// them, applies B_V and normalises (for calls with too few q tiles to fill the chip).
// ROPE_K = true (with HAS_BK = false) is the rotary key side of App. D.1: the cached keys are
// rotated ones and the adapter's contribution has to be rotated by its key's position before
// the score, so it cannot ride on Qt.  Instead every key tile is completed in LDS before the
// scores are taken: E^T = B_K^T . L^T for the tile's 64 keys (two MFMAs per wave and 16
// ranks: a wave owns 32 keys and the two 32-feature blocks that hold the halves of its rotary
// pairs, so both halves of a pair sit in the same lane and register), rotated, and added to
// the K_base rows of the tile (8-byte read-modify-writes in bf16).  One more barrier per
// tile; the score loop is the value-only one.
// POOL = true: a paged cache whose blocks lie within 32-bit byte offsets (see PfTileLoader).
template <int D, int RP, bool PAGED, bool HAS_BK, bool SPLIT, bool ROPE_K = false, bool KC16 = false>
__global__ __launch_bounds__(256, 2) void prefill_mfma_kernel(Params p) {
  constexpr bool POOL = false;
#include "lra_prefill_body.h"
}
// paged caches within 32-bit byte offsets, without in-kernel completion of the keys
template <int D, int RP, bool HAS_BK, bool SPLIT, bool KC16>
__device__ __forceinline__ void prefill_pool_tiles(const Params p) {
  constexpr bool PAGED = true, ROPE_K = false, POOL = true;
#include "lra_prefill_body.h"
}
template <int D, int RP, bool HAS_BK, bool SPLIT, bool KC16>
__global__ __launch_bounds__(256, 2) void prefill_pool_kernel(Params p) {
  prefill_pool_tiles<D, RP, HAS_BK, SPLIT, KC16>(p);
}

template <int D, int RP, bool SPLIT>
static hipError_t launch_pf2(const Params& p, dim3 grid, hipStream_t s) {
  const bool paged = p.block_size != 0, has_bk = p.b_k != nullptr;
  if (has_bk && p.key_rope_theta > 0.f) {
    if (paged) hipLaunchKernelGGL((prefill_mfma_kernel<D, RP, true, false, SPLIT, true>), grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((prefill_mfma_kernel<D, RP, false, false, SPLIT, true>), grid, dim3(256), 0, s, p);
    return hipGetLastError();
  }
  if (paged && prefill_pool_fits(p)) {
    if (p.keys_f16 && has_bk) return hipErrorInvalidValue;
    if (p.keys_f16) hipLaunchKernelGGL((prefill_pool_kernel<D, RP, false, SPLIT, true>), grid, dim3(256), 0, s, p);
    else if (has_bk) hipLaunchKernelGGL((prefill_pool_kernel<D, RP, true, SPLIT, false>), grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((prefill_pool_kernel<D, RP, false, SPLIT, false>), grid, dim3(256), 0, s, p);
    return hipGetLastError();
  }
  if (p.keys_f16) {  // (set by the host only where the pre-pass has completed the keys)
    if (has_bk) return hipErrorInvalidValue;
    if (paged) hipLaunchKernelGGL((prefill_mfma_kernel<D, RP, true, false, SPLIT, false, true>), grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((prefill_mfma_kernel<D, RP, false, false, SPLIT, false, true>), grid, dim3(256), 0, s, p);
    return hipGetLastError();
  }
  if (paged && has_bk)
    hipLaunchKernelGGL((prefill_mfma_kernel<D, RP, true, true, SPLIT>), grid, dim3(256), 0, s, p);
  else if (paged)
    hipLaunchKernelGGL((prefill_mfma_kernel<D, RP, true, false, SPLIT>), grid, dim3(256), 0, s, p);
  else if (has_bk)
    hipLaunchKernelGGL((prefill_mfma_kernel<D, RP, false, true, SPLIT>), grid, dim3(256), 0, s, p);
  else
    hipLaunchKernelGGL((prefill_mfma_kernel<D, RP, false, false, SPLIT>), grid, dim3(256), 0, s, p);
  return hipGetLastError();
}

template <int D, int RP>
static hipError_t launch_pf(const Params& p, dim3 grid, hipStream_t s) {
  return p.n_splits > 1 ? launch_pf2<D, RP, true>(p, grid, s) : launch_pf2<D, RP, false>(p, grid, s);
}

hipError_t launch_prefill_mfma(const Params& p, hipStream_t s) {
  const int q_tiles = (p.n_new * p.tile_group + 127) / 128;
  dim3 grid(q_tiles * p.n_kv_heads * (p.group / p.tile_group), p.n_splits);
  const int rp = p.rank <= 16 ? 16 : (p.rank <= 32 ? 32 : 64);
  if (p.head_dim == 128) {
    if (rp == 16) return launch_pf<128, 16>(p, grid, s);
    if (rp == 32) return launch_pf<128, 32>(p, grid, s);
    return launch_pf<128, 64>(p, grid, s);
  }
  if (rp == 16) return launch_pf<64, 16>(p, grid, s);
  if (rp == 32) return launch_pf<64, 32>(p, grid, s);
  return launch_pf<64, 64>(p, grid, s);
}

// ---------------------------------------------------------------------------------------
// Rotary key side, contiguous caches: the keys of the call's one adapter, formed once.
//   K_j = K_base,j + RoPE_j(L_j B_K^a)             (App. D.1: with LoRA on the key projection the
//                                                   adapter's part is rebuilt in the head dimension
//                                                   before the rotation)
// The tile-walking kernel can complete every key tile in LDS itself, but a call of many q tiles
// then repeats that work in every workgroup that walks the tile (q tiles x q heads of the kv head:
// 64 times at 2048 new tokens and a group of 4).  This pre-pass writes the completed keys of all
// visible tokens into the workspace, in the layout of K_base (same strides), and the call then
// runs the plain kernel without a key-side adapter on them.  HBM bound: K_base read and written
// once (+ L); rank x d multiply-adds per key and head on the vector ALU.
// One workgroup per (16 keys, kv head); lane (key, group g of 16): the pairs (dd, dd + d/2),
// dd = PPL g .. PPL g + PPL - 1, PPL = d/32.  E in fp32, angle = fractional part of position x rate
// in double precision, as in the producer of the caches.
// ---------------------------------------------------------------------------------------
template <int D, bool PAGED>
__global__ __launch_bounds__(256) void complete_rope_keys_kernel(Params p, unsigned short* kc) {
  constexpr int PPL = D / 32;              // rotary pairs per lane
  __shared__ __align__(16) unsigned short b_lds[64 * D];  // B_K^a rows of this kv head, [rho][d]
  __shared__ double rate[D / 2];
  const int tid = threadIdx.x;
  const int h = blockIdx.y;
  const int r = p.rank;
  const int n_t = min(PF_CONST_I32(p.seq_lens)[p.seq_index], p.max_seq_len);
  const int j = blockIdx.x * 16 + (tid >> 4);
  if (blockIdx.x * 16 >= n_t) return;
  const int a = min(max(p.adapter_index, 0), p.n_adapters - 1);
  const unsigned short* bk = static_cast<const unsigned short*>(p.b_k) +
                             (static_cast<int64_t>(a) * r * p.n_kv_heads + h) * D;
  for (int i = tid; i < r * (D / 8); i += 256) {
    const int rho = i / (D / 8), c = i - rho * (D / 8);
    *reinterpret_cast<uint4*>(b_lds + rho * D + c * 8) =
        *reinterpret_cast<const uint4*>(bk + static_cast<int64_t>(rho) * p.n_kv_heads * D + c * 8);
  }
  if (tid < D / 2) rate[tid] = rope_rate_rev(tid, D, p.key_rope_theta);
  __syncthreads();
  if (j >= n_t) return;
  const int g = tid & 15;
  // paged: the key's block comes from the sequence's row of the block table; the completed keys are written at
  // the block's LOGICAL index (the kernel that reads them needs no table for them)
  const int blk = PAGED ? PF_CONST_I32(p.block_table)[static_cast<int64_t>(p.seq_index) * p.max_blocks_per_seq + (j >> 4)] : 0;
  const int64_t l_index = PAGED ? static_cast<int64_t>(blk) * 16 + (j & 15) : j;
  const unsigned short* lrow = static_cast<const unsigned short*>(p.l) + static_cast<int64_t>(a) * p.l_adapter_stride +
                               l_index * p.l_row_stride;
  float lo[PPL], hi[PPL];
#pragma unroll
  for (int i = 0; i < PPL; ++i) lo[i] = hi[i] = 0.f;
  for (int r0 = 0; r0 < r; r0 += 8) {  // the rank is a multiple of 8
    const uint4 lv = *reinterpret_cast<const uint4*>(lrow + r0);
    const uint32_t lw[4] = {lv.x, lv.y, lv.z, lv.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float lf = __uint_as_float((e & 1) ? (lw[e >> 1] & 0xffff0000u) : (lw[e >> 1] << 16));
      const unsigned short* brow = b_lds + (r0 + e) * D + PPL * g;
#pragma unroll
      for (int i = 0; i < PPL; ++i) {
        lo[i] = fmaf(lf, __uint_as_float(static_cast<uint32_t>(brow[i]) << 16), lo[i]);
        hi[i] = fmaf(lf, __uint_as_float(static_cast<uint32_t>(brow[D / 2 + i]) << 16), hi[i]);
      }
    }
  }
  const int64_t in_blk = static_cast<int64_t>(PAGED ? (j & 15) : j) * p.kv_token_stride + static_cast<int64_t>(h) * p.kv_head_stride + PPL * g;
  const int64_t off_src = in_blk + (PAGED ? static_cast<int64_t>(blk) * p.kv_block_stride : 0);
  const int64_t off_dst = in_blk + (PAGED ? static_cast<int64_t>(j >> 4) * p.kv_block_stride : 0);
  // the lane's PPL consecutive features of either half: one 8-byte (d = 128) or 4-byte (d = 64) piece
  struct alignas(PPL * 2) Piece { unsigned short v[PPL]; };
  const unsigned short* ksrc = static_cast<const unsigned short*>(p.k_base) + off_src;
  unsigned short* kdst = kc + off_dst;
  const Piece klo = *reinterpret_cast<const Piece*>(ksrc), khi = *reinterpret_cast<const Piece*>(ksrc + D / 2);
  Piece olo, ohi;
#pragma unroll
  for (int i = 0; i < PPL; ++i) {
    float sn, cs;
    rope_sincos(rate[PPL * g + i], j, sn, cs);
    // (as fp16: see prefill_mfma_kernel)
    olo.v[i] = __builtin_bit_cast(unsigned short, static_cast<_Float16>(__uint_as_float(static_cast<uint32_t>(klo.v[i]) << 16) + (lo[i] * cs - hi[i] * sn)));
    ohi.v[i] = __builtin_bit_cast(unsigned short, static_cast<_Float16>(__uint_as_float(static_cast<uint32_t>(khi.v[i]) << 16) + (hi[i] * cs + lo[i] * sn)));
  }
  *reinterpret_cast<Piece*>(kdst) = olo;
  *reinterpret_cast<Piece*>(kdst + D / 2) = ohi;
}

hipError_t launch_complete_rope_keys(const Params& p, void* kc, hipStream_t s) {
  const dim3 grid((p.max_seq_len + 15) / 16, p.n_kv_heads);
  unsigned short* dst = static_cast<unsigned short*>(kc);
  if (p.block_size != 0) {
    if (p.head_dim == 128) hipLaunchKernelGGL((complete_rope_keys_kernel<128, true>), grid, dim3(256), 0, s, p, dst);
    else hipLaunchKernelGGL((complete_rope_keys_kernel<64, true>), grid, dim3(256), 0, s, p, dst);
  } else {
    if (p.head_dim == 128) hipLaunchKernelGGL((complete_rope_keys_kernel<128, false>), grid, dim3(256), 0, s, p, dst);
    else hipLaunchKernelGGL((complete_rope_keys_kernel<64, false>), grid, dim3(256), 0, s, p, dst);
  }
  return hipGetLastError();
}

}  // namespace lra
