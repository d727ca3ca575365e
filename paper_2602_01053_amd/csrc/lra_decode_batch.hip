// Split-KV MFMA decode of a batch in a paged cache (bf16, gfx950): the key shares of all sequences in one row, as many
// as the chip has places for.
//
// The grid of decode_mfma_kernel gives every sequence the same number of key shares: workgroups beyond the end of a
// short sequence find nothing, the last share of each is a remainder, and where the live ones land decides the time
// (16 sequences of 4 k to 64 k tokens: 5.0 TB/s, of equal lengths 5.5).  Here the shares of all sequences stand in one
// row and workgroup w of a (kv head, row group) takes the w-th: every compute unit holds two live workgroups, all of
// them from the start, and a sequence divides its 128-key tiles evenly.  The share size is the smallest with which the
// shares fit batch_wgs places.
//
// The lengths are read on the device: lane t of every wave holds sequence t (at most 64), a scan over the lanes places
// the shares.  The host's share size (from its copy of the lengths, 0: none) is where the search for one that fits
// begins; batch_min_tiles keeps the longest sequence within p.n_splits partial states.  A sequence's last workgroup
// leaves the states behind its own empty.
#include "lra_common.h"
#include "lra_decode_rope.h"
#include "lra_decode_util.h"
#include "lra_plan.h"
#include "lra_prefill_util.h"

namespace lra {

// inclusive sum over the lanes of a wave
__device__ __forceinline__ int scan_lanes(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);  // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, true);  // row_bcast:15
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, true);  // row_bcast:31
  return v;
}

// One share.  (A function of its own: with the body's text in the kernel itself a step took 1.5 % longer, 32 sequences of
// 300 to 40000 tokens 91.7 and 93.4 us.)
template <int D, int RT, int RP, bool HAS_BK, bool PA>
__device__ __forceinline__ void decode_share(const Params& p, const int h, const int t, const int rg, const int split, const int j0,
                                             const int keys, const bool last_of_seq, const int first_query, const int end_query) {
  constexpr bool PAGED = true, CAUSAL = false, LAST = true;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
#include "lra_decode_mfma_body.h"
}

template <int D, int RT, int RP, bool HAS_BK, int RPE, bool PA>
__global__ __launch_bounds__(256, RPE == 64 ? 1 : 2) void decode_batch_kernel(Params p) {
  const int lane = threadIdx.x & 63;
  const int h = blockIdx.x;
  // row groups of a share lcm(8, Hkv) workgroups apart: the same XCD, the next round of the dispatcher (m = rg_interleave)
  int w = blockIdx.y, rg = 0;
  if (p.row_groups > 1) {
    const int m = p.rg_interleave, hi = w >> __builtin_ctz(m), q = hi / p.row_groups;
    rg = hi - q * p.row_groups;
    w = (w & (m - 1)) + m * q;
  }
  int tiles = 0;
  // (the queries of the sequences travel with the lengths: one round trip for both)
  const int q_start = p.seq_query_start[min(lane, p.n_seqs)], q_next = p.seq_query_start[min(lane + 1, p.n_seqs)];
  if (lane < p.n_seqs) tiles = max((min(p.seq_lens[lane], p.max_seq_len) + 127) >> 7, 1);
  const int wgs = p.batch_wgs;
  int size = p.batch_tiles;
  if (size == 0) size = max(p.batch_min_tiles, (__builtin_amdgcn_readlane(scan_lanes(tiles), 63) + wgs - 1) / wgs);
  int shares, end;
  while (true) {  // (ends: with a share the size of the longest sequence there are n_seqs <= batch_wgs of them)
    shares = (tiles + size - 1) / size;
    end = scan_lanes(shares);
    if (__builtin_amdgcn_readlane(end, 63) <= wgs) break;
    size += (size >> 4) + 1;
  }
  if (w >= __builtin_amdgcn_readlane(end, 63)) return;
  const int t = __builtin_popcountll(__builtin_amdgcn_ballot_w64(end <= w) & (p.n_seqs == 64 ? ~0ull : (1ull << p.n_seqs) - 1));
  const int n = __builtin_amdgcn_readlane(shares, t), idx = w - (__builtin_amdgcn_readlane(end, t) - n);
  const int all = __builtin_amdgcn_readlane(tiles, t), len = all / n, more = all - len * n;  // the first `more` shares hold a tile more
  const int j0 = (idx * len + min(idx, more)) * 128, keys = (len + (idx < more ? 1 : 0)) * 128;
  const int first = t > 0 ? __builtin_amdgcn_readlane(q_start, t) : 0, last = t + 1 < p.n_seqs ? __builtin_amdgcn_readlane(q_next, t) : p.n_queries;
  if constexpr (RPE > 0) decode_rope_share<D, RPE, true, false, true>(p, h, t, rg, idx, j0, keys, idx == n - 1, first, last);
  else decode_share<D, RT, RP, HAS_BK, PA>(p, h, t, rg, idx, j0, keys, idx == n - 1, first, last);
}

template <int D, int RT, int RP>
static void launch_batch2(const Params& p, dim3 grid, hipStream_t s) {
  if (p.l_block != 0) {
    if constexpr (RT == 1) {
      if (p.b_k != nullptr) hipLaunchKernelGGL((decode_batch_kernel<D, 1, RP, true, 0, true>), grid, dim3(256), 0, s, p);
      else hipLaunchKernelGGL((decode_batch_kernel<D, 1, RP, false, 0, true>), grid, dim3(256), 0, s, p);
    }
  } else if (p.b_k != nullptr) {
    hipLaunchKernelGGL((decode_batch_kernel<D, RT, RP, true, 0, false>), grid, dim3(256), 0, s, p);
  } else {
    hipLaunchKernelGGL((decode_batch_kernel<D, RT, RP, false, 0, false>), grid, dim3(256), 0, s, p);
  }
}

// (at d = 128 the B_K^T operands of ranks above 32 leave no registers for this form)
static hipError_t launch_batch_rope(const Params& p, dim3 grid, hipStream_t s) {
  const dim3 block(256);
  if (p.head_dim == 128) {
    if (p.rank > 32) return hipErrorInvalidValue;
    if (p.rank <= 16) hipLaunchKernelGGL((decode_batch_kernel<128, 1, 32, true, 16, false>), grid, block, 0, s, p);
    else hipLaunchKernelGGL((decode_batch_kernel<128, 1, 32, true, 32, false>), grid, block, 0, s, p);
  } else if (p.rank <= 16) {
    hipLaunchKernelGGL((decode_batch_kernel<64, 1, 32, true, 16, false>), grid, block, 0, s, p);
  } else if (p.rank <= 32) {
    hipLaunchKernelGGL((decode_batch_kernel<64, 1, 32, true, 32, false>), grid, block, 0, s, p);
  } else {
    hipLaunchKernelGGL((decode_batch_kernel<64, 1, 64, true, 64, false>), grid, block, 0, s, p);
  }
  return hipGetLastError();
}

hipError_t launch_decode_batch(const Params& pp, int row_tiles, hipStream_t s) {
  Params p = pp;
  if (p.block_size == 0 || p.is_prefill || p.n_seqs > 64 || p.batch_wgs < p.n_seqs || p.batch_min_tiles < 1) return hipErrorInvalidValue;
  int g = p.n_kv_heads, e = 8;
  while (e) { const int tmp = g % e; g = e; e = tmp; }  // g = gcd(Hkv, 8)
  const int m = 8 / g;
  p.rg_interleave = m;
  const int gy = p.row_groups > 1 ? (p.batch_wgs + m - 1) / m * m * p.row_groups : p.batch_wgs;
  const dim3 grid(p.n_kv_heads, gy);
  if (p.key_rope_theta > 0.f && p.b_k != nullptr) {
    if (row_tiles != 1 || 16 / p.group_pad > decode_mfma_rope_slots(p.rank)) return hipErrorInvalidValue;
    return launch_batch_rope(p, grid, s);
  }
  const int tile_rank = p.l_block != 0 ? (16 / p.group_pad) * p.l_block : p.rank;
  const int key = (p.head_dim == 128 ? 4 : 0) | (row_tiles == 2 ? 2 : 0) | (tile_rank > 32 ? 1 : 0);
  if (p.l_block != 0 && row_tiles != 1) return hipErrorInvalidValue;
  switch (key) {
    case 0: launch_batch2<64, 1, 32>(p, grid, s); break;
    case 1: launch_batch2<64, 1, 64>(p, grid, s); break;
    case 2: launch_batch2<64, 2, 32>(p, grid, s); break;
    case 3: launch_batch2<64, 2, 64>(p, grid, s); break;
    case 4: launch_batch2<128, 1, 32>(p, grid, s); break;
    case 5: launch_batch2<128, 1, 64>(p, grid, s); break;
    case 6: launch_batch2<128, 2, 32>(p, grid, s); break;
    default: launch_batch2<128, 2, 64>(p, grid, s); break;
  }
  return hipGetLastError();
}

}  // namespace lra
