// MFMA decode kernel of the Flash-LoRA-Attention library (bf16, gfx950).
//
// One workgroup streams one range of keys of one (sequence, kv head) for ALL
// query rows that share that stream: every agent decoding on the sequence times
// the q heads of the GQA group.  Those rows form the 16-wide N dimension of
// v_mfma_f32_16x16x32_bf16, so K_base, V_base and L are read from HBM once for
// all agents (LRAgent Sec. 3.2: one base cache and one LR cache for the system).
//
// Per 32-key step (the inner loop of Alg. 1 with the App. D.1 key-side reordering):
//   S^T[key][row]  = K_base[key][:] . Q[row][:]  +  L[key][:] . Qt[row][:]     (MFMA)
//   online softmax along keys (per row = per lane column)
//   O^T[d][row]   += V_base^T[d][key] . P^T[key][row]                          (MFMA)
//   Olr^T[p][row] += L^T[p][key]      . P^T[key][row]                          (MFMA)
// with Qt = Q B_K^T computed once per workgroup in the prologue (MFMA, shared
// through LDS).  Computing S transposed makes the C-layout of the score tile
// coincide with the B-operand layout of the second product, so P never moves
// between lanes.
//
// Data path: buffer_load ... lds (16 bytes per lane, straight from HBM into
// wave-private LDS, no staging registers; K_base and V_base non-temporal, since
// nobody reads them twice, L cached for the workgroups of the other kv heads).  Each lane fetches the 16-byte chunk
// that belongs at ITS LDS slot under an XOR swizzle, so the later ds_read_b128
// (K operand), ds_read_b64 (L operand) and ds_read_b64_tr_b16 (transposed V and
// L operands) avoid bank conflicts.  Keys past the end of a wave's range are
// outside the buffer resource: the hardware returns zeros for them and touches
// no memory, so there is no tail branch on the load side.  A wave holds one
// tile; latency is hidden by the eight waves a CU holds, not by a software
// pipeline inside the wave.  The waves of a workgroup own disjoint key ranges
// and never synchronise inside the loop; their states are merged through LDS at
// the end (flash-decoding rule) and one partial (m, l, O, O_lr) per workgroup
// goes to the workspace.
#include "lra_common.h"
#include "lra_decode_rope.h"
#include "lra_decode_util.h"
#include "lra_plan.h"
#include "lra_prefill_util.h"

namespace lra {

// HAS_BK = false is the value-only setting (b_k == NULL, keys fully shared): no Qt, no
// adapter lookup on the key side, no L term in the scores; L is still streamed for P.L.
// CAUSAL = true serves lra_attn_prefill with a handful of new tokens: the new tokens of the
// one sequence take the place of the agents (same adapter for all), and row i only sees the
// keys up to n - n_new + i (the mask of Alg. 1); a long context is then split over the whole chip
// like any decode call instead of being walked by one workgroup per q head.
//
// RPE > 0 is the rotary key side (lra_decode_rope.h): 16, 32 or 64, the padded rank of its E product, for 4, 2 or 4 agent slots
// per tile with operands in registers; at 64 one workgroup fills a compute unit and its waves have 512 registers.
//
// PA = true is the decode form for one low-rank cache per adapter (BaseShared, Sec. 3.2) outside the rotary key
// side: the L tile is a row of column blocks [agent slot][32 keys][l_block ranks], block s requested from the cache
// of the adapter of agent slot s; Qt of a row stands in the block of its slot and is zero elsewhere, so the same
// products give Qt_a . L_a^T and P . L_a per agent, and a row keeps only its own block of O_lr.  K_base and V_base are
// then read once for all agents of a tile, and no zero padding is streamed.
// The body as a function of its own, for the form whose registers come out better behind that boundary: value-only adapters
// with their own low-rank caches on pages, d = 64, 20.0 us at the text, 19.7 at the function.
template <bool PAGED, bool HAS_BK, bool PA>
constexpr bool kDecodeByFunction = PA && PAGED && !HAS_BK;
template <int D, int RT, int RP, bool PAGED, bool HAS_BK, bool CAUSAL, bool PA>
__device__ __forceinline__ void decode_mfma_keys(const Params& p, const int h, const int t, const int rg, const int split,
                                                 const int j0, const int keys) {
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr bool LAST = false, last_of_seq = false;
  constexpr int first_query = 0, end_query = 0;
#include "lra_decode_mfma_body.h"
}

template <int D, int RT, int RP, bool PAGED, bool HAS_BK, bool CAUSAL, int RPE = 0, bool PA = false>
__global__ __launch_bounds__(256, RPE == 64 ? 1 : 2) void decode_mfma_kernel(Params p) {
  [[maybe_unused]] const int lane = threadIdx.x & 63;
  [[maybe_unused]] const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // kv head is the fastest grid index: workgroups go round-robin over the XCDs, so with 8 kv
  // heads all workgroups of a head run on one XCD and share Q and B_K in its L2
  const int h = blockIdx.x;
  int split = blockIdx.y;
  int t = CAUSAL ? p.seq_index : blockIdx.z / p.row_groups;
  int rg = CAUSAL ? blockIdx.z : blockIdx.z - t * p.row_groups;
  if (p.rg_interleave > 0) {
    // Several row groups share the keys of a (sequence, kv head, key share): only the first to ask reads them from
    // HBM if the others ask the same L2 soon after.  Workgroups go round-robin over the 8 XCDs in the order of
    // their linear index x + Hkv * y, so with m = lcm(8, Hkv) / Hkv and y = (share mod m) + m * (row group +
    // row_groups * (share / m)) the row groups of a share are lcm(8, Hkv) workgroups apart: the same XCD, the next
    // round of the dispatcher.  (z is the sequence.)  Key shares are padded to a multiple of m; in the rotary form, where a
    // workgroup without keys can push another into the next round, those behind the last multiple stand in the order of
    // the plain grid.
    const int m = p.rg_interleave, y = blockIdx.y;
    const int whole = RPE > 0 ? p.n_splits & ~(m - 1) : p.n_splits;
    if (RPE > 0 && y >= whole * p.row_groups) {
      const int rest = p.n_splits - whole, at = y - whole * p.row_groups;
      rg = at / rest;
      split = whole + at - rg * rest;
    } else {
      const int hi = y >> __builtin_ctz(m);
      const int q = hi / p.row_groups;
      rg = hi - q * p.row_groups;
      split = (y & (m - 1)) + m * q;
    }
    t = CAUSAL ? p.seq_index : blockIdx.z;
    if (split >= p.n_splits) return;
  }
  if constexpr (RPE > 0) {
    int j0 = split * p.split_keys, keys = p.split_keys;
    if (p.split_more > 0 && split >= p.split_more) {
      j0 -= (split - p.split_more) * 128;
      keys -= 128;
    }
    decode_rope_share<D, RPE, PAGED, CAUSAL, false>(p, h, t, rg, split, j0, keys, false, 0, 0);
  } else if constexpr (kDecodeByFunction<PAGED, HAS_BK, PA>) {
    decode_mfma_keys<D, RT, RP, PAGED, HAS_BK, CAUSAL, PA>(p, h, t, rg, split, split * p.split_keys, p.split_keys);
  } else {
    constexpr bool LAST = false, last_of_seq = false;
    constexpr int first_query = 0, end_query = 0;
    const int j0 = split * p.split_keys, keys = p.split_keys;
#include "lra_decode_mfma_body.h"
  }
}

template <int D, int RT, int RP, bool CAUSAL>
static hipError_t launch_cfg2(const Params& p, dim3 grid, hipStream_t s) {
  const dim3 block(256);
  const bool paged = p.block_size != 0, has_bk = p.b_k != nullptr;
  if (p.l_block != 0) {
    // per-adapter low-rank caches, one column block of the L tile per agent slot: decode, one row tile
    if constexpr (RT == 1 && !CAUSAL) {
      if (paged && has_bk) hipLaunchKernelGGL((decode_mfma_kernel<D, 1, RP, true, true, false, 0, true>), grid, block, 0, s, p);
      else if (paged) hipLaunchKernelGGL((decode_mfma_kernel<D, 1, RP, true, false, false, 0, true>), grid, block, 0, s, p);
      else if (has_bk) hipLaunchKernelGGL((decode_mfma_kernel<D, 1, RP, false, true, false, 0, true>), grid, block, 0, s, p);
      else hipLaunchKernelGGL((decode_mfma_kernel<D, 1, RP, false, false, false, 0, true>), grid, block, 0, s, p);
      return hipGetLastError();
    } else {
      return hipErrorInvalidValue;
    }
  }
  if (paged && has_bk)
    hipLaunchKernelGGL((decode_mfma_kernel<D, RT, RP, true, true, CAUSAL>), grid, block, 0, s, p);
  else if (paged)
    hipLaunchKernelGGL((decode_mfma_kernel<D, RT, RP, true, false, CAUSAL>), grid, block, 0, s, p);
  else if (has_bk)
    hipLaunchKernelGGL((decode_mfma_kernel<D, RT, RP, false, true, CAUSAL>), grid, block, 0, s, p);
  else
    hipLaunchKernelGGL((decode_mfma_kernel<D, RT, RP, false, false, CAUSAL>), grid, block, 0, s, p);
  return hipGetLastError();
}

template <int D, int RT, int RP>
static hipError_t launch_cfg(const Params& p, dim3 grid, hipStream_t s) {
  return p.is_prefill ? launch_cfg2<D, RT, RP, true>(p, grid, s) : launch_cfg2<D, RT, RP, false>(p, grid, s);
}

template <int D, int RP, int RPE>
static hipError_t launch_rope(const Params& p, dim3 grid, hipStream_t s) {
  const bool paged = p.block_size != 0;
  if (p.is_prefill) {
    if (paged) hipLaunchKernelGGL((decode_mfma_kernel<D, 1, RP, true, true, true, RPE>), grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((decode_mfma_kernel<D, 1, RP, false, true, true, RPE>), grid, dim3(256), 0, s, p);
  } else {
    if (paged) hipLaunchKernelGGL((decode_mfma_kernel<D, 1, RP, true, true, false, RPE>), grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((decode_mfma_kernel<D, 1, RP, false, true, false, RPE>), grid, dim3(256), 0, s, p);
  }
  return hipGetLastError();
}

static hipError_t launch_decode_mfma_grid(const Params& p, int row_tiles, dim3 grid, hipStream_t s);

hipError_t launch_decode_mfma(const Params& p, int row_tiles, bool allow_stream_form, bool main_kernel_only, hipStream_t s) {
  // calls that give a compute unit at most one workgroup: the form with two tile stages per wave
  if (allow_stream_form && decode_stream_applies(p, row_tiles, 256)) return launch_decode_stream(p, row_tiles, main_kernel_only, s);
  dim3 grid(p.n_kv_heads, p.n_splits, (p.is_prefill ? 1 : p.n_seqs) * p.row_groups);
  Params pi = p;
  pi.rg_interleave = 0;
  const int n_seqs = p.is_prefill ? 1 : p.n_seqs;
  const bool rotary = p.key_rope_theta > 0.f && p.b_k != nullptr;
  const int m = mfma_interleave(p.n_kv_heads, p.n_splits, p.row_groups, rotary);
  if (m > 0) {
    // (see the kernel: row groups of a key share next to each other on one XCD)
    pi.rg_interleave = m;
    const int shares = rotary ? p.n_splits : (p.n_splits + m - 1) / m * m;
    grid = dim3(p.n_kv_heads, static_cast<unsigned>(shares * p.row_groups), n_seqs);
  }
  return launch_decode_mfma_grid(pi, row_tiles, grid, s);
}

static hipError_t launch_decode_mfma_grid(const Params& p, int row_tiles, dim3 grid, hipStream_t s) {
  if (p.key_rope_theta > 0.f && p.b_k != nullptr) {
    if (row_tiles != 1 || (!p.is_prefill && 16 / p.group_pad > decode_mfma_rope_slots(p.rank))) return hipErrorInvalidValue;
    const int sel = (p.head_dim == 128 ? 3 : 0) + (p.rank <= 16 ? 0 : (p.rank <= 32 ? 1 : 2));
    switch (sel) {
      case 0: return launch_rope<64, 32, 16>(p, grid, s);
      case 1: return launch_rope<64, 32, 32>(p, grid, s);
      case 2: return launch_rope<64, 64, 64>(p, grid, s);
      case 3: return launch_rope<128, 32, 16>(p, grid, s);
      case 4: return launch_rope<128, 32, 32>(p, grid, s);
      default: return launch_rope<128, 64, 64>(p, grid, s);
    }
  }
  // columns of the L tile: the rank, or with per-adapter low-rank caches one block per agent slot of a row tile
  const int tile_rank = (p.l_block != 0 && !p.is_prefill) ? (16 / p.group_pad) * p.l_block : p.rank;
  const int rp = tile_rank <= 32 ? 32 : 64;
  const int key = (p.head_dim == 128 ? 4 : 0) | (row_tiles == 2 ? 2 : 0) | (rp == 64 ? 1 : 0);
  switch (key) {
    case 0: return launch_cfg<64, 1, 32>(p, grid, s);
    case 1: return launch_cfg<64, 1, 64>(p, grid, s);
    case 2: return launch_cfg<64, 2, 32>(p, grid, s);
    case 3: return launch_cfg<64, 2, 64>(p, grid, s);
    case 4: return launch_cfg<128, 1, 32>(p, grid, s);
    case 5: return launch_cfg<128, 1, 64>(p, grid, s);
    case 6: return launch_cfg<128, 2, 32>(p, grid, s);
    default: return launch_cfg<128, 2, 64>(p, grid, s);
  }
}

}  // namespace lra
