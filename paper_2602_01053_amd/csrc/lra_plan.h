// Host-side launch planning of the Flash-LoRA-Attention library: argument checks and the choice
// of kernel family, key shares, row packing and workspace layout.  Plain C++ with no HIP
// dependency, so that the arithmetic (32-bit offset caps, workspace sizes) can also be compiled
// for the CPU alone and run under the address and undefined-behaviour sanitizers.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include "lra_attn.h"

namespace lra {

constexpr int kCUs = 256;  // MI355X

// lra_tuning with every "0 = automatic" resolved.
struct Tuning {
  int variant = 0;          // 0 automatic, 1 vector-ALU kernels, 2 MFMA kernels without the streaming form
  int split_keys = 0;       // keys per workgroup in decode, 0 = automatic
  int short_prefill = 32;   // new tokens up to which a prefill takes the split-KV path (0 = never)
  int prefill_splits = 0;   // workgroups sharing the key tiles of a q tile, 0 = automatic, -1 = one, q tiles as automatic
  bool rope_key_prepass = true;  // rotary prefill on contiguous caches: completed keys by a pre-pass
  int append_skinny = 64;   // new tokens up to which lra_cache_append streams the weights (0 = never)
  int append_stages = 0;    // LDS stages of the tiled append GEMM, 0 = chosen from the grid
  int append_tile = 0;      // output tile of the append GEMM, 0 = chosen from the grid
  int append_k_splits = 0;  // parts of d_model in the append GEMM: 0 = chosen from the grid, 1 = never split
  bool stream_shares = true;      // shares and calls of the streaming kernel beside the rest of a plan (false: a workspace without room for them)
  bool main_kernel_only = false;  // measurement: enqueue only the dominant kernel of a call
};
Tuning resolve_tuning(const lra_tuning* t);

struct Plan {
  bool mfma;
  bool short_prefill;  // prefill served by the split-KV decode kernels (few new tokens)
  int rows;        // query rows = (queries | new tokens) x Hq
  int split_keys;  // keys per split
  int n_splits;    // splits per sequence at max_seq_len
  int split_more;  // 0: all splits alike; else only the first so many hold split_keys, those behind them 128 keys less
  bool split_kv_sized;  // prefill: few new tokens behind a context, the sizes the split-KV path is for (whatever path it takes)
  bool wave_rows;  // prefill: workgroups of 32 rows whose waves divide the keys (prefill_rows_kernel), whatever the rest says
  int wave_shares;  // ... or, if not 0, that kernel with this many workgroups dividing the keys of 32 rows, then the merge kernel
  // The streaming kernel (stream_keys > 0; nothing is rotated then, one sequence, at most one workgroup per unit) with other key shares
  // than the rest says, or in place of the kernel that the rest is for: keys of a share (a multiple of 32), shares, row packing.  The
  // workspace has room for either; as_run() is the plan of what runs.
  int stream_keys, stream_splits, stream_pad, stream_row_tiles, stream_row_groups;
  bool stream_prefill;
  int tile_group;  // tile-walking prefill: q heads whose rows share a q tile (all of a kv head's, or one)
  int group_pad, row_tiles, row_groups;  // MFMA decode row packing
  int l_block;     // split-KV MFMA kernels with per-adapter low-rank caches: padded rank of one slot's column block, else 0
  // decode of a batch by decode_batch_kernel (batch_wgs > 0, else decode_mfma_kernel): workgroups per (kv head, row group),
  // 128-key tiles of a share to begin with (0: from the lengths on the device) and at least, partial states per row
  int batch_wgs, batch_tiles, batch_min_tiles, batch_splits;
  bool workspace_optional;  // prefill: without room for the plan's workspace the call runs with one share per q tile
  bool launchable;  // false: a grid dimension would exceed the limit of 65535 in y or z (LRA_ERR_UNSUPPORTED)
  size_t off_ml, off_o, off_lr, off_adapter, off_qt, qt_bytes, bytes;
  // rotary prefill with the completed keys in the workspace: their offset and size (0: none), and
  // the size the plan has without them
  size_t off_kc, kc_bytes, bytes_without_kc;
};

lra_status check_common(const lra_shape* sh, const lra_cache* c);
// false: the call is too large for the planner's 32-bit row arithmetic (LRA_ERR_UNSUPPORTED)
bool plan_sizes_fit(const lra_shape* sh, const lra_cache* c, int32_t tokens, int32_t max_queries_per_seq);
// key_adapter: whether the call has a B_K.  lra_workspace_bytes cannot know and plans with one; the plan without one
// never needs more workspace.
Plan make_plan(const lra_shape* sh, const lra_cache* c, int tokens, int max_queries_per_seq, bool prefill,
               const Tuning& tune, bool key_adapter = true);

// The plan with its key shares, row packing and path those of the streaming kernel where that runs.
Plan as_run(const Plan& pl);

// lra_cache_append: parts of d_model the tiled GEMM is divided into (1: none), the token side of its
// tile, and the fp32 workspace the parts need.
struct AppendSplit {
  int k_splits, bt;
  size_t bytes;
};
// Whether tiles of 64 features x 64 tokens run instead (append_quarter_kernel); such a call is not split, whatever the
// split's plan says (what a call is told to bring as workspace does not depend on it).
bool append_quarter_tiles(int n_new, int n_kv_heads, int head_dim, int rank, int d_model, const Tuning& tune);
// Whether the weight-streaming kernel runs in place of the divided GEMM (as above: whatever the split's plan says).
bool append_streams(int n_new, int n_kv_heads, int head_dim, int d_model, const Tuning& tune);
AppendSplit plan_append_split(int n_new, int n_kv_heads, int head_dim, int rank, int d_model, const Tuning& tune);

// Key shares of the streaming kernel's grid where the kv head is its fastest index: the call's, or more, which end at once.
int stream_grid_shares(int n_kv_heads, int n_splits, int row_groups);
// rg_interleave of the split-KV kernel's grid (see there), 0: kv head, key share, (sequence, row group).
int mfma_interleave(int n_kv_heads, int n_splits, int row_groups, bool rotary);

// Kernel that merges the states of `shares` key shares per row: merge_kernel, merge_rows_kernel, merge_wave_kernel, merge_tokens_kernel
// (which has room for kMergeTokenShares).
enum class MergeForm { kColumns, kRows, kWave, kTokens };
constexpr int kMergeTokenShares = 16;
MergeForm merge_form(bool bf16, int head_dim, int rank, int n_q_heads, int n_kv_heads, int shares, bool prefill, int rows);

// Row tiles per workgroup the split-KV MFMA kernels are built for.
int decode_mfma_row_tiles(int rows_needed);
// Agent slots a 16-row tile may hold in the rotary form of the split-KV kernel.
int decode_mfma_rope_slots(int rank);
// Bytes of workspace the Qt pre-pass of the streaming form takes (0: Qt is formed per workgroup).
size_t decode_stream_qt_bytes(int group_pad, int rank, int row_tiles, int row_groups, int n_kv_heads);

}  // namespace lra
