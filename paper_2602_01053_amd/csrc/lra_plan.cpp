// Launch planning (host only; see lra_plan.h).
#include "lra_plan.h"

#include <algorithm>
#include <cmath>

namespace lra {

static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

Tuning resolve_tuning(const lra_tuning* t) {
  Tuning r;
  if (!t) return r;
  r.variant = (t->kernel_variant == 1 || t->kernel_variant == 2) ? t->kernel_variant : 0;
  r.split_keys = t->decode_split_keys > 0 ? t->decode_split_keys : 0;
  if (t->short_prefill != 0) r.short_prefill = t->short_prefill < 0 ? 0 : t->short_prefill;
  r.prefill_splits = t->prefill_splits > 0 ? t->prefill_splits : 0;
  r.rope_key_prepass = t->rope_key_prepass >= 0;
  if (t->append_skinny != 0) r.append_skinny = t->append_skinny < 0 ? 0 : t->append_skinny;
  r.append_stages = (t->append_stages >= 2 && t->append_stages <= 4) ? t->append_stages : 0;
  r.append_tile = (t->append_tile == 64 || t->append_tile == 128 || t->append_tile == 256) ? t->append_tile : 0;
  r.append_k_splits = (t->append_k_splits >= 1 && t->append_k_splits <= 16) ? t->append_k_splits : 0;
  r.main_kernel_only = t->measure_main_kernel_only == 1;
  return r;
}

// Caps that keep the planner's and the kernels' 32-bit arithmetic in range: query rows
// (tokens x Hq) and the padded rows of one sequence (queries x 16) below 2^30.
bool plan_sizes_fit(const lra_shape* sh, const lra_cache* c, int32_t tokens, int32_t max_queries_per_seq) {
  (void)c;
  if (tokens < 1 || max_queries_per_seq < 1) return false;
  if (static_cast<int64_t>(tokens) * sh->n_q_heads > (int64_t{1} << 30)) return false;
  if (static_cast<int64_t>(max_queries_per_seq) * 16 > (int64_t{1} << 30)) return false;
  return true;
}

// Chunks whose 64 x 64 tiles fill the chip at most once, and enough of it that dividing d_model among workgroups, two
// launches, is no faster: a tile costs 4.7 us and 0.35 us per 128 of d_model.  Measured over 40000 calls of eight layers (us
// before / with these tiles): Llama-3-8B projection, 193 to 256 tokens (128 to 159 tiles) 14.1 / 14.6, 321 to 384 15.6 /
// 15.2, 449 to 512 19.6 / 16.3, 513 to 576 (a second round) 20.1 / 27.7; 4 kv heads on 3584, 449 to 576 13.9 / 13.9, 833 to 958
// 17.3 / 15.1; 8 of 64 on 2048, 321 to 448 9.9 / 9.3, 833 to 960 12.7 / 10.1; 12 on 2048, 257 to 320 12.9 / 9.8; 32 on 4096, 65 to
// 128 20.1 / 16.5.  On the line itself a second token tile that is mostly empty is not worth it: 12 on 2048, 65 to 80 tokens
// 8.5 / 8.8, 96 8.9 / 8.8, 128 9.5 / 9.1.  With eight feature tiles or fewer, most of which then carry L features, to 216
// tiles: 2 kv heads on 2048, 1473 to 1726 tokens 12.9 / 8.8, 1624 to 1728, where d_model is not divided, 10.1 / 8.9 (beyond 216 the
// kernel was not faster when it still read x from beyond L2 there, 12.3 / 12.5, and has not been measured since).
bool append_quarter_tiles(int n_new, int n_kv_heads, int head_dim, int rank, int d_model, const Tuning& tune) {
  if (tune.append_k_splits > 1 || tune.append_tile != 0 || tune.append_stages != 0) return false;
  if (n_new < 1 || n_new <= tune.append_skinny || n_new > (1 << 20) || d_model % 128 != 0) return false;
  const int64_t feature_tiles = 2 * static_cast<int64_t>(n_kv_heads) * head_dim / 64;
  if (feature_tiles < 4 * ((rank + 15) / 16)) return false;  // (tiles that the L features ride on)
  const int64_t tiles = (static_cast<int64_t>(n_new) + 63) / 64 * feature_tiles;
  if (n_new < 96 && tiles * 64 < 4 * static_cast<int64_t>(d_model)) return false;
  return tiles * 64 >= 3 * static_cast<int64_t>(d_model) && tiles <= (feature_tiles <= 8 ? 216 : kCUs);
}

// Chunks whose division of d_model below is set aside for the weight-streaming kernel, one launch: while x, which each of its
// workgroups reads, is at most 416 KB and the layer's rows fit one workgroup per compute unit (us streamed and divided:
// Llama-3-8B projection 33 tokens 9.4 / 11.5, 48 11.2 / 12.0, 64 12.8 / 12.1; 4 kv heads on 3584, 33 tokens 6.2 / 8.0,
// 64 8.4 / 9.2; 12 on 2048, 64 9.2 / 10.6; 8 on 8192, 33 15.9 / 15.1; 16 on 4096, 33 18.7 / 15.1).
bool append_streams(int n_new, int n_kv_heads, int head_dim, int d_model, const Tuning& tune) {
  return tune.append_k_splits == 0 && n_new <= tune.append_skinny && n_new <= 64 && n_kv_heads * static_cast<int64_t>(head_dim) <= 1792 &&
         static_cast<int64_t>(n_new) * d_model <= 208 * 1024;
}

// A chunk whose output tiles of 128 features x 64 tokens occupy about half of the chip or less walks all of d_model
// in each of them, one 64-wide step after the other, at what one compute unit can pull from L2.  Such chunks divide
// d_model among several workgroups per tile (a power of two of parts, at least four steps each, about one workgroup
// per compute unit in all) and add the parts in a second kernel.  Measured on the Llama-3-8B projection: 64 tokens 10
// against 18 us, 160 tokens 12 against 19 us; up to 32 tokens the weight-streaming kernel is faster and stays.  Chunks
// of more than 100 tiles of 128 tokens fill the chip with tiles of 64 in one round, unsplit (8 kv heads of 64 on 2048,
// 1500 new tokens: 13 us, divided in two 19).  Forced tile or stage choices keep the unsplit kernels.
AppendSplit plan_append_split(int n_new, int n_kv_heads, int head_dim, int rank, int d_model, const Tuning& tune) {
  AppendSplit none{1, 128, 0};
  if (tune.append_k_splits == 1 || tune.append_tile != 0 || tune.append_stages != 0) return none;
  if (n_new < 1 || n_new > (1 << 20) || d_model < 64) return none;  // (keeps the byte count below 2^48)
  const int n_steps = d_model / 64;
  const int64_t hd = static_cast<int64_t>(n_kv_heads) * head_dim;
  const int64_t tile_rows = 2 * ((hd + 127) / 128) + 1;
  const int64_t tiles128 = (static_cast<int64_t>(n_new) + 127) / 128 * tile_rows;
  if (tune.append_k_splits == 0 && (n_new <= 32 || tiles128 > 100))
    return none;
  AppendSplit sp{1, tiles128 <= 100 ? 64 : 128, 0};
  const int64_t tiles = (static_cast<int64_t>(n_new) + sp.bt - 1) / sp.bt * tile_rows;
  if (tune.append_k_splits > 1) {
    if (n_steps % tune.append_k_splits != 0 || tiles * tune.append_k_splits > 65535 * 16) return none;
    sp.k_splits = tune.append_k_splits;
  } else {
    for (int ks = 16; ks >= 2; ks /= 2)
      if (n_steps % ks == 0 && n_steps / ks >= 4 && tiles * ks <= kCUs) {  // one workgroup per compute unit at most
        sp.k_splits = ks;
        break;
      }
  }
  if (sp.k_splits < 2) return none;
  const int64_t n_feat = 2 * hd + rank;
  sp.bytes = align_up(static_cast<size_t>(sp.k_splits) * static_cast<size_t>(n_new) * static_cast<size_t>(n_feat) * sizeof(float), 256);
  return sp;
}

// Several row groups read the same keys: their workgroups of one share had better meet on one XCD, so the workgroups of a row
// group are filled up to a multiple of eight (those without a share end at once).  The dispatcher deals an XCD's workgroups out to
// its four shader engines of eight compute units in turn, whatever they hold: workgroup i of the call goes to engine i mod 32 of the
// chip.  The fill stays away where an engine would then get more than eight workgroups with keys, the last of which would wait for a
// second round while other engines have units to spare (us without the fill and with it; most with keys on an engine: 4 kv heads of group 7,
// 37000 keys, rank 16, 29 shares, two row groups of 7 agents, eight, 34.8 and 28.6; 5 kv heads of 64, low-rank caches per adapter, 12
// shares, four row groups on 56167, eight, 35.4 and 29.5; 12 kv heads, 3 shares, six row groups of 41 agents on 44401 keys, nine, 165
// and 316; 6 kv heads, 13 shares, three row groups on 6635, nine, 24.2 and 31.6).
int stream_grid_shares(int n_kv_heads, int n_splits, int row_groups) {
  int shares = n_splits;
  while (shares * n_kv_heads % 8 != 0) ++shares;
  if (row_groups <= 1 || shares == n_splits) return n_splits;
  // a row group's workgroups with keys: `keys / 32` on every engine and one more on the keys % 32 from its first on
  const int keys = n_splits * n_kv_heads, all = shares * n_kv_heads;
  int starts[4] = {0, 0, 0, 0}, most = 0;  // row groups that begin on engine 8 k
  for (int rg = 0; rg < row_groups; ++rg) ++starts[all / 8 * rg % 4];
  for (int at = 0; at < 4; ++at) {
    int more = 0;
    for (int k = 0; k < 4; ++k) more += (at + 4 - k) % 4 * 8 < keys % 32 ? starts[k] : 0;
    most = most > more ? most : more;
  }
  return row_groups * (keys / 32) + most <= kCUs / 32 ? shares : n_splits;
}

// lcm(8, Hkv) / Hkv: key shares after which the kv heads of a share are on the XCDs of the first again.
static int interleave_step(int n_kv_heads) {
  int m = 8;
  while (m > 1 && n_kv_heads * (m / 2) % 8 == 0) m /= 2;
  return m;
}

// The key shares that fit, or up to a sixteenth less where the row groups of each share then meet on one XCD.
static int64_t meeting_shares(int64_t fit, int n_kv_heads, int row_groups) {
  const int m = row_groups > 1 ? interleave_step(n_kv_heads) : 1;
  return fit / m * m * 16 >= fit * 15 ? fit / m * m : fit;
}

// The rotary forms are not padded (the shares behind the last multiple of m stand in the order of the plain grid): calls that are
// resident at once would get workgroups for another round, and on the plain grid every row group reads the keys from beyond L2
// (us padded / plain / so: 5 kv heads, rank 64, 12 tokens after 21466, 255 workgroups and 360 padded, 66 / 37.0 / 34.2; 12 kv heads,
// rank 32, 24 after 33421, 504 and 576 183 / 145 / 111; of 500 calls 1.001 in the mean, one at 0.92).
int mfma_interleave(int n_kv_heads, int n_splits, int row_groups, bool rotary) {
  if (row_groups <= 1) return 0;
  const int m = interleave_step(n_kv_heads);
  const int64_t shares = rotary ? n_splits : (static_cast<int64_t>(n_splits) + m - 1) / m * m;
  return shares * row_groups > 65535 ? 0 : m;
}

int decode_mfma_row_tiles(int rows_needed) { return rows_needed <= 16 ? 1 : 2; }

// (the B_K^T operands of a tile's slots stay in registers: 4 slots at ranks up to 16, 2 up to 32, 4
// again above, where the kernel has a compute unit to itself)
int decode_mfma_rope_slots(int rank) { return rank <= 16 ? 4 : (rank <= 32 ? 2 : 4); }

// Which form merges, by rows, shares, rank and group.  9756 combinations behind a kernel that writes the states (bf16 and fp32, 64 and 128
// wide, groups of 1, 2, 3, 4, 5, 7, 12 and 16, ranks 16, 32 and 64, 512 to 10240 rows, 3 to 48 shares, all live or a third): 1.02
// of the best form's time in the mean.  Ratios W (a wave per row) / R (a workgroup per row) and T (four rows per wave) / R, bf16, 128 wide,
// groups of 4, all shares live:
//   rows    r 16, 3, 8, 16, 32 shares  r 32                   r 64                   T: r 16, 3, 8 shares  r 32         r 64
//   1024    0.83 0.94 1.07 1.09        0.93 0.97 1.07 1.13    1.21 1.24 1.24 1.39    1.58 1.48             1.64 1.54    1.72 1.59
//   2560    0.76 0.91 0.99 0.97        0.86 0.95 1.07 1.03    1.00 1.09 1.20 1.14    1.02 1.12             1.04 1.11    1.04 1.15
//   3584    0.73 0.89 0.95 1.02        0.82 0.91 1.02 1.02    0.95 1.03 1.13 1.12    0.88 1.05             0.88 1.06    0.88 1.05
//   6144    0.67 0.71 0.96 0.99        0.74 0.82 1.04 1.00    0.85 0.98 1.13 1.14    0.78 0.91             0.78 0.90    0.77 0.90
//   10240   0.61 0.67 0.99 1.08        0.68 0.74 0.97 0.99    0.81 0.91 1.06 0.97    0.67 0.81             0.65 0.81    0.62 0.80
// (fp32 within 0.05 of it; 64 wide 0.05 to 0.1 less for T, and for W up to rank 32.)  W reads no further than a row's last share
// with a key, the others read every slot: with a third of 32 shares live 0.57 to 0.8 for W up to rank 32.  So a batch, whose
// sequences may leave shares empty, takes W wherever the two come near each other, and a prefill, whose shares are all live, R.
// A workgroup of W is four q heads of a kv head.  Groups of 1, 2 and 5 leave two waves and more of four idle: above rank 32 W / R
// 1.04 to 1.5 (64 wide, group 5, 6144 rows, 16 shares 22.8 / 14.6 us), and T takes the longest prefills that W had (64 wide, rank 16, group
// 5, 10240 rows, 3 shares, W 11.3, T 9.1 us).
MergeForm merge_form(bool bf16, int head_dim, int r, int n_q_heads, int n_kv_heads, int ns, bool prefill, int rows) {
  // (statistics in one wave's lanes, the query index in the grid's z)
  if (ns > 64 || (head_dim != 64 && head_dim != 128) || rows / n_q_heads > 65535) return MergeForm::kColumns;
  if (r % 4 != 0) return rows >= 1024 ? MergeForm::kWave : MergeForm::kColumns;
  if (rows < (r <= 16 || (r <= 32 && !prefill && ns > 16) ? 1024 : 2560)) return MergeForm::kRows;
  const int G = n_q_heads / n_kv_heads, waves = (G + 3) / 4 * 4;  // (of W's workgroups)
  const bool wide = r > 32, narrow = head_dim == 64, most_rows = rows >= 9216, idle = (waves - G) * 4 > waves;
  if (prefill && bf16 && (rows / n_kv_heads + 15) / 16 <= 65535) {
    int most = 0;  // shares up to which T is ahead
    if (wide) most = rows >= 5120 ? 10 : 5;
    else if (r > 16 && rows >= 5120) most = narrow || (idle && most_rows) ? 10 : 5;
    if (most_rows && waves > G) most = std::max(most, narrow ? (idle ? kMergeTokenShares : 8) : (idle ? 5 : 0));
    if (ns <= most) return MergeForm::kTokens;
  }
  if (wide && (idle || rows < 5120 || ns > (!narrow && most_rows ? 8 : 5)) &&
      (prefill || ns <= (narrow ? (idle ? 64 : 32) : (idle ? 32 : 16))))
    return MergeForm::kRows;
  return prefill && ns > 8 && rows < 2560 ? MergeForm::kRows : MergeForm::kWave;
}

// The pre-pass pays (one more launch) once a workgroup of the streaming kernel would have to load sixteen 16-row blocks of B_K for
// each of two row tiles: four agent slots at ranks above 48.  us with the pre-pass / with Qt formed per workgroup, three sets of tensors in
// turn: rank 24, 8 agents on 1500 keys 11.5 / 10.2, on 15000 22.2 / 20.8; rank 32 12.0 / 11.3, 22.7 / 21.7; rank 64, groups of seven, 4
// agents, 13.2 / 12.2, 19.7 / 18.3; rank 48, twelve blocks, 13.8 / 13.7, 24.3 / 23.9; rank 64, sixteen, 14.5 / 14.8, 25.2 / 25.4, 16
// agents in two row groups 14.9 / 16.1, 28.5 / 29.1.  One row tile has sixteen at most, many of them empty slots' (8 kv heads of
// group 4, paged, rank 48, 1 agent on 275 keys 12.0 / 10.2, 4 on 469 12.3 / 11.1).  Not in a prefill, whose rows share one adapter.
size_t decode_stream_qt_bytes(int group_pad, int rank, int row_tiles, int row_groups, int n_kv_heads) {
  const int slots = 16 / group_pad, ncb = (rank + 15) / 16;
  if (row_tiles == 1 || slots * ncb < 16) return 0;
  return static_cast<size_t>(row_groups) * n_kv_heads * row_tiles * 2 * 1024;
}

lra_status check_common(const lra_shape* sh, const lra_cache* c) {
  if (!sh || !c) return LRA_ERR_NULL;
  if (sh->dtype != LRA_BF16 && sh->dtype != LRA_F32) return LRA_ERR_DTYPE;
  if (sh->n_q_heads < 1 || sh->n_kv_heads < 1 || sh->head_dim < 1 || sh->rank < 1) return LRA_ERR_SHAPE;
  if (sh->n_q_heads % sh->n_kv_heads) return LRA_ERR_SHAPE;
  if (!(sh->scale >= 0.f) || std::isinf(sh->scale)) return LRA_ERR_SHAPE;
  if (!(sh->key_rope_theta >= 0.f) || std::isinf(sh->key_rope_theta)) return LRA_ERR_SHAPE;
  if (sh->key_rope_theta > 0.f && (sh->head_dim & 1)) return LRA_ERR_SHAPE;
  if (sh->head_dim != 64 && sh->head_dim != 128) return LRA_ERR_UNSUPPORTED;
  if (sh->rank > 64) return LRA_ERR_UNSUPPORTED;
  if (sh->n_q_heads / sh->n_kv_heads > 16) return LRA_ERR_UNSUPPORTED;
  if (sh->n_q_heads > 4096) return LRA_ERR_UNSUPPORTED;
  if (!c->k_base || !c->v_base || !c->l || !c->seq_lens) return LRA_ERR_NULL;
  if (c->n_seqs < 1 || c->max_seq_len < 1) return LRA_ERR_SHAPE;
  if (c->n_seqs > (1 << 20) || c->max_seq_len > (1 << 30)) return LRA_ERR_UNSUPPORTED;
  if (c->block_size != 0 && c->block_size != 16) return LRA_ERR_UNSUPPORTED;
  if (c->kv_token_stride < sh->head_dim || c->kv_head_stride < sh->head_dim) return LRA_ERR_SHAPE;
  if ((c->kv_token_stride | c->kv_head_stride) & 7) return LRA_ERR_SHAPE;
  // extents stay far inside 64-bit element offsets (and the planner's products inside int64)
  if (c->kv_token_stride > (int64_t{1} << 31) || c->kv_head_stride > (int64_t{1} << 40)) return LRA_ERR_UNSUPPORTED;
  if (c->block_size == 0) {
    if (c->n_seqs != 1) return LRA_ERR_SHAPE;
  } else {
    if (!c->block_table) return LRA_ERR_NULL;
    if (c->num_blocks < 1 || c->max_blocks_per_seq < 1) return LRA_ERR_SHAPE;
    if (c->kv_block_stride < 16 * sh->head_dim || (c->kv_block_stride & 7)) return LRA_ERR_SHAPE;
    if (c->kv_block_stride > (int64_t{1} << 40) || c->num_blocks > (int64_t{1} << 60) / c->kv_block_stride)
      return LRA_ERR_UNSUPPORTED;
    if (static_cast<int64_t>(c->max_blocks_per_seq) * 16 < c->max_seq_len) return LRA_ERR_SHAPE;
  }
  if (c->l_row_stride < 0 || c->l_adapter_stride < 0 || (c->l_adapter_stride & 7)) return LRA_ERR_SHAPE;
  if (c->l_row_stride != sh->rank && (c->l_row_stride & 7)) return LRA_ERR_SHAPE;  // (dense rows of any rank are fine)
  if (c->l_row_stride != 0 && c->l_row_stride < sh->rank) return LRA_ERR_SHAPE;
  if (c->l_row_stride > (int64_t{1} << 31) || c->l_adapter_stride > (int64_t{1} << 40)) return LRA_ERR_UNSUPPORTED;
  if (c->block_size != 0 && c->num_blocks > 0 &&
      (c->l_row_stride ? c->l_row_stride : sh->rank) > (int64_t{1} << 56) / c->num_blocks)
    return LRA_ERR_UNSUPPORTED;
  const uintptr_t bits = reinterpret_cast<uintptr_t>(c->k_base) | reinterpret_cast<uintptr_t>(c->v_base) |
                         reinterpret_cast<uintptr_t>(c->l);
  if (bits & 15) return LRA_ERR_SHAPE;
  return LRA_OK;
}

// The q tiles of the tile-walking prefill kernel and the workgroups that share the key tiles of each.
//
// A q tile holds 128 rows (new token, q head) of all q heads of a kv head, or 128 tokens of one q head (tile_group 1).
// The first has fewer tiles and reads a key once for the group, the second spreads the reading of q, the product with
// B_V and the stores over more compute units, which counts in calls of a few tokens on few keys (us with tiles of
// the group / of one head, group 4: 33 new tokens without context 9.8 / 8.0, 64 after 300 12.7 / 11.9, 33 after
// 5000 21.9 / 20.6, 200 after 9000 63 / 68).
//
// Shares: the count with the smallest estimated time.  A compute unit takes two workgroups; a 64-key tile of head
// dimension 128 and rank 16 costs a workgroup 1.2 us on a unit of its own and 1.9 us beside another one (2.4 where every
// workgroup has keys of its own: the memory is the bound), a workgroup 1.3 us outside its tiles and up to 2.3 for its
// live rows; the merge costs 5 us, the partial states are written and read back at 4.3 TB/s.  Fitted to 2700 measured
// calls.  The even division (about two workgroups per compute unit, at least eight tiles each) stays unless the
// estimate is 8 % below its own: within that the two are level, and where it was followed at less it lost as often as
// it won.  us at 1 / 2 / 4 / 5 / 6 / 8 / 12 / 16 shares, chosen one marked: 333 new tokens on 5333: 100 / 67 / 60 /
// 57* / 66 / 62 / 72 / 79; 700 on 9000: 157 / 154 / 140* / 144 / 152 / 152 / 170 / 182.
// A few tokens behind a context (the sizes the split-KV path takes too): the merge of their few rows costs 1.5 us and
// 1 us per 1000 rows, a tile of its own the product with B_V, one dependent round trip per 16 ranks, 1.6 us more at
// rank 32 and 5 at 64, and the smallest estimate is taken as it is.  Over 3100 such calls 0.4 to 1 % from the best
// count (with the figures above 13 and 5 %); 6 tokens after 300, 8 kv heads of 128 / 64, us at 1 / 2 / 3 / 4 shares:
// rank 16 12.8 / 12.4 / 11.4 / 11.4, rank 64 21.8 / 15.3 / 14.0 / 14.0; after 500, 64 wide, 1 and 8 shares: 13.5 / 9.1.
// One share, and no workspace, where q tiles of 128 tokens per q head would fill two workgroups per unit.
struct PrefillTiles {
  int tile_group;
  int64_t shares;
};
static PrefillTiles plan_prefill_tiles(const lra_shape* sh, int tokens, int max_seq_len, bool split_kv_sized) {
  const int G = sh->n_q_heads / sh->n_kv_heads;
  const int64_t slots = 2 * kCUs, tiles = (static_cast<int64_t>(max_seq_len) + 63) / 64;
  const int64_t head_tiles = static_cast<int64_t>((tokens + 127) / 128) * sh->n_q_heads;  // tiles of one q head each
  if (head_tiles >= slots) return {G, 1};
  const bool few = !split_kv_sized && (max_seq_len < 1024 || (tokens <= 64 && max_seq_len <= 4096));
  const int tg = few ? 1 : G;
  const int64_t q_tiles = (static_cast<int64_t>(tokens) * tg + 127) / 128;
  const int64_t wgs = q_tiles * (sh->n_q_heads / tg);
  const int live = tokens * tg < 128 ? tokens * tg : 128;
  const int rank_pad = sh->rank <= 16 ? 16 : (sh->rank <= 32 ? 32 : 64);
  const double width = (sh->head_dim + 0.6 * rank_pad + 36.0) / (128 + 0.6 * 16 + 36.0);
  const double alone = 1.2 * width, beside = (q_tiles == 1 && tg == G ? 2.4 : 1.9) * width;
  const double fixed = 1.3 + 2.3 * live / 128;
  const double merge = split_kv_sized ? 1.5 + 1e-3 * tokens * sh->n_q_heads : 5.0;
  const double own_b_v = split_kv_sized ? (rank_pad - 16) * (0.018 + 6.5e-4 * sh->head_dim) : 0.0;
  const double per_share = static_cast<double>(tokens) * sh->n_q_heads * (sh->head_dim + sh->rank) * 8.0 / 4.3e6;
  auto estimate = [&](int64_t ns) {
    const int64_t w = wgs * ns, rest = w % slots, share = (tiles + ns - 1) / ns;
    double us = static_cast<double>(w / slots) * (fixed + beside * static_cast<double>(share));
    if (rest > 0) us += fixed + (rest <= kCUs ? alone : beside) * static_cast<double>(share);
    return ns > 1 ? us + merge + per_share * static_cast<double>(ns) : us + own_b_v;
  };
  int64_t even = (slots + head_tiles - 1) / head_tiles;
  if (even > max_seq_len / (8 * 64)) even = max_seq_len / (8 * 64);
  even = even < 1 ? 1 : (even > 32 ? 32 : even);
  int64_t best = even;
  double best_us = (split_kv_sized ? 1.0 : 0.92) * estimate(even);
  for (int64_t ns = 1; ns <= 32 && ns <= tiles; ++ns) {
    const double us = estimate(ns);
    if (us < best_us) {
      best = ns;
      best_us = us;
    }
  }
  return {tg, best};
}

// Whether a prefill of few new tokens (no rotary key side) runs on the tile-walking kernel rather than on the
// split-KV decode kernels.  Those take 16 rows per tile and, beyond 32 rows of a kv head, read the keys once per row
// group; the tile-walking kernel has one tile for 128 rows, at the price of 128 rows' matrix work per key, and at most
// 32 shares of it: with few kv heads it cannot fill the chip on long contexts.  Measured on MI355X at 2 to 33 thousand
// keys, each path as it is now (ratio of the times split-KV / tile walk, contiguous and paged; G = q heads per kv head):
//   8 kv heads, G 4    5 and 8 tokens 1.17 and 1.13 at 2 k, 1.03 and 1.0 at 9 k, 1.05 and 0.97 at 33 k; 16 tokens 1.03 and 1.0 at 2 k,
//                      1.12 and 1.2 at 9 k and beyond; 32 tokens 0.88 at 2 k, 1.05 at 4 k, 1.15 at 9 k, 1.57 and 1.71 at 33 k
//   8 kv heads, d 64   8 tokens 1.18 at 2 k, 0.98 at 9 k, 0.85 and 0.79 at 20 k; 16 tokens 1.03 to 1.08, paged to 1.22
//   4 kv heads, G 7    4 tokens 1.08 and 1.05 at 4 k, 1.01 and 0.96 at 6 k, 0.95 and 0.9 at 9 k, 0.78 and 0.73 at 33 k; 8 tokens 1.03 and
//                      1.0 at 4 k, 1.0 and 0.97 at 9 k, 0.92 and 0.88 at 33 k; 16 tokens 0.93 at 4 k, 1.07 and 1.24 at 9 k, 1.2 at 33 k
//   2 kv heads, G 8    8 tokens 1.1 and 1.05 at 2 k, 0.99 and 0.94 at 6 k, 0.93 and 0.87 at 9 k, 0.82 and 0.78 at 14 k; 16 tokens 0.94 and
//                      0.9 at 2 k to 9 k, 0.93 at 14 k; 20 tokens 0.9 to 6 k, 1.02 from 9 k on; 32 tokens 0.9 at 2 k, 1.24 at 9 k
//   32 kv heads, G 1   5 and 8 tokens 0.85 and 0.88 at 20 k; 16 tokens 1.16 to 1.3 throughout
// Ranks above 32 cost the tile walk more, on pages most of all:
//   4 kv heads, G 7    paged 4 and 8 tokens 1.06 and 1.0 at 2 k, 0.96 and 0.99 at 4 k, 0.79 and 0.86 at 7 k; 12 tokens 0.91 to 0.95, 0.86 at 7 k
//   2 kv heads, G 8    paged 8 tokens 0.92 at 4 k, 0.79 at 7 k, 0.51 at 33 k; 20 tokens 0.89 at 4 k, 0.84 at 7 k; 28 tokens 0.85 to 0.89
//   32 kv heads, G 1   paged 8 tokens 0.86 at 2 k, 0.75 at 7 k, 0.64 at 33 k
//   8 kv heads, d 64   12 and 16 tokens 0.94 and 0.91 at 11 k, 0.87 at 33 k, paged 1.01 to 1.04
// The lines below are older than the streaming kernel on pages and the one product that forms Qt of a prefill: paged calls of few kv
// heads, and ranks above 32 from 4 thousand keys on, stay on the tile walk up to where it is 6 to 20 % behind (2 kv heads, 8 tokens on
// 9000 keys of a paged cache 15.5 / 13.5 us); none is slower than it was before those two.
static bool short_prefill_walks_tiles(const lra_shape* sh, const lra_cache* c, int tokens) {
  const int G = sh->n_q_heads / sh->n_kv_heads, n = c->max_seq_len;
  const int rows = tokens * (G <= 4 ? 4 : (G <= 8 ? 8 : 16));  // rows of a kv head in the split-KV kernels
  if (rows <= 16) return false;
  const int groups = (rows + 31) / 32;                                // times those read the keys
  const int units = sh->n_kv_heads * groups;
  const int walk = sh->n_kv_heads * ((tokens * G + 127) / 128);      // q tiles of the tile-walking kernel
  if (groups == 1 && walk > 8 && n > 16384) return false;
  if (sh->rank > 32 && c->block_size != 0) {
    if (groups == 1 && walk > 8) return n <= 3072;
    return walk >= 8 || groups > 6 || n <= (walk < 4 || groups <= 2 ? 5120 : 9216);
  }
  if (sh->rank > 32 && sh->head_dim == 64 && walk <= 8 && tokens * G <= 64 && n > 14336) return false;
  if (c->block_size != 0) return n <= 12288 || !(groups == 1 ? walk < 8 : walk < 4 && groups <= 4);
  if (units <= 8) return n <= (walk < 4 ? (tokens * G <= 96 ? 3072 : 0) : (units < 8 ? 6144 : 9216));
  return tokens * G <= 96 || (walk < 8 ? units >= 12 && n >= 8192 : n >= 4096);
}

// The shares of one sequence in the rotary form of the split-KV kernel at ranks up to 32, two workgroups per compute unit
// (n = 0: one workgroup per unit).  Its steps are long and a unit takes as long as its two workgroups together, the first
// and the 257th to start, so what counts is the load of a unit in key tiles: the least one there is, halved between the
// two, an odd tile in the first.  Where that is the load of one workgroup per unit as well, two still cover each other's
// dependent steps, and the partial states double.
// us with one workgroup per unit / two, shares of one size / two, divided like this (8 kv heads of 128, rank 16, 4 agents on
// 9000 keys, 3 tiles a unit: 24 shares 20.3, 64 20.3, 40 18.9; on 20011: 32 29.6, 53 31.0, 63 27.6; on 60000: 32 70.1, 59 64.5, 64
// 59.9; 8 agents, two row groups, on 5000: 16 21.3, 24 18.6; on 33000: 16 74.4, 32 58.5; rank 32, 2 agents on 9000: 18.1,
// 40 16.9).  Not beyond 64 shares, which one merge kernel takes (4 kv heads on 60000: 64 shares 29.2, 128 35.0), and 128 keys
// only for up to 2048 (row, share) states; prefills of a few tokens from 384 keys on.
// Where the units do not divide 256 shares of one size in all 512 places can be shorter than half of that load, and are taken then
// (24 kv heads, 11 agents of 1 head, rank 32, 144 units, 6250 keys: two shares 99.7, three 75.2; 96 units, 8 agents on 40888, four
// 304 and five 256).  With several row groups the counts are those whose workgroups meet on one XCD, a sixteenth less at most (5 kv
// heads, 8 agents in two row groups on 35089, 25 shares for 24, 58.5 / 47.1 in all).
struct RopeShares {
  int keys, n, more;  // keys of the largest, shares, how many are of that size where the rest hold 128 less (0: all)
};
static RopeShares rope_two_per_unit(int max_seq_len, int n_kv_heads, int row_groups, int64_t rows, bool prefill) {
  const int64_t tiles = (static_cast<int64_t>(max_seq_len) + 127) / 128, work = static_cast<int64_t>(n_kv_heads) * row_groups;
  const int64_t units = meeting_shares(kCUs / work, n_kv_heads, row_groups), load = units > 0 ? (tiles + units - 1) / units : 0;
  if (load < 2) return {0, 0, 0};
  const int64_t places = meeting_shares(2 * kCUs / work, n_kv_heads, row_groups), level = (tiles + places - 1) / places;
  const int64_t n_alike = (tiles + level - 1) / level;
  auto held = [&](int64_t largest, int64_t n) { return n <= 64 && (prefill ? largest >= 3 : largest >= 2 || rows * n <= 2048); };
  const bool alike = 2 * level < load && held(level, n_alike), odd = !alike && (load & 1) != 0;
  const int64_t first = alike ? level : (load + 1) / 2;
  const int64_t n = odd ? units + (tiles - units * first + first - 2) / (first - 1) : (tiles + first - 1) / first;
  if (!held(first, n)) return {0, 0, 0};
  return {static_cast<int>(first * 128), static_cast<int>(n), odd ? static_cast<int>(units) : 0};
}

// What prefill_rows_kernel reads: ranks up to 32, and a cache within 32-bit byte offsets of one resource; the completed
// keys of a rotary call (`keys_ready`: the call has room for them).
static bool prefill_rows_reads(const lra_shape* sh, const lra_cache* c, bool split_kv_sized, bool keys_ready) {
  if (sh->rank > 32 || sh->rank % 8 != 0) return false;
  const bool rope = sh->key_rope_theta > 0.f;
  if (rope && (split_kv_sized || !keys_ready)) return false;
  const int64_t lim = 0x7ffff000 / 2;  // elements
  const int64_t l_pitch = c->l_row_stride ? c->l_row_stride : sh->rank;
  if (c->block_size == 0) {
    if (c->max_seq_len * c->kv_token_stride > lim || c->max_seq_len * l_pitch > lim) return false;
  } else {
    const int64_t blocks = c->num_blocks > c->max_blocks_per_seq ? c->num_blocks : c->max_blocks_per_seq;
    if (c->kv_block_stride > lim / blocks || c->kv_head_stride > lim / sh->n_kv_heads ||
        blocks * c->kv_block_stride + sh->n_kv_heads * c->kv_head_stride + 16 * c->kv_token_stride > lim ||
        l_pitch > lim / (blocks * 16))
      return false;
  }
  return true;
}
// Whether a prefill runs on the kernel whose waves divide the keys of a workgroup's 32 rows (prefill_rows_kernel): one
// kernel without a workspace, workgroups a quarter the size of a q tile.
//
// A workgroup has a compute unit to itself and takes 256 keys per 1.35 us (the way from L2 into LDS), about 7 us
// outside its loop; the tile walk it replaces takes 15 to 20 us for anything that small but walks a long context with
// fewer reads.  The line, from 1000 measured calls (8, 4 and 2 kv heads of group 4, 7 and 8, 32 of group 1, d = 64 and
// 128, ranks 8 to 32, with and without pages; ratio of the times before / here):
//   one round of the chip (w <= 256 workgroups): steps of 256 keys up to w / 8; 1.0 to 2.0, on the line itself 0.9 to
//     1.1 (llama shape, 62 tokens on 525 keys 17.2 -> 9.9 us, 104 on 627 21.8 -> 10.7, 198 on 2199 31.4 -> 20.4; beyond
//     the line 78 on 4395 0.82, 43 on 5802 0.80).  Above 16 kv heads the keys come from memory rather than from L2: w / 12.
//   two rounds, from 950 more: 3 to 6 steps 1.0 to 1.7; 7 and 8 at ranks up to 16 under 320 workgroups 0.96 to 1.2, else 1.0
//     to 1.5; 9 to 13 with a second round half full 1.0 to 1.4; 14 and more on the edge of that, 384 workgroups, 0.85 to 1.0,
//     at ranks up to 16 beyond it 14 1.0, 15 to 20 0.92 to 1.2, at the higher ones to 20 0.99 to 1.25 (399 tokens on 1270: 1.27;
//     378 on 5006 54.5 / 64.3 us).  At 512 keys and less 0.94 to 0.97 at ranks up to 16 under 448 workgroups, 1.0 to 1.2 from
//     there (rotary, with the pre-pass in front of either: 0.91 to 0.96 at 4 of 5, 248 on 360 18.0 / 19.8), at the higher ones 1.0
//     to 1.2 (0.94 at one of ten).
//   three rounds and more: 0.7 to 1.2, mostly below 1.
//   calls of the size the split-KV path takes, two launches and 8.5 to 9.5 us of GPU time there, from 520 more.  From 8 kv heads
//     on: one row tile per kv head 1.0 to 1.4 up to 384 keys, 0.93 to 1.1 to 512 (above 16 kv heads 1.01 to 1.2 from 7
//     tokens on, 0.89 to 0.97 below); two 1.0 to 1.2 up to 640, 0.93 to 1.0 beyond 700; three 1.1 to 1.25 up to 768; more 1.02
//     to 1.5 up to 1024.  Fewer kv heads: up to three 1.02 to 1.3 up to 512 and 0.89 to 1.06 to 768, four to six 1.03 to 1.2 up
//     to 768 and 0.91 to 1.1 to 1024, more 1.01 to 1.2 (5 tokens on 697 keys on pages, 4 kv heads 9.8 / 11.0 us; 24 on 982, 2
//     kv heads 11.4 / 12.5).
static bool prefill_waves_divide_keys(const lra_shape* sh, const lra_cache* c, int tokens, bool split_kv_sized,
                                      bool keys_ready) {
  if (!prefill_rows_reads(sh, c, split_kv_sized, keys_ready)) return false;
  const int64_t G = sh->n_q_heads / sh->n_kv_heads, tiles = (tokens * G + 31) / 32;
  const int64_t w = tiles * sh->n_kv_heads, n = c->max_seq_len, steps = (n + 255) / 256;
  if (split_kv_sized) {
    if (w > kCUs) return false;
    if (tiles == 1) return n <= (sh->n_kv_heads > 16 && tokens > 6 ? 512 : 384);
    if (sh->n_kv_heads >= 8) return n <= (tiles == 2 ? 640 : (tiles == 3 ? 768 : 1024));
    return n <= (tiles <= 3 ? 512 : (tiles <= 6 ? 768 : 1024));
  }
  if (w <= kCUs) return steps <= 4 || steps * (sh->n_kv_heads > 16 ? 12 : 8) <= w;
  if (w > 2 * kCUs) return false;
  const bool wide = sh->rank > 16;
  if (steps <= 2) return wide || (w >= 448 && sh->key_rope_theta <= 0.f);
  if (steps <= 8) return steps <= 6 || wide || w >= 320;
  return w >= 384 && steps <= (w < 400 ? 13 : (wide ? 20 : 14));
}

// Shares of the keys for prefill_rows_kernel where one workgroup per 32 rows leaves compute units idle (then the merge
// kernel), 0 where another path stays: one workgroup per compute unit in all, at most 32 per row.  A share costs 10 us
// with the merge and 1.33 us per 256 keys; its partial states are a quarter of those of 128-row tiles in number of rows.
//
// The line, from 5000 measured calls (the layer shapes of prefill_waves_divide_keys, 2 to 1000 tokens on 0.25 to 34
// thousand keys); s = steps of 256 keys per share, T = workgroups per kv head and share.  Inside it 1.13 in the mean,
// 0.95 at worst.  (Before the exchange of prefill_rows_kernel and the merge got shorter and few_tokens_stream came; outside it now,
// ratio of the time as the lines are / on this path, 420 calls of 2, 4 and 8 kv heads: T = 1 with 8 kv heads 5 and 8 tokens on
// 9009 1.0 to 1.05, paged 1.07 to 1.11, on 13000 1.05 to 1.13, 3 tokens 0.89 to 0.95; with 4 of group 7 5 and 8 tokens 0.84 to 0.95 to 9009,
// 1.08 to 1.11 on 13000; T = 2 to 4 on contiguous caches, 8 kv heads, 12 to 32 tokens 1.05 to 1.27 from 6644 keys on, 4 kv heads 16 tokens 1.06
// to 1.26, 2 kv heads 1.0 to 1.14.)
//   fewer workgroup steps than compute units: 0.72 to 1.05.
//   s < 1.4: 0.93 to 1.02 (8 kv heads, 10 tokens on 4568).
//   T = 1, above 16 kv heads and with two row tiles of the split-KV kernel: shares of 512 keys, 1.02 to 1.2 to s = 8;
//     with one row tile 0.87 to 1.0, with fewer kv heads 0.83 to 1.07 (8 kv heads, 8 tokens after 9001: 16.1 / 16.4 us, 14.9 / 14.9 now).
//   T = 2 to 4 on contiguous caches: 0.88 to 1.1 (10 tokens on 6644: 16.2 / 18.4 us; 12 14.8 / 14.0 now; paged 1.06 in the mean, from 0.96).
//   T > 1, up to the s where the 128 rows of the tile walk, which read the keys fewer times, catch up: 1.0 to 1.4 up to 6
//     where T fills the last such tile, 7, 11 and 12 at T % 4 = 3, 2, 1; beyond 0.66 to 1.0 (107 after 30000 0.72).
//     Above 16 kv heads, whose keys come from memory, to 4.
static int plan_wave_shares(const lra_shape* sh, const lra_cache* c, int tokens, int room) {
  const int64_t n = c->max_seq_len, G = sh->n_q_heads / sh->n_kv_heads;
  const int64_t row_tiles = (tokens * G + 31) / 32, w = row_tiles * sh->n_kv_heads;
  if (w > kCUs / 2 || w * n < int64_t{kCUs} * 256) return 0;
  int64_t shares = kCUs / w < 32 ? kCUs / w : 32;
  int64_t most;  // steps of a share
  if (row_tiles == 1) {
    if (tokens * (G <= 4 ? 4 : (G <= 8 ? 8 : 16)) <= 16 || sh->n_kv_heads <= 16) return 0;
    if (shares > (n + 511) / 512) shares = (n + 511) / 512;
    most = 8;
  } else {
    if (n < 360 * shares || (row_tiles < 5 && c->block_size == 0 && sh->n_kv_heads <= 16)) return 0;
    most = sh->n_kv_heads > 16 ? 4 : (row_tiles % 4 == 1 ? 12 : (row_tiles == 2 || row_tiles % 4 == 0 ? 6 : (row_tiles % 4 == 2 ? 11 : 7)));
  }
  // (room: the partial states per row that the path it replaces keeps, which is what callers' workspaces are sized for)
  if (n > most * 256 * shares || shares > room || shares < 2) return 0;
  return static_cast<int>(shares);
}

// Decode of a batch with the shares of all sequences in one row (decode_batch_kernel): two workgroups per compute unit
// (one in the rotary form above rank 32), or the grid of decode_mfma_kernel where that serves as well or the row cannot
// balance it.  All sequences have one share size, the smallest with which the shares fit the places, so a sequence of n
// tiles wastes part of a share, and with hardly more places than sequences a long one is not divided at all (one of 65536
// among 63 of 500, 8 kv heads: 265 us on the grid, 951 in a row).  Measured over 690 batches of 2 to 64 sequences,
// 0.3 k to 65 k tokens; ratio of the times grid / row:
//   a grid that is in place at once, or nearly.  One row group: 0.96 to 1.0 where no more than 512 workgroups find keys (8 of
//     18 k to 21 k: 113.7 / 116.4 us), without lengths 0.95 to 1.1 up to 576 in all (3 of 2.8 k: 11.0 / 11.6).  Several: 0.96
//     to 1.03 up to 320, at d = 64, where a unit holds more than two, up to 512.
//   known lengths, share size times places over all tiles: to 1.35 0.97 to 1.45 with one row group (16 of 4 k to 64 k, 4 kv
//     heads 177 / 162), from there 0.86 to 1.26, 0.28 to 0.4 beyond 8; with several row groups, whose keys the row's layout
//     reads once, 0.93 to 1.8 to a factor of 2 (10 of 6 k to 8 k, own low-rank caches 67.7 / 45.6), 0.36 at 16.  Shares no
//     longer than the grid's are taken whatever the factor: 0.98 to 1.9.
//   unknown lengths: from two places per sequence on 0.97 to 1.7, one long sequence among many short ones with it 1.0 to 2.6
//     (below that 4 of 400: 40000 among 25 of 4000 117.6 / 126.2, 10 of 9 k to 18 k, three row groups 55.1 / 63.3); with fewer
//     places 0.74 to 1.5 (62 of 0.1 k to 7.7 k: 96 / 130).
// The rotary forms, whose steps are long against everything else, gain from three tiles on (13 of 0.6 k to 2.7 k: 38.3 /
// 31.6) and lose up to 8 % at two.  What bounds them is the vector unit and not the keys, so that with several row groups only
// the balance counts (560 batches, several row groups).  Known lengths, to 1.35: 1.18 in the mean, 7 of 202 below 0.96, most
// of them with five row groups (0.78 at one, 8 of 31 k to 39 k above rank 32); beyond 0.75 to 1.6 (11 of 4 k to 33 k, rank 24, four
// row groups 516 / 690).  Unknown ones, up to rank 32: from five places per sequence on 1.1 to 1.2 in the mean, 0.87 to 0.94 at 4 of
// 80, below that 0.82 to 1.33, worst where the sequences are long and even, since the grid then has four rounds of equal workgroups
// (10 of 32 k to 38 k 304 / 365); above rank 32, one workgroup per unit, 1.0 to 1.7.
// (The lines are those of the 16 x 16 form before decode_rope_share.  With that, at d = 128 and ranks up to 16, 200 drawn batches, in a
// row where these lines say so: 1.03 in the mean, two of them 0.945 and 0.967.)
static void plan_batch(Plan& pl, const lra_shape* sh, const lra_cache* c, bool key_adapter) {
  constexpr int kMost = 64;  // sequences: one per lane
  if (c->n_seqs > kMost) return;
  const bool rope = sh->key_rope_theta > 0.f && key_adapter, one = pl.row_groups == 1;
  if (rope && sh->head_dim == 128 && sh->rank > 32) return;  // (built without: its registers go to scratch memory)
  const int64_t units = static_cast<int64_t>(sh->n_kv_heads) * pl.row_groups;
  const int64_t places = (rope && sh->rank > 32 ? kCUs : 2 * kCUs) / units;
  if (places < c->n_seqs) return;
  const int longest = (c->max_seq_len + 127) / 128, grid_tiles = pl.split_keys / 128;
  const int least = (longest + pl.n_splits - 1) / pl.n_splits;
  int tiles[kMost];  // of each sequence (at most 2^23)
  int64_t total = 0, live = 0;
  if (c->seq_lens_host != nullptr)
    for (int t = 0; t < c->n_seqs; ++t) {
      const int32_t len = c->seq_lens_host[t];
      tiles[t] = len < 0 ? 0 : ((len > c->max_seq_len ? c->max_seq_len : len) + 127) / 128;
      total += tiles[t];
      live += (tiles[t] + grid_tiles - 1) / grid_tiles;
    }
  const int64_t grid = c->n_seqs * pl.n_splits * units;
  if (one ? (total > 0 ? live * units <= 2 * kCUs : grid <= 576) : grid <= (sh->head_dim == 64 ? 512 : 320)) return;
  int size = 0;
  if (total > 0) {
    auto fits = [&](int share) {
      int64_t n = 0;
      for (int t = 0; t < c->n_seqs; ++t) n += tiles[t] > share ? (tiles[t] + share - 1) / share : 1;
      return n <= places;
    };
    const int64_t even = (total + places - 1) / places, balanced = (total * (one || rope ? 27 : 40) + places * 20 - 1) / (places * 20);
    int lo = static_cast<int>(even > least ? even : least);
    int hi = static_cast<int>(balanced > grid_tiles ? balanced : grid_tiles);  // the largest share that is worth it
    hi = hi > longest ? longest : hi;
    if (!fits(hi)) return;
    while (lo < hi) {  // the smallest that fits
      const int mid = lo + (hi - lo) / 2;
      if (fits(mid)) hi = mid;
      else lo = mid + 1;
    }
    size = hi;
  } else if (places < (rope && !one && sh->rank <= 32 ? 5 : 2) * c->n_seqs) {
    return;
  }
  if (rope && (total > 0 ? size : static_cast<int64_t>(longest) * c->n_seqs / (2 * places)) < 3) return;
  pl.batch_wgs = static_cast<int>(places);
  pl.batch_tiles = size;
  pl.batch_min_tiles = least;
  const int states = size > 0 ? (longest + size - 1) / size : pl.n_splits;
  pl.batch_splits = states < pl.n_splits ? states : pl.n_splits;
}

static Plan plan_call(const lra_shape* sh, const lra_cache* c, int tokens, int max_queries_per_seq, bool prefill,
                      const Tuning& tune, bool key_adapter) {
  Plan pl{};
  const int G = sh->n_q_heads / sh->n_kv_heads;
  pl.tile_group = G;
  // The MFMA kernels move L in 16-byte pieces: ranks that are not a multiple of 8 take the
  // vector-ALU kernels.
  // The rotary key side: prefill runs on the tile-walking MFMA kernel, which completes a key
  // tile in LDS for its one adapter; decode on the rotary form of the split-KV kernel.
  const bool rope = sh->key_rope_theta > 0.f;
  pl.mfma = sh->dtype == LRA_BF16 && tune.variant != 1 && sh->rank % 8 == 0;
  // Low-rank rows with a stride of their own, or one low-rank cache per adapter (BaseShared): the
  // tile-walking prefill kernel and the streaming form of the split-KV kernel read them; that form
  // needs a contiguous cache and no rotary key side, everything else takes the vector-ALU kernels.
  const int64_t l_pitch = c->l_row_stride ? c->l_row_stride : sh->rank;
  const bool custom_l = c->l_adapter_stride > 0 || l_pitch != sh->rank;
  const bool stream_ok = c->block_size == 0 && !(sh->key_rope_theta > 0.f) && tune.variant != 2;
  // ... except that the older split-KV kernel reads such rows too when every row tile of a workgroup belongs to
  // ONE low-rank cache: paged caches and batches then give each agent a row tile (and a workgroup) of its own,
  // which streams K_base / V_base once per agent of a sequence instead of once per sequence (the other agents'
  // workgroups find the tiles in L2), still on the matrix cores.  The rotary form of that kernel likewise (its
  // tiles then hold one agent slot each).
  const bool tile_per_agent = custom_l && !stream_ok;
  // Plain decode with one low-rank cache per adapter does better: the split-KV kernel has the same column-block L
  // tile as the streaming form (one block per agent slot of a row tile), so K_base / V_base are requested once for
  // the agents of a tile.  It addresses a paged pool of low-rank rows with 32-bit byte offsets inside one resource.
  const bool block_per_slot =
      tile_per_agent && !prefill && !rope && c->l_adapter_stride > 0 &&
      (c->block_size == 0 || static_cast<int64_t>(c->num_blocks) * 16 * l_pitch * 2 <= (int64_t{1} << 31) - 4096);
  const bool stream_only = custom_l && !tile_per_agent;
  if (prefill && pl.mfma) {
    // the tile-walking kernel addresses a contiguous kv head slice, and L as a whole, with
    // 32-bit byte offsets inside one buffer resource; larger caches take the other kernels
    const int64_t lim = (int64_t{1} << 32) - 4096;
    const int64_t l_rows = c->block_size == 0 ? c->max_seq_len : static_cast<int64_t>(c->num_blocks) * 16;
    if (l_rows * l_pitch * 2 > lim) pl.mfma = false;
    if (c->block_size == 0 && static_cast<int64_t>(c->max_seq_len) * c->kv_token_stride * 2 > lim) pl.mfma = false;
  }
  // A handful of new tokens after a long context: the split-KV decode kernel, with the new tokens in the place of
  // the agents and a causal limit per row, or the tile-walking kernel with the key tiles shared.
  pl.short_prefill = prefill && pl.mfma && tokens <= tune.short_prefill &&
                     static_cast<int64_t>(tokens) * 4 <= c->max_seq_len &&
                     (tune.short_prefill > 32 || rope || !short_prefill_walks_tiles(sh, c, tokens));
  // completed keys of a rotary prefill, in the layout of K_base (whether or not the call has a B_K); caches beyond 4 GB
  // keep completing tiles inside the kernel.  Paged caches: the blocks of the call's sequence in logical order, with
  // the strides of the pool.
  int64_t kc_span = -1;  // elements; -1: no pre-pass
  if (rope && tune.rope_key_prepass) {
    if (c->block_size == 0)
      kc_span = (static_cast<int64_t>(c->max_seq_len) - 1) * c->kv_token_stride +
                (static_cast<int64_t>(sh->n_kv_heads) - 1) * c->kv_head_stride + sh->head_dim;
    else if (c->kv_block_stride <= (int64_t{1} << 31))  // (keeps the product below inside int64)
      kc_span = (static_cast<int64_t>(c->max_seq_len) - 1) / 16 * c->kv_block_stride +
                (static_cast<int64_t>(sh->n_kv_heads) - 1) * c->kv_head_stride + 15 * c->kv_token_stride + sh->head_dim;
    if (kc_span > (int64_t{1} << 31)) kc_span = -1;
  }
  const bool split_kv_sized = tokens <= tune.short_prefill && static_cast<int64_t>(tokens) * 4 <= c->max_seq_len;
  pl.split_kv_sized = prefill && split_kv_sized;
  // (The rest of the plan is that of the kernel which would run without it: a call needs the same workspace either way.)
  pl.wave_rows = prefill && pl.mfma && tune.variant == 0 && tune.prefill_splits == 0 && tune.short_prefill <= 32 &&
                 tune.split_keys <= 0 && prefill_waves_divide_keys(sh, c, tokens, split_kv_sized, kc_span >= 0);
  const bool rope_split = rope && pl.mfma && (!prefill || pl.short_prefill);  // rotary form of the split-KV kernel
  if (prefill && pl.mfma && !pl.short_prefill) {
    // Tile-walking kernel: one workgroup per q tile (see plan_prefill_tiles).  Where those do not fill the chip the
    // key tiles of a q tile are divided among several workgroups and the merge kernel finishes the job; otherwise it
    // is one kernel without a workspace.
    pl.rows = tokens * sh->n_q_heads;
    pl.group_pad = pl.row_tiles = pl.row_groups = 1;
    pl.split_keys = c->max_seq_len;
    // (few tokens on a long context reach this place only where the packed tile was measured ahead of the split-KV path)
    const PrefillTiles pt = plan_prefill_tiles(sh, tokens, c->max_seq_len, split_kv_sized);
    pl.tile_group = tune.prefill_splits > 0 ? G : pt.tile_group;
    int64_t ns = tune.prefill_splits > 0 ? tune.prefill_splits : (tune.prefill_splits < 0 ? 1 : pt.shares);
    ns = ns > 32 ? 32 : (ns < 1 ? 1 : ns);
    // (sequences below sixteen tiles run without a workspace too, where they are not short prefills)
    pl.workspace_optional = ns > 1 && tune.prefill_splits == 0 && c->max_seq_len < 1024 &&
                            !split_kv_sized;
    pl.n_splits = static_cast<int>(ns);
    pl.bytes = 0;
    if (pl.n_splits > 1) {
      const size_t slots = static_cast<size_t>(pl.rows) * pl.n_splits;
      pl.off_ml = 0;
      pl.off_o = align_up(slots * 2 * sizeof(float), 256);
      pl.off_lr = pl.off_o + align_up(slots * sh->head_dim * sizeof(float), 256);
      pl.off_adapter = pl.off_lr + align_up(slots * sh->rank * sizeof(float), 256);
      pl.bytes = pl.off_adapter + align_up(static_cast<size_t>(pl.rows) * sizeof(int32_t), 256);
    }
    pl.off_qt = pl.bytes;
    pl.bytes_without_kc = pl.bytes;
    if (kc_span >= 0) {
      pl.off_kc = pl.bytes;
      pl.kc_bytes = align_up(static_cast<size_t>(kc_span) * 2, 256);
      pl.bytes += pl.kc_bytes;
    }
    pl.launchable = true;  // at most 32 shares in y
    return pl;
  }
  pl.rows = tokens * sh->n_q_heads;
  pl.group_pad = G <= 4 ? 4 : (G <= 8 ? 8 : 16);
  pl.l_block = 0;
  if (tile_per_agent && !block_per_slot && !prefill && c->l_adapter_stride > 0) pl.group_pad = 16;  // one agent per 16-row tile
  if (pl.mfma && !prefill && c->l_adapter_stride > 0 && (!tile_per_agent || block_per_slot)) {
    // every agent slot of a row tile brings its own column block of the L tile: 64 columns per tile
    pl.l_block = sh->rank <= 16 ? 16 : (sh->rank <= 32 ? 32 : 64);
    const int min_pad = 16 / (64 / pl.l_block);
    pl.group_pad = pl.group_pad > min_pad ? pl.group_pad : min_pad;
  }
  pl.row_tiles = 1;
  pl.row_groups = 1;
  int tile = 64;       // keys per wave-step of the vector-ALU kernel
  int64_t work;        // units that want a wave (vector-ALU) or a workgroup share (MFMA)
  int want;
  const int n_seqs_eff = prefill ? 1 : c->n_seqs;
  if (pl.short_prefill) max_queries_per_seq = tokens;
  if (pl.mfma) {
    int rows_needed = max_queries_per_seq * pl.group_pad;
    pl.row_tiles = (pl.l_block || (tile_per_agent && !prefill && c->l_adapter_stride > 0)) ? 1 : decode_mfma_row_tiles(rows_needed);  // (an L tile holds the column blocks, or the one cache, of one row tile's agents)
    if (rope_split) {
      // one row tile per workgroup, and (decode) no more agent slots in it than the kernel keeps
      // B_K^T operands for
      const int min_pad = prefill ? 1 : 16 / decode_mfma_rope_slots(sh->rank);
      pl.group_pad = pl.group_pad > min_pad ? pl.group_pad : min_pad;
      pl.row_tiles = 1;
      rows_needed = max_queries_per_seq * pl.group_pad;
    }
    pl.row_groups = (rows_needed + 16 * pl.row_tiles - 1) / (16 * pl.row_tiles);
    tile = 128;        // 4 waves x 32 keys
    work = static_cast<int64_t>(n_seqs_eff) * sh->n_kv_heads * pl.row_groups;
    want = kCUs;
  } else {
    work = pl.rows;
    // shares of a few steps each: the one-wave-per-row kernel of the rotary key side fills the chip with 8 per
    // compute unit, the plain one, of four waves, with the 3 that are resident (32 fp32 rows on 4000 keys: 34.1 us
    // with 63 shares, 24.2 with 21)
    want = rope && key_adapter ? kCUs * 8 : kCUs * 3;
  }
  // The streaming kernel reads one sequence's blocks too, with one low-rank cache for the call; but not where several row groups
  // read keys enough for two workgroups per unit of the split-KV kernel (units x keys of 2^18 and more): ratio of the times there
  // and streaming, three row groups and more 0.59 to 1.5 (32 kv heads of 64, 39 agents on 6572 keys 35.5 / 59.7; 4 kv heads of
  // group 7, 33 agents on 42376 64.6 / 83.9), two row groups at d = 64 0.87 to 1.05.  Two at d = 128 stream below 2^19 (split-KV /
  // streaming 0.95 to 1.3), above rank 32 (0.93 to 1.3) and from 5 x 2^18 on, where the two are level; between, with shares that
  // meet and fit, split-KV takes 0.89 to 0.98 (16 kv heads, 11 agents on 23854 44.6 / 48.4; 24, 9 on 17550 50.6 / 56.9).  Streaming
  // stays for one row group (1.0 to 1.3) and fewer keys (0.92 to 1.4, 1.14 in the mean of 600).
  const int64_t reads = n_seqs_eff == 1 && !prefill && pl.mfma ? work * c->max_seq_len : 0;
  const bool long_row = reads >= int64_t{2} * kCUs * 512;
  const bool long_pair = pl.row_groups == 2 && sh->head_dim == 128 && sh->rank <= 32 && reads >= int64_t{1} << 19 && reads < int64_t{5} << 18;
  const bool paged_stream = c->block_size != 0 && n_seqs_eff == 1 && tune.variant != 2 && (prefill || c->l_adapter_stride == 0) &&
                            !(long_row && (pl.row_groups > 2 || (pl.row_groups == 2 && sh->head_dim == 64) || long_pair));
  int split_keys = tune.split_keys;
  RopeShares two{0, 0, 0};
  if (split_keys <= 0 && pl.mfma) {
    // Measured on MI355X: one sequence runs best with about one workgroup per CU (the
    // per-workgroup prologue is not amortised otherwise); a ragged batch wants about four
    // times as many, equal-sized pieces so the CUs stay balanced.  A batch is assumed to be
    // half as long on average as its longest sequence.
    const bool batch = n_seqs_eff > 1;
    int64_t wgs = batch ? kCUs * 4 : kCUs;
    // ... and one long sequence in a paged cache with two, where it takes the split-KV kernel, two workgroups per compute
    // unit, as long as a share then still has 512 keys (on that kernel, 32768 tokens x 8 kv heads: 35.7 against 38.6 us, 65536:
    // 49.2 against 53.7; at 256 keys per share the doubling loses)
    if (long_row && c->block_size != 0 && !paged_stream && !rope) wgs = 2 * kCUs;
    // ... and one sequence in the rotary form at ranks up to 32 likewise.  Above rank 32 a unit holds one workgroup.  Nor
    // without a B_K: nothing is rotated then, and one workgroup per unit keeps the streaming form.
    if (!batch && rope_split && key_adapter && sh->rank <= 32) two = rope_two_per_unit(c->max_seq_len, sh->n_kv_heads, pl.row_groups, pl.rows, prefill);
    if (two.n > 0) {
      split_keys = two.keys < c->max_seq_len ? two.keys : c->max_seq_len;
    } else if (work >= 2 * wgs) {
      split_keys = c->max_seq_len;  // more units than workgroups wanted: one share per sequence
    } else {
      const int64_t key_heads = work * c->max_seq_len / (batch ? 2 : 1);
      int64_t sk = (key_heads + wgs - 1) / wgs;
      // One sequence: no last share more than fit, for a second round, where the units do not divide the workgroups.  (us before
      // and now: 12 kv heads, 12 agents in two row groups, rank 32, 20000 keys, eleven shares and ten 45 / 38; paged, 8 kv heads,
      // 6 agents with low-rank caches of their own at rank 32, 30000 keys, 22 shares and 21 64 / 44; rotary, 4 kv heads, 5 agents
      // of 7 heads at rank 64, 30000 keys, 22 and 20 77 / 56.)  Not where less than three quarters of the places are taken then (12 kv
      // heads, 96 agents in twelve row groups, rank 32, 13895 keys, two shares 125 and one 156; 160 units of 256 0.90 to 1.12 of 32
      // calls, 192 and more 1.0 to 1.4 of 140), nor on the split-KV kernel while it has places left, two per unit (paged, 16 kv
      // heads, 6 agents with low-rank caches of their own at rank 32, 1304 keys, six shares 13.1, four 14.8; with one cache for the
      // call, five shares of 96 units in place of six lose 3 %).  In the rotary form, whose tiles take longest, a last share may
      // stay that is no longer than what the others would grow by: 24 units, 9000 keys, ten shares of seven tiles and one of one
      // 48 us, nine of eight 53.  (Without a B_K
      // nothing is rotated, and the call streams where one round fills the chip.)
      const bool full = wgs / work * work * 4 >= 3 * wgs, rotates = rope && (key_adapter || !full);
      const bool streams = !rotates && tune.variant != 2 && (c->block_size == 0 || paged_stream);
      // (two workgroups per unit, several row groups: the shares that fit, or up to a fifth less where they then meet; without
      // that the padded grid has another round.  28 q heads over 4, 50 agents on 10232 paged keys, rank 24 56.6 / 45; 64 over 8, 83 agents
      // on 10908, rank 64 105.7 / 94.7; 500 calls of 9 to 60 agents 1.08 in the mean, two of them 0.94 and 0.97.  At d = 64, where a
      // unit holds three, 0.94 to 1.0, and only kv heads that are no multiple of eight, whose grid is padded: 1.04 in the mean of 250,
      // 0.94 at worst.)
      const int64_t fit = wgs / work, block = interleave_step(sh->n_kv_heads), meets = fit / block * block;
      const bool pair_rows = wgs > kCUs && pl.row_groups > 1 && (sh->head_dim == 128 || block > 1) && pl.l_block == 0 && !rope && meets * 5 >= fit * 4 && meets > 0;
      if (!batch && work <= wgs && (rope || pair_rows || (wgs > kCUs && pl.l_block != 0) || (streams && full))) {
        const int64_t shares = pair_rows ? meets : (streams ? meeting_shares(fit, sh->n_kv_heads, pl.row_groups) : fit);
        const int64_t least = (c->max_seq_len + shares - 1) / shares;
        const int64_t t = (sk + tile - 1) / tile, t_least = (least + tile - 1) / tile, all = (static_cast<int64_t>(c->max_seq_len) + tile - 1) / tile;
        const int64_t last = all - (all - 1) / t * t;
        if ((all + t - 1) / t > shares && (!rotates || t + last > t_least)) sk = sk > least ? sk : least;
      }
      split_keys = sk > c->max_seq_len ? c->max_seq_len : static_cast<int>(sk);
    }
  } else if (split_keys <= 0) {
    int64_t ns = (want + work - 1) / work;
    const int64_t max_ns = (c->max_seq_len + tile - 1) / tile;
    ns = ns < 1 ? 1 : (ns > max_ns ? max_ns : ns);
    split_keys = static_cast<int>((c->max_seq_len + ns - 1) / ns);
  }
  if (split_keys > (1 << 30)) split_keys = 1 << 30;  // (a tuning value; max_seq_len itself is capped there)
  split_keys = (split_keys + tile - 1) / tile * tile;
  if (tune.split_keys <= 0 && pl.mfma && !prefill && c->n_seqs > 1 && c->seq_lens_host != nullptr && c->n_seqs <= 16384) {
    // The lengths are known (what follows is the grid of decode_mfma_kernel, which plan_batch may replace by a row of
    // shares).  A batch of sequences of about the same length runs best when the workgroups that find
    // keys are all resident at once, two per compute unit, and equal in size (measured on MI355X, 16 sequences of
    // 32768 tokens: 5.7 TB/s at 512 workgroups, 5.0 at 2048, 4.9 at 704): the smallest share size that keeps them
    // within that; never smaller than the choice above, so the workspace of a call without the lengths is large
    // enough for any call with them.  A ragged batch (shortest sequence below three quarters of the longest) does
    // best in two rounds - its shares are unequal, and twice as many workgroups as there are places level that out
    // (16 sequences of 6.5 k to 65 k tokens: 173-175 us at 840 to 960 workgroups, 199 us at 512) - but not in two
    // rounds and a bit: the time jumps by a tenth between 960 and 1020 workgroups (a second batch, 24 sequences of
    // 2 k to 40 k tokens: 190 us at 916, 206 us at 1036).  There the bound is 940.
    const int64_t units = static_cast<int64_t>(sh->n_kv_heads) * pl.row_groups;
    int64_t shortest = c->max_seq_len, longest = 0;
    for (int t = 0; t < c->n_seqs; ++t) {
      int64_t len = c->seq_lens_host[t];
      len = len < 0 ? 0 : (len > c->max_seq_len ? c->max_seq_len : len);
      shortest = len < shortest ? len : shortest;
      longest = len > longest ? len : longest;
    }
    const bool even_lengths = shortest * 4 >= longest * 3 && longest > 0;
    auto workgroups = [&](int64_t share) {
      int64_t n = 0;
      for (int t = 0; t < c->n_seqs; ++t) {
        int64_t len = c->seq_lens_host[t];
        len = len < 0 ? 0 : (len > c->max_seq_len ? c->max_seq_len : len);
        n += (len + share - 1) / share;
      }
      return n * units;
    };
    int64_t lo = split_keys / tile, hi = (static_cast<int64_t>(c->max_seq_len) + tile - 1) / tile;  // in tiles
    if (hi < lo) hi = lo;
    const int64_t bound = even_lengths ? 2 * kCUs : 940;
    if (longest > 0 && workgroups(lo * tile) > bound) {
      while (lo < hi) {  // smallest share in (lo, hi] within the bound, else hi
        const int64_t mid = lo + (hi - lo) / 2;
        if (workgroups(mid * tile) <= bound) hi = mid;
        else lo = mid + 1;
      }
      split_keys = static_cast<int>(hi * tile);
    }
  }
  if (pl.mfma && c->block_size == 0) {
    // the kernel addresses one split of a contiguous cache with 32-bit byte offsets
    const int64_t cap = ((int64_t{1} << 31) - 4096) / (c->kv_token_stride * 2) / tile * tile;
    if (cap < tile) pl.mfma = false;
    else if (split_keys > cap) split_keys = static_cast<int>(cap);
  }
  if (pl.mfma && tile_per_agent && c->block_size == 0) {
    // a wave addresses the L rows of its keys with 32-bit byte offsets
    const int64_t cap_l = ((int64_t{1} << 31) - 4096) / (l_pitch * 2) * 4 / tile * tile;
    if (cap_l < tile) pl.mfma = false;
    else if (split_keys > cap_l) split_keys = static_cast<int>(cap_l);
  }
  if (!pl.mfma) pl.short_prefill = false;
  if (pl.mfma && stream_only) {
    // These calls want the streaming form: at most one workgroup per compute unit, and a wave's L rows inside 32-bit
    // byte offsets.  Where that does not fit (more (kv head, row group) units than compute units, a very wide row
    // pitch) the split-KV kernel reads the same layouts, a wave addressing a quarter of a key share.
    const int64_t max_shares = kCUs / work;
    const int64_t cap_l = ((int64_t{1} << 31) - 4096) / (l_pitch * 2) / tile * tile;
    int64_t sk = split_keys;
    bool fits = max_shares >= 1 && cap_l >= tile;
    if (fits) {
      const int64_t need = ((c->max_seq_len + max_shares - 1) / max_shares + tile - 1) / tile * tile;
      if (sk < need) sk = need;
      fits = sk <= cap_l && sk <= ((int64_t{1} << 31) - 4096) / (c->kv_token_stride * 2) / tile * tile;
    }
    if (fits) {
      split_keys = static_cast<int>(sk);
    } else {
      const int64_t cap4 = ((int64_t{1} << 31) - 4096) / (l_pitch * 2) * 4 / tile * tile;
      if (cap4 < tile) pl.mfma = false;
      else if (split_keys > cap4) split_keys = static_cast<int>(cap4);
    }
  }
  if (!pl.mfma) pl.l_block = 0;
  pl.split_keys = split_keys;
  pl.n_splits = static_cast<int>((static_cast<int64_t>(c->max_seq_len) + split_keys - 1) / split_keys);
  if (pl.mfma && two.n > 0 && split_keys == two.keys) {
    pl.n_splits = two.n;
    pl.split_more = two.more;
  }
  if (pl.mfma && !prefill && c->block_size != 0 && c->n_seqs > 1 && tune.variant == 0 && tune.split_keys <= 0)
    plan_batch(pl, sh, c, key_adapter);
  // grids: (kv head, share, sequence x row group) for the MFMA kernels, (row, share) otherwise
  pl.launchable = pl.n_splits <= 65535 &&
                  (!pl.mfma || static_cast<int64_t>(n_seqs_eff) * pl.row_groups <= 65535);
  const size_t slots = static_cast<size_t>(pl.rows) * pl.n_splits;
  pl.off_ml = 0;
  pl.off_o = align_up(slots * 2 * sizeof(float), 256);
  pl.off_lr = pl.off_o + align_up(slots * sh->head_dim * sizeof(float), 256);
  pl.off_adapter = pl.off_lr + align_up(slots * sh->rank * sizeof(float), 256);
  pl.bytes = pl.off_adapter + align_up(static_cast<size_t>(pl.rows) * sizeof(int32_t), 256);
  // room for Qt of the whole call where the streaming form of the split-KV kernel, which takes at most one workgroup per
  // compute unit, would otherwise reload many B_K rows per workgroup (reserved whether or not the call has a B_K)
  pl.off_qt = pl.bytes;
  pl.qt_bytes = 0;
  if (pl.mfma && !prefill && (c->block_size == 0 || paged_stream) && work * pl.n_splits <= kCUs && !rope_split && tune.variant != 2 && pl.l_block == 0)
    pl.qt_bytes = decode_stream_qt_bytes(pl.group_pad, sh->rank, pl.row_tiles, pl.row_groups, sh->n_kv_heads);
  pl.bytes += align_up(pl.qt_bytes, 256);
  pl.bytes_without_kc = pl.bytes;
  return pl;
}

// Whether a prefill of few new tokens that the lines above give to the tile walk, or the shares of prefill_rows_kernel, runs on the
// streaming kernel.  Four to eight kv heads of 128, ranks up to 32, up to three row groups; ratio of the times there / streaming, three
// sets of tensors taken in turn, ranks 16 / 32 where they differ, at 1, 2, 3, 4.5, 6, 9 and 13 thousand keys:
//   8 kv heads, G 4    8 tokens 0.97 1.11 1.10 1.01 1.03 0.96 0.97 / 0.94 1.04 1.00 0.95 0.99 0.95 1.0, paged 0.98 1.11 1.12 1.03 1.02 0.97 0.97 /
//                      0.95 1.07 1.05 0.97 1.01 0.99 1.0; 16 tokens 1.06 1.09 1.09 0.99 1.04 0.89 0.94 / 1.02 1.11 1.09 1.02 1.05 0.98 0.99, paged
//                      1.10 1.11 1.07 0.99 0.95 0.88 0.85 / 1.03 1.14 1.10 1.04 0.98 0.90 0.88; 24 tokens 1.16 1.15 1.06 1.04 0.97 0.89 0.83, paged
//                      1.21 1.14 1.05 0.90 0.85 0.77 0.70
//   4 kv heads, G 7    3 and 4 tokens 0.92 0.96 1.03 1.08 1.07 1.02 1.0, paged 0.96 0.98 1.07 1.13 1.13 1.15 0.99; 6 and 8 1.02 1.06 1.10 1.08 1.08
//                      1.05 0.99, paged 1.07 1.09 1.13 1.10 1.10 1.09 1.13; 12 1.11 1.18 1.10 1.15 1.05 1.05 1.0, paged 1.15 1.20 1.12 1.17 1.05 1.0
//                      0.95 (9 tokens 0.96 to 0.97 at 5.8 k)
// (Two row groups on the pages of fewer than six kv heads beyond 14 k keep the shares of prefill_rows_kernel: not measured there.)
// 5, 6 and 7 kv heads, groups of 1 to 16, value-side adapters only, 3300 more calls after the exchange of prefill_rows_kernel and the
// merge got shorter: 1.07 in the mean, 0.96 at worst.  Groups of one and two q heads fill a quarter and a half of their padded rows: one
// row group 0.92 to 0.97 to 1800 keys, several 1.0 to 1.15 to 2100 and 0.80 to 0.96 beyond, except with 4 and 5 kv heads (1.0 to 1.1); three of
// group 1 0.80 to 0.96 from 1750 on.  6 kv heads: one row group 0.96 to 0.99 at 6 thousand (7: 1.0 to 1.04), three 0.89 to 0.97 from 3300 on.
static bool few_tokens_stream(const lra_shape* sh, const lra_cache* c, int tokens, int row_groups) {
  if (sh->head_dim != 128 || sh->rank > 32 || sh->n_kv_heads < 4 || sh->n_kv_heads > 8 || row_groups > 3) return false;
  const int hkv = sh->n_kv_heads, G = sh->n_q_heads / hkv, rows = tokens * G, n = c->max_seq_len;
  const bool pages = c->block_size != 0, wide = sh->rank > 16, few = hkv < 6;
  if (row_groups == 1) return few ? n > (pages ? 2304 : 2560) : n > (G < 3 ? 1920 : 1536) && n <= (wide ? 3328 : (hkv == 6 ? 5120 : 7168));
  if (n <= 900 || (G == 1 && row_groups == 3)) return false;
  if (few) return row_groups == 2 ? !pages || n <= 14336 : n <= 5120 || (!pages && rows >= 84);
  if (G < 3) return n <= 2304;
  return n <= (row_groups == 2 ? (wide ? (pages ? 4608 : 6144) : 3584) : (hkv == 6 ? 3072 : (pages ? 3584 : 5120)));
}

// What the streaming kernel does with a call: key shares of any number of 32-key tiles, which its waves divide as they come.  Shares of
// 129 to 1024 keys (two row tiles or several row groups: 384; pages: 256) are as long as the places ask for, not the next multiple of
// 128.  Ratio of the times with multiples of 128 / so, three sets of tensors in turn, rank 16: 8 kv heads of group 4, 1 and 4 agents on
// 4300 keys 1.07 to 1.12, 5000 1.05 to 1.07 (paged 1.03), 5700 1.04, 9009 to 13000 1.01 to 1.03 (paged 0.98 to 1.01), beyond 1.0 to 1.01 (paged
// 0.98 to 1.0); 8 agents, two row tiles, 1.07, 1.02, 1.04, 1.0 to 1.04 on 9009 to 11200, 0.99 on 13000 and 15000 (paged 0.97 on 9009); 4 kv
// heads of group 7, twice as many shares, on 9009 1.05 to 1.08, 10000 1.03 to 1.07, 11200 1.01 to 1.04.  Where a pre-pass forms Qt 0.97 to
// 1.02; shares below 128 add one more per row and cost what the shorter ones save.  By kv heads (groups of 4 and 8, ranks 16, 32 and
// 64, 650 calls; n x kv heads / 256 = 140, 170, 200, 300, 420, 700): 4, 8, 12 ... 48 1.03 to 1.17, 1.0 to 1.1, 1.0 to 1.07, 1.0 to 1.06, 0.99 to 1.1,
// 0.99 to 1.03; 5 and those above 8 that are no multiple of four 1.01 to 1.08, 0.97 to 1.05, 0.95 to 1.04, then 0.91 to 1.03; 6 and 7 0.91 to
// 1.02 throughout; 1 to 3, whose more than 64 shares take the slow form of the merge, 0.7 to 0.99 (3 on 23037 at rank 64 0.70).
// 64 wide with two row tiles at 140 0.95 to 1.0 up to 12 kv heads, from 170 on 0.98 to 1.05.
static void plan_stream(Plan& pl, const lra_shape* sh, const lra_cache* c, int tokens, int max_queries_per_seq, bool prefill,
                        const Tuning& tune, bool key_adapter) {
  if (sh->key_rope_theta > 0.f || (!prefill && c->n_seqs != 1)) return;
  Plan st = pl;
  if (prefill && (!pl.short_prefill || pl.wave_shares > 0)) {
    // (a call that needs no workspace goes on without one)
    if (tune.short_prefill != 32 || tune.prefill_splits != 0 || !pl.split_kv_sized || pl.bytes == 0) return;
    const int G = sh->n_q_heads / sh->n_kv_heads, rows = tokens * (G <= 4 ? 4 : (G <= 8 ? 8 : 16));
    if (!few_tokens_stream(sh, c, tokens, (rows + 31) / 32)) return;
    Tuning forced = tune;
    forced.short_prefill = 33;
    if (!pl.short_prefill) st = plan_call(sh, c, tokens, max_queries_per_seq, true, forced, key_adapter);
    if (!st.mfma || !st.short_prefill) return;
  }
  // as in plan_call: the call streams (a paged decode of low-rank caches per adapter does not, nor one that it gives two workgroups
  // per unit), and one round of its shares fills the chip
  const int64_t work = static_cast<int64_t>(sh->n_kv_heads) * st.row_groups, n = c->max_seq_len;
  if (work * st.n_splits > kCUs || (c->block_size != 0 && !prefill && c->l_adapter_stride != 0)) return;
  const bool finer = kCUs / work * work * 4 >= 3 * kCUs && (prefill || st.qt_bytes == 0);
  int64_t keys = st.split_keys;
  if (finer) {
    const int64_t fit = kCUs / work, even = (n * work + kCUs - 1) / kCUs;
    const int hkv = sh->n_kv_heads;
    const int64_t most = hkv % 4 != 0 ? (hkv == 5 || hkv > 8 ? 192 : 0)
                                      : (c->block_size != 0 ? 256 : (st.row_tiles > 1 || st.row_groups > 1 ? 384 : 1024));
    const int64_t from = sh->head_dim == 64 && st.row_tiles > 1 ? 160 : 128;
    if (even > from && even <= most) {
      const int64_t shares = meeting_shares(fit, sh->n_kv_heads, st.row_groups);
      const int64_t least = ((n + shares - 1) / shares + 31) / 32 * 32;
      keys = least < keys ? least : keys;
    }
  }
  if (keys == st.split_keys && st.short_prefill == pl.short_prefill && pl.wave_shares == 0) return;
  pl.stream_keys = static_cast<int>(keys);
  pl.stream_splits = static_cast<int>((n + keys - 1) / keys);
  pl.stream_pad = st.group_pad;
  pl.stream_row_tiles = st.row_tiles;
  pl.stream_row_groups = st.row_groups;
  pl.stream_prefill = prefill;
  if (pl.stream_splits > pl.n_splits) {  // room for either
    const size_t slots = static_cast<size_t>(pl.rows) * pl.stream_splits;
    pl.off_ml = 0;
    pl.off_o = align_up(slots * 2 * sizeof(float), 256);
    pl.off_lr = pl.off_o + align_up(slots * sh->head_dim * sizeof(float), 256);
    pl.off_adapter = pl.off_lr + align_up(slots * sh->rank * sizeof(float), 256);
    pl.off_qt = pl.off_adapter + align_up(static_cast<size_t>(pl.rows) * sizeof(int32_t), 256);
    pl.bytes = pl.off_qt + align_up(pl.qt_bytes, 256);
    pl.bytes_without_kc = pl.bytes;
  }
}

Plan make_plan(const lra_shape* sh, const lra_cache* c, int tokens, int max_queries_per_seq, bool prefill,
               const Tuning& tune, bool key_adapter) {
  Plan pl = plan_call(sh, c, tokens, max_queries_per_seq, prefill, tune, key_adapter);
  pl.wave_shares = 0;
  if (prefill && pl.mfma && pl.n_splits > 1 && !pl.wave_rows && tune.variant == 0 && tune.prefill_splits == 0 && tune.short_prefill <= 32 &&
      tune.split_keys <= 0) {
    if (prefill_rows_reads(sh, c, pl.split_kv_sized, pl.kc_bytes > 0))
      pl.wave_shares = plan_wave_shares(sh, c, tokens, pl.n_splits);
  }
  if (pl.mfma && !pl.wave_rows && pl.launchable && tune.variant == 0 && tune.split_keys <= 0 && tune.stream_shares)
    plan_stream(pl, sh, c, tokens, max_queries_per_seq, prefill, tune, key_adapter);
  return pl;
}

Plan as_run(const Plan& plan) {
  Plan pl = plan;
  if (pl.stream_keys == 0) return pl;
  pl.split_keys = pl.stream_keys;
  pl.n_splits = pl.stream_splits;
  pl.group_pad = pl.stream_pad;
  pl.row_tiles = pl.stream_row_tiles;
  pl.row_groups = pl.stream_row_groups;
  pl.short_prefill = pl.stream_prefill;
  pl.wave_shares = 0;
  return pl;
}

}  // namespace lra
