// What the launch planner answers for one call, for tests that name the kernel they run (tests/test_gpu_cases_plan_cpu.py).
#include "lra_plan.h"

extern "C" void plan_query(const lra_shape* sh, const lra_cache* c, int tokens, int max_queries_per_seq, int prefill,
                           int key_adapter, const lra_tuning* tuning, int32_t* out) {
  const lra::Plan pl = lra::make_plan(sh, c, tokens, max_queries_per_seq, prefill != 0, lra::resolve_tuning(tuning), key_adapter != 0);
  out[0] = pl.mfma;
  out[1] = pl.short_prefill;
  out[2] = pl.wave_rows;
  out[3] = pl.wave_shares;
  out[4] = pl.n_splits;
  out[5] = pl.tile_group;
  out[6] = pl.batch_wgs;
  out[7] = pl.batch_tiles;
  out[8] = pl.row_tiles;
  out[9] = pl.row_groups;
  out[10] = pl.l_block;
  out[11] = pl.workspace_optional;
  out[12] = pl.group_pad;
  out[13] = pl.split_keys;
  out[14] = pl.split_more;
  out[15] = static_cast<int32_t>(pl.qt_bytes);
  out[16] = static_cast<int32_t>(pl.bytes >> 8);
}

// The merge kernel that a call ends with (0 merge_kernel, 1 merge_rows_kernel, 2 merge_wave_kernel, 3 merge_tokens_kernel; -1: none) and
// the shares per row that it takes.
extern "C" int merge_query(const lra_shape* sh, const lra_cache* c, int tokens, int max_queries_per_seq, int prefill, int key_adapter,
                           const lra_tuning* tuning, int32_t* shares) {
  const lra::Plan pl = lra::as_run(lra::make_plan(sh, c, tokens, max_queries_per_seq, prefill != 0, lra::resolve_tuning(tuning), key_adapter != 0));
  *shares = pl.batch_wgs > 0 ? pl.batch_splits : pl.n_splits;
  const int wave = pl.wave_rows ? 1 : pl.wave_shares;
  if (prefill && pl.mfma && !(pl.short_prefill && wave == 0)) {
    *shares = wave > 0 ? wave : pl.n_splits;
    if (*shares == 1) return -1;
  }
  return static_cast<int>(lra::merge_form(sh->dtype == LRA_BF16, sh->head_dim, sh->rank, sh->n_q_heads, sh->n_kv_heads, *shares, prefill != 0,
                                          tokens * sh->n_q_heads));
}

extern "C" int stream_grid_query(int n_kv_heads, int n_splits, int row_groups) { return lra::stream_grid_shares(n_kv_heads, n_splits, row_groups); }

extern "C" int interleave_query(int n_kv_heads, int n_splits, int row_groups, int rotary) {
  return lra::mfma_interleave(n_kv_heads, n_splits, row_groups, rotary != 0);
}

extern "C" int append_query(int n_new, int n_kv_heads, int head_dim, int rank, int d_model, const lra_tuning* tuning) {
  const lra::Tuning t = lra::resolve_tuning(tuning);
  if (lra::append_quarter_tiles(n_new, n_kv_heads, head_dim, rank, d_model, t)) return -1;
  const int parts = lra::plan_append_split(n_new, n_kv_heads, head_dim, rank, d_model, t).k_splits;
  return parts > 1 && lra::append_streams(n_new, n_kv_heads, head_dim, d_model, t) ? -2 : parts;
}
