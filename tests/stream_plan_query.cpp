// What runs of a call's plan (as_run: the streaming kernel's own key shares and calls), in the fields of tests/plan_query.cpp, for
// tests/test_stream_shares_cpu.py and tests/test_stream_shares_gpu.py.
#include "lra_plan.h"

extern "C" void plan_query(const lra_shape* sh, const lra_cache* c, int tokens, int max_queries_per_seq, int prefill,
                           int key_adapter, const lra_tuning* tuning, int32_t* out) {
  const lra::Plan pl = lra::as_run(lra::make_plan(sh, c, tokens, max_queries_per_seq, prefill != 0, lra::resolve_tuning(tuning), key_adapter != 0));
  const int32_t fields[] = {pl.mfma, pl.short_prefill, pl.wave_rows, pl.wave_shares, pl.n_splits, pl.tile_group, pl.batch_wgs, pl.batch_tiles,
                            pl.row_tiles, pl.row_groups, pl.l_block, pl.workspace_optional, pl.group_pad, pl.split_keys, pl.split_more,
                            static_cast<int32_t>(pl.qt_bytes), static_cast<int32_t>(pl.bytes >> 8)};
  for (int i = 0; i < 17; ++i) out[i] = fields[i];
}
