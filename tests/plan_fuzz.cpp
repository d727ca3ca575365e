// Fuzz driver for the host-side launch planning (csrc/lra_plan.cpp), built for the CPU alone with
// -fsanitize=address,undefined by tests/test_plan_sanitized.py: random and extreme shapes, strides
// and sizes go through the argument checks and, where those accept them, through the planner; every
// plan must keep its invariants, and the sanitizers must stay silent (signed overflow in the 32-bit
// offset caps and workspace sizes is what this is after).
#include <vector>
#include <cinttypes>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#include "lra_plan.h"

using namespace lra;

static uint64_t state = 0x9e3779b97f4a7c15ull;
static uint64_t rnd() {
  state ^= state << 13;
  state ^= state >> 7;
  state ^= state << 17;
  return state;
}
static int64_t pick(std::initializer_list<int64_t> v) { return *(v.begin() + rnd() % v.size()); }

#define CHECK(cond)                                                                     \
  do {                                                                                  \
    if (!(cond)) {                                                                      \
      std::fprintf(stderr, "plan_fuzz: %s failed at case %d (line %d)\n", #cond, it, __LINE__); \
      return 1;                                                                         \
    }                                                                                   \
  } while (0)

// Every key is in a share and no share is empty; those behind the first split_more hold 128 keys less.
static bool shares_cover(const Plan& pl, int64_t keys) {
  if (pl.split_more < 0 || pl.split_more >= pl.n_splits || (pl.split_more > 0 && pl.split_keys < 256)) return false;
  const int64_t large = pl.split_more > 0 ? pl.split_more : pl.n_splits, last = pl.split_keys - (pl.split_more > 0 ? 128 : 0);
  const int64_t all = large * pl.split_keys + (pl.n_splits - large) * last;
  return all >= keys && all - last < keys;
}

int main(int argc, char** argv) {
  const int cases = argc > 1 ? std::atoi(argv[1]) : 200000;
  static char dummy[64];
  int accepted = 0, uneven = 0;
  for (int it = 0; it < cases; ++it) {
    // every field: usually from the values the library supports, now and then a bad one
    auto pv = [&](std::initializer_list<int64_t> good, std::initializer_list<int64_t> bad) { return rnd() % 12 ? pick(good) : pick(bad); };
    lra_shape sh{};
    sh.n_kv_heads = static_cast<int32_t>(pv({1, 2, 4, 8, 3}, {0, -1, 1 << 20}));
    sh.n_q_heads = sh.n_kv_heads > 0 && rnd() % 12 ? sh.n_kv_heads * static_cast<int32_t>(pv({1, 2, 4, 7, 8, 16}, {17}))
                                                   : static_cast<int32_t>(pick({0, 5, 32, INT32_MAX}));
    sh.head_dim = static_cast<int32_t>(pv({64, 128}, {96, 0, 256}));
    sh.rank = static_cast<int32_t>(pv({1, 4, 8, 12, 16, 24, 32, 40, 64}, {65, 0, -3}));
    sh.dtype = static_cast<int32_t>(pv({0, 0, 0, 1}, {2, -1}));
    sh.scale = rnd() % 6 ? 0.f : static_cast<float>(pick({1, -1})) * 0.125f;
    sh.key_rope_theta = rnd() % 4 ? 0.f : 500000.f;
    lra_cache c{};
    c.k_base = c.v_base = c.l = dummy;
    c.seq_lens = reinterpret_cast<const int32_t*>(dummy);
    const bool paged = rnd() % 2;
    c.block_size = paged ? 16 : static_cast<int32_t>(pv({0}, {8}));
    c.n_seqs = paged ? static_cast<int32_t>(pv({1, 2, 16, 1000, 1 << 20}, {0, (1 << 20) + 1})) : static_cast<int32_t>(pv({1}, {2}));
    c.max_seq_len = static_cast<int32_t>(pv({1, 2, 31, 32, 33, 127, 128, 129, 1000, 8192, 65536, 1 << 20, 1 << 27, 1 << 30},
                                            {INT32_MAX, 0, -1}));
    const int64_t d = sh.head_dim > 0 ? sh.head_dim : 8;
    c.kv_token_stride = pv({d, d * 8, d * 8 + 8, d * 1024, int64_t{1} << 33}, {d - 8, 0, d + 4});
    c.kv_head_stride = pv({d, d * 16, static_cast<int64_t>(c.max_seq_len > 0 ? c.max_seq_len : 1) * d, int64_t{1} << 40}, {0});
    c.kv_block_stride = paged ? pv({16 * d, 16 * d * 8, int64_t{1} << 36}, {8, 0}) : 0;
    c.max_blocks_per_seq = paged ? static_cast<int32_t>(pv({(static_cast<int64_t>(c.max_seq_len > 0 ? c.max_seq_len : 1) + 15) / 16, INT32_MAX}, {1, 4})) : 0;
    c.num_blocks = paged ? static_cast<int32_t>(pv({1, 100, 1 << 20, INT32_MAX}, {0})) : 0;
    c.block_table = paged && rnd() % 16 ? reinterpret_cast<const int32_t*>(dummy) : nullptr;
    const int64_t rk = sh.rank > 0 ? sh.rank : 8;
    c.l_row_stride = pv({0, 0, (rk + 7) / 8 * 8, rk * 4 / 8 * 8 + 8, 4096, int64_t{1} << 31}, {rk - 1 > 0 ? (rk - 1) / 8 * 8 : 8, 12, -8, (int64_t{1} << 31) + 8});
    c.l_adapter_stride = pv({0, 0, 0, 16, 64, int64_t{1} << 30, int64_t{1} << 40}, {-8, 4, (int64_t{1} << 40) + 8});
    lra_tuning t{};
    t.kernel_variant = static_cast<int32_t>(pick({0, 0, 1, 2, 7}));
    t.decode_split_keys = static_cast<int32_t>(pick({0, 0, 1, 64, 100, 1 << 20, INT32_MAX, -5}));
    t.short_prefill = static_cast<int32_t>(pick({0, -1, 1, 64, INT32_MAX}));
    t.prefill_splits = static_cast<int32_t>(pick({0, 1, 5, 32, 1000, -1}));
    t.rope_key_prepass = static_cast<int32_t>(pick({0, 0, -1, 1}));
    const Tuning tune = resolve_tuning(rnd() % 4 ? &t : nullptr);
    if (check_common(&sh, &c) != LRA_OK) continue;
    ++accepted;
    const int G = sh.n_q_heads / sh.n_kv_heads;
    for (int prefill = 0; prefill < 2; ++prefill) {
      int64_t tokens = pick({1, 2, 3, 4, 8, 16, 17, 33, 64, 1000, 4096, 1 << 20, 1 << 26, INT32_MAX});
      if (prefill && tokens > c.max_seq_len) tokens = c.max_seq_len;
      int64_t mq = prefill ? 1 : pick({1, 1, 2, 4, 5, 9, 64, tokens});
      if (mq > tokens) mq = tokens;
      if (!plan_sizes_fit(&sh, &c, static_cast<int32_t>(tokens), static_cast<int32_t>(mq))) continue;
      const Plan pl = make_plan(&sh, &c, static_cast<int>(tokens), static_cast<int>(mq), prefill != 0, tune);
      CHECK(pl.rows == tokens * sh.n_q_heads);
      CHECK(pl.n_splits >= 1 && pl.split_keys >= 1);
      CHECK(pl.split_more == 0 || !prefill || pl.short_prefill);
      CHECK((prefill && pl.mfma && !pl.short_prefill) || shares_cover(pl, c.max_seq_len));
      CHECK(pl.off_ml % 256 == 0 && pl.off_o % 256 == 0 && pl.off_lr % 256 == 0 && pl.off_adapter % 256 == 0 && pl.off_qt % 256 == 0);
      CHECK(pl.bytes % 256 == 0);
      CHECK(pl.bytes == pl.bytes_without_kc + pl.kc_bytes && pl.off_kc % 256 == 0 && pl.kc_bytes % 256 == 0);
      {
        // a call without a B_K runs in a workspace that was sized without knowing that
        const Plan pk = make_plan(&sh, &c, static_cast<int>(tokens), static_cast<int>(mq), prefill != 0, tune, false);
        CHECK(pk.mfma == pl.mfma && pk.bytes <= pl.bytes && pk.bytes_without_kc <= pl.bytes_without_kc);
        CHECK(pk.n_splits <= pl.n_splits && pk.split_keys >= pl.split_keys);
      }
      if (prefill && pl.mfma && !pl.short_prefill) {
        CHECK(pl.tile_group == 1 || pl.tile_group == G);
        Tuning alone = tune;  // what a call falls back to where the workspace is optional and missing
        alone.prefill_splits = -1;
        const Plan pa = make_plan(&sh, &c, static_cast<int>(tokens), 1, true, alone);
        CHECK(pa.n_splits == 1 && pa.bytes_without_kc == 0 && !pa.workspace_optional && (tune.prefill_splits > 0 || pa.tile_group == pl.tile_group));
        CHECK(!pl.workspace_optional || (c.max_seq_len < 1024 && pl.n_splits > 1));
        if (tune.prefill_splits > 0) CHECK(pl.tile_group == G);
      }
      if (pl.wave_rows) {  // 32-row workgroups in at most two rounds, every byte offset within 2 GB, completed keys where a B_K is rotated
        CHECK(prefill && pl.mfma && sh.rank <= 32 && (tokens * G + 31) / 32 * sh.n_kv_heads <= 512);
        CHECK(!(sh.key_rope_theta > 0.f) || pl.kc_bytes > 0);
        const int64_t pitch = c.l_row_stride ? c.l_row_stride : sh.rank, top = 0x7ffff000;
        if (c.block_size == 0) CHECK(int64_t{c.max_seq_len} * c.kv_token_stride * 2 <= top && int64_t{c.max_seq_len} * pitch * 2 <= top);
        else CHECK(c.max_seq_len <= 8192 && int64_t{c.num_blocks} * c.kv_block_stride * 2 <= top && int64_t{c.num_blocks} * 16 * pitch * 2 <= top);
      }
      if (pl.wave_shares) {  // that kernel with shares: one workgroup per compute unit, states inside the plan's slots, a wave's block ids in one register
        CHECK(prefill && pl.mfma && !pl.wave_rows && sh.rank <= 32 && pl.wave_shares >= 2 && pl.wave_shares <= 32 && pl.wave_shares <= pl.n_splits);
        CHECK((tokens * G + 31) / 32 * sh.n_kv_heads * pl.wave_shares <= 256 && (int64_t{c.max_seq_len} + 31) / 32 <= 256 * pl.wave_shares);
        CHECK(!(sh.key_rope_theta > 0.f) || pl.kc_bytes > 0);
        CHECK(tune.variant == 0 && tune.prefill_splits == 0 && tune.split_keys == 0);
        const int64_t pitch = c.l_row_stride ? c.l_row_stride : sh.rank, top = 0x7ffff000;
        if (c.block_size == 0) CHECK(int64_t{c.max_seq_len} * c.kv_token_stride * 2 <= top && int64_t{c.max_seq_len} * pitch * 2 <= top);
        else CHECK(int64_t{c.num_blocks} * c.kv_block_stride * 2 <= top && int64_t{c.num_blocks} * 16 * pitch * 2 <= top);
      }
      if (pl.batch_wgs) {  // a batch's shares in one row: a place for every sequence, every state inside the workspace's slots
        CHECK(!prefill && pl.mfma && c.block_size != 0 && c.n_seqs > 1 && c.n_seqs <= 64 && pl.batch_wgs >= c.n_seqs);
        CHECK(static_cast<int64_t>(pl.batch_wgs) * sh.n_kv_heads * pl.row_groups <= 512);
        CHECK(pl.batch_splits >= 1 && pl.batch_splits <= pl.n_splits && pl.batch_min_tiles >= 1);
        const int64_t size = pl.batch_tiles > 0 ? pl.batch_tiles : pl.batch_min_tiles;
        CHECK(size >= pl.batch_min_tiles && size * 128 * pl.batch_splits >= c.max_seq_len);
      }
      if (pl.kc_bytes) {  // completed keys of a rotary prefill: a copy of the K_base extent behind everything else
        CHECK(prefill && pl.mfma && !pl.short_prefill && sh.key_rope_theta > 0.f);
        CHECK(pl.off_kc >= pl.bytes_without_kc);
        // contiguous: the extent of K_base; paged: the sequence's blocks in logical order at the strides of the pool
        const int64_t span = c.block_size == 0
            ? (static_cast<int64_t>(c.max_seq_len) - 1) * c.kv_token_stride +
                  (static_cast<int64_t>(sh.n_kv_heads) - 1) * c.kv_head_stride + sh.head_dim
            : (static_cast<int64_t>(c.max_seq_len) - 1) / 16 * c.kv_block_stride +
                  (static_cast<int64_t>(sh.n_kv_heads) - 1) * c.kv_head_stride + 15 * c.kv_token_stride + sh.head_dim;
        CHECK(pl.kc_bytes >= static_cast<size_t>(span) * 2 && pl.kc_bytes <= (size_t{1} << 32) + 256);
      }
      if (pl.bytes_without_kc) {
        const size_t slots = static_cast<size_t>(pl.rows) * pl.n_splits;
        CHECK(pl.off_o >= slots * 8 && pl.off_lr >= pl.off_o + slots * sh.head_dim * 4);
        CHECK(pl.off_adapter >= pl.off_lr + slots * sh.rank * 4 && pl.off_qt >= pl.off_adapter + static_cast<size_t>(pl.rows) * 4);
        CHECK(pl.bytes_without_kc >= pl.off_qt + pl.qt_bytes);
      }
      if (pl.l_block) {  // per-adapter low-rank caches on the MFMA decode path, one column block of the L tile per agent slot
        CHECK(!prefill && pl.mfma && c.l_adapter_stride > 0 && pl.row_tiles == 1 && !(sh.key_rope_theta > 0.f));
        CHECK(pl.l_block * (16 / pl.group_pad) <= 64 && pl.l_block >= sh.rank && pl.qt_bytes == 0);
        const int64_t pitch = c.l_row_stride ? c.l_row_stride : sh.rank;
        if (c.block_size == 0) {
          // contiguous cache (streaming form with at most one workgroup per compute unit, else split-KV form): a
          // wave's L rows inside 32-bit byte offsets
          CHECK(static_cast<int64_t>(pl.split_keys) / 4 * pitch * 2 < (int64_t{1} << 31));
        } else {
          // split-KV form on a paged cache: the whole pool of an adapter's L rows inside them
          CHECK(static_cast<int64_t>(c.num_blocks) * 16 * pitch * 2 < (int64_t{1} << 31));
        }
      }
      if (!prefill && c.n_seqs > 1 && c.n_seqs <= 2000) {
        // with a host copy of the lengths (any values: they are clamped) the key shares only grow, the workspace
        // only shrinks, and nothing else of the plan moves
        std::vector<int32_t> lens(static_cast<size_t>(c.n_seqs));
        for (auto& v : lens) v = static_cast<int32_t>(pick({-3, 0, 1, 17, c.max_seq_len / 2, c.max_seq_len, c.max_seq_len, INT32_MAX}));
        lra_cache cm = c;
        cm.seq_lens_host = lens.data();
        const Plan pm = make_plan(&sh, &cm, static_cast<int>(tokens), static_cast<int>(mq), false, tune);
        CHECK(pm.mfma == pl.mfma && pm.group_pad == pl.group_pad && pm.row_groups == pl.row_groups && pm.l_block == pl.l_block);
        CHECK(pm.split_keys >= pl.split_keys && pm.n_splits <= pl.n_splits && pm.bytes <= pl.bytes);
        CHECK(pm.split_keys % (pm.mfma ? 128 : 64) == 0);
        if (c.block_size == 0 && pm.mfma) CHECK(static_cast<int64_t>(pm.split_keys) * c.kv_token_stride * 2 < (int64_t{1} << 31));
      }
      const bool split_path = !prefill || pl.short_prefill || !pl.mfma;
      if (split_path && pl.mfma) {
        CHECK(pl.split_keys % 128 == 0);
        CHECK(pl.group_pad == 4 || pl.group_pad == 8 || pl.group_pad == 16);
        CHECK(pl.group_pad >= G && (pl.row_tiles == 1 || pl.row_tiles == 2));
        CHECK(static_cast<int64_t>(pl.row_groups) * pl.row_tiles * 16 >= (prefill ? tokens : mq) * pl.group_pad);
        if (c.block_size == 0) CHECK(static_cast<int64_t>(pl.split_keys) * c.kv_token_stride * 2 < (int64_t{1} << 31));
        CHECK(!pl.launchable || (pl.n_splits <= 65535 && static_cast<int64_t>(pl.row_groups) * (prefill ? 1 : c.n_seqs) <= 65535));
      } else if (split_path) {
        CHECK(pl.split_keys % 64 == 0);
      }
    }
  }
  // two workgroups per compute unit for rotary decodes of one sequence: not where that makes more than 64 shares of
  // fewer than 384 keys, whatever the length (multiples of the key tile and their neighbours among them)
  for (int it = 0; it < cases; ++it) {
    lra_shape sh{};
    sh.n_kv_heads = static_cast<int32_t>(pick({1, 2, 4, 8, 16, 32}));
    sh.n_q_heads = sh.n_kv_heads * static_cast<int32_t>(pick({1, 2, 4, 7, 8, 16}));
    sh.head_dim = 128;
    sh.rank = static_cast<int32_t>(pick({8, 16, 32, 64}));
    sh.key_rope_theta = 500000.f;
    lra_cache c{};
    c.k_base = c.v_base = c.l = dummy;
    c.seq_lens = reinterpret_cast<const int32_t*>(dummy);
    c.n_seqs = 1;
    c.max_seq_len = static_cast<int32_t>(pick({128, 1024, 4096, 8192, 16384, 20011, 32768, 50000, 65536, 131072})) +
                    static_cast<int32_t>(pick({-1, 0, 0, 1}));
    c.kv_token_stride = sh.head_dim * sh.n_kv_heads;
    c.kv_head_stride = sh.head_dim;
    const int agents = static_cast<int>(pick({1, 2, 4, 8, 16}));
    const Plan two = make_plan(&sh, &c, agents, agents, false, Tuning{}), one = make_plan(&sh, &c, agents, agents, false, Tuning{}, false);
    CHECK(!two.mfma || shares_cover(two, c.max_seq_len));
    uneven += two.split_more > 0;
    // (with a B_K one workgroup per unit may leave a short last share, the first of a second round, which without one it may not)
    if (two.split_keys == one.split_keys || (two.n_splits - 1) * sh.n_kv_heads * two.row_groups <= 256) continue;
    CHECK(sh.rank <= 32 && two.split_keys < one.split_keys);
    CHECK(two.n_splits <= 64 || two.split_keys >= 384);
    CHECK(two.split_keys >= 256 || static_cast<int64_t>(two.rows) * two.n_splits <= 2048);
  }
  // ... and for rotary prefills of a few tokens: only where a share keeps 384 keys
  for (int it = 0; it < cases; ++it) {
    lra_shape sh{};
    sh.n_kv_heads = static_cast<int32_t>(pick({1, 2, 4, 8, 16, 32}));
    sh.n_q_heads = sh.n_kv_heads * static_cast<int32_t>(pick({1, 2, 4, 7, 8, 16}));
    sh.head_dim = 64;
    sh.rank = static_cast<int32_t>(pick({8, 16, 32, 64}));
    sh.key_rope_theta = 500000.f;
    lra_cache c{};
    c.k_base = c.v_base = c.l = dummy;
    c.seq_lens = reinterpret_cast<const int32_t*>(dummy);
    c.n_seqs = 1;
    c.max_seq_len = static_cast<int32_t>(pick({128, 1024, 4096, 8192, 16384, 20011, 32768, 50000, 65536})) + static_cast<int32_t>(pick({-1, 0, 1}));
    c.kv_token_stride = sh.head_dim * sh.n_kv_heads;
    c.kv_head_stride = sh.head_dim;
    const int n_new = static_cast<int>(pick({1, 4, 8, 16, 31, 32}));
    const Plan two = make_plan(&sh, &c, n_new, 1, true, Tuning{}), one = make_plan(&sh, &c, n_new, 1, true, Tuning{}, false);
    CHECK((two.mfma && !two.short_prefill) || shares_cover(two, c.max_seq_len));
    uneven += two.split_more > 0;
    // (with a B_K one workgroup per unit may leave a short last share, the first of a second round, which without one it may not)
    if (two.split_keys == one.split_keys || (two.n_splits - 1) * sh.n_kv_heads * two.row_groups <= 256) continue;
    CHECK(two.short_prefill && two.split_keys >= 384 && two.n_splits <= 64);
  }
  // ... and every workgroup of theirs finds a place at once: 8 kv heads, 9 tokens of a group of 4, three row groups
  {
    lra_shape sh{};
    sh.n_kv_heads = 8;
    sh.n_q_heads = 32;
    sh.head_dim = 128;
    sh.rank = 32;
    sh.key_rope_theta = 500000.f;
    lra_cache c{};
    c.n_seqs = 1;
    c.kv_token_stride = 1024;
    c.kv_head_stride = 128;
    for (int it = 9000; it < 21000; it += 37) {
      c.max_seq_len = it;
      const Plan pl = make_plan(&sh, &c, 9, 1, true, Tuning{});
      CHECK(pl.short_prefill && pl.row_groups == 3 && pl.n_splits * 24 > 256 && pl.n_splits * 24 <= 512);
    }
  }
  // prefills of a few tokens: the path that was measured ahead on either side of each bound
  struct ShortCase { int hkv, G, n_new, n; bool paged, split_kv; int rank = 16, d = 128; };
  const ShortCase shorts[] = {
      {8, 4, 4, 9004, false, true},   {8, 4, 8, 9009, false, false},  {8, 4, 8, 33008, false, true},  {8, 4, 8, 33008, true, false},
      {8, 4, 32, 2032, false, true},  {8, 4, 32, 9032, false, false}, {4, 7, 4, 6004, false, false},  {4, 7, 4, 9004, false, true},
      {4, 7, 4, 9004, true, false},   {4, 7, 4, 14004, true, true},   {4, 7, 8, 33008, true, false},  {2, 8, 8, 2008, false, false},
      {2, 8, 8, 9008, false, true},   {2, 8, 8, 9008, true, false},   {2, 8, 8, 14008, true, true},   {2, 8, 16, 2016, false, true},
      {2, 8, 32, 6032, false, true},  {2, 8, 32, 9032, false, false}, {32, 1, 8, 14008, false, false}, {32, 1, 8, 20008, true, true},
      {2, 8, 20, 11020, false, true}, {2, 8, 20, 11020, true, false}, {2, 8, 8, 4008, true, false, 64}, {2, 8, 8, 7008, true, true, 64},
      {2, 8, 20, 11020, true, true, 64}, {2, 8, 28, 20028, true, false, 64}, {4, 7, 8, 4008, true, false, 64}, {4, 7, 8, 11008, true, true, 64},
      {4, 7, 12, 7012, true, false, 64}, {4, 7, 12, 20012, true, true, 48}, {4, 7, 20, 20020, true, false, 64}, {32, 1, 8, 2008, true, false, 64},
      {32, 1, 8, 7008, true, true, 64}, {8, 4, 8, 33008, true, false, 64}, {8, 4, 12, 11012, false, false, 64, 64}, {8, 4, 12, 33012, false, true, 64, 64}};
  for (int it = 0; it < static_cast<int>(sizeof(shorts) / sizeof(shorts[0])); ++it) {
    const ShortCase& t = shorts[it];
    lra_shape sh{};
    sh.n_kv_heads = t.hkv;
    sh.n_q_heads = t.hkv * t.G;
    sh.head_dim = t.d;
    sh.rank = t.rank;
    lra_cache c{};
    c.n_seqs = 1;
    c.max_seq_len = t.n;
    c.kv_token_stride = c.kv_head_stride = t.d;
    c.block_size = t.paged ? 16 : 0;
    c.kv_block_stride = t.paged ? 16 * t.d * t.hkv : 0;
    c.max_blocks_per_seq = c.num_blocks = t.paged ? (t.n + 15) / 16 : 0;
    CHECK(make_plan(&sh, &c, t.n_new, 1, true, Tuning{}).short_prefill == t.split_kv);
  }
  // shares of a tile-walking prefill of a few tokens: about as many as were measured fastest
  struct ShareCase { int hkv, G, d, rank, n_new, n; bool paged; int least, most; };
  const ShareCase share_cases[] = {{8, 4, 128, 64, 6, 306, false, 3, 5}, {8, 4, 128, 16, 6, 306, false, 3, 5}, {2, 8, 128, 64, 6, 206, true, 4, 4},
                                   {8, 4, 64, 16, 6, 506, true, 6, 8},   {4, 7, 128, 32, 10, 224, false, 3, 4}, {8, 4, 128, 16, 24, 142, false, 1, 1}};
  for (int it = 0; it < static_cast<int>(sizeof(share_cases) / sizeof(share_cases[0])); ++it) {
    const ShareCase& t = share_cases[it];
    lra_shape sh{};
    sh.n_kv_heads = t.hkv;
    sh.n_q_heads = t.hkv * t.G;
    sh.head_dim = t.d;
    sh.rank = t.rank;
    lra_cache c{};
    c.n_seqs = 1;
    c.max_seq_len = t.n;
    c.kv_token_stride = c.kv_head_stride = t.d;
    c.block_size = t.paged ? 16 : 0;
    c.kv_block_stride = t.paged ? 16 * t.d * t.hkv : 0;
    c.max_blocks_per_seq = c.num_blocks = t.paged ? (t.n + 15) / 16 : 0;
    const Plan pl = make_plan(&sh, &c, t.n_new, 1, true, Tuning{});
    CHECK(!pl.short_prefill && pl.n_splits >= t.least && pl.n_splits <= t.most);
  }
  // batches: shares in one row where that balances what the other grid does not (row: with the lengths known, blind: without)
  auto many = [](int first, int n, int rest) {
    std::vector<int32_t> v(static_cast<size_t>(n), rest);
    v[0] = first;
    return v;
  };
  auto spread = [](int n, int lo, int hi) {
    std::vector<int32_t> v;
    for (int i = 0; i < n; ++i) v.push_back(lo + static_cast<int>(static_cast<int64_t>(hi - lo) * ((i * 37) % n) / (n - 1)));
    return v;
  };
  struct BatchCase { std::vector<int32_t> lens; int hkv, G, queries; bool row, blind; float theta; };
  const BatchCase batch_cases[] = {
      {{65536, 4096, 30000, 9000}, 4, 7, 4, true, true, 0.f}, {{20000, 20000, 20000, 20000}, 8, 4, 4, false, true, 0.f},
      {{7000, 3000, 5000, 2000}, 8, 4, 4, true, true, 0.f},   {{900, 300}, 8, 4, 1, false, false, 0.f},
      {{2048, 1100, 700}, 8, 4, 4, false, false, 1e4f},       {{20480, 11000, 7000}, 8, 4, 4, true, true, 1e4f},
      // one long sequence among many: a common share size would leave it whole
      {many(65536, 16, 2000), 32, 1, 2, false, false, 0.f},   {many(65536, 64, 500), 8, 4, 2, false, false, 0.f},
      {many(65536, 32, 2000), 8, 4, 16, false, false, 0.f},   {many(65536, 64, 500), 4, 7, 8, false, false, 0.f},
      {many(20000, 32, 2000), 8, 4, 4, false, false, 1e4f},   {many(40000, 32, 300), 8, 4, 2, false, true, 0.f},
      // hardly more places than sequences, several per sequence
      {spread(56, 2000, 20000), 8, 4, 4, false, false, 0.f},  {spread(64, 2000, 20000), 8, 4, 1, false, false, 0.f},
      {spread(24, 2000, 36000), 8, 4, 4, true, true, 0.f},    {spread(64, 2000, 20000), 2, 8, 4, true, true, 0.f},
      {spread(12, 2000, 40000), 32, 1, 4, false, false, 0.f}, {spread(12, 2000, 40000), 8, 4, 16, true, true, 0.f},
      // rotary, several row groups: four, uneven; three, even; three with places enough
      {spread(11, 4000, 33000), 8, 4, 8, false, false, 1e4f}, {spread(10, 32000, 38000), 8, 4, 6, true, false, 1e4f},
      {spread(4, 3000, 17000), 8, 4, 6, true, true, 1e4f},
      // in place at once
      {{670, 500, 520, 530}, 2, 8, 9, false, false, 0.f},     {{6000, 5600, 5700}, 2, 8, 9, true, true, 0.f}};
  for (int it = 0; it < static_cast<int>(sizeof(batch_cases) / sizeof(batch_cases[0])); ++it) {
    const BatchCase& t = batch_cases[it];
    lra_shape sh{};
    sh.n_kv_heads = t.hkv;
    sh.n_q_heads = t.hkv * t.G;
    sh.head_dim = 128;
    sh.rank = 24;
    sh.key_rope_theta = t.theta;
    lra_cache c{};
    c.n_seqs = static_cast<int32_t>(t.lens.size());
    c.block_size = 16;
    c.kv_token_stride = 128;
    c.kv_head_stride = 16 * 128;
    c.kv_block_stride = 16 * 128 * t.hkv;
    c.seq_lens_host = t.lens.data();
    for (int32_t n : t.lens) c.max_seq_len = n > c.max_seq_len ? n : c.max_seq_len;
    c.num_blocks = c.max_blocks_per_seq = (c.max_seq_len + 15) / 16;
    const Plan pl = make_plan(&sh, &c, t.queries * c.n_seqs, t.queries, false, Tuning{});
    CHECK((pl.batch_wgs > 0) == t.row);
    c.seq_lens_host = nullptr;
    const Plan blind = make_plan(&sh, &c, t.queries * c.n_seqs, t.queries, false, Tuning{});
    CHECK((blind.batch_wgs > 0) == t.blind && blind.batch_tiles == 0 && blind.bytes >= pl.bytes);
    if (!t.row) continue;
    int64_t shares = 0, fewer = 0;
    for (int32_t n : t.lens) {
      shares += ((n + 127) / 128 + pl.batch_tiles - 1) / pl.batch_tiles;
      if (pl.batch_tiles > 1) fewer += ((n + 127) / 128 + pl.batch_tiles - 2) / (pl.batch_tiles - 1);
    }
    CHECK(shares <= pl.batch_wgs && (fewer == 0 || fewer > pl.batch_wgs || pl.batch_tiles == pl.batch_min_tiles));
    Tuning other;
    other.variant = 2;
    CHECK(make_plan(&sh, &c, t.queries * c.n_seqs, t.queries, false, other).batch_wgs == 0);
  }
  // prefills whose waves divide the keys: either side of the measured lines
  struct WaveCase { int hkv, G, rank, n_new, n; bool waves; float theta; };
  const WaveCase wave_cases[] = {
      {8, 4, 16, 62, 525, true, 0.f},    {8, 4, 16, 64, 2048, true, 0.f},   {8, 4, 16, 64, 2049, false, 0.f}, {8, 4, 16, 256, 8192, true, 0.f},
      {8, 4, 16, 256, 8193, false, 0.f}, {8, 4, 16, 257, 512, false, 0.f},  {8, 4, 24, 257, 512, true, 0.f},  {8, 4, 24, 257, 2048, true, 0.f},
      {8, 4, 24, 257, 2049, false, 0.f}, {8, 4, 24, 512, 5120, true, 0.f},  {8, 4, 16, 513, 2000, false, 0.f}, {8, 4, 64, 62, 525, false, 0.f},
      {8, 4, 16, 62, 525, true, 1e4f},   {8, 4, 16, 8, 384, false, 1e4f},   {32, 1, 16, 64, 1280, true, 0.f}, {32, 1, 16, 64, 1281, false, 0.f},
      // two rounds at ranks up to 16
      {8, 4, 16, 433, 512, false, 0.f},  {8, 4, 16, 448, 512, true, 0.f},   {8, 4, 16, 257, 1536, true, 0.f}, {8, 4, 16, 257, 1537, false, 0.f},
      {8, 4, 16, 320, 2048, true, 0.f},  {8, 4, 16, 312, 2048, false, 0.f}, {8, 4, 16, 384, 3328, true, 0.f}, {8, 4, 24, 384, 3329, false, 0.f},
      {8, 4, 16, 512, 3584, true, 0.f},  {8, 4, 16, 512, 3585, false, 0.f},
      {8, 8, 8, 248, 360, true, 0.f},    {8, 8, 8, 248, 360, false, 1e4f},  {8, 8, 24, 248, 360, true, 1e4f},
      // the split-KV path's sizes
      {8, 4, 16, 8, 384, true, 0.f},     {8, 4, 16, 8, 385, false, 0.f},    {32, 1, 16, 8, 512, true, 0.f},   {32, 1, 16, 8, 513, false, 0.f},
      {32, 1, 16, 6, 384, true, 0.f},    {32, 1, 16, 6, 385, false, 0.f},
      {8, 4, 16, 9, 640, true, 0.f},     {8, 4, 16, 9, 641, false, 0.f},    {8, 4, 16, 17, 768, true, 0.f},   {8, 4, 16, 17, 769, false, 0.f},
      {8, 4, 16, 32, 1024, true, 0.f},   {8, 4, 16, 32, 1025, false, 0.f},  {4, 7, 16, 5, 512, true, 0.f},    {4, 7, 16, 5, 513, false, 0.f},
      {2, 8, 16, 24, 768, true, 0.f},    {2, 8, 16, 24, 769, false, 0.f},   {2, 8, 16, 32, 1024, true, 0.f},  {2, 8, 16, 32, 1025, false, 0.f}};
  for (int it = 0; it < static_cast<int>(sizeof(wave_cases) / sizeof(wave_cases[0])); ++it) {
    const WaveCase& t = wave_cases[it];
    lra_shape sh{};
    sh.n_kv_heads = t.hkv;
    sh.n_q_heads = t.hkv * t.G;
    sh.head_dim = 128;
    sh.rank = t.rank;
    sh.key_rope_theta = t.theta;
    lra_cache c{};
    c.n_seqs = 1;
    c.max_seq_len = t.n;
    c.kv_token_stride = t.hkv * 128;
    c.kv_head_stride = 128;
    CHECK(make_plan(&sh, &c, t.n_new, 1, true, resolve_tuning(nullptr)).wave_rows == t.waves);
    lra_tuning forced{};
    forced.kernel_variant = 2;
    CHECK(!make_plan(&sh, &c, t.n_new, 1, true, resolve_tuning(&forced)).wave_rows);
    lra_tuning keys{};  // key shares asked for: the path that takes them
    keys.decode_split_keys = 128;
    const Plan split = make_plan(&sh, &c, t.n_new, 1, true, resolve_tuning(&keys));
    CHECK(!split.wave_rows && split.wave_shares == 0 && (!split.short_prefill || split.split_keys == 128));
    lra_tuning many{};
    many.short_prefill = 64;
    CHECK(!make_plan(&sh, &c, t.n_new, 1, true, resolve_tuning(&many)).wave_rows);
  }
  // ... with shares: either side of the measured lines
  struct WaveShareCase { int hkv, G, d, rank, n_new, n, shares; float theta; };
  const WaveShareCase wave_share_cases[] = {
      {8, 4, 128, 16, 8, 9009, 0, 0.f},    {32, 1, 128, 16, 16, 9009, 8, 0.f},  {32, 1, 128, 16, 4, 9009, 0, 0.f},    {32, 1, 128, 16, 5, 2047, 0, 0.f},
      {32, 1, 128, 16, 5, 16385, 0, 0.f},  {8, 4, 128, 16, 48, 1800, 5, 0.f},   {8, 4, 128, 16, 48, 1799, 0, 0.f},   {8, 4, 128, 16, 32, 2880, 0, 0.f},    {8, 4, 128, 16, 64, 2880, 4, 0.f},
      {8, 4, 128, 16, 64, 6144, 4, 0.f},   {8, 4, 128, 16, 64, 6145, 0, 0.f},   {8, 4, 128, 32, 33, 18432, 6, 0.f},   {8, 4, 128, 32, 33, 18433, 0, 0.f},
      {8, 4, 128, 64, 64, 2880, 0, 0.f},   {8, 4, 128, 16, 129, 5000, 0, 0.f},  {32, 1, 128, 16, 64, 4096, 4, 0.f},   {32, 1, 128, 16, 64, 4097, 0, 0.f},
      {8, 4, 128, 16, 33, 4000, 6, 1e4f},  {8, 4, 128, 16, 16, 9000, 0, 1e4f}};
  for (int it = 0; it < static_cast<int>(sizeof(wave_share_cases) / sizeof(wave_share_cases[0])); ++it) {
    const WaveShareCase& t = wave_share_cases[it];
    lra_shape sh{};
    sh.n_kv_heads = t.hkv;
    sh.n_q_heads = t.hkv * t.G;
    sh.head_dim = t.d;
    sh.rank = t.rank;
    sh.key_rope_theta = t.theta;
    lra_cache c{};
    c.n_seqs = 1;
    c.max_seq_len = t.n;
    c.kv_token_stride = t.hkv * t.d;
    c.kv_head_stride = t.d;
    const Plan pl = make_plan(&sh, &c, t.n_new, 1, true, resolve_tuning(nullptr));
    CHECK(pl.wave_shares == t.shares);
  }
  // the split of lra_cache_append over d_model
  for (int it = 0; it < cases; ++it) {
    const int64_t n_new = pick({1, 16, 32, 33, 64, 100, 128, 129, 512, 1000, 1024, 4096, 1 << 20, (1 << 20) + 1, INT32_MAX});
    const int hkv = static_cast<int>(pick({1, 2, 3, 8, 64, 4096}));
    const int d = static_cast<int>(pick({64, 128}));
    const int r = static_cast<int>(pick({8, 16, 24, 64}));
    const int dm = static_cast<int>(pick({64, 128, 704, 768, 1024, 4096, 8192, 1 << 20}));
    lra_tuning t{};
    t.append_k_splits = static_cast<int32_t>(pick({0, 0, 1, 2, 3, 8, 16, 17, -1}));
    t.append_tile = static_cast<int32_t>(pick({0, 0, 0, 64, 128}));
    t.append_stages = static_cast<int32_t>(pick({0, 0, 0, 3}));
    const Tuning tune = resolve_tuning(&t);
    if (append_quarter_tiles(static_cast<int>(n_new), hkv, d, r, dm, tune)) {  // one round, whole steps, a place for every L block
      const int64_t ft = 2LL * hkv * d / 64, tiles = (n_new + 63) / 64 * ft;
      CHECK(n_new > tune.append_skinny && tiles <= 256 && dm % 128 == 0 && ft >= 4 * ((r + 15) / 16));
      CHECK(tune.append_tile == 0 && tune.append_stages == 0 && tune.append_k_splits <= 1);
    }
    const AppendSplit sp = plan_append_split(static_cast<int>(n_new), hkv, d, r, dm, tune);
    CHECK(sp.k_splits >= 1 && sp.k_splits <= 16 && (sp.bt == 64 || sp.bt == 128));
    CHECK((sp.k_splits == 1) == (sp.bytes == 0));
    if (sp.k_splits > 1) {
      const int64_t n_feat = 2LL * hkv * d + r;
      CHECK((dm / 64) % sp.k_splits == 0 && n_new <= (1 << 20));
      CHECK(sp.bytes >= static_cast<size_t>(sp.k_splits) * n_new * n_feat * 4 && sp.bytes % 256 == 0);
      CHECK(tune.append_tile == 0 && tune.append_stages == 0 && tune.append_k_splits != 1);
      if (tune.append_k_splits == 0) {
        const int64_t tiles = (n_new + sp.bt - 1) / sp.bt * (2 * ((static_cast<int64_t>(hkv) * d + 127) / 128) + 1);
        CHECK(tiles * sp.k_splits <= kCUs && dm / 64 / sp.k_splits >= 4 && n_new > 32 && sp.bt == 64);
      }
    }
  }
  // 64 x 64 tiles: either side of the measured lines (kv heads, d, rank, d_model, new tokens)
  const struct { int hkv, d, r, dm, n_new; bool quarter; } quarter_cases[] = {
      {8, 128, 16, 4096, 321, true}, {8, 128, 16, 4096, 320, false}, {8, 128, 16, 4096, 512, true}, {8, 128, 16, 4096, 513, false},
      {8, 64, 64, 2048, 321, true},  {8, 64, 64, 2048, 320, false},  {2, 128, 32, 2048, 1728, true}, {2, 128, 32, 2048, 1729, false},
      {2, 128, 40, 2048, 1000, false}, {4, 64, 16, 1088, 700, false}, {4, 64, 16, 1024, 65, false}, {8, 128, 16, 256, 64, false}, {8, 128, 16, 256, 65, true},
      {12, 128, 16, 2048, 95, false}, {12, 128, 16, 2048, 96, true}, {32, 128, 16, 4096, 65, true}};
  for (int it = 0; it < static_cast<int>(sizeof(quarter_cases) / sizeof(quarter_cases[0])); ++it) {
    const auto& t = quarter_cases[it];
    CHECK(append_quarter_tiles(t.n_new, t.hkv, t.d, t.r, t.dm, resolve_tuning(nullptr)) == t.quarter);
  }
  if (uneven < cases / 100) {
    std::fprintf(stderr, "plan_fuzz: %d plans with shares of two sizes\n", uneven);
    return 1;
  }
  std::printf("plan_fuzz: %d cases, %d accepted by the argument checks, all plans consistent\n", cases, accepted);
  return accepted > cases / 10 ? 0 : 2;
}
