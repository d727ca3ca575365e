"""Parity of the cache-append producer (lra_cache_append) against the fp64 oracle, through
the C ABI.  Bar as for the attention calls: relative L2 <= 5e-3 over every written tensor
and over every token, max-abs <= 2e-2 (outputs are O(1): x ~ N(0,1), w ~ N(0, 1/d_model))."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_01053_amd as lra
from tests.harness import MAX_ABS_TOL, REL_L2_TOL, errors

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
SENTINEL = 7.0   # value of every cache element before the call: rows that are not appended must keep it


def _inputs(seed, n_new, d_model, hkv, d, r):
    gen = torch.Generator().manual_seed(seed)
    x = torch.randn(n_new, d_model, generator=gen).to(torch.bfloat16)
    w = (torch.randn(2 * hkv * d + r, d_model, generator=gen) / d_model ** 0.5).to(torch.bfloat16)
    return x, w


def _gate(got, ref, label):
    rel, mx = errors(got, ref)
    print(f"{label}: relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL, (label, rel, mx)


CASES = [
    # n (after the append), n_new, d_model, Hkv, d, r, rope_theta
    (1, 1, 64, 1, 64, 8, 10000.0),
    (200, 129, 256, 2, 128, 16, 500000.0),      # ragged token tile
    (300, 300, 512, 3, 64, 24, 10000.0),        # no old rows; Hkv*d = 192: a partly filled feature tile
    (70000, 130, 1024, 8, 128, 16, 500000.0),   # positions in the tens of thousands
    (513, 257, 4096, 8, 128, 64, 0.0),          # Llama-3-8B projection shape, keys stored unrotated
    (1000, 512, 1024, 4, 128, 32, 500000.0),
]


# few new tokens: the weight-streaming kernel (and, with it switched off, the tiled one on the same inputs)
SMALL = [
    (1, 1, 64, 1, 64, 8, 10000.0),
    (4097, 1, 4096, 8, 128, 16, 500000.0),     # a decode step at the Llama-3-8B shape
    (9, 2, 192, 2, 64, 8, 10000.0),
    (9, 1, 192, 2, 64, 8, 10000.0),            # matrix-vector kernel, d_model/8 = 24 pieces: lanes without one
    (19, 1, 1088, 2, 128, 24, 500000.0),       # ... 136 pieces: a third piece on some lanes
    (300, 1, 4160, 3, 128, 16, 10000.0),       # ... 520 pieces: a second round of eight per lane, of one
    (20, 1, 128, 2, 64, 8, 0.0),               # ... unrotated keys
    (31, 3, 1088, 2, 128, 24, 500000.0),
    (40000, 4, 4096, 8, 128, 16, 500000.0),
    (50, 7, 320, 2, 64, 24, 10000.0),          # five pieces of d_model over 8 waves
    (100, 16, 512, 2, 128, 16, 500000.0),
    (100, 17, 512, 2, 128, 40, 500000.0),
    (65000, 33, 1024, 4, 128, 16, 500000.0),
    (64, 64, 768, 3, 64, 64, 10000.0),
    (300, 150, 512, 2, 128, 16, 500000.0),     # beyond the default limit: runs streamed only when the limit is raised
    (20, 3, 128, 2, 64, 8, 0.0),               # unrotated keys
    (40, 12, 256, 2, 128, 16, 0.0),
]


@pytest.mark.parametrize("skinny", [0, 64, 1 << 30], ids=["tiled", "default", "streamed"])
@pytest.mark.parametrize("case", SMALL, ids=lambda c: "n%d_new%d_dm%d_hkv%d_d%d_r%d_th%g" % c)
def test_append_few_tokens(case, skinny):
    prev = lra.lra_set_append_skinny(skinny)
    try:
        test_append_contiguous(case)
    finally:
        lra.lra_set_append_skinny(prev)


@pytest.mark.parametrize("stages", [2, 3, 4])
@pytest.mark.parametrize("case", [SMALL[0], (200, 129, 256, 2, 128, 16, 500000.0), (700, 300, 704, 3, 64, 24, 10000.0)],
                         ids=lambda c: "n%d_new%d_dm%d_hkv%d_d%d_r%d_th%g" % c)
def test_append_tiled_stage_counts(case, stages):
    """The tiled GEMM with 2, 3 and 4 LDS stages (d_model of 1, 4 and 11 steps: shorter than the ring, and ragged against it)."""
    prev_s, prev_k = lra.lra_set_append_stages(stages), lra.lra_set_append_skinny(0)
    try:
        test_append_contiguous(case)
    finally:
        lra.lra_set_append_stages(prev_s)
        lra.lra_set_append_skinny(prev_k)


@pytest.mark.parametrize("case", [SMALL[0], (200, 129, 256, 2, 128, 16, 500000.0), (700, 300, 704, 3, 64, 24, 10000.0),
                                  (66000, 515, 1024, 8, 128, 64, 500000.0), (520, 520, 512, 1, 64, 8, 10000.0),
                                  (1000, 257, 4096, 8, 128, 16, 0.0)],
                         ids=lambda c: "n%d_new%d_dm%d_hkv%d_d%d_r%d_th%g" % c)
@pytest.mark.parametrize("tile", [64, 128, 256])
def test_append_tile_sizes(case, tile):
    """Every tile size of the GEMM kernels, forced: ragged token tiles, feature regions of 64, 192 and 1024
    (a tile that is partly filled, one that straddles the K and V rows of w), rank 8 to 64.  Regions of up to 256
    features have no 256-wide form: asked for it, they run on the automatic choice."""
    prev_t, prev_k = lra.lra_set_append_tile(tile), lra.lra_set_append_skinny(0)
    try:
        test_append_contiguous(case)
    finally:
        lra.lra_set_append_tile(prev_t)
        lra.lra_set_append_skinny(prev_k)


WIDE_CASES = [
    # the 256 x 256 tiles need K and V regions of more than 256 features; their feature tiles divide the L features
    (300, 300, 64, 4, 128, 8, 10000.0),        # one step of d_model; four feature tiles: two token blocks each, ragged tokens
    (900, 515, 192, 5, 64, 40, 500000.0),      # region of 320: a partly filled tile; rank 40: two blocks of L rows
    (2200, 2100, 128, 5, 128, 64, 0.0),        # six feature tiles (blocks 6 and 7 on the first two), nine token tiles
    (1000, 257, 256, 16, 128, 32, 10000.0),    # sixteen feature tiles: eight of them without L features
]


@pytest.mark.parametrize("case", WIDE_CASES, ids=lambda c: "n%d_new%d_dm%d_hkv%d_d%d_r%d_th%g" % c)
def test_append_wide_tiles(case):
    prev_t, prev_k = lra.lra_set_append_tile(256), lra.lra_set_append_skinny(0)
    try:
        test_append_contiguous(case)
    finally:
        lra.lra_set_append_tile(prev_t)
        lra.lra_set_append_skinny(prev_k)


ORDER_CASES = [
    # 128-token tiles, two stages: the orders in which the tiles are dealt out (three feature tiles here)
    (600, 512, 64, 1, 64, 8, 10000.0),          # four token tiles, one round: the plain order
    (700, 513, 64, 1, 64, 16, 10000.0),         # five: a stretch per XCD, L tiles on five of them
    (30000, 22528, 64, 1, 64, 8, 10000.0),      # 176 token tiles, above a round: the plain order (a multiple of 8)
    (30000, 22529, 64, 1, 64, 8, 0.0),          # 177: stretches
    (44100, 44032, 64, 1, 64, 8, 10000.0),      # 344 token tiles, above two rounds: stretches
    (100, 100, 128, 5, 128, 24, 10000.0),       # fewer tokens than features
]


@pytest.mark.parametrize("case", ORDER_CASES, ids=lambda c: "n%d_new%d_dm%d_hkv%d_d%d_r%d_th%g" % c)
def test_append_tile_orders(case):
    prev_t, prev_s, prev_k = lra.lra_set_append_tile(128), lra.lra_set_append_stages(2), lra.lra_set_append_skinny(0)
    try:
        test_append_contiguous(case)
    finally:
        lra.lra_set_append_tile(prev_t)
        lra.lra_set_append_stages(prev_s)
        lra.lra_set_append_skinny(prev_k)


GUARD = 4096  # bytes of a bit pattern on either side of a workspace


def _guarded_workspace(nbytes):
    """A 256-byte aligned workspace of nbytes between two guard bands; returns (workspace view, whole buffer)."""
    whole = torch.full((nbytes + 2 * GUARD,), 0xA5, dtype=torch.uint8, device=DEV)
    return whole[GUARD:GUARD + nbytes], whole


def _guards_intact(whole):
    return bool((whole[:GUARD] == 0xA5).all()) and bool((whole[-GUARD:] == 0xA5).all())


@pytest.mark.parametrize("case", CASES, ids=lambda c: "n%d_new%d_dm%d_hkv%d_d%d_r%d_th%g" % c)
def test_append_contiguous(case):
    _append_contiguous(case, False)


def _append_contiguous(case, with_workspace):
    """Runs one append on a contiguous cache against the oracle; returns the workspace bytes the library asked for."""
    n, n_new, d_model, hkv, d, r, theta = case
    x, w = _inputs(5000 + n + n_new, n_new, d_model, hkv, d, r)
    k_base = torch.full((n, hkv, d), SENTINEL, dtype=torch.bfloat16, device=DEV)
    v_base = torch.full_like(k_base, SENTINEL)
    l = torch.full((n, r), SENTINEL, dtype=torch.bfloat16, device=DEV)
    seq_lens = torch.tensor([n], dtype=torch.int32, device=DEV)
    q_like = torch.empty(1, hkv, d, dtype=torch.bfloat16, device=DEV)
    shape = lra.make_shape(q_like, hkv, r, 0.0)
    cache = lra.make_cache(k_base, v_base, l, seq_lens, n, None)
    xd, wd = x.to(DEV), w.to(DEV)
    need = 0
    if with_workspace:
        need = lra.lra_append_workspace_bytes(shape, cache, wd, theta, n_new)
        ws, whole = _guarded_workspace(max(need, 256))
        lra.lra_cache_append(shape, cache, wd, theta, xd, 0, workspace=ws)
    else:
        lra.lra_cache_append(shape, cache, wd, theta, xd, 0)
    torch.cuda.synchronize()
    if with_workspace:
        assert _guards_intact(whole)
    f = lambda t: t.to(torch.float64).cpu().numpy()
    pos = np.arange(n - n_new, n)
    k_ref, v_ref, l_ref = oracle.project_new_tokens(f(x), f(w), hkv, d, r, pos, theta)
    _gate(f(k_base)[n - n_new:], k_ref, "K rows")
    _gate(f(v_base)[n - n_new:], v_ref, "V rows")
    _gate(f(l)[n - n_new:], l_ref, "L rows")
    for t in (k_base, v_base, l):   # older rows untouched
        assert bool((t[:n - n_new] == SENTINEL).all())
    return need


SPLIT_CASES = [
    # n, n_new, d_model, Hkv, d, r, theta, parts the automatic choice takes (0: it keeps one kernel)
    (100, 17, 512, 2, 128, 16, 500000.0, 0),        # up to 32 tokens: the weight-streaming kernel
    (200, 40, 512, 2, 128, 16, 500000.0, 2),        # told a size, and streamed: x is small
    (65000, 33, 1024, 4, 128, 16, 500000.0, 4),     # ... likewise
    (64, 64, 768, 3, 64, 64, 10000.0, 2),           # ... likewise
    (200, 65, 512, 2, 128, 16, 500000.0, 2),        # 8 steps of d_model: two parts of four
    (200, 65, 768, 3, 64, 64, 10000.0, 2),          # 12 steps: two parts of six; 64 wide
    (90, 90, 1280, 5, 64, 24, 500000.0, 4),         # 20 steps: four parts of five
    (300, 64, 4096, 2, 64, 8, 0.0, 16),             # x beyond 416 KB: sixteen parts of four
    (70, 33, 2048, 15, 128, 16, 10000.0, 8),        # more features than one workgroup per unit has
    (200, 129, 256, 2, 128, 16, 500000.0, 0),       # 4 steps: too short to divide
    (700, 300, 704, 3, 64, 24, 10000.0, 0),         # 11 steps: no part count divides them
    (513, 257, 4096, 8, 128, 64, 0.0, 2),           # Llama-3-8B projection shape, r = 64, unrotated keys
    (1000, 512, 1024, 4, 128, 32, 500000.0, 2),
    (4300, 100, 4096, 8, 128, 16, 500000.0, 4),     # Llama-3-8B shape, a trace-sized chunk
    (40000, 400, 4096, 8, 128, 16, 500000.0, 2),    # ... a chunk that asks for the parts and runs on 64 x 64 tiles, as the row above
    (40000, 320, 4096, 8, 128, 16, 500000.0, 2),    # ... the largest that still divides
    (1000, 128, 1024, 4, 128, 32, 500000.0, 4),
    (40000, 1000, 4096, 8, 128, 16, 500000.0, 0),   # more than half a chip of tiles: one kernel
    (2048, 2048, 4096, 8, 128, 16, 500000.0, 0),    # enough tiles for the chip: one kernel
    (31, 16, 4096, 8, 128, 16, 500000.0, 0),        # few tokens: the weight-streaming kernel
]


@pytest.mark.parametrize("case", SPLIT_CASES, ids=lambda c: "n%d_new%d_dm%d_hkv%d_d%d_r%d_th%g_auto%d" % c)
def test_append_split_over_d_model_automatic(case):
    """lra_cache_append with a workspace: mid-sized chunks divide d_model among several workgroups per output
    tile and finish in a second kernel.  Same oracle, same gate, guard bands around the workspace intact, and
    the workspace asked for is the size of the parts the automatic choice takes."""
    *plain, parts = case
    n, n_new, d_model, hkv, d, r, theta = plain
    need = _append_contiguous(tuple(plain), True)
    expect = parts * n_new * (2 * hkv * d + r) * 4 if parts else 0
    assert need == (expect + 255) // 256 * 256


@pytest.mark.parametrize("parts", [2, 4, 16])
@pytest.mark.parametrize("case", [(200, 129, 256, 2, 128, 16, 500000.0), (5000, 40, 1024, 2, 64, 8, 10000.0),
                                  (513, 257, 4096, 8, 128, 64, 0.0), (300, 300, 512, 3, 64, 24, 10000.0)],
                         ids=lambda c: "n%d_new%d_dm%d_hkv%d_d%d_r%d_th%g" % c)
def test_append_split_over_d_model_forced(case, parts):
    """Part counts forced through the tuning struct, down to one step of d_model per part; counts that do not
    divide the steps leave the call on one kernel (and the workspace request at 0)."""
    prev = lra.lra_set_append_k_splits(parts)
    try:
        need = _append_contiguous(case, True)
    finally:
        lra.lra_set_append_k_splits(prev)
    n, n_new, d_model, hkv, d, r, theta = case
    divides = (d_model // 64) % parts == 0
    assert (need > 0) == divides


@pytest.mark.parametrize("skinny,tile,parts", [(0, 64, 0), (0, 128, 0), (0, 256, 0), (1 << 30, 0, 0), (64, 0, 2), (64, 0, 8)],
                         ids=["tile64", "tiled", "wide", "streamed", "two_parts", "eight_parts"])
def test_append_paged_then_attend(skinny, tile, parts):
    prev, prev_t, prev_p = lra.lra_set_append_skinny(skinny), lra.lra_set_append_tile(tile), lra.lra_set_append_k_splits(parts)
    try:
        _paged_then_attend(parts > 1, hkv=4 if tile == 256 else 2)  # (the 256-wide tiles need more than 256 features)
    finally:
        lra.lra_set_append_skinny(prev)
        lra.lra_set_append_tile(prev_t)
        lra.lra_set_append_k_splits(prev_p)


def _paged_then_attend(with_workspace=False, hkv=2):
    """Appends to two sequences of a paged cache (a last block that is partly filled, blocks in
    permuted order), checks the written rows and that nothing else moved, then runs the
    attention prefill on the appended tokens and compares it with the oracle evaluated on
    the cache the producer wrote."""
    hq, d, r, d_model, theta = 8, 128, 16, 512, 500000.0
    seq_lens = [77, 300]
    n_new = [30, 130]
    bs, max_blocks = 16, 20
    num_blocks = 45
    gen = torch.Generator().manual_seed(6001)
    perm = torch.randperm(num_blocks, generator=gen).to(torch.int32)
    table = torch.stack([perm[:max_blocks], perm[max_blocks:2 * max_blocks]])
    k_pool = torch.randn(num_blocks, hkv, bs, d, generator=gen).to(torch.bfloat16)
    v_pool = torch.randn(num_blocks, hkv, bs, d, generator=gen).to(torch.bfloat16)
    l_pool = torch.randn(num_blocks, bs, r, generator=gen).to(torch.bfloat16)
    kd, vd, ld = k_pool.to(DEV), v_pool.to(DEV), l_pool.to(DEV)
    lens_d = torch.tensor(seq_lens, dtype=torch.int32, device=DEV)
    table_d = table.to(DEV)
    q_like = torch.empty(1, hq, d, dtype=torch.bfloat16, device=DEV)
    shape = lra.make_shape(q_like, hkv, r, 0.0)
    cache = lra.make_cache(kd, vd, ld, lens_d, max(seq_lens), table_d)
    f = lambda t: t.to(torch.float64).cpu().numpy()
    k_exp, v_exp, l_exp = f(k_pool).copy(), f(v_pool).copy(), f(l_pool).copy()
    w = None
    for s in range(2):
        x, w = _inputs(6100 + s, n_new[s], d_model, hkv, d, r)
        if with_workspace:
            wd = w.to(DEV)
            need = lra.lra_append_workspace_bytes(shape, cache, wd, theta, n_new[s])
            assert need > 0
            ws, whole = _guarded_workspace(need)
            lra.lra_cache_append(shape, cache, wd, theta, x.to(DEV), s, workspace=ws)
            torch.cuda.synchronize()
            assert _guards_intact(whole)
        else:
            lra.lra_cache_append(shape, cache, w.to(DEV), theta, x.to(DEV), s)
        torch.cuda.synchronize()
        pos = np.arange(seq_lens[s] - n_new[s], seq_lens[s])
        k_ref, v_ref, l_ref = oracle.project_new_tokens(f(x), f(w), hkv, d, r, pos, theta)
        ids = table[s].numpy()
        got_k = oracle.gather_paged(f(kd), ids, seq_lens[s])[seq_lens[s] - n_new[s]:]
        got_v = oracle.gather_paged(f(vd), ids, seq_lens[s])[seq_lens[s] - n_new[s]:]
        got_l = oracle.lra_oracle.gather_paged_l(f(ld), ids, seq_lens[s])[seq_lens[s] - n_new[s]:]
        _gate(got_k, k_ref, f"paged K rows seq {s}")
        _gate(got_v, v_ref, f"paged V rows seq {s}")
        _gate(got_l, l_ref, f"paged L rows seq {s}")
        # everything except the appended rows is bit-identical to before
        oracle.scatter_paged(k_exp, ids, seq_lens[s] - n_new[s], got_k)
        oracle.scatter_paged(v_exp, ids, seq_lens[s] - n_new[s], got_v)
        oracle.scatter_paged_l(l_exp, ids, seq_lens[s] - n_new[s], got_l)
        np.testing.assert_array_equal(f(kd), k_exp)
        np.testing.assert_array_equal(f(vd), v_exp)
        np.testing.assert_array_equal(f(ld), l_exp)
    # attention over the cache the producer wrote (sequence 1, its 130 new tokens)
    s = 1
    gen = torch.Generator().manual_seed(6200)
    q = torch.randn(n_new[s], hq, d, generator=gen).to(torch.bfloat16)
    b_k = (0.05 * torch.randn(2, r, hkv * d, generator=gen)).to(torch.bfloat16)
    b_v = (0.05 * torch.randn(2, r, hkv * d, generator=gen)).to(torch.bfloat16)
    qd = q.to(DEV)
    out = torch.full_like(qd, float("nan"))
    ws = torch.empty(max(lra.lra_workspace_bytes(shape, cache, 1, 1, n_new[s]), 256), dtype=torch.uint8, device=DEV)
    lra.lra_attn_prefill(shape, cache, b_k.to(DEV), b_v.to(DEV), 2, qd, s, 1, out, ws)
    torch.cuda.synchronize()
    ids = table[s].numpy()
    kb = oracle.gather_paged(f(kd), ids, seq_lens[s])
    vb = oracle.gather_paged(f(vd), ids, seq_lens[s])
    lr = oracle.lra_oracle.gather_paged_l(f(ld), ids, seq_lens[s])
    ref = oracle.prefill(f(q), kb, vb, lr, f(b_k[1]), f(b_v[1]), n=seq_lens[s], scale=1.0 / d ** 0.5)
    _gate(f(out), ref, "attention over the appended cache")


PAGED_WIDE_CASES = [
    # lengths and new tokens of two sequences, d_model, Hkv, d, r: 256 x 256 tiles on paged caches
    ([300, 77], [300, 5], 64, 4, 128, 8),          # four feature tiles of one step: two token blocks of L each; a second tile of 44 tokens
    ([70, 900], [1, 515], 192, 5, 64, 40),         # a feature tile filled in part, two blocks of L rows, three token tiles
    ([257, 1100], [256, 1000], 128, 8, 64, 64),    # exactly one token tile; a ragged last block
    ([513, 40], [511, 40], 256, 6, 128, 24),       # six feature tiles: the first two take token blocks 6 and 7 too
]


@pytest.mark.parametrize("case", PAGED_WIDE_CASES, ids=lambda c: "n%d_new%d_n%d_new%d_dm%d_hkv%d_d%d_r%d" % (c[0][0], c[1][0], c[0][1], c[1][1], *c[2:]))
def test_append_wide_tiles_on_paged_caches(case):
    """The rows of K, V and L land in their blocks, and every other byte of the pools stays what it was."""
    lens, n_new, d_model, hkv, d, r = case
    blocks = [(n + 15) // 16 for n in lens]
    gen = torch.Generator().manual_seed(6500 + lens[0])
    num_blocks = sum(blocks) + 3
    perm = torch.randperm(num_blocks, generator=gen).to(torch.int32)
    table = torch.full((2, max(blocks)), -1, dtype=torch.int32)
    table[0, :blocks[0]], table[1, :blocks[1]] = perm[:blocks[0]], perm[blocks[0]:sum(blocks)]
    pools = [torch.randn(num_blocks, hkv, 16, d, generator=gen).to(torch.bfloat16) for _ in range(2)]
    pools.append(torch.randn(num_blocks, 16, r, generator=gen).to(torch.bfloat16))
    kd, vd, ld = (t.to(DEV) for t in pools)
    shape = lra.make_shape(torch.empty(1, hkv, d, dtype=torch.bfloat16, device=DEV), hkv, r, 0.0)
    lens_d, table_d = torch.tensor(lens, dtype=torch.int32, device=DEV), table.to(DEV)  # (the cache holds addresses only)
    cache = lra.make_cache(kd, vd, ld, lens_d, max(lens), table_d)
    f = lambda t: t.to(torch.float64).cpu().numpy()
    exp = [f(t).copy() for t in pools]
    prev_t, prev_k = lra.lra_set_append_tile(256), lra.lra_set_append_skinny(0)
    try:
        for s in range(2):
            x, w = _inputs(6600 + s, n_new[s], d_model, hkv, d, r)
            lra.lra_cache_append(shape, cache, w.to(DEV), 10000.0, x.to(DEV), s)
            torch.cuda.synchronize()
            first = lens[s] - n_new[s]
            refs = oracle.project_new_tokens(f(x), f(w), hkv, d, r, np.arange(first, lens[s]), 10000.0)
            ids = table[s, :blocks[s]].numpy()
            got = [oracle.gather_paged(f(kd), ids, lens[s])[first:], oracle.gather_paged(f(vd), ids, lens[s])[first:],
                   oracle.lra_oracle.gather_paged_l(f(ld), ids, lens[s])[first:]]
            for name, g, ref in zip("KVL", got, refs):
                _gate(g, ref, f"paged {name} rows seq {s}")
            oracle.scatter_paged(exp[0], ids, first, got[0])
            oracle.scatter_paged(exp[1], ids, first, got[1])
            oracle.scatter_paged_l(exp[2], ids, first, got[2])
            for t, e in zip((kd, vd, ld), exp):
                np.testing.assert_array_equal(f(t), e)
    finally:
        lra.lra_set_append_tile(prev_t)
        lra.lra_set_append_skinny(prev_k)


def test_append_rejects_what_it_cannot_do():
    hkv, d, r = 2, 128, 16
    k_base = torch.zeros(64, hkv, d, dtype=torch.bfloat16, device=DEV)
    l = torch.zeros(64, r, dtype=torch.bfloat16, device=DEV)
    seq_lens = torch.tensor([64], dtype=torch.int32, device=DEV)
    shape = lra.make_shape(torch.empty(1, hkv, d, dtype=torch.bfloat16, device=DEV), hkv, r, 0.0)
    cache = lra.make_cache(k_base, k_base.clone(), l, seq_lens, 64, None)
    w = torch.zeros(2 * hkv * d + r, 96, dtype=torch.bfloat16, device=DEV)   # d_model not a multiple of 64
    x = torch.zeros(4, 96, dtype=torch.bfloat16, device=DEV)
    with pytest.raises(lra.LraError) as e:
        lra.lra_cache_append(shape, cache, w, 10000.0, x, 0)
    assert e.value.status == 4
    w = torch.zeros(2 * hkv * d + r, 128, dtype=torch.bfloat16, device=DEV)
    x = torch.zeros(65, 128, dtype=torch.bfloat16, device=DEV)              # more new tokens than the cache holds
    with pytest.raises(lra.LraError) as e:
        lra.lra_cache_append(shape, cache, w, 10000.0, x, 0)
    assert e.value.status == 2


@pytest.mark.parametrize("n_new,prior", [(2048, 16384), (16384, 0), (1, 40000)], ids=["2048_after_16384", "16384_from_empty", "decode_step"])
def test_append_llama3_8b_full_size_sampled_rows(n_new, prior):
    """The benchmark's configuration (d_model 4096 -> 8 kv heads x 128 + rank 16, rotary base 500000) in the
    launch shape bench.py times; the oracle evaluates a sample of the new tokens (rows are independent)."""
    hkv, d, r, dm, theta = 8, 128, 16, 4096, 500000.0
    n = prior + n_new
    x, w = _inputs(7000 + n_new, n_new, dm, hkv, d, r)
    k_base = torch.full((n, hkv, d), SENTINEL, dtype=torch.bfloat16, device=DEV)
    v_base = torch.full_like(k_base, SENTINEL)
    l = torch.full((n, r), SENTINEL, dtype=torch.bfloat16, device=DEV)
    seq_lens = torch.tensor([n], dtype=torch.int32, device=DEV)
    shape = lra.make_shape(torch.empty(1, hkv, d, dtype=torch.bfloat16, device=DEV), hkv, r, 0.0)
    cache = lra.make_cache(k_base, v_base, l, seq_lens, n, None)
    lra.lra_cache_append(shape, cache, w.to(DEV), theta, x.to(DEV), 0)
    torch.cuda.synchronize()
    rng = np.random.default_rng(n_new)
    rows = np.unique(np.concatenate([[0, n_new - 1], rng.integers(0, n_new, size=min(96, n_new))]))
    f = lambda t: t.to(torch.float64).cpu().numpy()
    k_ref, v_ref, l_ref = oracle.project_new_tokens(f(x[rows]), f(w), hkv, d, r, prior + rows, theta)
    _gate(f(k_base[prior + rows]), k_ref, "K rows")
    _gate(f(v_base[prior + rows]), v_ref, "V rows")
    _gate(f(l[prior + rows]), l_ref, "L rows")
    if prior:
        assert bool((k_base[:prior] == SENTINEL).all()) and bool((l[:prior] == SENTINEL).all())


@pytest.mark.parametrize("n_new", [1, 5, 200, 2048], ids=lambda n: f"new{n}")
def test_append_writes_nothing_when_the_device_length_exceeds_the_bound(n_new):
    """max_seq_len sizes the caches: a device-side sequence length beyond it cannot be honoured, and the call must
    leave every cache row as it was (all four kernels: matrix-vector, weight-streaming, tiled, wide tile)."""
    hkv, d, r, d_model, rows = 2, 128, 16, 256, 2100
    x, w = _inputs(900 + n_new, n_new, d_model, hkv, d, r)
    k = torch.full((rows, hkv, d), SENTINEL, dtype=torch.bfloat16, device=DEV)
    v = torch.full_like(k, SENTINEL)
    l = torch.full((rows, r), SENTINEL, dtype=torch.bfloat16, device=DEV)
    lens = torch.tensor([rows + 50], dtype=torch.int32, device=DEV)       # longer than the cache can hold
    shape = lra.make_shape(torch.empty(1, hkv, d, dtype=torch.bfloat16, device=DEV), hkv, r, 0.0)
    wd, xd = w.to(DEV), x.to(DEV)   # referenced until the synchronisation: the call only enqueues
    lra.lra_cache_append(shape, lra.make_cache(k, v, l, lens, rows, None), wd, 500000.0, xd, 0)
    torch.cuda.synchronize()
    for name, t in (("K", k), ("V", v), ("L", l)):
        assert bool((t == SENTINEL).all()), f"{name} rows were overwritten"


QUARTER_CASES = [
    # n, n_new, d_model, Hkv, d, r, theta, paged: 64 x 64 tiles
    (66, 65, 128, 2, 64, 8, 10000.0, False),          # one step; one token in the second tile; L on every feature tile
    (700, 128, 256, 2, 128, 32, 500000.0, True),      # two steps, both L blocks, no remainder
    (400, 250, 384, 4, 64, 24, 500000.0, False),      # three steps; half of the second L block; six tokens short
    (70000, 161, 640, 3, 128, 16, 500000.0, False),   # five steps, one more than the ring holds; far positions
    (900, 320, 1024, 8, 128, 64, 0.0, True),          # four L blocks, unrotated keys
    (2000, 511, 4096, 8, 128, 16, 500000.0, False),   # a full round of the chip
    (1500, 1025, 128, 1, 128, 16, 10000.0, True),     # four feature tiles, all with L blocks; more tokens than features: an XCD's stretch by tokens
    (900, 833, 256, 3, 64, 16, 500000.0, False),      # ... 84 tiles on 8 XCDs, the last stretch four short
]


@pytest.mark.parametrize("case", QUARTER_CASES, ids=lambda c: "n%d_new%d_dm%d_hkv%d_d%d_r%d_th%g_paged%d" % c)
def test_append_quarter_tiles(case):
    """Against the oracle, all other cache elements keep their value, and an offered workspace is left alone (the
    parts of a divided d_model would be in it)."""
    n, n_new, d_model, hkv, d, r, theta, paged = case
    x, w = _inputs(7300 + n, n_new, d_model, hkv, d, r)
    blocks = (n + 15) // 16
    order = torch.randperm(blocks, generator=torch.Generator().manual_seed(n))
    if paged:
        k = torch.full((blocks, hkv, 16, d), SENTINEL, dtype=torch.bfloat16, device=DEV)
        l = torch.full((blocks, 16, r), SENTINEL, dtype=torch.bfloat16, device=DEV)
    else:
        k = torch.full((n, hkv, d), SENTINEL, dtype=torch.bfloat16, device=DEV)
        l = torch.full((n, r), SENTINEL, dtype=torch.bfloat16, device=DEV)
    v = k.clone()
    lens = torch.tensor([n], dtype=torch.int32, device=DEV)
    table = order.to(torch.int32).view(1, -1).to(DEV) if paged else None  # (the cache holds addresses only)
    cache = lra.make_cache(k, v, l, lens, n, table)
    shape = lra.make_shape(torch.empty(1, hkv, d, dtype=torch.bfloat16, device=DEV), hkv, r, 0.0)
    ws = torch.full((8 << 20,), 0xA5, dtype=torch.uint8, device=DEV)
    lra.lra_cache_append(shape, cache, w.to(DEV), theta, x.to(DEV), 0, workspace=ws)
    torch.cuda.synchronize()
    assert bool((ws == 0xA5).all())
    rows = lambda t, lead: (t.transpose(1, 2) if lead else t)[order.to(DEV)].flatten(0, 1) if paged else t
    f = lambda t: t.to(torch.float64).cpu().numpy()
    refs = oracle.project_new_tokens(f(x), f(w), hkv, d, r, np.arange(n - n_new, n), theta)
    for name, t, lead, ref in zip("KVL", (k, v, l), (True, True, False), refs):
        t = rows(t, lead)
        _gate(f(t[n - n_new:n]), ref, f"{case} {name}")
        assert bool((t[:n - n_new] == SENTINEL).all()) and bool((t[n:] == SENTINEL).all())
