"""The GPU tests name the kernels their cases run on; this asks the launch planner, compiled for the CPU
(tests/plan_query.cpp), whether the calls still get there."""
from __future__ import annotations

import ctypes
import os
import shutil
import subprocess

import pytest

from paper_2602_01053_amd.binding import LraCache, LraShape, LraTuning
from tests import test_append_gpu as A
from tests import test_merge_forms_gpu as F
from tests import test_merge_tokens_gpu as M
from tests import test_parity_gpu as P
from tests import test_rope_shares_gpu as R

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
FIELDS = ("mfma", "short_prefill", "wave_rows", "wave_shares", "n_splits", "tile_group", "batch_wgs", "batch_tiles", "row_tiles",
          "row_groups", "l_block", "workspace_optional", "group_pad", "split_keys", "split_more", "qt_bytes", "pages")


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    lib = str(tmp_path_factory.mktemp("plan") / "plan_query.so")
    csrc = os.path.join(ROOT, "paper_2602_01053_amd", "csrc")
    subprocess.run([gxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                    os.path.join(csrc, "lra_plan.cpp"), os.path.join(ROOT, "tests", "plan_query.cpp"), "-o", lib], check=True)
    return ctypes.CDLL(lib)


def _call(hq, hkv, d, r, lens, *, longest=None, agents=0, n_new=0, paged, side="bk", host=None, variant=0, fp32=False, split_keys=0, splits=0, short_prefill=0):
    """The planner's arguments for a call."""
    n = longest or max(lens)
    shape = LraShape(hq, hkv, d, r, int(fp32), 0.0, 500000.0 if side.startswith("rotary") else 0.0)
    cache = LraCache(n_seqs=len(lens), max_seq_len=n, l_row_stride=r)
    if paged:
        blocks = sum((x + 15) // 16 for x in lens) if longest is None else (n + 15) // 16
        cache.block_size, cache.num_blocks, cache.max_blocks_per_seq = 16, blocks, (n + 15) // 16
        cache.kv_token_stride, cache.kv_head_stride, cache.kv_block_stride = d, 16 * d, 16 * d * hkv
        if side in ("own", "own_none"):
            cache.l_adapter_stride = blocks * 16 * r
    else:
        cache.kv_token_stride, cache.kv_head_stride = hkv * d, d
    if host is not None:
        mirror = (ctypes.c_int32 * len(host))(*host)
        cache.seq_lens_host = ctypes.cast(mirror, ctypes.c_void_p)
    return (ctypes.byref(shape), ctypes.byref(cache), n_new or agents * len(lens), max(agents, 1), int(n_new > 0),
            int(side not in ("none", "own_none", "rotary_none")),
            ctypes.byref(LraTuning(kernel_variant=variant, decode_split_keys=split_keys, prefill_splits=splits, short_prefill=short_prefill)))


def _plan(planner, *call, **kw):
    out = (ctypes.c_int32 * len(FIELDS))()
    planner.plan_query(*_call(*call, **kw), out)
    return dict(zip(FIELDS, out))


def _merge(planner, *call, **kw):
    """The merge kernel that a call ends with, and its shares."""
    shares = ctypes.c_int32()
    form = planner.merge_query(*_call(*call, **kw), ctypes.byref(shares))
    return (("columns", "rows", "wave", "tokens")[form] if form >= 0 else None), shares.value


def test_batches_in_one_row(planner):
    seen = set()
    for lens, agents, hq, hkv, d, r, side in P.BATCH_ROW_CASES:
        for host in (lens, None):
            pl = _plan(planner, hq, hkv, d, r, lens, agents=agents, paged=True, side=side, host=host)
            assert pl["batch_wgs"] >= len(lens) and (pl["batch_tiles"] > 0) == (host is not None), (lens, agents, hq, hkv, d, r, side)
        tile_rank = 16 // pl["group_pad"] * pl["l_block"] if pl["l_block"] else r
        rotary = (16 if r <= 16 else 32 if r <= 32 else 64) if side == "rotary" else 0
        seen.add((d, pl["row_tiles"], 32 if tile_rank <= 32 else 64, side in ("bk", "own", "rotary"), rotary, pl["l_block"] > 0))
    assert len(seen) == 29  # the instantiations of decode_batch_kernel
    # ... of the shared list, the ones below, whatever the host believes
    rows = [i for i, (lens, agents, hq, hkv, d, r, side) in enumerate(P.BATCH_CASES)
            if all(_plan(planner, hq, hkv, d, r, lens, agents=agents, paged=True, side=side, host=h)["batch_wgs"]
                   for h in (lens, None, [2 * n for n in lens]))]
    assert rows == [1, 4, 7]


def test_prefills_whose_waves_divide_the_keys(planner):
    for n, n_new, hq, hkv, d, r, paged, side in P.WAVE_CASES:
        assert _plan(planner, hq, hkv, d, r, [n], n_new=n_new, paged=paged, side=side)["wave_rows"], (n, n_new)
    shares = {}
    for n, n_new, hq, hkv, d, r, paged, side, longest in P.WAVE_SHARE_CASES:
        pl = _plan(planner, hq, hkv, d, r, [n], longest=longest, n_new=n_new, paged=paged, side=side)
        assert not pl["wave_rows"]
        shares[n, n_new] = pl["wave_shares"]
    assert shares == {(2100, 9): 5, (2880, 64): 4, (6144, 61): 4, (18432, 33): 6, (11521, 7): 0, (11777, 15): 0, (14001, 9): 32,
                      (16000, 8): 32, (20000, 8): 32, (4096, 64): 4, (2200, 33): 6, (4401, 40): 12, (100, 64): 4, (40, 40): 12}


def test_prefills_on_the_tile_walk(planner):
    groups = set()
    for n, n_new, hq, hkv, d, r in P.TILE_CASES:
        pl = _plan(planner, hq, hkv, d, r, [n], n_new=n_new, paged=False, variant=2)
        assert not (pl["wave_rows"] or pl["wave_shares"] or pl["short_prefill"])
        groups.add((pl["tile_group"] == 1, pl["n_splits"] > 1))
    assert groups >= {(True, True), (False, True), (True, False)}
    for n, n_new in ((417, 84), (1023, 300)):  # without room for its shares, one per q tile
        pl = _plan(planner, 8, 2, 128, 16, [n], n_new=n_new, paged=False, variant=2)
        assert pl["workspace_optional"] and pl["n_splits"] > 1 and not pl["wave_rows"]


def test_long_prefills_that_merge(planner):
    forms = []
    for n_new, n, hq, hkv, d, r, _ in M.CASES:
        pl = _plan(planner, hq, hkv, d, r, [n], n_new=n_new, paged=True)
        assert n_new * hq >= 9216 and not pl["wave_rows"] and not pl["short_prefill"], (n_new, n)
        assert 2 <= pl["n_splits"] <= 16 if pl["mfma"] else (pl["n_splits"] == 1 and r % 8), (n_new, n)
        forms.append(_merge(planner, hq, hkv, d, r, [n], n_new=n_new, paged=True))
    assert forms == [("tokens", 3), ("wave", 3), ("tokens", 3), ("wave", 3), ("tokens", 7), ("tokens", 1)]
    reach = set()
    for n_new, n, hq, hkv, d, r, value_side, shares in M.SHARE_CASES:
        assert _merge(planner, hq, hkv, d, r, [n], n_new=n_new, paged=False, splits=shares) == ("tokens", shares), (n_new, n)
        reach.add((d, value_side, shares > 8))
    assert reach == {(128, True, True), (128, True, False), (128, False, False), (64, True, True), (64, False, True), (64, False, False)}


def test_merges_of_many_rows(planner):
    """A wave per row, in the instantiations that the cases stand for."""
    def call(case, split, **kw):
        seqs, agents, hq, hkv, d, r, longest = case
        return _merge(planner, hq, hkv, d, r, [longest] * seqs, longest=longest, agents=agents, paged=True, split_keys=split, **kw)
    reach = set()
    for case in F.WAVE_CASES:
        form, shares = call(case, 128)
        assert form == "wave", case
        reach.add((case[4], 16 if case[5] <= 16 else 32 if case[5] <= 32 else 64, shares <= 4))
    assert reach >= {(128, 64, True), (128, 64, False), (64, 64, False), (64, 32, False), (128, 32, True)}
    forms = [call((*c, 699), 128)[0] for c in P.test_many_rows_take_the_wave_per_row_merge.pytestmark[0].args[1]]
    assert forms == ["wave", "rows", "rows", "wave"]
    forms = [call(c, 64) for c in F.test_many_rows_of_ragged_batches.pytestmark[0].args[1]]
    assert [f[0] for f in forms] == ["wave", "rows", "wave", "rows", "wave"]


def test_merge_lines(planner):
    """Which form merges, on both sides of every line of the rule."""
    def prefill(rows, shares, r, d=128, hq=32, hkv=8, **kw):
        return _merge(planner, hq, hkv, d, r, [4 * rows], n_new=rows // hq, paged=False, splits=shares, **kw)[0]

    def batch(rows, shares, r, d=128, hq=32, hkv=8):
        return _merge(planner, hq, hkv, d, r, [128 * shares] * 8, agents=rows // hq // 8, paged=True, split_keys=128)[0]

    for form, args in [
            ("rows", (992, 5, 16)), ("wave", (1024, 5, 16)), ("rows", (2528, 9, 16)), ("wave", (2560, 9, 16)), ("rows", (2528, 5, 32)),
            ("wave", (2560, 5, 32)), ("wave", (5088, 5, 32)), ("tokens", (5120, 5, 32)), ("wave", (5120, 6, 32)), ("tokens", (5120, 10, 32, 64)),
            ("wave", (5120, 11, 32, 64)), ("rows", (2528, 5, 64)), ("tokens", (2560, 5, 64)), ("rows", (2560, 6, 64)), ("tokens", (5120, 10, 64)),
            ("rows", (5120, 11, 64)), ("wave", (9216, 5, 16)), ("wave", (9216, 5, 16, 64)), ("tokens", (9240, 8, 16, 64, 28, 4)),
            ("wave", (9240, 9, 16, 64, 28, 4)), ("tokens", (9240, 16, 16, 64, 40, 8)), ("wave", (9240, 17, 16, 64, 40, 8)),
            ("tokens", (9240, 5, 16, 128, 40, 8)), ("wave", (9240, 6, 16, 128, 40, 8)), ("tokens", (9240, 10, 32, 128, 40, 8)),
            ("wave", (9200, 5, 16, 64, 40, 8))]:
        assert prefill(*args) == form, args
    for form, args in [
            ("rows", (768, 5, 16)), ("wave", (1024, 5, 16)), ("wave", (1024, 17, 32)), ("rows", (1024, 16, 32)), ("wave", (2560, 16, 32)),
            ("rows", (2304, 5, 64)), ("rows", (5120 - 256, 5, 64)), ("wave", (5120, 5, 64)), ("rows", (5120, 6, 64)), ("rows", (9216 - 256, 8, 64)),
            ("wave", (9216, 8, 64)), ("rows", (9216, 9, 64)), ("rows", (2560, 16, 64)), ("wave", (2560, 17, 64)), ("rows", (2560, 32, 64, 64)),
            ("wave", (2560, 33, 64, 64)), ("rows", (5120, 5, 64, 128, 32, 32)), ("rows", (2560, 32, 64, 128, 32, 32)),
            ("wave", (2560, 33, 64, 128, 32, 32)), ("rows", (2560, 64, 64, 64, 32, 32)), ("columns", (2560, 65, 64, 64))]:
        assert batch(*args) == form, args


def test_rotary_calls_with_shares_of_two_sizes(planner):
    for n, n_new, hq, hkv, d, r in R.PREFILL_CASES:
        for paged in (False, True):
            pl = _plan(planner, hq, hkv, d, r, [n], n_new=n_new, paged=paged, side="rotary")
            assert pl["short_prefill"] and 0 < pl["split_more"] < pl["n_splits"], (n, n_new)
    rests = []
    for n, n_new, hq, hkv, d, r in R.REST_CASES:
        pl = _plan(planner, hq, hkv, d, r, [n], n_new=n_new, paged=True, side="rotary")
        m = planner.interleave_query(hkv, pl["n_splits"], pl["row_groups"], 1)
        assert pl["short_prefill"]
        rests.append((m, pl["n_splits"]))
    assert rests == [(8, 12), (2, 7), (8, 6)]
    for host in (R.ROW_LENS, None):
        pl = _plan(planner, 32, 8, 128, 16, R.ROW_LENS, agents=3, paged=True, side="rotary", host=host)
        assert pl["batch_wgs"] >= len(R.ROW_LENS) and (pl["batch_tiles"] > 0) == (host is not None)


def test_appends_that_divide_d_model(planner):
    """-1: 64 x 64 tiles, -2: the weight-streaming kernel where d_model would be divided; else the parts."""
    tiles_of_64 = {(129, 256), (512, 1024), (400, 4096)}  # (a size is told for the last two, and not used)
    streamed = {(40, 512), (33, 1024), (64, 768)}         # (here too)
    for n, n_new, d_model, hkv, d, r, theta, parts in A.SPLIT_CASES:
        expect = -1 if (n_new, d_model) in tiles_of_64 else (-2 if (n_new, d_model) in streamed else max(parts, 1))
        assert planner.append_query(n_new, hkv, d, r, d_model, None) == expect, (n_new, d_model)
