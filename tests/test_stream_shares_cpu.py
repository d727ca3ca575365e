"""The streaming kernel's own key shares, and the few-token prefills that it takes: only calls that stream have them, in one round of
workgroups that covers the keys, with room in the workspace."""
import ctypes
import os
import shutil
import subprocess

import pytest

from tests import test_parity_gpu as P
from tests import test_stream_prologue_gpu as S
from tests.test_gpu_cases_plan_cpu import ROOT, _plan, planner  # noqa: F401 (a fixture)


@pytest.fixture(scope="module")
def runs(tmp_path_factory):
    """_plan's library for the plan as it runs."""
    gxx = shutil.which("g++")
    if gxx is None:
        pytest.skip("no host C++ compiler")
    lib = str(tmp_path_factory.mktemp("plan") / "stream_plan_query.so")
    csrc = os.path.join(ROOT, "paper_2602_01053_amd", "csrc")
    subprocess.run([gxx, "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "include"), "-I", csrc,
                    os.path.join(csrc, "lra_plan.cpp"), os.path.join(ROOT, "tests", "stream_plan_query.cpp"), "-o", lib], check=True)
    return ctypes.CDLL(lib)


def _check(pl, run, units, n, hq, rows, d, r):
    assert run["split_keys"] % 32 == 0 and units * run["n_splits"] <= 256 and not run["wave_shares"]
    assert run["n_splits"] * run["split_keys"] >= n > (run["n_splits"] - 1) * run["split_keys"]
    assert run["pages"] == pl["pages"]  # one workspace for both
    align = lambda x: (x + 255) // 256
    slots = rows * max(run["n_splits"], pl["n_splits"])
    assert pl["pages"] == align(slots * 8) + align(slots * d * 4) + align(slots * r * 4) + align(rows * 4) + align(run["qt_bytes"])


def test_only_calls_that_stream(planner, runs):  # noqa: F811
    own = forms = 0
    for hkv in (1, 2, 4, 5, 8, 12, 24, 32, 48):
        for group in (1, 4, 7, 16):
            for agents in (1, 4, 9, 17):
                for r in (16, 64):
                    for n in (500, 1500, 4500, 9009, 13000, 25000, 66000):
                        for paged in (False, True):
                            for side in ("bk", "none", "own", "rotary"):
                                a = dict(agents=agents, paged=paged, side=side)
                                pl, run = (_plan(x, hkv * group, hkv, 128, r, [n], **a) for x in (planner, runs))
                                if pl == run:
                                    continue
                                own += 1
                                assert side != "rotary" and not (paged and side == "own") and 128 < run["split_keys"] < pl["split_keys"]
                                _check(pl, run, hkv * run["row_groups"], n, hkv * group, agents * hkv * group, 128, r)
                                assert _plan(runs, hkv * group, hkv, 128, r, [n], variant=2, **a)["split_keys"] % 128 == 0
            for n_new in (1, 3, 5, 8, 12, 16, 24, 32, 33):
                for r in (16, 32, 64):
                    for n in (800, 1400, 2700, 4500, 9009, 20000):
                        for paged in (False, True):
                            for side in ("bk", "none", "rotary"):
                                a = dict(n_new=n_new, paged=paged, side=side)
                                pl, run = (_plan(x, hkv * group, hkv, 128, r, [n], **a) for x in (planner, runs))
                                if pl == run:
                                    continue
                                forms += not pl["short_prefill"]
                                assert run["short_prefill"] and side != "rotary" and n_new <= 32 and n_new * 4 <= n and not run["wave_rows"]
                                _check(pl, run, hkv * run["row_groups"], n, hkv * group, n_new * hkv * group, 128, r)
    assert own > 150 and forms > 100
    batch = dict(agents=4, paged=True)
    assert _plan(planner, 32, 8, 128, 16, [4500, 4400], **batch) == _plan(runs, 32, 8, 128, 16, [4500, 4400], **batch)


def test_which_few_token_prefills_stream(runs):
    for hkv, group, n_new, n, paged, r, streams in [
            (8, 4, 8, 9009, False, 16, False), (8, 4, 8, 1536, False, 16, False), (8, 4, 8, 1537, False, 16, True), (8, 4, 8, 7168, False, 16, True),
            (8, 4, 8, 5000, False, 32, False), (8, 4, 6, 2000, True, 32, True), (4, 7, 4, 6004, False, 16, True), (4, 7, 4, 2200, True, 16, False),
            (4, 7, 8, 14000, True, 24, True), (4, 7, 8, 14400, True, 24, False), (8, 4, 16, 3500, False, 8, True), (8, 4, 16, 6000, False, 8, False),
            (8, 4, 16, 6000, False, 32, True), (8, 4, 16, 4000, True, 8, False), (8, 4, 24, 5000, False, 16, True), (8, 4, 24, 4000, True, 16, False),
            (4, 7, 12, 6000, True, 16, False), (4, 7, 12, 6000, False, 16, True), (4, 7, 9, 6000, False, 16, False)]:
        assert _plan(runs, hkv * group, hkv, 128, r, [n], n_new=n_new, paged=paged)["short_prefill"] == streams, (hkv, n_new, n, paged, r)


def test_cases_of_the_kernel_whose_waves_divide_the_keys_keep_it(planner, runs):  # noqa: F811
    for n, n_new, hq, hkv, d, r, paged, side, longest in P.WAVE_SHARE_CASES:
        a = dict(longest=longest, n_new=n_new, paged=paged, side=side)
        shares = _plan(planner, hq, hkv, d, r, [n], **a)["wave_shares"]
        assert _plan(runs, hq, hkv, d, r, [n], **a)["wave_shares"] == shares, (n, n_new)


def test_kv_heads_whose_calls_have_them(planner, runs):  # noqa: F811
    """Key shares of any number of tiles by kv heads: 1 to 3, 6 and 7 keep multiples of 128, 5 and those above 8 that are no multiple of
    four leave them only for shares of at most 192 keys."""
    for hkv in (1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 12, 14, 16, 20, 32):
        for even in (140, 180, 201, 241, 300, 420, 700):
            n = even * 256 // hkv
            for r in (16, 64):
                for paged in (False, True):
                    a = (hkv * 4, hkv, 128, r, [n])
                    pl, run = (_plan(x, *a, agents=2, paged=paged) for x in (planner, runs))
                    most = (256 if paged else 1024) if hkv % 4 == 0 else (192 if hkv == 5 or hkv > 8 else 0)
                    if even > most:
                        assert run == pl, (hkv, even, r, paged)
                    elif even < 241:  # (an even share close below a multiple of 128 is that multiple)
                        assert run["split_keys"] < pl["split_keys"], (hkv, even, r, paged)
    for hkv, n, own in ((8, 4500, False), (8, 5500, True)):  # 64 wide, two row tiles
        pl, run = (_plan(x, hkv * 8, hkv, 64, 32, [n], agents=4, paged=True) for x in (planner, runs))
        assert (run != pl) == own


def test_few_token_prefills_of_other_groups_and_heads(runs):
    """Groups of one and two q heads, whose rows are padded to four, and 6 kv heads leave streaming earlier."""
    for hkv, group, n_new, n, paged, r, streams in [
            (8, 2, 8, 1800, False, 16, False), (8, 2, 8, 2000, False, 16, True), (8, 3, 8, 1800, False, 16, True),
            (8, 2, 24, 2300, False, 16, True), (8, 2, 24, 2600, False, 16, False), (8, 2, 16, 3000, True, 32, False), (6, 1, 16, 2300, True, 16, True),
            (6, 1, 16, 2600, True, 16, False), (8, 1, 24, 2000, False, 16, False), (4, 1, 24, 4500, False, 16, False), (4, 2, 24, 4500, False, 16, True),
            (4, 1, 16, 4500, False, 16, True), (6, 4, 24, 3000, False, 16, True), (6, 4, 24, 3300, False, 16, False), (7, 4, 24, 4500, False, 16, True),
            (6, 4, 8, 5000, False, 16, True), (6, 4, 8, 6000, False, 16, False), (7, 4, 8, 6000, False, 16, True)]:
        assert _plan(runs, hkv * group, hkv, 128, r, [n], n_new=n_new, paged=paged)["short_prefill"] == streams, (hkv, group, n_new, n, paged, r)


def test_calls_of_the_prologue_tests_stream(runs):
    seen = set()
    for n, agents, hq, hkv, d, r, key_side in S.CASES:
        pl = _plan(runs, hq, hkv, d, r, [n], agents=agents, paged=False, side="bk" if key_side else "none")
        assert pl["mfma"] and hkv * pl["n_splits"] * pl["row_groups"] <= 256, (n, agents)
        seen.add((pl["row_tiles"], d, pl["qt_bytes"] > 0, key_side))
    assert seen >= {(1, 64, False, True), (1, 128, False, True), (2, 64, False, True), (2, 128, False, True), (2, 128, True, True), (2, 64, True, True),
                    (2, 128, False, False)}
    tiles = set()
    for n_new, n, hq, hkv, d, r in S.PREFILL_CASES:
        pl = _plan(runs, hq, hkv, d, r, [n], n_new=n_new, paged=False, short_prefill=33)
        assert pl["short_prefill"] and not pl["wave_rows"] and hkv * pl["n_splits"] * pl["row_groups"] <= 256, (n_new, n)
        tiles.add(pl["row_tiles"])
    assert tiles == {1, 2}
    pl = _plan(runs, 32, 8, 128, 64, [11000], agents=17, paged=True, split_keys=11000)  # (three row groups, one share)
    assert pl["row_groups"] == 3 and pl["n_splits"] == 1 and pl["qt_bytes"] == 0 and pl["row_tiles"] == 2
