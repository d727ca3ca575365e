"""Decode of one sequence: key shares of all kv heads and row groups fill one round of workgroups."""
import pytest

from tests.test_gpu_cases_plan_cpu import _plan, planner  # noqa: F401 (a fixture)


@pytest.mark.parametrize("paged,side", [(False, "bk"), (False, "none"), (False, "own"), (True, "bk"), (True, "own"),
                                        (False, "rotary"), (True, "rotary")])
def test_one_round(planner, paged, side):  # noqa: F811
    for hkv in (1, 2, 3, 5, 7, 8, 9, 12, 24, 32):
        for group in (1, 4, 7):
            for agents in (1, 3, 6, 12):
                for r in (64,) if side == "rotary" else (16, 64):
                    for n in (129, 1000, 5000, 20000, 65537):
                        pl = _plan(planner, hkv * group, hkv, 128, r, [n], agents=agents, paged=paged, side=side)
                        units = hkv * pl["row_groups"]
                        # the split-KV kernel, two workgroups per unit, reads caches of blocks with low-rank rows per adapter
                        room = 512 if paged and side == "own" else 256
                        # ... and long ones that several row groups read, where a last share may begin another round
                        if paged and side == "bk" and pl["row_groups"] > 2 and units * n >= 512 * 512:
                            assert units * (pl["n_splits"] - 1) <= 512 or pl["n_splits"] == 1
                            continue
                        # ... or two, between 2^19 and 5 x 2^18, at ranks up to 32
                        if paged and side == "bk" and pl["row_groups"] == 2 and r <= 32 and 1 << 19 <= units * n < 5 << 18:
                            room = 512
                        if pl["mfma"] and units <= room:
                            short = 1 if side == "rotary" else 0  # (a last, short share may begin a second one)
                            assert units * (pl["n_splits"] - short) <= room, (hkv, group, agents, r, n, units, pl["n_splits"])


def test_one_round_fills_the_chip(planner):  # noqa: F811
    """The shares are cut down to one round only where that leaves three quarters of the places taken, and with several row groups
    to a count whose workgroups meet on one XCD where there is one within a sixteenth."""
    def splits(hkv, group, agents, n, r=16, paged=False, side="bk"):
        pl = _plan(planner, hkv * group, hkv, 128, r, [n], agents=agents, paged=paged, side=side)
        return hkv * pl["row_groups"], pl["n_splits"]

    assert splits(24, 1, 45, 4465) == (144, 2)    # 144 of 256 in one round: two
    assert splits(32, 1, 35, 22237) == (160, 2)
    assert splits(32, 1, 41, 8000) == (192, 1)    # 192: one
    assert splits(12, 2, 38, 5918) == (60, 4)
    assert splits(5, 4, 10, 55301) == (10, 23)    # 25 fit; 24 meet, 23 of 19 tiles are enough
    assert splits(6, 4, 10, 34074) == (12, 20)    # 21 fit; 20 meet
    assert splits(8, 4, 12, 20000)[1] == 16
    # low-rank caches per adapter on pages: the split-KV kernel, two workgroups per unit
    assert splits(16, 2, 6, 1304, r=32, paged=True, side="own") == (48, 6)
    assert splits(8, 8, 10, 2353, r=32, paged=True, side="own") == (40, 7)
    assert splits(8, 4, 6, 30000, r=32, paged=True, side="own") == (24, 20)


def test_long_paged_sequences_of_several_row_groups(planner):  # noqa: F811
    """The split-KV kernel, two workgroups per unit, where three row groups (64 wide: two) read 2^18 keys and more in all units."""
    def workgroups(hkv, group, d, agents, n):
        pl = _plan(planner, hkv * group, hkv, d, 16, [n], agents=agents, paged=True)
        return pl["row_groups"], hkv * pl["row_groups"] * pl["n_splits"]

    assert workgroups(32, 1, 64, 39, 6572) == (5, 640)
    assert workgroups(4, 7, 128, 33, 42376)[1] > 460
    assert workgroups(8, 4, 128, 17, 10922)[1] <= 256 < workgroups(8, 4, 128, 17, 10923)[1]  # 24 units
    assert workgroups(32, 1, 64, 14, 13256) == (2, 512) and workgroups(32, 1, 128, 14, 4700) == (2, 256)
    # two row groups at d = 128: between 2^19 and 5 x 2^18, shares that meet on an XCD
    assert workgroups(32, 1, 128, 14, 8191) == (2, 256) and workgroups(32, 1, 128, 14, 8192) == (2, 512)
    assert workgroups(32, 1, 128, 14, 20479) == (2, 512) and workgroups(32, 1, 128, 14, 20480) == (2, 256)
    assert workgroups(12, 2, 128, 10, 40000) == (2, 480) and workgroups(5, 4, 128, 9, 55000)[1] <= 480
    assert workgroups(8, 4, 128, 8, 65536) == (1, 256)
    # shares that fit two workgroups per unit, or up to a fifth less where they then meet on an XCD
    assert workgroups(4, 7, 128, 50, 10232) == (13, 416) and workgroups(8, 8, 128, 83, 10908) == (21, 504)
    assert workgroups(12, 2, 128, 31, 42330) == (4, 480) and workgroups(7, 2, 128, 26, 33554) == (4, 448)  # (18 fit, 16 meet)


def test_no_room_for_a_pre_pass_that_does_not_run(planner):  # noqa: F811
    """Room for Qt only where the streaming kernel can run: without it a decode of many agents stays within the 64 MiB of the
    library's own workspace."""
    for paged in (False, True):
        pl = _plan(planner, 256, 32, 128, 64, [9300], agents=289, paged=paged)
        assert pl["row_groups"] * 32 > 256 and pl["qt_bytes"] == 0 and pl["pages"] * 256 <= 64 << 20
        pl = _plan(planner, 32, 8, 128, 64, [9300], agents=8, paged=paged)
        assert pl["row_groups"] * 8 * pl["n_splits"] <= 256 and pl["qt_bytes"] > 0


def test_the_pre_pass_runs_for_two_row_tiles(planner):  # noqa: F811
    for paged in (False, True):
        for agents in (1, 2, 3, 4):
            pl = _plan(planner, 32, 8, 128, 64, [3000], agents=agents, paged=paged)
            assert pl["row_tiles"] == 1 and pl["qt_bytes"] == 0
        assert _plan(planner, 32, 8, 128, 64, [3000], agents=5, paged=paged)["qt_bytes"] > 0
        assert _plan(planner, 28, 4, 128, 64, [3000], agents=2, paged=paged)["qt_bytes"] == 0


def test_two_workgroups_per_unit_in_the_rotary_form(planner):  # noqa: F811
    """One size for all shares where the units do not divide the chip and that makes the longest load shorter; else the first ones a
    tile longer; with several row groups counts that meet on one XCD."""
    def shares(hkv, group, agents, n, r):
        pl = _plan(planner, hkv * group, hkv, 128, r, [n], agents=agents, paged=False, side="rotary")
        return hkv * pl["row_groups"], pl["n_splits"], pl["split_keys"], pl["split_more"]

    assert shares(24, 1, 11, 6250, 32) == (144, 3, 17 * 128, 0)
    assert shares(24, 1, 8, 40888, 32) == (96, 5, 64 * 128, 0)
    assert shares(32, 1, 5, 8187, 24) == (96, 5, 13 * 128, 0)
    assert shares(8, 4, 4, 9000, 16) == (8, 39, 2 * 128, 32)      # 71 tiles on 32 units: loads of three
    assert shares(5, 4, 4, 41459, 32) == (10, 47, 7 * 128, 0)     # 25 units fit, 24 meet: loads of 14
    assert shares(5, 4, 8, 35089, 8)[:2] == (10, 46)
    assert shares(2, 8, 11, 38848, 16)[:2] == (12, 38)
    # a prefill of a few tokens keeps 384 keys and more per share: 14 tiles on three units of 72, shares of three and two
    pl = _plan(planner, 24, 24, 128, 8, [1686], n_new=10, paged=False, side="rotary")
    assert (pl["n_splits"], pl["split_keys"], pl["split_more"]) == (6, 384, 3)
    pl = _plan(planner, 32, 8, 64, 16, [2621], agents=12, paged=False, side="rotary")  # (one tile for all: too many states)
    assert (pl["n_splits"], pl["split_keys"], pl["split_more"]) == (11, 256, 10)


def test_rotary_shapes_without_a_key_adapter_keep_one_round(planner):  # noqa: F811
    """Nothing is rotated without a B_K: the call runs on the streaming kernel, which has no second round."""
    for paged in (False, True):
        for hkv, agents, n, r in ((24, 1, 9000, 16), (12, 8, 9000, 16), (24, 2, 9000, 64), (5, 4, 20000, 48)):
            pl = _plan(planner, 4 * hkv, hkv, 128, r, [n], agents=agents, paged=paged, side="rotary_none")
            units = hkv * pl["row_groups"]
            assert units * 2 <= 256 and 192 <= units * pl["n_splits"] <= 256, (hkv, agents, n, r, pl["n_splits"])
