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
                        room = 512 if paged and side == "own" and units * n >= 512 * 512 else 256
                        if pl["mfma"] and units <= room:
                            short = 1 if side == "rotary" else 0  # (a last, short share may begin a second one)
                            assert units * (pl["n_splits"] - short) <= room, (hkv, group, agents, r, n, units, pl["n_splits"])
