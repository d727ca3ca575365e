"""Where the workgroups of several row groups run: workgroup i goes to XCD i mod 8, each of 32 compute units."""
from collections import Counter

from tests.test_gpu_cases_plan_cpu import planner  # noqa: F401 (a fixture)


def test_streaming_grids_fit_one_round(planner):  # noqa: F811
    """A grid filled up so that the row groups of a key share meet on one XCD does not give an XCD more workgroups, empty ones
    among them, than it has compute units."""
    filled = 0
    for hkv in range(1, 41):
        for row_groups in range(1, 12):
            for splits in range(1, 256 // (hkv * row_groups) + 1):
                shares = planner.stream_grid_query(hkv, splits, row_groups)
                assert splits <= shares < splits + 8
                if shares == splits:
                    continue
                filled += 1
                where = [Counter((x + hkv * y + hkv * shares * rg) % 8 for y in range(shares) for x in range(hkv)) for rg in range(row_groups)]
                assert all(w == where[0] for w in where) and max(where[0].values()) * row_groups <= 32, (hkv, splits, row_groups)
    assert filled > 100
