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


def test_interleaved_grids_of_rotary_calls(planner):  # noqa: F811
    """The padding of an interleaved grid does not cost a rotary call that is resident at once another workgroup per compute unit;
    where it is taken the row groups of a share are on one XCD."""
    taken = refused = 0
    for hkv in (1, 2, 3, 4, 5, 6, 7, 8, 12, 24, 32, 40):
        for row_groups in range(2, 12):
            for rank, room in ((16, 512), (32, 512), (40, 256), (64, 256)):
                for splits in range(1, room // (hkv * row_groups) + 1):
                    m = planner.interleave_query(hkv, splits, row_groups, 1, 1, rank)
                    if m == 0:
                        refused += 1
                        continue
                    taken += 1
                    padded = -(-splits // m) * m
                    assert hkv * m % 8 == 0 and hkv * row_groups * padded <= room
                    assert -(-hkv * row_groups * padded // 256) == -(-hkv * row_groups * splits // 256)
    assert taken > 100 and refused > 100
    assert planner.interleave_query(5, 17, 3, 1, 1, 64) == 0 and planner.interleave_query(5, 50, 2, 1, 1, 32) == 0
    assert planner.interleave_query(5, 48, 2, 1, 1, 32) == 8 and planner.interleave_query(8, 31, 2, 1, 1, 16) == 1
    assert planner.interleave_query(5, 17, 3, 1, 0, 64) == 8  # no rotation: as ever
