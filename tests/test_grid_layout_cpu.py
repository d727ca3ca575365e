"""Where the workgroups of several row groups run: workgroup i goes to XCD i mod 8 and, of its four shader engines of eight
compute units, to the one that i mod 32 stands for."""
from collections import Counter

from tests.test_gpu_cases_plan_cpu import planner  # noqa: F401 (a fixture)


def test_streaming_grids_fit_one_round(planner):  # noqa: F811
    """A grid filled up so that the row groups of a key share meet on one XCD does not give a shader engine more workgroups with keys
    than it has compute units; one that is left as it is would."""
    filled = left = 0
    for hkv in range(1, 41):
        for row_groups in range(1, 12):
            for splits in range(1, 256 // (hkv * row_groups) + 1):
                shares = planner.stream_grid_query(hkv, splits, row_groups)
                full = next(n for n in range(splits, splits + 8) if n * hkv % 8 == 0)
                assert shares in (splits, full)
                if row_groups == 1 or full == splits:
                    assert shares == splits
                    continue
                where = [[x + hkv * y + hkv * full * rg for y in range(splits) for x in range(hkv)] for rg in range(row_groups)]
                most = max(Counter(i % 32 for w in where for i in w).values())
                assert (shares == full) == (most <= 8), (hkv, splits, row_groups)
                filled, left = filled + (shares == full), left + (shares != full)
                if shares == full:
                    on = [Counter(i % 8 for i in w) for w in where]
                    assert all(c == on[0] for c in on)
    assert filled > 100 and left > 100
    assert planner.stream_grid_query(4, 29, 2) == 30 and planner.stream_grid_query(5, 12, 4) == 16 and planner.stream_grid_query(12, 3, 6) == 3


def test_interleaved_grids_of_rotary_calls(planner):  # noqa: F811
    """The kernel's walk of its grid: every (share, row group) once, nothing beyond them, and the row groups of every share in a
    whole block of m on one XCD."""
    met = 0
    for hkv in (1, 2, 3, 4, 5, 6, 7, 8, 12, 24, 32, 40):
        for row_groups in range(2, 12):
            for splits in range(1, 512 // (hkv * row_groups) + 1):
                m = planner.interleave_query(hkv, splits, row_groups, 1)
                assert m in (1, 2, 4, 8) and hkv * m % 8 == 0
                whole = splits & ~(m - 1)
                seen = {}
                for y in range(splits * row_groups):
                    if y >= whole * row_groups:
                        rest, at = splits - whole, y - whole * row_groups
                        rg, split = at // rest, whole + at % rest
                    else:
                        hi = y // m
                        rg, split = hi % row_groups, y % m + m * (hi // row_groups)
                    assert (split, rg) not in seen and split < splits and rg < row_groups
                    seen[split, rg] = y
                assert len(seen) == splits * row_groups
                for split in range(whole):
                    for x in (0, hkv - 1):
                        assert len({(x + hkv * seen[split, rg]) % 8 for rg in range(row_groups)}) == 1
                        met += 1
    assert met > 1000
    assert planner.interleave_query(5, 17, 1, 1) == 0 and planner.interleave_query(5, 17, 3, 0) == 8
    assert planner.interleave_query(5, 65530, 2, 0) == 0  # (131072 in the grid's second dimension)
