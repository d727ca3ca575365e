"""The weight-streaming append of few tokens against the oracle, where its division can go wrong: every count of eight-row token
requests, groups of one to seven rotary pairs (a last group that is not full, groups across K and V, as many L features as
workgroups), waves without a piece of d_model, with unequal numbers and with more than their ring holds.  Same gate as the other appends."""
import pytest

import paper_2602_01053_amd as lra
from tests.test_append_gpu import _append_contiguous

pytestmark = pytest.mark.gpu

CASES = [
    # n, n_new, d_model, Hkv, d, r, theta
    (90, 2, 64, 1, 64, 64, 10000.0),         # one pair, 64 workgroups, 64 L features; one piece
    (90, 9, 576, 5, 64, 24, 10000.0),        # two pairs, nine pieces over eight waves
    (90, 24, 1088, 5, 128, 64, 500000.0),    # three pairs: 213 1/3 workgroups, one group across K and V
    (40000, 25, 4096, 7, 128, 16, 500000.0), # four pairs
    (90, 41, 1600, 9, 128, 8, 0.0),          # five pairs, 230 2/5 workgroups
    (90, 49, 256, 11, 128, 40, 10000.0),     # six pairs; four of the eight waves have no piece
    (90, 57, 640, 14, 128, 48, 10000.0),     # seven pairs
    (90, 8, 512, 15, 128, 16, 10000.0),      # four pairs, two workgroups per unit
    (90, 17, 512, 25, 128, 32, 10000.0),     # six pairs, 533 1/3 workgroups
    (90, 32, 8192, 2, 64, 16, 10000.0),      # sixteen pieces per wave
    (200, 64, 1024, 3, 64, 16, 10000.0),
    (200, 131, 704, 3, 128, 16, 10000.0),    # three chunks of 64 tokens, the last of three
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "n%d_new%d_dm%d_hkv%d_d%d_r%d_th%g" % c)
def test_few_tokens(case):
    prev = lra.lra_set_append_skinny(1 << 30)
    try:
        _append_contiguous(case, False)
    finally:
        lra.lra_set_append_skinny(prev)
