"""The merge of the key shares against the oracle where its forms and their bounds meet: 16 / 17, 32 / 33 and 64 shares, ranks at
and behind 16 and 32, shares that hold no key (ragged batches, causal rows), the row counts at which one form hands over to
another.  bf16: the gate of the parity tests (2e-3 is what bf16 operands leave); fp32: 2e-5, sums of at most 4000 terms."""
import numpy as np
import pytest
import torch

import paper_2602_01053_amd as lra
from paper_2602_01053_amd import workloads as W
from tests.harness import MAX_ABS_TOL, REL_L2_TOL, errors, oracle_decode, oracle_prefill, run_decode, run_prefill

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _check(got, ref, fp32=False):
    rel, mx = errors(got, ref)
    print(f"relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= (2e-5 if fp32 else REL_L2_TOL) and mx <= MAX_ABS_TOL


@pytest.mark.parametrize("case", [
    # shares of 64 keys (the last of one key), rank, d, Hq, Hkv, fp32
    (1, 8, 128, 8, 2, False), (16, 16, 128, 8, 2, False), (17, 24, 128, 8, 8, False), (32, 32, 64, 8, 2, False),
    (33, 40, 128, 8, 2, False), (64, 64, 64, 6, 3, False), (64, 16, 128, 4, 1, False), (65, 16, 128, 4, 1, False),
    (2, 4, 64, 4, 4, True), (16, 20, 128, 4, 2, True), (17, 64, 64, 4, 4, True), (33, 12, 128, 4, 4, True), (3, 6, 64, 4, 4, True),
], ids=lambda c: "s%d_r%d_d%d_%dover%d_%s" % (*c[:5], "fp32" if c[5] else "bf16"))
def test_shares_and_ranks(case):
    shares, r, d, hq, hkv, fp32 = case
    w = W.make_contiguous("merge", "decode", seed=sum(case), dtype=torch.float32 if fp32 else torch.bfloat16, n_agents=3, n_q_heads=hq,
                          n_kv_heads=hkv, head_dim=d, rank=r, n=64 * (shares - 1) + 1, b_std=0.1)
    old = lra.lra_set_decode_split_keys(64)
    try:
        _check(run_decode(w, DEV), oracle_decode(w), fp32)
    finally:
        lra.lra_set_decode_split_keys(old)


@pytest.mark.parametrize("case", [
    # sequences, agents, Hq, Hkv, d, r, longest: rows from 1024 on, shares of 64 keys of which most rows have fewer than the longest
    (8, 4, 32, 8, 128, 16, 1100),    # 1024 rows
    (9, 4, 28, 4, 128, 32, 1300),    # 1008, one per workgroup
    (10, 4, 28, 4, 128, 32, 2100),   # 1120, more than 32 shares
    (20, 4, 32, 8, 64, 40, 700),     # 2560 rows above rank 32
    (6, 11, 16, 2, 128, 6, 300),     # 1056 of an odd rank (vector-ALU kernels)
], ids=lambda c: "q%dx%d_%dover%d_d%d_r%d_n%d" % c)
def test_many_rows_of_ragged_batches(case):
    seqs, agents, hq, hkv, d, r, longest = case
    lens = [longest] + [int(x) for x in np.random.default_rng(sum(case)).integers(1, longest, size=seqs - 1)]
    w = W.make_paged("merge", seed=sum(case), seq_lens=lens, agents_per_seq=agents, n_adapters=3, n_q_heads=hq, n_kv_heads=hkv,
                     head_dim=d, rank=r, d_model=None, b_std=0.05)
    old = lra.lra_set_decode_split_keys(64)
    try:
        _check(run_decode(w, DEV), oracle_decode(w))
    finally:
        lra.lra_set_decode_split_keys(old)


# sequences, agents, Hq, Hkv, d, r, longest (shares of 128 keys): a wave per row at ranks above 16, up to four shares and more (a second
# request of B_V above rank 32), more than 16 and 32, groups of 16, 7 and 4
WAVE_CASES = [
    (40, 8, 16, 1, 128, 64, 500), (40, 8, 16, 1, 128, 36, 600), (20, 8, 16, 1, 128, 40, 2300), (20, 8, 32, 8, 64, 48, 4300),
    (37, 5, 14, 2, 64, 24, 700), (21, 4, 32, 8, 128, 32, 450),
]


@pytest.mark.parametrize("case", WAVE_CASES, ids=lambda c: "q%dx%d_%dover%d_d%d_r%d_n%d" % c)
def test_a_wave_per_row(case):
    seqs, agents, hq, hkv, d, r, longest = case
    lens = [longest] + [int(x) for x in np.random.default_rng(sum(case)).integers(1, longest, size=seqs - 1)]
    w = W.make_paged("merge", seed=sum(case), seq_lens=lens, agents_per_seq=agents, n_adapters=3, n_q_heads=hq, n_kv_heads=hkv,
                     head_dim=d, rank=r, d_model=None, b_std=0.05)
    old = lra.lra_set_decode_split_keys(128)
    try:
        _check(run_decode(w, DEV), oracle_decode(w))
    finally:
        lra.lra_set_decode_split_keys(old)


@pytest.mark.parametrize("case", [
    # new tokens, keys, Hq, Hkv, d, r, shares
    (70, 700, 32, 8, 128, 16, 4), (70, 1400, 32, 8, 128, 16, 9), (90, 1300, 32, 8, 64, 16, 11), (90, 700, 28, 4, 128, 24, 3),
    (170, 900, 32, 8, 128, 32, 5), (81, 1500, 32, 8, 128, 64, 8), (81, 1500, 32, 8, 64, 48, 13),
], ids=lambda c: "n%dof%d_%dover%d_d%d_r%d_s%d" % c)
def test_many_rows_of_prefills(case):
    n_new, n, hq, hkv, d, r, shares = case
    w = W.make_contiguous("merge", "prefill", seed=sum(case), n_agents=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, rank=r, n=n,
                          n_new=n_new, b_std=0.05)
    old = lra.lra_set_prefill_splits(shares)
    try:
        _check(run_prefill(w, DEV), oracle_prefill(w))
    finally:
        lra.lra_set_prefill_splits(old)
