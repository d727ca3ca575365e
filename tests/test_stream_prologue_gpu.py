"""Streaming decode and few-token prefills where the prologue's division can go wrong: one and two row tiles, two waves to a tile, Qt
blocks from one to sixteen per tile (empty agent slots, ranks that end inside a block, Qt from the pre-pass and without one), no
key-side adapter, and streaming waves without a key, whose states the merge of the eight waves reads too.  (That these calls stream is
asked of the planner in tests/test_stream_shares_cpu.py.)  Same gate as everywhere."""
import pytest
import torch

import paper_2602_01053_amd as lra
from paper_2602_01053_amd import workloads as W
from paper_2602_01053_amd.runner import DeviceWorkload
from tests.harness import MAX_ABS_TOL, REL_L2_TOL, errors, oracle_decode, oracle_prefill, run_prefill

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _check(got, ref):
    rel, mx = errors(got, ref)
    print(f"relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL


CASES = [
    # keys, agents, Hq, Hkv, d, r, key side
    (31, 1, 8, 8, 64, 8, True), (97, 8, 32, 8, 128, 16, False), (300, 5, 32, 8, 128, 16, True), (700, 8, 32, 8, 64, 16, True),
    (1100, 3, 28, 4, 128, 16, True), (600, 4, 28, 4, 128, 32, True), (700, 2, 16, 1, 128, 64, True), (513, 2, 16, 1, 64, 48, True),
    (600, 7, 32, 8, 128, 24, True), (900, 2, 32, 8, 128, 64, True), (260, 6, 32, 8, 128, 40, False),
    (900, 8, 32, 8, 128, 64, True), (1000, 7, 32, 8, 64, 56, True),  # (with the pre-pass)
]


@pytest.mark.parametrize("n,agents,hq,hkv,d,r,key_side", CASES)
def test_decode(n, agents, hq, hkv, d, r, key_side):
    w = W.make_contiguous("prologue", "decode", seed=n + r, n_agents=agents, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, rank=r, n=n, b_std=0.1)
    if not key_side:
        w.b_k.zero_()
    dw = DeviceWorkload(w, DEV)
    dw.b_k = dw.b_k if key_side else None
    dw.alloc_workspace()
    dw.out.fill_(float("nan"))
    dw.decode()
    torch.cuda.synchronize()
    _check(dw.out.to(torch.float64).cpu().numpy(), oracle_decode(w))


def test_sixteen_blocks_of_each_of_two_row_tiles():
    """One forced share of a long paged sequence that three row groups read: its plan has no room for the pre-pass."""
    w = W.make_paged("prologue", seed=5, seq_lens=[11000], agents_per_seq=17, n_adapters=17, n_q_heads=32, n_kv_heads=8, head_dim=128,
                     rank=64, d_model=None, b_std=0.1)
    dw = DeviceWorkload(w, DEV)
    old = lra.lra_set_decode_split_keys(11000)
    try:
        dw.alloc_workspace()
        dw.out.fill_(float("nan"))
        dw.decode()
        torch.cuda.synchronize()
    finally:
        lra.lra_set_decode_split_keys(old)
    _check(dw.out.to(torch.float64).cpu().numpy(), oracle_decode(w))


PREFILL_CASES = [(1, 40, 8, 8, 64, 8), (7, 1000, 32, 8, 128, 16), (5, 900, 32, 8, 128, 64), (3, 700, 28, 4, 128, 24), (13, 600, 8, 2, 128, 48)]


@pytest.mark.parametrize("n_new,n,hq,hkv,d,r", PREFILL_CASES)
def test_few_new_tokens(n_new, n, hq, hkv, d, r):
    w = W.make_contiguous("prologue", "prefill", seed=n, n_agents=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, rank=r, n=n, n_new=n_new, b_std=0.1)
    old = lra.lra_set_short_prefill(33)  # (the split-KV path, whatever the sizes)
    try:
        _check(run_prefill(w, DEV), oracle_prefill(w))
    finally:
        lra.lra_set_short_prefill(old)
