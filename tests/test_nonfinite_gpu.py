"""Scores of minus infinity and NaN in the kernels that keep several softmax states per row: keys whose score falls below the
type (a mask of its lowest value) have no weight, wherever in a wave, a step or a key share they stand; a key of NaN reaches every
output that reads it, through every form of the merge."""
import numpy as np
import pytest
import torch

import paper_2602_01053_amd as lra
from paper_2602_01053_amd import workloads as W
from paper_2602_01053_amd.runner import DeviceWorkload
from tests.harness import MAX_ABS_TOL, REL_L2_TOL, errors, oracle_decode, oracle_prefill

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _run(w, prefill=False):
    dw = DeviceWorkload(w, DEV)
    dw.alloc_workspace()
    dw.out.fill_(float("nan"))
    dw.prefill() if prefill else dw.decode()
    torch.cuda.synchronize()
    return dw.out.to(torch.float64).cpu().numpy()


# (keys without weight, a range: the first sixteen, a wave's of the first and of a later step, a whole step, a whole share of 256,
# all but the last)
MASKS = [(0, 16), (16, 32), (112, 128), (0, 64), (320, 384), (256, 512), (0, 599)]


@pytest.mark.parametrize("lo,hi", MASKS)
@pytest.mark.parametrize("fp32,d,prefill", [(True, 64, False), (True, 128, True), (False, 128, False), (False, 64, True)])
def test_vector_alu_partials_with_keys_below_the_type(lo, hi, fp32, d, prefill):
    n, n_new = 600, 40
    if prefill and hi > n - n_new:
        hi = n - n_new  # (every new token keeps a key)
    w = W.make_contiguous("mask", "prefill" if prefill else "decode", seed=lo + hi, dtype=torch.float32 if fp32 else torch.bfloat16,
                          n_agents=1 if prefill else 2, n_q_heads=4, n_kv_heads=2, head_dim=d, rank=12, n=n,
                          n_new=n_new if prefill else 1, b_std=0.1)
    w.q.abs_().add_(0.5)                            # (so that the lowest value gives minus infinity)
    w.k_base[lo:hi] = torch.finfo(w.k_base.dtype).min
    old = lra.lra_set_kernel_variant(1), lra.lra_set_decode_split_keys(256)
    try:
        got = _run(w, prefill)
    finally:
        lra.lra_set_kernel_variant(old[0])
        lra.lra_set_decode_split_keys(old[1])
    rel, mx = errors(got, oracle_prefill(w) if prefill else oracle_decode(w))
    print(f"relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= (2e-5 if fp32 else REL_L2_TOL) and mx <= MAX_ABS_TOL


def _nan_rows(got, ref, nan):
    """Rows of `nan` all NaN, the others as the oracle has them without that key."""
    assert np.isnan(got[nan]).all(), f"{np.isnan(got[nan]).mean():.3f} of the outputs that read the key are NaN"
    rel, mx = errors(got[~nan], ref[~nan])
    print(f"relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL


@pytest.mark.parametrize("valu", [False, True])
@pytest.mark.parametrize("d,r,shares", [(128, 16, 9), (64, 40, 40), (128, 24, 70)])
def test_nan_of_one_share_reaches_the_output(d, r, shares, valu):
    """A key row of NaN in the last of several shares, in calls of few rows (one workgroup per row, and beyond 64 shares the form for
    any number): its kv head's outputs are NaN, not the attention over the other shares."""
    n = 64 * (shares - 1) + (128 if not valu else 9)
    w = W.make_contiguous("nan", "decode", seed=n, n_agents=2, n_q_heads=8, n_kv_heads=2, head_dim=d, rank=r, n=n, b_std=0.1)
    ref = oracle_decode(w)
    w.k_base[n - 3, 1] = float("nan")
    old = lra.lra_set_kernel_variant(int(valu)), lra.lra_set_decode_split_keys(64)
    try:
        got = _run(w)
    finally:
        lra.lra_set_kernel_variant(old[0])
        lra.lra_set_decode_split_keys(old[1])
    nan = np.zeros(got.shape[:2], bool)
    nan[:, 4:] = True
    _nan_rows(got, ref, nan)


@pytest.mark.parametrize("valu", [False, True])
@pytest.mark.parametrize("d,r", [(128, 16), (64, 8), (128, 40)])
def test_nan_of_one_share_in_many_rows(d, r, valu):
    """The same with a wave per row: 2560 rows of a ragged batch, the key in the longest sequence's last share."""
    lens = [700, 690, 120, 333, 64, 500, 9, 650, 480, 256, 300, 610, 77, 420, 512, 20, 640, 350, 128, 699]
    w = W.make_paged("nan", seed=d + r, seq_lens=lens, agents_per_seq=4, n_adapters=3, n_q_heads=32, n_kv_heads=8, head_dim=d, rank=r,
                     d_model=None, b_std=0.05)
    ref = oracle_decode(w)
    w.k_base[int(w.block_table[0, 690 // 16]), 5, 690 % 16] = float("nan")
    old = lra.lra_set_kernel_variant(int(valu)), lra.lra_set_decode_split_keys(128)
    try:
        got = _run(w)
    finally:
        lra.lra_set_kernel_variant(old[0])
        lra.lra_set_decode_split_keys(old[1])
    nan = np.zeros(got.shape[:2], bool)
    nan[:4, 20:24] = True
    _nan_rows(got, ref, nan)


@pytest.mark.parametrize("d,r,shares", [(128, 48, 4), (64, 64, 9), (128, 16, 5)])
def test_nan_of_one_share_of_a_prefill(d, r, shares):
    """Rows of new tokens, shares of the keys: four rows per wave, and one."""
    n, n_new = 1300, 90
    w = W.make_contiguous("nan", "prefill", seed=shares, n_agents=1, n_q_heads=32, n_kv_heads=8, head_dim=d, rank=r, n=n, n_new=n_new, b_std=0.05)
    ref = oracle_prefill(w)
    w.k_base[n - n_new - 2, 3] = float("nan")
    old = lra.lra_set_prefill_splits(shares)
    try:
        got = _run(w, prefill=True)
    finally:
        lra.lra_set_prefill_splits(old)
    nan = np.zeros(got.shape[:2], bool)
    nan[:, 12:16] = True
    _nan_rows(got, ref, nan)


@pytest.mark.parametrize("lo,hi", [(0, 32), (128, 160), (160, 192), (192, 224), (480, 512), (160, 320), (0, 480), (0, 4099)])
@pytest.mark.parametrize("agents,prefill", [(2, False), (8, False), (1, True)])
def test_streaming_kernel_with_keys_below_the_type(lo, hi, agents, prefill):
    """Key shares of 160 keys, of which a wave of the streaming kernel has one 32-key tile or two: a tile, a share or several without
    weight, where a wave or a share begins and elsewhere."""
    n = 4100 if agents < 8 else 4500
    if prefill:
        n, hi = 4500, min(hi, 4492)
    w = W.make_contiguous("mask", "prefill" if prefill else "decode", seed=lo + hi + agents, n_agents=agents, n_q_heads=32, n_kv_heads=8,
                          head_dim=128, rank=16, n=n, n_new=8 if prefill else 1, b_std=0.1)
    w.q.abs_().add_(0.5)
    w.k_base[lo:hi] = torch.finfo(w.k_base.dtype).min
    rel, mx = errors(_run(w, prefill), oracle_prefill(w) if prefill else oracle_decode(w))
    print(f"relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL
