"""Scores of minus infinity and NaN in the kernels that keep several softmax states per row: keys whose score falls below the
type (a mask of its lowest value) have no weight, wherever in a wave, a step or a key share they stand."""
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
