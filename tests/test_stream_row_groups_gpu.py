"""Decode of one sequence by more agents than a workgroup's rows hold, the workgroups of a row group filled up to a multiple of
eight or not: share counts and kv heads that do not make one, two row groups and three.  Same gate as everywhere."""
import pytest
import torch

from paper_2602_01053_amd import workloads as W
from paper_2602_01053_amd.runner import DeviceWorkload
from tests.harness import MAX_ABS_TOL, REL_L2_TOL, errors, oracle_decode

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # keys, agents, Hq, Hkv, d, r
    (3700, 7, 28, 4, 128, 16),   # 29 shares of 4 heads, two row groups: three workgroups without a share
    (2570, 9, 28, 4, 128, 24),   # three row groups: not filled up
    (1700, 9, 20, 5, 64, 16),    # 14 shares of 5 heads
    (1000, 12, 16, 1, 128, 16),  # one kv head
    (900, 5, 24, 3, 128, 16),
]


@pytest.mark.parametrize("n,agents,hq,hkv,d,r", CASES)
@pytest.mark.parametrize("paged", [False, True], ids=["contiguous", "paged"])
def test_decode(n, agents, hq, hkv, d, r, paged):
    if paged:
        w = W.make_paged("paged", seed=n, seq_lens=[n], agents_per_seq=agents, n_adapters=agents, n_q_heads=hq, n_kv_heads=hkv, head_dim=d,
                         rank=r, d_model=None, b_std=0.1)
    else:
        w = W.make_contiguous("contiguous", "decode", seed=n, n_agents=agents, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, rank=r, n=n, b_std=0.1)
    dw = DeviceWorkload(w, DEV)
    dw.alloc_workspace()
    dw.out.fill_(float("nan"))
    dw.decode()
    torch.cuda.synchronize()
    rel, mx = errors(dw.out.to(torch.float64).cpu().numpy(), oracle_decode(w))
    print(f"relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL
