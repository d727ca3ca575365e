"""The exchange of prefill_rows_kernel where its layout can go wrong: one to nine 32-key tiles (waves without a key, a wave with two), rows of a
tile that end inside it, ranks that end inside a part of eight or sixteen, head dimensions with four and eight half blocks, no
value-side adapter, shares of the keys.  Same gate as everywhere."""
import pytest
import torch

from paper_2602_01053_amd import workloads as W
from paper_2602_01053_amd.runner import DeviceWorkload
from tests.harness import MAX_ABS_TOL, REL_L2_TOL, errors, oracle_prefill
from tests.test_stream_shares_cpu import _plan, runs  # noqa: F401 (a fixture)

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("d,r", [(128, 8), (128, 16), (128, 24), (128, 32), (64, 16), (64, 32)])
@pytest.mark.parametrize("n,n_new", [(9, 9), (33, 20), (130, 5), (255, 40), (280, 33), (2600, 38)])
@pytest.mark.parametrize("value_side", [True, False], ids=["value", "no_value"])
def test_prefill(runs, n, n_new, d, r, value_side):  # noqa: F811
    hq, hkv = 32, 8
    pl = _plan(runs, hq, hkv, d, r, [n], n_new=n_new, paged=False)
    assert pl["wave_rows"] or n == 2600
    w = W.make_contiguous("rows", "prefill", seed=n + r, n_agents=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, rank=r, n=n, n_new=n_new, b_std=0.1)
    if not value_side:
        w.b_v.zero_()
    dw = DeviceWorkload(w, DEV)
    dw.b_v = dw.b_v if value_side else None
    dw.alloc_workspace()
    dw.out.fill_(float("nan"))
    dw.prefill()
    torch.cuda.synchronize()
    rel, mx = errors(dw.out.to(torch.float64).cpu().numpy(), oracle_prefill(w))
    print(f"relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL
