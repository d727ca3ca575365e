"""Decode with one low-rank cache per adapter on one contiguous sequence, in both layouts of the workgroup index (key shares that
fill the XCDs evenly, and not): one to eight row groups, share counts on and off a multiple of eight.  Same gate as everywhere."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_01053_amd as lra
from tests.harness import MAX_ABS_TOL, REL_L2_TOL, errors

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # keys, agents, Hq, Hkv, d, r
    (3900, 4, 32, 8, 128, 16),   # one row group, 31 shares
    (1500, 6, 32, 8, 128, 32),   # three, ten or eleven shares
    (700, 8, 16, 8, 128, 64),    # eight row groups of one agent, four shares
    (900, 3, 28, 4, 128, 64),    # three, eight shares
    (1025, 6, 28, 4, 128, 16),   # three row groups of two agents of seven heads
    (2100, 5, 12, 12, 64, 32),
]


@pytest.mark.parametrize("key_side", [True, False], ids=["key", "value"])
@pytest.mark.parametrize("n,agents,hq,hkv,d,r", CASES)
def test_decode(n, agents, hq, hkv, d, r, key_side):
    gen = torch.Generator().manual_seed(n)
    k, v = (torch.randn(n, hkv, d, generator=gen).to(torch.bfloat16) for _ in range(2))
    ls = torch.randn(agents, n, r, generator=gen).to(torch.bfloat16)
    bk, bv = ((0.05 * torch.randn(agents, r, hkv * d, generator=gen)).to(torch.bfloat16) for _ in range(2))
    q = torch.randn(agents, hq, d, generator=gen).to(torch.bfloat16)
    kd, vd, ld, bkd, bvd, qd = (t.to(DEV) for t in (k, v, ls, bk, bv, q))
    lens = torch.tensor([n], dtype=torch.int32, device=DEV)
    adapter_of = [(3 * a + 1) % agents for a in range(agents)]
    shape = lra.make_shape(qd, hkv, r, 0.0)
    cache = lra.make_cache(kd, vd, ld, lens, n, None, l_per_adapter=True)
    out = torch.full_like(qd, float("nan"))
    ws = torch.empty(lra.lra_workspace_bytes(shape, cache, agents, agents), dtype=torch.uint8, device=DEV)
    qa, qs = torch.tensor(adapter_of, dtype=torch.int32, device=DEV), torch.tensor([0, agents], dtype=torch.int32, device=DEV)
    lra.lra_attn_decode(shape, cache, bkd if key_side else None, bvd, agents, qd, qa, qs, agents, out, ws)
    torch.cuda.synchronize()
    f = lambda t: t.to(torch.float64).cpu().numpy()
    ref = np.concatenate([oracle.decode(f(q[i:i + 1]), f(k), f(v), f(ls[a]), f(bk) * key_side, f(bv), np.array([a]), np.array([0, 1]), [n],
                                        1.0 / d ** 0.5) for i, a in enumerate(adapter_of)])
    rel, mx = errors(f(out), ref)
    print(f"relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL
