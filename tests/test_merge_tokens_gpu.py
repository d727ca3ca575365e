"""The merge of long prefills whose keys are dealt to shares (four rows of a kv head per wave; the two cases of rank 8: a wave per row)
against the oracle: rows that do not fill a wave, a share that the first rows do not reach, ranks below, at and above sixteen rows
of B_V, both head dims, no value side, three shares to sixteen.  tests/test_gpu_cases_plan_cpu.py asks which form each case takes.
Same gate as everywhere."""
import pytest
import torch

import oracle
import paper_2602_01053_amd as lra
from paper_2602_01053_amd import workloads as W
from paper_2602_01053_amd.runner import DeviceWorkload
from tests.harness import MAX_ABS_TOL, REL_L2_TOL, _f64, errors, oracle_prefill

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # new tokens, keys, Hq, Hkv, d, r, value side
    (331, 3000, 28, 4, 128, 24, True),   # 2317 rows of a kv head: a wave with one row
    (577, 2400, 16, 2, 128, 8, True),    # group of 8
    (293, 2500, 32, 8, 64, 64, True),
    (289, 2049, 32, 8, 64, 8, False),
    (384, 4000, 24, 2, 128, 40, True),   # 9216 rows
    (297, 1100, 32, 8, 128, 20, True),   # a rank that is no multiple of eight: the vector kernel's states, one share
]

SHARE_CASES = [
    # ... and the shares, told: four rows per wave for each
    (90, 1300, 32, 8, 128, 48, True, 5), (90, 1301, 32, 8, 64, 64, False, 4), (170, 1400, 32, 8, 128, 64, True, 9),
    (170, 1401, 32, 8, 64, 40, False, 10), (171, 1402, 32, 8, 128, 24, False, 3), (170, 1403, 32, 8, 64, 24, True, 10),
    (1845, 2500, 5, 1, 64, 16, True, 13), (1845, 2501, 5, 1, 64, 8, False, 16), (1845, 2502, 5, 1, 128, 8, True, 5),
]


@pytest.mark.parametrize("n_new,n,hq,hkv,d,r,value_side,shares", SHARE_CASES)
def test_shares(n_new, n, hq, hkv, d, r, value_side, shares):
    w = W.make_contiguous("merge", "prefill", seed=n, n_agents=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, rank=r, n=n, n_new=n_new, b_std=0.1)
    if not value_side:
        w.b_v.zero_()
    dw = DeviceWorkload(w, DEV)
    dw.b_v = dw.b_v if value_side else None
    old = lra.lra_set_prefill_splits(shares)
    try:
        dw.alloc_workspace()
        dw.out.fill_(float("nan"))
        dw.prefill()
        torch.cuda.synchronize()
    finally:
        lra.lra_set_prefill_splits(old)
    rel, mx = errors(dw.out.to(torch.float64).cpu().numpy(), oracle_prefill(w))
    print(f"relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL


@pytest.mark.parametrize("n_new,n,hq,hkv,d,r,value_side", CASES)
def test_prefill(n_new, n, hq, hkv, d, r, value_side):
    w = W.make_paged("paged", seed=n, seq_lens=[n], agents_per_seq=1, n_adapters=2, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, rank=r,
                     d_model=None, b_std=0.1)
    dw = DeviceWorkload(w, DEV)
    shares = lra.lra_workspace_bytes(dw.shape, dw.cache, 1, 1, n_new) // (n_new * hq * (d + r) * 4)
    assert 2 <= shares <= 16 or (shares == 1 and r % 8)
    q = torch.randn(n_new, hq, d, generator=torch.Generator().manual_seed(n)).to(torch.bfloat16)
    out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device=DEV)
    ws = torch.empty(lra.lra_workspace_bytes(dw.shape, dw.cache, 1, 1, n_new), dtype=torch.uint8, device=DEV)
    lra.lra_attn_prefill(dw.shape, dw.cache, dw.b_k, dw.b_v if value_side else None, 2, q.to(DEV), 0, 1, out, ws)
    torch.cuda.synchronize()
    b_v = _f64(w.b_v[1]) * (1.0 if value_side else 0.0)
    j = torch.arange(n)
    blk = w.block_table[0, j // 16].long()
    k, v, l = (_f64(t) for t in (w.k_base[blk, :, j % 16], w.v_base[blk, :, j % 16], w.l[blk, j % 16]))
    ref = oracle.prefill(_f64(q), k, v, l, _f64(w.b_k[1]), b_v, n=n, scale=w.scale)
    rel, mx = errors(out.to(torch.float64).cpu().numpy(), ref)
    print(f"relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL
