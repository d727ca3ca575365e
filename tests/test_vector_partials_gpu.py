"""The vector-ALU partial kernel against the oracle where its layout can go wrong: sixteen keys to a wave and 64 to a step, so
lengths around both; ranks around the bound of 16 and no multiple of four; paged blocks; no key-side adapter; causal rows.
fp32 is held to 2e-5 (sums of a few hundred terms in fp32), bf16 to the gate of the parity tests."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_01053_amd as lra
from paper_2602_01053_amd import workloads as W
from paper_2602_01053_amd.runner import DeviceWorkload
from tests.harness import MAX_ABS_TOL, REL_L2_TOL, _f64, errors, oracle_prefill, run_prefill

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _check(got, ref, fp32):
    rel, mx = errors(got, ref)
    print(f"relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= (2e-5 if fp32 else REL_L2_TOL) and mx <= MAX_ABS_TOL


CASES = [
    # keys, rank, d, Hq, Hkv, fp32, paged, key-side adapter
    (1, 1, 64, 2, 2, True, False, True), (15, 5, 64, 4, 4, True, True, True), (16, 8, 128, 4, 2, True, False, False),
    (17, 16, 128, 6, 3, True, True, True), (63, 17, 64, 4, 1, True, False, True), (64, 64, 64, 4, 4, True, True, False),
    (65, 64, 128, 4, 4, True, False, True), (129, 24, 128, 7, 1, True, True, True), (700, 16, 64, 4, 4, True, False, True),
    (17, 12, 64, 4, 2, False, False, True), (65, 3, 128, 8, 8, False, True, True), (700, 63, 128, 4, 2, False, True, False),
    (300, 64, 64, 6, 2, False, False, True),
]


@pytest.mark.parametrize("case", CASES, ids=["n%d_r%d_d%d_%dover%d_%s%s%s" % (*c[:5], "fp32" if c[5] else "bf16", "_paged" * c[6], "" if c[7] else "_value")
                                             for c in CASES])
def test_decode(case):
    n, r, d, hq, hkv, fp32, paged, key_side = case
    kw = dict(seed=n + r, dtype=torch.float32 if fp32 else torch.bfloat16, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, rank=r, d_model=None,
              b_std=0.1)
    if paged:
        w = W.make_paged("valu", seq_lens=[n, 1, max(n // 2, 1)], agents_per_seq=2, n_adapters=3, **kw)
    else:
        w = W.make_contiguous("valu", "decode", n_agents=3, n=n, **kw)
    dw = DeviceWorkload(w, DEV)
    b_k = _f64(w.b_k)
    if not key_side:
        dw.b_k, b_k = None, np.zeros_like(b_k)
    old = lra.lra_set_kernel_variant(1)
    try:
        dw.alloc_workspace()
        dw.out.fill_(float("nan"))
        dw.decode()
        torch.cuda.synchronize()
    finally:
        lra.lra_set_kernel_variant(old)
    ref = oracle.decode(_f64(w.q), _f64(w.k_base), _f64(w.v_base), _f64(w.l), b_k, _f64(w.b_v), w.query_adapter.numpy(),
                        w.seq_query_start.numpy(), w.seq_lens, w.scale, block_size=w.block_size,
                        block_table=None if w.block_table is None else w.block_table.numpy())
    _check(dw.out.to(torch.float64).cpu().numpy(), ref, fp32)


@pytest.mark.parametrize("case", [(70, 70, 8, 128, 4, 2, True), (33, 200, 20, 64, 4, 4, True), (20, 150, 12, 128, 8, 1, False)],
                         ids=lambda c: "new%dof%d_r%d_d%d_%dover%d_%s" % (*c[:6], "fp32" if c[6] else "bf16"))
def test_causal_rows(case):
    n_new, n, r, d, hq, hkv, fp32 = case
    w = W.make_contiguous("valu", "prefill", seed=n, dtype=torch.float32 if fp32 else torch.bfloat16, n_agents=1, n_q_heads=hq,
                          n_kv_heads=hkv, head_dim=d, rank=r, n=n, n_new=n_new, b_std=0.1)
    old = lra.lra_set_kernel_variant(1)
    try:
        _check(run_prefill(w, DEV), oracle_prefill(w), fp32)
    finally:
        lra.lra_set_kernel_variant(old)
