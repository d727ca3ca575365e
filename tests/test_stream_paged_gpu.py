"""One sequence of a paged cache on the streaming kernel against the oracle: tiles that end inside a block, key ranges of one,
two and more tiles per wave, one and two row tiles, Qt from the pre-pass, low-rank rows with a pitch, tables whose places behind
the sequence name no block, sequences shorter than the plan's longest, few-token prefills.  Same gate as everywhere."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_01053_amd as lra
from paper_2602_01053_amd import workloads as W
from paper_2602_01053_amd.runner import DeviceWorkload
from tests.harness import MAX_ABS_TOL, REL_L2_TOL, _f64, errors, oracle_decode

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # keys, agents, Hq, Hkv, d, r, key side, places of the table beyond the sequence
    (1, 1, 8, 2, 128, 16, True, 3),
    (127, 3, 28, 4, 128, 24, True, 0),
    (1009, 5, 32, 8, 128, 32, True, 0),      # two row tiles, split issue
    (4113, 4, 8, 8, 64, 8, False, 900),      # group of one; two thirds of the shares find nothing
    (9001, 2, 32, 8, 128, 64, True, 1),      # more than two tiles per wave, hand-over in a stage
    (8193, 8, 32, 8, 128, 64, True, 0),      # ... with Qt from the pre-pass
    (1100, 4, 32, 8, 128, 64, True, 0),      # one row tile of four slots: sixteen blocks of B_K in the prologue
    (500, 3, 16, 4, 64, 40, True, 2),        # ... one slot empty, the last block half beyond the rank
    (5003, 3, 16, 1, 64, 48, True, 0),       # group of 16: two row groups, the second with a row tile of no agent
]


@pytest.mark.parametrize("case", CASES, ids=[f"n{c[0]}_a{c[1]}_{c[2]}over{c[3]}_d{c[4]}_r{c[5]}" for c in CASES])
@pytest.mark.parametrize("pitch", [0, 8], ids=["dense", "pitch"])
def test_decode(case, pitch):
    n, agents, hq, hkv, d, r, key_side, beyond = case
    w = W.make_paged("paged", seed=n + r, seq_lens=[n], agents_per_seq=agents, n_adapters=max(agents, 2), n_q_heads=hq, n_kv_heads=hkv,
                     head_dim=d, rank=r, d_model=None, b_std=0.1)
    if not key_side:
        w.b_k.zero_()
    dw = DeviceWorkload(w, DEV)
    table = torch.full((1, dw.block_table.shape[1] + beyond), -1, dtype=torch.int32, device=DEV)
    table[:, :dw.block_table.shape[1]] = dw.block_table
    l = dw.l
    if pitch:
        l = torch.full((*dw.l.shape[:2], r + pitch), float("nan"), dtype=dw.l.dtype, device=DEV)
        l[:, :, :r] = dw.l
        l = l[:, :, :r]
    dw.cache = lra.make_cache(dw.k_base, dw.v_base, l, dw.seq_lens, n + 16 * beyond, table)
    dw.b_k = dw.b_k if key_side else None
    dw.alloc_workspace()
    dw.out.fill_(float("nan"))
    dw.decode()
    torch.cuda.synchronize()
    rel, mx = errors(dw.out.to(torch.float64).cpu().numpy(), oracle_decode(w))
    print(f"relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL


@pytest.mark.parametrize("n_new,n,r", [(4, 20000, 16), (3, 9005, 64), (4, 777, 32)])
def test_prefill_of_a_few_tokens(n_new, n, r):
    """The second of two sequences: its row of the table, its length, its adapter."""
    hq, hkv, d = 32, 8, 128
    gen = torch.Generator().manual_seed(n)
    w = W.make_paged("paged", seed=n, seq_lens=[333, n], agents_per_seq=1, n_adapters=3, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, rank=r,
                     d_model=None, b_std=0.1)
    dw = DeviceWorkload(w, DEV)
    q = torch.randn(n_new, hq, d, generator=gen).to(torch.bfloat16)
    out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device=DEV)
    ws = torch.empty(lra.lra_workspace_bytes(dw.shape, dw.cache, 1, 1, n_new), dtype=torch.uint8, device=DEV)
    lra.lra_attn_prefill(dw.shape, dw.cache, dw.b_k, dw.b_v, 3, q.to(DEV), 1, 2, out, ws)
    torch.cuda.synchronize()
    rows = [(int(w.block_table[1, j // 16]), j % 16) for j in range(n)]
    b, o = torch.tensor([x for x, _ in rows]), torch.tensor([x for _, x in rows])
    k, v, l = (_f64(t) for t in (w.k_base[b, :, o], w.v_base[b, :, o], w.l[b, o]))
    ref = oracle.prefill(_f64(q), k, v, l, _f64(w.b_k[2]), _f64(w.b_v[2]), n=n, scale=w.scale)
    rel, mx = errors(out.to(torch.float64).cpu().numpy(), ref)
    print(f"relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL
