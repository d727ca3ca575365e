"""Key shares of the streaming kernel that are no multiple of 128 keys (four waves, some with a 32-key tile more than the others):
counts of tiles per share from five on, short last shares, waves and whole shares without a key, paged and contiguous, one and two row
tiles, low-rank caches per adapter, the causal form.  Same gate as everywhere."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_01053_amd as lra
from paper_2602_01053_amd import workloads as W
from paper_2602_01053_amd.runner import DeviceWorkload
from tests.harness import MAX_ABS_TOL, REL_L2_TOL, _f64, errors, oracle_decode, oracle_prefill, run_prefill
from tests.test_gpu_cases_plan_cpu import _plan, planner  # noqa: F401 (a fixture)
from tests.test_stream_shares_cpu import runs  # noqa: F401 (a fixture)

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

CASES = [
    # keys, longest of the plan, agents, Hq, Hkv, d, r, paged, key share
    (4100, 4100, 4, 32, 8, 128, 16, False, 160), (4100, 5200, 4, 32, 8, 128, 16, True, 192), (6400, 6400, 8, 32, 8, 128, 16, False, 224),
    (9009, 9009, 4, 32, 8, 128, 24, False, 288), (10000, 10300, 2, 32, 8, 128, 64, False, 352), (3001, 3001, 3, 32, 32, 128, 8, False, 384),
    (13000, 13000, 4, 8, 8, 64, 16, False, 416), (9009, 9009, 3, 28, 4, 128, 16, True, 160),
]


def _check(got, ref):
    rel, mx = errors(got, ref)
    print(f"relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL


@pytest.mark.parametrize("n,longest,agents,hq,hkv,d,r,paged,share", CASES)
def test_decode(runs, n, longest, agents, hq, hkv, d, r, paged, share):  # noqa: F811
    assert _plan(runs, hq, hkv, d, r, [n], longest=longest, agents=agents, paged=paged)["split_keys"] == share
    kw = dict(seed=n + r, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, rank=r, b_std=0.1)
    if paged:
        w = W.make_paged("shares", seq_lens=[n], agents_per_seq=agents, n_adapters=agents, d_model=None, **kw)
    else:
        w = W.make_contiguous("shares", "decode", n_agents=agents, n=n, **kw)
    dw = DeviceWorkload(w, DEV)
    table = None
    if paged:
        table = torch.full((1, (longest + 15) // 16), -1, dtype=torch.int32, device=DEV)
        table[:, :dw.block_table.shape[1]] = dw.block_table
    dw.cache = lra.make_cache(dw.k_base, dw.v_base, dw.l, dw.seq_lens, longest, table)
    dw.alloc_workspace()
    dw.out.fill_(float("nan"))
    dw.decode()
    torch.cuda.synchronize()
    _check(dw.out.to(torch.float64).cpu().numpy(), oracle_decode(w))


def test_low_rank_cache_per_adapter():
    n, agents, hq, hkv, d, r = 6001, 4, 32, 8, 128, 16
    gen = torch.Generator().manual_seed(n)
    k, v = (torch.randn(n, hkv, d, generator=gen).to(torch.bfloat16) for _ in range(2))
    ls = torch.randn(agents, n, r, generator=gen).to(torch.bfloat16)
    bk, bv = ((0.05 * torch.randn(agents, r, hkv * d, generator=gen)).to(torch.bfloat16) for _ in range(2))
    q = torch.randn(agents, hq, d, generator=gen).to(torch.bfloat16)
    kd, vd, ld, bkd, bvd, qd = (t.to(DEV) for t in (k, v, ls, bk, bv, q))
    lens = torch.tensor([n], dtype=torch.int32, device=DEV)
    shape, cache = lra.make_shape(qd, hkv, r, 0.0), lra.make_cache(kd, vd, ld, lens, n, None, l_per_adapter=True)
    out = torch.full_like(qd, float("nan"))
    ws = torch.empty(lra.lra_workspace_bytes(shape, cache, agents, agents), dtype=torch.uint8, device=DEV)
    qa, qs = torch.arange(agents, dtype=torch.int32, device=DEV), torch.tensor([0, agents], dtype=torch.int32, device=DEV)
    lra.lra_attn_decode(shape, cache, bkd, bvd, agents, qd, qa, qs, agents, out, ws)
    torch.cuda.synchronize()
    ref = np.concatenate([oracle.decode(_f64(q[a:a + 1]), _f64(k), _f64(v), _f64(ls[a]), _f64(bk), _f64(bv), np.array([a]), np.array([0, 1]),
                                        [n], 1.0 / d ** 0.5) for a in range(agents)])
    _check(out.to(torch.float64).cpu().numpy(), ref)


@pytest.mark.parametrize("n_new,n,hq,hkv,r", [(8, 6001, 32, 8, 16), (3, 10000, 28, 4, 24), (12, 3500, 32, 8, 8)])
def test_few_new_tokens(runs, n_new, n, hq, hkv, r):  # noqa: F811
    pl = _plan(runs, hq, hkv, 128, r, [n], n_new=n_new, paged=False)
    assert pl["short_prefill"] and pl["wave_shares"] == 0 and not pl["wave_rows"] and pl["split_keys"] % 32 == 0
    w = W.make_contiguous("shares", "prefill", seed=n, n_agents=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=128, rank=r, n=n, n_new=n_new, b_std=0.1)
    _check(run_prefill(w, DEV), oracle_prefill(w))


def test_workspace_without_room_for_these_shares():
    """17 shares of 256 keys where 26 of 160 do not fit; below that the call is refused."""
    n, agents, hq, hkv, d, r = 4100, 4, 32, 8, 128, 16
    w = W.make_contiguous("shares", "decode", seed=3, n_agents=agents, n=n, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, rank=r, b_std=0.1)
    dw = DeviceWorkload(w, DEV)
    dw.alloc_workspace()
    slots, align = agents * hq * 17, lambda x: (x + 255) // 256 * 256
    least = align(slots * 8) + align(slots * d * 4) + align(slots * r * 4) + align(agents * hq * 4)
    assert least < dw.workspace.numel()
    dw.workspace = torch.empty(least, dtype=torch.uint8, device=DEV)
    dw.out.fill_(float("nan"))
    dw.decode()
    torch.cuda.synchronize()
    _check(dw.out.to(torch.float64).cpu().numpy(), oracle_decode(w))
    dw.workspace = torch.empty(least - 256, dtype=torch.uint8, device=DEV)
    with pytest.raises(lra.LraError):
        dw.decode()


def test_few_new_tokens_without_room_for_these_shares(runs, planner):  # noqa: F811
    """A few-token prefill whose workspace has room for the shares of its other path only: that path runs, and below its need the
    call is refused."""
    n_new, n, hq, hkv, d, r = 8, 4500, 32, 8, 128, 16
    a = (hq, hkv, d, r, [n])
    other, run = (_plan(x, *a, n_new=n_new, paged=False) for x in (planner, runs))
    assert run["short_prefill"] and not other["short_prefill"] and not other["wave_rows"]
    align = lambda x: (x + 255) // 256 * 256
    rows, shares = n_new * hq, other["n_splits"]
    need = lambda k: align(rows * k * 8) + align(rows * k * d * 4) + align(rows * k * r * 4) + align(rows * 4)
    assert need(shares) < need(run["n_splits"])
    w = W.make_contiguous("shares", "prefill", seed=4, n_agents=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, rank=r, n=n, n_new=n_new, b_std=0.1)
    ref = oracle_prefill(w)
    dw = DeviceWorkload(w, DEV)
    dw.alloc_workspace()
    assert dw.workspace.numel() == need(run["n_splits"])
    outs = []
    for nbytes in (need(run["n_splits"]), need(run["n_splits"]) - 256, need(shares)):
        dw.workspace = torch.empty(nbytes, dtype=torch.uint8, device=DEV)
        dw.out.fill_(float("nan"))
        dw.prefill()
        torch.cuda.synchronize()
        outs.append(dw.out.to(torch.float64).cpu().numpy())
        _check(outs[-1], ref)
    assert (outs[1] == outs[2]).all() and (outs[0] != outs[1]).any()  # (one path with either of the smaller ones, another with the largest)
    dw.workspace = torch.empty(need(shares) - 256, dtype=torch.uint8, device=DEV)
    with pytest.raises(lra.LraError):
        dw.prefill()
