"""The rotary form of the split-KV kernel against the oracle where its layout can go wrong: units whose two workgroups hold
unequal shares, last tiles of one key, agent slots that are empty, one wave without keys, blocks of 16 keys that end inside a
request of 32 low-rank rows, sequences shorter than the plan's longest.  Same gate as everywhere: bf16 operands of the
products (2^-9 each) leave 2e-3 of the output, of which 1.7e-3 is the rounding of the result itself."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_01053_amd as lra
from paper_2602_01053_amd import workloads as W
from paper_2602_01053_amd.runner import DeviceWorkload
from tests.harness import MAX_ABS_TOL, REL_L2_TOL, _f64, errors

pytestmark = pytest.mark.gpu
THETA = 500000.0

CASES = [
    # keys, agents, Hq, Hkv, d, r, paged, longest the plan allows for (0: the sequence)
    (8193, 4, 32, 8, 128, 8, False, 0),     # 65 tiles on 32 units: loads of 3, the first 32 shares twice the size of the rest
    (9088, 1, 32, 8, 128, 16, True, 0),     # ... and one of four slots
    (12417, 3, 28, 4, 128, 32, True, 0),    # two row groups, the second with an empty slot
    (6145, 5, 8, 8, 128, 24, False, 0),     # group of one, 5 agents in two row groups
    (20011, 2, 16, 8, 64, 16, True, 0),     # 64 wide
    (5000, 3, 32, 8, 128, 16, False, 20011),  # most shares find nothing
    (129, 4, 8, 2, 128, 8, True, 0),        # a tile and a key
    (17, 2, 8, 2, 64, 40, True, 0),         # one workgroup, three waves without keys
    (3001, 4, 16, 1, 128, 64, True, 0),     # group of 16: a slot fills the tile
    (2500, 9, 20, 5, 64, 40, True, 0),      # three row groups, ten shares of which eight meet on an XCD
    (3001, 7, 20, 5, 128, 24, False, 0),    # four, twelve of which eight
]


@pytest.mark.parametrize("case", CASES, ids=[f"n{c[0]}_a{c[1]}_{c[2]}over{c[3]}_d{c[4]}_r{c[5]}{'_paged' if c[6] else ''}" for c in CASES])
def test_decode(case):
    n, agents, hq, hkv, d, r, paged, longest = case
    kw = dict(seed=n, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, rank=r, d_model=None, b_std=0.1)
    if paged:
        w = W.make_paged("rope", seq_lens=[n], agents_per_seq=agents, n_adapters=max(agents, 2), **kw)
    else:
        w = W.make_contiguous("rope", "decode", n_agents=agents, n=n, **kw)
    dw = DeviceWorkload(w, "cuda:0", key_rope_theta=THETA)
    if longest:
        dw.cache.max_seq_len = longest
    dw.alloc_workspace()
    dw.out.fill_(float("nan"))
    dw.decode()
    torch.cuda.synchronize()
    ref = oracle.decode(_f64(w.q), _f64(w.k_base), _f64(w.v_base), _f64(w.l), _f64(w.b_k), _f64(w.b_v), w.query_adapter.numpy(),
                        w.seq_query_start.numpy(), w.seq_lens, w.scale, block_size=w.block_size,
                        block_table=None if w.block_table is None else w.block_table.numpy(), key_rope_theta=THETA)
    rel, mx = errors(dw.out.to(torch.float64).cpu().numpy(), ref)
    print(f"relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL


ROW_LENS = [9000, 8700, 129, 1, 2500, 4000]


def test_batch_in_one_row_at_rank_16():
    """128 wide, ranks up to 16, the shares of all sequences in one row."""
    w = W.make_paged("rope", seed=5, seq_lens=ROW_LENS, agents_per_seq=3, n_adapters=3, n_q_heads=32, n_kv_heads=8,
                     head_dim=128, rank=16, d_model=None, b_std=0.1)
    ref = oracle.decode(_f64(w.q), _f64(w.k_base), _f64(w.v_base), _f64(w.l), _f64(w.b_k), _f64(w.b_v), w.query_adapter.numpy(),
                        w.seq_query_start.numpy(), w.seq_lens, w.scale, block_size=w.block_size, block_table=w.block_table.numpy(),
                        key_rope_theta=THETA)
    for host_lens in (True, False):
        dw = DeviceWorkload(w, "cuda:0", key_rope_theta=THETA, host_lens=host_lens)
        dw.alloc_workspace()
        dw.out.fill_(float("nan"))
        dw.decode()
        torch.cuda.synchronize()
        rel, mx = errors(dw.out.to(torch.float64).cpu().numpy(), ref)
        assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL


PREFILL_CASES = [
    # keys, new tokens, Hq, Hkv, d, r: the first shares a tile longer than the rest
    (9000, 8, 32, 8, 128, 8),       # 71 tiles, 16 shares of three and 12 of two; two row groups
    (9089, 5, 32, 8, 128, 16),      # 72 tiles, the last of one key; a row group of one token
    (12417, 6, 32, 8, 128, 24),
    (10348, 25, 12, 12, 128, 16),   # seven row groups, six shares
    (16584, 27, 16, 16, 64, 16),
]
REST_CASES = [
    # ... and as many shares as do not all meet on an XCD: whole blocks of eight, eight and two, none, with a rest
    (3001, 12, 20, 5, 128, 24),     # twelve shares, three row groups
    (4000, 21, 12, 12, 128, 32),    # seven, six row groups
    (700, 10, 20, 5, 128, 48),      # six
]


@pytest.mark.parametrize("paged", [False, True], ids=["contiguous", "paged"])
@pytest.mark.parametrize("case", PREFILL_CASES + REST_CASES, ids=lambda c: f"n{c[0]}_new{c[1]}_{c[2]}over{c[3]}_d{c[4]}_r{c[5]}")
def test_prefill_of_a_few_tokens(case, paged):
    n, n_new, hq, hkv, d, r = case
    w = W.make_paged("rope", seed=n, seq_lens=[n], agents_per_seq=1, n_adapters=2, n_q_heads=hq, n_kv_heads=hkv, head_dim=d, rank=r,
                     d_model=None, b_std=0.1)
    j = torch.arange(n)
    blk = w.block_table[0, j // 16].long()
    k, v, l = w.k_base[blk, :, j % 16], w.v_base[blk, :, j % 16], w.l[blk, j % 16]
    dw = DeviceWorkload(w, "cuda:0", key_rope_theta=THETA)
    held = [t.contiguous().to("cuda:0") for t in (k, v, l)]  # (the cache holds addresses only)
    cache = dw.cache if paged else lra.make_cache(*held, dw.seq_lens, n, None)
    q = torch.randn(n_new, hq, d, generator=torch.Generator().manual_seed(n)).to(torch.bfloat16)
    out = torch.full(q.shape, float("nan"), dtype=torch.bfloat16, device="cuda:0")
    ws = torch.full((lra.lra_workspace_bytes(dw.shape, cache, 1, 1, n_new),), 0xFF, dtype=torch.uint8, device="cuda:0")
    qd = q.to("cuda:0")
    lra.lra_attn_prefill(dw.shape, cache, dw.b_k, dw.b_v, 2, qd, 0, 1, out, ws)
    torch.cuda.synchronize()
    ref = oracle.prefill(_f64(q), _f64(k), _f64(v), _f64(l), _f64(w.b_k[1]), _f64(w.b_v[1]), n=n, scale=w.scale, key_rope_theta=THETA)
    rel, mx = errors(out.to(torch.float64).cpu().numpy(), ref)
    print(f"relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL
