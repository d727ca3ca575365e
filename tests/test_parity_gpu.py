"""Parity of the HIP library against the fp64 oracle, through the C ABI.

Bar (stated for bf16 inputs with fp32 accumulation): relative L2 <= 5e-3 over the
whole output AND over every single query / new token, max-abs <= 2e-2.  fp32
inputs are additionally held to relative L2 <= 2e-5.
"""
import numpy as np
import pytest
import torch

import paper_2602_01053_amd as lra
from paper_2602_01053_amd import workloads as W
from tests.harness import (MAX_ABS_TOL, REL_L2_TOL, DeviceWorkload, errors, oracle_decode,
                           oracle_prefill, oracle_prefill_by_blocks, run_decode, run_prefill)

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


# 0: automatic choice (bf16: MFMA kernels, and among them the one-workgroup-per-CU streaming form of the
# split-KV kernel wherever a call qualifies); 1: vector-ALU kernels; 2: MFMA kernels without the streaming form
@pytest.fixture(params=[0, 1, 2], ids=["auto", "valu", "mfma_no_stream_form"])
def variant(request):
    old = lra.lra_set_kernel_variant(request.param)
    yield request.param
    lra.lra_set_kernel_variant(old)


def _gate(got, ref, fp32=False, label=""):
    rel, mx = errors(got, ref)
    print(f"{label}: relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL, (label, rel, mx)
    if fp32:
        assert rel <= 2e-5, (label, rel)


# ---- the five named configurations at full size -----------------------------
def test_config1_tiny_decode_fp32(variant):
    w = W.config(1)
    _gate(run_decode(w, DEV), oracle_decode(w), fp32=True, label=w.name)


@pytest.mark.parametrize("head_major", [False, True], ids=["token_major", "head_major"])
def test_config2_llama_decode(variant, head_major):
    w = W.config(2)
    _gate(run_decode(w, DEV, head_major), oracle_decode(w), label=w.name)


def test_config4_long_multi_agent_decode(variant):
    w = W.config(4)
    _gate(run_decode(w, DEV), oracle_decode(w), label=w.name)


def test_config5_ragged_paged_decode():
    w = W.config(5)
    print("sum of lengths", sum(w.seq_lens), flush=True)
    _gate(run_decode(w, DEV), oracle_decode(w), label=w.name)


def test_config3_prefill_every_row():
    """Full-size causal prefill in the launch configuration the benchmark times, compared with the
    oracle on every one of its 2048 x 32 output rows."""
    w = W.config(3)
    got = run_prefill(w, DEV)
    assert np.isfinite(got).all()
    _gate(got, oracle_prefill_by_blocks(w), label=w.name)


# ---- small shapes: several tiles, ragged tails, odd groups ------------------
DECODE_CASES = [
    # n, agents, Hq, Hkv, d, r
    (1, 1, 4, 4, 64, 8),
    (17, 3, 8, 2, 128, 16),
    (63, 2, 4, 1, 64, 4),
    (64, 5, 8, 8, 128, 1),
    (65, 1, 14, 2, 128, 32),     # group of 7
    (257, 4, 32, 8, 128, 16),
    (1000, 7, 16, 4, 64, 24),
    (1031, 9, 16, 1, 128, 64),   # group of 16, > 8 agents
    (4099, 17, 4, 2, 128, 48),
]


@pytest.mark.parametrize("case", DECODE_CASES, ids=lambda c: "n%d_a%d_hq%d_hkv%d_d%d_r%d" % c)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
def test_decode_small_shapes(variant, case, dtype):
    n, agents, hq, hkv, d, r = case
    w = W.make_contiguous("small", "decode", seed=1000 + n, dtype=dtype, n_agents=agents,
                          n_q_heads=hq, n_kv_heads=hkv, head_dim=d, rank=r, n=n, d_model=None,
                          b_std=0.05)
    _gate(run_decode(w, DEV), oracle_decode(w), fp32=dtype == torch.float32, label=str(case))


PREFILL_CASES = [
    # n, n_new, Hq, Hkv, d, r
    (1, 1, 4, 4, 64, 8),
    (40, 40, 4, 2, 128, 16),       # no old context
    (130, 3, 8, 2, 128, 16),
    (200, 129, 4, 4, 64, 8),
    (513, 257, 14, 2, 128, 32),
    (1500, 300, 8, 1, 128, 64),
    (700, 200, 8, 2, 128, 24),     # rank padded to 32 inside the MFMA kernel
    (391, 150, 6, 2, 64, 48),      # rank padded to 64, half-empty last block
    (260, 131, 4, 4, 128, 20),     # rank not a multiple of 8: vector-ALU kernels
]


@pytest.mark.parametrize("case", PREFILL_CASES, ids=lambda c: "n%d_new%d_hq%d_hkv%d_d%d_r%d" % c)
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32], ids=["bf16", "fp32"])
def test_prefill_small_shapes(variant, case, dtype):
    n, n_new, hq, hkv, d, r = case
    w = W.make_contiguous("small", "prefill", seed=2000 + n, dtype=dtype, n_agents=1, n_q_heads=hq,
                          n_kv_heads=hkv, head_dim=d, rank=r, n=n, n_new=n_new, d_model=None,
                          b_std=0.05)
    _gate(run_prefill(w, DEV), oracle_prefill(w), fp32=dtype == torch.float32, label=str(case))


SHORT_PREFILL_CASES = [
    # n, n_new, Hq, Hkv, d, r
    (1000, 1, 8, 2, 128, 16),
    (1000, 7, 8, 2, 128, 16),
    (4099, 16, 32, 8, 128, 16),    # two row tiles, several splits
    (300, 13, 14, 2, 128, 32),     # group of 7: 8 rows per token, several row groups
    (777, 16, 16, 1, 64, 64),      # group of 16
    (64, 16, 4, 4, 64, 8),         # context exactly four times the new tokens
    (2000, 8, 8, 2, 128, 64),      # 4 token slots x 4 rank blocks x 2 row tiles: Qt comes from the pre-pass kernel
    (1500, 6, 16, 4, 64, 40),      # the same at d = 64, rank 40 (3 rank blocks), a ragged last row tile
]


@pytest.mark.parametrize("case", SHORT_PREFILL_CASES, ids=lambda c: "n%d_new%d_hq%d_hkv%d_d%d_r%d" % c)
@pytest.mark.parametrize("path", ["split_kv", "tile_walk"])
def test_short_prefill_both_paths(case, path):
    """A few new tokens after a longer context: served by the split-KV decode kernels with a
    causal limit per row (default) or by the tile-walking prefill kernel (path switched off);
    both must match the oracle."""
    n, n_new, hq, hkv, d, r = case
    w = W.make_contiguous("short_prefill", "prefill", seed=3000 + n + n_new, n_agents=1, n_q_heads=hq,
                          n_kv_heads=hkv, head_dim=d, rank=r, n=n, n_new=n_new, d_model=None, b_std=0.05)
    old = lra.lra_set_short_prefill(64 if path == "split_kv" else 0)
    old_s = lra.lra_set_prefill_splits(1)
    try:
        dw = DeviceWorkload(w, DEV)
        nbytes = dw.alloc_workspace()
        assert (nbytes > 0) == (path == "split_kv")
        dw.out.fill_(float("nan"))
        dw.prefill()
        torch.cuda.synchronize()
        got = dw.out.to(torch.float64).cpu().numpy()
    finally:
        lra.lra_set_short_prefill(old)
        lra.lra_set_prefill_splits(old_s)
    _gate(got, oracle_prefill(w), label=f"{case} {path}")


SPLIT_PREFILL_CASES = [
    # n, n_new, Hq, Hkv, d, r, splits (0 = automatic)
    (3000, 200, 8, 2, 128, 16, 0),     # automatic: few q tiles, several shares
    (2048, 130, 4, 4, 64, 8, 3),
    (5000, 700, 14, 2, 128, 32, 4),    # ragged last q tile, group of 7
    (1100, 1100, 4, 1, 128, 64, 2),    # no old context: later shares hold rows that see nothing of them
    (700, 300, 8, 2, 64, 48, 32),      # more shares than key tiles: empty shares
]


@pytest.mark.parametrize("case", SPLIT_PREFILL_CASES, ids=lambda c: "n%d_new%d_hq%d_hkv%d_d%d_r%d_s%d" % c)
def test_prefill_key_tiles_shared_by_workgroups(case):
    """The tile-walking prefill kernel with the key tiles of each q tile divided among several
    workgroups plus the merge kernel."""
    n, n_new, hq, hkv, d, r, splits = case
    w = W.make_contiguous("split_prefill", "prefill", seed=4000 + n + n_new, n_agents=1, n_q_heads=hq,
                          n_kv_heads=hkv, head_dim=d, rank=r, n=n, n_new=n_new, d_model=None, b_std=0.05)
    old_s = lra.lra_set_prefill_splits(splits)
    old_t = lra.lra_set_short_prefill(0)
    try:
        dw = DeviceWorkload(w, DEV)
        nbytes = dw.alloc_workspace()
        assert nbytes > 0
        dw.out.fill_(float("nan"))
        dw.prefill()
        torch.cuda.synchronize()
        got = dw.out.to(torch.float64).cpu().numpy()
    finally:
        lra.lra_set_prefill_splits(old_s)
        lra.lra_set_short_prefill(old_t)
    _gate(got, oracle_prefill(w), label=str(case))


PACKED_ROW_CASES = [
    # n, n_new, Hq, Hkv, d, r: the rows of a q tile are (new token, q head of the group) pairs
    (1300, 32, 8, 2, 128, 16),     # 128 rows: exactly one tile
    (1300, 33, 8, 2, 128, 16),     # 132: four rows in the second
    (97, 43, 9, 3, 128, 16),       # 129 rows in groups of 3: a token's heads lie in two tiles
    (55, 55, 7, 1, 128, 24),       # 385 rows in groups of 7, no old context: limits differ inside a wave
    (140, 129, 32, 2, 64, 8),      # group of 16
    (300, 129, 4, 4, 128, 64),     # group of 1
]


@pytest.mark.parametrize("case", PACKED_ROW_CASES, ids=lambda c: "n%d_new%d_hq%d_hkv%d_d%d_r%d" % c)
@pytest.mark.parametrize("splits", [1, 2])
def test_prefill_rows_of_all_heads_of_a_group_in_one_tile(case, splits):
    n, n_new, hq, hkv, d, r = case
    w = W.make_contiguous("packed_prefill", "prefill", seed=4500 + n + n_new, n_agents=1, n_q_heads=hq,
                          n_kv_heads=hkv, head_dim=d, rank=r, n=n, n_new=n_new, d_model=None, b_std=0.05)
    old_s = lra.lra_set_prefill_splits(splits)
    old_t = lra.lra_set_short_prefill(0)
    try:
        got = run_prefill(w, DEV)
    finally:
        lra.lra_set_prefill_splits(old_s)
        lra.lra_set_short_prefill(old_t)
    _gate(got, oracle_prefill(w), label=str(case))


TILE_CASES = [
    # n, n_new, Hq, Hkv, d, r: automatic plans on either side of the lengths and token counts where a q tile holds
    # 128 tokens of one q head (up to 1023 keys, or 64 tokens on up to 4096) or the rows of all heads of a group
    (1023, 300, 9, 3, 128, 16),
    (1024, 300, 9, 3, 128, 16),
    (1023, 64, 14, 2, 64, 64),
    (4096, 64, 14, 2, 64, 8),
    (4097, 64, 14, 2, 64, 8),
    (4096, 65, 16, 1, 128, 40),
    (130, 129, 16, 1, 128, 24),    # sixteen tile sets per kv head, one live row in the second tile of each
    (2500, 1300, 5, 1, 64, 16),    # several rounds of q tiles per head set
]


@pytest.mark.parametrize("kernels", [0, 2], ids=["auto", "tile_walk"])
@pytest.mark.parametrize("case", TILE_CASES, ids=lambda c: "n%d_new%d_hq%d_hkv%d_d%d_r%d" % c)
def test_prefill_tiles_of_one_head_or_of_a_group(case, kernels):
    """(Variant 2: at ranks up to 32 the automatic choice is the kernel whose waves divide the keys.)"""
    n, n_new, hq, hkv, d, r = case
    w = W.make_contiguous("head_tiles", "prefill", seed=4600 + n + n_new, n_agents=1, n_q_heads=hq, n_kv_heads=hkv,
                          head_dim=d, rank=r, n=n, n_new=n_new, d_model=None, b_std=0.05)
    old = lra.lra_set_kernel_variant(kernels)
    try:
        got = run_prefill(w, DEV)
    finally:
        lra.lra_set_kernel_variant(old)
    _gate(got, oracle_prefill(w), label=str(case))


WAVE_CASES = [
    # n, n_new, Hq, Hkv, d, r, paged, key side: 32 rows per workgroup, 32-key tiles dealt to eight waves
    (1, 1, 4, 4, 128, 16, False, "bk"),        # one key: seven waves without a tile
    (31, 31, 4, 1, 64, 8, True, "bk"),         # one tile, no old context
    (32, 8, 8, 2, 128, 24, False, "bk"),       # a full tile, exactly 32 rows
    (33, 9, 8, 2, 128, 32, True, "none"),      # two tiles, 36 rows: four in the second workgroup
    (255, 40, 14, 2, 128, 16, False, "none"),  # group of 7; the last tile one key short
    (256, 33, 9, 3, 64, 32, True, "bk"),       # group of 3; a tile for every wave
    (257, 65, 16, 1, 128, 8, True, "bk"),      # group of 16; one wave takes a second tile of one key
    (513, 150, 3, 3, 128, 16, True, "rotary"),
    (700, 64, 8, 2, 64, 16, False, "rotary"),
    (1500, 90, 28, 4, 128, 32, False, "bk"),
    (8192, 512, 16, 2, 64, 8, True, "none"),   # 32 tiles per wave, all that its block ids reach
    (600, 500, 16, 4, 128, 24, False, "bk"),   # two rounds of workgroups
]


@pytest.mark.parametrize("case", WAVE_CASES, ids=lambda c: "n%d_new%d_hq%d_hkv%d_d%d_r%d_paged%d_%s" % c)
def test_prefill_whose_waves_divide_the_keys(case):
    """Against the oracle, twice with the same bits; the workspace, without completed keys in it, is left alone (partial
    states would mean another kernel ran), and the kernels of variant 2 pass the same bar."""
    n, n_new, hq, hkv, d, r, paged, side = case
    theta = 500000.0 if side == "rotary" else 0.0
    w = W.make_contiguous("waves", "prefill", seed=4700 + n + n_new, n_agents=1, n_q_heads=hq, n_kv_heads=hkv,
                          head_dim=d, rank=r, n=n, n_new=n_new, d_model=None, b_std=0.05)
    k, v, l, table = w.k_base.to(DEV), w.v_base.to(DEV), w.l.to(DEV), None
    if paged:
        blocks = (n + 15) // 16
        order = torch.randperm(blocks + 3, generator=torch.Generator().manual_seed(n))[:blocks]
        def pool(t, lead):  # [n][...] -> [blocks][lead][16][...], NaN in the free slots
            out = torch.full((blocks + 3, 16, *t.shape[1:]), float("nan"), dtype=t.dtype)
            pad = torch.full((blocks * 16, *t.shape[1:]), float("nan"), dtype=t.dtype)
            pad[:n] = t
            out[order] = pad.view(blocks, 16, *t.shape[1:])
            return (out.transpose(1, 2).contiguous() if lead else out).to(DEV)
        k, v, l = pool(w.k_base, True), pool(w.v_base, True), pool(w.l, False)
        table = order.to(torch.int32).view(1, -1).to(DEV)
    lens = torch.tensor([n], dtype=torch.int32, device=DEV)
    cache = lra.make_cache(k, v, l, lens, n, table)
    q = w.q.to(DEV)
    shape = lra.make_shape(q, hkv, r, 0.0, theta)
    b_k = None if side == "none" else w.b_k.to(DEV)
    b_v = w.b_v.to(DEV)
    outs = []
    for variant in (0, 0, 2):
        old = lra.lra_set_kernel_variant(variant)
        try:
            need = lra.lra_workspace_bytes(shape, cache, 1, 1, n_new)
            ws = torch.full((max(need, 256),), 0xA5 + len(outs), dtype=torch.uint8, device=DEV)
            out = torch.full_like(q, float("nan"))
            lra.lra_attn_prefill(shape, cache, b_k, b_v, w.n_adapters, q, 0, 0, out, ws)
            torch.cuda.synchronize()
            assert variant != 0 or side == "rotary" or bool((ws == 0xA5 + len(outs)).all())
            outs.append(out)
        finally:
            lra.lra_set_kernel_variant(old)
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))
    import oracle
    f = lambda t: t.to(torch.float64).numpy()
    bk0 = np.zeros_like(f(w.b_k[0])) if side == "none" else f(w.b_k[0])
    ref = oracle.prefill(f(w.q), f(w.k_base), f(w.v_base), f(w.l), bk0, f(w.b_v[0]), n=n, scale=w.scale, key_rope_theta=theta)
    for out in outs[1:]:
        _gate(out.to(torch.float64).cpu().numpy(), ref, label=str(case))


WAVE_SHARE_CASES = [
    # n, n_new, Hq, Hkv, d, r, paged, key side, longest: the keys of 32 rows divided among workgroups
    (2100, 9, 32, 32, 128, 16, False, "bk", 2100),     # 5 shares of one row tile, nine live rows
    (2880, 64, 32, 8, 128, 16, False, "bk", 2880),     # 4 shares of eight row tiles
    (6144, 61, 32, 8, 64, 32, True, "none", 6144),     # the longest share of full 128-row tiles
    (18432, 33, 32, 8, 128, 24, True, "bk", 18432),    # the longest share of all, four live rows in the fifth tile
    (11521, 7, 28, 4, 128, 8, True, "bk", 11521),      # group of 7, and no room for its 32 shares: the tile walk
    (11777, 15, 16, 2, 64, 16, True, "bk", 11777),     # ... of 8
    (14001, 9, 28, 4, 128, 8, True, "bk", 14001),      # 32 shares of two row tiles, group of 7
    (16000, 8, 32, 4, 128, 24, True, "none", 16000),   # ... of 8
    (20000, 8, 16, 1, 64, 32, True, "bk", 20000),      # 32 shares of four row tiles
    (4096, 64, 32, 32, 128, 32, False, "none", 4096),  # group of 1
    (2200, 33, 32, 8, 128, 8, False, "rotary", 2200),
    (4401, 40, 16, 4, 64, 16, True, "rotary", 4401),
    (100, 64, 32, 8, 128, 16, True, "bk", 2880),       # shorter than the longest it was planned for: 2 to 4 tiles,
    (40, 40, 16, 4, 128, 32, False, "bk", 4400),       # so shares without a key, and (here) rows without one in theirs
]


@pytest.mark.parametrize("case", WAVE_SHARE_CASES, ids=lambda c: "n%d_new%d_hq%d_hkv%d_d%d_r%d_paged%d_%s_of%d" % c)
def test_prefill_whose_waves_divide_the_keys_of_a_share(case):
    """Against the oracle, twice with the same bits, on a workspace of NaN bytes; variant 2 passes the same bar."""
    n, n_new, hq, hkv, d, r, paged, side, longest = case
    theta = 500000.0 if side == "rotary" else 0.0
    w = W.make_contiguous("wave_shares", "prefill", seed=4800 + n + n_new, n_agents=1, n_q_heads=hq, n_kv_heads=hkv,
                          head_dim=d, rank=r, n=n, n_new=n_new, d_model=None, b_std=0.05)
    blocks = (longest + 15) // 16
    order = torch.randperm(blocks, generator=torch.Generator().manual_seed(n))
    def store(t, lead):  # rows past the sequence's end hold NaN
        pad = torch.full((blocks * 16, *t.shape[1:]), float("nan"), dtype=t.dtype)
        pad[:n] = t
        if not paged:
            return pad[:longest].to(DEV)
        out = torch.empty((blocks, 16, *t.shape[1:]), dtype=t.dtype)
        out[order] = pad.view(blocks, 16, *t.shape[1:])
        return (out.transpose(1, 2).contiguous() if lead else out).to(DEV)
    k, v, l = store(w.k_base, True), store(w.v_base, True), store(w.l, False)
    table = order.to(torch.int32).view(1, -1).to(DEV) if paged else None
    lens = torch.tensor([n], dtype=torch.int32, device=DEV)
    cache = lra.make_cache(k, v, l, lens, longest, table)
    q = w.q.to(DEV)
    shape = lra.make_shape(q, hkv, r, 0.0, theta)
    b_k = None if side == "none" else w.b_k.to(DEV)
    b_v = w.b_v.to(DEV)
    outs = []
    for variant in (0, 0, 2):
        old = lra.lra_set_kernel_variant(variant)
        try:
            need = lra.lra_workspace_bytes(shape, cache, 1, 1, n_new)
            ws = torch.full((need,), 0xff, dtype=torch.uint8, device=DEV)
            out = torch.full_like(q, float("nan"))
            lra.lra_attn_prefill(shape, cache, b_k, b_v, w.n_adapters, q, 0, 0, out, ws)
            torch.cuda.synchronize()
            outs.append(out)
        finally:
            lra.lra_set_kernel_variant(old)
    assert torch.equal(outs[0].view(torch.int16), outs[1].view(torch.int16))
    import oracle
    f = lambda t: t.to(torch.float64).numpy()
    bk0 = np.zeros_like(f(w.b_k[0])) if side == "none" else f(w.b_k[0])
    ref = oracle.prefill(f(w.q), f(w.k_base), f(w.v_base), f(w.l), bk0, f(w.b_v[0]), n=n, scale=w.scale, key_rope_theta=theta)
    for out in outs[1:]:
        _gate(out.to(torch.float64).cpu().numpy(), ref, label=str(case))


@pytest.mark.parametrize("n,n_new,hq,hkv,d,r", [(846, 31, 28, 4, 128, 24), (931, 20, 16, 2, 128, 24), (700, 24, 32, 8, 128, 16), (500, 32, 32, 8, 64, 32)])
def test_few_token_prefill_is_no_further_off_than_the_split_kv_path(n, n_new, hq, hkv, d, r):
    """The kernel whose waves divide the keys against variant 2, both against float64.  The errors are norms over 40000
    values and more, so a ratio of equal ones stays within 3 / sqrt(40000) of 1; a softmax reference that is only raised
    lazily shows as 1.05 to 1.11."""
    w = W.make_contiguous("few_tokens", "prefill", seed=4900 + n, n_agents=1, n_q_heads=hq, n_kv_heads=hkv, head_dim=d,
                          rank=r, n=n, n_new=n_new, d_model=None, b_std=0.05)
    ref = oracle_prefill(w)
    err = []
    for variant in (0, 2):
        old = lra.lra_set_kernel_variant(variant)
        try:
            err.append(errors(run_prefill(w, DEV), ref)[0])
        finally:
            lra.lra_set_kernel_variant(old)
    print("relL2 %.4e and %.4e" % tuple(err))
    assert err[0] <= 1.015 * err[1]


@pytest.mark.parametrize("kernels", [0, 2], ids=["auto", "tile_walk"])
@pytest.mark.parametrize("n,n_new", [(417, 84), (1023, 300)])
def test_short_sequence_prefill_with_and_without_a_workspace(n, n_new, kernels):
    """(Variant 2: the tile walk, with key shares and, where it has no room for them, without.)"""
    w = W.make_contiguous("short_sequence", "prefill", seed=4700 + n, n_agents=1, n_q_heads=8, n_kv_heads=2,
                          head_dim=128, rank=16, n=n, n_new=n_new, d_model=None, b_std=0.05)
    ref = oracle_prefill(w)
    old = lra.lra_set_kernel_variant(kernels)
    try:
        for with_workspace in (True, False):
            dw = DeviceWorkload(w, DEV)
            assert dw.alloc_workspace() > 0
            if not with_workspace:
                dw.workspace = None
            dw.out.fill_(float("nan"))
            dw.prefill()
            torch.cuda.synchronize()
            _gate(dw.out.to(torch.float64).cpu().numpy(), ref, label=f"workspace {with_workspace}")
    finally:
        lra.lra_set_kernel_variant(old)


@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("paged", [False, True], ids=["contiguous", "paged"])
@pytest.mark.parametrize("d,r", [(128, 16), (64, 24), (128, 64)])
def test_prefill_holds_the_low_rank_sums_in_fp32_until_the_output(d, r, paged, splits):
    """L rows of about 4 and B_V rows that cancel: what is left of P.L.B_V is a tenth of its terms, so a P.L rounded to
    bf16 (2^-9 of 4 per rank) would show as several percent.  The probabilities' own rounding does not: it scales all
    ranks alike up to a spread of 2^-9 / sqrt(keys) per rank, below 1e-2 of what is left."""
    n, n_new = 900, 140
    make = lambda **kw: W.make_contiguous("cancelling", "prefill", n=n, n_new=n_new, n_agents=1, **kw)
    w = make(seed=4800 + r, n_q_heads=8, n_kv_heads=2, head_dim=d, rank=r, d_model=None, b_std=0.05)
    w.l = (4.0 + w.l.float()).to(torch.bfloat16)
    w.v_base.mul_(1e-3)
    signs = torch.tensor([1.0, -1.0]).repeat(r // 2)[:, None]
    w.b_v = (signs * torch.ones_like(w.b_v[0].float()))[None].to(torch.bfloat16)
    ref = oracle_prefill(w)
    table = None
    k, v, l = w.k_base.to(DEV), w.v_base.to(DEV), w.l.to(DEV)
    if paged:  # the same rows in blocks of 16, the last one partly filled
        blocks = (n + 15) // 16
        pad = lambda t: torch.cat([t, torch.full((blocks * 16 - n, *t.shape[1:]), float("nan"), dtype=t.dtype, device=DEV)])
        k, v = (pad(t).view(blocks, 16, 2, d).permute(0, 2, 1, 3).contiguous() for t in (k, v))
        l = pad(l).view(blocks, 16, r)
        table = torch.arange(blocks, dtype=torch.int32, device=DEV)[None].contiguous()
    q = w.q.to(DEV)
    shape = lra.make_shape(q, 2, r, w.scale)
    lens = torch.tensor([n], dtype=torch.int32, device=DEV)
    cache = lra.make_cache(k, v, l, lens, n, table)
    out = torch.full_like(q, float("nan"))
    old = lra.lra_set_prefill_splits(splits)
    try:
        ws = torch.empty(max(256, lra.lra_workspace_bytes(shape, cache, 1, 1, n_new)), dtype=torch.uint8, device=DEV)
        lra.lra_attn_prefill(shape, cache, w.b_k.to(DEV), w.b_v.to(DEV), 1, q, 0, 0, out, ws)
        torch.cuda.synchronize()
    finally:
        lra.lra_set_prefill_splits(old)
    got = out.to(torch.float64).cpu().numpy()
    rel = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    print(f"relL2 {rel:.3e}", flush=True)
    assert rel <= 1e-2


@pytest.mark.parametrize("seq,n_new,path", [(0, 5, "split_kv"), (1, 16, "split_kv"), (2, 9, "split_kv"), (0, 1, "default"),
                                            (1, 4, "default"), (2, 3, "default"), (1, 16, "default")])
def test_short_prefill_on_paged_cache_value_only(seq, n_new, path):
    """Prefill of a few new tokens on a paged, ragged cache without B_K: the split-KV kernel, asked for or (up to 4
    tokens at a group of 4) by itself, and the tile walk that takes 16 tokens by itself."""
    w = W.make_paged("paged_short_prefill", seed=92, seq_lens=[40, 333, 1500], agents_per_seq=1, n_adapters=3,
                     n_q_heads=8, n_kv_heads=2, head_dim=128, rank=16, d_model=None, b_std=0.05)
    import oracle
    f = lambda t: t.to(torch.float64).numpy()
    gen = torch.Generator().manual_seed(600 + seq)
    q = torch.randn(n_new, 8, 128, generator=gen).to(torch.bfloat16)
    adapter = seq % 3
    dw = DeviceWorkload(w, DEV)
    qd = q.to(DEV)
    out = torch.full_like(qd, float("nan"))
    need = lambda: lra.lra_workspace_bytes(dw.shape, dw.cache, 1, 1, n_new)
    old = lra.lra_set_short_prefill(64)
    try:
        split_kv = need()
        lra.lra_set_short_prefill(0)
        assert need() != split_kv  # (the two paths are told apart by the workspace they ask for)
        lra.lra_set_short_prefill(64 if path == "split_kv" else old)
        assert (need() == split_kv) == (n_new < 16 or path == "split_kv") and need() > 0
        ws = torch.empty(need(), dtype=torch.uint8, device=DEV)
        lra.lra_attn_prefill(dw.shape, dw.cache, None, dw.b_v, w.n_adapters, qd, seq, adapter, out, ws)
        torch.cuda.synchronize()
    finally:
        lra.lra_set_short_prefill(old)
    n_t = w.seq_lens[seq]
    ids = w.block_table[seq].numpy()
    kb = oracle.gather_paged(f(w.k_base), ids, n_t)
    vb = oracle.gather_paged(f(w.v_base), ids, n_t)
    lr = oracle.lra_oracle.gather_paged_l(f(w.l), ids, n_t)
    ref = oracle.prefill(f(q), kb, vb, lr, np.zeros_like(f(w.b_k[adapter])), f(w.b_v[adapter]), n=n_t, scale=w.scale)
    _gate(out.to(torch.float64).cpu().numpy(), ref, label=f"paged short prefill seq {seq} n_new {n_new}")


@pytest.mark.parametrize("seq,n_new", [(0, 1), (1, 77), (2, 300), (3, 1027)])
def test_prefill_on_paged_cache(variant, seq, n_new):
    """Causal prefill of the last n_new tokens of one sequence of a paged, ragged cache
    (block table lookups, a last block that is partly filled, NaN in the free slots)."""
    w = W.make_paged("paged_prefill", seed=91, seq_lens=[1, 130, 300, 1027], agents_per_seq=1, n_adapters=3,
                     n_q_heads=8, n_kv_heads=2, head_dim=128, rank=16, d_model=None, b_std=0.05)
    gen = torch.Generator().manual_seed(500 + seq)
    q = torch.randn(n_new, 8, 128, generator=gen).to(torch.bfloat16)
    adapter = (seq + 1) % 3
    dw = DeviceWorkload(w, DEV)
    dw.alloc_workspace()
    qd = q.to(DEV)
    out = torch.full_like(qd, float("nan"))
    ws_bytes = lra.lra_workspace_bytes(dw.shape, dw.cache, 1, 1, n_new)
    ws = torch.empty(max(ws_bytes, 256), dtype=torch.uint8, device=DEV)
    lra.lra_attn_prefill(dw.shape, dw.cache, dw.b_k, dw.b_v, w.n_adapters, qd, seq, adapter, out, ws)
    torch.cuda.synchronize()
    import oracle
    f = lambda t: t.to(torch.float64).numpy()
    n_t = w.seq_lens[seq]
    ids = w.block_table[seq].numpy()
    kb = oracle.gather_paged(f(w.k_base), ids, n_t)
    vb = oracle.gather_paged(f(w.v_base), ids, n_t)
    lr = oracle.lra_oracle.gather_paged_l(f(w.l), ids, n_t)
    ref = oracle.prefill(f(q), kb, vb, lr, f(w.b_k[adapter]), f(w.b_v[adapter]), n=n_t, scale=w.scale)
    _gate(out.to(torch.float64).cpu().numpy(), ref, label=f"paged prefill seq {seq} n_new {n_new}")


FAR_POOL_CASES = [
    # n_new, splits, d, r, key side: with a B_K, without, rotary with the completed keys in the workspace
    (40, 1, 128, 16, "bk"), (333, 3, 128, 16, "bk"), (40, 3, 128, 16, "none"), (333, 1, 128, 64, "none"),
    (100, 1, 128, 32, "rotary"), (333, 2, 128, 16, "rotary"), (129, 1, 64, 64, "bk"), (65, 2, 64, 32, "none"),
    (200, 2, 64, 64, "rotary"), (333, 2, 128, 64, "bk"), (50, 1, 64, 16, "bk"),
]


@pytest.mark.parametrize("n_new,splits,d,r,key_side", FAR_POOL_CASES)
def test_prefill_on_a_pool_beyond_two_gigabytes(n_new, splits, d, r, key_side):
    """Pools within 32-bit byte offsets and larger ones take different kernels: the same blocks, once dense and once
    128 MiB apart (3.2 GB), give the same bits."""
    w = W.make_paged("far_blocks", seed=95, seq_lens=[1, 333], agents_per_seq=1, n_adapters=2, n_q_heads=8,
                     n_kv_heads=2, head_dim=d, rank=r, d_model=None, b_std=0.05)
    dw = DeviceWorkload(w, DEV, key_rope_theta=500000.0 if key_side == "rotary" else 0.0)
    b_k = None if key_side == "none" else dw.b_k
    nb, hkv, bs, _ = dw.k_base.shape
    far = [torch.empty(nb << 26, dtype=torch.bfloat16, device=DEV).as_strided((nb, hkv, bs, d), (1 << 26, bs * d, d, 1))
           for _ in range(2)]
    far[0].copy_(dw.k_base)
    far[1].copy_(dw.v_base)
    assert nb << 27 > 1 << 31
    far_cache = lra.make_cache(far[0], far[1], dw.l, dw.seq_lens, max(w.seq_lens), dw.block_table)
    q = torch.randn(n_new, 8, d, generator=torch.Generator().manual_seed(96)).to(torch.bfloat16).to(DEV)
    old_s, old_t = lra.lra_set_prefill_splits(splits), lra.lra_set_short_prefill(0)
    try:
        outs = []
        for cache in (dw.cache, far_cache):
            out = torch.full_like(q, float("nan"))
            need = lra.lra_workspace_bytes(dw.shape, cache, 1, 1, n_new)
            ws = torch.empty(max(256, need), dtype=torch.uint8, device=DEV)
            lra.lra_attn_prefill(dw.shape, cache, b_k, dw.b_v, w.n_adapters, q, 1, 1, out, ws)
            outs.append(out)
        torch.cuda.synchronize()
    finally:
        lra.lra_set_prefill_splits(old_s)
        lra.lra_set_short_prefill(old_t)
    assert torch.isfinite(outs[0]).all() and torch.equal(outs[0], outs[1])


def test_paged_small_ragged_distinct_adapters(variant):
    """Lengths that end inside a block, one adapter per query, NaN-poisoned free
    slots: nothing outside a sequence's own tokens may reach its output."""
    w = W.make_paged("paged_small", seed=77, seq_lens=[1, 15, 16, 17, 250, 1027], agents_per_seq=3,
                     n_adapters=0, n_q_heads=14, n_kv_heads=2, head_dim=128, rank=32, d_model=None,
                     distinct_adapter_per_query=True, b_std=0.05)
    _gate(run_decode(w, DEV), oracle_decode(w), label=w.name)


@pytest.mark.parametrize("mirror", ["none", "exact", "all_zero", "too_long"])
def test_host_copy_of_the_lengths_only_steers_planning(mirror):
    """lra_cache.seq_lens_host: the decode of a batch sizes its key shares from it; the results do not depend on
    it, whatever it holds, and a workspace sized without it serves the call with it."""
    import paper_2602_01053_amd as lra
    from paper_2602_01053_amd.runner import DeviceWorkload
    lens = [6000, 5500, 7000, 6500, 5300, 6900, 5251, 7001]
    w = W.make_paged("mirror", seed=79, seq_lens=lens, agents_per_seq=2, n_adapters=3, n_q_heads=16, n_kv_heads=4,
                     head_dim=128, rank=16, d_model=None, b_std=0.05)
    host = {"none": None, "exact": lens, "all_zero": [0] * len(lens), "too_long": [10 ** 6] * len(lens)}[mirror]
    dw = DeviceWorkload(w, DEV, host_lens=False)
    need_without = dw.alloc_workspace()
    dw.cache = lra.make_cache(dw.k_base, dw.v_base, dw.l, dw.seq_lens, max(lens), dw.block_table, seq_lens_host=host)
    need_with = lra.lra_workspace_bytes(dw.shape, dw.cache, w.n_queries, dw.max_queries_per_seq, 0)
    assert need_with <= need_without
    if mirror in ("exact", "too_long"):
        assert need_with < need_without  # 8 sequences x 4 kv heads of 5251 to 7001 keys: fewer, longer key shares
    dw.out.fill_(float("nan"))
    dw.decode()                        # on the workspace sized without the lengths
    torch.cuda.synchronize()
    _gate(dw.out.to(torch.float64).cpu().numpy(), oracle_decode(w), label=f"{w.name} {mirror}")


def test_one_long_sequence_in_a_paged_cache():
    """One sequence of 33000 tokens in a paged cache with 8 kv heads: long enough that the planner gives the split-KV
    kernel two workgroups per compute unit (512 key shares x kv heads), with a ragged last share and last block."""
    w = W.make_paged("long_paged", seed=80, seq_lens=[33001], agents_per_seq=3, n_adapters=3, n_q_heads=32, n_kv_heads=8,
                     head_dim=128, rank=16, d_model=None, b_std=0.05)
    _gate(run_decode(w, DEV), oracle_decode(w), label=w.name)


BATCH_CASES = [
    # lengths, agents, Hq, Hkv, d, r, side: about half of them small enough for the grid of equal shares, the others with the
    # key shares of all sequences in one row, dealt to 512 workgroups
    ([3000, 129, 128, 1, 2500], 2, 8, 2, 128, 16, "bk"),        # a tile and a key, a tile, one key; up to 24 shares
    ([6000, 700], 5, 28, 4, 128, 32, "bk"),                     # group of 7: 40 rows, two row groups of two row tiles
    ([5000, 40, 1900], 3, 8, 8, 64, 24, "none"),
    ([4100, 2100, 900, 3300], 4, 16, 4, 128, 16, "own"),        # a low-rank cache per adapter
    ([9000, 2222, 333], 3, 28, 4, 128, 32, "own"),              # ... in two row groups
    ([9000, 500, 4000], 4, 8, 2, 128, 24, "rotary"),
    ([7000, 900], 2, 8, 4, 64, 64, "rotary"),                   # one workgroup per compute unit
    ([40 * (i + 3) for i in range(64)], 1, 4, 1, 64, 8, "bk"),  # a sequence in every lane
]
_A, _B, _C = [4000, 1501, 3000, 700], [5200, 900, 2600], [2817, 3000, 129, 1, 2500]
BATCH_ROW_CASES = [
    # ... in one row with the lengths known and without, one case and more for every instantiation of that kernel
    (_C, 2, 32, 8, 128, 16, "bk"), (_A, 3, 32, 8, 128, 24, "none"), (_A, 1, 32, 8, 128, 40, "bk"), (_A, 4, 32, 8, 128, 64, "none"),
    (_A, 7, 32, 8, 128, 8, "bk"), (_A, 5, 32, 8, 128, 32, "none"), (_B, 6, 32, 8, 128, 64, "bk"), (_B, 8, 32, 8, 128, 40, "none"),
    (_C, 2, 32, 8, 64, 16, "none"), (_A, 3, 32, 8, 64, 32, "bk"), (_A, 1, 32, 8, 64, 64, "none"), (_A, 4, 32, 8, 64, 40, "bk"),
    (_A, 7, 32, 8, 64, 24, "none"), (_A, 5, 32, 8, 64, 8, "bk"), (_B, 6, 32, 8, 64, 40, "none"), (_B, 8, 32, 8, 64, 64, "bk"),
    # a low-rank cache per adapter, two row groups at a group of 7
    (_B, 3, 28, 4, 128, 16, "own"), (_A, 2, 32, 8, 128, 16, "own"), (_B, 3, 28, 4, 64, 16, "own"), (_A, 3, 32, 8, 64, 8, "own"),
    (_B, 3, 28, 4, 128, 16, "own_none"), (_A, 2, 32, 8, 128, 16, "own_none"), (_B, 3, 28, 4, 64, 16, "own_none"), (_A, 3, 32, 8, 64, 8, "own_none"),
    # rotary: three and five row groups, one workgroup per compute unit at rank 40
    ([9000, 2000, 5000, 7000, 6100, 8000], 5, 28, 4, 64, 16, "rotary"), ([20000, 9000, 16000], 2, 32, 8, 64, 24, "rotary"),
    ([9000, 3000, 6100, 2000], 3, 16, 8, 64, 40, "rotary"), ([9000, 2000, 5000], 9, 28, 4, 128, 24, "rotary"),
    ([20000, 3000, 9000, 1000], 3, 32, 8, 128, 16, "rotary"),
    # batches of some tens of sequences, two row groups in the second
    ([300 + 141 * (7 * i % 20) for i in range(20)], 2, 16, 4, 128, 16, "bk"), ([1200 + 90 * (11 * i % 48) for i in range(48)], 6, 14, 2, 64, 32, "none"),
]


@pytest.mark.parametrize("case,mirror", [(c, m) for c in BATCH_CASES for m in ("exact", "none", "half", "double")] +
                         [(c, m) for c in BATCH_ROW_CASES for m in ("exact", "none")],
                         ids=lambda v: v if isinstance(v, str) else "s%d_a%d_hq%d_hkv%d_d%d_r%d_%s" % (len(v[0]), *v[1:]))
def test_batch_whose_shares_stand_in_one_row(case, mirror):
    """Ragged batches against the oracle, with the right lengths on the host, with none, and with wrong ones (shares that
    do not fit their places are enlarged on the device); NaN in the workspace, so that a state nobody wrote would show."""
    lens, agents, hq, hkv, d, r, side = case
    theta = 500000.0 if side == "rotary" else 0.0
    w = W.make_paged("batch_row", seed=4800 + sum(lens), seq_lens=lens, agents_per_seq=agents, n_adapters=max(agents, 2),
                     n_q_heads=hq, n_kv_heads=hkv, head_dim=d, rank=r, d_model=None, b_std=0.05)
    dev = lambda t: t.to(DEV)
    f = lambda t: t.to(torch.float64).numpy()
    l = w.l
    own = side in ("own", "own_none")
    if own:  # adapter a attends over a low-rank cache of its own
        l = torch.stack([w.l.roll(a, dims=-1) * (1 + a) for a in range(w.n_adapters)])
    q = dev(w.q)
    b_k = None if side in ("none", "own_none") else dev(w.b_k)
    host = {"exact": lens, "none": None, "half": [n // 2 for n in lens], "double": [2 * n for n in lens]}[mirror]
    cache_t = [dev(w.k_base), dev(w.v_base), dev(l), torch.tensor(lens, dtype=torch.int32, device=DEV), dev(w.block_table)]
    cache = lra.make_cache(cache_t[0], cache_t[1], cache_t[2], cache_t[3], max(lens), cache_t[4], l_per_adapter=own,
                           seq_lens_host=host)
    shape = lra.make_shape(q, hkv, r, 0.0, theta)
    b_v, ids, start = dev(w.b_v), dev(w.query_adapter), dev(w.seq_query_start)
    need = lra.lra_workspace_bytes(shape, cache, q.shape[0], agents)
    out = torch.full_like(q, float("nan"))
    ws = torch.full((need,), 0xFF, dtype=torch.uint8, device=DEV)
    lra.lra_attn_decode(shape, cache, b_k, b_v, w.n_adapters, q, ids, start, agents, out, ws)
    torch.cuda.synchronize()
    import oracle
    got, ref = out.to(torch.float64).cpu().numpy(), np.empty(tuple(q.shape))
    qf, kf, vf, lf, bk, bv = f(w.q), f(w.k_base), f(w.v_base), f(l), f(w.b_k) * (b_k is not None), f(w.b_v)
    for i in range(q.shape[0]):  # one query at a time: its sequence's rows, its adapter's low-rank cache
        t, a = i // agents, int(w.query_adapter[i])
        table = w.block_table[t].numpy()
        kb, vb = oracle.gather_paged(kf, table, lens[t]), oracle.gather_paged(vf, table, lens[t])
        lr = oracle.lra_oracle.gather_paged_l(lf[a] if own else lf, table, lens[t])
        ref[i] = oracle.prefill(qf[i:i + 1], kb, vb, lr, bk[a], bv[a], n=lens[t], scale=w.scale, key_rope_theta=theta)[0]
    _gate(got, ref, label=f"{case} {mirror}")


@pytest.mark.parametrize("lens,agents,hq,hkv,r", [([700 + 170 * (4 * i % 9) for i in range(9)], 4, 32, 8, 24), ([3000 + 800 * i for i in range(5)], 6, 28, 4, 16)])
def test_batch_in_one_row_is_no_further_off_than_the_grid(lens, agents, hq, hkv, r):
    """The row's longer key shares against variant 2, both against float64.  The errors are norms over 100000 values and
    more, so a ratio of equal ones stays within 3 / sqrt(100000) of 1; the running maximum as softmax reference shows as
    1.018 in the first call and as 1.008 in the second."""
    w = W.make_paged("row_error", seed=4990 + len(lens), seq_lens=lens, agents_per_seq=agents, n_adapters=3, n_q_heads=hq,
                     n_kv_heads=hkv, head_dim=128, rank=r, d_model=None, b_std=0.05)
    ref = oracle_decode(w)
    err = []
    for variant in (0, 2):
        old = lra.lra_set_kernel_variant(variant)
        try:
            err.append(errors(run_decode(w, DEV), ref)[0])
        finally:
            lra.lra_set_kernel_variant(old)
    print("relL2 %.4e and %.4e" % tuple(err))
    assert err[0] <= 1.01 * err[1]


def test_uneven_queries_per_sequence(variant):
    """Sequences with 0, 1 and many queries in one call."""
    w = W.make_paged("uneven", seed=78, seq_lens=[300, 77, 129, 512], agents_per_seq=2, n_adapters=3,
                     n_q_heads=8, n_kv_heads=2, head_dim=64, rank=16, d_model=None, b_std=0.05)
    w.seq_query_start = torch.tensor([0, 5, 5, 6, 8], dtype=torch.int32)   # 5, 0, 1, 2 queries
    _gate(run_decode(w, DEV), oracle_decode(w), label=w.name)


def test_null_adapters_reduce_to_plain_attention(variant):
    """b_k = b_v = NULL is the fully shared cache: equals the oracle with B = 0."""
    w = W.config(2, shrink=8)
    dw = DeviceWorkload(w, DEV)
    dw.alloc_workspace()
    dw.b_k = None
    dw.b_v = None
    dw.decode()
    torch.cuda.synchronize()
    w.b_k.zero_()
    w.b_v.zero_()
    _gate(dw.out.to(torch.float64).cpu().numpy(), oracle_decode(w), label="null adapters")


@pytest.mark.parametrize("kind", ["decode_contiguous", "decode_paged", "prefill_contiguous", "prefill_r64"])
def test_value_only_adapters(variant, kind):
    """b_k = NULL with b_v present: the paper's main setting (keys fully shared, LoRA on the
    value side only, Sec. 3.2).  Equals the oracle with B_K = 0."""
    if kind == "decode_contiguous":
        w = W.config(2, shrink=8)
    elif kind == "decode_paged":
        w = W.make_paged("value_only_paged", seed=79, seq_lens=[5, 64, 333, 1500], agents_per_seq=3, n_adapters=4,
                         n_q_heads=14, n_kv_heads=2, head_dim=128, rank=32, d_model=None, b_std=0.05)
    elif kind == "prefill_contiguous":
        w = W.make_contiguous("value_only_prefill", "prefill", seed=80, n_agents=1, n_q_heads=8, n_kv_heads=2,
                              head_dim=128, rank=16, n=700, n_new=300, d_model=None, b_std=0.05)
    else:
        w = W.make_contiguous("value_only_prefill_r64", "prefill", seed=81, n_agents=1, n_q_heads=4, n_kv_heads=4,
                              head_dim=64, rank=64, n=391, n_new=391, d_model=None, b_std=0.05)
    dw = DeviceWorkload(w, DEV)
    dw.alloc_workspace()
    dw.b_k = None
    dw.out.fill_(float("nan"))
    if w.kind == "decode":
        dw.decode()
    else:
        dw.prefill()
    torch.cuda.synchronize()
    w.b_k.zero_()
    ref = oracle_decode(w) if w.kind == "decode" else oracle_prefill(w)
    _gate(dw.out.to(torch.float64).cpu().numpy(), ref, label=kind)


def test_deterministic_and_inputs_untouched(variant):
    w = W.config(2, shrink=4)
    dw = DeviceWorkload(w, DEV)
    dw.alloc_workspace()
    dw.decode()
    torch.cuda.synchronize()
    first = dw.out.clone()
    dw.workspace.fill_(0xFF)
    dw.out.zero_()
    dw.decode()
    torch.cuda.synchronize()
    assert torch.equal(first.view(torch.int16), dw.out.view(torch.int16))
    assert torch.equal(dw.k_base.cpu(), w.k_base) and torch.equal(dw.l.cpu(), w.l)
    assert torch.equal(dw.q.cpu(), w.q) and torch.equal(dw.b_v.cpu(), w.b_v)


def test_split_size_does_not_change_result_beyond_rounding():
    w = W.config(2, shrink=4)
    ref = oracle_decode(w)
    try:
        for keys in (64, 192, 1024, 1 << 20):
            lra.lra_set_decode_split_keys(keys)
            _gate(run_decode(w, DEV), ref, label=f"split_keys={keys}")
    finally:
        lra.lra_set_decode_split_keys(0)


def test_runs_on_a_side_stream():
    w = W.config(2, shrink=8)
    dw = DeviceWorkload(w, DEV)
    dw.alloc_workspace()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        dw.decode(s)
    s.synchronize()
    _gate(dw.out.to(torch.float64).cpu().numpy(), oracle_decode(w), label="side stream")


def test_machine_probes_run():
    """The benchmark's two probe kernels complete, leave their sink alone and report their work."""
    sink = torch.zeros(4, dtype=torch.int32, device=DEV)
    buf = torch.arange(1 << 20, dtype=torch.int32, device=DEV)
    lra.lra_probe_stream_read(buf, sink)
    lra.lra_probe_stream_read(buf[:1000], sink)       # a length that leaves a remainder pass
    flops = lra.lra_probe_mfma_bf16(100, sink)
    assert lra.lra_probe_mfma_bf16(100, sink, random_operands=True) == flops
    torch.cuda.synchronize()
    assert flops == 512 * 4 * 4 * 100 * 2 * 32 * 32 * 16
    assert int(sink.abs().sum()) == 0


@pytest.mark.parametrize("case", [
    # sequences, agents per sequence, Hq, Hkv, d, r  -> rows = sequences x agents x Hq
    (40, 8, 4, 1, 128, 16),     # 1280 rows, group of 4
    (30, 5, 14, 2, 64, 24),     # 2100 rows, group of 7 (two workgroups of four waves per kv head, one wave idle)
    (20, 4, 16, 1, 128, 64),    # 1280 rows, group of 16
    (70, 3, 5, 5, 64, 8),       # 1050 rows, group of 1 (three of four waves idle)
], ids=lambda c: "s%d_a%d_hq%d_hkv%d_d%d_r%d" % c)
def test_many_rows_take_the_wave_per_row_merge(case):
    """Ragged paged batches of 1024 rows and more with many short sequences (so that most key shares of most rows are
    empty), every group size class: at ranks up to 16 the merge is a wave per row, at the two above a workgroup per row
    (tests/test_merge_forms_gpu.py has the wave per row of those ranks, from 2560 rows on)."""
    n_seqs, agents, hq, hkv, d, r = case
    rng = np.random.default_rng(sum(case))
    lens = [int(x) for x in rng.integers(1, 700, size=n_seqs)]
    w = W.make_paged("many_rows", seed=4000 + sum(case), seq_lens=lens, agents_per_seq=agents, n_adapters=3,
                     n_q_heads=hq, n_kv_heads=hkv, head_dim=d, rank=r, d_model=None, b_std=0.05)
    assert w.q.shape[0] * hq >= 1024
    prev = lra.lra_set_decode_split_keys(128)   # up to six shares per sequence
    try:
        got = run_decode(w, DEV)
    finally:
        lra.lra_set_decode_split_keys(prev)
    _gate(got, oracle_decode(w), label=w.name)


def test_many_rows_fp32_and_vector_alu_partials():
    """The wave-per-row merge behind the vector-ALU partial kernels: fp32 (held to 2e-5), and bf16 with the
    vector-ALU kernels forced."""
    lens = [int(x) for x in np.random.default_rng(77).integers(1, 400, size=36)]
    for dtype, variant, fp32 in ((torch.float32, 0, True), (torch.bfloat16, 1, False)):
        w = W.make_paged("many_rows_valu", seed=4200, dtype=dtype, seq_lens=lens, agents_per_seq=4, n_adapters=3,
                         n_q_heads=8, n_kv_heads=2, head_dim=64, rank=12, d_model=None, b_std=0.05)
        assert w.q.shape[0] * 8 >= 1024
        prev = lra.lra_set_kernel_variant(variant)
        try:
            got = run_decode(w, DEV)
        finally:
            lra.lra_set_kernel_variant(prev)
        _gate(got, oracle_decode(w), fp32=fp32, label=f"{w.name} {dtype}")


def test_vector_alu_kernel_beyond_2_to_24_rows():
    """4100 queries of 4096 heads, all the same: 16.8 million rows of 256 threads each, more threads than one grid
    dimension holds.  Every query's output equals the first one's, bit for bit, and that one the oracle's."""
    nq, hq, hkv, d, r, n = 4100, 4096, 256, 64, 8, 40
    w = W.make_contiguous("many_rows", "decode", seed=97, dtype=torch.float32, n_agents=1, n_q_heads=hq, n_kv_heads=hkv,
                          head_dim=d, rank=r, n=n, n_new=1, d_model=None, b_std=0.05)
    dw = DeviceWorkload(w, DEV)
    q = dw.q.expand(nq, hq, d).contiguous()
    out = torch.full_like(q, float("nan"))
    ids = torch.zeros(nq, dtype=torch.int32, device=DEV)
    start = torch.tensor([0, nq], dtype=torch.int32, device=DEV)
    ws = torch.empty(lra.lra_workspace_bytes(dw.shape, dw.cache, nq, nq), dtype=torch.uint8, device=DEV)
    lra.lra_attn_decode(dw.shape, dw.cache, dw.b_k, dw.b_v, 1, q, ids, start, nq, out, ws)
    torch.cuda.synchronize()
    _gate(out[:1].to(torch.float64).cpu().numpy(), oracle_decode(w), fp32=True, label="first query")
    assert all(torch.equal(out[i:i + 100], out[:1].expand(100, hq, d)) for i in range(0, nq, 100))


def test_prefill_with_shared_key_tiles_and_many_rows():
    """64 new tokens x 16 q heads = 1024 rows, key tiles shared by 4 workgroups: the wave-per-row merge after the
    tile-walking prefill kernel."""
    w = W.make_contiguous("pf_many_rows", "prefill", seed=4100, n_agents=1, n_q_heads=16, n_kv_heads=4, head_dim=128,
                          rank=16, n=1500, n_new=64, d_model=None, b_std=0.05)
    prev_s, prev_p = lra.lra_set_short_prefill(0), lra.lra_set_prefill_splits(4)
    try:
        got = run_prefill(w, DEV)
    finally:
        lra.lra_set_short_prefill(prev_s)
        lra.lra_set_prefill_splits(prev_p)
    _gate(got, oracle_prefill(w), label=w.name)


def test_adapter_ids_outside_the_table_are_clamped(variant):
    """query_adapter is device data the host cannot check: every kernel keeps an id inside [0, n_adapters) by
    clamping, so a bad id gives the result of the nearest valid adapter and no read outside B_K / B_V."""
    w = W.make_contiguous("bad_ids", "decode", seed=88, n_agents=5, n_q_heads=8, n_kv_heads=2, head_dim=128, rank=16,
                          n=700, d_model=None, b_std=0.05)
    good = w.query_adapter.clone()
    bad = good.clone()
    bad[1], bad[3] = 99, -7                       # clamp to the last and to the first adapter
    good[1], good[3] = w.n_adapters - 1, 0
    w.query_adapter = bad
    got = run_decode(w, DEV)
    w.query_adapter = good
    _gate(got, oracle_decode(w), label="clamped adapter ids")
