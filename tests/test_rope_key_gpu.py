"""The rotary key side (lra_shape.key_rope_theta > 0: K_j = K_base,j + RoPE_j(L_j B_K), the
setting of the paper's qkvo ablation, App. D.1) against the oracle, through the C ABI:
decode and prefill, contiguous and paged, bf16 and fp32.  Same gate as everywhere
(relative L2 <= 5e-3, max-abs <= 2e-2); fp32 is also held to 1e-4."""
import numpy as np
import pytest
import torch

import oracle
import paper_2602_01053_amd as lra
from paper_2602_01053_amd import workloads as W
from paper_2602_01053_amd.runner import DeviceWorkload
from tests.harness import MAX_ABS_TOL, REL_L2_TOL, _f64, errors, oracle_prefill_by_blocks

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _run(w, theta):
    dw = DeviceWorkload(w, DEV, key_rope_theta=theta)
    dw.alloc_workspace()
    dw.out.fill_(float("nan"))
    if w.kind == "decode":
        dw.decode()
    else:
        dw.prefill()
    torch.cuda.synchronize()
    return dw.out.to(torch.float64).cpu().numpy()


def _oracle(w, theta):
    if w.kind == "decode":
        return oracle.decode(_f64(w.q), _f64(w.k_base), _f64(w.v_base), _f64(w.l), _f64(w.b_k), _f64(w.b_v),
                             w.query_adapter.numpy(), w.seq_query_start.numpy(), w.seq_lens, w.scale,
                             block_size=w.block_size,
                             block_table=None if w.block_table is None else w.block_table.numpy(),
                             key_rope_theta=theta)
    a = int(w.query_adapter[0])
    return oracle.prefill(_f64(w.q), _f64(w.k_base), _f64(w.v_base), _f64(w.l), _f64(w.b_k[a]), _f64(w.b_v[a]),
                          n=w.seq_lens[0], scale=w.scale, key_rope_theta=theta)


def _cases():
    yield "decode_llama_shape", W.make_contiguous("rope_dec", "decode", seed=301, n_agents=4, n_q_heads=32, n_kv_heads=8,
                                                  head_dim=128, rank=16, n=1500, n_new=1, d_model=None, b_std=0.1), 500000.0, None
    yield "decode_d64_r24", W.make_contiguous("rope_dec64", "decode", seed=302, n_agents=3, n_q_heads=8, n_kv_heads=2,
                                              head_dim=64, rank=24, n=333, n_new=1, d_model=None, b_std=0.1), 10000.0, None
    yield "decode_paged", W.make_paged("rope_paged", seed=303, seq_lens=[5, 64, 700], agents_per_seq=2, n_adapters=3,
                                       n_q_heads=8, n_kv_heads=2, head_dim=128, rank=8, d_model=None, b_std=0.1), 500000.0, None
    yield "decode_paged_batch", W.make_paged("rope_paged2", seed=307, seq_lens=[1, 63, 64, 65, 1000, 2500], agents_per_seq=4,
                                             n_adapters=4, n_q_heads=28, n_kv_heads=4, head_dim=128, rank=32, d_model=None,
                                             b_std=0.1), 500000.0, None
    yield "decode_r64_8_agents", W.make_contiguous("rope_dec_r64", "decode", seed=308, n_agents=8, n_q_heads=32, n_kv_heads=8,
                                                   head_dim=128, rank=64, n=2100, n_new=1, d_model=None, b_std=0.05), 500000.0, None
    yield "decode_r48_d64", W.make_contiguous("rope_dec_r48", "decode", seed=309, n_agents=2, n_q_heads=16, n_kv_heads=2,
                                              head_dim=64, rank=48, n=777, n_new=1, d_model=None, b_std=0.05), 10000.0, None
    yield "decode_9_agents_r16", W.make_contiguous("rope_dec_9", "decode", seed=310, n_agents=9, n_q_heads=16, n_kv_heads=4,
                                                   head_dim=128, rank=16, n=4100, n_new=1, d_model=None, b_std=0.1), 500000.0, None
    yield "decode_d64_r8_group1", W.make_contiguous("rope_dec_g1", "decode", seed=311, n_agents=5, n_q_heads=4, n_kv_heads=4,
                                                    head_dim=64, rank=8, n=129, n_new=1, d_model=None, b_std=0.1), 10000.0, None
    yield "decode_long_positions", W.make_contiguous("rope_dec_long", "decode", seed=312, n_agents=4, n_q_heads=8, n_kv_heads=2,
                                                     head_dim=128, rank=16, n=70001, n_new=1, d_model=None, b_std=0.1), 500000.0, None
    yield "prefill", W.make_contiguous("rope_pre", "prefill", seed=304, n_agents=1, n_q_heads=8, n_kv_heads=2,
                                       head_dim=128, rank=16, n=400, n_new=150, d_model=None, b_std=0.1), 500000.0, None
    yield "decode_fp32", W.make_contiguous("rope_f32", "decode", seed=305, dtype=torch.float32, n_agents=2, n_q_heads=4,
                                           n_kv_heads=2, head_dim=64, rank=5, n=200, n_new=1, d_model=None, b_std=0.1), 10000.0, 1e-4


@pytest.mark.parametrize("variant", [0, 1], ids=["mfma", "vector_alu"])
@pytest.mark.parametrize("name,w,theta,tight", list(_cases()), ids=[c[0] for c in _cases()])
def test_rotary_key_side(name, w, theta, tight, variant):
    """bf16 decode runs on the rotary form of the split-KV MFMA kernel (variant 0: 4, 2 or 1 agent slots per
    workgroup for ranks up to 16, 32, 64), or on the vector-ALU kernels (variant 1, and fp32 always)."""
    prev = lra.lra_set_kernel_variant(variant)
    try:
        got = _run(w, theta)
    finally:
        lra.lra_set_kernel_variant(prev)
    ref = _oracle(w, theta)
    rel, mx = errors(got, ref)
    plain = _oracle(w, 0.0)
    moved = np.linalg.norm(ref - plain) / np.linalg.norm(ref)
    print(f"{name}: relL2={rel:.3e} maxabs={mx:.3e}; the rotation moves the output by {moved:.3e}", flush=True)
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL
    if tight:
        assert rel <= tight
    assert moved > 4 * REL_L2_TOL      # the gate would see a missing rotation


@pytest.mark.parametrize("cfg", [2, 4, 5])
def test_rotary_decode_at_the_named_configurations(cfg):
    """The decode configurations at full size (4 slots per tile at rank 16, one at rank 64, two at rank 32 on a
    ragged paged batch), in the launch configuration the benchmark's rotary leg times."""
    w = W.config(cfg)
    got = _run(w, 500000.0)
    ref = _oracle(w, 500000.0)
    rel, mx = errors(got, ref)
    print(f"{w.name}: relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL


def test_rotary_prefill_at_configuration_3_every_row():
    """The full-size causal prefill with the rotary key side, in the launch configuration the benchmark's rotary
    leg times (keys completed by the pre-pass) and with the key tiles completed inside the kernel, compared
    with the oracle on every output row."""
    w = W.config(3)
    ref = oracle_prefill_by_blocks(w, key_rope_theta=500000.0)
    for prepass in (True, False):
        prev = lra.lra_set_rope_key_prepass(prepass)
        try:
            got = _run(w, 500000.0)
        finally:
            lra.lra_set_rope_key_prepass(prev)
        rel, mx = errors(got, ref)
        print(f"{w.name} rotary, {'key pre-pass' if prepass else 'tiles completed in the kernel'}: relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
        assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL


def test_rotary_prefill_with_large_key_adapters_at_configuration_3_shape():
    """Configuration 3's shape with five times larger adapters (B ~ N(0, 0.1^2): the rotated adapter part is a
    large share of every key, so the second rounding of the completed keys to bf16 weighs most), both ways of
    completing the keys, on a spread of rows that includes the first and last rows of q tiles."""
    w = W.make_contiguous("cfg3_b01", "prefill", seed=322, n_agents=1, n_q_heads=32, n_kv_heads=8, head_dim=128, rank=16,
                          n=18432, n_new=2048, d_model=None, b_std=0.1)
    rows = np.unique(np.concatenate([np.arange(0, 2048, 24), np.arange(127, 2048, 128), np.arange(128, 2048, 128), [2047]]))
    a = int(w.query_adapter[0])
    ref = oracle.prefill(_f64(w.q), _f64(w.k_base), _f64(w.v_base), _f64(w.l), _f64(w.b_k[a]), _f64(w.b_v[a]),
                         n=w.seq_lens[0], scale=w.scale, rows=rows, key_rope_theta=500000.0)
    for prepass in (True, False):
        prev = lra.lra_set_rope_key_prepass(prepass)
        try:
            got = _run(w, 500000.0)[rows]
        finally:
            lra.lra_set_rope_key_prepass(prev)
        rel, mx = errors(got, ref)
        print(f"b_std 0.1, {'key pre-pass' if prepass else 'tiles completed in the kernel'}: relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
        assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL


def test_rotary_prefill_key_prepass_layouts_and_small_workspace():
    """The pre-pass writes the completed keys in the layout of K_base: token-major and head-major caches give
    the same output; a call whose workspace has no room for them (here: none at all) completes the tiles in the
    kernel and still matches the oracle."""
    w = W.make_contiguous("rp_hm", "prefill", seed=321, n_agents=1, n_q_heads=8, n_kv_heads=4, head_dim=128, rank=16,
                          n=1300, n_new=513, d_model=None, b_std=0.1)
    ref = _oracle(w, 500000.0)
    outs = []
    for head_major in (False, True):
        dw = DeviceWorkload(w, DEV, head_major, key_rope_theta=500000.0)
        need = dw.alloc_workspace()
        assert need >= w.k_base.numel() * 2          # room for a copy of the keys
        dw.out.fill_(float("nan"))
        dw.prefill()
        torch.cuda.synchronize()
        outs.append(dw.out.to(torch.float64).cpu().numpy())
        rel, mx = errors(outs[-1], ref)
        print(f"head_major={head_major}: relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
        assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL
    assert np.array_equal(outs[0], outs[1])
    dw = DeviceWorkload(w, DEV, key_rope_theta=500000.0)
    prev = lra.lra_set_rope_key_prepass(False)
    try:
        small = dw.alloc_workspace()                  # what the call needs without the completed keys
    finally:
        lra.lra_set_rope_key_prepass(prev)
    assert small < need - w.k_base.numel() * 2 + 4096
    dw.out.fill_(float("nan"))
    dw.prefill()                                      # pre-pass allowed, but no room for its keys
    torch.cuda.synchronize()
    rel, mx = errors(dw.out.to(torch.float64).cpu().numpy(), ref)
    print(f"workspace without room for the keys: relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL


def _random_decode_cases(count=28, seed=2026):
    """Seeded draws over the shapes the rotary decode kernel distinguishes: head dimension, rank class (16 / 32 /
    64 and ranks inside a class), group size (row padding 4, 8, 16), more agents than slots of a tile, lengths
    around the 32-key step and the share boundaries, contiguous and paged."""
    rng = np.random.default_rng(seed)
    for i in range(count):
        d = int(rng.choice([64, 128]))
        rank = int(rng.choice([8, 16, 24, 32, 40, 64]))
        group = int(rng.choice([1, 2, 4, 7, 8, 16]))
        hkv = int(rng.choice([1, 2, 4]))
        agents = int(rng.integers(1, 10))
        theta = float(rng.choice([10000.0, 500000.0]))
        if i % 2 == 0:
            n = int(rng.choice([1, 31, 32, 33, 127, 128, 129, 500, 1025, 2600]))
            w = W.make_contiguous(f"rnd{i}", "decode", seed=1000 + i, n_agents=agents, n_q_heads=group * hkv, n_kv_heads=hkv,
                                  head_dim=d, rank=rank, n=n, n_new=1, d_model=None, b_std=0.1)
        else:
            lens = [int(x) for x in rng.choice([1, 15, 16, 17, 100, 129, 700, 1500], size=int(rng.integers(1, 5)))]
            w = W.make_paged(f"rnd{i}", seed=1000 + i, seq_lens=lens, agents_per_seq=agents, n_adapters=3,
                             n_q_heads=group * hkv, n_kv_heads=hkv, head_dim=d, rank=rank, d_model=None, b_std=0.1)
        yield f"{i}_d{d}_r{rank}_g{group}_kv{hkv}_a{agents}_{'paged' if i % 2 else 'contig'}", w, theta


@pytest.mark.parametrize("name,w,theta", list(_random_decode_cases()), ids=[c[0] for c in _random_decode_cases()])
def test_rotary_decode_random_shapes(name, w, theta):
    got = _run(w, theta)
    ref = _oracle(w, theta)
    rel, mx = errors(got, ref)
    print(f"{name}: relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert np.isfinite(got).all()
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL


def test_rotary_key_side_without_key_adapter_is_the_plain_path():
    """b_k = NULL: nothing to rotate; the result agrees with key_rope_theta = 0 (which runs on the MFMA kernels)."""
    w = W.make_contiguous("rope_nobk", "decode", seed=306, n_agents=2, n_q_heads=8, n_kv_heads=2, head_dim=128,
                          rank=16, n=300, n_new=1, d_model=None, b_std=0.1)
    outs = []
    for theta in (0.0, 500000.0):
        dw = DeviceWorkload(w, DEV, key_rope_theta=theta)
        dw.alloc_workspace()
        dw.b_k = None
        dw.decode()
        torch.cuda.synchronize()
        outs.append(dw.out.to(torch.float64).cpu().numpy())
    w.b_k.zero_()
    rel, mx = errors(outs[1], _oracle(w, 500000.0))
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL
    rel, mx = errors(outs[0], outs[1])
    assert rel <= REL_L2_TOL


@pytest.mark.parametrize("paged", [False, True], ids=["contiguous", "paged"])
@pytest.mark.parametrize("n,agents", [(8192, 4), (20011, 4), (60000, 8)])
def test_static_and_ordinary_decode_without_a_key_adapter_give_the_same_bits(n, agents, paged):
    """One plan for both entry points, whatever the size of the workspace: the bytes asked for, and four times that."""
    hq, hkv, d, r = 32, 8, 128, 16
    gen = torch.Generator(device=DEV).manual_seed(1700 + n)
    rn = lambda *sh: torch.randn(*sh, generator=gen, device=DEV, dtype=torch.bfloat16)
    blocks = (n + 15) // 16
    k, v = (rn(blocks, hkv, 16, d), rn(blocks, hkv, 16, d)) if paged else (rn(n, hkv, d), rn(n, hkv, d))
    l = rn(blocks, 16, r) if paged else rn(n, r)
    table = torch.randperm(blocks, generator=gen, device=DEV).to(torch.int32)[None] if paged else None
    b_v, q = rn(agents, r, hkv * d).mul_(0.1), rn(agents, hq, d)
    lens = torch.tensor([n], dtype=torch.int32, device=DEV)
    ids = torch.arange(agents, dtype=torch.int32, device=DEV)
    start = torch.tensor([0, agents], dtype=torch.int32, device=DEV)
    shape, cache = lra.make_shape(q, hkv, r, 0.0, 500000.0), lra.make_cache(k, v, l, lens, n, table)
    need = lra.lra_workspace_bytes(shape, cache, agents, agents)
    outs = []
    for size in (need, 4 * need):
        outs.append(torch.full_like(q, float("nan")))
        ws = torch.empty(size, dtype=torch.uint8, device=DEV)
        lra.lra_attn_decode(shape, cache, None, b_v, agents, q, ids, start, agents, outs[-1], ws)
    outs.append(torch.full_like(q, float("nan")))
    lra.lra_attn_decode_static(shape, cache, None, b_v, agents, q, ids, start, agents, outs[-1])
    torch.cuda.synchronize()
    assert torch.isfinite(outs[0]).all()
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])


def _prefill_cases():
    mk = W.make_contiguous
    yield "d128_r16_ragged", mk("rp1", "prefill", seed=311, n_agents=1, n_q_heads=8, n_kv_heads=2, head_dim=128, rank=16,
                                n=700, n_new=300, d_model=None, b_std=0.1), 500000.0
    yield "d64_r24", mk("rp2", "prefill", seed=312, n_agents=1, n_q_heads=6, n_kv_heads=3, head_dim=64, rank=24,
                        n=391, n_new=391, d_model=None, b_std=0.1), 10000.0
    yield "d128_r64", mk("rp3", "prefill", seed=313, n_agents=1, n_q_heads=4, n_kv_heads=4, head_dim=128, rank=64,
                         n=260, n_new=129, d_model=None, b_std=0.05), 500000.0
    yield "positions_beyond_40000", mk("rp4", "prefill", seed=314, n_agents=1, n_q_heads=4, n_kv_heads=1, head_dim=128, rank=16,
                                       n=41000, n_new=70, d_model=None, b_std=0.1), 500000.0
    # the same positions with a handful of rows, so that the vector-ALU kernels (one wave per row and key
    # share) finish it quickly as well
    yield "positions_beyond_40000_few_rows", mk("rp4b", "prefill", seed=320, n_agents=1, n_q_heads=2, n_kv_heads=1, head_dim=128,
                                                rank=16, n=41000, n_new=3, d_model=None, b_std=0.1), 500000.0
    yield "paged_second_sequence", None, 500000.0
    # few new tokens after a long context: the causal form of the split-KV kernel
    yield "short_7_tokens_r16", mk("rp6", "prefill", seed=317, n_agents=1, n_q_heads=32, n_kv_heads=8, head_dim=128, rank=16,
                                   n=3000, n_new=7, d_model=None, b_std=0.1), 500000.0
    yield "short_1_token_r32_g7", mk("rp7", "prefill", seed=318, n_agents=1, n_q_heads=28, n_kv_heads=4, head_dim=128, rank=32,
                                     n=1234, n_new=1, d_model=None, b_std=0.1), 500000.0
    yield "short_32_tokens_r64_d64", mk("rp8", "prefill", seed=319, n_agents=1, n_q_heads=4, n_kv_heads=2, head_dim=64, rank=64,
                                        n=900, n_new=32, d_model=None, b_std=0.05), 10000.0
    yield "paged_short", None, 500000.0


def _prefill_params():
    """Every case on both kernel families, except the 70-token case at 41000 positions on the vector-ALU
    kernels (280 rows walking 41000 keys each): its few-row sibling covers those positions there.  On the MFMA
    kernels every case runs twice: with the completed keys written to the workspace by the pre-pass (what a
    contiguous cache gets by default) and with every key tile completed inside the kernel."""
    for variant, vid, prepass in ((0, "mfma_key_prepass", True), (0, "mfma_in_kernel", False), (1, "vector_alu", True)):
        for name, w, theta in _prefill_cases():
            if variant == 1 and name == "positions_beyond_40000":
                continue
            yield pytest.param(name, w, theta, variant, prepass, id=f"{name}-{vid}")


@pytest.mark.parametrize("name,w,theta,variant,prepass", list(_prefill_params()))
def test_rotary_key_side_prefill(name, w, theta, variant, prepass):
    """The MFMA prefill kernel runs on keys completed once by a pre-pass (contiguous caches) or completes every
    key tile in LDS itself (E = L B_K rotated and added to the K_base rows) before the scores; a handful of new
    tokens after a long context takes the causal rotary form of the split-KV kernel; the vector-ALU kernels
    serve the same calls when asked to (kernel variant 1)."""
    prev = lra.lra_set_kernel_variant(variant)
    prev_pp = lra.lra_set_rope_key_prepass(prepass)
    try:
        if w is None:
            _paged_prefill(theta, 9 if name == "paged_short" else 130)
            return
        got = _run(w, theta)
    finally:
        lra.lra_set_kernel_variant(prev)
        lra.lra_set_rope_key_prepass(prev_pp)
    ref = _oracle(w, theta)
    rel, mx = errors(got, ref)
    moved = np.linalg.norm(ref - _oracle(w, 0.0)) / np.linalg.norm(ref)
    print(f"{name}: relL2={rel:.3e} maxabs={mx:.3e}; the rotation moves the output by {moved:.3e}", flush=True)
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL
    assert moved > 4 * REL_L2_TOL


def _paged_prefill(theta, n_new):
    """New tokens at the end of the second sequence of a paged cache (blocks in permuted order)."""
    hkv, hq, d, r = 2, 8, 128, 16
    seq_lens, s = [77, 500], 1
    bs, max_blocks, num_blocks = 16, 32, 70
    gen = torch.Generator().manual_seed(315)
    perm = torch.randperm(num_blocks, generator=gen).to(torch.int32)
    table = torch.stack([perm[:max_blocks], perm[max_blocks:2 * max_blocks]])
    rn = lambda *sh, std=1.0: (std * torch.randn(*sh, generator=gen)).to(torch.bfloat16)
    k_pool, v_pool, l_pool = rn(num_blocks, hkv, bs, d), rn(num_blocks, hkv, bs, d), rn(num_blocks, bs, r)
    q, b_k, b_v = rn(n_new, hq, d), rn(2, r, hkv * d, std=0.1), rn(2, r, hkv * d, std=0.1)
    dev = lambda t: t.to(DEV)
    lens_d = torch.tensor(seq_lens, dtype=torch.int32, device=DEV)
    qd, kd, vd, ld, td, bkd, bvd = dev(q), dev(k_pool), dev(v_pool), dev(l_pool), dev(table), dev(b_k), dev(b_v)
    shape = lra.make_shape(qd, hkv, r, 0.0, theta)
    cache = lra.make_cache(kd, vd, ld, lens_d, max(seq_lens), td)   # holds raw pointers: the tensors stay alive above
    out = torch.full_like(qd, float("nan"))
    ws = torch.empty(max(lra.lra_workspace_bytes(shape, cache, 1, 1, n_new), 256), dtype=torch.uint8, device=DEV)
    lra.lra_attn_prefill(shape, cache, bkd, bvd, 2, qd, s, 1, out, ws)
    torch.cuda.synchronize()
    f = lambda t: t.to(torch.float64).cpu().numpy()
    ids = table[s].numpy()
    kb, vb = oracle.gather_paged(f(k_pool), ids, seq_lens[s]), oracle.gather_paged(f(v_pool), ids, seq_lens[s])
    lr = oracle.lra_oracle.gather_paged_l(f(l_pool), ids, seq_lens[s])
    ref = oracle.prefill(f(q), kb, vb, lr, f(b_k[1]), f(b_v[1]), n=seq_lens[s], scale=1.0 / d ** 0.5, key_rope_theta=theta)
    rel, mx = errors(f(out), ref)
    print(f"paged prefill: relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
    assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL


def test_rotary_key_side_prefill_with_shared_key_tiles():
    """Few q tiles: the key tiles of a q tile are shared by several workgroups (forced to 5, then 32 with empty
    shares) and merged; every share completes its own tiles."""
    w = W.make_contiguous("rp5", "prefill", seed=316, n_agents=1, n_q_heads=4, n_kv_heads=2, head_dim=128, rank=16,
                          n=2000, n_new=40, d_model=None, b_std=0.1)
    ref = _oracle(w, 500000.0)
    for splits in (5, 32):
        prev = lra.lra_set_prefill_splits(splits)
        try:
            got = _run(w, 500000.0)
        finally:
            lra.lra_set_prefill_splits(prev)
        rel, mx = errors(got, ref)
        print(f"splits {splits}: relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
        assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL


def test_rotary_decode_with_more_key_shares_than_tiles():
    """Rotary decode on a ragged paged batch with 128 keys per share (sequences of 1 to 65 tokens leave
    most shares of the batch empty, and every share, empty or not, must leave what the merge kernel reads),
    then with one share per sequence."""
    w = W.make_paged("rope_paged3", seed=308, seq_lens=[1, 63, 64, 65, 1000, 2500], agents_per_seq=3, n_adapters=3,
                     n_q_heads=8, n_kv_heads=2, head_dim=128, rank=16, d_model=None, b_std=0.1)
    ref = _oracle(w, 500000.0)
    for keys in (128, 4096):
        prev = lra.lra_set_decode_split_keys(keys)
        try:
            got = _run(w, 500000.0)
        finally:
            lra.lra_set_decode_split_keys(prev)
        rel, mx = errors(got, ref)
        print(f"{keys} keys per share: relL2={rel:.3e} maxabs={mx:.3e}", flush=True)
        assert rel <= REL_L2_TOL and mx <= MAX_ABS_TOL
