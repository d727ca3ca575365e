"""The work that is timed when this library's speed is judged: one attention layer's calls of a
multi-LoRA agent system, through the public entry points.

A case describes one call (or, for a token step, the two calls a layer makes per generated token):
`op` decode | prefill | append | token, the attention heads, rank, agents, sequences and lengths,
whether the cache is paged, whether every adapter has its own low-rank cache, whether the keys carry
an adapter, and whether that adapter's contribution is rotated.  Lengths follow from the case alone
(`length_seed` for a ragged batch), values from the seed.
"""
from __future__ import annotations

import random

import torch

import paper_2602_01053_amd as lra
from paper_2602_01053_amd.workloads import BASE_SEED, ragged_lengths

ROPE_THETA = 500000.0
BLOCK = 16

# Attention layers: query heads, kv heads, head dimension, model width.
LAYERS = {
    "llama3_8b": (32, 8, 128, 4096),
    "qwen25_7b": (28, 4, 128, 3584),
    "tiny": (4, 4, 64, 256),
}


def _case(name, op, layer, n, *, rank=16, agents=1, seqs=1, shortest=0, length_seed=0, n_new=1,
          dtype="bf16", paged=False, lr_per_adapter=False, key_side=True, rope=False):
    """n: cached tokens (the longest sequence's upper bound in a ragged batch), the new ones included."""
    c = {"op": op, "layer": layer, "n": n, "rank": rank, "agents": agents, "seqs": seqs,
         "shortest": shortest or n, "length_seed": length_seed, "n_new": n_new, "dtype": dtype,
         "paged": paged, "lr_per_adapter": lr_per_adapter, "key_side": key_side, "rope": rope}
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest call: a unit-test sized fp32 decode of two agents, all latency.
        _case("decode_fp32_tiny", "decode", "tiny", 512, rank=8, agents=2, dtype="fp32"),
        # One generated token of a short agent trajectory (the trace's 1.9k tokens): project the token
        # into the caches, then attend; adapters on queries and values only, the usual LoRA setting.
        _case("token_step_n1877", "token", "llama3_8b", 1877, key_side=False),
        # The headline decode: four agents on one shared 8k context.
        _case("decode_a4_n8192", "decode", "llama3_8b", 8192, agents=4),
        # A long trajectory with eight agents and the largest rank.
        _case("decode_a8_n32768_r64", "decode", "llama3_8b", 32768, rank=64, agents=8),
        # Serving: 16 trajectories of 4k to 64k tokens in a paged cache, four agents each.
        _case("decode_ragged_paged", "decode", "qwen25_7b", 65536, rank=32, agents=4, seqs=16,
              shortest=4096, length_seed=BASE_SEED + 5, paged=True),
        # LoRA on the key projection of a rotary model (the qkvo ablation), an odd length.
        _case("decode_rotary_n20011", "decode", "llama3_8b", 20011, rank=8, agents=4, rope=True),
        # BaseShared: every agent brings its own low-rank cache; a smaller ragged paged batch.
        _case("decode_own_lr_paged", "decode", "llama3_8b", 24000, agents=4, seqs=8,
              shortest=1500, length_seed=BASE_SEED + 7, paged=True, lr_per_adapter=True),
        # The trace's most frequent prefill: an 8-token turn on a long context.
        _case("prefill_8_after_9001", "prefill", "llama3_8b", 9009, n_new=8),
        # A tool's answer of a few hundred tokens, paged cache, adapters on queries and values only.
        _case("prefill_333_paged", "prefill", "llama3_8b", 5333, n_new=333, paged=True, key_side=False),
        # The headline prefill: 2048 new tokens after a shared 16k context.
        _case("prefill_2048_after_16384", "prefill", "llama3_8b", 18432, n_new=2048),
        # The caches of a few hundred new tokens (an ordinary prompt chunk, ragged).
        _case("append_509", "append", "llama3_8b", 1021, n_new=509),
        # The caches of a retrieved document: the largest chunk of the trace.
        _case("append_16384", "append", "llama3_8b", 16896, n_new=16384),
    ]


def _log(rng, lo, hi):
    """An integer of [lo, hi], spread over its logarithm."""
    return min(hi, max(lo, int(round(lo * (hi / lo) ** rng.random()))))


def draw(rng):
    layer = rng.choice(("llama3_8b", "llama3_8b", "qwen25_7b"))
    rank = rng.choice((8, 16, 16, 24, 32, 64))
    op = rng.choice(("decode", "decode", "decode", "batch", "batch", "token", "prefill", "prefill", "prefill",
                     "append", "append", "tiny"))
    paged = rng.random() < 0.4
    key_side = rng.random() < 0.7
    rope = key_side and rng.random() < 0.25
    if op == "tiny":
        return _case(None, "decode", "tiny", _log(rng, 100, 4000), rank=rng.choice((8, 16)),
                     agents=rng.randint(1, 4), dtype="fp32")
    if op == "decode":
        return _case(None, "decode", layer, _log(rng, 700, 66000), rank=rank, agents=_log(rng, 1, 8), paged=paged,
                     key_side=key_side, rope=rope, lr_per_adapter=not rope and rng.random() < 0.2)
    if op == "batch":
        rope = rope and rng.random() < 0.5
        longest = _log(rng, 2000, 12000 if rope else 32000)
        return _case(None, "decode", layer, longest, rank=min(rank, 32), agents=rng.randint(1, 4), seqs=_log(rng, 2, 16),
                     shortest=max(64, int(longest * rng.uniform(0.05, 1.0))), length_seed=rng.randrange(1 << 20),
                     paged=True, key_side=key_side, rope=rope,
                     lr_per_adapter=not rope and rng.random() < 0.25)
    if op == "token":
        return _case(None, "token", layer, _log(rng, 300, 33000), rank=rank, key_side=key_side, paged=paged)
    if op == "prefill":
        n_new = _log(rng, 4, 1800)
        return _case(None, "prefill", layer, n_new + _log(rng, 200, 16384), rank=min(rank, 32), n_new=n_new, paged=paged,
                     key_side=key_side, rope=rope)
    n_new = _log(rng, 2, 16384)
    return _case(None, "append", layer, n_new + _log(rng, 16, 512), rank=rank, n_new=n_new, paged=paged)


def _lengths(case):
    if case["seqs"] == 1:
        return [case["n"]]
    return ragged_lengths(case["length_seed"], case["seqs"], case["shortest"], case["n"])


class _State:
    """Tensors and descriptors that a serving program holds for one layer."""


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev).manual_seed(seed)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    hq, hkv, d, d_model = LAYERS[case["layer"]]
    r, agents, op, n_new = case["rank"], case["agents"], case["op"], case["n_new"]

    def randn(*shape, std=1.0):
        return torch.randn(*shape, generator=gen, device=dev, dtype=dt).mul_(std)

    s = _State()
    s.op = op
    lengths = _lengths(case)
    n_seqs = len(lengths)
    n_adapters = max(agents, 3)
    if case["paged"]:
        per_seq = [(n + BLOCK - 1) // BLOCK for n in lengths]
        blocks = sum(per_seq)
        order = torch.randperm(blocks, generator=gen, device=dev).to(torch.int32)
        s.block_table = torch.full((n_seqs, max(per_seq)), -1, dtype=torch.int32, device=dev)
        at = 0
        for t, nb in enumerate(per_seq):
            s.block_table[t, :nb] = order[at:at + nb]
            at += nb
        kv_shape, l_shape = (blocks, hkv, BLOCK, d), (blocks, BLOCK, r)
    else:
        s.block_table = None
        kv_shape, l_shape = (lengths[0], hkv, d), (lengths[0], r)
    s.k, s.v = randn(*kv_shape), randn(*kv_shape)
    own = case["lr_per_adapter"]
    s.l = randn(n_adapters, *l_shape) if own else randn(*l_shape)
    s.seq_lens = torch.tensor(lengths, dtype=torch.int32, device=dev)
    s.cache = lra.make_cache(s.k, s.v, s.l, s.seq_lens, max(lengths), s.block_table, l_per_adapter=own,
                             seq_lens_host=lengths)
    s.b_k = randn(n_adapters, r, hkv * d, std=0.02) if case["key_side"] else None
    s.b_v = randn(n_adapters, r, hkv * d, std=0.02)
    s.n_adapters = n_adapters
    s.n_queries = n_new if op == "prefill" else n_seqs * agents
    s.q = randn(s.n_queries, hq, d)
    s.shape = lra.make_shape(s.q, hkv, r, 0.0, ROPE_THETA if case["rope"] else 0.0)
    s.out = torch.empty_like(s.q)
    s.agents = agents
    if op in ("decode", "token"):
        s.query_adapter = (torch.arange(s.n_queries, device=dev) % n_adapters).to(torch.int32)
        s.seq_query_start = (torch.arange(n_seqs + 1, device=dev) * agents).to(torch.int32)
    if op != "append":
        need = lra.lra_workspace_bytes(s.shape, s.cache, s.n_queries, agents, n_new if op == "prefill" else 0)
        s.workspace = torch.empty(max(need, 256), dtype=torch.uint8, device=dev)
    if op in ("append", "token"):
        s.w = randn(2 * hkv * d + r, d_model, std=d_model ** -0.5)
        s.x = randn(n_new, d_model)
        need = lra.lra_append_workspace_bytes(s.shape, s.cache, s.w, ROPE_THETA, n_new)
        s.append_workspace = torch.empty(max(need, 256), dtype=torch.uint8, device=dev)
        s.written = _written_rows(s, case, lengths[0], n_new)
    return s


def _written_rows(s, case, n, n_new):
    """Where an append writes: the last n_new rows, or on a paged cache the blocks that hold them."""
    if not case["paged"]:
        return s.k[n - n_new:n], s.v[n - n_new:n], s.l[n - n_new:n]
    return s.k, s.v, s.l


def run(s):
    if s.op in ("append", "token"):
        lra.lra_cache_append(s.shape, s.cache, s.w, ROPE_THETA, s.x, 0, workspace=s.append_workspace)
        if s.op == "append":
            return s.written
    if s.op == "prefill":
        lra.lra_attn_prefill(s.shape, s.cache, s.b_k, s.b_v, s.n_adapters, s.q, 0, 1, s.out, s.workspace)
        return s.out
    lra.lra_attn_decode(s.shape, s.cache, s.b_k, s.b_v, s.n_adapters, s.q, s.query_adapter, s.seq_query_start,
                        s.agents, s.out, s.workspace)
    return (s.out, *s.written) if s.op == "token" else s.out


def work(case):
    """Bytes: every visible cached row, the adapters in use, queries and outputs once.  Operations: 4(d + r)
    per visible pair of query row and key (less 2r without a key-side adapter; with a rotated one 2rd per
    key, agent and kv head instead of 2r per pair) and the rank-r projections of each row."""
    hq, hkv, d, d_model = LAYERS[case["layer"]]
    es = 2 if case["dtype"] == "bf16" else 4
    r, agents, op, n_new = case["rank"], case["agents"], case["op"], case["n_new"]
    lengths = _lengths(case)
    tokens = sum(lengths)
    nbytes, flops = 0, 0
    if op in ("append", "token"):
        feats = 2 * hkv * d + r
        nbytes += es * (feats * d_model + n_new * d_model + n_new * feats)
        flops += 2 * n_new * d_model * feats
    if op != "append":
        if op == "prefill":
            rows = n_new * hq
            pairs = hq * (n_new * (tokens - n_new) + n_new * (n_new + 1) // 2)
            users = 1
        else:
            rows = len(lengths) * agents * hq
            pairs = agents * hq * tokens
            users = agents
        sides = 2 if case["key_side"] else 1
        used = min(max(agents, 3), len(lengths) * agents) if op != "prefill" else 1
        l_rows = tokens * (users if case["lr_per_adapter"] else 1)
        nbytes += es * (2 * tokens * hkv * d + l_rows * r + sides * used * r * hkv * d + 2 * rows * d)
        flops += pairs * (4 * d + 2 * r) + 2 * rows * d * r
        if case["rope"]:
            flops += 2 * tokens * users * hkv * r * d
        elif case["key_side"]:
            flops += pairs * 2 * r + 2 * rows * d * r
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """About four times what the listed cases show.  bf16: against a float64 evaluation 1.9e-3 to 2.4e-3 (of
    which the rounding of the output alone is 1.7e-3), with another split of the keys 2.0e-3 to 2.5e-3 and at
    most 1.3e-2 on one value; fp32: 5e-7 and 1.5e-6 at 512 keys, more with the length."""
    if case["dtype"] == "fp32":
        return {"rel": 5e-6, "max": 2e-5}
    return {"rel": 1e-2, "max": 6e-2}
