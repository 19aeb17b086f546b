"""Performance cases of the library: what a program that uses it has it do.

Three kinds of pass, each through the public binding:

  step    ``ChunkedPrefill.run``: a whole prompt, chunk by chunk (append, then
          attention), as one pipeline stage runs it.  Returns O, every chunk's
          LSE and the block pools.
  attend  one chunk's attention behind a prefix that is already stored:
          ``mocap_chunk_attn`` ("plain"), ``mocap_chunk_attn_noalloc``
          ("noalloc"), or ``mocap_chunk_attn_two_store`` with the first half of
          the prefix in a second store ("two_store").  Returns O and LSE.
  append  ``mocap_kv_append`` of one chunk at a start position.  Returns the
          block pools.

Inputs are the synthetic ones used throughout: Q, K, V ~ N(0, 1) in bf16,
score scale 1/sqrt(head_dim); block tables are the identity or a permutation.
"""
import math

import torch

from paper_2606_22968_amd import binding
from paper_2606_22968_amd.prefill import ChunkedPrefill

# (query heads, KV heads, head_dim): the attention layers of Llama-3-8B and
# Llama-3-70B, and the other layouts (multi-head, grouped, odd groups,
# multi-query) that the library is tested with.
HEADS = ((32, 8, 128), (64, 8, 128), (8, 8, 64), (8, 4, 128), (8, 2, 128), (16, 2, 64), (12, 4, 128),
         (32, 1, 128), (64, 1, 64), (6, 3, 128))


def listed():
    """Twelve cases, from a 572-token prompt to a 131072-token one."""
    return [
        # The smallest workload: four short chunks, bound by launches and latency.
        dict(name="step_small_d64", kind="step", h_q=8, h_kv=8, d=64, seq=1024, chunks=4, plan="uniform", bs=256,
             permuted=False),
        # A short prompt cut at odd places (prefixes and lengths off every tile edge).
        dict(name="step_ragged", kind="step", h_q=8, h_kv=2, d=128, seq=572, chunks=8,
             plan="1,7,100,129,13,255,64,3", bs=64, permuted=True),
        # The benchmark: a Llama-3-8B layer, 32768 tokens in 16 chunks of 2048.
        dict(name="step_8b_32k", kind="step", h_q=32, h_kv=8, d=128, seq=32768, chunks=16, plan="uniform", bs=256,
             permuted=False),
        # The latency-balanced plan of a 131072-token prompt: long first chunk, short late ones.  The largest case.
        dict(name="step_8b_128k_balanced", kind="step", h_q=32, h_kv=8, d=128, seq=131072, chunks=16,
             plan="balanced", bs=256, permuted=False),
        # The last chunk of a 65536-token prompt at the Llama-3-70B shape.
        dict(name="attend_70b_64k", kind="attend", h_q=64, h_kv=8, d=128, prefix=63488, len=2048, bs=256,
             permuted=False, via="plain"),
        # A debtor stage: half of a long prefix in a second store, permuted blocks.
        dict(name="attend_8b_two_store", kind="attend", h_q=32, h_kv=8, d=128, prefix=126976, len=4096, bs=256,
             permuted=True, via="two_store"),
        # The remainder that ends a prompt whose length is no multiple of the chunk, in a serving loop that
        # must not allocate.
        dict(name="attend_8b_tail", kind="attend", h_q=32, h_kv=8, d=128, prefix=30720, len=137, bs=256,
             permuted=True, via="noalloc"),
        # A few new tokens behind a cached history (prefill-only scoring of short continuations).
        dict(name="attend_8b_few_tokens", kind="attend", h_q=32, h_kv=8, d=128, prefix=9001, len=7, bs=256,
             permuted=True, via="plain"),
        # A short chunk behind about a million tokens.
        dict(name="attend_8b_1m_prefix", kind="attend", h_q=32, h_kv=8, d=128, prefix=(1 << 20) + 64, len=300,
             bs=256, permuted=True, via="plain"),
        # Head dimension 64, multi-query heads, off-grid lengths.
        dict(name="attend_mqa_d64", kind="attend", h_q=64, h_kv=1, d=64, prefix=16001, len=1000, bs=320,
             permuted=True, via="plain"),
        # The KV write of one ordinary chunk.
        dict(name="append_8b_2048", kind="append", h_q=32, h_kv=8, d=128, prefix=30720, len=2048, bs=256,
             permuted=False),
        # The KV write of a long chunk that starts off every boundary.
        dict(name="append_offset", kind="append", h_q=64, h_kv=8, d=128, prefix=8191, len=20011, bs=192,
             permuted=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# Drawn cases stay below this much arithmetic (the largest listed case has 1.4e14).
MAX_FLOPS = 2e13


def draw(rng):
    """Another case of the listed ranges: prompts of 200 to 65536 tokens in 1
    to 16 chunks; chunks of 1 to 8192 tokens behind prefixes of 0 to about a
    million; appends of 1 to 32768 tokens; every head layout, block sizes from
    64 to 1600, odd lengths and positions among them."""
    kind = rng.choice(("step", "attend", "attend", "attend", "append"))
    h_q, h_kv, d = rng.choice(HEADS[:2] + HEADS)
    case = dict(kind=kind, h_q=h_q, h_kv=h_kv, d=d, bs=rng.choice((64, 128, 192, 256, 256, 320, 1600)),
                permuted=rng.random() < 0.5)
    pair_flops = 4.0 * d * h_q
    if kind == "step":
        seq = min(_log_int(rng, 200, 65536), int(math.sqrt(2 * MAX_FLOPS / pair_flops)))
        chunks = rng.randint(1, 16)
        plan = rng.choice(("uniform", "balanced", "ragged"))
        if plan == "balanced":
            seq = max(seq // 512, chunks) * 512
        elif plan == "ragged":
            cuts = sorted(rng.sample(range(1, seq), min(chunks, 64) - 1))
            plan = ",".join(str(b - a) for a, b in zip([0] + cuts, cuts + [seq]))
        return dict(case, seq=seq, chunks=chunks, plan=plan)
    if kind == "append":
        return dict(case, len=_log_int(rng, 1, 32768), prefix=rng.choice((0, 256 * rng.randint(1, 256),
                                                                          rng.randint(1, 65536))))
    n = _log_int(rng, 1, 8192)
    prefix = rng.choice((0, 256 * rng.randint(1, 512), _log_int(rng, 64, 1 << 20), _log_int(rng, 64, 1 << 18)))
    prefix = min(prefix, int(MAX_FLOPS / pair_flops / n))
    via = rng.choice(("plain", "plain", "noalloc", "two_store"))
    if via == "two_store" and prefix < 128:
        via = "plain"
    return dict(case, prefix=prefix, len=n, via=via)


def _lengths(case):
    if case["plan"] in ("uniform", "balanced"):
        return binding.mocap_chunk_plan(case["seq"], case["chunks"], 128, balanced=case["plan"] == "balanced")
    return [int(x) for x in case["plan"].split(",")]


def _scale(case):
    return float(torch.tensor(1.0 / case["d"] ** 0.5, dtype=torch.float32))


def _qkv(case, seed, n_q, n_kv):
    """Q [n_q][Hq][d], K and V [n_kv][Hkv][d] on the GPU."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return tuple(torch.randn((n, h, case["d"]), generator=g, device="cuda", dtype=torch.bfloat16)
                 for n, h in ((n_q, case["h_q"]), (n_kv, case["h_kv"]), (n_kv, case["h_kv"])))


def _table(case, seed, n_tokens):
    blocks = -(-n_tokens // case["bs"])
    if not case["permuted"]:
        return torch.arange(blocks, dtype=torch.int32)
    g = torch.Generator(device="cpu")
    g.manual_seed(seed + 1)
    return torch.randperm(blocks, generator=g).to(torch.int32)


def _remote_end(case):
    """The first half of the prefix, in whole 64-key tiles, is in the second store."""
    return case["prefix"] // 2 // 64 * 64 if case.get("via") == "two_store" else 0


def prepare(case, seed):
    d, h_kv, bs = case["d"], case["h_kv"], case["bs"]
    if case["kind"] == "step":
        table = _table(case, seed, case["seq"])
        runner = ChunkedPrefill(case["h_q"], h_kv, d, _lengths(case), block_size=bs, table=table, pool_fill=0.0)
        q, k, v = _qkv(case, seed, case["seq"], case["seq"])
        return dict(case=case, runner=runner, q=q, k=k, v=v, scale=_scale(case),
                    lse=[runner.lse(c) for c in range(len(runner.lengths))])
    p, n = case["prefix"], case["len"]
    table = _table(case, seed, p + n).cuda()
    store = binding.KvStore(table.numel(), bs, h_kv, d, fill=0.0)
    if case["kind"] == "append":
        _, k, v = _qkv(case, seed, 0, n)
        return dict(case=case, store=store, table=table, k=k, v=v)
    q, k, v = _qkv(case, seed, n, p + n)
    binding.mocap_kv_append(store, table, 0, k, v)
    state = dict(case=case, store=store, table=table, q=q, scale=_scale(case), o=torch.empty_like(q),
                 lse=torch.empty((case["h_q"], n), dtype=torch.float32, device="cuda"))
    remote_end = _remote_end(case)
    if remote_end:
        remote_table = _table(case, seed + 7, remote_end).cuda()
        state.update(remote=binding.KvStore(remote_table.numel(), bs, h_kv, d, fill=0.0), remote_table=remote_table,
                     remote_end=remote_end)
        binding.mocap_kv_append(state["remote"], remote_table, 0, k[:remote_end], v[:remote_end])
    if case["via"] != "noalloc":
        _, ws_bytes = binding.mocap_chunk_attn_workspace_size(p, n, case["h_q"], h_kv, d, 0)
        state["workspace"] = torch.empty(max(ws_bytes, 16), dtype=torch.uint8, device="cuda")
    return state


def run(state):
    case = state["case"]
    if case["kind"] == "step":
        runner = state["runner"]
        runner.run(state["q"], state["k"], state["v"], state["scale"])
        return dict(o=runner.o, lse=state["lse"], k_pool=runner.store.k_pool, v_pool=runner.store.v_pool)
    store, table, p = state["store"], state["table"], case["prefix"]
    if case["kind"] == "append":
        binding.mocap_kv_append(store, table, p, state["k"], state["v"])
        return dict(k_pool=store.k_pool, v_pool=store.v_pool)
    q, scale, o, lse = state["q"], state["scale"], state["o"], state["lse"]
    if case["via"] == "noalloc":
        binding.mocap_chunk_attn_noalloc(store, table, q, p, scale, o, lse)
    elif case["via"] == "two_store":
        binding.mocap_chunk_attn_two_store(store, table, state["remote"], state["remote_table"], 0,
                                           state["remote_end"], q, p, scale, o, lse, state["workspace"])
    else:
        binding.mocap_chunk_attn(store, table, q, p, scale, o, lse, state["workspace"])
    return dict(o=o, lse=lse)


def work(case):
    """K and V read once (and written once where the pass stores them), Q read,
    O and LSE written; 4 d FLOP per head and visible (query, key) pair."""
    h_q, h_kv, d = case["h_q"], case["h_kv"], case["d"]
    if case["kind"] == "append":
        return dict(bytes=8 * case["len"] * h_kv * d, flops=0)
    if case["kind"] == "step":
        s = case["seq"]
        return dict(bytes=4 * s * h_q * d + 4 * s * h_q + 8 * s * h_kv * d,
                    flops=4 * d * h_q * (s * (s + 1) // 2))
    p, n = case["prefix"], case["len"]
    return dict(bytes=4 * n * h_q * d + 4 * n * h_q + 4 * (p + n) * h_kv * d,
                flops=4 * d * h_q * (n * p + n * (n + 1) // 2))


def tolerance(case):
    """Appends copy bits.  Attention rounds the probabilities and O to bf16;
    another block order or reference exponent rounds them elsewhere.  Between
    split counts, O differs by up to 3.1e-3 (2-norm) and single values by up
    to 1.6e-2 of the larger of themselves and the root mean square; against
    float64 by 2.4e-3.  Stated: four times that."""
    if case["kind"] == "append":
        return "exact"
    return dict(rel=1.2e-2, max=6.4e-2)


def _exact_attn(q, k, v, prefix, scale):
    """Attention of the rows q behind `prefix` keys in float64: O [n][Hq][d], LSE [Hq][n]."""
    n, h_q, d = q.shape
    h_kv, keys = k.shape[1], prefix + n
    group = h_q // h_kv
    o = torch.empty((n, h_q, d), dtype=torch.float64, device=q.device)
    lse = torch.empty((h_q, n), dtype=torch.float64, device=q.device)
    rows = max(1, min(n, (1 << 27) // keys))
    at = torch.arange(keys, device=q.device)
    for h in range(h_kv):
        kt, vd = k[:keys, h].double().t().contiguous(), v[:keys, h].double()
        for g in range(h * group, (h + 1) * group):
            for r in range(0, n, rows):
                e = min(n, r + rows)
                s = (q[r:e, g].double() @ kt) * scale
                s.masked_fill_(at[None, :] > prefix + torch.arange(r, e, device=q.device)[:, None], -math.inf)
                lse[g, r:e] = torch.logsumexp(s, 1)
                o[r:e, g] = s.sub_(lse[g, r:e, None]).exp_() @ vd
    return o, lse


def _exact_pools(case, table, start, k, v):
    """The pools after K, V are stored at positions start, start + 1, ..."""
    bs, h_kv, d = case["bs"], case["h_kv"], case["d"]
    pos = torch.arange(start, start + k.shape[0])
    block, slot = table.cpu().long()[pos // bs].cuda(), (pos % bs).cuda()
    k_pool = torch.zeros((table.numel(), h_kv, bs, d), dtype=torch.float64, device="cuda")
    v_pool = torch.zeros((table.numel(), h_kv, d, bs), dtype=torch.float64, device="cuda")
    k_pool[block, :, slot] = k.double()
    v_pool[block, :, :, slot] = v.double()
    return k_pool, v_pool


def exact(case, seed):
    """What run() returns, in float64 torch (None where that takes too long)."""
    if work(case)["flops"] > 2.5e13:
        return None
    if case["kind"] == "append":
        _, k, v = _qkv(case, seed, 0, case["len"])
        k_pool, v_pool = _exact_pools(case, _table(case, seed, case["prefix"] + case["len"]), case["prefix"], k, v)
        return dict(k_pool=k_pool, v_pool=v_pool)
    scale = _scale(case)
    if case["kind"] == "attend":
        q, k, v = _qkv(case, seed, case["len"], case["prefix"] + case["len"])
        o, lse = _exact_attn(q, k, v, case["prefix"], scale)
        return dict(o=o, lse=lse)
    q, k, v = _qkv(case, seed, case["seq"], case["seq"])
    o, lse, p = [], [], 0
    for n in _lengths(case):
        part = _exact_attn(q[p:p + n], k[:p + n], v[:p + n], p, scale)
        o.append(part[0])
        lse.append(part[1])
        p += n
    k_pool, v_pool = _exact_pools(case, _table(case, seed, case["seq"]), 0, k, v)
    return dict(o=torch.cat(o), lse=lse, k_pool=k_pool, v_pool=v_pool)
