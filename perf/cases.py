"""The work that a user of this library has it do, as cases that can be timed and compared.

A case is one pass of a program through the public entry points: the attention of one or more
blocks of a FedAttn stack over a prompt that N participants share (prefill), one decoding step
of such blocks over their KV caches (decode), or whole decoder blocks with their projections and
element-wise passes (block).  Sizes are those of the workloads in fedattn_inputs.py, of the tests
and of bench.py, or generic ones; inputs are normal draws as there.

Fields of a case
  kind              "prefill", "decode" or "block"
  n, lo, hi, layout  participants, and segment lengths drawn from lo..hi (layout seeds the draw)
  hq, hkv, d, dtype  heads, head dimension, "bf16" or "f32"
  blocks, h         consecutive blocks 0 .. blocks-1 of a stack with sync interval h
  causal            decoder (True) or encoder (False) attention
  chunk, keep       sparse KV exchange in sync blocks: chunk length and kept share (chunk 0: dense)
  kv                where a sync block finds K and V: "global" (one aggregated matrix),
                    "in_place" (the participants' own matrices, back to back), "apart" (allocated
                    one by one, aggregated by the call)
  call              decode: "blocks" (one call for all blocks), "each" (one call per block)
  generated         decode: rows of each cache that are not shown to other participants
  d_model, hidden   block: widths of the residual stream and of the feed-forward network
"""
import random

import numpy as np
import torch

import paper_2511_02647_amd as fa
from paper_2511_02647_amd.block import BlockBuffers, BlockWeights, block_forward


def _prefill(name, n, lo, hi, hq, hkv, d, dtype="bf16", blocks=1, h=1, causal=True, chunk=0, keep=1.0, kv="global", layout=1):
    return dict(name=name, kind="prefill", n=n, lo=lo, hi=hi, layout=layout, hq=hq, hkv=hkv, d=d, dtype=dtype, blocks=blocks, h=h,
                causal=causal, chunk=chunk, keep=keep, kv=kv)


def _decode(name, n, lo, hi, hq, hkv, d, dtype="bf16", blocks=1, h=1, call="blocks", generated=0, layout=1):
    return dict(name=name, kind="decode", n=n, lo=lo, hi=hi, layout=layout, hq=hq, hkv=hkv, d=d, dtype=dtype, blocks=blocks, h=h,
                call=call, generated=generated)


def _block(name, n, lo, hi, hq, hkv, d, d_model, hidden, blocks=2, h=2, chunk=0, keep=1.0, layout=1):
    return dict(name=name, kind="block", n=n, lo=lo, hi=hi, layout=layout, hq=hq, hkv=hkv, d=d, dtype="bf16", blocks=blocks, h=h,
                causal=True, chunk=chunk, keep=keep, d_model=d_model, hidden=hidden)


def listed():
    return [
        # the smallest call: the tiny fp32 stack (2 x 32 tokens, 4 blocks, every second one synchronised); launches and host work
        _prefill("tiny_stack_f32", 2, 32, 32, 2, 2, 64, "f32", blocks=4, h=2),
        # one communication round (3 local blocks, 1 sync block) of a short prompt at Llama-3-8B's attention shape
        _prefill("round_short_prompt", 4, 512, 512, 32, 8, 128, blocks=4, h=4, kv="in_place"),
        # the same round on a long prompt cut unevenly (semantic segmentation): the throughput case
        _prefill("round_uneven_prompt", 8, 1024, 3072, 32, 8, 128, blocks=4, h=4, kv="in_place", layout=3),
        # a local and a sparsely synchronised block on 64k tokens, a quarter of the 64-token chunks exchanged: the largest prompt
        _prefill("round_sparse_64k", 16, 4096, 4096, 16, 4, 128, blocks=2, h=2, chunk=64, keep=0.25),
        # token-granular sparse exchange on odd lengths, every participant's K and V in an allocation of its own
        _prefill("sync_sparse_tokens", 8, 300, 1500, 16, 4, 128, blocks=1, h=1, chunk=1, keep=0.3, kv="apart", layout=5),
        # encoder attention, one KV head per query head, head dimension 64, odd and very short segments among long ones
        _prefill("encoder_ragged_d64", 6, 1, 900, 16, 16, 64, blocks=2, h=2, causal=False, kv="apart", layout=2),
        # fp32 runs (checking a bf16 deployment against full precision): a local and a sync block
        _prefill("prefill_f32", 4, 100, 900, 8, 2, 128, "f32", blocks=2, h=2, layout=4),
        # a model whose head dimension is neither 64 nor 128, bf16
        _prefill("prefill_d96", 4, 100, 900, 8, 2, 96, blocks=2, h=2, layout=4),
        # decoding with few participants and short caches, block after block as a model calls it: latency
        _decode("decode_short_cache", 3, 64, 400, 8, 2, 128, blocks=4, h=4, call="each"),
        # a decoding step of 8 blocks for 16 participants with 1152 cached rows each (6 local, 2 sync): the bandwidth case
        _decode("decode_16_participants", 16, 1152, 1152, 32, 8, 128, blocks=8, h=4),
        # fp32 decoding, ragged caches, the rows generated since the prompt kept private
        _decode("decode_f32_ragged", 5, 200, 1500, 8, 2, 64, "f32", blocks=2, h=2, generated=100, layout=7),
        # two whole decoder blocks (local, sparse sync) of the end-to-end configuration on 16 x 1024 tokens
        _block("decoder_blocks", 16, 1024, 1024, 16, 4, 128, 2048, 5632, blocks=2, h=2, chunk=64, keep=0.25),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def _heads(rng, most):
    while True:
        hkv, g = rng.choice([1, 2, 3, 4, 8]), rng.choice([1, 2, 3, 4, 4, 8])
        if hkv * g <= most:
            return hkv * g, hkv


def draw(rng):
    """One more case: a kind of the list, its sizes spread over the range that the listed ones span."""
    sort = rng.choice(["bf16", "bf16", "bf16", "sparse", "general", "decode", "decode", "decode_general", "block"])
    while True:
        seed = rng.randrange(1 << 30)
        blocks = rng.randint(1, 4)
        h = rng.choice([1, 2, 4])
        n = _log_int(rng, 1, 32)
        hi = _log_int(rng, 16, 4096)
        lo = hi if rng.random() < 0.3 else max(1, int(hi * rng.choice([0.02, 0.3, 0.6])))
        if sort in ("bf16", "sparse"):
            hq, hkv = _heads(rng, 32)
            c = _prefill("", n, lo, hi, hq, hkv, rng.choice([64, 128, 128]), blocks=blocks, h=h, causal=rng.random() < 0.8,
                         kv=rng.choice(["global", "in_place", "apart"]), layout=seed)
            if sort == "sparse":
                c.update(chunk=rng.choice([1, 16, 64, 64, 100, 256]), keep=rng.choice([0.1, 0.25, 0.5]), h=1)
        elif sort == "general":
            hq, hkv = _heads(rng, 8)
            dtype = rng.choice(["f32", "bf16"])
            d = rng.choice([64, 128, 128, 96] if dtype == "f32" else [32, 80, 96, 160, 256])
            c = _prefill("", min(n, 8), lo, hi, hq, hkv, d, dtype, blocks=min(blocks, 2), h=h, causal=rng.random() < 0.8, layout=seed)
        elif sort == "decode":
            hi = _log_int(rng, 64, 8192)
            lo = hi if rng.random() < 0.4 else max(1, int(hi * 0.3))
            hq, hkv = _heads(rng, 32)
            c = _decode("", n, lo, hi, hq, hkv, rng.choice([64, 128, 128]), blocks=rng.choice([1, 2, 4, 8]), h=rng.choice([1, 2, 4]),
                        call=rng.choice(["blocks", "blocks", "each"]), generated=rng.choice([0, 0, lo // 4]), layout=seed)
        elif sort == "decode_general":
            hi = _log_int(rng, 64, 1500)
            lo = max(1, int(hi * 0.3))
            hq, hkv = _heads(rng, 8)
            dtype = rng.choice(["f32", "bf16"])
            c = _decode("", min(n, 8), lo, hi, hq, hkv, rng.choice([64, 128] if dtype == "f32" else [80, 96, 256]), dtype,
                        blocks=min(blocks, 2), h=h, call=rng.choice(["blocks", "each"]), generated=rng.choice([0, lo // 4]), layout=seed)
        else:
            hi = _log_int(rng, 32, 1024)
            hkv = rng.choice([2, 4])
            hq, d = hkv * rng.choice([2, 4]), rng.choice([64, 128])
            c = _block("", min(n, 16), max(1, int(hi * rng.choice([0.3, 1.0]))), hi, hq, hkv, d, hq * d, 8 * _log_int(rng, 64, 704),
                       blocks=blocks, h=h, chunk=rng.choice([0, 1, 64]), keep=0.25, layout=seed)
        if c["n"] * c["hi"] > 65536:
            continue
        w = work(c)
        most = {"general": 6e9, "decode_general": 5e8, "block": 2e12}.get(sort, 1.2e12)
        if w["flops"] <= most and w["bytes"] <= 1.5e9:
            del c["name"]
            return c


def _lens(c):
    r = random.Random(c["layout"])
    return [r.randint(c["lo"], c["hi"]) for _ in range(c["n"])]


def _syncs(c):
    return [(b + 1) % c["h"] == 0 for b in range(c["blocks"])]


def _chunks(lens, chunk):
    return [-(-x // chunk) for x in lens]


def _visible(c, lens, sync):
    """Visible (query, key) pairs of one block and query head."""
    own = sum(x * (x + 1) // 2 if c["causal"] else x * x for x in lens)
    if not sync:
        return own
    kept = lens
    if c["chunk"]:
        kept = [min(x, round(c["keep"] * k) * c["chunk"]) for x, k in zip(lens, _chunks(lens, c["chunk"]))]
    before, remote = 0, 0
    for x, k in zip(lens, kept):
        remote += x * (before if c["causal"] else sum(kept) - k)
        before += k
    return own + remote


def work(c):
    lens, syncs = _lens(c), _syncs(c)
    t = sum(lens)
    es = 2 if c["dtype"] == "bf16" else 4
    row = c["d"] * es
    if c["kind"] == "decode":
        one = c["n"] * c["hq"] * row * 2 + t * c["hkv"] * row * 2
        shown = sum(max(0, x - c["generated"]) for x in lens)
        keys = [sum(x + (shown - max(0, x - c["generated"]) if s else 0) for x in lens) for s in syncs]
        return {"bytes": c["blocks"] * one, "flops": sum(4 * c["d"] * c["hq"] * k for k in keys)}
    fl = sum(4 * c["d"] * c["hq"] * _visible(c, lens, s) for s in syncs)
    if c["kind"] == "prefill":
        flags = sum(_chunks(lens, c["chunk"])) * sum(syncs) if c["chunk"] else 0
        return {"bytes": c["blocks"] * t * row * 2 * (c["hq"] + c["hkv"]) + flags, "flops": fl}
    dm, f, wide = c["d_model"], c["hidden"], (c["hq"] + 2 * c["hkv"]) * c["d"]
    mats = dm * wide + c["hq"] * c["d"] * dm + 3 * dm * f
    # weights, q, k, v and the attention's output, the residual stream in and out and its start copied
    by = c["blocks"] * (2 * mats + t * row * 2 * (c["hq"] + c["hkv"]) + 8 * t * dm) + 4 * t * dm
    return {"bytes": by, "flops": fl + 2 * t * mats * c["blocks"]}


def tolerance(c):
    """About four times the relative error measured against the same function in 64 bits (attention)
    or against the block computed step by step in fp32 with bf16 between the steps (block): bf16 with
    weights rounded to bf16 0.0019-0.0029, other bf16 shapes 0.0016, fp32 2e-7-1e-6, block 0.0035."""
    if c["kind"] == "block":
        return {"rel": 1.4e-2}
    if c["dtype"] == "f32":
        return {"rel": 4e-6}
    return {"rel": 1e-2 if c["d"] in (64, 128) else 6.5e-3}


def _dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def prepare(c, seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dt = _dtype(c)

    def normal(*shape, std=1.0, dtype=dt):
        x = torch.randn(*shape, generator=g, device="cuda", dtype=dtype)
        return x if std == 1.0 else x.mul_(std)

    lens, syncs = _lens(c), _syncs(c)
    seg = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    t = int(seg[-1])
    n, hq, hkv, d = c["n"], c["hq"], c["hkv"], c["d"]
    params = fa.make_params(n, hq, hkv, d, c["h"], dt, causal=c.get("causal", True))
    s = dict(case=c, params=params, seg=seg, syncs=syncs)
    if c["kind"] == "decode":
        # caches with room for 128 more rows per participant, as a serving program keeps them
        cap = (np.arange(n + 1) * (c["hi"] + 128)).astype(np.int32)
        s["cap"], s["lens"] = cap, np.asarray(lens, dtype=np.int32)
        s["shown"] = np.maximum(s["lens"] - c["generated"], 0).astype(np.int32) if c["generated"] else None
        rows = int(cap[-1])
        s["q"] = normal(c["blocks"], n, hq, d)
        s["k"], s["v"] = (normal(c["blocks"], rows, hkv, d) for _ in range(2))
        s["out"] = torch.empty_like(s["q"])
        s["ws"] = torch.empty(max(16, fa.fedattn_workspace_bytes(params, fa.FEDATTN_OP_DECODE, rows)), dtype=torch.uint8, device="cuda")
        return s
    chunk = c["chunk"]
    s["keep"] = [None] * c["blocks"]
    if chunk:
        for b in range(c["blocks"]):
            if syncs[b]:
                flags = []
                for k in _chunks(lens, chunk):
                    f = torch.zeros(k, dtype=torch.uint8, device="cuda")
                    f[torch.rand(k, generator=g, device="cuda").argsort()[:round(c["keep"] * k)]] = 1
                    flags.append(f)
                s["keep"][b] = torch.cat(flags)
    if c["kind"] == "block":
        dm, f = c["d_model"], c["hidden"]
        s["x0"] = normal(t, dm, dtype=torch.float32)
        s["x"] = torch.empty_like(s["x0"])
        s["w"] = [BlockWeights(normal(dm, (hq + 2 * hkv) * d, std=0.02), normal(hq * d, dm, std=0.02), normal(dm, 2 * f, std=0.02),
                               normal(f, dm, std=0.02)) for _ in range(c["blocks"])]
        s["buf"] = BlockBuffers(params, t, dm, f, chunk_tokens=chunk)
        return s
    s["q"] = [normal(t, hq, d) for _ in range(c["blocks"])]
    s["k"], s["v"] = ([normal(t, hkv, d) for _ in range(c["blocks"])] for _ in range(2))
    s["out"] = [torch.empty_like(x) for x in s["q"]]
    op = fa.FEDATTN_OP_PREFILL if c["kv"] == "global" else fa.FEDATTN_OP_PREFILL_SYNC_LOCAL_KV
    s["ws"] = torch.empty(max(16, fa.fedattn_workspace_bytes(params, op, t, chunk)), dtype=torch.uint8, device="cuda")
    s["k_own"], s["v_own"] = [None] * c["blocks"], [None] * c["blocks"]
    for b in range(c["blocks"]):
        if syncs[b] and c["kv"] != "global":
            for own, x in (("k_own", s["k"][b]), ("v_own", s["v"][b])):
                parts = [x[seg[i]:seg[i + 1]] for i in range(n)]
                s[own][b] = [p.clone() for p in parts] if c["kv"] == "apart" else parts
    return s


def run(s):
    c, p, seg = s["case"], s["params"], s["seg"]
    if c["kind"] == "decode":
        if c["call"] == "blocks":
            fa.fedattn_decode_blocks(p, 0, c["blocks"], s["q"], s["k"], s["v"], s["out"], s["q"][0].numel(), s["k"][0].numel(),
                                     s["cap"], s["lens"], remote_lens=s["shown"], workspace=s["ws"])
        else:
            for b in range(c["blocks"]):
                fa.fedattn_decode(p, b, s["q"][b], s["k"][b], s["v"][b], s["out"][b], s["cap"], s["lens"], remote_lens=s["shown"],
                                  workspace=s["ws"])
        return s["out"]
    if c["kind"] == "block":
        x, pending = s["x"], None
        x.copy_(s["x0"])
        for b in range(c["blocks"]):
            keep = s["keep"][b]
            pending = block_forward(p, b, x, s["w"][b], seg, s["buf"], keep_chunks=keep, chunk_tokens=c["chunk"] if keep is not None else 0,
                                    pending=pending, defer_update=True)["pending"]
        fa.fedattn_residual_add(x, pending)
        return x
    for b in range(c["blocks"]):
        keep = s["keep"][b]
        chunk = c["chunk"] if keep is not None else 0
        if s["k_own"][b] is not None:
            fa.fedattn_prefill_sync_local_kv(p, s["q"][b], s["k_own"][b], s["v_own"][b], s["out"][b], seg, keep_chunks=keep,
                                             chunk_tokens=chunk, workspace=s["ws"])
        else:
            fa.fedattn_prefill(p, b, s["q"][b], s["k"][b], s["v"][b], s["out"][b], seg, keep_chunks=keep, chunk_tokens=chunk,
                               workspace=s["ws"] if keep is not None else None)
    return s["out"]
