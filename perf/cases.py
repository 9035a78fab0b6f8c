"""The work this library is asked to do, as cases that can be timed: one device's share of sequence-parallel attention.

A case is a dict of plain values.  `kind` says which entry points a pass goes through:

  train    attention forward and backward over a packed batch with a plan that is kept (the layers of one
           micro-batch share it): flexsp_attn_varlen_fwd, flexsp_attn_varlen_bwd
  step     one layer of a micro-batch whose lengths are new: plan, pack q k v, forward, unpack o, pack dO,
           backward, unpack dq dk dv (what bench.py times)
  infer    flexsp_attn_varlen_fwd_static, the forward without a plan
  ring     one device's pass of a context-parallel ring of p devices, the device with the last 1/p of every
           sequence's rows: p shard forwards folded into the fp32 running result, then p shard backwards that
           add up (flexsp_attn_varlen_fwd_kvshard_acc, flexsp_attn_varlen_bwd_kvshard)
  permute  flexsp_pack_many of q, k, v and flexsp_unpack of o: the local halves of the exchanges alone

`recipe`, `tokens` and `lens_seed` give the sequence lengths (the length recipes of workloads.py, equal or
uniformly drawn lengths); seeds of prepare() change the data, not the lengths.  Data is N(0,1) in bf16, as the
benchmark and the tests draw it.
"""
import dataclasses
import math
import random

import torch

from paper_2412_01523_amd import binding as fx
from paper_2412_01523_amd import workloads as wl

_RECIPE = {"tiny": 0, "lognormal": 1, "pareto": 2, "single": 3, "bimodal": 4}
_ctx = None


def _context():
    """One context per process, as a user's program keeps it."""
    global _ctx
    if _ctx is None:
        _ctx = fx.Context(0)
    return _ctx


def listed():
    return [
        # the smallest batch of the benchmark configurations (436 tokens in four odd sequences): launches and latency
        dict(name="tiny_436_train", kind="train", recipe="tiny", tokens=436, lens_seed=0, hq=4, hkv=4, d=64, causal=True, f32=False),
        # fine-tuning data: nothing but short sequences of odd lengths, which the corpora of the paper mostly consist of
        dict(name="short_48k_train", kind="train", recipe="uniform", low=64, high=1024, tokens=49152, lens_seed=5, hq=8, hkv=8, d=128, causal=True, f32=False),
        # one layer of the 32K-token log-normal micro-batch, 32 heads over 8 devices
        dict(name="lognormal_32k_step", kind="step", recipe="lognormal", tokens=32768, lens_seed=20243201, hq=4, hkv=4, d=128, p=8),
        # one layer of the 64K-token long-tail micro-batch (the headline workload)
        dict(name="pareto_64k_step", kind="step", recipe="pareto", tokens=65536, lens_seed=20244201, hq=8, hkv=8, d=128, p=8),
        # one 131 072-token sequence: the longest context of the benchmark configurations
        dict(name="single_128k_train", kind="train", recipe="single", tokens=131072, lens_seed=0, hq=8, hkv=8, d=128, causal=True, f32=False),
        # grouped-query heads, 256K tokens, long and short sequences in one pack
        dict(name="bimodal_256k_gqa_train", kind="train", recipe="bimodal", tokens=262144, lens_seed=20246201, hq=16, hkv=2, d=128, causal=True, f32=False),
        # a large sequence-parallel group leaves one head of a long sequence on each device
        dict(name="one_head_32k_train", kind="train", recipe="single", tokens=32768, lens_seed=0, hq=1, hkv=1, d=128, causal=True, f32=False),
        # an encoder: no mask, head dim 64, grouped heads, ragged medium lengths, gradients wanted in fp32
        dict(name="encoder_d64_train", kind="train", recipe="uniform", low=200, high=4000, tokens=30011, lens_seed=7, hq=12, hkv=4, d=64, causal=False, f32=True),
        # the long-tail batch as a ring of four devices sees it
        dict(name="pareto_64k_ring", kind="ring", recipe="pareto", tokens=65536, lens_seed=20244201, hq=8, hkv=8, d=128, p=4, causal=True),
        # prompt processing without a plan, grouped-query heads
        dict(name="prompt_16k_infer", kind="infer", recipe="lognormal", tokens=16384, lens_seed=11, hq=16, hkv=2, d=128, causal=True),
        # the permutes alone: q, k, v in and o back, 32 heads over 8 devices
        dict(name="permute_32k", kind="permute", tokens=32768, hq=32, hkv=32, d=128, p=8, elem=2),
        # the permutes on odd sizes and another element type: 24 and 6 heads over 3 devices, 30 011 tokens, fp32
        dict(name="permute_odd_f32", kind="permute", tokens=30011, hq=24, hkv=6, d=80, p=3, elem=4),
    ]


def draw(rng):
    """One more case of the ranges above; no dearer than the dearest listed one."""
    def size(low, high):
        return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))

    kind = rng.choice(("train", "train", "train", "step", "step", "infer", "ring", "permute"))
    p = rng.choice((2, 4, 8))
    if kind == "permute":
        hkv = p * rng.choice((1, 1, 2, 3, 4))
        hq = hkv * rng.choice((1, 1, 2, 4))
        d, elem = rng.choice((64, 72, 80, 128, 128)), rng.choice((1, 2, 2, 4))
        return dict(kind=kind, tokens=size(64, min(131072, (1 << 30) // (hq * d * elem))), hq=hq, hkv=hkv, d=d, p=p, elem=elem)
    group = rng.choice((1, 1, 1, 2, 4, 8))
    hkv = rng.choice((1, 1, 2, 3, 4, 8))
    hq = min(16, hkv * group)
    hkv = hq // group if hq % group == 0 else hq
    recipe = rng.choice(("uniform", "uniform", "lognormal", "pareto", "pareto", "single"))
    c = dict(kind=kind, recipe=recipe, tokens=size(256, 131072), lens_seed=rng.randrange(1 << 20), hq=hq, hkv=hkv, d=rng.choice((64, 128, 128)))
    if recipe == "uniform":
        c["low"] = size(64, 1024)
        c["high"] = c["low"] * rng.choice((1, 2, 8))
    if kind == "step":
        c["p"] = p
        c["tokens"] = max(p, c["tokens"] // p * p)
    else:
        c["causal"] = rng.random() < 0.8
    if kind == "train":
        c["f32"] = rng.random() < 0.3
    if kind == "ring":
        c["p"] = p
        c["tokens"] = max(1024, c["tokens"])
    while _flops(c) > 9e13 * c["d"] / 128:  # the dearest listed case takes 1.4e14 with d = 128, and head dim 64 runs at half the rate
        c["tokens"] = c["tokens"] // 2 // 8 * 8
    return c


# ------------------------------------------------------------------------------------------------ lengths and work
def _lengths(c):
    if c["recipe"] == "uniform":
        rng = random.Random(c["lens_seed"])
        out, left = [], c["tokens"]
        while left > 0:
            out.append(min(left, rng.randint(c["low"], c["high"])))
            left -= out[-1]
        return out
    cfg = dataclasses.replace(wl.CONFIGS[_RECIPE[c["recipe"]]], tokens=c["tokens"])
    return wl.lengths(cfg, c["lens_seed"] or None)


def _shard_cuts(lens, p):
    return [[(j * s) // p for j in range(p + 1)] for s in lens]


def _ring_pairs(c):
    """(query, key) pairs the last device of the ring looks at."""
    pairs = 0
    for s in _lengths(c):
        n = s - ((c["p"] - 1) * s) // c["p"]
        pairs += n * (n + 1) // 2 + n * (s - n) if c["causal"] else n * s
    return pairs


def _flops(c):
    """Counted as everywhere in this repository: two products forward, five backward, masked pairs not at all."""
    if c["kind"] == "permute":
        return 0
    if c["kind"] == "ring":
        return 14 * c["d"] * c["hq"] * _ring_pairs(c)
    fwd, bwd = wl.attn_flops(_lengths(c), c["hq"], c["d"], c.get("causal", True))
    return fwd if c["kind"] == "infer" else fwd + bwd


def work(case):
    c = case
    t, d = c["tokens"], c["d"]
    q, kv = t * c["hq"] * d, t * c["hkv"] * d  # elements of a query-side and of a key-side tensor
    lse = 4 * t * c["hq"]
    if c["kind"] == "permute":
        return {"bytes": 2 * c["elem"] * (2 * q + 2 * kv), "flops": 0}
    forward = 2 * (2 * q + 2 * kv) + lse  # q k v in, o and the log-sum-exp out
    if c["kind"] == "infer":
        return {"bytes": forward, "flops": _flops(c)}
    if c["kind"] == "ring":
        rows = sum(s - ((c["p"] - 1) * s) // c["p"] for s in _lengths(c))
        q, lse = rows * c["hq"] * d, 4 * rows * c["hq"]
        # q, the shards' k and v, o in both precisions; then q, k, v, o, dO again, dq and the shards' dk, dv in fp32
        return {"bytes": 2 * (q + 2 * kv) + 6 * q + lse + 2 * (3 * q + 2 * kv) + lse + 4 * (q + 2 * kv), "flops": _flops(c)}
    grad = 4 if c.get("f32") else 2
    backward = 2 * (3 * q + 2 * kv) + lse + grad * (q + 2 * kv)  # q k v o dO in, dq dk dv out
    permutes = 2 * 2 * (4 * q + 4 * kv) if c["kind"] == "step" else 0  # q k v o dO dq dk dv, read and written
    return {"bytes": forward + backward + permutes, "flops": _flops(c)}


def tolerance(case):
    if case["kind"] == "permute":
        return "exact"
    # P, dS and the bf16 outputs carry one rounding to bf16 each (at most 2^-8 of the value).  Measured against the same
    # attention in fp64 on 4 099 tokens: 1.7e-3 to 2.6e-3 off in the 2-norm, and 0.07 of an output's root mean square
    # where it is off most (rows that see few keys have gradients far above the mean).
    return {"rel": 1e-2, "max": 0.25}



# ------------------------------------------------------------------------------------------------ inputs
def _normal(gen, *shape):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).to(torch.bfloat16)


def prepare(case, seed):
    c = case
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return {"case": c, "ctx": _context(), **_PREPARE[c["kind"]](c, gen)}


def _prepare_train(c, gen):
    t, hq, hkv, d = c["tokens"], c["hq"], c["hkv"], c["d"]
    cu = wl.cu_seqlens(_lengths(c))
    grad = torch.float32 if c["f32"] else torch.bfloat16
    new = lambda h, dtype: torch.empty((t, h, d), dtype=dtype, device="cuda")  # noqa: E731
    return dict(q=_normal(gen, t, hq, d), k=_normal(gen, t, hkv, d), v=_normal(gen, t, hkv, d), g=_normal(gen, t, hq, d),
                o=new(hq, torch.bfloat16), lse=torch.empty((hq, t), dtype=torch.float32, device="cuda"),
                dq=new(hq, grad), dk=new(hkv, grad), dv=new(hkv, grad), cu=torch.from_numpy(cu).cuda(),
                plan=fx.Plan(_context(), cu, hq, hkv, d, c["causal"]))


def _prepare_step(c, gen):
    t, hq, hkv, d, p = c["tokens"], c["hq"], c["hkv"], c["d"], c["p"]
    cu = wl.cu_seqlens(_lengths(c))
    sharded = lambda h: torch.empty((t // p, p * h, d), dtype=torch.bfloat16, device="cuda")  # noqa: E731
    slabs = lambda h: torch.empty((p, t // p, h, d), dtype=torch.bfloat16, device="cuda")  # noqa: E731
    s = dict(cu_host=cu, cu=torch.from_numpy(cu).cuda(), lse=torch.empty((hq, t), dtype=torch.float32, device="cuda"))
    for name, h in (("q", hq), ("k", hkv), ("v", hkv), ("g", hq)):
        s["x" + name] = _normal(gen, t // p, p * h, d)
    for name, h in (("q", hq), ("k", hkv), ("v", hkv), ("g", hq), ("o", hq), ("dq", hq), ("dk", hkv), ("dv", hkv)):
        s["s" + name] = slabs(h)
    for name, h in (("o", hq), ("dq", hq), ("dk", hkv), ("dv", hkv)):
        s["y" + name] = sharded(h)
    return s


def _prepare_infer(c, gen):
    t, hq, hkv, d = c["tokens"], c["hq"], c["hkv"], c["d"]
    return dict(q=_normal(gen, t, hq, d), k=_normal(gen, t, hkv, d), v=_normal(gen, t, hkv, d),
                o=torch.empty((t, hq, d), dtype=torch.bfloat16, device="cuda"),
                lse=torch.empty((hq, t), dtype=torch.float32, device="cuda"),
                cu=torch.from_numpy(wl.cu_seqlens(_lengths(c))).cuda())


def _prepare_ring(c, gen):
    hq, hkv, d, p = c["hq"], c["hkv"], c["d"], c["p"]
    cuts = _shard_cuts(_lengths(c), p)
    cu_q = wl.cu_seqlens([x[p] - x[p - 1] for x in cuts])
    tq = int(cu_q[-1])
    shards = []
    for j in range(p - 1, -1, -1):  # its own shard first, then the earlier ones as they come by
        cu_k = wl.cu_seqlens([x[j + 1] - x[j] for x in cuts])
        tk = int(cu_k[-1])
        shards.append(dict(plan=fx.ShardPlan(_context(), cu_q, cu_k, [x[p - 1] - x[j] for x in cuts], hq, hkv, d, c["causal"]),
                           k=_normal(gen, tk, hkv, d), v=_normal(gen, tk, hkv, d),
                           dk=torch.empty((tk, hkv, d), dtype=torch.float32, device="cuda"),
                           dv=torch.empty((tk, hkv, d), dtype=torch.float32, device="cuda")))
    return dict(shards=shards, q=_normal(gen, tq, hq, d), g=_normal(gen, tq, hq, d),
                o_acc=torch.empty((tq, hq, d), dtype=torch.float32, device="cuda"),
                o=torch.empty((tq, hq, d), dtype=torch.bfloat16, device="cuda"),
                lse=torch.empty((hq, tq), dtype=torch.float32, device="cuda"),
                dq=torch.empty((tq, hq, d), dtype=torch.float32, device="cuda"))


def _prepare_permute(c, gen):
    t, d, p = c["tokens"], c["d"], c["p"]
    dtype = {1: torch.uint8, 2: torch.bfloat16, 4: torch.float32}[c["elem"]]
    s = {}
    for name, h in (("q", c["hq"]), ("k", c["hkv"]), ("v", c["hkv"]), ("o", c["hq"])):
        packed = name == "o"  # o comes back as slabs and is regrouped by token
        wide, slab = (t, h, d), (p, t, h // p, d)
        if c["elem"] == 1:
            x = torch.randint(0, 256, slab if packed else wide, generator=gen, device="cuda", dtype=torch.uint8)
        else:
            x = torch.randn(slab if packed else wide, generator=gen, device="cuda", dtype=torch.float32).to(dtype)
        s["x" + name], s["y" + name] = x, torch.empty(wide if packed else slab, dtype=dtype, device="cuda")
    return s


_PREPARE = {"train": _prepare_train, "step": _prepare_step, "infer": _prepare_infer, "ring": _prepare_ring, "permute": _prepare_permute}


# ------------------------------------------------------------------------------------------------ one pass
def run(state):
    return _RUN[state["case"]["kind"]](state)


def _run_train(s):
    ctx, plan, causal = s["ctx"], s["plan"], s["case"]["causal"]
    fx.flexsp_attn_varlen_fwd(ctx, plan, s["q"], s["k"], s["v"], s["cu"], s["o"], s["lse"], causal=causal)
    fx.flexsp_attn_varlen_bwd(ctx, plan, s["q"], s["k"], s["v"], s["o"], s["g"], s["lse"], s["cu"], s["dq"], s["dk"], s["dv"],
                              causal=causal)
    return {n: s[n] for n in ("o", "lse", "dq", "dk", "dv")}


def _run_step(s):
    ctx, c = s["ctx"], s["case"]
    tokens = lambda x: x.view(c["tokens"], x.shape[2], c["d"])  # noqa: E731
    q, k, v, g, o, dq, dk, dv = (tokens(s["s" + n]) for n in ("q", "k", "v", "g", "o", "dq", "dk", "dv"))
    plan = fx.Plan(ctx, s["cu_host"], c["hq"], c["hkv"], c["d"], True)
    fx.flexsp_pack_many(ctx, [s["xq"], s["xk"], s["xv"]], [s["sq"], s["sk"], s["sv"]], c["p"])
    fx.flexsp_attn_varlen_fwd(ctx, plan, q, k, v, s["cu"], o, s["lse"])
    fx.flexsp_unpack(ctx, s["so"], s["yo"])
    fx.flexsp_pack(ctx, s["xg"], s["sg"], c["p"])
    fx.flexsp_attn_varlen_bwd(ctx, plan, q, k, v, o, g, s["lse"], s["cu"], dq, dk, dv)
    fx.flexsp_unpack_many(ctx, [s["sdq"], s["sdk"], s["sdv"]], [s["ydq"], s["ydk"], s["ydv"]])
    plan.close()
    return {n: s[n] for n in ("yo", "lse", "ydq", "ydk", "ydv")}


def _run_infer(s):
    fx.flexsp_attn_varlen_fwd_static(s["ctx"], s["q"], s["k"], s["v"], s["cu"], s["o"], s["lse"], causal=s["case"]["causal"])
    return {n: s[n] for n in ("o", "lse")}


def _run_ring(s):
    ctx, causal, shards = s["ctx"], s["case"]["causal"], s["shards"]
    s["lse"].fill_(float("-inf"))  # an empty running result
    for n, x in enumerate(shards):
        fx.flexsp_attn_varlen_fwd_kvshard_acc(ctx, x["plan"], s["q"], x["k"], x["v"], s["o_acc"], s["lse"],
                                              s["o"] if n == len(shards) - 1 else None, causal=causal)
    s["dq"].zero_()
    for x in shards:
        x["dk"].zero_()
        x["dv"].zero_()
        fx.flexsp_attn_varlen_bwd_kvshard(ctx, x["plan"], s["q"], x["k"], x["v"], s["o"], s["g"], s["lse"], s["dq"], x["dk"],
                                          x["dv"], causal=causal, accumulate=True)
    return {"o": s["o"], "o_acc": s["o_acc"], "lse": s["lse"], "dq": s["dq"], "dk": [x["dk"] for x in shards],
            "dv": [x["dv"] for x in shards]}


def _run_permute(s):
    fx.flexsp_pack_many(s["ctx"], [s["xq"], s["xk"], s["xv"]], [s["yq"], s["yk"], s["yv"]], s["case"]["p"])
    fx.flexsp_unpack(s["ctx"], s["xo"], s["yo"])
    return {n: s[n] for n in ("yq", "yk", "yv", "yo")}


_RUN = {"train": _run_train, "step": _run_step, "infer": _run_infer, "ring": _run_ring, "permute": _run_permute}
