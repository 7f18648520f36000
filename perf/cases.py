"""The work that users of the paged-attention library have it do, as measurable cases.

A serving instance runs phase-pure batches: prefill-only batches (append the prompts' K/V, then causal attention over
the paged cache) and decode-only steps (append one token per sequence, then attention over the whole context), layer
after layer of a model.  A case is one such step over a few layers, every layer with its own cache.  Head shapes and
length distributions are those of paper_2504_18154_amd/workloads.py, of the tests and of bench.py, or generic ones
(one K/V head per GPU under tensor parallelism, head size 64, a chunk of a prompt behind a long cached prefix).

Lengths follow from the case (`len_seed`), everything else - block tables, K/V, queries - from prepare()'s seed.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2504_18154_amd import binding
from paper_2504_18154_amd import workloads as wl

BS = wl.BLOCK_SIZE


def _decode(name, heads, B, lo, hi, layers, *, D=128, dtype="bf16", mean=0.0, entry="append", lse=False, adaptive=False,
            graph=False, len_seed=1):
    """A decode-only step.  Context lengths (with the new token) are uniform in [lo, hi], or lognormal around `mean` and
    clipped to [lo, hi].  entry: "append" the fused append + attention call, "separate" the two calls, "noalloc" the
    append and the call that needs no context.  graph: the step's launches are recorded once and replayed."""
    return {"name": name, "kind": "decode", "Hq": heads[0], "Hkv": heads[1], "D": D, "dtype": dtype, "B": B, "lo": lo, "hi": hi,
            "mean": float(mean), "layers": layers, "entry": entry, "lse": lse, "adaptive": adaptive, "graph": graph,
            "len_seed": len_seed}


def _prefill(name, heads, B, lo, hi, layers, *, D=128, dtype="bf16", mean=0.0, pre_lo=0, pre_hi=0, fused_rows=False, lse=False,
             len_seed=1):
    """A prefill-only step: B prompts (or chunks of prompts) of lo..hi new tokens behind pre_lo..pre_hi cached ones.
    fused_rows: Q, K and V are slices of one projection output row per token."""
    return {"name": name, "kind": "prefill", "Hq": heads[0], "Hkv": heads[1], "D": D, "dtype": dtype, "B": B, "lo": lo, "hi": hi,
            "mean": float(mean), "pre_lo": pre_lo, "pre_hi": pre_hi, "layers": layers, "fused_rows": fused_rows, "lse": lse,
            "len_seed": len_seed}


def _cycle(name, heads, B, lo, hi, steps, *, D, dtype, len_seed=1):
    """A prefill-only batch and `steps` decode-only steps after it, one layer."""
    return {"name": name, "kind": "cycle", "Hq": heads[0], "Hkv": heads[1], "D": D, "dtype": dtype, "B": B, "lo": lo, "hi": hi,
            "mean": 0.0, "steps": steps, "len_seed": len_seed}


def listed():
    return [
        # one user at a time: an interactive session of ~800 tokens; latency and the number of launches are everything
        _decode("decode_one", (40, 8), 1, 777, 777, 16),
        # a lightly loaded chat server (the lengths of the ShareGPT row of the paper's Table 4), its step recorded as a graph
        # with the call that needs no context
        _decode("decode_chat_graph", (64, 8), 16, 20, 2000, 16, mean=460.0, entry="noalloc", graph=True),
        # many short conversations at once: contexts of ~100 tokens (the Alpaca row of Table 4), ragged last blocks
        _decode("decode_short_many", (40, 8), 1024, 2, 800, 2, mean=103.0),
        # the benchmark's decode batch: 128 sequences of 512..4096 tokens, shares that follow the XCDs as bench.py has them
        _decode("decode_30b", (40, 8), 128, 512, 4096, 2, adaptive=True, len_seed=2),
        # the largest decode batch of the benchmark (70B-scale heads)
        _decode("decode_70b", (64, 8), 256, 1024, 4096, 1, len_seed=4),
        # multi-head attention without K/V sharing (the paper's third model), append as a call of its own, log-sum-exp wanted
        _decode("decode_mha", (52, 52), 24, 300, 3000, 2, entry="separate", lse=True, len_seed=3),
        # a single short prompt: time to first token of an idle instance
        _prefill("prefill_one", (40, 8), 1, 93, 93, 16),
        # the benchmark's prefill batch: 16 prompts, lognormal around 1024 tokens, 128..4096
        _prefill("prefill_30b", (40, 8), 16, 128, 4096, 2, mean=1024.0, len_seed=3),
        # the benchmark's prefill burst: 8 prompts of 8192 tokens (70B-scale heads), the largest case
        _prefill("prefill_burst", (64, 8), 8, 8192, 8192, 1),
        # chunked prefill: a step's budget of about 512 new tokens, taken from two long prompts behind what earlier chunks left
        # in the cache, read in place from the projection's output rows
        _prefill("prefill_chunk", (64, 8), 2, 150, 400, 4, pre_lo=3000, pre_hi=12000, fused_rows=True, len_seed=5),
        # the fp32 model of the benchmark's tiny configuration (checks against a reference in full precision)
        _cycle("cycle_f32", (4, 2), 4, 37, 700, 8, D=64, dtype="f32"),
        # a small model with head size 64 in bf16
        _cycle("cycle_d64", (32, 8), 4, 50, 600, 8, D=64, dtype="bf16"),
    ]


_HEADS = ((40, 8), (64, 8), (52, 52), (8, 1), (32, 8), (5, 1))


def _log(rng: random.Random, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    kind = rng.choice(("decode", "decode", "prefill", "prefill", "cycle"))
    ls = rng.randrange(1, 1 << 30)
    if kind == "decode":
        heads = rng.choice(_HEADS)
        B = _log(rng, 1, 1024)
        # at most 2.7 GB of K/V in a layer, as in the largest listed case
        cap = max(64, min(16384, int(2.7e9 / (512 * heads[1] * B))))
        hi = _log(rng, 32, cap)
        lo = max(1, hi // rng.choice((1, 2, 8, 64)))
        mean = float((lo + hi) // 3) if rng.random() < 0.4 else 0.0
        kv = 512 * heads[1] * B * (mean or (lo + hi) / 2)
        layers = 1 if kv > 1e9 else 2 if kv > 1e8 else 8
        entry = rng.choice(("append", "append", "separate", "noalloc"))
        c = _decode("", heads, B, lo, hi, layers, mean=mean, entry=entry, lse=rng.random() < 0.3,
                    adaptive=entry == "append" and rng.random() < 0.3, graph=entry == "noalloc", len_seed=ls)
    elif kind == "prefill":
        heads = rng.choice(_HEADS)
        B = _log(rng, 1, 512)
        hi = _log(rng, 16, max(32, min(8192, 40000 // B)))
        lo = max(1, hi // rng.choice((1, 2, 8, 32)))
        mean = float((lo + hi) // 3) if rng.random() < 0.4 else 0.0
        pre = (0, 0)
        if rng.random() < 0.5:
            pre_hi = _log(rng, 16, max(32, min(16384, 800000 // (B * heads[1]))))
            pre = (rng.choice((0, pre_hi // 2, pre_hi)), pre_hi)
        # the rows times what they see, kept to an eighth of the largest listed case's products
        while 4.0 * heads[0] * 128 * B * hi * (pre[1] + hi / 2) > 1.1e12:
            B, hi = max(1, B // 2), max(16, hi * 3 // 4)
            lo = min(lo, hi)
        mean = min(mean, float(hi))
        small = B * hi * heads[0] < 200000 and B * (hi + pre[1]) * heads[1] < 200000
        c = _prefill("", heads, B, lo, hi, 8 if small else 2, mean=mean, pre_lo=pre[0], pre_hi=pre[1],
                     fused_rows=rng.random() < 0.4, lse=rng.random() < 0.3, len_seed=ls)
    else:
        dtype, D, heads = rng.choice((("f32", 64, (4, 2)), ("f32", 128, (6, 3)), ("bf16", 64, (32, 8)), ("bf16", 80, (8, 8)),
                                      ("bf16", 96, (8, 2)), ("bf16", 256, (8, 1))))
        hi = _log(rng, 16, 800)
        B = max(1, min(_log(rng, 1, 64), int(4.0e7 / (heads[0] * D * hi))))
        c = _cycle("", heads, B, max(1, hi // rng.choice((1, 4, 16))), hi, rng.randrange(1, 9), D=D, dtype=dtype, len_seed=ls)
    del c["name"]
    return c


# ---- lengths and accounting ---------------------------------------------------------------------


def _lengths(c):
    """Per sequence: (tokens cached before the step, new tokens), int64 arrays."""
    rng = wl.rng_for(c["len_seed"])
    n = (wl.lengths_lognormal(rng, c["B"], c["mean"], 1.0, c["lo"], c["hi"]) if c["mean"]
         else wl.lengths_uniform(rng, c["B"], c["lo"], c["hi"])).astype(np.int64)
    if c["kind"] == "decode":
        return n - 1, np.ones_like(n)
    if c["kind"] == "prefill":
        return wl.lengths_uniform(rng, c["B"], c["pre_lo"], c["pre_hi"]).astype(np.int64), n
    return np.zeros_like(n), n


def _step_work(c, before, new, lse):
    """Bytes and FLOPs one layer of one step cannot do without: the cached K/V and the new rows read once, the new rows
    written into the cache once, queries read, outputs written; both products under the causal mask."""
    es = 2 if c["dtype"] == "bf16" else 4
    row = c["Hkv"] * c["D"] * es
    total = before + new
    kv = 2 * row * int(total.sum()) + 2 * row * int(new.sum())
    qo = 2 * c["Hq"] * c["D"] * es * int(new.sum()) + (4 * c["Hq"] * int(new.sum()) if lse else 0)
    meta = 4 * int(((total + BS - 1) // BS).sum()) + 8 * len(new)
    return kv + qo + meta, 4 * c["Hq"] * c["D"] * int((new * before + new * (new + 1) // 2).sum())


def work(case):
    before, new = _lengths(case)
    if case["kind"] != "cycle":
        b, f = _step_work(case, before, new, case["lse"])
        return {"bytes": b * case["layers"], "flops": f * case["layers"]}
    b, f = _step_work(case, before, new, False)
    for s in range(case["steps"]):
        sb, sf = _step_work(case, new + s, np.ones_like(new), False)
        b, f = b + sb, f + sf
    return {"bytes": b, "flops": f}


def tolerance(case):
    # four times the relative 2-norm measured against an fp64 evaluation of the same inputs: bf16 outputs 1.6e-3 to 2.4e-3 (their own
    # rounding and that of the weights), fp32 outputs 2.2e-7
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-6}


# ---- a user's program ---------------------------------------------------------------------------


def _randn(shape, dtype, gen):
    """N(0, 1) on the GPU in the storage type, drawn in pieces so that a pool of gigabytes needs no fp32 copy of itself."""
    t = torch.empty(shape, dtype=torch.bfloat16 if dtype == "bf16" else torch.float32, device="cuda")
    flat = t.view(-1)
    for o in range(0, flat.numel(), 1 << 28):
        n = min(1 << 28, flat.numel() - o)
        flat[o:o + n] = torch.randn(n, generator=gen, device="cuda", dtype=torch.float32)
    return t


def _i32(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.int32), device="cuda")


def prepare(case, seed):
    c = dict(case)
    before, new = _lengths(c)
    B, Hq, Hkv, D = c["B"], c["Hq"], c["Hkv"], c["D"]
    layers, steps = c.get("layers", 1), c.get("steps", 0)
    rng, gen = wl.rng_for(seed), torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    table, num_blocks = wl.make_block_table(rng, before + new + steps)
    ctx = binding.Context(Hq, Hkv, D, num_blocks, c["dtype"], B, table.shape[1])
    if c.get("adaptive"):
        ctx.set_option(binding.OPT_DECODE_ADAPTIVE, 1)
    T = int(new.sum())
    n = num_blocks * Hkv * BS * D
    s = {"case": c, "ctx": ctx, "bt": _i32(table), "before": _i32(before),
         "cu": _i32(wl.cu_from_lengths(new)), "total": _i32(before + new), "max_new": int(new.max()), "max_total": int((before + new).max()),
         "k": _randn((layers, n), c["dtype"], gen), "v": _randn((layers, n), c["dtype"], gen),
         "out": torch.zeros((layers, T, Hq, D), dtype=ctx.torch_dtype, device="cuda"),
         "lse": torch.zeros((layers, T, Hq), dtype=torch.float32, device="cuda") if c.get("lse") else None}
    if c.get("fused_rows"):
        rows = _randn((layers, T, Hq + 2 * Hkv, D), c["dtype"], gen)
        q, kn, vn = rows[:, :, :Hq], rows[:, :, Hq:Hq + Hkv], rows[:, :, Hq + Hkv:]
    else:
        q, kn, vn = (_randn((layers, T, h, D), c["dtype"], gen) for h in (Hq, Hkv, Hkv))
    # each layer's tensors, as a model's layers hold them
    s["layers"] = list(zip(*((t.unbind(0) if t is not None else (None,) * layers)
                             for t in (q, kn, vn, s["k"], s["v"], s["out"], s["lse"]))))
    if c["kind"] == "cycle":
        s["steps"] = [{"q": _randn((B, Hq, D), c["dtype"], gen), "kn": _randn((B, Hkv, D), c["dtype"], gen),
                       "vn": _randn((B, Hkv, D), c["dtype"], gen), "total": _i32(new + i + 1), "max_total": int(new.max()) + i + 1,
                       "out": torch.zeros((B, Hq, D), dtype=ctx.torch_dtype, device="cuda")} for i in range(steps)]
    if c.get("graph"):
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            _decode_step(s)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        s["graph"] = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s["graph"]):
            _decode_step(s)
    return s


def _decode_step(s):
    ctx, entry = s["ctx"], s["case"]["entry"]
    for q, kn, vn, k, v, out, lse in s["layers"]:
        if entry == "append":
            ctx.attn_decode_append(q, kn, vn, k, v, s["bt"], s["total"], out, s["max_total"], lse)
            continue
        ctx.kv_append(k, v, kn, vn, s["cu"], s["before"], s["bt"], max_new_len=1)
        if entry == "separate":
            ctx.attn_decode(q, k, v, s["bt"], s["total"], out, s["max_total"], lse)
        else:
            status = binding.attn_decode_noalloc(ctx.layout, q, k, v, s["bt"], s["total"], out, s["max_total"], lse)
            if status != binding.OK:
                raise RuntimeError(binding.strerror(status))


def _prefill_step(s):
    ctx, fused = s["ctx"], s["case"].get("fused_rows")
    append, attend = (ctx.kv_append_strided, ctx.attn_prefill_strided) if fused else (ctx.kv_append, ctx.attn_prefill)
    ctx.set_option(binding.OPT_PREFILL_REUSE_PLAN, 1)  # the layers of this step share their list of query tiles
    for q, kn, vn, k, v, out, lse in s["layers"]:
        append(k, v, kn, vn, s["cu"], s["before"], s["bt"], max_new_len=s["max_new"])
        attend(q, k, v, s["cu"], s["before"], s["bt"], out, lse, max_q_len=s["max_new"])


def run(state):
    kind = state["case"]["kind"]
    if kind == "decode":
        if "graph" in state:
            state["graph"].replay()
        else:
            _decode_step(state)
    else:
        _prefill_step(state)
    got = {"out": state["out"], "lse": state["lse"], "k": state["k"], "v": state["v"]}
    if kind == "cycle":
        ctx = state["ctx"]
        for t in state["steps"]:
            _, _, _, k, v, _, _ = state["layers"][0]
            ctx.attn_decode_append(t["q"], t["kn"], t["vn"], k, v, state["bt"], t["total"], t["out"], t["max_total"])
        got["steps"] = [t["out"] for t in state["steps"]]
    return got


# ---- the same in 64 bits ------------------------------------------------------------------------


def _cached(pool, c, blocks, n, is_k):
    """The first n cached tokens of a sequence as fp64 [Hkv, n, D], taken out of a pool's blocks."""
    Hkv, D, x = c["Hkv"], c["D"], 8 if c["dtype"] == "bf16" else 4
    if is_k:
        t = pool.view(-1, Hkv, D // x, BS, x)[blocks].permute(1, 0, 3, 2, 4)
    else:
        t = pool.view(-1, Hkv, D, BS)[blocks].permute(1, 0, 3, 2)
    return t.reshape(Hkv, -1, D)[:, :n].double()


def _attend(c, q, k, v):
    """fp64 (out, log-sum-exp) of the last len(q) positions of k/v [Hkv, n, D], each seeing itself and what precedes it."""
    S, (Hkv, n, D) = q.shape[0], k.shape
    G = c["Hq"] // Hkv
    kt = k.transpose(1, 2).contiguous()
    out = torch.empty((S, c["Hq"], D), dtype=torch.float64, device="cuda")
    lse = torch.empty((S, c["Hq"]), dtype=torch.float64, device="cuda")
    step = max(1, min(S, int(1.2e8 / (c["Hq"] * n))))
    for r in range(0, S, step):
        e = min(S, r + step)
        seen = n - S + e  # keys that the last row of this piece sees
        qs = q[r:e].double().view(e - r, Hkv, G, D).permute(1, 2, 0, 3).reshape(Hkv, G * (e - r), D)
        s = torch.bmm(qs, kt[:, :, :seen].contiguous()).view(Hkv, G, e - r, seen) / math.sqrt(D)
        if S > 1:
            pos = torch.arange(n - S + r, seen, device="cuda")
            s.masked_fill_(torch.arange(seen, device="cuda") > pos[:, None], -math.inf)
        z = torch.logsumexp(s, -1)
        p = s.sub_(z[..., None]).exp_().view(Hkv, G * (e - r), seen)
        o = torch.bmm(p, v[:, :seen].contiguous()).view(Hkv, G, e - r, D)
        out[r:e] = o.permute(2, 0, 1, 3).reshape(e - r, c["Hq"], D)
        lse[r:e] = z.permute(2, 0, 1).reshape(e - r, c["Hq"])
    return out, lse


def exact(case, seed):
    c = dict(case)
    s = prepare(case, seed)
    before, new = _lengths(c)
    cu, bt = np.concatenate(([0], np.cumsum(new))), s["bt"].long()
    outs, lses, steps = [], [], [torch.empty(t["out"].shape, dtype=torch.float64, device="cuda") for t in s.get("steps", ())]
    for q, kn, vn, kp, vp, _, _ in s["layers"]:
        rows = []
        for b in range(c["B"]):
            a, e, n = int(cu[b]), int(cu[b + 1]), int(before[b])
            k, v = (x[a:e].double().transpose(0, 1) for x in (kn, vn))
            if n:
                blocks = bt[b, :(n + BS - 1) // BS]
                k = torch.cat((_cached(kp, c, blocks, n, True), k), 1)
                v = torch.cat((_cached(vp, c, blocks, n, False), v), 1)
            rows.append(_attend(c, q[a:e], k, v))
            for i, t in enumerate(s.get("steps", ())):
                k = torch.cat((k, t["kn"][b:b + 1].double().transpose(0, 1)), 1)
                v = torch.cat((v, t["vn"][b:b + 1].double().transpose(0, 1)), 1)
                steps[i][b:b + 1] = _attend(c, t["q"][b:b + 1], k, v)[0]
        outs.append(torch.cat([o for o, _ in rows]))
        lses.append(torch.cat([z for _, z in rows]))
    # the pools hold copies of the inputs: no computed numbers
    got = {"out": torch.stack(outs), "lse": torch.stack(lses) if c.get("lse") else None, "k": None, "v": None}
    if c["kind"] == "cycle":
        got["steps"] = steps
    return got
