"""The work that a user of this framework has it do, as measurable cases.

One process plays one rank: it holds the K and V of the whole sequence and its own query rows, and asks for its
share of the attention (forward), for the gradients of it (backward), or, where the sub-chunks of the other ranks
arrive one step at a time, for one step's partial result after the other.  The shapes are those of this repository's
own workloads and of the paper's benchmark grid (heads of dimension 64, batches of up to 128 short sequences), from
the smallest, where launches and latency count, to a sequence of a million tokens.

  op      "call"    tasp_chunk_attn: outputs and workspace allocated by the call
          "plan"    ChunkAttnPlan.run: buffers kept, as in a training or serving loop
          "static"  tasp_chunk_attn_static: nothing allocated, for callers under graph capture or in tight loops
          "bwd"     ChunkAttnBwdPlan.run
          "steps"   tasp_step_attn for every step of the schedule, each partial result folded in as it arrives
                    (fold = "pair": tasp_lse_merge) or all of them at the end (fold = "many": tasp_lse_merge_many)
  n, rank, nodes    ranks of the schedule, the rank played, nodes they are spread over (1: one node)
  S, hq, hkv, d, batch, dtype, mask ("full" or "zigzag"), order ("tasp" or "ring"), fuse_merge, fuse_steps, aux
  k_scale, outliers keys scaled (a power of two), and the share of the key rows that is eight times as large
"""
import math

import torch

from paper_2509_26541_amd import binding as tb

_BASE = {"op": "plan", "n": 8, "rank": 3, "nodes": 1, "S": 0, "hq": 8, "hkv": 8, "d": 128, "batch": 1, "dtype": "bf16",
         "mask": "zigzag", "order": "tasp", "fuse_merge": True, "fuse_steps": False, "aux": False, "fold": "pair",
         "k_scale": 1.0, "outliers": 0.0}


def _case(name=None, **kw):
    c = dict(_BASE, **kw)
    return dict({"name": name}, **c) if name else c


def listed():
    return [
        # The smallest workload of the repository, in fp32: a check of one short sequence, called as a function.
        _case("fp32 1k call", op="call", n=4, rank=0, S=1024, hq=4, hkv=4, d=64, dtype="fp32", mask="full", fuse_merge=False),
        # One short request of a grouped-query model in a tight serving loop: K and V are there, nothing is allocated.
        _case("bf16 4k static", op="static", S=4096, hq=8, hkv=2, fuse_steps=True),
        # The short end of the paper's grid: many small sequences, a launch per step as in its Algorithm 3.
        _case("grid 20x3k batch 128", S=3072, hq=20, hkv=20, d=64, batch=128),
        # The same grid further up, all steps in one launch.
        _case("grid 4x12k batch 32 fused", S=12288, hq=4, hkv=4, d=64, batch=32, fuse_steps=True),
        # Training on the grid's middle sizes: gradients of multi-head attention with heads of 64.
        _case("bwd grid 12x24k batch 8", op="bwd", S=24576, hq=12, hkv=12, d=64, batch=8),
        # Two nodes of eight ranks, a length that no tile or sub-chunk divides, merge kernel after every step (the default).
        _case("two nodes 33k ragged", n=16, nodes=2, rank=5, S=32 * 1043, hq=24, hkv=8, batch=2, fuse_merge=False),
        # What a distributed run does: every step's partial as soon as its sub-chunks are there, folded into the running pair.
        _case("steps 64k", op="steps", S=65536, rank=6, hq=16, hkv=4, mask="full"),
        # The forward pass that the repository's benchmark is quoted on.
        _case("fwd 128k", S=131072, hq=32, hkv=8),
        # And its backward pass.
        _case("bwd 128k", op="bwd", S=131072, hq=32, hkv=8),
        # fp32 in earnest: an evaluation in full precision, grouped heads of 128.
        _case("fp32 fwd 16k", n=8, rank=2, S=16384, hq=16, hkv=4, dtype="fp32"),
        # Gradients in full precision, as for a gradient check or a sensitive layer; a ragged length.
        _case("fp32 bwd 6k ragged", op="bwd", n=12, rank=7, S=24 * 257, hq=8, hkv=8, d=64, dtype="fp32"),
        # The longest workload of the repository: a million tokens, one in a hundred keys an outlier, all steps in one launch.
        _case("fwd 1M fused", rank=7, S=1048576, hq=32, hkv=8, fuse_steps=True, outliers=0.01),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above: sizes over their logarithm, lengths of no particular divisor."""
    while True:
        kind = rng.choice(["fp32", "fp32", "short", "short", "grid", "grid", "bwd", "bwd", "steps", "long"])
        nodes = 2 if rng.random() < 0.15 else 1
        n = 16 if nodes == 2 else rng.choice([4, 8, 8, 8, 12, 16])
        c = _case(n=n, nodes=nodes, rank=rng.randrange(n), mask=rng.choice(["zigzag", "zigzag", "full"]),
                  order=rng.choice(["tasp", "tasp", "tasp", "ring"]), fuse_merge=rng.random() < 0.6, fuse_steps=rng.random() < 0.4,
                  k_scale=rng.choice([1.0, 1.0, 2.0]))
        if kind == "grid" or (kind in ("bwd", "fp32") and rng.random() < 0.5):
            h = rng.choice([4, 12, 20])
            c.update(hq=h, hkv=h, d=64)
        else:
            hkv = rng.choice([1, 2, 4, 8])
            c.update(hq=hkv * rng.choice([1, 3, 4, 8]), hkv=hkv, d=128)
        if kind == "fp32":
            c.update(op=rng.choice(["call", "plan", "plan", "bwd"]), dtype="fp32")
            tokens, batch = (512, 24576), (1, 4)
            c["fuse_steps"] = c["fuse_steps"] and c["op"] != "bwd"
        elif kind == "short":
            c["op"] = rng.choice(["call", "plan", "static"])
            tokens, batch = (1024, 32768), (1, 2)
        elif kind == "grid":
            tokens, batch = (3072, 196608), (1, 128)
        elif kind == "bwd":
            c.update(op="bwd", aux=rng.random() < 0.3, k_scale=1.0)
            tokens, batch = (2048, 131072), (1, 64)
        elif kind == "steps":
            c.update(op="steps", fold=rng.choice(["pair", "many"]))
            tokens, batch = (4096, 131072), (1, 1)
        else:
            tokens, batch = (65536, 524288), (1, 2)
            c["outliers"] = rng.choice([0.0, 0.01])
        unit = 2 * n
        c["S"] = max(1, _log_int(rng, tokens[0], tokens[1]) // unit) * unit
        c["batch"] = _log_int(rng, batch[0], batch[1])
        w = work(c)
        # 32-bit sums take the chip far longer than bf16 products: bounded for themselves
        most = {"fp32 fwd": 1.2e11, "fp32 bwd": 4e10, "bf16 fwd": 3e14, "bf16 bwd": 1.2e14}[c["dtype"] + (" bwd" if c["op"] == "bwd" else " fwd")]
        elems = c["batch"] * (c["S"] // n * c["hq"] + 2 * c["S"] * c["hkv"]) * c["d"]
        small = c["op"] != "static" or c["batch"] * (c["S"] // n) * c["hq"] * c["d"] <= (6 << 20)
        if w["flops"] <= most and elems <= 1.5e9 and small:
            return c


def _mask(c):
    return tb.MASK_ZIGZAG_CAUSAL if c["mask"] == "zigzag" else tb.MASK_FULL


def _order(c):
    return tb.ORDER_RING if c["order"] == "ring" else tb.ORDER_TASP


def prepare(case, seed):
    c = dict(case)
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    dt = torch.float32 if c["dtype"] == "fp32" else torch.bfloat16
    lead = (c["batch"],) if c["batch"] > 1 else ()

    def normal(rows, heads):
        return torch.empty(lead + (rows, heads, c["d"]), dtype=dt, device=dev).normal_(generator=gen)

    q = normal(c["S"] // c["n"], c["hq"])
    k = normal(c["S"], c["hkv"])
    v = normal(c["S"], c["hkv"])
    if c["k_scale"] != 1.0:
        k *= c["k_scale"]
    if c["outliers"] > 0:
        rows = torch.randperm(c["S"], generator=gen, device=dev)[: int(c["outliers"] * c["S"])]
        k[..., rows, :, :] *= 8.0
    sched = tb.tasp_schedule_multinode(c["n"] // c["nodes"], c["nodes"], c["rank"]) if c["nodes"] > 1 else tb.tasp_schedule(c["n"], c["rank"])
    s = {"op": c["op"], "q": q, "k": k, "v": v, "schedule": sched, "mask": _mask(c), "order": _order(c), "fold": c["fold"],
         "fuse_merge": c["fuse_merge"], "fuse_steps": c["fuse_steps"]}
    if c["op"] == "plan":
        s["plan"] = tb.ChunkAttnPlan(sched, q, k, v, s["mask"], s["order"], s["fuse_merge"], 0.0, s["fuse_steps"])
    elif c["op"] == "static":
        s["out"] = torch.empty_like(q)
        s["lse"] = torch.empty(q.shape[:-1], dtype=torch.float32, device=dev)
    elif c["op"] == "bwd":
        out, lse = tb.tasp_chunk_attn(q, k, v, sched, s["mask"], s["order"], fuse_merge=True)
        dout = normal(c["S"] // c["n"], c["hq"])
        aux = torch.cuda.Stream() if c["aux"] else None
        s["plan"] = tb.ChunkAttnBwdPlan(sched, q, k, v, out, lse, dout, s["mask"], s["order"], 0.0, aux, s["fuse_steps"])
    return s


def run(s):
    op = s["op"]
    if op in ("plan", "bwd"):
        return s["plan"].run()
    if op == "call":
        return tb.tasp_chunk_attn(s["q"], s["k"], s["v"], s["schedule"], s["mask"], s["order"], s["fuse_merge"], 0.0, s["fuse_steps"])
    if op == "static":
        return tb.tasp_chunk_attn_static(s["q"], s["k"], s["v"], s["out"], s["lse"], s["schedule"], s["mask"], s["order"],
                                         s["fuse_merge"], 0.0, s["fuse_steps"])
    if s["fold"] == "many":
        parts = [tb.tasp_step_attn(s["q"], s["k"], s["v"], s["schedule"], s["mask"], i, s["order"]) for i in range(s["schedule"].n_ranks)]
        return tb.tasp_lse_merge_many([o for o, _ in parts], [l for _, l in parts])
    o, lse = tb.tasp_step_attn(s["q"], s["k"], s["v"], s["schedule"], s["mask"], 0, s["order"])
    for i in range(1, s["schedule"].n_ranks):
        o_i, lse_i = tb.tasp_step_attn(s["q"], s["k"], s["v"], s["schedule"], s["mask"], i, s["order"])
        tb.tasp_lse_merge(o, lse, o_i, lse_i)
    return o, lse


def _pairs_and_keys(c):
    """(query, key) pairs of one head of one sequence that the mask leaves, and keys that some local row sees."""
    S, n, r = c["S"], c["n"], c["rank"]
    if c["mask"] == "full":
        return S // n * S, S
    h = S // (2 * n)
    a, b = r * h, S - (r + 1) * h                        # first positions of the two half-chunks
    return h * a + h * b + h * (h + 1), b + h            # row p of a half-chunk sees p + 1 keys


def work(case):
    c = case
    size = 4 if c["dtype"] == "fp32" else 2
    rows = c["S"] // c["n"]
    pairs, keys = _pairs_and_keys(c)
    q = rows * c["hq"] * c["d"]
    kv = keys * c["hkv"] * c["d"]
    lse = rows * c["hq"] * 4
    flops = 4.0 * c["d"] * c["hq"] * pairs
    if c["op"] == "bwd":                                 # q, out, dout, k, v, lse in; dq, dk, dv out (every row of dk, dv)
        total = (4 * q + 2 * kv + 2 * c["S"] * c["hkv"] * c["d"]) * size + lse
        flops *= 2.5
    else:
        out = q * (4 if c["op"] == "steps" else size)
        total = (q + 2 * kv) * size + out + lse
    return {"bytes": float(c["batch"] * total), "flops": c["batch"] * flops}


def tolerance(case):
    # fp32: sums of a few thousand 32-bit products in another order.  bf16: products of bf16 values summed in 32 bits with
    # the probabilities rounded to bf16 on the way (relative 2^-9 at most), and the results too where they are stored so;
    # in the backward pass the probabilities' derivatives are rounded as well, behind a difference of like numbers.
    if case["dtype"] == "fp32":
        return {"rel": 1e-5, "max": 2e-4}
    if case["op"] == "bwd":
        return {"rel": 1e-2, "max": 0.1}
    return {"rel": 3e-3 if case["op"] == "steps" else 5e-3, "max": 0.05}
