"""The work an attention server does, as measurable cases.

Every case is one pass through the public entry points: `ca_forward`, `ca_forward` + `ca_backward` (a "step"), the
differentiable `AttentionServer` op (a "train" pass), key-window tasks with `ca_merge_partials` / `ca_sum_partial_dq`,
or the merge alone.  Batches have the shapes of this repository's workloads, of its profiler's latency grid and of its
shard-length experiment; documents and shards are ragged unless a workload fixes them.  Q, K, V and dO are N(0,1)
rounded to bf16, as everywhere in this repository.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2510_18121_amd import binding as B
from paper_2510_18121_amd import workloads as W
from paper_2510_18121_amd.autograd import AttentionServer

DEV = "cuda:0"


# ------------------------------------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest server call: workload 1, two short documents in four ragged shards, a small head layout
        {"name": "tiny_step", "kind": "workload", "index": 1, "div": 1, "run": "step"},
        # a small micro-batch: a few thousand tokens of packed ragged documents, 8B-class heads
        {"name": "docs_4k_step", "kind": "docs", "tokens": 4001, "median": 1024, "shard": 512, "hq": 32, "hkv": 8, "d": 128,
         "run": "step", "layout": 11},
        # training code that uses the differentiable op: 16K packed tokens, multi-head (no GQA), head_dim 64
        {"name": "mha_d64_16k_train", "kind": "docs", "tokens": 16411, "median": 2048, "shard": 0, "hq": 16, "hkv": 16, "d": 64,
         "run": "train", "layout": 12},
        # workload 2: a 64K-token chunk of documents of a median of 2K tokens, 8B-class heads
        {"name": "packed_64k_step", "kind": "workload", "index": 2, "div": 1, "run": "step"},
        # workload 3, the benchmark: 128K tokens, long and short documents in shuffled shards of 16 to 16K rows
        {"name": "composability_128k_step", "kind": "workload", "index": 3, "div": 1, "run": "step"},
        # workload 5 at a quarter of its tokens: 64/8 heads, documents of 8K to 16K and a tail of short ones
        {"name": "gqa8_64k_step", "kind": "workload", "index": 5, "div": 4, "run": "step"},
        # a point of the profiler's latency grid: a server that got one CA-task, 256 rows with a 16K context (prefill)
        {"name": "task_256x16k_fwd", "kind": "tasks", "n": 1, "q_len": 256, "kv_len": 16384, "hq": 32, "hkv": 8, "d": 128,
         "run": "fwd", "layout": 13},
        # the same with both directions, a ragged shard at the end of a 128K context
        {"name": "task_1000x128k_step", "kind": "tasks", "n": 1, "q_len": 1000, "kv_len": 130001, "hq": 32, "hkv": 8, "d": 128,
         "run": "step", "layout": 14},
        # the shard-length experiment: lone 64-token shards with contexts of up to 16K, 32K query tokens in one call
        {"name": "chunk_64_step", "kind": "chunk", "shard": 64, "context": 16384, "hq": 8, "hkv": 2, "d": 128, "run": "step",
         "layout": 0},
        # the same at 120 rows, forward only, head_dim 64
        {"name": "chunk_120_d64_fwd", "kind": "chunk", "shard": 120, "context": 16384, "hq": 8, "hkv": 2, "d": 64, "run": "fwd",
         "layout": 1},
        # a shard whose 128K context is cut into key windows: partial forward, merge, partial backward, sum of dQ
        {"name": "window_256x128k_step", "kind": "window", "q_len": 256, "kv_len": 131072, "window": 8192, "hq": 32, "hkv": 8,
         "d": 128, "layout": 15},
        # the home GPU's share of that for a whole chunk: 16K rows merged from four windows, written back for backward
        {"name": "merge_16k_x4", "kind": "merge", "rows": 16384, "parts": 4, "hq": 32, "d": 128},
    ]


HEADS = ((4, 2), (8, 1), (8, 2), (6, 2), (16, 16), (32, 8), (64, 8))


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    limit = _flops(listed()[4])
    while True:
        kind = rng.choice(("docs", "docs", "docs", "tasks", "tasks", "chunk", "window", "merge"))
        hq, hkv = rng.choice(HEADS)
        d = rng.choice((64, 128, 128))
        layout = rng.randrange(1 << 20)
        run = rng.choice(("fwd", "step", "step", "train"))
        if kind == "docs":
            c = {"kind": kind, "tokens": _log(rng, 300, 65536), "median": _log(rng, 128, 16384),
                 "shard": rng.choice((0, _log(rng, 16, 4096))), "hq": hq, "hkv": hkv, "d": d, "run": run, "layout": layout}
        elif kind == "tasks":
            kv = _log(rng, 128, 131072)
            c = {"kind": kind, "n": rng.choice((1, 1, 2, 5)), "q_len": min(kv, _log(rng, 1, 8192)), "kv_len": kv, "hq": hq,
                 "hkv": hkv, "d": d, "run": run, "layout": layout}
        elif kind == "chunk":
            c = {"kind": kind, "shard": _log(rng, 16, 2048), "context": _log(rng, 1024, 16384), "hq": hq, "hkv": hkv, "d": d,
                 "run": "fwd" if run == "fwd" else "step", "layout": layout}
        elif kind == "window":
            kv = _log(rng, 2048, 131072)
            c = {"kind": kind, "q_len": min(kv, _log(rng, 1, 2048)), "kv_len": kv, "window": max(kv // 48 + 1, _log(rng, 256, 16384)),
                 "hq": hq, "hkv": hkv, "d": d, "layout": layout}
        else:
            c = {"kind": kind, "rows": _log(rng, 64, 32768), "parts": rng.choice((2, 3, 4, 7)), "hq": hq, "d": d}
        if _flops(c) <= limit and _pair_heads(c) < 2e11:
            return c


# ------------------------------------------------------------------------------------------------ batches
def _batch(c):
    """The batch of CA-tasks of a case: it follows from the case's values alone."""
    if c["kind"] == "workload":
        return W.config(c["index"], c["div"])
    if c["kind"] == "chunk":
        return W.shard_chunk(c["shard"], "distinct", seed=c["layout"], chunk_tokens=32768 // c["shard"] * c["shard"],
                             max_context=c["context"], hq=c["hq"], hkv=c["hkv"], d=c["d"])
    rng = random.Random(c["layout"])
    if c["kind"] == "docs":  # whole ragged documents, each cut into shards of `shard` rows (0: not cut), shards shuffled
        lens, left = [], c["tokens"]
        while left > 0:
            lens.append(min(left, max(1, round(rng.lognormvariate(math.log(c["median"]), 1.0)))))
            left -= lens[-1]
        tasks = [(i, a, min(c["shard"] or n, n - a)) for i, n in enumerate(lens) for a in range(0, n, c["shard"] or n)]
    else:  # `n` tasks, each the last q_len rows of a document of its own
        n = c.get("n", 1)
        lens = [c["kv_len"]] * n
        tasks = [(i, c["kv_len"] - c["q_len"], c["q_len"]) for i in range(n)]
    order = list(range(len(tasks)))
    rng.shuffle(order)
    return W.custom(lens, tasks, c["hq"], c["hkv"], c["d"], task_order=order)


def _pairs(b):
    return sum(n * (2 * a + n + 1) // 2 for a, n in zip(b.task_q_pos.tolist(), b.task_q_len.tolist()))


def _pair_heads(c):
    if c["kind"] == "merge":
        return 0
    b = _batch(c)
    return _pairs(b) * b.n_q_heads


def _flops(c):
    if c["kind"] == "merge":
        return 2 * c["rows"] * c["parts"] * c["hq"] * c["d"]
    b = _batch(c)
    return (4 if c.get("run") == "fwd" else 14) * b.head_dim * b.n_q_heads * _pairs(b)


# ------------------------------------------------------------------------------------------------ prepare and run
def _normal(gen, *shape):
    out = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
    flat = out.view(-1)
    for i in range(0, flat.numel(), 1 << 26):  # in pieces, so that the fp32 staging stays small
        m = min(1 << 26, flat.numel() - i)
        flat[i:i + m] = torch.randn(m, generator=gen, device=DEV)
    return out


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(seed)


def _inputs(c, seed):
    b, g = _batch(c), _gen(seed)
    q, k, v = (_normal(g, n, h, b.head_dim) for n, h in ((b.total_q, b.n_q_heads), (b.total_kv, b.n_kv_heads), (b.total_kv, b.n_kv_heads)))
    return b, q, k, v, (None if c.get("run") == "fwd" else _normal(g, b.total_q, b.n_q_heads, b.head_dim))


def _merge_inputs(c, seed):
    g = _gen(seed)
    n, p, h, d = c["rows"], c["parts"], c["hq"], c["d"]
    o = _normal(g, n * p, h, d)
    # log-sum-exps of windows of unlike length: around ln(keys), a unit apart
    lse = 8.0 + torch.randn(h, n * p, generator=g, device=DEV)
    # as split_kv lays them out: a window's partial rows are one run, and early rows have no part in the last windows
    rows = torch.arange(n * p, device=DEV, dtype=torch.int32).view(p, n)
    rows[p - 1, :n // 4] = -1
    return rows, o, lse


def prepare(c, seed):
    if c["kind"] == "merge":
        rows, o_part, lse_part = _merge_inputs(c, seed)
        n, h, d = c["rows"], c["hq"], c["d"]
        return {"case": c, "rows": rows, "o_part": o_part, "lse_part": lse_part,
                "o": torch.empty(n, h, d, dtype=torch.bfloat16, device=DEV), "lse": torch.empty(h, n, device=DEV),
                "o_back": torch.zeros_like(o_part), "lse_back": torch.zeros_like(lse_part)}
    b, q, k, v, do = _inputs(c, seed)
    s = {"case": c, "k": k, "v": v}
    if c.get("run") == "train":
        s["server"] = AttentionServer(b, DEV)
        s["q"], s["k"], s["v"], s["do"] = q.requires_grad_(), k.requires_grad_(), v.requires_grad_(), do
        return s
    if c["kind"] == "window":
        pb, gather, part_rows = W.split_kv(b, c["window"])
        at = torch.as_tensor(gather, device=DEV)
        s["rows"] = torch.as_tensor(part_rows, device=DEV).contiguous()
        s["o"], s["dq"] = torch.empty_like(q), torch.empty_like(q)
        s["lse"] = torch.empty(b.n_q_heads, b.total_q, device=DEV)
        q, do, b = q.index_select(0, at), do.index_select(0, at), pb
    s["plan"] = B.ca_plan(b)
    s["ws"] = B.alloc_workspace(s["plan"], DEV)
    s["q"], s["do"], s["o_q"] = q, do, torch.empty_like(q)
    s["lse_q"] = torch.empty(b.n_q_heads, b.total_q, device=DEV)
    if do is not None:
        s["dq_q"], s["dk"], s["dv"] = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)
    return s


def run(s):
    c = s["case"]
    if c["kind"] == "merge":
        B.ca_merge_partials(s["rows"], s["o_part"], s["lse_part"], s["o"], s["lse"], s["o_back"], s["lse_back"])
        return {n: s[n] for n in ("o", "lse", "o_back", "lse_back")}
    if c.get("run") == "train":
        o = s["server"](s["q"], s["k"], s["v"])
        dq, dk, dv = torch.autograd.grad(o, (s["q"], s["k"], s["v"]), s["do"])
        return {"o": o, "dq": dq, "dk": dk, "dv": dv}
    B.ca_forward(s["plan"], s["q"], s["k"], s["v"], s["o_q"], s["lse_q"], s["ws"])
    if c["kind"] == "window":
        B.ca_merge_partials(s["rows"], s["o_q"], s["lse_q"], s["o"], s["lse"], s["o_q"], s["lse_q"])
    if c.get("run") == "fwd":
        return {"o": s["o_q"], "lse": s["lse_q"]}
    B.ca_backward(s["plan"], s["q"], s["k"], s["v"], s["o_q"], s["do"], s["lse_q"], s["dq_q"], s["dk"], s["dv"], s["ws"])
    if c["kind"] == "window":
        B.ca_sum_partial_dq(s["rows"], s["dq_q"], s["dq"])
        return {n: s[n] for n in ("o", "lse", "dq", "dk", "dv")}
    return {"o": s["o_q"], "lse": s["lse_q"], "dq": s["dq_q"], "dk": s["dk"], "dv": s["dv"]}


# ------------------------------------------------------------------------------------------------ what is asked of them
def work(c):
    if c["kind"] == "merge":  # partial rows in, merged rows out and back into every partial row
        row = c["hq"] * (2 * c["d"] + 4)
        return {"bytes": c["rows"] * (row * (2 * c["parts"] + 1) + 4 * c["parts"]), "flops": _flops(c)}
    b = _batch(c)
    qb, kb, lb = 2 * b.total_q * b.n_q_heads * b.head_dim, 2 * b.total_kv * b.n_kv_heads * b.head_dim, 4 * b.n_q_heads * b.total_q
    # forward: Q, K, V in, O and LSE out; with backward also dO in, dQ, dK, dV out
    return {"bytes": 2 * qb + 2 * kb + lb if c.get("run") == "fwd" else 4 * qb + 4 * kb + lb, "flops": _flops(c)}


def tolerance(c):
    # bf16 results of bf16 inputs.  Against 64 bits the attention outputs are off by 2.2e-3 to 2.9e-3 and the merged
    # ones by 1.7e-3 (2-norm); the largest single difference is in gradients of the first rows of a document, where O, a
    # bf16 input of backward, is as large as a single V row.
    return {"rel": 7e-3, "max": 0.1} if c["kind"] == "merge" else {"rel": 1e-2, "max": 0.4}


def exact(c, seed):
    if c["kind"] == "merge":
        return _exact_merge(c, seed)
    if _pair_heads(c) > 2e11:
        return None
    b, q, k, v, do = _inputs(c, seed)
    f64 = torch.float64
    hq, hkv, d, g = b.n_q_heads, b.n_kv_heads, b.head_dim, b.n_q_heads // b.n_kv_heads
    scale = 1.0 / math.sqrt(d)
    o = torch.zeros(q.shape, dtype=f64, device=DEV)
    lse = torch.zeros(hq, b.total_q, dtype=f64, device=DEV)
    dq = torch.zeros_like(o) if do is not None else None
    dk, dv = (torch.zeros(k.shape, dtype=f64, device=DEV) for _ in range(2)) if do is not None else (None, None)
    for t in range(b.n_tasks):
        doc, q0, n, pos = (int(x[t]) for x in (b.task_doc, b.task_q_start, b.task_q_len, b.task_q_pos))
        kv0 = int(b.doc_kv_start[doc])
        step = max(1, (1 << 26) // (g * (pos + n)))
        for a in range(0, n, step):  # rows [a, e) of the task see keys [0, pos + e)
            e = min(n, a + step)
            rows, keys = slice(q0 + a, q0 + e), slice(kv0, kv0 + pos + e)
            hidden = torch.arange(pos + e, device=DEV)[None, :] > pos + torch.arange(a, e, device=DEV)[:, None]
            for h in range(hkv):
                heads = slice(h * g, (h + 1) * g)
                # the g query heads of a group stacked: [g (e - a), d]
                qt, kt, vt = q[rows, heads].to(f64).transpose(0, 1).reshape(-1, d), k[keys, h].to(f64), v[keys, h].to(f64)
                p = (qt @ kt.t()).mul_(scale)
                p.view(g, e - a, -1).masked_fill_(hidden, -math.inf)
                m = p.amax(1, keepdim=True)
                p.sub_(m).exp_()
                total = p.sum(1, keepdim=True)
                p.div_(total)
                ot = p @ vt
                o[rows, heads] = ot.view(g, e - a, d).transpose(0, 1)
                lse[heads, rows] = (m + total.log()).view(g, e - a)
                if do is not None:
                    dt = do[rows, heads].to(f64).transpose(0, 1).reshape(-1, d)
                    dv[keys, h] += p.t() @ dt
                    ds = (dt @ vt.t()).sub_((dt * ot).sum(1, keepdim=True)).mul_(p)
                    dq[rows, heads] = (ds @ kt).mul_(scale).view(g, e - a, d).transpose(0, 1)
                    dk[keys, h] += (ds.t() @ qt).mul_(scale)
    if do is None:
        return {"o": o, "lse": lse}
    if c.get("run") == "train":
        return {"o": o, "dq": dq, "dk": dk, "dv": dv}
    return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}


def _exact_merge(c, seed):
    rows, o_part, lse_part = _merge_inputs(c, seed)
    n, h, d = c["rows"], c["hq"], c["d"]
    at, has = rows.clamp(min=0).long(), rows >= 0
    o, lse = torch.zeros(n, h, d, dtype=torch.float64, device=DEV), torch.zeros(h, n, dtype=torch.float64, device=DEV)
    o_back, lse_back = torch.zeros(o_part.shape, dtype=torch.float64, device=DEV), torch.zeros(lse_part.shape, dtype=torch.float64, device=DEV)
    for i in range(h):
        part = lse_part[i].double()[at].masked_fill(~has, -math.inf)
        lse[i] = torch.logsumexp(part, 0)
        o[:, i] = ((part - lse[i]).exp()[:, :, None] * o_part[:, i].double()[at]).sum(0)
    for p in range(c["parts"]):
        o_back[at[p][has[p]]] = o[has[p]]
        lse_back[:, at[p][has[p]]] = lse[:, has[p]]
    return {"o": o, "lse": lse, "o_back": o_back, "lse_back": lse_back}
