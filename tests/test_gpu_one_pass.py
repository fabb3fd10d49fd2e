"""The backward in one pass against whole units in the other kernels, which the oracle checks: the same sums in the same order, so the
same bits; whatever the workspace held, on two streams at once, and from a graph."""
import pytest
import torch

from one_pass_batches import BATCHES
from paper_2510_18121_amd import binding as B
from paper_2510_18121_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _setup(name):
    b = BATCHES[name]()
    q, k, v, d_o = W.make_tensors(b, DEV)
    p = B.ca_plan(b)
    o, lse = torch.zeros_like(q), torch.zeros(b.n_q_heads, b.total_q, device=DEV)
    B.ca_forward(p, q, k, v, o, lse)
    one, base = p.workspace_bytes_one_pass(), p.workspace_bytes()[1]
    assert one > base

    def run(n_bytes, fill, out=None):
        ws = torch.full((n_bytes,), fill, dtype=torch.uint8, device=DEV)
        out = out or [torch.full_like(x, 7.0) for x in (q, k, v)]
        B.ca_backward(p, q, k, v, o, d_o, lse, *out, ws)
        return out, ws
    return b, p, (q, k, v, d_o), o, lse, one, base, run


@pytest.mark.parametrize("name", sorted(BATCHES))
def test_same_bits_as_whole_units(name):
    *_, one, base, run = _setup(name)
    whole = run(base, 0)[0]
    for fill in (0, 0xFF, 0x3F):
        for got, want in zip(run(one, fill)[0], whole):
            assert torch.equal(got, want)


def test_sum_identities():
    """For every document and KV head: sum of dV = sum of dO, sum of dK = 0 (size independent rounding: 2e-2 of the norm)."""
    b, p, (q, k, v, d_o), o, lse, one, base, run = _setup("gaps_and_keys_nobody_sees")
    dq, dk, dv = run(one, 0)[0]
    row_doc = torch.full((b.total_q,), -1, device=DEV)
    for t in range(b.n_tasks):
        row_doc[b.task_q_start[t]:b.task_q_start[t] + b.task_q_len[t]] = int(b.task_doc[t])
    g = b.n_q_heads // b.n_kv_heads
    for d in sorted(set(b.task_doc.tolist())):
        keys = slice(int(b.doc_kv_start[d]), int(b.doc_kv_start[d] + b.doc_kv_len[d]))
        want = d_o[row_doc == d].float().view(-1, b.n_kv_heads, g, b.head_dim).sum((0, 2))
        assert (dv[keys].float().sum(0) - want).norm() <= 2e-2 * max(1.0, float(dv[keys].float().norm()))
        assert dk[keys].float().sum(0).norm() <= 2e-2 * max(1.0, float(dk[keys].float().norm()))


def test_two_streams_and_a_graph():
    b, p, (q, k, v, d_o), o, lse, one, base, run = _setup("documents")
    want, _ = run(one, 0)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    outs = [[torch.zeros_like(x) for x in (q, k, v)] for _ in range(2)]
    spaces = [torch.zeros(one, dtype=torch.uint8, device=DEV) for _ in range(2)]
    torch.cuda.synchronize()
    for _ in range(2):
        for s, out, ws in zip(streams, outs, spaces):
            B.ca_backward(p, q, k, v, o, d_o, lse, *out, ws, stream=s)
    torch.cuda.synchronize()
    for out in outs:
        assert all(torch.equal(x, y) for x, y in zip(out, want))
    out, ws = [torch.zeros_like(x) for x in (q, k, v)], spaces[0]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        B.ca_backward(p, q, k, v, o, d_o, lse, *out, ws)
    for _ in range(3):
        for x in out:
            x.zero_()
        ws.fill_(0x5A)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(out, want))


def test_timing_and_smaller_workspaces():
    b, p, (q, k, v, d_o), o, lse, one, base, run = _setup("documents")
    want, _ = run(one, 0)
    p.profile_enable(True)
    timed, _ = run(one, 0)
    t = p.profile_read()
    p.profile_enable(False)
    assert t["bwd_dkv_ms"] > 0 and t["bwd_dq_ms"] < t["bwd_dkv_ms"] / 10
    assert all(torch.equal(x, y) for x, y in zip(timed, want))
    less, _ = run(one - 1, 0)  # the lists of units, cut or whole
    for x, y in zip(less, want):
        assert (x.float() - y.float()).norm() <= 1e-2 * y.float().norm()
    assert B.alloc_workspace(p, DEV).numel() >= one


def _poisoned(b, x, rows, value):
    x = x.clone()
    x[rows] = value
    return x


def _backward(p, q, k, v, o, d_o, lse, n_bytes):
    out = [torch.full_like(x, 7.0) for x in (q, k, v)]
    B.ca_backward(p, q, k, v, o, d_o, lse, *out, torch.full((n_bytes,), 0x5A, dtype=torch.uint8, device=DEV))
    return out


@pytest.mark.parametrize("name", ["gaps_and_keys_nobody_sees", "shards_d64"])
def test_keys_that_nobody_sees_may_hold_anything(name):
    """NaN or Inf in K and V behind a document's last query: every gradient as with finite values there, zero for those keys."""
    b, p, (q, k, v, d_o), o, lse, one, base, run = _setup(name)
    if name == "shards_d64":  # (this batch has no such keys: the same queries without the last rows of each document)
        n = b.task_q_len.copy()
        n[n > 40] -= 37
        b = W.custom(b.doc_kv_len.tolist(), list(zip(b.task_doc.tolist(), b.task_q_pos.tolist(), n.tolist())), b.n_q_heads, b.n_kv_heads, b.head_dim)
        q, k, v, d_o = W.make_tensors(b, DEV)
        p = B.ca_plan(b)
        o, lse = torch.zeros_like(q), torch.zeros(b.n_q_heads, b.total_q, device=DEV)
        B.ca_forward(p, q, k, v, o, lse)
        one = p.workspace_bytes_one_pass()
        assert one > 0
    unseen = torch.ones(b.total_kv, dtype=torch.bool, device=DEV)
    for t in range(b.n_tasks):
        at = int(b.doc_kv_start[b.task_doc[t]])
        unseen[at:at + int(b.task_q_pos[t] + b.task_q_len[t])] = False
    assert unseen.any()
    want = _backward(p, q, k, v, o, d_o, lse, one)
    for value in (float("nan"), float("inf")):
        for kk, vv in ((_poisoned(b, k, unseen, value), v), (k, _poisoned(b, v, unseen, value))):
            got = _backward(p, q, kk, vv, o, d_o, lse, one)
            for x, y in zip(got, want):
                assert torch.equal(x, y)
            assert not got[1][unseen].any() and not got[2][unseen].any()


@pytest.mark.parametrize("what", ["k", "v", "q", "d_o"])
@pytest.mark.parametrize("name", ["documents", "gaps_and_keys_nobody_sees", "windows", "documents_d64"])
def test_non_finite_rows_reach_no_further_than_in_whole_units(name, what):
    """One NaN row of Q or dO, or key or value, in every document: what is finite from whole units is the same bits here."""
    b, p, (q, k, v, d_o), o, lse, one, base, run = _setup(name)
    x = {"q": q, "k": k, "v": v, "d_o": d_o}
    rows = []
    for d in sorted(set(b.task_doc.tolist())):
        tasks = [t for t in range(b.n_tasks) if b.task_doc[t] == d]
        t = tasks[len(tasks) * 2 // 3]
        at = (7 * d + 13) % int(b.task_q_len[t])
        rows.append(int(b.task_q_start[t]) + at if what in ("q", "d_o") else int(b.doc_kv_start[d] + min(b.task_q_pos[t] + at, b.task_kv_len[t] - 1)))
    x[what] = _poisoned(b, x[what], torch.tensor(rows, device=DEV), float("nan"))
    args = (x["q"], x["k"], x["v"], o, x["d_o"], lse)
    whole, got = _backward(p, *args, base), _backward(p, *args, one)
    for w, g in zip(whole, got):
        finite = torch.isfinite(w)
        assert finite.any() and torch.equal(g[finite], w[finite])
    assert not all(torch.isfinite(w).all() for w in whole)
