"""Work units cut into pieces (partial results in the workspace, added up by the combine kernels), against the oracle and
against whole units: lone shards with long contexts, small batches, rows scattered so that some see none of a piece's keys,
clipped windows, every head packing, both head_dims; the workspace sizes at which the calls change over; graph replays."""
import numpy as np
import pytest
import torch

import parity_util as P
from paper_2510_18121_amd import binding as B
from paper_2510_18121_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"

BATCHES = {
    # name: (documents, tasks, heads, KV heads, head_dim)
    "lone ragged shard": ([5000], [(0, 4711, 289)], 8, 2, 128),
    "lone ragged shard d64": ([5000], [(0, 4711, 289)], 8, 2, 64),
    "one row": ([4099], [(0, 4098, 1)], 4, 1, 128),
    # units of 256 slots whose rows are in one wave of one half
    "few rows, no GQA": ([6000], [(0, 5990, 5)], 3, 3, 128),
    "few rows, no GQA d64": ([6000], [(0, 5950, 34)], 3, 3, 64),
    "one document": ([2111], [(0, 0, 2111)], 4, 2, 128),
    "one document d64, no GQA": ([1900], [(0, 0, 1900)], 3, 3, 64),
    "GQA 8, two documents": ([1500, 700], [(0, 0, 811), (0, 811, 689), (1, 100, 600)], 8, 1, 128),
    # the parts of dQ take the place of those of dK/dV, so that the batch still fits the static workspace
    "shared parts": ([4400], [(0, 2300, 2100)], 8, 2, 128),
    # one 256-slot tile holds rows at the document's start and at its end: windows some rows see in full, some not at all
    "scattered rows": ([3000], [(0, 0, 3), (0, 70, 60), (0, 1000, 65), (0, 2040, 30), (0, 2900, 100)], 4, 4, 128),
    "scattered rows d64": ([3000], [(0, 0, 3), (0, 70, 60), (0, 1000, 65), (0, 2040, 30), (0, 2900, 100)], 4, 4, 64),
}


def tensors_of(name):
    docs, tasks, hq, hkv, d = BATCHES[name]
    b = W.custom(docs, tasks, hq, hkv, d, seed=90)
    return b, W.make_tensors(b, DEV)


def run(b, t, ws_bytes_f, ws_bytes_b, plan):
    q, k, v, d_o = t
    o, dq, dk, dv = (torch.full_like(x, float("nan")) for x in (q, q, k, v))
    lse = torch.full((b.n_q_heads, b.total_q), float("nan"), device=DEV)
    # what the workspace held before must not matter
    wf = torch.full((ws_bytes_f,), 255, dtype=torch.uint8, device=DEV) if ws_bytes_f else None
    B.ca_forward(plan, q, k, v, o, lse, wf)
    B.ca_backward(plan, q, k, v, o, d_o, lse, dq, dk, dv, torch.full((ws_bytes_b,), 255, dtype=torch.uint8, device=DEV))
    torch.cuda.synchronize()
    return {"o": o, "lse": lse, "dq": dq, "dk": dk, "dv": dv}


@pytest.mark.parametrize("name", list(BATCHES))
def test_pieces_match_the_oracle_and_whole_units(name):
    b, t = tensors_of(name)
    plan = B.ca_plan(b)
    (f0, b0), (f1, b1) = plan.workspace_bytes(), plan.workspace_bytes_split()
    assert f1 > 0 and b1 > b0, "the batch is there because its units are cut"
    pc = plan.pieces()
    n_parts = int(pc["fwd_combine"][:, 1].sum() + pc["bwd_combine"][:, 1].sum())
    assert (b1 - b0 < n_parts * 256 * b.head_dim * 4) == (name == "shared parts")
    cut, whole = run(b, t, f1, b1, plan), run(b, t, 0, b0, plan)
    ref = P.run_oracle(b, *t)
    for r, tag in ((cut, "pieces"), (whole, "whole units")):
        e = P.errors(r, ref)
        print(name, tag, e, flush=True)
        P.assert_parity(e, (name, tag))
    # one byte less than the pieces need: whole units, bit for bit, as without a workspace; more: pieces, and the same again
    less, more = run(b, t, f1 - 1, b1 - 1, plan), run(b, t, f1 + 256, b1 + 256, plan)
    for n in cut:
        assert torch.equal(less[n], whole[n]), n
        assert torch.equal(more[n], cut[n]), n


@pytest.mark.parametrize("hq,hkv,d,shards", [(4, 2, 128, [(0, 300)]), (3, 1, 64, [(0, 65), (100, 31)]), (8, 1, 128, [(40, 1)]),
                                             (16, 2, 64, [(0, 200), (37, 500)]), (6, 2, 128, [(500, 16), (3, 129)]),
                                             (4, 1, 64, [(1000, 20)])])
def test_joint_backward_matches_separate_launches(hq, hkv, d, shards):
    """Small batches run dK/dV and dQ units in one launch (dQ units in halves of 128 rows: all head packings, halves that
    see fewer keys than their unit, rows that fill no half); with timing enabled their workgroups run as two launches."""
    b = W.custom([a + n for a, n in shards], [(i, a, n) for i, (a, n) in enumerate(shards)], hq, hkv, d, seed=92)
    t = W.make_tensors(b, DEV)
    plan = B.ca_plan(b)
    assert plan.info()["joint_backward"] == 1
    joint = P.run_hip(b, *t, plan=plan)
    plan.profile_enable(True)
    apart = P.run_hip(b, *t, plan=plan)
    plan.profile_enable(False)
    ref = P.run_oracle(b, *t)
    for r, tag in ((joint, "joint"), (apart, "apart")):
        e = P.errors(r, ref)
        print(hq, hkv, d, tag, e, flush=True)
        P.assert_parity(e, tag)
    assert torch.equal(joint["dk"], apart["dk"]) and torch.equal(joint["dv"], apart["dv"])


def test_pieces_at_scores_that_outgrow_the_reference():
    """A piece whose scores leave the finite range is repeated by the general path; its weight dominates the others'."""
    b = W.custom([4000], [(0, 3800, 200)], 2, 1, 128, seed=91, scale=1.0)
    q, k, v, _ = W.make_tensors(b, DEV)
    q = torch.full_like(q, 1.0)
    k = (k.float() * 0.01).to(torch.bfloat16)
    k[2100:2110] = (200.0 * np.log(2.0)) / 128
    plan = B.ca_plan(b)
    assert plan.workspace_bytes_split()[0] > 0 and plan.info()["forward_piece_halves"] == 1
    hip = P.run_hip(b, q, k, v, plan=plan)
    e = P.errors(hip, P.run_oracle(b, q, k, v))
    print(e, flush=True)
    assert e["o_err_over_bound"] <= 1.0 and e["lse_max_abs"] <= P.LSE_MAX_ABS, e


def test_pieces_that_are_whole_units_at_head_dim_64():
    """The batches above run their pieces as halves of units; this one's are whole."""
    b = W.custom([5000], [(0, 0, 5000)], 8, 1, 64, seed=95)
    q, k, v, _ = W.make_tensors(b, DEV)
    plan = B.ca_plan(b)
    assert len(plan.pieces()["fwd"]) > 0 and plan.info()["forward_piece_halves"] == 0
    e = P.errors(P.run_hip(b, q, k, v, plan=plan), P.run_oracle(b, q, k, v))
    print(e, flush=True)
    assert e["o_err_over_bound"] <= 1.0 and e["lse_max_abs"] <= P.LSE_MAX_ABS, e


def test_pieces_replay_from_a_graph():
    b, (q, k, v, d_o) = tensors_of("lone ragged shard")
    plan = B.ca_plan(b)
    ws = B.alloc_workspace(plan, DEV)
    assert ws.numel() == max(plan.workspace_bytes_split())
    outs = [torch.empty_like(x) for x in (q, q, k, v)] + [torch.empty((b.n_q_heads, b.total_q), device=DEV)]
    o, dq, dk, dv, lse = outs

    def step():
        B.ca_forward(plan, q, k, v, o, lse, ws)
        B.ca_backward(plan, q, k, v, o, d_o, lse, dq, dk, dv, ws)

    step()
    torch.cuda.synchronize()
    want = [t.clone() for t in outs]
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for _ in range(3):
        for t in outs:
            t.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        for t, w in zip(outs, want):
            assert torch.equal(t, w)


@pytest.mark.parametrize("hq,hkv,d,shards", [(4, 2, 128, [(0, 300)]), (6, 2, 128, [(500, 16), (3, 129)]), (8, 1, 64, [(40, 700)]),
                                             (8, 2, 128, [(0, 1024), (100, 411)])])
def test_timing_does_not_change_results(hq, hkv, d, shards):
    """Joint batches, with and without cut units: all results bit for bit the same with timing enabled, which reports a time for
    each kind of unit."""
    b = W.custom([a + n for a, n in shards], [(i, a, n) for i, (a, n) in enumerate(shards)], hq, hkv, d, seed=93)
    t = W.make_tensors(b, DEV)
    plan = B.ca_plan(b)
    assert plan.info()["joint_backward"] == 1
    want = P.run_hip(b, *t, plan=plan)
    plan.profile_enable(True)
    got = P.run_hip(b, *t, plan=plan)
    times = plan.profile_read()
    plan.profile_enable(False)
    for n in ("o", "lse", "dq", "dk", "dv"):
        assert torch.equal(got[n], want[n]), n
    assert times["bwd_dkv_ms"] > 0 and times["bwd_dq_ms"] > 0, times


@pytest.mark.parametrize("hq,hkv,d,n,length", [(32, 8, 128, 4, 800), (16, 16, 64, 2, 500)])
def test_whole_units_do_not_depend_on_the_batch(hq, hkv, d, n, length):
    """With the workspace of whole units, a document's results are the same bit for bit whatever else is in the batch: on its
    own, where dK/dV and dQ units share a launch, and next to long documents, where they do not."""
    long = [16384, 9001]
    small = W.custom([length] * n, [(i, 0, length) for i in range(n)], hq, hkv, d, seed=94)
    large = W.custom([length] * n + long, [(i, 0, length) for i in range(n)] + [(n + i, 0, m) for i, m in enumerate(long)],
                     hq, hkv, d, seed=94)
    t = W.make_tensors(large, DEV)
    rows, results = n * length, []
    for b, joint in ((large, 0), (small, 1)):
        plan = B.ca_plan(b)
        assert plan.info()["joint_backward"] == joint
        tb = t if b is large else tuple(x[:rows].contiguous() for x in t)
        results.append(run(b, tb, 0, plan.workspace_bytes()[1], plan))
    assert plan.workspace_bytes()[1] == plan.workspace_bytes_split()[1], "nothing is cut: the small batch runs its one launch"
    for name in ("o", "dq", "dk", "dv"):
        assert torch.equal(results[0][name][:rows], results[1][name]), name
    assert torch.equal(results[0]["lse"][:, :rows], results[1]["lse"])


@pytest.mark.parametrize("hq,hkv,d,shard", [(8, 1, 128, (0, 9000)), (32, 4, 64, (50, 5000))])
def test_pieces_beyond_and_inside_the_static_workspace(hq, hkv, d, shard):
    """Partial results that go beyond the static workspace, which whole units fit: with room for them, with the static
    workspace's size (pieces that stay inside it), through the static workspace itself, and as whole units."""
    a, n = shard
    b = W.custom([a + n], [(0, a, n)], hq, hkv, d, seed=96)
    t = W.make_tensors(b, DEV)
    plan, static = B.ca_plan(b), B.lib().ca_static_workspace_bytes()
    (_, b0), (f1, b1) = plan.workspace_bytes(), plan.workspace_bytes_split()
    assert b0 <= static < b1
    ref = P.run_oracle(b, *t)
    results = {}
    for ws_f, ws_b in ((f1, b1), (0, b1 - 1), (0, static), (0, b0)):
        r = results[ws_b] = run(b, t, ws_f, ws_b, plan)
        e = P.errors(r, ref)
        print(hq, hkv, d, ws_f, ws_b, e, flush=True)
        P.assert_parity(e, (ws_f, ws_b))
    q, k, v, d_o = t
    r = results[static]
    dq, dk, dv = (torch.full_like(x, float("nan")) for x in (q, k, v))
    B.ca_backward_static_ws(plan, q, k, v, r["o"], d_o, r["lse"], dq, dk, dv)
    torch.cuda.synchronize()
    for name, got in (("dq", dq), ("dk", dk), ("dv", dv)):
        assert torch.equal(got, r[name]) and torch.equal(results[b1 - 1][name], r[name]), name
