"""Planner: the lists in which long work units are cut into pieces (no GPU).  Whatever is cut, the pieces of a unit cover
exactly what the unit covers, once, and the combine lists name exactly their partial results."""
import numpy as np
import pytest

from paper_2510_18121_amd import binding as B
from paper_2510_18121_amd import workloads as W


def check_pieces(b):
    p = B.ca_plan_host(b)
    pc, step = p.pieces(), p.info()["fwd_kv_step"]
    (fwd0, bwd0), (fwd1, bwd1) = p.workspace_bytes(), p.workspace_bytes_split()
    part = 256 * b.head_dim * 4
    n_fwd = int(pc["fwd_combine"][:, 1].sum())
    n_bwd = int(pc["bwd_combine"][:, 1].sum())
    # workspace: nothing more where nothing is cut, room for every part otherwise, and bounded
    assert (fwd1 > fwd0) == (n_fwd > 0) == (len(pc["fwd"]) > 0)
    assert (bwd1 > bwd0) == (n_fwd + n_bwd > 0) and (n_bwd > 0) == (len(pc["bwd"]) > 0)
    assert fwd1 == n_fwd * (part + 4096) and (bwd1 == bwd0 or bwd1 >= bwd0 + max(n_fwd, n_bwd) * part)
    assert bwd1 - bwd0 <= 256 << 20
    # forward / dQ: every unit whole, or cut into consecutive windows of whole tiles that a combine entry names
    if n_fwd:
        whole = {(u[0], u[3], u[4]): u for u in p.fwd_units().tolist()}
        combine = {(c[2], c[3], c[4]): c for c in pc["fwd_combine"].tolist()}
        got = {}
        for i, (s0, kv, nk, h, hp, k0, part_i, _) in enumerate(pc["fwd"].tolist()):
            assert i % b.n_kv_heads == h // (b.n_q_heads // b.n_kv_heads), "unit index modulo n_kv_heads is the KV head"
            got.setdefault((s0, h, hp), []).append((k0, nk, kv, part_i))
        assert set(got) == set(whole)
        for key, pieces in got.items():
            _, kv, nk, _, _ = whole[key]
            pieces.sort()
            if key not in combine:
                assert pieces == [(0, nk, kv, -1)]
                continue
            first, n = combine[key][:2]
            assert len(pieces) == n > 1 and [x[3] for x in pieces] == list(range(first, first + n))
            end = 0
            for k0, m, row, _ in pieces:
                assert k0 == end and k0 % step == 0 and row == kv + k0 and m >= 1
                end = k0 + m
            assert end == nk
        parts = sorted(i for c in pc["fwd_combine"].tolist() for i in range(c[0], c[0] + c[1]))
        assert parts == list(range(n_fwd))
        costs = -(-pc["fwd"][:, 2] // step)
        assert np.all(np.diff(costs) <= 0), "longest first"
    # dK/dV: the same over the query blocks; chains stay as they are
    if n_bwd:
        n_wg = p.info()["n_bwd_workgroups"]
        key_of = lambda u: (u[3], u[6])
        whole = {key_of(u): u for u in p.bwd_units().tolist()}
        combine = {(c[2], c[4]): c for c in pc["bwd_combine"].tolist()}
        got, bw, steps = {}, pc["bwd"].tolist(), []
        for i, u in enumerate(bw):
            if i < pc["bwd_workgroups"]:
                assert i % b.n_kv_heads == u[6] and u[8] >= 1
                mine = [u] + (bw[u[7]:u[7] + u[8] - 1] if u[8] > 1 else [])
                assert all(x[6] == u[6] for x in mine) and (u[8] == 1 or pc["bwd_workgroups"] <= u[7])
                steps.append(sum((x[1] - x[0]) // 64 * x[9] for x in mine))
            else:
                assert u[8] == 0
            got.setdefault(key_of(u), []).append(u)
        assert np.all(np.diff(steps) <= 0) and sum(u[8] for u in bw) == len(bw)
        assert set(got) == set(whole)
        for key, pieces in got.items():
            w = whole[key]
            if key not in combine:
                assert len(pieces) == 1 and pieces[0][:7] == w[:7] and pieces[0][9] == w[9] and pieces[0][7] >= 0
                continue
            first, n, kv_row, n_valid, hk, _ = combine[key]
            pieces.sort(key=lambda u: u[0])
            assert len(pieces) == n > 1 and [-1 - u[7] for u in pieces] == list(range(first, first + n))
            assert (kv_row, hk, n_valid) == (w[3], w[6], w[4])
            end = w[0]
            for u in pieces:
                assert u[0] == end and u[1] > u[0] and (u[1] - u[0]) % 64 == 0 and u[8] == 1
                assert u[2] == min(max(w[2], u[0]), u[1]) and u[3:7] == w[3:7] and u[9] == w[9]
                end = u[1]
            assert end == w[1]
        parts = sorted(i for c in pc["bwd_combine"].tolist() for i in range(c[0], c[0] + c[1]))
        assert parts == list(range(n_bwd))
    return n_fwd, n_bwd


def test_where_units_are_cut():
    """Few long units: cut.  Enough of them, or only short ones: not."""
    lone = W.custom([16384], [(0, 16384 - 256, 256)], 32, 8, 128)
    n_fwd, n_bwd = check_pieces(lone)
    assert n_fwd >= 128 and n_bwd == 0  # 32 units of 256 tiles; the dK/dV units are 1024 of 16 steps
    n_fwd, n_bwd = check_pieces(W.custom([4096], [(0, 0, 4096)], 32, 8, 128))
    assert n_bwd > 0  # 256 dK/dV units of up to 256 steps, 132 on average
    for b in (W.config(2), W.config(3), W.config(5), W.shard_chunk(64, "distinct")):
        assert check_pieces(b) == (0, 0)
    assert check_pieces(W.custom([200], [(0, 0, 200)], 8, 2, 128))[0] == 0
    assert check_pieces(W.custom([8], [], 4, 2, 64)) == (0, 0)


@pytest.mark.parametrize("hq,hkv,sizes", [(8, 1, (9000, 12000, 15800, 16500)), (64, 8, (1500, 1900, 2200))])
def test_units_are_cut_on_both_sides_of_the_static_workspace(hq, hkv, sizes):
    """One document: its dK/dV units are too few and too long whether whole units take a half, nearly all or more of the static
    workspace."""
    static, base = B.lib().ca_static_workspace_bytes(), []
    for n in sizes:
        b = W.custom([n], [(0, 0, n)], hq, hkv, 128)
        assert check_pieces(b)[1] > 0, n
        base.append(B.ca_plan_host(b).workspace_bytes()[1])
    assert base[0] < 0.8 * static and 0.9 * static < base[-2] <= static < base[-1]


@pytest.mark.parametrize("seed", range(30))
def test_pieces_cover_their_units(seed):
    rng = np.random.default_rng(8000 + seed)
    hkv = int(rng.choice([1, 2, 3, 8]))
    g = int(rng.choice([1, 2, 3, 4, 8]))
    docs = [int(np.exp(rng.uniform(0, np.log(30000)))) for _ in range(int(rng.integers(1, 4)))]
    tasks = []
    for dd, n in enumerate(docs):
        for _ in range(int(rng.integers(1, 4))):
            a = int(rng.integers(0, n))
            tasks.append((dd, a, int(min(n - a, np.exp(rng.uniform(0, np.log(3000)))) // 1 or 1)))
    b = W.custom(docs, tasks, hkv * g, hkv, int(rng.choice([64, 128])),
                 doc_order=[int(x) for x in rng.permutation(len(docs))], task_order=[int(x) for x in rng.permutation(len(tasks))])
    for t in range(b.n_tasks):
        if rng.random() < 0.25:
            b.task_kv_len[t] = int(rng.integers(1, b.task_kv_len[t] + 1))
    check_pieces(b)
