"""Planner: in which form the forward runs its units and pieces (no GPU)."""
import pytest

from paper_2510_18121_amd import binding as B
from paper_2510_18121_amd import workloads as W


@pytest.mark.parametrize("n,rows,keys,hq,hkv,d,pieces,halves,turns", [
    # 32 units of 256 tiles: 256 pieces, whose 512 halves share the CUs evenly
    (1, 256, 16384, 32, 8, 128, 256, 1, 1),
    # 128 units of 2032 tiles: two whole pieces per CU beat two halves of one twice as long by more than their parts cost
    (1, 1000, 130001, 32, 8, 128, 512, 0, 1),
    # 176 of 938: fewer units than CUs, but too many to ignore that two share one
    (2, 700, 60000, 32, 8, 128, 704, 0, 0),
    # head_dim 64 has three workgroups per CU and takes no turns
    (1, 256, 16384, 32, 8, 64, 256, 1, 0),
])
def test_lone_shards(n, rows, keys, hq, hkv, d, pieces, halves, turns):
    p = B.ca_plan_host(W.custom([keys] * n, [(i, keys - rows, rows) for i in range(n)], hq, hkv, d))
    info = p.info()
    got = len(p.pieces()["fwd"]), info["forward_piece_halves"], info["forward_piece_turns"]
    assert got == (pieces, halves, turns)


def test_parts_beyond_the_static_workspace_leave_a_plan_inside_it():
    """Callers with the static workspace run the pieces that fit it."""
    b = W.custom([130001], [(0, 129001, 1000)], 32, 8, 128)
    p = B.ca_plan_host(b)
    static = B.lib().ca_static_workspace_bytes()
    assert p.workspace_bytes()[1] < static < p.workspace_bytes_split()[1]


def test_units_of_unlike_length_take_no_turns():
    """The longest are the oldest on their CU and served first."""
    lens = [64 * (i + 1) + 256 for i in range(16)]
    info = B.ca_plan_host(W.custom(lens, [(i, n - 256, 256) for i, n in enumerate(lens)], 32, 8, 128)).info()
    assert info["n_fwd_units"] == 512 and info["forward_turns"] == 0
    info = B.ca_plan_host(W.custom([1280] * 16, [(i, 1024, 256) for i in range(16)], 32, 8, 128)).info()
    assert info["n_fwd_units"] == 512 and info["forward_turns"] == 1


@pytest.mark.parametrize("hq,hkv,shards", [(3, 3, [(5990, 5)]), (4, 1, [(4000, 70), (3900, 33)]), (16, 2, [(3000, 300), (10, 290)])])
def test_units_know_how_many_of_their_slots_hold_rows(hq, hkv, shards):
    """The forward kernel leaves out halves and waves behind a unit's last row."""
    p = B.ca_plan_host(W.custom([a + n for a, n in shards], [(i, a, n) for i, (a, n) in enumerate(shards)], hq, hkv, 128))
    row, units = p.rows()[0], p.pieces()["fwd"].tolist()
    assert units
    for slot0, _, _, _, hp, _, _, rows in units:
        held = row[slot0:slot0 + 256 // hp] >= 0
        assert rows == held.sum() > 0 and held[:rows].all()
