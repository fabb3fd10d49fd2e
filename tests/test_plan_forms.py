"""Planner: in which form the forward runs its units and pieces (no GPU)."""
import pytest

from paper_2510_18121_amd import binding as B
from paper_2510_18121_amd import workloads as W


@pytest.mark.parametrize("n,rows,keys,hq,hkv,d,pieces,halves,turns", [
    # 32 units of 256 tiles: 256 pieces, whose 512 halves share the CUs evenly
    (1, 256, 16384, 32, 8, 128, 256, 1, 1),
    # head_dim 64 has three workgroups per CU and takes no turns
    (1, 256, 16384, 32, 8, 64, 256, 1, 0),
])
def test_lone_shards(n, rows, keys, hq, hkv, d, pieces, halves, turns):
    p = B.ca_plan_host(W.custom([keys] * n, [(i, keys - rows, rows) for i in range(n)], hq, hkv, d))
    info = p.info()
    got = len(p.pieces()["fwd"]), info["forward_piece_halves"], info["forward_piece_turns"]
    assert got == (pieces, halves, turns)


def test_units_of_unlike_length_take_no_turns():
    """The longest are the oldest on their CU and served first."""
    lens = [64 * (i + 1) + 256 for i in range(16)]
    info = B.ca_plan_host(W.custom(lens, [(i, n - 256, 256) for i, n in enumerate(lens)], 32, 8, 128)).info()
    assert info["n_fwd_units"] == 512 and info["forward_turns"] == 0
    info = B.ca_plan_host(W.custom([1280] * 16, [(i, 1024, 256) for i in range(16)], 32, 8, 128)).info()
    assert info["n_fwd_units"] == 512 and info["forward_turns"] == 1
