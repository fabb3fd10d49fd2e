"""The forward kernel runs whole units of 256 rows, or, where a list has few of them, their halves: the same results bit for bit,
on shards that begin and end anywhere and in units that hold several heads."""
import pytest
import torch

import parity_util as P
from paper_2510_18121_amd import binding as B
from paper_2510_18121_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("d,hq,hkv", [(64, 8, 1), (128, 8, 8), (128, 8, 2)])
def test_halves_equal_whole_units(d, hq, hkv):
    # (first position, rows): around the edges of keys tiles (64), waves (32, 64 rows), halves (128) and units (256)
    shards = [(0, 1), (0, 129), (17, 300), (40, 64), (63, 130), (64, 257), (100, 513), (200, 31), (1000, 256)]
    few = [a + n for a, n in shards]
    tasks = [(i, a, n) for i, (a, n) in enumerate(shards)]
    fill = -(-1100 // hq)  # documents of one unit per head: beyond 1024 units every list runs whole ones
    small = W.custom(few, tasks, hq, hkv, d, seed=97)
    large = W.custom(few + [300] * fill, tasks + [(len(few) + i, 44, 256) for i in range(fill)], hq, hkv, d, seed=97)
    q, k, v, d_o = W.make_tensors(large, DEV)
    nq, nk = small.total_q, small.total_kv
    results = []
    for b, (qq, kk, vv) in ((large, (q, k, v)), (small, (q[:nq].contiguous(), k[:nk].contiguous(), v[:nk].contiguous()))):
        plan = B.ca_plan(b)
        assert (len(plan.fwd_units()) > 1024) == (b is large)
        o, lse = torch.full_like(qq, float("nan")), torch.full((hq, b.total_q), float("nan"), device=DEV)
        B.ca_forward(plan, qq, kk, vv, o, lse)  # no workspace: whole units or halves of them, no pieces
        torch.cuda.synchronize()
        results.append((o[:nq], lse[:, :nq]))
    assert torch.equal(results[0][0], results[1][0]) and torch.equal(results[0][1], results[1][1])
    t = (q[:nq].contiguous(), k[:nk].contiguous(), v[:nk].contiguous())
    e = P.errors({"o": results[1][0], "lse": results[1][1]}, P.run_oracle(small, *t))
    print(d, hq, hkv, e, flush=True)
    assert e["o_err_over_bound"] <= 1.0 and e["lse_max_abs"] <= P.LSE_MAX_ABS, e
