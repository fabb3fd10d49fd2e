"""The forward kernel runs whole units of 256 rows, or, where a list has few of them, their halves: the same results bit for bit,
on shards that begin and end anywhere and in units that hold several heads.  Both forms repeat what leaves the finite range."""
import numpy as np
import pytest
import torch

import parity_util as P
from paper_2510_18121_amd import binding as B
from paper_2510_18121_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def batches(docs, tasks, hq, hkv, d, **kw):
    """The batch alone, and in front of as many more documents, of a unit per head each, as make its list run whole units (lists
    of more than 1024 units)."""
    fill = -(-1100 // hq)
    small = W.custom(docs, tasks, hq, hkv, d, seed=97, **kw)
    large = W.custom(docs + [300] * fill, tasks + [(len(docs) + i, 44, 256) for i in range(fill)], hq, hkv, d, seed=97, **kw)
    return small, large


def both_forms(small, large, q, k, v):
    """Results of the small batch's rows from whole units (as part of the large one) and from halves."""
    nq, nk, results = small.total_q, small.total_kv, []
    for b, (qq, kk, vv) in ((large, (q, k, v)), (small, (q[:nq].contiguous(), k[:nk].contiguous(), v[:nk].contiguous()))):
        plan = B.ca_plan(b)
        assert plan.info()["forward_halves"] == (b is small)
        o, lse = torch.full_like(qq, float("nan")), torch.full((b.n_q_heads, b.total_q), float("nan"), device=DEV)
        B.ca_forward(plan, qq, kk, vv, o, lse)  # no workspace: whole units or halves of them, no pieces
        torch.cuda.synchronize()
        results.append({"o": o[:nq], "lse": lse[:, :nq]})
    return results


@pytest.mark.parametrize("d,hq,hkv", [(64, 8, 1), (128, 8, 8), (128, 8, 2)])
def test_halves_equal_whole_units(d, hq, hkv):
    # (first position, rows): around the edges of keys tiles (64), waves (32, 64 rows), halves (128) and units (256)
    shards = [(0, 1), (0, 129), (17, 300), (40, 64), (63, 130), (64, 257), (100, 513), (200, 31), (1000, 256)]
    small, large = batches([a + n for a, n in shards], [(i, a, n) for i, (a, n) in enumerate(shards)], hq, hkv, d)
    q, k, v, _ = W.make_tensors(large, DEV)
    whole, halves = both_forms(small, large, q, k, v)
    assert torch.equal(whole["o"], halves["o"]) and torch.equal(whole["lse"], halves["lse"])
    e = P.errors(halves, P.run_oracle(small, q[:small.total_q], k[:small.total_kv], v[:small.total_kv]))
    print(d, hq, hkv, e, flush=True)
    assert e["o_err_over_bound"] <= 1.0 and e["lse_max_abs"] <= P.LSE_MAX_ABS, e


@pytest.mark.parametrize("d", [64, 128])
def test_both_forms_repeat_after_an_overflow(d):
    """The last 20 keys of a document score about 2^200 above everything before (in probability)."""
    n = 300
    small, large = batches([n], [(0, 0, n)], 2, 1, d, scale=1.0)
    q, k, v, _ = W.make_tensors(large, DEV)
    q = torch.full_like(q, 1.0)
    k = (k.float() * 0.01).to(torch.bfloat16)
    k[n - 20:n] = (200.0 * np.log(2.0)) / d
    ref = P.run_oracle(small, q[:n], k[:n], v[:n])
    for got, form in zip(both_forms(small, large, q, k, v), ("whole units", "halves")):
        e = P.errors(got, ref)
        print(d, form, e, flush=True)
        assert e["o_err_over_bound"] <= 1.0 and e["lse_max_abs"] <= P.LSE_MAX_ABS, (form, e)


@pytest.mark.parametrize("d", [64, 128])
def test_the_reference_is_the_maximum_of_the_first_32_keys(d):
    """Keys 20 and 21 share the weight (what the others have, 2^-60 each, is lost in fp32).  Referred to their own score their
    probabilities are 1, which bf16 holds, so that O is the mean of their V rows, rounded once; referred to a smaller score
    they are 2^60.37, and O carries their rounding."""
    n = 300
    small, large = batches([n], [(0, 0, n)], 2, 1, d, scale=1.0)
    q, k, v, _ = W.make_tensors(large, DEV)
    q, k = torch.full_like(q, 1.0), torch.zeros_like(k)
    k[20:22] = 60.37 * np.log(2.0) / d
    mean = (v[20].float() + v[21].float()) / 2
    # (a score times log2(e) and its fp32 rounding, which is subtracted, are 2^-19 apart: where that decides how O is rounded, skip)
    sure = (mean * (1 + 1e-5)).to(torch.bfloat16) == (mean * (1 - 1e-5)).to(torch.bfloat16)
    sure = (sure & (mean.abs() > 1e-3)).expand(n - 21, 2, d)  # (where the two cancel, the others show)
    assert sure.float().mean() > 0.4
    for got in both_forms(small, large, q, k, v):
        assert torch.equal(got["o"][21:][sure], mean.to(torch.bfloat16).expand(n - 21, 2, d)[sure])


@pytest.mark.parametrize("d", [64, 128])
def test_an_overflow_in_one_half_leaves_the_other_alone(d):
    """Rows 200 and up of a unit leave the finite range and are computed again with the rest of their half; the other half is not,
    in either form."""
    n = 256
    small, large = batches([n], [(0, 0, n)], 2, 1, d, scale=1.0)
    q, k, v, _ = W.make_tensors(large, DEV)
    q = torch.full_like(q, 1.0)
    k = (k.float() * 0.05).to(torch.bfloat16)
    k[200:204] = (200.0 * np.log(2.0)) / d
    whole, halves = both_forms(small, large, q, k, v)
    assert torch.isfinite(whole["o"]).all() and float(whole["lse"][:, 200:].min()) > 130
    assert torch.equal(whole["o"], halves["o"]) and torch.equal(whole["lse"], halves["lse"])


@pytest.mark.parametrize("kind", [float("inf"), float("nan")])
@pytest.mark.parametrize("d", [64, 128])
def test_whom_a_non_finite_value_reaches_does_not_depend_on_the_form(d, kind):
    """A masked key multiplies its value by 0, so a non-finite one reaches the rows that are multiplied with its 32 keys: those of
    the 64 that share a wave in whole units."""
    shards = [(10, 290), (0, 256), (100, 40)]
    small, large = batches([a + n for a, n in shards], [(i, a, n) for i, (a, n) in enumerate(shards)], 2, 2, d)
    q, k, v, _ = W.make_tensors(large, DEV)
    for key in (20, 40, 57, 100, 130, 170, 210):
        bad = v.clone()
        for i, (a, n) in enumerate(shards):
            if key < a + n:
                bad[sum(x + y for x, y in shards[:i]) + key] = kind
        whole, halves = both_forms(small, large, q, k, bad)
        assert torch.equal(whole["o"].isnan(), halves["o"].isnan()) and not torch.isfinite(whole["o"]).all()
        assert torch.equal(whole["o"].nan_to_num(0.0), halves["o"].nan_to_num(0.0)) and torch.equal(whole["lse"], halves["lse"])


def test_taking_turns_does_not_change_results():
    """512 units of equal length, two per CU, which take turns at having priority, against the same among 1632 that do not."""
    small, large = batches([1280] * 16, [(i, 1024, 256) for i in range(16)], 32, 8, 128)
    q, k, v, _ = W.make_tensors(large, DEV)
    nq, nk, results = small.total_q, small.total_kv, []
    for b, (qq, kk, vv) in ((large, (q, k, v)), (small, (q[:nq].contiguous(), k[:nk].contiguous(), v[:nk].contiguous()))):
        plan = B.ca_plan(b)
        assert plan.info()["forward_turns"] == (b is small) and plan.info()["forward_halves"] == 0
        results.append(P.run_hip(b, qq, kk, vv, plan=plan))
    assert torch.equal(results[0]["o"][:nq], results[1]["o"]) and torch.equal(results[0]["lse"][:, :nq], results[1]["lse"])
