"""Plan upload: small arrays go up in one transfer, large ones by themselves; plans with both, uploaded again."""
import pytest
import torch

import parity_util as P
from paper_2510_18121_amd import binding as B
from paper_2510_18121_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def test_plan_with_large_and_small_arrays_uploaded_twice():
    """1500 lone 20-row shards: unit lists of 12K and 24K entries (beyond 256 KiB) next to small arrays."""
    n, q = 1500, 20
    docs = [q + 7 * (i % 40) for i in range(n)]
    b = W.custom(docs, [(i, docs[i] - q, q) for i in range(n)], 8, 8, 64, seed=95)
    t = W.make_tensors(b, DEV)
    plan = B.ca_plan(b)
    assert plan.fwd_units().nbytes > 200 << 10 and plan.bwd_units().nbytes > 256 << 10
    first = P.run_hip(b, *t, plan=plan)
    P.assert_parity(P.errors(first, P.run_oracle(b, *t)), "large plan")
    plan.upload()
    again = P.run_hip(b, *t, plan=plan)
    for name in ("o", "lse", "dq", "dk", "dv"):
        assert torch.equal(first[name], again[name]), name
