"""The forward kernel's diagonal: every tile a wave sees, except tile 0 for rows that see less than a tile, takes the
pipelined path, masked where rows of the wave end inside the tile.  Shards whose first row and length sit on and around
the edges of tiles (64 keys), waves (64 rows) and units (256 rows), waves whose rows are scattered over the document, and
scores that overflow the pipeline's reference inside a masked tile, against the oracle."""
import numpy as np
import pytest
import torch

import parity_util as P
from paper_2510_18121_amd import workloads as W

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def forward_errors(b, q, k, v):
    return P.errors(P.run_hip(b, q, k, v), P.run_oracle(b, q, k, v))


@pytest.mark.parametrize("d,hq,hkv", [(64, 4, 2), (128, 2, 2), (128, 8, 1)])
def test_shards_around_tile_edges(d, hq, hkv):
    # (first position, rows): one document each, so every shard starts a unit of its own
    shards = [(0, 1), (0, 63), (0, 64), (0, 65), (1, 64), (62, 2), (63, 1), (63, 130), (64, 64), (64, 257), (65, 63), (95, 33),
              (127, 65), (128, 256), (191, 1), (192, 31), (255, 300), (320, 7)]
    docs = [a + n for a, n in shards]
    b = W.custom(docs, [(i, a, n) for i, (a, n) in enumerate(shards)], hq, hkv, d, seed=81)
    q, k, v, _ = W.make_tensors(b, DEV)
    e = forward_errors(b, q, k, v)
    print(d, hq, hkv, e, flush=True)
    assert e["o_err_over_bound"] <= 1.0 and e["lse_max_abs"] <= P.LSE_MAX_ABS, e


@pytest.mark.parametrize("d", [64, 128])
def test_waves_with_scattered_rows(d):
    """Rows of many small shards of one document share a wave: its tiles are seen in full by some rows, in part or not at
    all by others, from tile 0 to the last."""
    rng = np.random.default_rng(82)
    starts = sorted(rng.choice(2000 // 8, size=60, replace=False).tolist())
    b = W.custom([2000], [(0, 8 * int(s) + int(rng.integers(0, 3)), int(rng.integers(1, 6))) for s in starts], 4, 2, d, seed=83)
    q, k, v, _ = W.make_tensors(b, DEV)
    e = forward_errors(b, q, k, v)
    print(d, e, flush=True)
    assert e["o_err_over_bound"] <= 1.0 and e["lse_max_abs"] <= P.LSE_MAX_ABS, e


@pytest.mark.parametrize("d", [64, 128])
def test_overflow_inside_a_masked_tile_repeats_the_unit(d):
    """The keys a row sees last score about 2^200 above everything before (in probability), and do so inside the diagonal
    tile: the pipeline's row sum leaves the finite range and the unit is computed again by the general path."""
    n = 300
    b = W.custom([n], [(0, 0, n)], 2, 1, d, seed=84, scale=1.0)
    q, k, v, _ = W.make_tensors(b, DEV)
    q = torch.full_like(q, 1.0)
    k = (k.float() * 0.01).to(torch.bfloat16)
    k[n - 20:] = (200.0 * np.log(2.0)) / d  # scores of about 139 = 200 ln 2
    hip = P.run_hip(b, q, k, v)
    e = P.errors(hip, P.run_oracle(b, q, k, v))
    print(d, e, flush=True)
    assert torch.isfinite(hip["o"]).all() and torch.isfinite(hip["lse"]).all()
    # rows that end among the last 20 keys average V rows with equal weights, whose bf16 probabilities are exact; LSE is
    # about 140 there, where an fp32 unit is 1.5e-5
    assert e["o_err_over_bound"] <= 1.0 and e["lse_max_abs"] <= P.LSE_MAX_ABS, e


@pytest.mark.parametrize("kind", [float("inf"), float("nan")])
@pytest.mark.parametrize("d,key,rows", [(64, 100, 64), (128, 100, 64), (64, 170, 128), (128, 170, 128)])
def test_values_beyond_a_waves_last_block_do_not_reach_its_rows(d, key, rows, kind):
    """Probabilities of masked keys are 0, but 0 times a non-finite value is not: a wave multiplies no values of a 32-key block
    that none of its rows sees.  Waves hold positions 10..73 and 74..137 here; their last tiles hold blocks from key 96 and from key 160
    on that they do not see."""
    b = W.custom([300], [(0, 10, 290)], 2, 2, d, seed=85)
    q, k, v, _ = W.make_tensors(b, DEV)
    want = P.run_hip(b, q, k, v)
    bad = v.clone()
    bad[key] = kind
    got = P.run_hip(b, q, k, bad)
    assert torch.isfinite(want["o"]).all() and not torch.isfinite(got["o"]).all()
    assert torch.equal(got["o"][:rows], want["o"][:rows]) and torch.equal(got["lse"], want["lse"])
