"""The backward in one pass without a GPU: the planner's queues, and static checks of the kernel's assembly."""
import os

import numpy as np
import pytest

from one_pass_batches import BATCHES
from paper_2510_18121_amd import binding as B
from paper_2510_18121_amd import isa_check as C
from paper_2510_18121_amd import workloads as W


@pytest.mark.parametrize("name", sorted(BATCHES))
def test_chains(name):
    """Every key of every KV head once; a chain in one queue, in the order of its tiles; blocks without a mask see a later key."""
    b = BATCHES[name]()
    p = B.ca_plan_host(b)
    assert p.info()["one_pass_backward"] == 1
    (units, queue), pos = p.one_pass_units(), p.rows()[1]
    keys = 256 if b.head_dim == 128 else 128
    assert queue[0] == 0 and queue[8] == len(units) and np.all(np.diff(queue) >= 0)
    seen, chain = np.zeros((b.total_kv, b.n_kv_heads), int), {}
    for q in range(8):
        for begin, end, full, row, n, k0, h, follow, count, heads in units[queue[q]:queue[q + 1]].tolist():
            seen[row:row + n, h] += 1
            at = chain.setdefault((row - k0, h), [q, 0, begin])
            assert at[0] == q and at[1] == k0 and at[2] <= begin, "one queue, first keys first, under no more rows than before"
            at[1], at[2] = k0 + keys, begin
            assert begin <= full <= end and (count, follow) == (1, 0) and begin % 64 == full % 64 == end % 64 == 0
            if full < end:
                assert pos[full] >= k0 + keys
            if begin < full:
                assert pos[begin + 63] >= k0, "some row of the first block sees the tile"
    held = np.zeros(b.total_kv, int)
    for d in set(b.task_doc.tolist()):
        held[b.doc_kv_start[d]:b.doc_kv_start[d] + b.doc_kv_len[d]] = 1
    assert np.array_equal(seen, np.repeat(held[:, None], b.n_kv_heads, 1))


@pytest.mark.parametrize("name", sorted(BATCHES))
def test_longest_first_inside_groups_of_chains(name):
    """A queue's units: longest first, of equal ones those of the earlier keys; where that starts again, only new chains follow."""
    units, queue = B.ca_plan_host(BATCHES[name]()).one_pass_units()
    for q in range(8):
        done, group, last = set(), set(), None
        for begin, end, full, row, n, k0, h, follow, count, heads in units[queue[q]:queue[q + 1]].tolist():
            key = (-(end - begin) * heads, k0)
            if last is not None and key < last:
                done, group = done | group, set()
            group.add((row - k0, h))
            assert (row - k0, h) not in done
            last = key


def test_workspace():
    """Sums of dQ and a counter per wave and 32 rows lie behind what whole units need; small batches have no one pass."""
    b = BATCHES["documents"]()
    p = B.ca_plan_host(b)
    rows, d = p.info()["padded_rows"] * b.n_q_heads, b.head_dim
    assert p.workspace_bytes_one_pass() == p.workspace_bytes()[1] + rows * d * 4 + rows // 32 * 8 * 4 + 8 * 256
    small = B.ca_plan_host(W.custom([4000], [(0, 0, 4000)], 32, 8, 128))
    assert small.workspace_bytes_one_pass() == 0 and small.info()["one_pass_backward"] == 0 and len(small.one_pass_units()[0]) == 0


def test_offsets_beyond_32_bits_take_other_kernels():
    b = W.custom([300000], [(0, 0, 300000)], 32, 8, 128)  # 4.9 GB of sums
    assert B.ca_plan_host(b).info()["one_pass_backward"] == 0


@pytest.mark.parametrize("last,taken", [(960, 1), (961, 0)])
def test_largest_offset(last, taken):
    """128 documents of whole 64-row blocks, 64 heads: 4 GiB less 2 MiB of sums, and one block more."""
    lens = [1024] * 127 + [last]
    info = B.ca_plan_host(W.custom(lens, [(i, 0, n) for i, n in enumerate(lens)], 64, 8, 128)).info()
    sums = info["padded_rows"] * 64 * 128 * 4
    assert info["one_pass_backward"] == taken and sums == (1 << 32) - (1 << 21) * taken


@pytest.mark.skipif(not os.path.exists(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")), reason="hipcc is needed to produce the assembly")
def test_kernel_keeps_everything_in_registers():
    asm = C.compile_to_asm("ca_bwd_fused.hip")
    bodies = C.kernel_bodies(asm, "ca_bwd_fused_kernel")
    assert len(bodies) == 2  # head_dim 128 and 64
    for body in bodies:
        assert body.count("v_mfma_f32_16x16x32_bf16") >= 80 and "scratch_" not in body
    assert C.assembly_vector_instructions(asm) == []
    n, bad = C.check_trans_use(asm)
    assert n >= 64 and not bad, bad
