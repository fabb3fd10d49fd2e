"""Workspace where device memory is short (no GPU): a batch that fits without the partial results of cut units goes on fitting,
as whole units."""
import types

import pytest
import torch

from one_pass_batches import BATCHES
from paper_2510_18121_amd import autograd as A
from paper_2510_18121_amd import binding as B
from paper_2510_18121_amd import workloads as W


@pytest.fixture
def limit(monkeypatch):
    """Allocations beyond `limit["bytes"]` fail like the device's."""
    box, empty = {"bytes": 1 << 40}, torch.empty

    def limited(*size, **kw):
        t = empty(*size, **{**kw, "device": "cpu"})
        if t.numel() * t.element_size() > box["bytes"]:
            raise torch.cuda.OutOfMemoryError("no room")
        return t

    monkeypatch.setattr(torch, "empty", limited)
    return box


def test_workspace_without_room_for_partial_results(limit):
    plan = B.ca_plan_host(W.custom([16384], [(0, 16384 - 256, 256)], 32, 8, 128))
    base, split = max(plan.workspace_bytes()), max(plan.workspace_bytes_split())
    assert base < split
    assert B.alloc_workspace(plan).numel() == split
    limit["bytes"] = split - 1
    assert B.alloc_workspace(plan).numel() == base
    limit["bytes"] = base - 1
    with pytest.raises(torch.cuda.OutOfMemoryError):
        B.alloc_workspace(plan)


def test_one_pass_leaves_memory_to_others(limit, monkeypatch):
    """The workspace holds the one pass's sums where they take at most an eighth of what is free, or where the caller says so."""
    plan = B.ca_plan_host(BATCHES["documents"]())
    base, split, one = max(plan.workspace_bytes()), max(plan.workspace_bytes_split()), plan.workspace_bytes_one_pass()
    assert base < one
    box = {"free": 0, "reserved": 1 << 30, "allocated": 1 << 30}
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: False)
    monkeypatch.setattr(torch.cuda, "mem_get_info", lambda device=None: (box["free"], 288 << 30))
    monkeypatch.setattr(torch.cuda, "memory_reserved", lambda device=None: box["reserved"])
    monkeypatch.setattr(torch.cuda, "memory_allocated", lambda device=None: box["allocated"])
    box["free"] = 8 * (one - base)
    assert B.alloc_workspace(plan).numel() == max(one, split)
    box["free"] -= 1
    assert B.alloc_workspace(plan).numel() == split
    assert B.alloc_workspace(plan, one_pass=True).numel() == max(one, split)
    box["allocated"] -= 1  # what torch holds for itself counts as free
    assert B.alloc_workspace(plan).numel() == max(one, split)
    assert B.alloc_workspace(plan, one_pass=False).numel() == split
    limit["bytes"] = max(one, split) - 1
    assert B.alloc_workspace(plan, one_pass=True).numel() == split


def test_forward_without_room_for_partial_results(limit, monkeypatch):
    b = W.custom([16384], [(0, 16384 - 256, 256)], 4, 1, 64)
    plan = B.ca_plan_host(b)
    n = plan.workspace_bytes_split()[0]
    given = []
    monkeypatch.setattr(B, "ca_forward", lambda plan, q, k, v, o, lse, ws=None, stream=None: given.append(ws))
    server = types.SimpleNamespace(plan=plan, fwd_ws_bytes=n)
    ctx = types.SimpleNamespace(save_for_backward=lambda *t: None)
    q, k = torch.zeros(b.total_q, 4, 64, dtype=torch.bfloat16), torch.zeros(b.total_kv, 1, 64, dtype=torch.bfloat16)
    A._CoreAttention.forward(ctx, q, k, k, server)
    limit["bytes"] = n - 1
    A._CoreAttention.forward(ctx, q, k, k, server)
    assert n > 0 and given[0].numel() == n and given[1] is None
