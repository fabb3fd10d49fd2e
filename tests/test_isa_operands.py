"""Static checks of the generated assembly: the kernels spill no registers, and are seen to their ends (no GPU)."""
import os

import pytest

from paper_2510_18121_amd import isa_check as C

pytestmark = pytest.mark.skipif(not os.path.exists(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")),
                                reason="hipcc is needed to produce the assembly")


def test_joint_kernel_keeps_everything_in_registers():
    bodies = C.kernel_bodies(C.compile_to_asm("ca_bwd.hip"), "ca_bwd_joint_kernel")
    assert len(bodies) == 2  # head_dim 128 and 64
    for body in bodies:
        assert "scratch_" not in body


def test_dq_kernel_keeps_everything_in_registers():
    asm = C.compile_to_asm("ca_bwd.hip")
    bodies = C.kernel_bodies(asm, "ca_bwd_dq_kernel")
    assert len(bodies) == 2  # head_dim 128 and 64
    for body in bodies:
        assert "scratch_" not in body


def test_kernels_that_return_early_are_seen_to_their_end():
    asm = "_Z1kv:\n\ts_endpgm\n.LBB0_1:\n\tscratch_store_dword off, v0, off\n\ts_endpgm\n.Lfunc_end0:\n\tv_nop\n"
    (body,) = C.kernel_bodies(asm, "1kv")
    assert "scratch_" in body and body.count("s_endpgm") == 2 and "v_nop" not in body
