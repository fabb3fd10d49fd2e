"""Hazards between vector instructions, checked in the generated instruction stream (no GPU): `isa_check` compiles the kernel
sources for gfx950 and walks the assembly.  No vector instruction of theirs is inline assembly, so that the compiler knows all that
it has to keep apart; planted violations show that the checks would see one."""
import os

import pytest

from paper_2510_18121_amd import isa_check as C

pytestmark = pytest.mark.skipif(not os.path.exists(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")),
                                reason="hipcc is needed to produce the assembly")


@pytest.fixture(scope="module")
def bwd_asm():
    return C.compile_to_asm("ca_bwd.hip")


def test_backward_kernels_leave_wait_states_to_the_compiler(bwd_asm):
    """The backward kernels have no assembly MFMAs: the compiler sees every one of them and places the wait states."""
    for name in ("ca_bwd_dkv_kernel", "ca_bwd_joint_kernel"):
        bodies = C.kernel_bodies(bwd_asm, name)
        assert len(bodies) == 2  # head_dim 128 and 64
        for body in bodies:
            assert body.count("v_mfma_f32_16x16x32_bf16") >= 100
            # the loops keep everything in registers
            assert "scratch_" not in body
    assert C.assembly_vector_instructions(bwd_asm) == []


def test_no_vector_instruction_reads_a_transcendental_in_the_next_slot(bwd_asm):
    n, bad = C.check_trans_use(bwd_asm)
    assert n > 100
    assert not bad, bad


def test_forward_kernel_transcendentals_and_registers():
    asm = C.compile_to_asm("ca_fwd.hip")
    n, bad = C.check_trans_use(asm)
    assert n > 50 and not bad, bad
    bodies = C.kernel_bodies(asm, "ca_fwd_kernel")
    assert len(bodies) == 4  # head_dim 128 and 64, units and halves of units
    for body in bodies:
        # the loops keep everything in registers
        assert "scratch_" not in body
    assert C.assembly_vector_instructions(asm) == []


def test_planted_violations_are_found():
    assert C.check_trans_use("\tv_exp_f32_e32 v5, v6\n\tv_add_f32_e32 v7, v5, v8\n")[1]
    assert not C.check_trans_use("\tv_exp_f32_e32 v5, v6\n\ts_nop 0\n\tv_add_f32_e32 v7, v5, v8\n")[1]
    assert not C.check_trans_use("\tv_exp_f32_e32 v5, v6\n\tv_add_f32_e32 v7, v9, v8\n")[1]
    assert not C.check_trans_use("\tv_exp_f32_e32 v5, v6\n\tv_exp_f32_e32 v7, v5\n")[1]
    by_hand = "\t;;#ASMSTART\n\tv_xor_b32 v1, 64, v2\n\t;;#ASMEND\n"
    assert C.assembly_vector_instructions(by_hand) == ["v_xor_b32 v1, 64, v2"]
    assert C.assembly_vector_instructions(by_hand.replace("v_xor_b32 v1, 64, v2", "global_load_lds_dwordx4 v1, s[2:3]")) == []
    assert C.assembly_vector_instructions("\tv_xor_b32 v1, 64, v2\n") == []
