"""Static checks of the generated assembly: operands of assembly MFMAs in all kernels, and the MFMA chains of the kernel that
runs dK/dV and dQ units in one launch (no GPU)."""
import os

import pytest

from paper_2510_18121_amd import isa_check as C

pytestmark = pytest.mark.skipif(not os.path.exists(os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")),
                                reason="hipcc is needed to produce the assembly")


@pytest.mark.parametrize("source", ["ca_bwd.hip", "ca_fwd.hip"])
def test_operands_of_assembly_mfmas_are_settled(source):
    asm = C.compile_to_asm(source)
    assert C.check_mfma_operands(asm) == (0, [])  # none is left to settle by hand
    for body in C.kernel_bodies(asm, "ca_bwd_joint_kernel"):
        assert "scratch_" not in body


def test_planted_copies_in_front_of_an_mfma_are_found():
    mfma = "\t;;#ASMSTART\n\tv_mfma_f32_32x32x16_bf16 v[0:15], v[40:43], a[64:67], v[0:15]\n\t;;#ASMEND\n"
    far = "\tv_accvgpr_write_b32 a67, v9\n\ts_nop 1\n" + mfma
    assert C.check_mfma_operands(far) == (1, [])
    assert len(C.check_mfma_operands("\tv_accvgpr_write_b32 a67, v9\n" + mfma)[1]) == 1
    assert len(C.check_mfma_operands("\tv_accvgpr_write_b32 a67, v9\n\ts_nop 0\n" + mfma)[1]) == 1
    assert len(C.check_mfma_operands("\tv_mov_b32_e32 v3, v9\n" + mfma)[1]) == 1
    assert C.check_mfma_operands("\tv_mov_b32_e32 v33, v9\n" + mfma) == (1, [])
    assert C.check_mfma_operands("\tv_mov_b32_e32 v3, v9\n" + mfma.replace(";;#ASMSTART", "").replace(";;#ASMEND", "")) == (0, [])


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
