"""Static checks of the generated gfx950 instruction stream.

The hardware needs wait states between some vector instructions (an MFMA and a reader of its result, or a later writer of its C
operand; a transcendental and its reader).  The compiler places them between instructions it knows, but does not look into inline
assembly, so vector instructions written there are the author's responsibility.  This module compiles a kernel source to assembly
and verifies:

1. that no vector instruction is inline assembly (`assembly_vector_instructions`; what is left there are direct loads to LDS,
   barriers and empty statements that pin or hide values), so that the compiler knows all that it has to keep apart;
2. transcendentals (`check_trans_use`): the instruction directly after a `v_exp_f32` (and its kin) does not read its
   result unless it is itself a transcendental or an `s_nop` (one wait state is required on this architecture).

    python -m paper_2510_18121_amd.isa_check            # compiles the attention kernels' sources, prints findings
"""
from __future__ import annotations

import os
import re
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
TRANS = ("v_exp_f32", "v_log_f32", "v_rcp_f32", "v_rsq_f32", "v_sqrt_f32", "v_sin_f32", "v_cos_f32")


def compile_to_asm(source: str) -> str:
    """Device-side assembly of one kernel source, with the flags of the library build."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    with tempfile.TemporaryDirectory() as tmp:
        out = os.path.join(tmp, "k.s")
        cmd = [hipcc, "--offload-arch=gfx950", "-O3", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
               "-packed-fp32-ops", "-Wno-unused-command-line-argument", "-Wno-unknown-attributes", "-Wno-inline-asm",
               "-Wno-int-to-pointer-cast", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-S", "--cuda-device-only",
               "-o", out, os.path.join(CSRC, source)]
        r = subprocess.run(cmd, capture_output=True, text=True)
        if r.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + r.stderr)
        return open(out).read()


def kernel_bodies(asm: str, name_part: str):
    """The instruction streams (label to the function's end: a kernel that returns early has several s_endpgm) of the kernels
    whose mangled name contains name_part."""
    out, cur = [], None
    for line in asm.split("\n"):
        if cur is None:
            if re.match(r"^_Z\w*" + re.escape(name_part) + r"\w*:", line):
                cur = [line]
        else:
            cur.append(line)
            if line.startswith(".Lfunc_end"):
                out.append("\n".join(cur))
                cur = None
    return out


def _vregs(text: str) -> set:
    out = set()
    for m in re.finditer(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b", text):
        if m.group(1):
            out.update(range(int(m.group(1)), int(m.group(2)) + 1))
        else:
            out.add(int(m.group(3)))
    return out


def assembly_vector_instructions(asm: str):
    """The vector ALU and matrix instructions that come from inline assembly."""
    out, inside = [], False
    for line in asm.split("\n"):
        t = line.strip()
        if t.startswith((";;#ASMSTART", ";;#ASMEND")):
            inside = t.startswith(";;#ASMSTART")
        elif inside and t.startswith("v_"):
            out.append(t)
    return out


def check_trans_use(asm: str):
    """Returns (number of transcendental instructions, list of findings)."""
    ins = []
    for line in asm.split("\n"):
        t = line.split(";")[0].strip()
        if t and not t.endswith(":") and not t.startswith(".") and not t.startswith("#"):
            ins.append(t)
    n, bad = 0, []
    for a, b in zip(ins, ins[1:]):
        if not a.split()[0].startswith(TRANS):
            continue
        n += 1
        dst = _vregs(a.split(None, 1)[1].split(",")[0])
        op = b.split()[0]
        if op.startswith(TRANS) or op.startswith("s_nop"):
            continue
        parts = b.split(None, 1)
        if len(parts) < 2:
            continue
        ops = parts[1].split(",")
        reads = set()
        for o in (ops if op.startswith(("v_mfma", "ds_write", "global_store")) else ops[1:]):
            reads |= _vregs(o)
        if dst & reads:
            bad.append((a, b))
    return n, bad


def main():
    status = 0
    for src in ("ca_bwd.hip", "ca_bwd_fused.hip", "ca_fwd.hip"):
        asm = compile_to_asm(src)
        bad = assembly_vector_instructions(asm)
        print(f"{src}: {len(bad)} vector instructions in inline assembly")
        for f in bad:
            print("  ", f)
        nt, badt = check_trans_use(asm)
        print(f"{src}: {nt} transcendental instructions, {len(badt)} findings")
        for f in badt:
            print("  ", *f)
        status |= bool(bad or badt)
    raise SystemExit(status)


if __name__ == "__main__":
    main()
