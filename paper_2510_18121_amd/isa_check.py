"""Static checks of the generated gfx950 instruction stream.

The hardware needs wait states between some vector instructions (an MFMA and a reader of its result, or a later writer of its C
operand; a transcendental and its reader).  The compiler places them between instructions it knows, but does not look into inline
assembly, so vector instructions written there are the author's responsibility.  This module compiles a kernel source to assembly
and verifies:

1. that no vector instruction is inline assembly (`assembly_vector_instructions`; what is left there are direct loads to LDS,
   barriers and empty statements that pin or hide values), so that 2 and 3 have nothing to find;
2. MFMA chains (`check_mfma_chains`): from the first assembly MFMA that writes an architectural tuple with a fresh C operand to
   the end of its chain (an `s_nop 11`, or the `; chain end` marker), nothing but MFMAs touches the chain's registers
   and no control flow intervenes; after a `; chain end` marker no non-MFMA instruction touches those registers for the next 16
   issue cycles at least;
3. operands of assembly MFMAs (`check_mfma_operands`): no vector instruction within two wait states before one writes a
   register it reads;
4. transcendentals (`check_trans_use`): the instruction directly after a `v_exp_f32` (and its kin) does not read its
   result unless it is itself a transcendental or an `s_nop` (one wait state is required on this architecture).

    python -m paper_2510_18121_amd.isa_check            # compiles csrc/ca_bwd.hip and csrc/ca_fwd.hip, prints findings
"""
from __future__ import annotations

import os
import re
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
MFMA = "v_mfma_f32_32x32x16_bf16"
TRANS = ("v_exp_f32", "v_log_f32", "v_rcp_f32", "v_rsq_f32", "v_sqrt_f32", "v_sin_f32", "v_cos_f32")
WINDOW = 16  # issue cycles after a "; chain end" marker in which the chain's registers must stay untouched


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


def check_mfma_chains(asm: str):
    """Returns (number of chains, number of '; chain end' markers, list of findings)."""
    first = re.compile(MFMA + r" v\[(\d+):(\d+)\], .*, (0|v\[(\d+):(\d+)\])$")
    any_v = re.compile(MFMA + r" v\[(\d+):(\d+)\]")
    flow = re.compile(r"(s_cbranch|s_branch|\.LBB|s_endpgm)")
    chain = watch = None
    left = n = marks = 0
    bad = []
    for no, line in enumerate(asm.split("\n"), 1):
        t = line.strip()
        if t.startswith("; chain end"):
            if chain is None:
                bad.append((no, "marker without an open chain"))
            watch, left, chain = chain, WINDOW, None
            marks += 1
            continue
        if not t or t.startswith(";"):
            continue
        if watch is not None:
            if flow.match(t):
                bad.append((no, "control flow inside the window after a chain end: " + t))
                watch = None
            else:
                is_mfma = t.startswith("v_mfma")
                if not is_mfma and _vregs(t) & watch:
                    bad.append((no, "chain registers touched inside the window: " + t))
                m = re.match(r"s_nop (\d+)", t)
                left -= int(m.group(1)) + 1 if m else 8 if is_mfma else 1
                if left <= 0:
                    watch = None
        m = first.match(t)
        if m and m.group(3) != "0" and m.group(4) == m.group(1):
            m = None  # accumulating onto itself: a later link, not a first MFMA
        if m:
            if chain is None:
                chain, n = set(), n + 1
            chain |= set(range(int(m.group(1)), int(m.group(2)) + 1))
            continue
        if chain is not None:
            if t.startswith("s_nop 11"):
                chain = None
            elif flow.match(t):
                bad.append((no, "control flow inside a chain: " + t))
                chain = None
            else:
                m2 = any_v.match(t)
                if m2:
                    chain |= set(range(int(m2.group(1)), int(m2.group(2)) + 1))
                elif _vregs(t) & chain:
                    bad.append((no, "chain registers touched before the chain's end: " + t))
    return n, marks, bad


def check_mfma_operands(asm: str):
    """Returns (number of MFMAs in inline assembly, list of findings)."""
    def regs(text):
        out = set()
        for m in re.finditer(r"\b([va])\[(\d+):(\d+)\]|\b([va])(\d+)\b", text):
            if m.group(1):
                out.update((m.group(1), i) for i in range(int(m.group(2)), int(m.group(3)) + 1))
            else:
                out.add((m.group(4), int(m.group(5))))
        return out

    ins, inside = [], False
    for line in asm.split("\n"):
        t = line.strip()
        if t.startswith((";;#ASMSTART", ";;#ASMEND")):
            inside = t.startswith(";;#ASMSTART")
            continue
        t = t.split(";")[0].strip()
        if t and not t.endswith(":") and not t.startswith("."):
            ins.append((t, inside))
    n, bad = 0, []
    for i, (t, in_asm) in enumerate(ins):
        if not in_asm or not t.startswith("v_mfma"):
            continue
        n += 1
        reads, waited = regs(t.split(",", 1)[1]), 0
        for p, _ in reversed(ins[max(0, i - 2):i]):
            if waited >= 2:
                break
            if p.startswith("v_") and not p.startswith("v_mfma") and regs(p.split(None, 1)[1].split(",")[0]) & reads:
                bad.append((p, t))
            m = re.match(r"s_nop (\d+)", p)
            waited += int(m.group(1)) + 1 if m else 1
    return n, bad


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
    for src in ("ca_bwd.hip", "ca_fwd.hip"):
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
