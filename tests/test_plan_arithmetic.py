"""Planner: no division by zero on its way to a plan (no GPU).  The planner is compiled with the host compiler's check for
floating-point divisions by zero, which ends the process at the first one, and plans batches whose documents have resident
keys beyond their last query row: their KV tiles are units without a single step."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CXX = shutil.which("g++")
pytestmark = pytest.mark.skipif(CXX is None, reason="needs g++")

PLAN_BATCHES = """
import ctypes, sys
sys.path.insert(0, sys.argv[1])
from paper_2510_18121_amd import binding as B, workloads as W
B.lib()  # declares the argument types; then the checked planner takes its place
lib = ctypes.CDLL(sys.argv[2])
lib.ca_plan_host.argtypes = B.lib().ca_plan_host.argtypes
lib.ca_plan_destroy_host.argtypes = [ctypes.c_void_p]
for docs, tasks, hq, hkv, d in (([20000], [(0, 0, 3000)], 4, 2, 128), ([65536], [(0, 0, 2048)], 8, 2, 128),
                                ([9000, 500], [(0, 17, 1300), (1, 0, 500)], 8, 1, 64), ([300], [], 4, 2, 64),
                                ([4096], [(0, 0, 4096)], 32, 8, 128)):
    keep, h = [], ctypes.c_void_p()
    desc = B.make_desc(W.custom(docs, tasks, hq, hkv, d), keep)
    assert lib.ca_plan_host(ctypes.byref(desc), ctypes.byref(h)) == 0
    lib.ca_plan_destroy_host(h)
print("planned")
"""


def test_planning_divides_by_no_zero(tmp_path):
    out = str(tmp_path / "planner.so")
    csrc = os.path.join(ROOT, "paper_2510_18121_amd", "csrc")
    main = tmp_path / "planner.cpp"  # the planner, and a destructor for its plans (the library's own also frees device memory)
    main.write_text('#include "ca_plan.cpp"\nextern "C" void ca_plan_destroy_host(ca_plan_t *p) { delete p; }\n')
    subprocess.run([CXX, "-O1", "-std=c++17", "-shared", "-fPIC", "-fsanitize=float-divide-by-zero", "-fno-sanitize-recover=all",
                    "-I", csrc, "-I", os.path.join(ROOT, "include"), "-o", out, str(main)], check=True)
    r = subprocess.run([sys.executable, "-c", PLAN_BATCHES, ROOT, out], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "planned" in r.stdout, r.stderr[-2000:]
