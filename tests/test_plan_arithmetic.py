"""Planner: no division by zero on its way to a plan, and the simulation of the list scheduling its rules rest on (no GPU).  The
planner is compiled with the host compiler's check for floating-point divisions by zero, which ends the process at the first
one, and plans batches whose documents have resident keys beyond their last query row: their KV tiles are units without a
single step."""
import ctypes
import heapq
import os
import shutil
import subprocess
import sys

import numpy as np
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


@pytest.fixture(scope="module")
def planner(tmp_path_factory):
    """The planner with that check, with a destructor for its plans (the library's own also frees device memory) and with its
    simulation exported."""
    tmp = tmp_path_factory.mktemp("planner")
    out, main = str(tmp / "planner.so"), tmp / "planner.cpp"
    main.write_text('#include "ca_plan.cpp"\nextern "C" void ca_plan_destroy_host(ca_plan_t *p) { delete p; }\n'
                    'extern "C" double simulate(const double *us, const int64_t *n, int64_t k, int64_t cus, double at_most) {\n'
                    "  std::vector<std::pair<double, int64_t>> u;\n  for (int64_t i = 0; i < k; ++i) u.push_back({us[i], n[i]});\n"
                    "  return ca::makespan(u, cus, at_most, 512);\n}\n"
                    'extern "C" int64_t within(const ca_plan_t *p, int64_t *out) {\n'
                    "  const ca_plan_t *s = p->within_static.get();\n  if (!s) return 0;\n"
                    "  const int64_t v[6] = {int64_t(s->ws_bwd), int64_t(s->ws_bwd_split), int64_t(p->ws_bwd_split), s->n_fwd_parts, s->n_bwd_parts,\n"
                    "                        int64_t(s->bwd_units.size()) - int64_t(p->bwd_units.size())};\n"
                    "  for (int i = 0; i < 6; ++i) out[i] = v[i];\n  return 1;\n}\n")
    csrc = os.path.join(ROOT, "paper_2510_18121_amd", "csrc")
    subprocess.run([CXX, "-O1", "-std=c++17", "-shared", "-fPIC", "-fsanitize=float-divide-by-zero", "-fno-sanitize-recover=all",
                    "-I", csrc, "-I", os.path.join(ROOT, "include"), "-o", out, str(main)], check=True)
    return out


def test_planning_divides_by_no_zero(planner):
    r = subprocess.run([sys.executable, "-c", PLAN_BATCHES, ROOT, planner], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "planned" in r.stdout, r.stderr[-2000:]


def list_schedule(units, cus):
    busy, end = [0.0] * cus, 0.0
    for us, n in units:
        for _ in range(n):
            t = heapq.heappop(busy) + us
            heapq.heappush(busy, t)
            end = max(end, t)
    return end


@pytest.mark.parametrize("seed", range(12))
def test_simulated_list_schedule(planner, seed):
    """Up to 512 units: the list schedule itself.  Longer lists are simulated with neighbours taken together: every CU's last
    unit may then end up to a unit's length earlier or later, and the list's mean load stays what it is."""
    lib = ctypes.CDLL(planner)
    lib.simulate.restype = ctypes.c_double
    lib.simulate.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int64, ctypes.c_int64, ctypes.c_double]
    rng = np.random.default_rng(seed)
    cus = int(rng.choice([256, 512, 128, 32, 2]))
    for total in (3, 200, 500, 3000):
        us, n = [], []
        while sum(n) < total:
            us.append(float(12 + 1.75 * rng.integers(0, 400)))
            n.append(int(min(total - sum(n), rng.integers(1, 9))))
        us = np.sort(np.asarray(us))[::-1].copy()
        n = np.asarray(n, np.int64)
        want = list_schedule(list(zip(us.tolist(), n.tolist())), cus)
        got = lib.simulate(us.ctypes.data, n.ctypes.data, len(us), cus, 1e30)
        if total <= 512:
            assert got == want, (seed, total, cus)
        else:
            mean = float((us * n).sum()) / cus
            assert max(0.99 * mean, us[0]) <= got and abs(got - want) <= 0.03 * want, (seed, total, cus, got, want)
        assert lib.simulate(us.ctypes.data, n.ctypes.data, len(us), cus, 0.5 * got) >= 0.5 * got


def test_plan_inside_the_static_workspace(planner):
    """Where partial results go beyond the static workspace, which whole units fit, the plan holds another one that stays inside."""
    from paper_2510_18121_amd import binding as B
    from paper_2510_18121_amd import workloads as W

    lib, static = ctypes.CDLL(planner), B.lib().ca_static_workspace_bytes()
    lib.ca_plan_host.argtypes = B.lib().ca_plan_host.argtypes
    lib.within.restype, lib.within.argtypes = ctypes.c_int64, [ctypes.c_void_p, ctypes.c_void_p]
    lib.ca_plan_destroy_host.argtypes = [ctypes.c_void_p]
    seen = 0
    for n, hq, hkv, d in ((6000, 8, 1, 128), (9000, 8, 1, 128), (15800, 8, 1, 128), (16500, 8, 1, 128), (1900, 64, 8, 128), (26000, 8, 1, 64)):
        keep, h = [], ctypes.c_void_p()
        desc = B.make_desc(W.custom([n], [(0, 0, n)], hq, hkv, d), keep)
        assert lib.ca_plan_host(ctypes.byref(desc), ctypes.byref(h)) == 0
        out = np.zeros(6, np.int64)
        if lib.within(h, out.ctypes.data):
            seen += 1
            base, inside, beyond, _, _, units = out.tolist()
            assert base <= inside <= static < beyond <= base + (256 << 20) and units == 0
        lib.ca_plan_destroy_host(h)
    assert seen >= 3
