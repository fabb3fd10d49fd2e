#!/usr/bin/env python3
"""Benchmark of the attention-server hot path on one MI355X.

A step is one pass of the whole path - ca_forward then ca_backward through the C ABI - over one fused
batch of CA-tasks with all inputs already resident in HBM.  The reported value is causal-FLOP
throughput, 14 * head_dim * n_q_heads * (visible query-key pairs) flops per step (2 contractions
forward, 5 backward).  Planning (ca_plan) and allocation are outside the timed region and reported
separately.  Prints ONE JSON line.
"""
from __future__ import annotations

import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_BF16_TFLOPS = 2500.0  # MI355X dense bf16 MFMA peak

# HBM bytes per launch of the backward's main kernel on workload 3 as counted by rocprofv3 (FETCH_SIZE / WRITE_SIZE passes,
# scaled by the plain-copy calibration): NOT measured in a plain run of this script.  The figure of the last counter
# passes over the kernel that ran is quoted under roofline.traffic_profiled with the file it comes from; roofline.traffic itself is null.
TRAFFIC_PROFILED_GIB = {"ca_bwd_fused_kernel": 219.5 + 132.4, "ca_bwd_dkv_kernel": 184.8 + 0.50}


def traffic_profiled(kernel, workload):
    if workload != 3 or kernel not in TRAFFIC_PROFILED_GIB:
        return None
    return {"bytes": int(TRAFFIC_PROFILED_GIB[kernel] * 2**30), "workload": workload,
            "source": "profiles/hot_path_cfg3_hbm_traffic.md"}


class EngineClockSampler:
    """Reads the engine clock (and the package power, where the driver exposes it) from sysfs every 20 ms on a host
    thread while a section of the benchmark runs.  Read-only; every failure just leaves the figures at None."""

    def __init__(self, drm_root="/sys/class/drm"):
        import glob
        self.sclk = next(iter(sorted(glob.glob(drm_root + "/card*/device/pp_dpm_sclk"))), None)
        dev = os.path.dirname(self.sclk) if self.sclk else None
        self.power = next(iter(sorted(glob.glob(dev + "/hwmon/hwmon*/power1_average") +
                                      glob.glob(dev + "/hwmon/hwmon*/power1_input"))), None) if dev else None
        self.temps = sorted(glob.glob(dev + "/hwmon/hwmon*/temp*_input")) if dev else []
        cap = next(iter(sorted(glob.glob(dev + "/hwmon/hwmon*/power1_cap"))), None) if dev else None
        self.power_cap_w = self._read_number(cap, 1e-6)
        self.max_mhz = None
        try:
            self.max_mhz = max(float(l.split(":")[1].lower().replace("mhz", "").replace("*", "").strip())
                               for l in open(self.sclk).read().splitlines() if ":" in l)
        except Exception:
            pass

    @staticmethod
    def _read_number(path, scale):
        try:
            return float(open(path).read().split()[0]) * scale
        except Exception:
            return None

    def _current_mhz(self):
        try:
            for l in open(self.sclk).read().splitlines():
                if "*" in l:
                    return float(l.split(":")[1].lower().replace("mhz", "").replace("*", "").strip())
        except Exception:
            pass
        return None

    def __enter__(self):
        import threading
        self.mhz, self.watts, self.temp_c, self._stop = [], [], [], threading.Event()

        def run():
            while not self._stop.is_set():
                c, w = self._current_mhz(), self._read_number(self.power, 1e-6)
                if c is not None:
                    self.mhz.append(c)
                if w is not None:
                    self.watts.append(w)
                t = [x for x in (self._read_number(f, 1e-3) for f in self.temps) if x is not None]
                if t:
                    self.temp_c.append(max(t))  # the hottest of the sensors the driver lists
                self._stop.wait(0.02)
        self._thread = threading.Thread(target=run, daemon=True)
        if self.sclk:
            self._thread.start()
        return self

    def __exit__(self, *exc):
        self._stop.set()
        if self.sclk:
            self._thread.join()

    def summary(self):
        med = lambda x: sorted(x)[len(x) // 2] if x else None
        return {"engine_clock_mhz_median": med(self.mhz), "engine_clock_mhz_min": min(self.mhz) if self.mhz else None,
                "engine_clock_mhz_max": max(self.mhz) if self.mhz else None, "samples": len(self.mhz),
                "power_w_median": med(self.watts), "power_cap_w": self.power_cap_w,
                "hottest_sensor_c_median": med(self.temp_c)}


def cpu_baseline(index: int):
    """The fp64 oracle, as it stands, timed on this host's cores on a bounded sample of the workload:
    the generator's token-count/8 twin (token-count/32 for the 512K workload) restricted to one KV head's
    query-head group; about ten seconds of work on 16 cores."""
    import numpy as np
    import oracle
    from paper_2510_18121_amd import workloads as W

    b = W.config(index, 1 if index == 1 else 8)
    if index != 1:
        b = W.one_kv_group(b)
    if index == 4:
        b = W.one_kv_group(W.config(4, 32))
    q, k, v, d_o = W.make_tensors(b, "cpu")
    f64 = lambda t: t.float().numpy().astype(np.float64)
    q, k, v, d_o = f64(q), f64(k), f64(v), f64(d_o)
    t0 = time.perf_counter()
    oracle.forward_backward(b, q, k, v, d_o)
    dt = time.perf_counter() - t0
    return {"value": b.flops()["total"] / dt / 1e12, "unit": "TFLOP/s", "cores": oracle.threads(), "kind": "oracle",
            "sample": f"{b.name}: {b.total_q} tokens, {b.n_q_heads}/{b.n_kv_heads} heads, "
                      f"{b.flops()['total']:.3e} causal flops in {dt:.1f} s (fp64)"}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=10)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--workload", type=int, default=3, help="1..5; 3 is the 8B-class 128K-token workload")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--calibration-copy-mib", type=int, default=0,
                    help="after the timed steps, run one plain device copy of this many MiB (a kernel of known "
                         "traffic next to which rocprofv3's FETCH_SIZE / WRITE_SIZE counters are scaled)")
    ap.add_argument("--no-sustained-probe", action="store_true",
                    help="skip the MFMA-only launches that measure the matrix pipes' sustained rate on this device")
    args = ap.parse_args()
    if args.gpus != 1:
        sys.exit("bench.py: this build runs on one GPU only; --gpus N with N > 1 is not supported "
                 "(no collectives or sharding are part of it)")

    import torch
    from paper_2510_18121_amd import binding as B
    from paper_2510_18121_amd import workloads as W

    if not torch.cuda.is_available():
        sys.exit("bench.py: no GPU visible")
    dev = torch.device("cuda:0")
    torch.cuda.set_device(dev)
    props = torch.cuda.get_device_properties(dev)

    b = W.config(args.workload)
    fl = b.flops()
    q, k, v, d_o = W.make_tensors(b, dev)
    # planning (host work + upload of the schedule): the first call in a process also pays for the runtime's first
    # allocations, so it is timed apart from a repeat, which is what a scheduler thread planning every batch sees
    t0 = time.perf_counter()
    plan = B.ca_plan(b)
    torch.cuda.synchronize()
    plan_first_ms = (time.perf_counter() - t0) * 1e3
    t0 = time.perf_counter()
    plan_again = B.ca_plan(b)
    torch.cuda.synchronize()
    plan_ms = (time.perf_counter() - t0) * 1e3
    plan = plan_again  # the first plan is freed here, outside both timings
    ws = B.alloc_workspace(plan, dev)
    o = torch.empty_like(q)
    lse = torch.empty((b.n_q_heads, b.total_q), dtype=torch.float32, device=dev)
    dq, dk, dv = torch.empty_like(q), torch.empty_like(k), torch.empty_like(v)

    def step():
        B.ca_forward(plan, q, k, v, o, lse, ws)
        B.ca_backward(plan, q, k, v, o, d_o, lse, dq, dk, dv, ws)

    for _ in range(args.warmup):
        step()
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    clocks = EngineClockSampler()
    wall0 = time.perf_counter()
    with clocks:
        e0.record()
        for _ in range(args.steps):
            step()
        e1.record()
        torch.cuda.synchronize()
    wall = time.perf_counter() - wall0
    ms_per_step = e0.elapsed_time(e1) / args.steps
    # per-kernel durations: HIP events recorded by the library on the launch stream, in passes of their own (with timing on,
    # small batches run their one backward launch as two)
    plan.profile_enable(True)
    kern = {"fwd_kernel_ms": [], "bwd_prep_ms": [], "bwd_dkv_ms": [], "bwd_dq_ms": []}
    for _ in range(max(1, min(args.steps, 3))):
        step()
        r = plan.profile_read()
        for kk in kern:
            kern[kk].append(r[kk])
    kavg = {kk: sum(vv) / len(vv) for kk, vv in kern.items()}
    plan.profile_enable(False)
    # what the matrix pipes sustain on this device, right after the timed work (chip warm): the library's MFMA-only
    # kernel on N(0,1) bf16 operands, in the attention kernels' shape (16x16x32) and at their two waves per SIMD, three launches
    # of about a quarter second each, the last one reported; then the same with the other work per MFMA issued alongside that the
    # backward kernels and the forward kernel have
    sustained = sustained_side = None
    if not args.no_sustained_probe:
        from paper_2510_18121_amd import mfma_rate
        probe_clocks = EngineClockSampler()
        with probe_clocks:
            sustained = mfma_rate.sustained_tflops("normal", 0, 2, device=dev, shape=16)[-1]
        sustained_side = mfma_rate.sustained_tflops("normal", 1, 2, device=dev, shape=16)[-1]
        sustained_fwd = mfma_rate.sustained_tflops("normal", 2, 2, device=dev, shape=16)[-1]
    if args.calibration_copy_mib > 0:
        src = torch.empty(args.calibration_copy_mib << 20, dtype=torch.uint8, device=dev).fill_(3)
        dst = torch.empty_like(src)
        torch.cuda.synchronize()
        dst.copy_(src)
        torch.cuda.synchronize()

    tflops = fl["total"] / (ms_per_step * 1e-3) / 1e12
    bwd_ms = kavg["bwd_prep_ms"] + kavg["bwd_dkv_ms"] + kavg["bwd_dq_ms"]
    bwd_tflops = fl["bwd"] / (bwd_ms * 1e-3) / 1e12 if bwd_ms > 0 else 0.0
    # the maximum engine clock: from the runtime's device properties, else the highest level the driver lists in sysfs
    clock_mhz = getattr(props, "clock_rate", 0) / 1e3 or clocks.max_mhz or 0.0
    # 4096 dense bf16 flops per clock per CU; None when neither source reports the engine clock
    peak_from_device = props.multi_processor_count * 4096 * clock_mhz * 1e6 / 1e12 if clock_mhz > 0 else None
    # the one-pass kernel executes the backward's 5 contractions: 10*D*Hq*pairs flops; where there are two kernels the dK/dV kernel
    # executes 4 of them (S, dP, dV, dK)
    one_pass = bool(plan.info()["one_pass_backward"]) and ws.numel() >= plan.workspace_bytes_one_pass()
    dkv_flops = fl["bwd"] * (1.0 if one_pass else 0.8)
    kernel = "ca_bwd_fused_kernel" if one_pass else "ca_bwd_dkv_kernel"
    bwd_main_tflops = dkv_flops / (kavg["bwd_dkv_ms"] * 1e-3) / 1e12 if kavg["bwd_dkv_ms"] > 0 else 0.0
    fwd_tflops = fl["fwd"] / (kavg["fwd_kernel_ms"] * 1e-3) / 1e12 if kavg["fwd_kernel_ms"] > 0 else 0.0
    # the dQ kernel executes 3 contractions (S, dP, dQ): 6*D*Hq*pairs flops
    dq_tflops = fl["bwd"] * 0.6 / (kavg["bwd_dq_ms"] * 1e-3) / 1e12 if kavg["bwd_dq_ms"] > 0 and not one_pass else 0.0
    out = {
        "metric": "core-attention fwd+bwd TFLOP/s (causal FLOPs), 1 GPU",
        "value": tflops, "unit": "TFLOP/s", "n_gpus": 1, "steps": args.steps, "warmup": args.warmup,
        "ms_per_step": ms_per_step, "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": "bf16", "data": "synthetic",
        "config": {"workload": b.name, "tokens": b.total_q, "n_q_heads": b.n_q_heads, "n_kv_heads": b.n_kv_heads,
                   "head_dim": b.head_dim, "docs": b.n_docs, "ca_tasks": b.n_tasks, "pairs": fl["pairs"],
                   "flops_fwd_bwd": fl["total"]},
        # against the peak read from the device (CUs x 4096 flop/clk x maximum engine clock); the published 2500 when
        # the device reports no clock
        "pct_of_bf16_mfma_peak": 100.0 * tflops / (peak_from_device or PEAK_BF16_TFLOPS),
        "pct_peak_denominator_tflops": peak_from_device or PEAK_BF16_TFLOPS,
        "device": {"name": props.name, "cus": props.multi_processor_count, "clock_mhz": clock_mhz,
                   "peak_bf16_tflops_from_device": peak_from_device, "during_timed_steps": clocks.summary()},
        "kernels_ms": kavg, "fwd_only_tflops": fwd_tflops, "bwd_only_tflops": bwd_tflops, "plan_ms": plan_ms, "plan_first_call_ms": plan_first_ms,
        "wall_s_timed": wall,
        "roofline": {"kernel": kernel, "bound": "mfma", "achieved": bwd_main_tflops,
                     "peak": PEAK_BF16_TFLOPS, "unit": "TFLOP/s", "frac": bwd_main_tflops / PEAK_BF16_TFLOPS,
                     "traffic": None,
                     "traffic_profiled": traffic_profiled(kernel, args.workload)},
    }
    # The metric credits 14*D flops per (pair, head), which is what the one pass executes; where there are two backward kernels they
    # execute 18*D (both recompute S and dP).  Executed rate next to the rate of back-to-back MFMAs measured in this run:
    executed = (fl["fwd"] + (1.0 if one_pass else 1.4) * fl["bwd"]) / (ms_per_step * 1e-3) / 1e12
    out["executed_tflops"] = executed
    if sustained is not None:
        out["roofline"]["sustained_mfma"] = {
            "tflops": sustained, "frac": bwd_main_tflops / sustained,
            "during_probe": probe_clocks.summary(), "with_side_work_tflops": sustained_side,
            "frac_with_side_work": bwd_main_tflops / sustained_side,
            "other_kernels": {
                "ca_fwd_kernel": {"executed_tflops": fwd_tflops, "stream_side_work_2_tflops": sustained_fwd,
                                  "frac": fwd_tflops / sustained_fwd},
                **({} if one_pass else {"ca_bwd_dq_kernel": {
                    "executed_tflops": dq_tflops, "stream_side_work_1_tflops": sustained_side, "frac": dq_tflops / sustained_side}})},
            "what": "ca_mfma_stream16 in this run after the timed steps: v_mfma_f32_16x16x32_bf16 back to back from registers, "
                    "N(0,1) bf16 operands, two waves per SIMD on all CUs; with_side_work and side_work_1 add one 16-byte LDS "
                    "read per lane and two multiply-adds per two MFMAs and an exponential per four, side_work_2 four "
                    "multiply-adds and an exponential per two and a read per four"}
    if not args.no_cpu_baseline:
        out["cpu_baseline"] = cpu_baseline(args.workload)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
