#!/usr/bin/env python3
"""Benchmark: deep Pauli-exponential circuit at 21 qubits on one MI355X.

Workload (one step): start from |0...0>, apply the 50,000-exponential
circuit (about 4.5e5 input gates: basis change, CNOT ladder, Rz, uncompute;
the synthetic stand-in for the paper's 21-qubit P9-P15 circuits, Section 5.1
Table 5), then evaluate <H> of a 100-term random Pauli sum in FP64.
The circuit is compiled (fusion + pass plan) once and its operator tables
are resident in HBM before the timed region, like the state.

Prints one JSON line: input gates/s, the achieved bandwidth of the dominant
kernel (span pass) against HBM peak, and the CPU oracle's rate on a bounded
prefix of the same circuit.
"""
from __future__ import annotations

import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0
# LDS: 128 bytes per clock per CU (32 banks of 4 bytes), 256 CUs at 2.4 GHz
LDS_PEAK_GBS = 128 * 256 * 2.4

# HBM bytes per launch of k_span at 21 qubits, from two counter runs of this
# benchmark (rocprofv3 --pmc FETCH_SIZE, then WRITE_SIZE; KiB per dispatch).  A
# plain device copy dispatch of 256 MiB reads FETCH_SIZE = 131,084 KiB and
# WRITE_SIZE = 262,144 KiB, so fetches scale by 2.0 and writes by 1.0.
# The figures hold for the kernel sources with the hash below (see
# kernel_source_hash); for any other source the traffic is reported as null.
MEASURED_TRAFFIC = {
    "kernels_sha256_16": "39d06d2581eeca87",
    "complex128": (16512.4 * 2.0 + 33698.4) * 1024,
    "complex64": (8325.2 * 2.0 + 16461.3) * 1024,
}


KERNEL_SOURCES = ("kernels.hip", "span.hip", "device.h", "launch.h", "swizzle.h", "host.h")


def kernel_source_hash():
    """sha256 prefix over the sources the kernels are compiled from."""
    import hashlib
    h = hashlib.sha256()
    for name in KERNEL_SOURCES:
        with open(os.path.join(ROOT, "paper_2310_17739_amd", "csrc", name), "rb") as f:
            h.update(f.read())
    return h.hexdigest()[:16]


def measured_traffic(dtype):
    return MEASURED_TRAFFIC.get(dtype) if kernel_source_hash() == MEASURED_TRAFFIC["kernels_sha256_16"] else None


WORKLOAD_TEXT = {"pauli": "{} Pauli-string exponentials",
                 "dense": "{} brick-wall layers of Haar-random two-qubit unitaries",
                 "dense5": "{} Haar-random 5-qubit unitaries on random qubits"}


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def cpu_baseline(n, g, target_s=12.0, target_1t_s=6.0):
    """The oracle (FP64, one gate at a time) on a prefix of the circuit, timed
    on the host's cores with OpenMP over the amplitude loop, then on one
    thread."""
    import oracle

    def timed(target):
        # calibrate on a short prefix, then time a prefix of about `target` s
        k = 100
        t0 = time.perf_counter()
        oracle.run(n, g[:k])
        dt = time.perf_counter() - t0
        k2 = int(min(len(g), max(k, k * target / max(dt, 1e-3))))
        t0 = time.perf_counter()
        oracle.run(n, g[:k2])
        return k2, time.perf_counter() - t0

    model = ""
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    cores = oracle.set_threads(0)
    k_all, dt_all = timed(target_s)
    oracle.set_threads(1)
    k_1, dt_1 = timed(target_1t_s)
    oracle.set_threads(cores)
    return {"value": k_all / dt_all, "unit": "gates/s", "cores": cores, "kind": "oracle",
            "sample": f"first {k_all} of {len(g)} gates of the same {n}-qubit circuit, FP64, "
                      f"{dt_all:.1f} s wall, OpenMP over the amplitude loop on {cores} threads ({model})",
            "single_thread": {"value": k_1 / dt_1, "unit": "gates/s", "cores": 1,
                              "sample": f"first {k_1} gates, {dt_1:.1f} s wall"}}


def pct(xs, q):
    import numpy as np
    return float(np.percentile(np.asarray(xs), q)) if len(xs) else None


def copy_ceiling(qsim, buf, reps=200):
    """Same-footprint ceilings of a tile pass over the state buffer `buf`,
    from the library's streaming-copy kernel run in place (bytes read plus
    bytes written per second, averaged over `reps` back-to-back launches):

    * stable: every 64 KiB block goes to the same workgroup (and XCD) on
      every launch, so a block written by one launch is read back from that
      XCD's L2 by the next;
    * rotated: each launch hands every block to the next workgroup, so
      blocks move between XCDs from launch to launch, as the tiles of
      successive passes over different qubit sets do;

    each with plain and with non-temporal loads and stores."""
    import torch
    nbytes = buf.numel() * buf.element_size()
    stream = torch.cuda.current_stream()
    out = {}
    for nt in (0, 1):
        for rot in (0, 1):
            for i in range(5):
                qsim.qsim_stream_copy(buf, buf, flags=nt, rotate=i * rot)
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record(stream)
            for i in range(reps):
                qsim.qsim_stream_copy(buf, buf, flags=nt, rotate=i * rot)
            b.record(stream)
            torch.cuda.synchronize()
            out[("nt_" if nt else "plain_") + ("rotated" if rot else "stable")] = \
                2 * nbytes * reps / (a.elapsed_time(b) * 1e-3) / 1e9
    out["best_stable"] = max(out["plain_stable"], out["nt_stable"])
    out["best_rotated"] = max(out["plain_rotated"], out["nt_rotated"])
    return out


FIXTURE = os.path.join(ROOT, "tests", "golden", "cfg2_21q_50k_oracle.npz")


def oracle_distance(W, psi, energy, H):
    """Against the oracle's stored results for the 21-qubit, 50,000-exponential
    circuit (written by tests/golden/make_cfg2_fixture.py, which runs only the
    oracle): the estimate of ||psi/|psi| - phi/|phi|||^2 from 48 seeded
    Gaussian probe overlaps (an upper bound of the infidelity of two unit
    states, up to the estimate's spread) and |<H> - <H>_oracle| / sum|c|."""
    import numpy as np
    fx = np.load(FIXTURE)
    a = np.asarray(psi, dtype=np.complex128)
    na = np.sqrt(np.vdot(a, a).real)
    nb = np.sqrt(float(fx["norm"]))
    acc = 0.0
    for k, r in enumerate(W.probe_vectors(int(fx["n"]), len(fx["probe"]))):
        acc += abs(np.vdot(r, a) / na - fx["probe"][k] / nb) ** 2
    d2 = acc / (2.0 * len(fx["probe"]))
    idx = fx["sample_idx"]
    amp = np.abs(a[idx] / na - fx["sample_amp"] / nb).max()
    return {"distance2_estimate": d2, "probes": int(len(fx["probe"])),
            "max_sampled_amplitude_error": float(amp),
            "dexpval_over_sum_abs_c": abs(energy - float(fx["energy"])) / float(np.abs(H["coeff"]).sum()),
            "oracle_energy": float(fx["energy"])}


def runs_as_rotations(stats):
    """Passes of rotations take none of the paper's fusion steps."""
    return stats["ops_after"][1] == -1


def flops_per_amplitude(stats):
    """Arithmetic of one run: in tiled passes a complex multiply-add (8 flops) per
    XOR-shift term of every operator; in passes of rotations two real multiply-adds
    per rotation (a controlled one takes four: these are counted low)."""
    return 4.0 * stats["fused_ops"] if runs_as_rotations(stats) else 8.0 * stats["terms"]


def run_trajectories(qsim, W, ntraj=1024, rounds=500):
    """Mid-circuit measurement form: 12 system + 2 ancilla qubits, complex64
    states with FP64 reductions, `rounds` rounds of gates + 2 measurements +
    2 resets, one trajectory per state, decisions on the device."""
    import numpy as np
    import torch
    g = W.trajectory_round_program(12, rounds, seed=4)
    u = W.uniforms((ntraj, 2 * rounds), seed=5)
    b = qsim.Batch([{"n": 14, "n_states": ntraj, "gates": g, "uniforms": u, "n_slots": 2 * rounds}],
                   dtype="complex64", use_graph=True)
    b.qsim_batch_run()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    b.qsim_batch_run()
    res = b.qsim_batch_results(0)
    dt = time.perf_counter() - t0
    info = b.qsim_batch_info()
    gs = b.qsim_batch_group_stats(0)
    b.close()
    p = res["probs"]
    # The 128 KiB state stays in one workgroup for the whole pass.  In tiled passes
    # every operator reads and writes the state in LDS once, and so does each
    # measurement or reset record (a reset that follows a measurement of its qubit
    # runs inside that measurement's record); passes of rotations do so once per
    # re-layout and keep it in registers in between.
    trips = gs["reg_relayouts"] if runs_as_rotations(gs) else info["fused_ops"] + info["records"]
    lds_bytes = ntraj * trips * 2 * 8 * (1 << 14)
    flops = ntraj * flops_per_amplitude(gs) * (1 << 14)
    return {"workload": f"{ntraj} trajectories x {rounds} rounds, 14 qubits, complex64",
            "seconds": dt, "trajectory_rounds_per_s": ntraj * rounds / dt,
            "input_gates_per_s": ntraj * len(g) / dt, "passes": info["passes"],
            "fused_ops_per_trajectory": info["fused_ops"], "records_per_trajectory": info["records"],
            "lds": {"bytes": lds_bytes, "achieved_GBps": lds_bytes / dt / 1e9, "peak_GBps": LDS_PEAK_GBS,
                    "frac": lds_bytes / dt / 1e9 / LDS_PEAK_GBS},
            # (see flops_per_amplitude) vector FP32 without packed instructions
            # peaks at the FP64 rate, 78.6 TFLOP/s
            "alu": {"flops": flops, "achieved_TFLOPs": flops / dt / 1e12, "peak_TFLOPs": 78.6,
                    "frac": flops / dt / 1e12 / 78.6},
            "failed": int((res["status"] != 0).sum()),
            "mean_p_outcome": float(p.mean()), "norm_max_dev": float(np.abs(res["norms"] - 1).max())}


def run_batched(qsim, W, n_circuits=4096, n_exp=500, sample_one_at_a_time=48):
    """Batched form: circuits of width U{10..20}, each a 500-exponential
    template with its own angles, complex64 with FP64 <H>, one graph launch;
    against the same circuits one at a time in complex128 on the same GPU."""
    import numpy as np
    import torch
    tmpl = W.batch_templates(10, 20, n_exp, 100)
    widths, thetas = W.batch_instances(n_circuits, 10, 20, n_exp)
    groups, index = [], []
    for w in range(10, 21):
        sel = np.nonzero(widths == w)[0]
        if len(sel) == 0:
            continue
        g, H = tmpl[w]
        groups.append({"n": w, "n_states": len(sel), "gates": g, "params": thetas[sel], "terms": H})
        index.append(sel)
    t0 = time.perf_counter()
    b = qsim.Batch(groups, dtype="complex64", use_graph=True, autotune=True)
    create_s = time.perf_counter() - t0
    gstats = [b.qsim_batch_group_stats(gi) for gi in range(len(groups))]
    widths_tuned = {int(gd["n"]): gs["tuned_width"] for gd, gs in zip(groups, gstats)}
    tiles_tuned = {int(gd["n"]): gs["tile_qubits"] for gd, gs in zip(groups, gstats)}
    t0 = time.perf_counter()
    b.qsim_batch_run()
    torch.cuda.synchronize()
    first_s = time.perf_counter() - t0
    times = []
    for _ in range(3):
        t0 = time.perf_counter()
        b.qsim_batch_run()
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t0)
    ev = np.zeros(n_circuits)
    for gi, sel in enumerate(index):
        ev[sel] = b.qsim_batch_results(gi)["expvals"]
    info = b.qsim_batch_info()
    b.close()
    best = min(times)
    # one circuit at a time, complex128, on a seeded sample: each circuit is
    # compiled (angles bound on the host, fusion, plan) and then run with
    # its <H>; compile and device time are kept apart so that both sides
    # can be compared with and without their host preparation
    rng = np.random.default_rng(11)
    pick = rng.choice(n_circuits, size=min(sample_one_at_a_time, n_circuits), replace=False)
    diffs = []
    compile_s = run_s = 0.0
    torch.cuda.synchronize()
    for c in pick:
        w = int(widths[c])
        g, H = tmpl[w]
        t0 = time.perf_counter()
        prog = qsim.Program(w, g, "complex128", params=thetas[c])
        t1 = time.perf_counter()
        sv = qsim.StateVector(w, "complex128")
        torch.cuda.synchronize()
        t2 = time.perf_counter()
        prog.qsim_run(sv)
        e = sv.qsim_expval(H)
        t3 = time.perf_counter()
        compile_s += t1 - t0
        run_s += t3 - t2
        diffs.append(abs(e - ev[c]) / np.abs(H["coeff"]).sum())
        prog.close()
        sv.close()
    one_run = run_s / len(pick)
    one_all = (run_s + compile_s) / len(pick)
    return {"workload": f"{n_circuits} circuits, widths U{{10..20}}, {n_exp} exponentials each, own angles, "
                        "complex64 + FP64 <H>, one HIP-graph launch",
            "circuits_per_s": n_circuits / best, "seconds": best, "create_s": create_s,
            "first_run_s": first_s,
            "circuits_per_s_with_create": n_circuits / (create_s + first_s),
            "state_bytes": info["state_bytes"], "passes": info["passes"],
            "tuned_fusion_width_by_qubits": widths_tuned, "tile_qubits_by_qubits": tiles_tuned,
            "tune_s": info["tune_seconds"],
            "one_at_a_time_c128_circuits_per_s": 1.0 / one_run,
            "one_at_a_time_c128_circuits_per_s_with_compile": 1.0 / one_all,
            "one_at_a_time_sample": int(len(pick)),
            "speedup_vs_one_at_a_time_c128": (n_circuits / best) * one_run,
            "speedup_with_host_preparation_on_both_sides": (n_circuits / (create_s + first_s)) * one_all,
            "max_rel_dexpval_vs_c128": float(max(diffs))}


def run_served(qsim, W, n_requests=48, loads=(0.5, 0.8, 1.0), wmax=30, n_compare=16, wcompare=24):
    """Serving form: requests with log-uniform widths 12..wmax and depths
    10^3..10^5 gates of the Pauli-exponential style, complex64, 8 slots, pool
    admission by state bytes.  First a closed-loop run (all requests at once)
    calibrates capacity; then Poisson arrivals at each offered load x capacity,
    each on its own request set; latency is completion - arrival.  Last, on
    requests of width <= wcompare, the served complex64 path against the plain
    one-circuit-at-a-time complex128 path on the same requests."""
    import numpy as np
    import torch
    nsets = 1 + len(loads)
    reqs = W.serving_requests(nsets * n_requests, 12, wmax, rate=1.0, seed=8)
    circuits = [(r["width"], W.request_circuit(r), W.pauli_sum(r["width"], 20, seed=r["seed"])) for r in reqs]

    def serve(batch, arrivals):
        srv = qsim.Server(dtype="complex64", slots=8, compile_threads=8, pool_bytes=48 << 30)
        t0 = srv.qsim_server_clock()
        ids = {}
        done = {}
        for (w, g, H), a in zip(batch, arrivals):
            while srv.qsim_server_clock() < t0 + a:
                for r in srv.qsim_server_poll(wait_ms=0):
                    done[r["id"]] = r
                time.sleep(0.0005)
            ids[srv.qsim_server_submit(w, g, terms=H)] = w
        while len(done) < len(ids):
            for r in srv.qsim_server_poll(wait_ms=100):
                done[r["id"]] = r
        st = srv.qsim_server_stats()
        srv.close()
        lat = [r["t_done"] - r["t_submit"] for r in done.values()]
        span = max(r["t_done"] for r in done.values()) - t0
        bad = sum(1 for r in done.values() if r["status"] != 0)
        return {"circuits_per_s": len(done) / span, "p50_s": pct(lat, 50), "p99_s": pct(lat, 99),
                "failed": bad, "pool_peak_bytes": st["pool_peak"]}, {i: done[i] for i in done}

    cap, _ = serve(circuits[:n_requests], [0.0] * n_requests)
    rng = np.random.default_rng(9)
    runs = []
    for j, load in enumerate(loads):
        rate = load * cap["circuits_per_s"]
        gaps = rng.exponential(1.0 / rate, size=n_requests)
        batch = circuits[(j + 1) * n_requests:(j + 2) * n_requests]
        res, _ = serve(batch, list(np.cumsum(gaps)))
        runs.append(dict(res, load=load, offered_per_s=rate))
    # served complex64 vs one-at-a-time complex128 on the same small requests
    small = [c for c in circuits if c[0] <= wcompare][:n_compare]
    served_small, got = serve(small, [0.0] * len(small))
    t0 = time.perf_counter()
    e128 = []
    for (w, g, H) in small:
        prog = qsim.Program(w, g, "complex128")
        sv = qsim.StateVector(w, "complex128")
        prog.qsim_run(sv)
        e128.append(sv.qsim_expval(H))
        prog.close()
        sv.close()
    torch.cuda.synchronize()
    one_s = time.perf_counter() - t0
    e64 = [got[i]["expval"] for i in sorted(got)]
    scale = [float(np.abs(H["coeff"]).sum()) for (_, _, H) in small]
    dmax = max(abs(a - b) / sc for a, b, sc in zip(e64, e128, scale))
    widths = [c[0] for c in circuits]
    depths = [len(c[1]) for c in circuits]
    return {"workload": f"{nsets} sets of {n_requests} requests, widths log-U[12,{wmax}] (max {max(widths)}), "
                        f"depths {min(depths)}..{max(depths)} gates, complex64, 8 slots, HBM-byte admission",
            "capacity": cap, "poisson": runs,
            "vs_one_at_a_time_c128": {"requests": len(small), "max_width": max(c[0] for c in small),
                                      "served_c64_circuits_per_s": served_small["circuits_per_s"],
                                      "one_at_a_time_c128_circuits_per_s": len(small) / one_s,
                                      "speedup": served_small["circuits_per_s"] / (len(small) / one_s),
                                      "max_dexpval_over_sum_abs_c": dmax}}


def run_mma(qsim, W, n_sys=20, steps=8, shots=1024, delta=0.3, dtype="complex128"):
    """Measurement assertion (Section 4.3) against shot-by-shot measurement,
    on the projection-filter workload (one ancilla, n_sys system qubits,
    synthetic diagonal Hamiltonian, t_i = t_(i-1)/2).

    MMA: one state; after each step the ancilla is asserted to 0 (its
    probability tracked) and reset; then all shots are drawn from the final
    state at once.  It runs as a one-state batch program with the assertions
    decided on the device, compiled once before the timed run like the
    shot-by-shot batch; the same chain through the synchronous single-state
    calls (qsim_apply per step, compile included, qsim_measure_assert and
    qsim_reset) is timed as well.  Shot by shot: `shots` trajectories in one
    batch, the ancilla measured with a draw after every step; a shot
    succeeds when every outcome is 0.  In the shape of the paper's Table 6,
    the report gives, per step, the asserted probability against the
    observed rate among the shots still successful."""
    import numpy as np
    import torch
    ga, info = W.projection_filter(n_sys, steps, seed=12, record="assert", delta=delta)
    gm, _ = W.projection_filter(n_sys, steps, seed=12, record="measure", delta=delta)
    n = info["n"]
    cuts = [i for i in range(len(ga)) if ga["kind"][i] == W.KIND_ASSERT0]
    # the single-state calls, one host round trip per assertion
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    sv = qsim.StateVector(n, dtype)
    p_host = []
    prev = 0
    for c in cuts:
        sv.qsim_apply(ga[prev:c])
        p_host.append(sv.qsim_measure_assert(0))
        sv.qsim_reset(0)
        prev = c + 2
    sv.qsim_sample(W.uniforms(shots, seed=13))
    torch.cuda.synchronize()
    t_host = time.perf_counter() - t0
    sv.close()
    # the device-side program: the batch runs in place on the state that
    # the sampler then reads
    tdt = torch.complex128 if dtype == "complex128" else torch.complex64
    psi = torch.empty(1 << n, dtype=tdt, device="cuda")
    sv = qsim.StateVector(n, dtype, tensor=psi)
    bm = qsim.Batch([{"n": n, "n_states": 1, "gates": ga, "n_slots": steps, "states": psi}], dtype=dtype)
    bm.qsim_batch_run()                      # warm-up, as for the shots
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    bm.qsim_batch_run()
    drawn = sv.qsim_sample(W.uniforms(shots, seed=13))
    torch.cuda.synchronize()
    t_mma = time.perf_counter() - t0
    resm = bm.qsim_batch_results(0)
    bm.close()
    sv.close()
    p_steps = [float(x) for x in resm["probs"][0]]
    p_dev_vs_host = max(abs(a - b) for a, b in zip(p_steps, p_host))
    b = qsim.Batch([{"n": n, "n_states": shots, "gates": gm, "uniforms": W.uniforms((shots, steps), seed=14),
                     "n_slots": steps}], dtype=dtype)
    b.qsim_batch_run()                       # warm-up (and graph-free)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    b.qsim_batch_run()
    torch.cuda.synchronize()
    t_shots = time.perf_counter() - t0
    res = b.qsim_batch_results(0)
    b.close()
    outc = res["outcomes"]
    alive = np.ones(shots, dtype=bool)
    table = []
    for i in range(steps):
        at_risk = int(alive.sum())
        zeros = int((alive & (outc[:, i] == 0)).sum())
        table.append({"step": i + 1, "asserted_p": p_steps[i], "shots_at_risk": at_risk,
                      "observed_zero": zeros, "expected_zero": at_risk * p_steps[i]})
        alive &= outc[:, i] == 0
    ptrack = float(np.prod(p_steps))
    k = int(alive.sum())
    sd = (shots * ptrack * (1 - ptrack)) ** 0.5
    return {"workload": f"projection filter, {n} qubits ({n_sys} system + 1 ancilla), {steps} steps, "
                        f"delta={delta}, {dtype}, {shots} shots",
            "mma": {"seconds": t_mma, "tracked_probability": ptrack, "shots_drawn": int(len(drawn)),
                    "ancilla_zero_in_all_drawn": bool((np.asarray(drawn) & 1 == 0).all()),
                    "status": int(resm["status"][0]),
                    "host_calls_seconds": t_host, "max_dp_device_vs_host_calls": p_dev_vs_host},
            "shot_by_shot": {"seconds": t_shots, "successful": k, "expected": shots * ptrack,
                             "z": (k - shots * ptrack) / sd if sd > 0 else 0.0,
                             "failed_status": int((res["status"] != 0).sum())},
            "speedup_mma_vs_shots": t_shots / t_mma, "speedup_host_calls_vs_shots": t_shots / t_host,
            "per_step": table}


def run_wide_job(qsim, W, n=30, n_exp=40000):
    """One 30-qubit complex64 job (8 GiB state, HBM-bound passes): about
    10^4 tile passes.  Beside HBM peak, the rate of a plain device copy of the
    same footprint (read 8 GiB, write 8 GiB) is reported as a ceiling, timed
    before and after the job (the job runs for tens of seconds)."""
    import torch
    g, _, _ = W.pauli_exponential_circuit(n, n_exp, seed=31)
    prog = qsim.Program(n, g, "complex64")
    st = prog.qsim_program_stats()
    sv = qsim.StateVector(n, "complex64")
    src = sv.tensor.view(torch.int64)
    dst = torch.empty_like(src)

    def copy_rate():
        dst.copy_(src)
        torch.cuda.synchronize()
        c0 = time.perf_counter()
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        return 2 * src.numel() * src.element_size() / ((time.perf_counter() - c0) / 3) / 1e9

    ceil = copy_ceiling(qsim, sv.tensor.view(torch.int64), reps=3)
    copy_before = copy_rate()
    sv.qsim_init_zero()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    prog.qsim_run(sv)
    torch.cuda.synchronize()
    dt = time.perf_counter() - t0
    nrm = sv.qsim_norm()
    copy_after = copy_rate()
    prog.close()
    del dst
    sv.close()
    pass_bytes = 2 * 8 * (1 << n)
    gbs = pass_bytes * st["passes"] / dt / 1e9
    return {"workload": f"{n} qubits, {n_exp} exponentials ({st['input_gates']} gates), complex64",
            "passes": st["passes"], "tile_qubits": st["tile_qubits"], "seconds": dt,
            "gates_per_s": st["input_gates"] / dt, "avg_pass_ms": 1e3 * dt / st["passes"], "pass_GBps": gbs,
            "frac_of_hbm_peak": gbs / HBM_PEAK_GBS, "stream_copy_GBps": ceil,
            "frac_of_stream_copy": gbs / max(ceil["best_stable"], ceil["best_rotated"]),
            "torch_copy_GBps_before": copy_before, "torch_copy_GBps_after": copy_after, "norm": nrm}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--dtype", default="complex128", choices=["complex128", "complex64"])
    ap.add_argument("--qubits", type=int, default=21)
    ap.add_argument("--n-exp", type=int, default=50_000)
    ap.add_argument("--workload", default="pauli", choices=["pauli", "dense", "dense5"],
                    help="pauli: the Pauli-exponential circuit; dense: brick-wall layers of Haar-random "
                         "two-qubit unitaries (--n-exp sets the number of layers); dense5: --n-exp "
                         "Haar-random 5-qubit unitaries on random qubits")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--graph", action="store_true", help="replay the passes as a HIP graph")
    ap.add_argument("--only", action="store_true", help="skip the other dtype")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="first run a plain 256 MiB device copy five times (a known byte count for "
                         "scaling memory counters)")
    ap.add_argument("--forms", default="trajectories,batched,served,mma,wide",
                    help="comma list of extra forms to run: trajectories,batched,served,mma,wide "
                         "(or 'all'; '' or --no-forms for none)")
    ap.add_argument("--no-forms", action="store_true")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for {args.gpus}): the library has no "
              "multi-GPU path; the states of a batch or a server are independent and would "
              "shard by whole states", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch

    import workloads as W
    from paper_2310_17739_amd import qsim

    if args.calibrate_copy:
        src = torch.ones(1 << 25, dtype=torch.float64, device="cuda")   # 256 MiB
        dst = torch.empty_like(src)
        for _ in range(5):
            dst.copy_(src)
        torch.cuda.synchronize()
        log("[bench] copy calibration: 5 x 256 MiB read + 256 MiB written")
        del src, dst

    n = args.qubits
    mats = None
    if args.workload == "dense5":
        log(f"[bench] generating circuit: {n} qubits, {args.n_exp} dense 5-qubit operators")
        g, mats = W.dense_operator_circuit(n, args.n_exp, 5, seed=43)
    elif args.workload == "dense":
        log(f"[bench] generating circuit: {n} qubits, {args.n_exp} dense brick-wall layers")
        g, mats = W.dense_brickwork_circuit(n, args.n_exp, seed=41)
    else:
        log(f"[bench] generating circuit: {n} qubits, {args.n_exp} exponentials")
        g, _, _ = W.pauli_exponential_circuit(n, args.n_exp, seed=2)
    H = W.pauli_sum(n, 100, seed=3)

    def measure(dtype):
        # the library's and the HIP runtime's one-time set-up for this precision
        # (kernel attributes, staging buffers) is not part of a circuit's compile
        qsim.Program(n, g[:8], dtype, mats=mats).close()
        log(f"[bench] compile {dtype}")
        t0 = time.perf_counter()
        prog = qsim.Program(n, g, dtype, mats=mats)
        compile_s = time.perf_counter() - t0
        st = prog.qsim_program_stats()
        sv = qsim.StateVector(n, dtype)
        if args.graph:
            prog.qsim_program_graph(sv, True)
        for i in range(args.warmup):
            sv.qsim_init_zero()
            prog.qsim_run(sv)
            sv.qsim_expval(H)
        log(f"[bench] {dtype}: warmup done; timing {args.steps} steps")
        torch.cuda.synchronize()
        # events on the stream the passes run on (the state's stream is
        # torch's current stream), around each step's program
        stream = sv.stream
        ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
              for _ in range(args.steps)]
        t0 = time.perf_counter()
        energy = None
        for i in range(args.steps):
            sv.qsim_init_zero()
            ev[i][0].record(stream)
            prog.qsim_run(sv)
            ev[i][1].record(stream)
            energy = sv.qsim_expval(H)      # synchronises the stream
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        prog_ms = [a.elapsed_time(b) for a, b in ev]
        ms_step = 1e3 * dt / args.steps
        elem = 16 if dtype == "complex128" else 8
        pass_bytes = 2 * elem * (1 << n)
        res = {"dtype": dtype, "ms_per_step": ms_step, "gates_per_s": st["input_gates"] / (dt / args.steps),
               "compile_s": compile_s, "stats": st, "energy": energy, "norm": sv.qsim_norm()}
        # a circuit run once: host compile (fusion + plan) plus one device run
        res["gates_per_s_with_compile"] = st["input_gates"] / (compile_s + dt / args.steps)
        if n == 21 and args.n_exp == 50_000 and args.workload == "pauli" and os.path.exists(FIXTURE):
            log(f"[bench] {dtype}: final state against the oracle's stored results")
            res["vs_oracle"] = oracle_distance(W, sv.qsim_get_state(), energy, H)
        if not args.graph:
            # average launch duration over the timed region: the program's
            # span divided by its launches (inter-launch gaps included)
            launches = st["passes"]
            avg_ms = float(np.mean(prog_ms)) / launches
            achieved = pass_bytes / (avg_ms * 1e-3) / 1e9
            res["program_ms_per_step"] = float(np.mean(prog_ms))
            res["avg_launch_us"] = avg_ms * 1e3
            ceil = copy_ceiling(qsim, sv.tensor.view(torch.int64))
            copy_gbs = max(ceil["best_stable"], ceil["best_rotated"])
            res["roofline"] = {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                               "frac": achieved / HBM_PEAK_GBS, "traffic": measured_traffic(dtype),
                               "copy_GBps": copy_gbs, "frac_of_copy": achieved / copy_gbs,
                               "copy_ceilings_GBps": ceil,
                               "frac_of_rotated_copy": achieved / ceil["best_rotated"],
                               "kernel": f"{'k_span' if runs_as_rotations(st) else 'k_tile'}"
                                         f"<{'double' if elem == 16 else 'float'}>",
                               "bytes_per_launch": pass_bytes, "launches_per_step": launches}
            # one more step with an event pair around every pass: pure kernel
            # time per launch (what a kernel trace reports)
            sv.qsim_init_zero()
            prog.qsim_run_timed(sv)
            kms, kl = prog.qsim_program_kernel_ms()
            res["per_pass_kernel_us"] = 1e3 * kms / kl
            # arithmetic of the same launches
            flops = flops_per_amplitude(st) * (1 << n)
            res["alu"] = {"flops_per_step": flops,
                          "achieved_TFLOPs": flops / (float(np.mean(prog_ms)) * 1e-3) / 1e12,
                          "peak_TFLOPs": 78.6,
                          "frac": flops / (float(np.mean(prog_ms)) * 1e-3) / 1e12 / 78.6}
            # LDS traffic of the same launches: in tiled passes every operator
            # reads and writes the whole tile once (coefficient reads not
            # counted), in passes of rotations every re-layout does
            lds_bytes = float(st["reg_relayouts"] if runs_as_rotations(st) else st["fused_ops"]) * pass_bytes
            lds_gbs = lds_bytes / (float(np.mean(prog_ms)) * 1e-3) / 1e9
            res["lds"] = {"bytes_per_step": lds_bytes, "achieved_GBps": lds_gbs,
                          "peak_GBps": LDS_PEAK_GBS, "frac": lds_gbs / LDS_PEAK_GBS}
        prog.close()
        sv.close()
        return res

    main_res = measure(args.dtype)
    forms = {}
    want = set(args.forms.split(",")) if (args.forms and not args.no_forms) else set()
    if "all" in want:
        want = {"trajectories", "batched", "served", "mma", "wide"}
    for name, fn in (("trajectories", run_trajectories), ("batched", run_batched),
                     ("served", run_served), ("mma", run_mma), ("wide", run_wide_job)):
        if name in want:
            log(f"[bench] form: {name}")
            forms[name] = fn(qsim, W)
            log(f"[bench] {name}: {json.dumps(forms[name])}")
    other = None
    if not args.only:
        other = measure("complex64" if args.dtype == "complex128" else "complex128")
    cpu = None
    if not args.no_cpu_baseline:
        log("[bench] cpu baseline (oracle)")
        cpu = cpu_baseline(n, g)
    st = main_res["stats"]
    out = {
        "metric": "gates/s + GB/s (roofline %) at 21q",
        "value": main_res["gates_per_s"],
        "unit": "gates/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": main_res["ms_per_step"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "c128 (f64)" if args.dtype == "complex128" else "c64 (f32) + f64 reductions",
        "data": "synthetic",
        "config": {"workload": f"{n}-qubit circuit of {WORKLOAD_TEXT[args.workload].format(args.n_exp)} "
                               f"({st['input_gates']} gates), then <H> of a 100-term Pauli sum",
                   "qubits": n, "input_gates": st["input_gates"], "fused_ops": st["fused_ops"],
                   "ops_after_fusion_levels": st["ops_after"], "passes": st["passes"],
                   "tile_qubits": st["tile_qubits"], "max_width": st["max_width"],
                   "compile_s": main_res["compile_s"], "graph": bool(args.graph),
                   "parallelism": "single GPU"},
        "roofline": main_res.get("roofline"),
        "cpu_baseline": cpu,
        "energy": main_res["energy"],
        "norm": main_res["norm"],
    }
    for k in ("program_ms_per_step", "avg_launch_us", "per_pass_kernel_us", "alu", "lds", "vs_oracle",
              "gates_per_s_with_compile"):
        if k in main_res:
            out[k] = main_res[k]
    if forms:
        out["forms"] = forms
    if other is not None:
        out["other_dtype"] = {k: other[k] for k in ("dtype", "ms_per_step", "gates_per_s", "energy")}
        for k in ("roofline", "avg_launch_us", "per_pass_kernel_us", "alu", "lds", "vs_oracle",
                  "gates_per_s_with_compile", "compile_s"):
            if k in other:
                out["other_dtype"][k] = other[k]
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
