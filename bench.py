#!/usr/bin/env python3
"""Benchmark of the state-vector hot path on one MI355X.

Headline workload: the 30-qubit layered circuit (20 layers of RY, RZ on every
qubit followed by the CNOT ladder 0->1 ... 28->29; 1780 gates, 1200 angles
uniform in [0, 2pi) from seed 0) applied to |0...0> in FP64 split planes
(16 GiB), then <Z_i> for every qubit.  One step = reset + all sweeps + one
Pauli pass; the state is resident in HBM throughout.

value = amplitude-gate updates per second = 1780 * 2^30 * steps / time.

Also reported: the roofline of the dominant kernel (tile sweep) from HIP
events around each sweep launch, the oracle's CPU rate on a bounded sample of
the same workload, and extras (paper-style width-5 fusion plan, complex64).

    python bench.py [--gpus 1] [--steps 5] [--warmup 2] [--no-cpu] [--no-extras]
"""
import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

HBM_PEAK_GBS = 8000.0          # MI355X HBM3E, published
METRIC = "amplitude-gate updates/s + % HBM roofline (30q); served req/s, p99 latency"


def log(*a):
    print("[bench]", *a, file=sys.stderr, flush=True)


def cpu_baseline(circ, budget_s: float):
    """The oracle (plain C, OpenMP over amplitude groups) applying the first gates of
    the same 30-qubit circuit until `budget_s` of CPU work; returns updates/s."""
    import ctypes as C
    import numpy as np
    from oracle import oracle as O
    n = circ.n
    N = 1 << n
    t_alloc = time.time()
    buf = np.zeros(2 * N, dtype=np.float64)
    buf[0] = 1.0
    log(f"cpu_baseline: allocated {buf.nbytes / 2**30:.1f} GiB in {time.time() - t_alloc:.1f}s")
    L = O.lib()
    p = np.ascontiguousarray(circ.params, dtype=np.float64)
    dp = p.ctypes.data_as(C.POINTER(C.c_double))
    bp = buf.ctypes.data_as(C.POINTER(C.c_double))
    done = 0
    per_gate = []
    t0 = time.time()
    while done < len(circ.ops) and time.time() - t0 < budget_s:
        oa = O.OpArray([circ.ops[done]])
        tg = time.perf_counter()
        rc = L.orc_apply(n, bp, oa.ptr(), 1, dp)
        per_gate.append(float(N) / (time.perf_counter() - tg))
        if rc != 0:
            raise RuntimeError("oracle failed")
        done += 1
    el = time.time() - t0
    rate = done * float(N) / el
    del buf
    q1, q2, q3 = np.percentile(per_gate, [25, 50, 75])
    return {"value": rate, "unit": "updates/s", "cores": O.threads(), "kind": "oracle",
            "sample": f"first {done} of {len(circ.ops)} gates of the same {n}-qubit circuit, "
                      f"{el:.1f} s wall, plain C FP64 gate-by-gate",
            "per_gate_updates_per_s": {"median": float(q2), "iqr": float(q3 - q1),
                                       "gates": done}}


def cpu_model() -> str:
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return "unknown"


def oracle_single_thread_child():
    """Runs in a child process started with OMP_NUM_THREADS=1 (never touches
    the GPU): the oracle on the 12-qubit layered circuit (state + <Z_i>) and on
    the 20-qubit HEA/TFIM energy + adjoint gradient; prints one JSON line."""
    import numpy as np
    from oracle import oracle as O
    from paper_2608_09733_amd import inputs as I
    out = {"threads": O.threads()}
    c1 = I.layered(12, 20, seed=0)
    z12 = I.hamiltonian(12, [("Z", [q], 1.0) for q in range(12)])
    ts = []
    for _ in range(5):
        t0 = time.time()
        psi = O.run_circuit(c1)
        O.expect(12, psi, z12)
        ts.append(time.time() - t0)
    out["layered_12q_20l_ms"] = float(np.median(ts) * 1e3)
    c3 = I.hea(20, 10, seed=0)
    t0 = time.time()
    O.adjoint_grad(c3, I.tfim(20, 0.7))
    out["adjoint_hea_20q_10l_tfim_ms"] = (time.time() - t0) * 1e3
    # the 512-circuit ragged batch (state + <Z0 Z1> per circuit), timed circuit
    # by circuit in batch order over those of at most 18 qubits until about
    # 12 s are spent, then projected to all 512 by gate-amplitude updates
    circs = I.batch_circuits(512, seed=0)
    upd = [len(c.ops) * float(1 << c.n) for c in circs]
    t_sum, u_sum, k = 0.0, 0.0, 0
    for c, u in zip(circs, upd):
        if c.n > 18:
            continue
        t0 = time.time()
        psi = O.run_circuit(c)
        O.expect(c.n, psi, I.z0z1(c.n))
        t_sum += time.time() - t0
        u_sum += u
        k += 1
        if t_sum > 12.0:
            break
    out["batch_512_ragged"] = {
        "sample": f"first {k} circuits of at most 18 qubits, in batch order, timed one by one",
        "circuits_timed": k, "sampled_s": t_sum, "sampled_updates": u_sum,
        "updates_per_s": u_sum / t_sum, "total_updates": float(sum(upd)),
        "projected_all_512_s": t_sum * float(sum(upd)) / u_sum}
    print(json.dumps(out), flush=True)


def oracle_single_thread():
    import subprocess
    env = dict(os.environ, OMP_NUM_THREADS="1")
    r = subprocess.run([sys.executable, os.path.abspath(__file__), "--oracle-single-child"],
                       env=env, capture_output=True, text=True, timeout=400)
    if r.returncode != 0:
        raise RuntimeError("single-thread oracle run failed: " + r.stderr[-2000:])
    return json.loads(r.stdout.strip().splitlines()[-1])


def measured_traffic():
    """Bytes per launch of the tile sweep from the committed counter summary
    (FETCH_SIZE / WRITE_SIZE scaled by a plain copy), or None when the kernel
    sources have changed since the counters were taken."""
    import hashlib
    path = os.path.join(ROOT, "profiles", "k_sweep_kron_30q_layered_fp64.md")
    try:
        txt = open(path).read()
    except OSError:
        return None
    vals = {}
    for line in txt.splitlines():
        line = line.strip()
        for key in ("traffic_bytes_per_launch:", "kernel_source_sha256:", "kernel_sources:"):
            if line.startswith(key):
                vals[key[:-1]] = line[len(key):].strip()
    if len(vals) != 3:
        return None
    h = hashlib.sha256()
    for f in vals["kernel_sources"].split():
        h.update(open(os.path.join(ROOT, "paper_2608_09733_amd", "csrc", f), "rb").read())
    if h.hexdigest() != vals["kernel_source_sha256"]:
        return None
    return float(vals["traffic_bytes_per_launch"])


def _median_ms(fn, reps, torch):
    """Median over `reps` calls of fn(), each bracketed by events on the current stream."""
    import numpy as np
    ts = []
    for _ in range(reps):
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record()
        fn()
        e1.record()
        torch.cuda.synchronize()
        ts.append(e0.elapsed_time(e1))
    return float(np.median(ts)), float(np.percentile(ts, 75) - np.percentile(ts, 25))


def sampling_and_exit(st, n, torch):
    """Terminal sampling and the explicit exit on a resident n-qubit FP64 state:
    2^20 shots of all qubits per call (chunk sums, blocked prefix, draws, 8 MiB
    of samples to the host), and 2^min(n,28) amplitudes copied into pinned host
    buffers."""
    import numpy as np
    out = {}
    shots = 1 << 20
    allq = list(range(n))
    st.sample(1, shots, allq)
    ts = []
    for k in range(5):
        t0 = time.time()
        st.sample(k + 2, shots, allq)
        ts.append((time.time() - t0) * 1e3)
    out["sampling_2p20_shots"] = {"ms_median": float(np.median(ts)), "shots": shots,
                                  "shots_per_s": shots / (np.median(ts) / 1e3),
                                  "state_read_bytes": 16.0 * (1 << n)}
    log(f"sampling: {np.median(ts):.2f} ms per {shots} shots")
    ts = []
    for k in range(5):
        t0 = time.time()
        st.sample(k + 2, 1000, allq)
        ts.append((time.time() - t0) * 1e3)
    out["sampling_1000_shots"] = {"ms_median": float(np.median(ts)), "shots": 1000}
    log(f"sampling: {np.median(ts):.2f} ms per 1000 shots")
    # grouped shot estimator: TFIM (ZZ group and X group), 2^20 shots in all
    from paper_2608_09733_amd import inputs as I
    ham = I.tfim(n, 0.7)
    st.shot_estimate(1, 1 << 20, ham)
    ts = []
    for k in range(3):
        t0 = time.time()
        vals, e, var, G = st.shot_estimate(k + 2, 1 << 20, ham)
        ts.append((time.time() - t0) * 1e3)
    out["shot_estimate_tfim_2p20_shots"] = {"ms_median": float(np.median(ts)), "shots": 1 << 20,
                                            "groups": G, "terms": len(ham), "energy": e,
                                            "std_error": math.sqrt(var)}
    log(f"shot estimator: {np.median(ts):.1f} ms, {G} groups, E = {e:.4f} +- {math.sqrt(var):.4f}")
    cnt = 1 << min(n, 28)
    pre = torch.empty(cnt, dtype=torch.float64, pin_memory=True)
    pim = torch.empty(cnt, dtype=torch.float64, pin_memory=True)
    bufs = (pre.numpy(), pim.numpy())
    st.planes(0, cnt, out=bufs)
    t0 = time.time()
    st.planes(0, cnt, out=bufs)
    tx = (time.time() - t0) * 1e3
    out["exit_to_pinned_host"] = {"amplitudes": cnt, "bytes": 16.0 * cnt, "ms": tx,
                                  "gb_s": 16.0 * cnt / (tx / 1e3) / 1e9}
    log(f"exit: {16.0 * cnt / 2**30:.0f} GiB in {tx:.1f} ms")
    return out


def density_matrix_run(st, n, sv, I, torch):
    """A density matrix of n/2 qubits on the n-qubit handle (the same 2^n
    amplitudes as the state-vector workload): 4 layers of the layered circuit,
    each followed by depolarizing noise (p = 0.01) on every qubit, then <Z_i>."""
    import numpy as np
    nd, Ld = n // 2, 4
    cd = I.layered(nd, Ld, seed=0)
    per = 3 * nd - 1
    arrays = [sv.OpArray(cd.ops[l * per:(l + 1) * per]) for l in range(Ld)]
    p = 0.01
    s3 = math.sqrt(p / 3)
    kr = [math.sqrt(1 - p) * np.eye(2), s3 * np.array([[0, 1], [1, 0]]),
          s3 * np.array([[0, -1j], [1j, 0]]), s3 * np.diag([1.0, -1.0])]
    zs = I.hamiltonian(nd, [("Z", [q], 1.0) for q in range(nd)])

    def run():
        st.reset()
        for oa in arrays:
            st.dm_apply(None, cd.params, op_array=oa)
            st.dm_apply_kraus(list(range(nd)), kr)
        return st.dm_expect(zs)
    run()
    torch.cuda.synchronize()
    ts = []
    for _ in range(3):
        t0 = time.time()
        vals, _ = run()
        ts.append((time.time() - t0) * 1e3)
    ms = float(np.median(ts))
    log(f"density matrix {nd}q ({n}-qubit vector), {Ld} noisy layers: {ms:.1f} ms")
    # checks: Tr(rho) = 1 after the channels; without the channels, <Z_i> of
    # rho equals <Z_i> of the same circuit run as an nd-qubit state vector
    zi = I.hamiltonian(nd, [("Z", [q], 1.0) for q in range(nd)] + [("I", [0], 1.0)])
    tr = st.dm_expect(zi)[0][-1]
    st.reset()
    for oa in arrays:
        st.dm_apply(None, cd.params, op_array=oa)
    zdm = st.dm_expect(zi)[0][:nd]
    sv_state = sv.State(nd)
    sv_state.apply(cd.ops, cd.params)
    zsv = sv_state.expect(zi)[0][:nd]
    sv_state.close()
    dz = float(np.max(np.abs(zdm - zsv)))
    log(f"density matrix checks: Tr(rho) - 1 = {tr - 1:.2e}, noiseless <Z_i> vs state vector {dz:.2e}")
    return {"density_matrix_%dq_%dl_depolarizing" % (nd, Ld): {
        "ms_median": ms, "qubits": nd, "vector_qubits": n, "layers": Ld,
        "gates": len(cd.ops), "channels": nd * Ld, "z0": float(vals[0]),
        "trace_minus_1": float(tr - 1.0), "noiseless_z_max_abs_diff_vs_state_vector": dz}}


def side_configs(sv, I, torch, serving=True):
    """The other workloads of the method at their own shapes: small-state
    latency (12 qubits), adjoint gradient (20-qubit HEA, TFIM), and the ragged
    batch of 512 circuits as one persistent launch vs the per-circuit loop."""
    out = {}
    # 12-qubit layered circuit, 20 layers, then <Z_i>: a 64 KiB state (latency-bound)
    c1 = I.layered(12, 20, seed=0)
    z12 = I.hamiltonian(12, [("Z", [q], 1.0) for q in range(12)])
    s1 = sv.State(12)
    oa1 = sv.OpArray(c1.ops)

    def f1():
        s1.reset()
        s1.apply(None, c1.params, op_array=oa1)
        s1.expect(z12)
    f1()
    ms, iqr = _median_ms(f1, 20, torch)
    out["layered_12q_20l"] = {"ms_median": ms, "ms_iqr": iqr, "gates": len(c1.ops),
                              "updates_per_s": len(c1.ops) * 4096 / (ms / 1e3)}
    s1.close()
    log(f"12q layered: {ms:.3f} ms")
    # adjoint gradient: 20-qubit HEA (RY/RZ + CZ ring), 10 layers, 400 angles, TFIM h=0.7
    c3 = I.hea(20, 10, seed=0)
    h3 = I.tfim(20, 0.7)
    s3 = sv.State(20, adjoint=True)
    oa3 = sv.OpArray(c3.ops)
    def f3():
        s3.reset()
        s3.adjoint_grad(None, c3.params, h3, op_array=oa3)
    f3()
    ms, iqr = _median_ms(f3, 10, torch)
    out["adjoint_hea_20q_10l_tfim"] = {"ms_median": ms, "ms_iqr": iqr, "params": int(len(c3.params)),
                                       "gates": len(c3.ops)}
    s3.close()
    log(f"20q adjoint: {ms:.3f} ms")
    # the same ansatz at 26 qubits (1 GiB per state: psi, lambda and the psi
    # copy live in HBM), against a forward pass + <H> on the same state
    c4 = I.hea(26, 10, seed=0)
    h4 = I.tfim(26, 0.7)
    s4 = sv.State(26, adjoint=True)
    oa4 = sv.OpArray(c4.ops)
    def f4():
        s4.reset()
        s4.adjoint_grad(None, c4.params, h4, op_array=oa4)
    def g4():
        s4.reset()
        s4.apply(None, c4.params, op_array=oa4)
        s4.expect(h4)
    f4()
    g4()
    ms, iqr = _median_ms(f4, 5, torch)
    fms, _ = _median_ms(g4, 5, torch)
    out["adjoint_hea_26q_10l_tfim"] = {"ms_median": ms, "ms_iqr": iqr, "params": int(len(c4.params)),
                                       "gates": len(c4.ops), "forward_expect_ms": fms,
                                       "ratio_to_forward": ms / fms}
    s4.close()
    log(f"26q adjoint: {ms:.2f} ms (forward + <H>: {fms:.2f} ms)")
    # ragged batch: 512 layered circuits, n in 8..22, L in 10..40, <Z0 Z1> each
    circs = I.batch_circuits(512, seed=0)
    hams = [I.z0z1(c.n) for c in circs]
    tune = sv.batch_autotune(circs, hams, reps=2)
    b = sv.Batch(circs, hams, low_bits=tune["low_bits"], group_bits=tune["group_bits"])
    b.run(graph=True)
    b.results()
    ms, iqr = _median_ms(lambda: b.run(graph=True), 5, torch)
    b.check()
    units, sweeps, updates, nbytes = b.stats()
    b.close()
    states = [sv.State(c.n) for c in circs]

    def plain():
        for stt, c, h in zip(states, circs, hams):
            stt.reset()
            stt.apply(c.ops, c.params)
            stt.expect(h)
    plain()
    pms, _ = _median_ms(plain, 2, torch)
    for stt in states:
        stt.close()
    out["batch_512_ragged"] = {"ms_median": ms, "ms_iqr": iqr, "circuits_per_s": 512 / (ms / 1e3),
                               "updates_per_s": updates / (ms / 1e3), "updates": updates,
                               "work_units": units, "sweeps": sweeps, "tiling": tune,
                               "algorithmic_bytes": nbytes, "hbm_gbs": nbytes / (ms / 1e3) / 1e9,
                               "plain_loop_ms": pms, "speedup_vs_plain_loop": pms / ms}
    log(f"batch 512: {ms:.1f} ms ({updates / (ms / 1e3):.3e} upd/s), plain loop {pms:.1f} ms, "
        f"tiling {tune}")
    if not serving:
        return out
    # serving: Poisson arrivals at 200 req/s, n log-uniform in [10, 28], TFIM,
    # (E, grad) per request; small requests batched into the serving kernel,
    # one big lane, one mid lane, against serial FIFO on one lane
    from paper_2608_09733_amd import serving as S
    srv = S.run(rate=200.0, count=500, lanes=2, budget_gb=200.0, seed=0)
    out["serving_200rps_500req"] = srv
    log(f"serving: {srv['served']['throughput_req_s']:.1f} req/s, p50 "
        f"{srv['served']['latency_p50_ms']:.1f} ms, p99 {srv['served']['latency_p99_ms']:.1f} ms; "
        f"serial {srv['serial_fifo']['throughput_req_s']:.1f} req/s, p50 "
        f"{srv['serial_fifo']['latency_p50_ms']:.1f} ms, p99 {srv['serial_fifo']['latency_p99_ms']:.1f} ms; "
        f"alone-vs-mix mismatches {srv['alone_vs_mix_mismatches']}")
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=2)
    ap.add_argument("--n", type=int, default=30)
    ap.add_argument("--layers", type=int, default=20)
    ap.add_argument("--tile", type=int, default=0)
    ap.add_argument("--low", type=int, default=0)
    ap.add_argument("--group", type=int, default=0)
    ap.add_argument("--fuse", type=int, default=-1)
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-extras", action="store_true")
    ap.add_argument("--cpu-budget", type=float, default=15.0)
    ap.add_argument("--side-only", action="store_true",
                    help="only the side workloads (12-qubit latency, adjoint, batch), no serving")
    ap.add_argument("--dm-only", action="store_true",
                    help="only the density-matrix workload on the --n qubit handle")
    ap.add_argument("--sample-only", action="store_true",
                    help="only sampling and the exit copy on the resident --n qubit state")
    ap.add_argument("--copy-probe", action="store_true",
                    help="only run a plain 2 GiB device-to-device copy (counter calibration)")
    ap.add_argument("--adjoint-only", action="store_true",
                    help="only the --n qubit HEA (10 layers, TFIM) adjoint, --steps times, then "
                         "as many forward passes with <H>; --tile/--low/--group set the backward "
                         "tiling (for profiling and tuning)")
    ap.add_argument("--batch-only", action="store_true",
                    help="only the 512-circuit ragged batch, --steps graph launches, tiling from "
                         "--low/--group or else the autotuner (for profiling)")
    ap.add_argument("--oracle-single-child", action="store_true", help=argparse.SUPPRESS)
    args = ap.parse_args()
    if args.oracle_single_child:
        oracle_single_thread_child()
        return

    if args.gpus != 1 or int(os.environ.get("WORLD_SIZE", "1")) != 1:
        print("bench.py: the state-vector path runs and is measured on one GPU only "
              "(one MI355X holds the whole 30-qubit state); --gpus must be 1", file=sys.stderr)
        sys.exit(2)

    import numpy as np
    import torch
    from paper_2608_09733_amd import inputs as I
    from paper_2608_09733_amd import sv

    torch.cuda.set_device(0)
    if args.copy_probe:
        # a plain copy of known size: 2 GiB read + 2 GiB written per dispatch
        a = torch.ones(1 << 28, dtype=torch.float64, device="cuda")
        b = torch.empty_like(a)
        for _ in range(3):
            b.copy_(a)
        torch.cuda.synchronize()
        log(f"copy probe: 3 copies of {a.numel() * 8} bytes")
        return
    if args.adjoint_only:
        c4 = I.hea(args.n, 10, seed=0)
        h4 = I.tfim(args.n, 0.7)
        s4 = sv.State(args.n, adjoint=True)
        if args.tile or args.low or args.group:
            s4.set_adjoint_tiling(args.tile, args.low, args.group)   # backward sweeps
        oa4 = sv.OpArray(c4.ops)
        res = {"workload": f"hea_{args.n}q_10l_tfim_adjoint", "adjoint_ms": [], "forward_expect_ms": [],
               "backward_tiling": [args.tile, args.low, args.group]}
        for key, fn in (("adjoint_ms", lambda: s4.adjoint_grad(None, c4.params, h4, op_array=oa4)),
                        ("forward_expect_ms", lambda: (s4.apply(None, c4.params, op_array=oa4),
                                                       s4.expect(h4)))):
            for _ in range(args.steps):
                s4.reset()
                torch.cuda.synchronize()
                t0 = time.perf_counter()
                fn()
                torch.cuda.synchronize()
                res[key].append((time.perf_counter() - t0) * 1e3)
                log(f"{key}: {res[key][-1]:.2f}")
        s4.close()
        print(json.dumps(res), flush=True)
        return
    if args.batch_only:
        circs = I.batch_circuits(512, seed=0)
        hams = [I.z0z1(c.n) for c in circs]
        if args.group and args.low:
            tune = {"low_bits": args.low, "group_bits": args.group}
        else:
            tune = sv.batch_autotune(circs, hams, reps=2)
        b = sv.Batch(circs, hams, low_bits=tune["low_bits"], group_bits=tune["group_bits"])
        res = {"workload": "batch_512_ragged", "tiling": tune, "ms": []}
        for _ in range(args.steps):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            b.run(graph=True)
            b.check()
            res["ms"].append((time.perf_counter() - t0) * 1e3)
        res["stats"] = list(b.stats())
        b.close()
        print(json.dumps(res), flush=True)
        return
    if args.side_only:
        from paper_2608_09733_amd import inputs as I
        from paper_2608_09733_amd import sv
        print(json.dumps(side_configs(sv, I, torch, serving=False)), flush=True)
        return
    if args.dm_only:
        st = sv.State(args.n, "c128")
        print(json.dumps(density_matrix_run(st, args.n, sv, I, torch)), flush=True)
        st.close()
        return
    if args.sample_only:
        circ = I.layered(args.n, args.layers, seed=0)
        st = sv.State(args.n, "c128")
        st.apply(None, circ.params, op_array=sv.OpArray(circ.ops))
        print(json.dumps(sampling_and_exit(st, args.n, torch)), flush=True)
        st.close()
        return
    n, L = args.n, args.layers
    circ = I.layered(n, L, seed=0)
    gates = len(circ.ops)
    zs = I.hamiltonian(n, [("Z", [q], 1.0) for q in range(n)])
    oa = sv.OpArray(circ.ops)
    # the plan of every step: from the |0..0> that it begins with
    sweeps, blocks = sv.plan_stats(n, circ.ops, args.fuse, args.tile, args.low, args.group,
                                   from_zero=True)
    log(f"workload n={n} L={L} gates={gates} plan fuse={args.fuse}: {sweeps} sweeps, {blocks} blocks")

    st = sv.State(n, "c128")
    dt = sv.default_tiling(n)
    tiling = (args.tile or dt[0], args.low or dt[1], args.group or dt[2])
    if args.tile or args.low or args.group:
        st.set_tiling(args.tile, args.low, args.group)

    def step():
        st.reset()
        st.apply(None, circ.params, fuse=args.fuse, op_array=oa)
        return st.expect(zs)

    for w in range(args.warmup):
        step()
        log(f"warmup {w} done")
    torch.cuda.synchronize()
    st.timing(True)
    evs = [torch.cuda.Event(enable_timing=True) for _ in range(args.steps + 1)]
    t0 = time.time()
    evs[0].record()
    for k in range(args.steps):
        z, _ = step()
        evs[k + 1].record()
        log(f"step {k} done")
    torch.cuda.synchronize()
    wall = time.time() - t0
    gpu_ms = evs[0].elapsed_time(evs[-1])
    step_ms = np.array([evs[k].elapsed_time(evs[k + 1]) for k in range(args.steps)])
    sweep_ms, launches, sweep_bytes = st.timing_read()
    st.timing(False)
    ms_per_step = gpu_ms / args.steps
    value = gates * float(1 << n) * args.steps / (gpu_ms / 1e3)
    avg_launch_ms = sweep_ms / max(1, launches)
    bytes_per_launch = sweep_bytes / max(1, launches)
    achieved = bytes_per_launch / (avg_launch_ms / 1e3) / 1e9
    log(f"GPU {ms_per_step:.2f} ms/step ({wall / args.steps * 1e3:.2f} wall), {value:.4e} updates/s, "
        f"sweep avg {avg_launch_ms:.3f} ms over {launches} launches -> {achieved:.0f} GB/s")

    result = {
        "metric": METRIC,
        "value": value,
        "unit": "amplitude-gate updates/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "ms_per_step_median": float(np.median(step_ms)),
        "ms_per_step_iqr": float(np.percentile(step_ms, 75) - np.percentile(step_ms, 25)),
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic",
        "config": {"workload": f"layered RY/RZ + CNOT-ladder circuit, {n} qubits, {L} layers, "
                               f"{gates} gates, angles U[0,2pi) seed 0, from |0..0>, then <Z_i> "
                               f"for all i", "n_qubits": n, "layers": L, "gates": gates,
                   "plan": "tile clusters (SV_FUSE_AUTO)" if args.fuse == -1 else f"fuse={args.fuse}",
                   "sweeps": sweeps, "register_blocks": blocks,
                   "state_bytes": 16 * (1 << n)},
        "roofline": {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                     "frac": achieved / HBM_PEAK_GBS, "traffic": measured_traffic(),
                     "kernel": f"svk::k_sweep_kron<double,{tiling[0]},{tiling[2]}> (tile sweep)",
                     "bytes_per_launch": bytes_per_launch, "avg_launch_ms": avg_launch_ms,
                     "launches": launches,
                     # every sweep over every tile (the first one only writing)
                     "bytes_per_launch_dense": (2 + 4 * (sweeps - 1)) * 8.0 * (1 << n) / sweeps,
                     "note": "from |0..0> the sweeps after the first run only the tiles on the "
                             "support reached so far (the others are zero before and after); "
                             "bytes_per_launch counts what the launches moved"},
    }
    extras = {}
    # whole-path HBM efficiency: counted sweep bytes / step time
    extras["path_hbm_gbs"] = (sweep_bytes / args.steps) / (ms_per_step / 1e3) / 1e9
    if not args.no_extras and args.fuse == -1:
        # paper-style fusion (greedy in-order blocks of <= 5 qubits, one sweep each)
        s5, _ = sv.plan_stats(n, circ.ops, 5)
        st.reset()
        st.apply(None, circ.params, fuse=5, op_array=oa)
        torch.cuda.synchronize()
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        st.reset()
        e0.record()
        st.apply(None, circ.params, fuse=5, op_array=oa)
        e1.record()
        torch.cuda.synchronize()
        t5 = e0.elapsed_time(e1)
        extras["fuse5_plan"] = {"sweeps": s5, "ms": t5,
                                "updates_per_s": gates * float(1 << n) / (t5 / 1e3),
                                "hbm_gbs": s5 * 32.0 * (1 << n) / (t5 / 1e3) / 1e9}
        log(f"fuse=5: {s5} sweeps, {t5:.1f} ms")
        # complex64 variant: same circuit in FP32 planes; error against the
        # oracle's FP64 amplitudes at the golden indices (the 30-qubit,
        # 20-layer, seed-0 workload), else against this run's FP64 state
        gold = os.path.join(ROOT, "tests", "golden", "layered30_seed0.npz")
        g = np.load(gold, allow_pickle=False) if os.path.exists(gold) else None
        if g is not None and tuple(g["meta"][:3]) != (n, L, 0):
            g = None
        if g is not None:
            ref_idx, ref_amp, ref_kind = g["idx"], g["amp"], "oracle_golden_65536_amps"
        else:
            st.reset()
            st.apply(None, circ.params, fuse=-1, op_array=oa)
            ref_idx = np.arange(1 << 16)
            ref_amp, ref_kind = st.gather(ref_idx), "gpu_fp64_first_65536_amps"
        s32 = sv.State(n, "c64")
        s32.apply(None, circ.params, fuse=-1, op_array=oa)
        torch.cuda.synchronize()
        e0.record()
        s32.reset()
        s32.apply(None, circ.params, fuse=-1, op_array=oa)
        e1.record()
        torch.cuda.synchronize()
        t32 = e0.elapsed_time(e1)
        err = float(np.max(np.abs(s32.gather(ref_idx) - ref_amp)))
        rms = math.sqrt(2.0 ** -n)
        extras["complex64"] = {"ms": t32, "updates_per_s": gates * float(1 << n) / (t32 / 1e3),
                               "max_abs_err": err, "max_abs_err_over_rms_amplitude": err / rms,
                               "reference": ref_kind}
        log(f"complex64: {t32:.1f} ms, max err {err:.2e} ({err / rms:.2e} x rms amplitude, "
            f"against {ref_kind})")
        s32.close()
        del s32
        extras.update(sampling_and_exit(st, n, torch))
        extras.update(density_matrix_run(st, n, sv, I, torch))
        # the paper's other circuit families at the same size (Section 9.1)
        for name, c in (("qft", I.qft(n)), ("ghz", I.ghz(n)),
                        ("random300", I.random_circuit(n, 300, seed=0))):
            oac = sv.OpArray(c.ops)
            st.reset()
            st.apply(None, c.params, op_array=oac)
            torch.cuda.synchronize()
            e0.record()
            for _ in range(3):
                st.reset()
                st.apply(None, c.params, op_array=oac)
            e1.record()
            torch.cuda.synchronize()
            tc = e0.elapsed_time(e1) / 3
            extras[f"{name}_{n}q"] = {"gates": len(c.ops), "ms": tc,
                                      "updates_per_s": len(c.ops) * float(1 << n) / (tc / 1e3)}
            log(f"{name} {n}q: {len(c.ops)} gates, {tc:.1f} ms")
    if not args.no_extras:
        st.close()
        del st
        st = None
        torch.cuda.empty_cache()
        extras.update(side_configs(sv, I, torch))
    if st is not None:
        st.close()
        del st
    torch.cuda.empty_cache()
    if not args.no_cpu:
        result["cpu_baseline"] = cpu_baseline(circ, args.cpu_budget)
        result["cpu_baseline"]["cpu_model"] = cpu_model()
        result["cpu_baseline"]["single_thread_oracle"] = oracle_single_thread()
        log(f"single-thread oracle: {result['cpu_baseline']['single_thread_oracle']}")
        log(f"cpu_baseline {result['cpu_baseline']['value']:.3e} updates/s on "
            f"{result['cpu_baseline']['cores']} threads")
    result["extras"] = extras
    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()
