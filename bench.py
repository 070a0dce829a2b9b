"""Benchmark: batched term-network contraction of Algorithm 1's level-l estimate.

Headline workload: 225 qubits on a 15x15 grid, 6 layers of Haar SU(2) + CZ
(colours A B C D A B), 20 amplitude+phase-damping noises (rates ~ U[1e-4,
1e-3]) at seeded random gate locations, input |0...0>, target = the noiseless
output state, level-3 expansion (32551 term networks).  Synthetic, seeded
(see workloads/).  The same line carries the 25-qubit grid (level 2), the
36-qubit QAOA (level 2) and the 64 packed circuits as secondary lines.

One step = one full estimate (every term network contracted, FP64 dominant
term, per-term values, level sums) with the plan and its schedule prepared
and all inputs resident in HBM.  The timed steps launch the prepared
schedule directly: by default the K estimates are spread round-robin over 4
streams, each with its own prepared schedule and two estimates in flight
(submit / collect), since one estimate of this workload is latency-bound and
fills few CUs (`one_stream` gives the one-stream figure, --streams 1 makes it
the headline); the same steps one after another give the latency
(time_to_estimate_ms), and a further pass launches the schedule with a HIP
event pair around every launch for the per-kernel durations of the roofline
entry.  Prints ONE JSON line.

  python bench.py [--steps K] [--warmup W] [--gpus 1]
"""
import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "term-network contractions/s and time-to-estimate at |err|<=1e-6, batched vs plain"
FP32_MFMA_PEAK_TFLOPS = 157.3
HBM_PEAK_GBS = 8000.0
FP64_PEAK_TFLOPS = 78.6


_oracle_state = {}


def _oracle_init(cfg):
    from threadpoolctl import threadpool_limits
    import workloads as W
    from oracle import network
    _oracle_state["limit"] = threadpool_limits(1)
    c = W.config(cfg)
    _oracle_state["net"] = network.KetNetwork(c, diagonal=True)
    _oracle_state["split"] = network.slot_split(c)


def _oracle_terms(tl):
    from oracle import network
    for t in tl:
        network.term_value(_oracle_state["net"], _oracle_state["split"], t)
    return len(tl)


def host_info():
    model = None
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    model = line.split(":", 1)[1].strip()
                    break
    except OSError:
        pass
    try:
        affinity = len(os.sched_getaffinity(0))
    except AttributeError:
        affinity = os.cpu_count()
    return {"nproc": affinity, "os_cpu_count": os.cpu_count(), "cpu_model": model}


def cpu_baseline(cfg, level, single_terms, all_terms, reps=3, max_procs=16):
    """The oracle as it stands (one FP64 ket-network contraction per term,
    numpy pairs in its own greedy order), timed on the host on a seeded random
    sample of the workload's term set: single-threaded (BLAS limited to one
    thread) and on all cores (one single-threaded process per core, the
    sample split among them), each the median of `reps` runs; the full term
    set's time is extrapolated from the rate.  Runs before the GPU is
    touched (worker processes are forked)."""
    import multiprocessing as mp
    import numpy as np
    from oracle import terms as oterms
    tl = oterms.enumerate_terms(__import__("workloads").config(cfg).n_noises, level)
    rng = np.random.default_rng(2211170280 + cfg)
    order = rng.permutation(len(tl))
    info = host_info()
    procs = max(1, min(max_procs, info["nproc"] or 1))
    ctx = mp.get_context("fork")
    runs1, runsn = [], []
    sample1 = [tl[j] for j in order[:single_terms]]
    with ctx.Pool(1, initializer=_oracle_init, initargs=(cfg,)) as pool:
        pool.map(_oracle_terms, [sample1[:4]])                     # warm
        for _ in range(reps):
            t0 = time.perf_counter()
            pool.map(_oracle_terms, [sample1])
            runs1.append(len(sample1) / (time.perf_counter() - t0))
    samplen = [tl[j] for j in order[:all_terms]]
    chunks = [samplen[i::procs] for i in range(procs)]
    with ctx.Pool(procs, initializer=_oracle_init, initargs=(cfg,)) as pool:
        pool.map(_oracle_terms, [c[:2] for c in chunks])            # warm every worker
        for _ in range(reps):
            t0 = time.perf_counter()
            pool.map(_oracle_terms, chunks, chunksize=1)
            runsn.append(len(samplen) / (time.perf_counter() - t0))
    med1, medn = sorted(runs1)[len(runs1) // 2], sorted(runsn)[len(runsn) // 2]
    return {"value": medn, "unit": "contractions/s", "cores": procs, "kind": "oracle",
            "sample": f"{len(samplen)} of the {len(tl)} terms (seeded random order), split over "
                      f"{procs} single-threaded processes, median of {reps} runs; one FP64 ket-network "
                      f"contraction per term (numpy pairs, the oracle's greedy order, diagonal gates as "
                      f"shared indices); network setup excluded",
            "runs": runsn,
            "single_thread": {"value": med1, "runs": runs1, "sample": f"{len(sample1)} terms, median of {reps}"},
            "extrapolated_full_estimate_s": {"all_cores": len(tl) / medn, "single_thread": len(tl) / med1},
            "host": info}


def traffic_record_path(workload):
    return os.path.join(ROOT, "profiles", f"traffic_{workload}.json")


def measured_traffic(kernel, workload):
    """HBM bytes per launch of `kernel` from the committed rocprofv3 --pmc
    record of `workload` (FETCH_SIZE and WRITE_SIZE scaled by a plain copy of
    known size), or None when there is no record or the kernel source changed
    since."""
    import hashlib
    rec = traffic_record_path(workload)
    if not os.path.exists(rec):
        return None
    with open(rec) as f:
        t = json.load(f)
    with open(os.path.join(ROOT, "paper_2211_17028_amd", "csrc", "kernels.hip"), "rb") as f:
        sha = hashlib.sha256(f.read()).hexdigest()
    if t.get("kernel") != kernel or t.get("kernels_hip_sha256") != sha:
        return None
    return t["traffic_bytes_per_launch"]


def _kernel_key(name):
    """'void tn::k_mfma_group<128, 64>(tn::MfmaJob const*, ...)' -> 'k_mfma_group<128,64>'."""
    n = name.split("(")[0].replace("void ", "").replace("tn::", "")
    if n.startswith("k_tile64_group"):
        return "k_tile64_group"
    if n.startswith("k_split_reduce"):
        return "k_split_reduce<double>" if "double" in n else "k_split_reduce<float>"
    n = n.replace("HIP_vector_type<float, 2u>", "").replace("HIP_vector_type<double, 2u>", "")
    n = n.replace(" ", "").replace(",>", ">")
    return n


def traffic_from_counters(fetch_csv, write_csv, kernel, out_path, symbol=None, grids=None):
    """HBM bytes per launch of `kernel` from two rocprofv3 --pmc runs of
    bench.py --copy-calibration (FETCH_SIZE, then WRITE_SIZE, KiB per
    dispatch).  Each counter is scaled by what it reads for the 512 MiB
    device-to-device copy of the calibration (the dispatches that write
    512 MiB), so the figure is in bytes moved.  `symbol`: the profiler's
    kernel name to match (default: `kernel`); `grids`: keep only dispatches of
    these workgroup counts (the launches of one estimate, not those run once
    when a schedule is bound)."""
    import csv
    import hashlib

    def load(path, counter):
        rows = [r for r in csv.DictReader(open(path)) if r["Counter_Name"] == counter]
        return rows

    def keep(r):
        if _kernel_key(r["Kernel_Name"]) != (symbol or kernel):
            return False
        return grids is None or int(r["Grid_Size"]) // int(r["Workgroup_Size"]) in grids
    fr, wr = load(fetch_csv, "FETCH_SIZE"), load(write_csv, "WRITE_SIZE")
    copy_ids = {r["Dispatch_Id"] for r in wr if "copyBuffer" in r["Kernel_Name"]
                and abs(float(r["Counter_Value"]) - 524288.0) < 1.0}
    copy_fetch = [float(r["Counter_Value"]) for r in fr if "copyBuffer" in r["Kernel_Name"]
                  and r["Dispatch_Id"] in copy_ids]
    copy_write = [float(r["Counter_Value"]) for r in wr if r["Dispatch_Id"] in copy_ids]
    if not copy_fetch or not copy_write:
        raise SystemExit("no 512 MiB calibration copy in the counter files")
    fs = 524288.0 / (sum(copy_fetch) / len(copy_fetch))
    ws = 524288.0 / (sum(copy_write) / len(copy_write))
    kf = [float(r["Counter_Value"]) for r in fr if keep(r)]
    kw = [float(r["Counter_Value"]) for r in wr if keep(r)]
    if not kf or not kw:
        raise SystemExit(f"kernel {kernel} not in the counter files")
    f_kib, w_kib = sum(kf) / len(kf), sum(kw) / len(kw)
    with open(os.path.join(ROOT, "paper_2211_17028_amd", "csrc", "kernels.hip"), "rb") as f:
        sha = hashlib.sha256(f.read()).hexdigest()
    rec = {"kernel": kernel, "kernels_hip_sha256": sha, "dispatches": len(kf),
           "grids": sorted(grids) if grids else None,
           "fetch_kib_per_launch": f_kib, "write_kib_per_launch": w_kib, "fetch_scale": fs,
           "write_scale": ws, "traffic_bytes_per_launch": 1024.0 * (f_kib * fs + w_kib * ws)}
    with open(out_path, "w") as f:
        json.dump(rec, f, indent=1)
    print(json.dumps(rec))


def roofline_of(name, st, per):
    """Roofline entry of one kernel from its accumulated event timing: FP32
    matrix-core kernels against the FP32 MFMA peak, FP64 FMA tile kernels
    against the FP64 peak, the rest (small steps, permutes) against HBM."""
    if name.startswith("k_mfma") or name.startswith("k_gemm_mfma"):
        achieved = st["flops"] / (st["ms"] * 1e-3) / 1e12
        roof = {"bound": "mfma", "achieved": achieved, "peak": FP32_MFMA_PEAK_TFLOPS, "unit": "TFLOP/s",
                "frac": achieved / FP32_MFMA_PEAK_TFLOPS}
    elif name.startswith("k_tile64") or name.startswith("k_gemm_tiled_c128"):
        achieved = st["flops"] / (st["ms"] * 1e-3) / 1e12
        roof = {"bound": "alu", "achieved": achieved, "peak": FP64_PEAK_TFLOPS, "unit": "TFLOP/s",
                "frac": achieved / FP64_PEAK_TFLOPS,
                "peak_note": "FP64 FMA: 256 CUs x 4 SIMDs x 16 lanes x 2 flops x 2.4 GHz"}
    else:
        achieved = st["bytes"] / (st["ms"] * 1e-3) / 1e9
        roof = {"bound": "hbm", "achieved": achieved, "peak": HBM_PEAK_GBS, "unit": "GB/s",
                "frac": achieved / HBM_PEAK_GBS}
    if roof["bound"] != "hbm" and st["bytes"] > 0:
        # attainable ceiling at the kernel's algorithmic intensity: min(peak, AI x HBM)
        ai = st["flops"] / st["bytes"]
        roof["intensity_flop_per_byte"] = ai
        roof["attainable"] = min(roof["peak"], ai * HBM_PEAK_GBS / 1000.0)
        roof["frac_attainable"] = roof["achieved"] / roof["attainable"]
    roof.update({"kernel": name, "launches_per_step": st["launches"] / per,
                 "avg_launch_us": 1000.0 * st["ms"] / st["launches"],
                 "algorithmic_per_launch": (st["bytes"] if roof["bound"] == "hbm" else st["flops"])
                 / st["launches"], "algorithmic_bytes_per_launch": st["bytes"] / st["launches"]})
    return roof


def exact_value(circ, level, res, reps):
    """The exact value of the bench workload: its doubled network (every noise
    as its whole superoperator, ket and bra halves in one network) contracted
    once per run by the FP64 pass; F - A(l) is the estimate's actual error."""
    import torch
    from paper_2211_17028_amd import tn
    t0 = time.perf_counter()
    pd = tn.tn_plan_build_doubled(circ, path_trials=16384)
    td = tn.tn_terms_enumerate(pd, 0)
    plan_s = time.perf_counter() - t0
    ed = tn.tn_exec_prepare([pd], [td], tn.exec_opts(use_graph=False))
    rd = ed.run()[0]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(reps):
        rd = ed.run()[0]
    torch.cuda.synchronize()
    ms = 1000.0 * (time.perf_counter() - t0) / reps
    del ed
    ek = tn.tn_exec_prepare([pd], [td], tn.exec_opts(use_graph=False, time_kernels=True))
    ek.run()
    ek.kernel_stats(reset=True)
    for _ in range(reps):
        ek.run()
    st = ek.kernel_stats(reset=True)
    del ek
    dname, dst = max(st.items(), key=lambda kv: kv[1]["ms"])
    info = pd.info()
    f = rd["A"][0]
    return {"workload": "grid5x5_12L_10depol doubled network", "F": f, "A_level": res["A"][level],
            "F_minus_A": f - res["A"][level], "bound_of_A": res["bound"], "ms_per_value": ms,
            "plan_s": plan_s, "flops_per_value": info["flops_per_term"],
            "max_log_size": info["max_log_size"],
            "tflops": info["flops_per_term"] / (ms * 1e-3) / 1e12,
            "roofline": roofline_of(dname, dst, reps),
            "kernels": {k: {"ms_per_value": v["ms"] / reps, "launches_per_value": v["launches"] / reps}
                        for k, v in sorted(st.items(), key=lambda kv: -kv[1]["ms"])}}


def offdiagonal_value(circ, level, reps):
    """<0..0|E|0..01> on the workload's ideal outputs (last qubit flipped):
    four estimates with the bond-2 targets of the polarization identity,
    packed in one schedule."""
    import numpy as np
    import torch
    from paper_2211_17028_amd import tn
    n = circ.n_qubits
    x = np.zeros((n, 2), dtype=np.complex128)
    x[:, 0] = 1
    y = x.copy()
    y[n - 1] = [0, 1]
    t0 = time.perf_counter()
    a, parts, ex = tn.offdiagonal(circ, x, y, level, True, opts=tn.exec_opts(use_graph=False))
    prep_s = time.perf_counter() - t0
    ex.run()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(reps):
        ex.run()
    torch.cuda.synchronize()
    ms = 1000.0 * (time.perf_counter() - t0) / reps
    return {"workload": "grid5x5_12L_10depol <0..0|E|0..01> level %d" % level,
            "A_xy": [[v.real, v.imag] for v in a], "ms_per_element": ms, "plan_prepare_s": prep_s,
            "terms": sum(p["n_terms"] for p in parts), "targets": 4}


def trajectories_value(circ, f_exact, reps):
    """The paper's comparison method on the same engine: 65536 quantum-trajectory
    draws of the workload's noises (seeded uniforms), one network per distinct
    draw, the sample mean through the level sums."""
    import numpy as np
    import torch
    import workloads as W
    from paper_2211_17028_amd import tn
    m = 65536
    u = W.trajectory_uniforms(m, circ.n_noises, 2211)
    t0 = time.perf_counter()
    plan = tn.tn_plan_build_trajectories(circ)
    terms = tn.tn_terms_trajectories(plan, u)
    ex = tn.tn_exec_prepare([plan], [terms], tn.exec_opts(use_graph=False))
    prep_s = time.perf_counter() - t0
    r = ex.run()[0]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(reps):
        r = ex.run()[0]
    torch.cuda.synchronize()
    ms = 1000.0 * (time.perf_counter() - t0) / reps
    x, _ = ex.values()
    x = x * m
    pat, _ = terms.get()
    return {"samples": m, "distinct_draws": len({bytes(row) for row in pat}), "ms_per_estimate": ms,
            "plan_prepare_s": prep_s, "mean": r["A"][0], "stderr": float(x.std(ddof=1) / np.sqrt(m)),
            "error_vs_exact": None if f_exact is None else r["A"][0] - f_exact}


def pruning_value(c5, plan5, terms5, ms_full, ms_full_seq, reps):
    """The learned pruning on the 225-qubit workload (level 3, held out): the
    network trained on the term values of the 25-qubit, 36-qubit and 16 of
    the packed circuits, threshold from a 1e-7 pruned-mass budget of the
    training estimates.  Timed twice: the pruned term set's estimate alone
    (prepared, as the full one), and end to end from the plan: the level-1
    pre-pass, features, network scores, the pruned enumeration, its prepare
    and one estimate (what selecting the terms costs on a new circuit)."""
    import numpy as np
    import torch
    import workloads as W
    from paper_2211_17028_amd import pruner, tn
    t0 = time.perf_counter()
    data = [pruner.training_data(W.config(2)), pruner.training_data(W.config(3))]
    for c in W.config(4)[:16]:
        data.append(pruner.training_data(c))
    net, hist, (f_dev, xs) = pruner.train(data, epochs=30)
    train_s = time.perf_counter() - t0
    total = sum(d[2]["A"][-1] for d in data)
    tau = pruner.threshold(pruner.score_candidates(net, f_dev.cpu().numpy(), "mlp"), xs, 1e-7 * total)
    full = tn.tn_exec_prepare([plan5], [terms5], tn.exec_opts(use_graph=False)).run()[0]
    # end to end from the plan, twice each (the first warms the allocator; the
    # second is reported): the full estimate (enumeration, prepare, one run)
    # and the pruned one (level-1 pre-pass, features, scores, pruned
    # enumeration, prepare, one run)
    for _ in range(2):
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        tf = tn.tn_terms_enumerate(plan5, c5.level)
        tn.tn_exec_prepare([plan5], [tf], tn.exec_opts(use_graph=False)).run()
        torch.cuda.synchronize()
        full_e2e_s = time.perf_counter() - t0
    for _ in range(2):
        sel = pruner.pruned_estimate(c5, net, tau, "mlp", plan=plan5)
    e2e_s = sel["seconds"]
    for _ in range(2):
        sel_np = pruner.pruned_estimate(c5, net, tau, "mlp")
    e2e_plan_s = sel_np["seconds"]
    keep = sel["keep"]
    tp = tn.tn_terms_enumerate(plan5, c5.level, keep=keep, min_level=2)
    ex = tn.tn_exec_prepare([plan5], [tp], tn.exec_opts(use_graph=False))
    r = ex.run()[0]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    prev = ex.submit()
    for _ in range(reps - 1):
        t = ex.submit()
        r = ex.collect(prev)[0]
        prev = t
    r = ex.collect(prev)[0]
    torch.cuda.synchronize()
    ms = 1000.0 * (time.perf_counter() - t0) / reps
    t0 = time.perf_counter()
    for _ in range(reps):
        r = ex.run()[0]
    ms_seq = 1000.0 * (time.perf_counter() - t0) / reps
    gold = os.path.join(ROOT, "tests", "golden", "config5_oracle.txt")
    g = np.loadtxt(gold) if os.path.exists(gold) else None
    return {"workload": "grid15x15_6L_20adpd_level3", "candidates": sel["candidates"], "kept": sel["kept"],
            "terms_full": full["n_terms"], "terms_contracted": r["n_contracted"],
            "contraction_factor": full["n_contracted"] / max(1, r["n_contracted"]),
            "ms_pruned": ms, "ms_full": ms_full, "time_factor_estimate_only": ms_full / ms,
            "ms_pruned_sequential": ms_seq, "ms_full_sequential": ms_full_seq,
            "end_to_end_ms": 1000.0 * e2e_s,
            "end_to_end_full_ms": 1000.0 * full_e2e_s,
            "end_to_end_with_plan_build_ms": 1000.0 * e2e_plan_s,
            "time_factor": full_e2e_s / e2e_s,
            "time_factor_note": "end to end from the plan: full estimate (enumeration, prepare, one run) / "
                                "pruned estimate (level-1 pre-pass, features, network scores, pruned "
                                "enumeration, prepare, one run)",
            "time_factor_prepared": ms_full_seq / (1000.0 * e2e_s),
            "time_factor_prepared_note": "full estimate with its schedule already prepared (one after another) / "
                                         "pruned estimate end to end from the plan",
            "error_vs_full": full["A"][-1] - r["A"][-1],
            "error_vs_oracle_full": None if g is None else g[-1] - r["A"][-1],
            "level1_error_vs_oracle_full": None if g is None else g[-1] - full["A"][1],
            "train_s": train_s}


def run_estimates(ex, steps, warmup):
    """(result, ms per estimate with two in flight, ms per estimate one after
    another) of a prepared schedule."""
    import torch
    for _ in range(warmup):
        r = ex.run()[0]
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    prev = ex.submit()
    for _ in range(steps - 1):
        t = ex.submit()
        r = ex.collect(prev)[0]
        prev = t
    r = ex.collect(prev)[0]
    torch.cuda.synchronize()
    el = time.perf_counter() - t0
    t0 = time.perf_counter()
    for _ in range(steps):
        r_seq = ex.run()
    torch.cuda.synchronize()
    el_seq = time.perf_counter() - t0
    assert [x["A"] for x in r_seq] == [x["A"] for x in ex.run()]
    return r, 1000.0 * el / steps, 1000.0 * el_seq / steps, r_seq


def run_estimates_streams(execs, streams, steps, warmup):
    """(last result, ms per estimate) of `steps` estimates spread round-robin
    over prepared schedules of the same estimate, one per stream, each with up
    to two estimates in flight: independent estimates overlap on the GPU (a
    latency-bound estimate fills a few of its CUs)."""
    import torch
    E = len(execs)
    pending = [[] for _ in range(E)]

    def step(i):
        e = i % E
        if len(pending[e]) == 2:
            execs[e].collect(pending[e].pop(0))
        pending[e].append(execs[e].submit(streams[e]))

    def drain():
        r = None
        for e in range(E):
            while pending[e]:
                r = execs[e].collect(pending[e].pop(0))[0]
        return r

    for i in range(max(warmup, 2 * E)):
        step(i)
    drain()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for i in range(steps):
        step(i)
    r = drain()
    torch.cuda.synchronize()
    return r, 1000.0 * (time.perf_counter() - t0) / steps


def kernel_pass(plans, terms, steps, warmup, tune):
    """Per-kernel durations: the schedule launched eagerly with a HIP event pair
    around every launch on that launch's stream, every level by itself (the
    estimates timed elsewhere run small consecutive levels in one launch), and
    the launches of an estimate as it is timed elsewhere."""
    import torch
    from paper_2211_17028_amd import tn
    ex = tn.tn_exec_prepare(plans, terms, tn.exec_opts(use_graph=False, time_kernels=True, tune=tune))
    for _ in range(warmup):
        ex.run()
    ex.kernel_stats(reset=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        re_ = ex.run()
    torch.cuda.synchronize()
    eel = time.perf_counter() - t0
    desc = ex.describe()
    stats = ex.kernel_stats(reset=True)
    del ex
    kernel_pass.last_desc = desc
    # launches of an estimate that is not timed launch by launch: it joins small levels
    timed = tn.tn_exec_prepare(plans, terms, tn.exec_opts(use_graph=False, tune=tune))
    launches = timed.describe()["estimate_launches"]
    del timed
    return stats, 1000.0 * eel / steps, re_, launches


def launch_floor(n_launch, ex, reps=50):
    """GPU-side latency of an estimate against the floor of its launch count.
    Both are queued behind a 1 ms spin kernel, so the host's issue time is
    hidden and the events time the GPU alone: a chain of `n_launch` dependent
    one-element kernels (torch's in-place add) on one stream, and one estimate
    of the prepared schedule `ex` (its own events, tn_exec_timing).  Medians of
    `reps` (microseconds)."""
    import torch
    x = torch.zeros(1, device="cuda")
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    floor, est = [], []
    for _ in range(reps):
        torch.cuda._sleep(2_000_000)
        e0.record()
        for _ in range(n_launch):
            x.add_(1.0)
        e1.record()
        torch.cuda.synchronize()
        floor.append(1000.0 * e0.elapsed_time(e1))
        torch.cuda._sleep(2_000_000)
        ex.run()
        est.append(1000.0 * ex.timing()[0])
    floor.sort()
    est.sort()
    return floor[len(floor) // 2], est[len(est) // 2]


def roofline_entry(stats, steps, workload):
    """Dominant kernel of the FP32 chain (the critical path; the FP64 pass
    runs beside it on its own stream and is summed in fp64_side_kernels)."""
    fp64_names = {k for k in stats if "double" in k or k.startswith("k_tile64") or k.startswith("k_gemm_tiled_c128")}
    main = {k: v for k, v in stats.items() if k not in fp64_names} or stats
    dom_name, dom = max(main.items(), key=lambda kv: kv[1]["ms"])
    roof = roofline_of(dom_name, dom, steps)
    roof["traffic"] = measured_traffic(dom_name, workload)
    side = [stats[k] for k in fp64_names]
    if side:
        roof["fp64_side_kernels"] = {"kernels": sorted(fp64_names),
                                     "ms_per_step": sum(v["ms"] for v in side) / steps,
                                     "launches_per_step": sum(v["launches"] for v in side) / steps}
    mf = [v for k, v in stats.items() if k.startswith("k_mfma")]
    if mf:
        ms_ = sum(v["ms"] for v in mf)
        roof["fp32_matrix_kernels"] = {"ms_per_step": ms_ / steps,
                                       "tflops": sum(v["flops"] for v in mf) / (ms_ * 1e-3) / 1e12,
                                       "frac": sum(v["flops"] for v in mf) / (ms_ * 1e-3) / 1e12
                                       / FP32_MFMA_PEAK_TFLOPS}
    kernels = {k: {"ms_per_step": v["ms"] / steps, "launches_per_step": v["launches"] / steps,
                   "tflops": v["flops"] / max(1e-9, v["ms"] * 1e-3) / 1e12,
                   "gbs": v["bytes"] / max(1e-9, v["ms"] * 1e-3) / 1e9}
               for k, v in sorted(stats.items(), key=lambda kv: -kv[1]["ms"])}
    return roof, kernels


def launch_roofline(desc, workload):
    """Roofline entry of the FP32 chain's longest launch (one launch of one tree
    level, durations from the kernel pass's HIP event pairs): its algorithmic
    flops (matrix-core launches) or bytes (others) per run / its average
    duration.  Secondary lines use it because the autotuner can give two levels
    the same tile shape, whose per-kernel totals then mix both launches."""
    cand = [L for L in desc["launches"] if L["phase"] == "batch" and L.get("t_n", 0) > 0 and not L["fp64"]]
    if not cand:
        return None
    L = max(cand, key=lambda x: x["t_ms"])
    name = L.get("kernel", "")
    st = {"flops": L["flops"] * L["t_n"], "bytes": L["bytes"] * L["t_n"], "ms": L["t_ms"], "launches": L["t_n"]}
    roof = roofline_of(name, st, L["t_n"])
    roof["level"] = L["level"]
    roof["tiles_or_blocks"] = L.get("n_tiles", L.get("blocks"))
    grids = None
    rec = traffic_record_path(workload)
    if os.path.exists(rec):
        with open(rec) as f:
            grids = json.load(f).get("grids")
    tiles = roof["tiles_or_blocks"]
    roof["traffic"] = measured_traffic(name, workload) if grids and tiles in grids else None
    return roof


def golden_err(cfg, A):
    import numpy as np
    gold = os.path.join(ROOT, "tests", "golden", f"config{cfg}_oracle.txt")
    if not os.path.exists(gold):
        return None
    g = np.loadtxt(gold)
    return max(abs(A[u] - g[u]) / abs(g[u]) for u in range(len(g)))


def secondary_line(cfg, args, with_roofline=False, with_plain=False):
    """One more workload, timed like the headline: the 25-qubit grid (level 2,
    436 terms), the 36-qubit QAOA (level 2, 1771 terms) or the 64 packed
    circuits (354814 terms)."""
    import workloads as W
    from paper_2211_17028_amd import tn
    cs = W.config(cfg)
    cs = cs if isinstance(cs, list) else [cs]
    t0 = time.perf_counter()
    plans = [tn.tn_plan_build(c, c.level) for c in cs]
    terms = [tn.tn_terms_enumerate(p, c.level) for p, c in zip(plans, cs)]
    plan_s = time.perf_counter() - t0
    t0 = time.perf_counter()
    ex = tn.tn_exec_prepare(plans, terms, tn.exec_opts(use_graph=False, tune=not args.no_tune))
    prep_s = time.perf_counter() - t0
    steps = max(3, args.steps // (4 if cfg == 4 else 1))
    r, ms, ms_seq, rs = run_estimates(ex, steps, max(1, args.warmup))
    del ex
    n_c = sum(x["n_contracted"] for x in rs)
    name = {2: "grid5x5_12L_10depol_level2", 3: "qaoa36_p2_20adpd_level2", 4: "mixed64_level2or3_packed"}[cfg]
    line = {"workload": name, "terms": sum(x["n_terms"] for x in rs), "contracted": n_c,
            "value": n_c / (ms * 1e-3), "unit": "contractions/s", "ms_per_estimate": ms,
            "time_to_estimate_ms": ms_seq, "plan_s": plan_s, "prepare_s": prep_s,
            "err_vs_oracle": golden_err(cfg, r["A"]) if cfg != 4 else None}
    if with_roofline:
        stats, eager_ms, _, n_launch = kernel_pass(plans, terms, steps, max(1, args.warmup), not args.no_tune)
        roof, kernels = roofline_entry(stats, steps, name)
        roof_l = launch_roofline(kernel_pass.last_desc, name)
        if roof_l is not None:
            for key in ("fp64_side_kernels", "fp32_matrix_kernels"):
                if key in roof:
                    roof_l[key] = roof[key]
            roof = roof_l
        line.update({"roofline": roof, "kernels": kernels, "launches_per_estimate": n_launch,
                     "flops_per_estimate": sum(v["flops"] for v in stats.values()) / steps})
    if with_plain:
        exp = tn.tn_exec_prepare(plans, terms, tn.exec_opts(mode=tn.TN_MODE_PLAIN, use_graph=False,
                                                            fp64_level0=False))
        exp.run()
        import torch
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        rp = exp.run()[0]
        torch.cuda.synchronize()
        pel = time.perf_counter() - t0
        line["plain"] = {"value": rp["n_contracted"] / pel, "ms_per_estimate": 1000 * pel,
                         "speedup_batched_vs_plain": line["value"] / (rp["n_contracted"] / pel)}
        del exp
    return line


def plain_rate_c5(plan5, c5):
    """PLAIN mode (the same kernels, one term at a time, no sharing, no graph)
    on the 225-qubit workload's level-1 terms (61 networks): every term runs
    the same steps, so its per-term time is that of the whole term set."""
    import torch
    from paper_2211_17028_amd import tn
    t1 = tn.tn_terms_enumerate(plan5, 1)
    exp = tn.tn_exec_prepare([plan5], [t1], tn.exec_opts(mode=tn.TN_MODE_PLAIN, use_graph=False,
                                                         fp64_level0=False))
    exp.run()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    rp = exp.run()[0]
    torch.cuda.synchronize()
    pel = time.perf_counter() - t0
    del exp
    return rp["n_contracted"] / pel, 1000.0 * pel, rp["n_contracted"]


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--traffic-from", nargs=2, metavar=("FETCH_CSV", "WRITE_CSV"),
                    help="write the HBM traffic record of --traffic-kernel on --traffic-workload from two "
                         "rocprofv3 --pmc counter files of bench.py --copy-calibration, then exit (no GPU needed)")
    ap.add_argument("--traffic-kernel", default="k_mfma_group<128,32>")
    ap.add_argument("--traffic-symbol", default=None,
                    help="the profiler's kernel name when it differs from --traffic-kernel")
    ap.add_argument("--traffic-grids", default=None,
                    help="comma-separated workgroup counts of the launches to keep")
    ap.add_argument("--traffic-workload", default="grid5x5_12L_10depol_level2")
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=20)
    ap.add_argument("--warmup", type=int, default=3)
    ap.add_argument("--headline-only", action="store_true",
                    help="only the headline workload (no secondary lines, no side measurements)")
    ap.add_argument("--secondary", type=int, default=0,
                    help="only the secondary line of config 2, 3 or 4 (with its roofline), e.g. for profiling")
    ap.add_argument("--no-plain", action="store_true")
    ap.add_argument("--no-cpu", action="store_true")
    ap.add_argument("--no-secondary", action="store_true", help="skip the 25-qubit, 36-qubit and packed lines")
    ap.add_argument("--cpu-single-terms", type=int, default=1500)
    ap.add_argument("--cpu-all-terms", type=int, default=12000)
    ap.add_argument("--no-exact", action="store_true", help="skip the exact value (doubled network)")
    ap.add_argument("--no-offdiag", action="store_true", help="skip the off-diagonal element")
    ap.add_argument("--no-trajectories", action="store_true", help="skip the quantum-trajectories comparison")
    ap.add_argument("--no-pruning", action="store_true", help="skip the learned-pruning measurement")
    ap.add_argument("--no-factored", action="store_true", help="skip the exact cross-term reuse line")
    ap.add_argument("--exact-only", action="store_true",
                    help="only the exact value of the 25-qubit workload (one estimate for A(l)); prints its JSON")
    ap.add_argument("--graph", action="store_true", help="headline from hipGraph replays instead of direct launches")
    ap.add_argument("--streams", type=int, default=4,
                    help="headline: independent estimates of the workload on this many streams (1 = one stream)")
    ap.add_argument("--no-tune", action="store_true", help="tiles by shape instead of the autotuner")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="run a 512 MiB device copy first (byte-counter calibration under rocprofv3)")
    args = ap.parse_args()
    if args.traffic_from:
        grids = {int(g) for g in args.traffic_grids.split(",")} if args.traffic_grids else None
        traffic_from_counters(args.traffic_from[0], args.traffic_from[1], args.traffic_kernel,
                              traffic_record_path(args.traffic_workload), args.traffic_symbol, grids)
        return
    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (asked for --gpus {args.gpus}); the term range would "
              f"shard across GPUs with one all-reduce of the level sums; runs on several GPUs are not implemented.",
              file=sys.stderr)
        sys.exit(2)

    import workloads as W
    c5 = W.config(5)
    level = c5.level
    # the oracle on the host first, before the GPU is touched (its workers are forked)
    cpu = None
    if not (args.no_cpu or args.headline_only or args.secondary or args.exact_only):
        cpu = cpu_baseline(5, level, args.cpu_single_terms, args.cpu_all_terms)
        print(f"cpu baseline done: {cpu['value']:.1f} contractions/s on {cpu['cores']} processes", file=sys.stderr,
              flush=True)

    import torch
    from paper_2211_17028_amd import tn

    assert torch.cuda.is_available(), "bench.py needs a HIP device"
    torch.cuda.set_device(0)
    if args.copy_calibration:
        src = torch.ones(64 << 20, dtype=torch.float64, device="cuda")   # 512 MiB
        dst = torch.empty_like(src)
        for _ in range(2):
            dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    if args.exact_only:
        c2 = W.config(2)
        p2 = tn.tn_plan_build(c2, c2.level)
        t2 = tn.tn_terms_enumerate(p2, c2.level)
        r1 = tn.tn_exec_prepare([p2], [t2], tn.exec_opts(use_graph=False)).run()[0]
        print(json.dumps({"exact_value": exact_value(c2, c2.level, r1, args.steps)}), flush=True)
        return
    if args.secondary:
        print(json.dumps({"secondary": secondary_line(args.secondary, args, with_roofline=True)}), flush=True)
        return

    workload = "grid15x15_6L_20adpd_level3"
    t0 = time.perf_counter()
    plan = tn.tn_plan_build(c5, level)
    plan_s = time.perf_counter() - t0
    terms = tn.tn_terms_enumerate(plan, level)
    # timed region: the prepared schedule run with direct launches (issued
    # level by level, the FP64 pass on its own stream), inputs resident in HBM,
    # two estimates in flight; the same steps one after another give the
    # latency of one estimate; the schedule replayed as a hipGraph beside it
    t0 = time.perf_counter()
    ex = tn.tn_exec_prepare([plan], [terms], tn.exec_opts(use_graph=args.graph, tune=not args.no_tune))
    prep_s = time.perf_counter() - t0
    res, ms_one, ms_seq, _ = run_estimates(ex, args.steps, args.warmup)
    # the same estimate on `streams` streams (one prepared schedule each),
    # estimates spread round-robin: the throughput of independent estimates
    ms_per_step, res_multi = ms_one, res
    if args.streams > 1 and not args.graph:
        execs = [ex] + [tn.tn_exec_prepare([plan], [terms], tn.exec_opts(use_graph=False, tune=not args.no_tune))
                        for _ in range(args.streams - 1)]
        strm = [torch.cuda.Stream() for _ in range(args.streams)]
        res_multi, ms_per_step = run_estimates_streams(execs, strm, args.steps, args.warmup)
        del execs, strm
    del ex
    eo = tn.tn_exec_prepare([plan], [terms], tn.exec_opts(use_graph=not args.graph, tune=not args.no_tune))
    res_o, ms_o, ms_o_seq, _ = run_estimates(eo, args.steps, args.warmup)
    del eo
    n_contracted = res["n_contracted"]
    value = n_contracted / (ms_per_step * 1e-3)
    one_stream = {"value": n_contracted / (ms_one * 1e-3), "ms_per_step": ms_one,
                  "note": "one prepared schedule, two estimates in flight on one stream"}
    other = {"mode": "direct launches" if args.graph else "hipGraph replay",
             "value": n_contracted / (ms_o * 1e-3), "ms_per_step": ms_o, "ms_per_step_sequential": ms_o_seq,
             "A_equal": res_o["A"] == res["A"]}
    # tn_estimate: the same estimate through the one-call entry point (its
    # first call builds, binds and uploads the schedule; later calls with the
    # same arguments reuse it and upload its constants again)
    _, full_ws = tn.tn_plan_workspace([plan], [terms])
    ws = torch.empty(full_ws, dtype=torch.uint8, device="cuda")
    tn.tn_release_cached()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    r_est = tn.tn_estimate([plan], [terms], ws=ws)[0]
    est_cold_ms = 1000.0 * (time.perf_counter() - t0)
    t0 = time.perf_counter()
    for _ in range(args.steps):
        r_est = tn.tn_estimate([plan], [terms], ws=ws)[0]
    est_warm_ms = 1000.0 * (time.perf_counter() - t0) / args.steps
    tn.tn_release_cached()
    del ws
    stats, eager_ms, re_, n_launch = kernel_pass([plan], [terms], args.steps, args.warmup, not args.no_tune)
    roof, kernels = roofline_entry(stats, args.steps, workload)
    eager = {"value": n_contracted / (eager_ms * 1e-3), "ms_per_step": eager_ms, "A_equal": re_[0]["A"] == res["A"],
             "note": "direct launches with a HIP event pair per launch, every level by itself (kernel durations "
                     "below)"}
    err = golden_err(5, res["A"])
    ex_f = tn.tn_exec_prepare([plan], [terms], tn.exec_opts(use_graph=False, tune=not args.no_tune))
    floor_us, est_gpu_us = launch_floor(n_launch, ex_f)
    del ex_f

    plain = None
    if not (args.no_plain or args.headline_only):
        rate, pms, pn = plain_rate_c5(plan, c5)
        plain = {"value": rate, "ms_for_sample": pms, "sample_terms": pn,
                 "note": "PLAIN mode on the workload's level-1 terms (every term runs the same steps)",
                 "speedup_batched_vs_plain": value / rate}

    factored = None
    if not (args.no_factored or args.headline_only):
        # exact cross-term reuse: the workload's 9 independent clusters
        # factored, at level 8 (1.03e9 terms in the full expansion)
        t0 = time.perf_counter()
        fe = tn.FactoredEstimate(c5, 8, opts=tn.exec_opts(use_graph=False))
        f_prep = time.perf_counter() - t0
        for _ in range(args.warmup):
            a8, _ = fe.run()
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(args.steps):
            a8, _ = fe.run()
        msf = 1000.0 * (time.perf_counter() - t0) / args.steps
        full8 = sum(math.comb(c5.n_noises, u) * 3 ** u for u in range(9))
        factored = {"level": 8, "terms_full_expansion": full8, "terms_factored": fe.terms.n,
                    "ms_per_estimate": msf, "plan_prepare_s": f_prep, "A": list(a8)}
        del fe

    secondary = None
    if not (args.no_secondary or args.headline_only):
        secondary = {
            "grid5x5_12L_10depol_level2": secondary_line(2, args, with_roofline=True, with_plain=not args.no_plain),
            "qaoa36_p2_20adpd_level2": secondary_line(3, args),
            "mixed64_level2or3_packed": secondary_line(4, args),
        }
    c2 = W.config(2)
    exact = None
    offd = traj = prune = None
    if not args.headline_only:
        if not args.no_exact:
            p2 = tn.tn_plan_build(c2, c2.level)
            t2 = tn.tn_terms_enumerate(p2, c2.level)
            r2 = tn.tn_exec_prepare([p2], [t2], tn.exec_opts(use_graph=False)).run()[0]
            exact = exact_value(c2, c2.level, r2, 5)
        offd = None if args.no_offdiag else offdiagonal_value(c2, c2.level, 20)
        traj = None if args.no_trajectories else trajectories_value(c2, exact["F"] if exact else None, 20)
        prune = None if args.no_pruning else pruning_value(c5, plan, terms, ms_one, ms_seq, args.steps)

    info = plan.info()
    line = {
        "metric": METRIC,
        "value": value,
        "unit": "contractions/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": ms_per_step,
        "time_to_estimate_ms": ms_seq,
        "time_to_estimate_note": "one estimate's latency: tn_exec_run of the prepared schedule, one after another",
        "tn_estimate_ms": est_warm_ms,
        "tn_estimate_first_call_ms": est_cold_ms,
        "tn_estimate_A_equal": r_est["A"] == res["A"],
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "c64",
        "dtype_detail": "complex64 term contractions on FP32 MFMA; complex128 all-dominant term; FP64 sums",
        "data": "synthetic",
        "config": {"workload": workload, "qubits": 225, "layers": 6, "noises": 20,
                   "level": level, "terms": res["n_terms"], "contracted": n_contracted},
        "err_vs_oracle": err,
        "A": res["A"],
        "T": res["T"],
        "paper_unit_value": 2 * value,
        "plan_s": plan_s,
        "prepare_s": prep_s,
        "launches_per_estimate": n_launch,
        "flops_per_estimate": sum(v["flops"] for v in stats.values()) / args.steps,
        "flops_per_term_plain": info["flops_per_term"],
        "roofline": roof,
        "latency_floor": {"launches": n_launch, "floor_us": floor_us, "estimate_gpu_us": est_gpu_us,
                          "frac": floor_us / est_gpu_us,
                          "note": "GPU-side times, both queued behind a spin kernel so the host's issue time is "
                                  "hidden (median of 50): floor_us = a chain of as many dependent one-element "
                                  "kernels on one stream, what an estimate of this many launches cannot go "
                                  "below on this GPU; estimate_gpu_us = one estimate of the prepared schedule; "
                                  "frac = floor / estimate"},
        "kernels": kernels,
        "timed": ("hipGraph replays, two estimates in flight (submit / collect)" if args.graph or args.streams < 2
                  else f"direct launches, {args.streams} streams with one prepared schedule each, estimates "
                       "spread round-robin, two in flight per stream (submit / collect)"),
        "streams": 1 if args.graph else max(1, args.streams),
        "one_stream": one_stream,
        "A_equal_streams": res_multi["A"] == res["A"],
        "other_mode": other,
        "eager": eager,
        "plain": plain,
        "paper_note": "the paper quotes about 1.8 h for 225 qubits with 20 noises on its own CPU server "
                      "and circuits (different circuits, level not stated; context only)",
        "factored": factored,
        "secondary": secondary,
        "exact_value": exact,
        "offdiagonal": offd,
        "trajectories": traj,
        "pruning": prune,
        "cpu_baseline": cpu,
    }
    print(json.dumps(line), flush=True)


if __name__ == "__main__":
    main()
