#!/usr/bin/env python3
"""Benchmark: loop hafnians/s and subset-terms/s at N = 50 (complex128) on one
MI355X, with the fraction of the FP64 vector peak.

A step is one full loop hafnian of the N = 50 workload matrix (all 2^25 pair
subsets: gather, Hessenberg reduction, La Budde, series, compensated sum), with
the input already resident in device memory.  The per-subset kernel's achieved
rate comes from HIP events recorded around every launch on the launch stream
(gbs_profile_*), over the same timed steps.

Prints exactly one JSON line on stdout; progress goes to stderr.
"""
import argparse
import json
import math
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

FP64_PEAK_TFLOPS = 78.6  # MI355X: 256 CU x 2.4 GHz x 128 FP64 flop/clk/CU (vector FMA)

# HBM bytes per launch (fetched, written) of the largest kernel instances of the
# N = 50 step, from rocprofv3 --pmc FETCH_SIZE and --pmc WRITE_SIZE runs scaled
# by the same counters on a plain 256 MiB device copy (fetch x2.0, write x1.0);
# the commands and raw figures are in profiles/tree_n50.md (subset tree) and
# profiles/charpoly_n50_traffic.md (register tiles, which FP64 sums of this size
# ran on before).  Valid only for the kernel sources hashed here: any change to
# them reports null until re-measured.
TREE_TRAFFIC_SOURCES = ("paper_2010_15595_amd/csrc/tree_device.h", "paper_2010_15595_amd/csrc/tree_kernels.h",
                        "paper_2010_15595_amd/csrc/tree_launch.h")
TREE_TRAFFIC = {
    "sha256": "056b912bbc1bae1dff4bb03d24a51cea2ed4b6f8f523f58752d67a5a28b92bcc",
    "kernels": {  # FETCH_SIZE / WRITE_SIZE KiB per dispatch
        "tree_sub_kernel<25>": (1920181008, 4194304),  # 937588.4 / 4096.0
    },
}
TRAFFIC_SOURCES = ("paper_2010_15595_amd/csrc/lhaf_device.h", "paper_2010_15595_amd/csrc/lhaf_kernels.h",
                   "paper_2010_15595_amd/csrc/charpoly_l88.hip", "paper_2010_15595_amd/csrc/charpoly_l84.hip",
                   "paper_2010_15595_amd/csrc/charpoly_l44.hip")
TRAFFIC = {
    "sha256": "6b2e424ae8298050ff7b6175df2aea57b3ec8a99a729673c550b9eb9d629ac1e",
    "kernels": {  # FETCH_SIZE / WRITE_SIZE KiB per dispatch
        "charpoly_kernel<8, 4, 3, 6, double2, 64, 0>": (1960755, 899399066),  # 957.4 / 878319.4
        "charpoly_kernel<8, 4, 4, 7, double2, 64, 2>": (1380634, 898611840),  # 674.1 / 877550.6
        "charpoly_kernel<8, 4, 3, 6, double2, 64, 2>": (1198259, 770238720),  # 585.1 / 752186.2
        "charpoly_kernel<8, 8, 4, 4, double2, 64, 4>": (1136717, 770238720),  # 555.0 / 752186.2
        "charpoly_kernel<8, 4, 3, 5, double2, 64, 0>": (1140992, 706052160),  # 557.1 / 689504.1
        "charpoly_kernel<8, 4, 4, 8, double2, 64, 2>": (1281472, 706052160),  # 625.7 / 689504.1
        "charpoly_kernel<4, 4, 5, 5, double2, 64, 2>": (1404928, 882565200),  # 686.0 / 861880.1
        "charpoly_kernel<8, 4, 4, 8, double2, 64, 0>": (1309888, 882565200),  # 639.6 / 861880.1
        "charpoly_kernel<4, 4, 4, 4, double2, 64, 0>": (1136128, 467240400),  # 554.8 / 456289.5
        "charpoly_kernel<8, 8, 5, 5, double2, 64, 6>": (1040064, 467240400),  # 507.8 / 456289.5
    },
}


def sources_sha256(sources=TRAFFIC_SOURCES):
    import hashlib

    h = hashlib.sha256()
    for rel in sources:
        with open(os.path.join(ROOT, rel), "rb") as f:
            h.update(f.read())
    return h.hexdigest()


def traffic_entry(kernel):
    """Measured HBM bytes per launch of `kernel`, if they were taken on it and on these sources."""
    for table, sources in ((TREE_TRAFFIC, TREE_TRAFFIC_SOURCES), (TRAFFIC, TRAFFIC_SOURCES)):
        if kernel in table["kernels"] and table["sha256"] == sources_sha256(sources):
            return sum(table["kernels"][kernel])
    return None


def log(*a):
    print(*a, file=sys.stderr, flush=True)


def workload(N):
    from paper_2010_15595_amd import workloads

    st = workloads.config3(N)
    return st


def cpu_model():
    try:
        with open("/proc/cpuinfo") as f:
            for line in f:
                if line.startswith("model name"):
                    return line.split(":", 1)[1].strip()
    except OSError:
        pass
    return None


def _terms_rate(A, n, seconds, threads, rng):
    """Subset terms per second of the fp64 oracle over uniform random pair
    subsets, on `threads` OpenMP threads, for about `seconds`."""
    import numpy as np

    import oracle

    probe = rng.integers(0, 1 << n, size=max(64, 8 * threads), dtype=np.uint64)
    t0 = time.perf_counter()
    oracle.terms(A, probe, prec="d", nthreads=threads)
    dt = time.perf_counter() - t0
    rate = len(probe) / dt
    # the probe underestimates the rate (thread start-up); resize once from a real sample
    cap = 1.5e7
    count = len(probe)
    for _ in range(2):
        count = int(max(len(probe), min(rate * seconds, cap)))
        sample = rng.integers(0, 1 << n, size=count, dtype=np.uint64)
        t0 = time.perf_counter()
        oracle.terms(A, sample, prec="d", nthreads=threads)
        dt = time.perf_counter() - t0
        rate = count / dt
        if dt >= 0.5 * seconds or count >= cap:
            break
    return rate, count, dt


def cpu_baseline(A, N, seconds, one_thread_seconds):
    """The oracle (double) on a uniform random sample of the workload's pair
    subsets, on all host threads and on one thread; scaled to lhaf/s by 2^n
    subsets per lhaf."""
    import numpy as np

    import oracle

    n = N // 2
    rng = np.random.default_rng(1234)
    threads = oracle.max_threads()
    rate, count, dt = _terms_rate(A, n, seconds, threads, rng)
    res = {
        "value": rate / float(1 << n),
        "unit": "lhaf/s",
        "cores": threads,
        "kind": "oracle",
        "cpu_model": cpu_model(),
        "subset_terms_per_s": rate,
        "seconds": dt,
        "sample": f"{count} pair subsets drawn uniformly from the 2^{n} of the N={N} workload, "
                  f"fp64 oracle (Householder Hessenberg + La Budde + mat-vec loop terms), "
                  f"{threads} OpenMP threads; lhaf/s = subset-terms/s / 2^{n}",
    }
    if one_thread_seconds > 0:
        r1, c1, d1 = _terms_rate(A, n, one_thread_seconds, 1, rng)
        res["one_thread"] = {"value": r1 / float(1 << n), "unit": "lhaf/s", "cores": 1,
                             "subset_terms_per_s": r1, "seconds": d1, "sample": f"{c1} pair subsets, 1 thread"}
    return res


def batch_cpu_baseline(mats, seconds, one_thread_seconds):
    """The oracle (double, full power-trace sums) on items drawn uniformly at
    random from the batch, on all host threads and on one thread: items/s over
    the sample (its mean cost estimates the batch's)."""
    import numpy as np

    import oracle

    rng = np.random.default_rng(4321)
    threads = oracle.max_threads()

    def leg(sec, nthr):
        done, t0 = 0, time.perf_counter()
        dims = []
        while done < 4 or time.perf_counter() - t0 < sec:
            A = mats[int(rng.integers(0, len(mats)))]
            oracle.lhaf_pt(A, prec="d", nthreads=nthr)
            dims.append(A.shape[0])
            done += 1
        dt = time.perf_counter() - t0
        return done / dt, done, dt, dims

    rate, done, dt, dims = leg(seconds, threads)
    res = {"value": rate, "unit": "lhaf/s", "cores": threads, "kind": "oracle", "cpu_model": cpu_model(),
           "seconds": dt,
           "sample": f"{done} items drawn uniformly from the {len(mats)} of the batch (mean N {np.mean(dims):.1f}), "
                     f"full fp64 oracle power-trace sums, {threads} OpenMP threads"}
    if one_thread_seconds > 0:
        r1, d1, t1, dm1 = leg(one_thread_seconds, 1)
        res["one_thread"] = {"value": r1, "unit": "lhaf/s", "cores": 1, "seconds": t1,
                             "sample": f"{d1} items (mean N {np.mean(dm1):.1f}), 1 thread"}
    return res


def roofline_from_profile(prof, steps, note):
    """Roofline entry of the dominant kernel instance: its operations (subset
    tree) or yardstick flops (per-subset kernels) per launch over its average launch duration (HIP event pairs on the
    launch streams)."""
    achieved = prof["dominant_flops"] / (prof["dominant_ms"] / 1000.0) / 1e12 if prof["dominant_ms"] > 0 else None
    achieved_all = prof["charpoly_flops"] / (prof["charpoly_ms"] / 1000.0) / 1e12 if prof["charpoly_ms"] > 0 else None
    return {
        "bound": "alu",
        "kernel": prof["dominant_kernel"],
        "kernel_note": note,
        "achieved": achieved,
        "peak": FP64_PEAK_TFLOPS,
        "unit": "TFLOP/s",
        "frac": (achieved / FP64_PEAK_TFLOPS) if achieved else None,
        "flops_per_launch": prof["dominant_flops"] / max(1, prof["dominant_launches"]),
        "avg_launch_ms": prof["dominant_ms"] / max(1, prof["dominant_launches"]),
        "launches_per_step": prof["dominant_launches"] / steps,
        "all_per_subset_kernels": {"achieved": achieved_all,
                                   "frac": (achieved_all / FP64_PEAK_TFLOPS) if achieved_all else None,
                                   "launches_per_step": prof["charpoly_launches"] / steps,
                                   "kernel_ms_per_step": prof["charpoly_ms"] / steps},
    }


def bench_batch(args, gbs):
    """One step = one replay of the captured batch plan over all items."""
    import numpy as np
    import torch

    from paper_2010_15595_amd import workloads

    st = workloads.config4(count=args.batch_count)
    mats = [gbs.expand(st["B"], st["gamma"], pat) for pat in st["patterns"]]
    dims = [a.shape[0] for a in mats]
    prec = gbs.GBS_FP64 if args.precision == "fp64" else gbs.GBS_FP32_COMP
    torch.cuda.set_device(0)
    gbs.init(0)
    dev = torch.device("cuda:0")
    t0 = time.perf_counter()
    plan = gbs.BatchPlan(dims, prec=prec, autotune=not args.no_autotune)
    info = plan.info()
    plan_s = time.perf_counter() - t0
    log(f"plan ({plan_s:.2f} s): {info}")
    packed = torch.from_numpy(gbs.pack(mats)).to(dev)
    out = torch.zeros(len(mats), dtype=torch.complex128, device=dev)
    ab = torch.zeros(len(mats), dtype=torch.float64, device=dev)
    stream = torch.cuda.current_stream(dev)
    for _ in range(args.warmup):
        plan.run(packed, out, ab, stream)
    torch.cuda.synchronize()
    ref_out = out.cpu().numpy().copy()
    ev0 = torch.cuda.Event(enable_timing=True)
    ev1 = torch.cuda.Event(enable_timing=True)
    ev0.record(stream)
    for _ in range(args.steps):
        plan.run(packed, out, ab, stream)
    ev1.record(stream)
    torch.cuda.synchronize()
    gpu_ms = ev0.elapsed_time(ev1)
    res = out.cpu().numpy()
    if args.warmup > 0 and not np.array_equal(res, ref_out):
        log("WARNING: batch results changed between replays")
    sec = gpu_ms / 1000.0
    items_per_s = args.steps * len(mats) / sec
    terms_per_s = args.steps * info["subset_terms"] / sec
    flops_per_s = args.steps * info["yardstick_flops"] / sec
    log(f"{args.steps} replays in {gpu_ms:.1f} ms: {items_per_s:.1f} lhaf/s, {terms_per_s:.4e} subset-terms/s, "
        f"{flops_per_s / 1e12:.2f} yardstick TFLOP/s")
    # the plain form: the same items one at a time through the single-matrix entry point
    plain = None
    if not args.no_plain:
        import torch as _t

        mats_dev = [_t.from_numpy(a).to(dev) for a in mats]
        o1 = _t.zeros(1, dtype=_t.complex128, device=dev)
        a1 = _t.zeros(1, dtype=_t.float64, device=dev)
        pv = np.zeros(len(mats), dtype=np.complex128)
        for a in mats_dev[:8]:
            gbs.lhaf_device(a, o1, a1, stream, prec)
        torch.cuda.synchronize()
        e0 = torch.cuda.Event(enable_timing=True)
        e1 = torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        outs = _t.zeros(len(mats), dtype=_t.complex128, device=dev)
        for i, a in enumerate(mats_dev):
            gbs.lhaf_device(a, outs[i:i + 1], None, stream, prec)
        e1.record(stream)
        torch.cuda.synchronize()
        pms = e0.elapsed_time(e1)
        pv = outs.cpu().numpy()
        scale = np.maximum(ab.cpu().numpy(), 1e-300)
        plain = {"lhaf_per_s": len(mats) / (pms / 1000.0), "ms": pms,
                 "max_normwise_diff_vs_batch": float(np.max(np.abs(pv - res) / scale))}
        log(f"plain form: {len(mats)} single lhaf_device calls in {pms:.1f} ms = {plain['lhaf_per_s']:.1f} lhaf/s; "
            f"batch speedup {plain['ms'] / (gpu_ms / args.steps):.2f}x; max |diff|/sum|t| {plain['max_normwise_diff_vs_batch']:.2e}")
    # roofline pass: the same schedule issued eagerly (graph replays cannot be
    # bracketed by events per launch) on one stream, every persistent launch
    # timed alone on the device
    gbs.profile_enable(True)
    for _ in range(args.roofline_steps):
        plan.run(packed, out, ab, stream)
    torch.cuda.synchronize()
    prof = gbs.profile_read()
    gbs.profile_enable(False)
    if not np.array_equal(out.cpu().numpy(), res):
        log("WARNING: eager (profiled) run differs from the graph replays")
    roof = roofline_from_profile(prof, args.roofline_steps,
                                 "subtree or elimination kernel of one order over a group of the batch's items; "
                                 f"average launch from {args.roofline_steps} eager profiled run(s) of the captured "
                                 "schedule right after the timed graph replays, one launch at a time")
    roof["traffic"] = None
    log(f"roofline: {roof['kernel']} {roof['achieved']:.2f} TFLOP/s ({100 * roof['frac']:.1f}% of FP64 peak); "
        f"all per-subset launches {roof['all_per_subset_kernels']['achieved']:.2f} TFLOP/s")
    result = {
        "metric": "loop hafnians/s and subset-terms/s, batched uneven N",
        "value": items_per_s,
        "unit": "lhaf/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": gpu_ms / args.steps,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "c128" if args.precision == "fp64" else "c128 Hessenberg + c64 La Budde/series (compensated)",
        "data": "synthetic",
        "config": {
            "workload": f"{len(mats)} loop hafnians of uneven even N in [10, 36] expanded from one 100-mode pure "
                        "state (r=1.0, sigma=0.2), chain-like photon patterns; one HIP graph replay per step",
            "items": len(mats),
            "subset_terms_per_step": info["subset_terms"],
            "tile_subsets": info["tile_subsets"],
            "graph_kernel_nodes": info["kernel_nodes"],
            "rounds": info["rounds"],
        },
        "subset_terms_per_s": terms_per_s,
        "yardstick_tflops": flops_per_s / 1e12,
        "pct_fp64_peak": 100.0 * prof["charpoly_flops"] / args.roofline_steps * args.steps / sec
                         / (FP64_PEAK_TFLOPS * 1e12),
        "plan_seconds": plan_s,
        "plain_form": plain,
        "roofline": roof,
    }
    plan.close()
    if not args.no_cpu_baseline:
        log(f"cpu baseline: oracle on items of the batch for ~{args.cpu_seconds:.0f} s ...")
        result["cpu_baseline"] = batch_cpu_baseline(mats, args.cpu_seconds, args.cpu_one_thread_seconds)
        log(f"cpu baseline: {result['cpu_baseline']['value']:.2f} lhaf/s on {result['cpu_baseline']['cores']} threads")
    print(json.dumps(result), flush=True)


FIG1_PAPER_TVD_PCT = {  # Fig. 1 of the paper: modes -> (expected TVD %, TVD % of the algorithm), 200000 samples
    1: (0.0673495237048602, 0.0647525723905912), 2: (0.160458530772439, 0.156253393597565),
    3: (0.326807192070019, 0.330725502822026), 4: (0.574908610108614, 0.560088803231853),
    5: (0.956263734732863, 0.945682615697726), 6: (1.60448581724988, 1.60403702590985),
}


def sampler_state(M, seed):
    """Fig. 1 setting: squeezing r = 0.5 in every mode into a Haar-random interferometer, no displacement."""
    from paper_2010_15595_amd import workloads

    return workloads.pure_state(M, 0.5, 0.0, seed=seed)


def bench_sampler(args, gbs):
    """One step = one gbs_sample_pure call drawing args.samples samples of the
    6-mode Fig. 1 state (r = 0.5, Haar interferometer, cutoff 6)."""
    import numpy as np

    M, cutoff = args.sampler_modes, 6
    st = sampler_state(M, seed=2024)
    rng = np.random.default_rng(7)
    n = args.samples
    z = rng.standard_normal((n, 2 * (M - 1)))
    u = rng.random((n, M))
    prec = gbs.GBS_FP64 if args.precision == "fp64" else gbs.GBS_FP32_COMP
    gbs.init(0)
    for _ in range(args.warmup):
        ref = gbs.sample_pure(st["Q"], st["alpha_vec"], cutoff, z, u, prec=prec)
    t0 = time.perf_counter()
    infos = []
    for _ in range(args.steps):
        s, info = gbs.sample_pure(st["Q"], st["alpha_vec"], cutoff, z, u, prec=prec, with_info=True)
        infos.append(info)
    sec = time.perf_counter() - t0
    if args.warmup > 0 and not np.array_equal(s, ref):
        log("WARNING: samples changed between identical calls")
    info = infos[-1]
    rate = args.steps * n / sec
    log(f"{args.steps} x {n} samples in {sec:.2f} s: {rate:.1f} samples/s, "
        f"{args.steps * info['loop_hafnians'] / sec:.3e} lhaf/s; info {info}")
    result = {
        "metric": "samples/s of the conditional sampling chain (Fig. 1 setting)",
        "value": rate,
        "unit": "samples/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": 1000.0 * sec / args.steps,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "c128" if args.precision == "fp64" else "c128 Hessenberg + c64 La Budde/series (compensated)",
        "data": "synthetic",
        "config": {
            "workload": f"{n} samples per step of a {M}-mode pure state: r = 0.5 squeezing in every mode into a "
                        f"Haar-random interferometer, cutoff {cutoff}; host random numbers, host samples out "
                        "(wall clock of the synchronous call, PCIe included)",
            "samples_per_step": n,
            "modes": M,
            "cutoff": cutoff,
        },
        "loop_hafnians_per_s": args.steps * info["loop_hafnians"] / sec,
        "subset_terms_per_step": info["subset_terms"],
        "max_dim": info["max_dim"],
        "host_setup_ms": info["setup_ms"],
        "mean_photons": float(s.sum(axis=1).mean()),
    }
    if not args.no_cpu_baseline:
        # the oracle chain (numpy conditioning, long-double loop hafnians) on the first samples of the
        # same random numbers, for about args.cpu_seconds; its draws must equal the GPU's
        from oracle import sampler as osampler

        t0 = time.perf_counter()
        done = 0
        while done < n and (done < 8 or time.perf_counter() - t0 < args.cpu_seconds):
            ref = osampler.sample_chain(st["Q"], st["alpha_vec"], cutoff, z[done], u[done])
            if list(ref) != [int(x) for x in s[done]]:
                log(f"WARNING: oracle sample {done} differs from the GPU's: {ref} vs {list(s[done])}")
            done += 1
        dt = time.perf_counter() - t0
        import oracle

        result["cpu_baseline"] = {"value": done / dt, "unit": "samples/s", "cores": oracle.max_threads(),
                                  "kind": "oracle", "seconds": dt,
                                  "sample": f"the first {done} samples of the same workload and random numbers "
                                  "through the oracle's sampling chain (numpy conditioning; its C loop hafnians may "
                                  "use the OpenMP threads counted in cores)"}
        log(f"cpu baseline: {done} oracle samples in {dt:.1f} s")
    print(json.dumps(result), flush=True)


def fig1_tvd(args, gbs):
    """Fig. 1 of the paper: for 1..6 modes and 10 Haar-random unitaries, the
    total variation distance between args.samples samples of the chain and the
    exact distribution of patterns with s_i <= 6, beside the TVD of as many
    samples drawn from the exact distribution itself.  Exact probabilities of
    all patterns with at most args.tvd_max_photons photons come from one batch
    plan of loop hafnians (the rest weigh below the statistical resolution)."""
    import itertools

    import numpy as np

    cutoff, n = 6, args.samples
    gbs.init(0)
    rows = {}
    for M in range(1, args.sampler_modes + 1):
        tv, ex = [], []
        for rep in range(args.tvd_unitaries):
            st = sampler_state(M, seed=1000 * M + rep)
            B, gamma, pvac = gbs.pure_state(st["Q"], st["alpha_vec"])
            pats = [p for p in itertools.product(range(cutoff + 1), repeat=M) if sum(p) <= args.tvd_max_photons]
            mats = [gbs.expand(B, gamma, p) for p in pats]
            plan = gbs.BatchPlan([a.shape[0] for a in mats])
            import torch

            dev = torch.device("cuda:0")
            packed = torch.from_numpy(gbs.pack(mats)).to(dev)
            out = torch.zeros(len(mats), dtype=torch.complex128, device=dev)
            plan.run(packed, out, None, torch.cuda.current_stream(dev))
            torch.cuda.synchronize()
            plan.close()
            lh = out.cpu().numpy()
            fact = np.array([np.prod([math.factorial(x) for x in p]) for p in pats], dtype=float)
            prob = pvac * np.abs(lh) ** 2 / fact
            prob = prob / prob.sum()
            rng = np.random.default_rng(rep + 17 * M)
            s = gbs.sample_pure(st["Q"], st["alpha_vec"], cutoff, rng.standard_normal((n, 2 * (M - 1))),
                                rng.random((n, M)))
            base = (cutoff + 1) ** np.arange(M - 1, -1, -1)
            codes = s @ base
            emp = np.bincount(codes, minlength=(cutoff + 1) ** M) / n
            ref = np.zeros_like(emp)
            ref[np.array(pats) @ base] = prob
            tv.append(50.0 * np.abs(emp - ref).sum())
            ex.append(50.0 * np.abs(rng.multinomial(n, ref) / n - ref).sum())
        rows[M] = {"tvd_pct": float(np.mean(tv)), "tvd_pct_std": float(np.std(tv)),
                   "expected_tvd_pct": float(np.mean(ex)), "expected_tvd_pct_std": float(np.std(ex)),
                   "paper_expected_pct": FIG1_PAPER_TVD_PCT[M][0], "paper_algorithm_pct": FIG1_PAPER_TVD_PCT[M][1]}
        log(f"M={M}: {rows[M]}")
    print(json.dumps({"metric": "total variation distance % (Fig. 1)", "samples": n, "cutoff": cutoff,
                      "unitaries": args.tvd_unitaries, "max_photons_in_reference": args.tvd_max_photons,
                      "modes": rows}), flush=True)


def fig2_accuracy(args, gbs):
    """Fig. 2 of the paper: relative error of the loop hafnian of the n x n
    all-ones matrix against the telephone number T(n), for the FP64 and the
    double-double paths, beside the paper's long-double errors."""
    from fractions import Fraction

    import numpy as np

    import oracle

    paper = {}
    with open(os.path.join(ROOT, "tests", "golden", "fig2_allones_relerr.txt")) as f:
        for line in f:
            if line.strip() and not line.startswith("#"):
                k, v = line.split()
                paper[int(k)] = float(v)
    gbs.init(0)
    rows = {}
    for n in args.fig2_sizes:
        A = np.ones((n, n), dtype=complex)
        T = oracle.telephone(n)
        t0 = time.perf_counter()
        v64 = gbs.lhaf(A)
        t64 = time.perf_counter() - t0
        t0 = time.perf_counter()
        hi, d = gbs.lhaf(A, prec=gbs.GBS_DD, with_diag=True)
        tdd = time.perf_counter() - t0
        lo = d["lhaf_lo"]
        e64 = float(abs(Fraction(v64.real) - T) / T) + abs(v64.imag) / T
        edd = float(abs(Fraction(hi.real) + Fraction(lo.real) - T) / T) + abs(hi.imag + lo.imag) / T
        rows[n] = {"fp64_relerr": e64, "dd_relerr": edd, "paper_long_double_relerr": paper.get(n),
                   "kappa": d["kappa"], "fp64_seconds": t64, "dd_seconds": tdd}
        log(f"n={n}: {rows[n]}")
    print(json.dumps({"metric": "relative error of lhaf(all-ones n x n) vs T(n) (Fig. 2)", "sizes": rows}),
          flush=True)


def fig3_sweep(args, gbs):
    """Fig. 3 of the paper: loop-hafnian time on random complex symmetric
    matrices (Re, Im ~ U[0, 1), symmetrised) for even N, FP64 (and double-double
    up to --fig3-dd-max) on the GPU beside the paper's long-double times on 96
    vCPUs, with the dominant per-subset instance's roofline at each N."""
    import numpy as np
    import torch

    from paper_2010_15595_amd import workloads

    paper = {}
    with open(os.path.join(ROOT, "tests", "golden", "fig3_times.txt")) as f:
        for line in f:
            if line.strip() and not line.startswith("#"):
                k, v = line.split()
                paper[int(k)] = float(v)
    torch.cuda.set_device(0)
    gbs.init(0)
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream(dev)
    out = torch.zeros(1, dtype=torch.complex128, device=dev)
    ab = torch.zeros(1, dtype=torch.float64, device=dev)
    rows = {}
    for N in args.fig3_sizes:
        A = workloads.random_uniform_symmetric(N, seed=N)
        A_dev = torch.from_numpy(A).to(dev)
        n = N // 2
        # (FP64 sums up to MAX_BATCH_DIM run on the subset tree, which has no lane grid to choose)
        if not args.no_autotune and N > gbs.MAX_BATCH_DIM:
            gbs.autotune(n)
        gbs.lhaf_device(A_dev, out, ab, stream)
        torch.cuda.synchronize()
        # at least ~1 s of GPU time per size, whole loop hafnians
        t0 = time.perf_counter()
        gbs.lhaf_device(A_dev, out, ab, stream)
        torch.cuda.synchronize()
        est = time.perf_counter() - t0
        steps = max(1, min(200, int(1.0 / max(est, 1e-6))))
        # whole loop hafnians timed without the per-launch profiling events,
        # then a profiled pass of the same calls for the dominant instance
        ev0, ev1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        ev0.record(stream)
        for _ in range(steps):
            gbs.lhaf_device(A_dev, out, ab, stream)
        ev1.record(stream)
        torch.cuda.synchronize()
        sec = ev0.elapsed_time(ev1) / 1000.0 / steps
        psteps = max(1, min(steps, 20))
        gbs.profile_enable(True)
        for _ in range(psteps):
            gbs.lhaf_device(A_dev, out, ab, stream)
        torch.cuda.synchronize()
        prof = gbs.profile_read()
        gbs.profile_enable(False)
        flops = gbs.yardstick_flops(N)
        roof = roofline_from_profile(prof, psteps, "subtree kernel, 32 subsets per wavefront")
        row = {"fp64_seconds": sec, "fp64_lhaf_per_s": 1.0 / sec, "subset_terms_per_s": float(1 << n) / sec,
               "pct_fp64_peak": 100.0 * prof["charpoly_flops"] / psteps / sec / (FP64_PEAK_TFLOPS * 1e12),
               "yardstick_tflops": flops / sec / 1e12,
               "dominant_kernel": roof["kernel"], "dominant_frac": roof["frac"],
               "paper_seconds": paper.get(N), "speedup_vs_paper": paper[N] / sec if N in paper else None,
               "steps": steps}
        if N <= args.fig3_dd_max:
            gbs.lhaf(A, prec=gbs.GBS_DD)
            t0 = time.perf_counter()
            _, d = gbs.lhaf(A, prec=gbs.GBS_DD, with_diag=True)
            row["dd_seconds"] = d["kernel_ms"] / 1000.0
            row["dd_speedup_vs_paper"] = paper[N] / row["dd_seconds"] if N in paper else None
        if not args.no_autotune and N > gbs.MAX_BATCH_DIM:
            gbs.set_layout(n, 0, -1)
        rows[N] = row
        log(f"N={N}: {row}")
    print(json.dumps({"metric": "loop-hafnian seconds vs N on Fig. 3 inputs (Sec. IV)", "unit": "s",
                      "higher_is_better": False, "n_gpus": 1, "data": "synthetic",
                      "config": {"workload": "random complex symmetric N x N, Re, Im ~ U[0,1), (R + R^T)/2, seed N",
                                 "paper": "long double, 96 vCPUs (Azure D96a v4, 2.345 GHz)"},
                      "sizes": rows}), flush=True)


def shard_split(args, gbs):
    """One GPU's share of a loop hafnian split over several GPUs: the N matrix
    of the default line split --shards ways (every shard the same share of
    every size class), each shard timed alone on the one GPU with HIP events
    on its stream, the records folded on the host and compared with the
    whole sum."""
    import numpy as np
    import torch

    N, G = args.N, args.shards
    st = workload(N)
    A = gbs.expand(st["B"], st["gamma"], st["pattern"])
    n = (N + 1) // 2
    torch.cuda.set_device(0)
    gbs.init(0)
    dev = torch.device("cuda:0")
    stream = torch.cuda.current_stream(dev)
    A_dev = torch.from_numpy(A).to(dev)
    if not args.no_autotune:
        gbs.autotune(n)
    out = torch.zeros(1, dtype=torch.complex128, device=dev)
    ab = torch.zeros(1, dtype=torch.float64, device=dev)
    rec = torch.zeros((G, 5), dtype=torch.float64, device=dev)

    def timed(fn):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record(stream)
        fn()
        e1.record(stream)
        torch.cuda.synchronize()
        return e0.elapsed_time(e1)

    gbs.lhaf_device(A_dev, out, ab, stream)  # warm-up
    torch.cuda.synchronize()
    whole_ms = timed(lambda: gbs.lhaf_device(A_dev, out, ab, stream))
    shard_ms = [timed(lambda g=g: gbs.lhaf_device_shard(A_dev, rec[g], g, G, stream)) for g in range(G)]
    val, abs_sum = gbs.combine_partials(rec.cpu().numpy())
    ref = complex(out.cpu().numpy()[0])
    diff = abs(val - ref) / float(ab.cpu().numpy()[0])
    log(f"N={N} in {G} shards: " + " ".join(f"{t:.1f}" for t in shard_ms) + f" ms; whole {whole_ms:.1f} ms; "
        f"|fold - whole| / sum|t| {diff:.2e}")
    print(json.dumps({
        "metric": f"ms per shard of one N={N} loop hafnian split {G} ways (one GPU's share, timed alone)",
        "value": max(shard_ms), "unit": "ms", "higher_is_better": False, "n_gpus": 1, "data": "synthetic",
        "dtype": "c128",
        "config": {"workload": f"the N={N} matrix of the default line; shard g of {G} takes colex ranks "
                               f"[C g / {G}, C (g + 1) / {G}) of every size class"},
        "shard_ms": shard_ms, "whole_ms": whole_ms, "sum_of_shards_over_whole": sum(shard_ms) / whole_ms,
        "max_over_mean": max(shard_ms) / (sum(shard_ms) / G), "fold_vs_whole_normwise": diff,
    }), flush=True)


def methods_comparison(args, gbs):
    """Sec. IV compares La Budde with diagonalisation: the same subset sum on
    the LDS-resident reference kernels with either method (FP64), beside the
    production FP64 kernels, each scored against the double-double value."""
    from paper_2010_15595_amd import workloads

    gbs.init(0)
    rows = {}
    for N in args.method_sizes:
        st = workloads.config3(N)
        A = gbs.expand(st["B"], st["gamma"], st["pattern"])
        ref, dref = gbs.lhaf(A, prec=gbs.GBS_DD, with_diag=True)
        row = {"kappa": dref["kappa"], "dd_kernel_ms": dref["kernel_ms"]}
        for name, fn in (("production_fp64", lambda: gbs.lhaf(A, with_diag=True)),
                         ("labudde_lds_fp64", lambda: gbs.lhaf_method(A, gbs.GBS_CHARPOLY_LABUDDE, with_diag=True)),
                         ("eigen_lds_fp64", lambda: gbs.lhaf_method(A, gbs.GBS_CHARPOLY_EIGEN, with_diag=True))):
            fn()  # warm
            v, d = fn()
            row[name] = {"kernel_ms": d["kernel_ms"], "err_over_sum_abs": abs(v - ref) / dref["abs_sum"],
                         "rel_err": abs(v - ref) / abs(ref)}
        row["eigen_over_labudde_time"] = row["eigen_lds_fp64"]["kernel_ms"] / row["labudde_lds_fp64"]["kernel_ms"]
        rows[N] = row
        log(f"N={N}: {row}")
    print(json.dumps({"metric": "La Budde vs eigenvalue characteristic polynomials (Sec. IV)", "sizes": rows}),
          flush=True)


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=5)
    ap.add_argument("--warmup", type=int, default=1)
    ap.add_argument("--N", type=int, default=50)
    ap.add_argument("--cpu-seconds", type=float, default=15.0)
    ap.add_argument("--cpu-one-thread-seconds", type=float, default=8.0,
                    help="length of the one-thread leg of the oracle baseline (0: skip)")
    ap.add_argument("--roofline-steps", type=int, default=2,
                    help="batch: eager profiled runs of the schedule for the roofline entry")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--precision", choices=["fp64", "fp32comp", "dd"], default="fp64",
                    help="fp32comp: La Budde, series and per-lane sums in complex FP32 (Hessenberg FP64); "
                         "dd: every step in double-double (single evaluations, N <= 56)")
    ap.add_argument("--no-autotune", action="store_true",
                    help="skip the lane-grid autotuner (use the heuristic or GBS_AUTOTUNE_CACHE)")
    ap.add_argument("--print-source-hash", action="store_true",
                    help="print the hash of the kernel sources the traffic figures are tied to")
    ap.add_argument("--copy-calibration", action="store_true",
                    help="only run a plain 256 MiB device-to-device copy (HBM counter calibration)")
    ap.add_argument("--workload", choices=["n50", "batch", "sampler", "tvd", "fig2", "fig3", "methods", "shard"],
                    default="n50",
                    help="batch: 4096 loop hafnians of uneven N in [10, 36] from one 100-mode state, "
                         "one captured graph of persistent launches per step; sampler: samples/s of the "
                         "conditional sampling chain in the Fig. 1 setting; tvd: the Fig. 1 experiment; "
                         "shard: the N loop hafnian split --shards ways, each share timed alone")
    ap.add_argument("--shards", type=int, default=8, help="shard: number of shares of the subset sum")
    ap.add_argument("--samples", type=int, default=200000, help="sampler / tvd: samples per step / per unitary")
    ap.add_argument("--sampler-modes", type=int, default=6)
    ap.add_argument("--tvd-unitaries", type=int, default=10)
    ap.add_argument("--tvd-max-photons", type=int, default=14)
    ap.add_argument("--method-sizes", type=int, nargs="+", default=[16, 24, 32, 36, 40])
    ap.add_argument("--fig2-sizes", type=int, nargs="+", default=[30, 34, 38, 42, 46, 48, 50])
    ap.add_argument("--batch-count", type=int, default=4096)
    ap.add_argument("--fig3-sizes", type=int, nargs="+", default=list(range(30, 57, 2)))
    ap.add_argument("--fig3-dd-max", type=int, default=44, help="fig3: largest N also timed in double-double")
    ap.add_argument("--no-plain", action="store_true", help="batch: skip timing the items one at a time")
    args = ap.parse_args()
    if args.print_source_hash:
        print(sources_sha256(TREE_TRAFFIC_SOURCES), sources_sha256())
        return
    if args.copy_calibration:
        import torch

        src = torch.ones(32 << 20, dtype=torch.float64, device="cuda:0")  # 256 MiB
        dst = torch.empty_like(src)
        for _ in range(3):
            dst.copy_(src)
        torch.cuda.synchronize()
        log("copied 3 x 268435456 bytes")
        return

    if args.gpus != 1:
        print(f"bench.py runs on one GPU only (got --gpus {args.gpus}); the subset sum shards by "
              "pair-subset rank ranges (gbs_lhaf_device_shard computes one GPU's share, "
              "--workload shard times G shares on one GPU), but no multi-GPU launch is provided.",
              file=sys.stderr)
        sys.exit(2)
    rank = int(os.environ.get("RANK", "0"))

    import numpy as np
    import torch

    from paper_2010_15595_amd import _lib

    if not os.path.exists(_lib.LIB_PATH):
        from paper_2010_15595_amd import build as libbuild

        log("building libgbs_lhaf.so ...")
        libbuild.build()
    import paper_2010_15595_amd as gbs

    if args.workload == "batch":
        return bench_batch(args, gbs)
    if args.workload == "sampler":
        return bench_sampler(args, gbs)
    if args.workload == "tvd":
        return fig1_tvd(args, gbs)
    if args.workload == "fig2":
        return fig2_accuracy(args, gbs)
    if args.workload == "methods":
        return methods_comparison(args, gbs)
    if args.workload == "fig3":
        return fig3_sweep(args, gbs)
    if args.workload == "shard":
        return shard_split(args, gbs)

    N = args.N
    st = workload(N)
    A = gbs.expand(st["B"], st["gamma"], st["pattern"])
    assert A.shape == (N, N)
    n = (N + 1) // 2
    terms = float(1 << n)
    flops = gbs.yardstick_flops(N)

    prec = {"fp64": gbs.GBS_FP64, "fp32comp": gbs.GBS_FP32_COMP, "dd": gbs.GBS_DD}[args.precision]
    torch.cuda.set_device(0)
    gbs.init(0)
    dev = torch.device("cuda:0")
    A_dev = torch.from_numpy(A).to(dev)
    out = torch.zeros(1, dtype=torch.complex128, device=dev)
    ab = torch.zeros(1, dtype=torch.float64, device=dev)
    stream = torch.cuda.current_stream(dev)

    tuned = None
    # FP64 sums up to MAX_BATCH_DIM run on the subset tree, which has no lane grid to choose
    if not args.no_autotune and (args.precision == "fp32comp" or (args.precision == "fp64" and N > gbs.MAX_BATCH_DIM)):
        t0 = time.perf_counter()
        rep = gbs.autotune(n)
        tuned = {s: lay for s, (lay, _) in rep.items()}
        log(f"autotune n={n} ({time.perf_counter() - t0:.2f} s): " + " ".join(f"{s}:{lay}" for s, lay in tuned.items()))
    log(f"warmup {args.warmup} step(s), N={N} ({int(terms)} subsets/step) ...")
    for _ in range(args.warmup):
        gbs.lhaf_device(A_dev, out, ab, stream, prec)
    torch.cuda.synchronize()
    ref_val = complex(out.cpu().numpy()[0])

    log(f"timing {args.steps} step(s) ...")
    gbs.profile_enable(True)
    ev0 = torch.cuda.Event(enable_timing=True)
    ev1 = torch.cuda.Event(enable_timing=True)
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    ev0.record(stream)
    for _ in range(args.steps):
        gbs.lhaf_device(A_dev, out, ab, stream, prec)
    ev1.record(stream)
    torch.cuda.synchronize()
    wall = time.perf_counter() - t0
    prof = gbs.profile_read()
    gbs.profile_enable(False)
    gpu_ms = ev0.elapsed_time(ev1)
    val = complex(out.cpu().numpy()[0])
    abs_sum = float(ab.cpu().numpy()[0])
    if args.warmup > 0 and val != ref_val:
        log("WARNING: result changed between steps (non-deterministic)")
    sec = gpu_ms / 1000.0
    lhaf_per_s = args.steps / sec
    # roofline of the dominant kernel instance: its operations per launch over its average launch duration (HIP events on the launch stream)
    achieved = prof["dominant_flops"] / (prof["dominant_ms"] / 1000.0) / 1e12 if prof["dominant_ms"] > 0 else None
    achieved_all = prof["charpoly_flops"] / (prof["charpoly_ms"] / 1000.0) / 1e12 if prof["charpoly_ms"] > 0 else None
    log(f"{args.steps} steps in {gpu_ms:.1f} ms (wall {wall * 1e3:.1f} ms): {lhaf_per_s:.4f} lhaf/s, "
        f"{terms * lhaf_per_s:.4e} subset-terms/s; subset kernels {prof['charpoly_ms']:.1f} ms over "
        f"{prof['charpoly_launches']} launches, series {prof['series_ms']:.1f} ms, reduce {prof['reduce_ms']:.2f} ms")
    log(f"lhaf = {val:.12e}, sum|t_S| = {abs_sum:.4e}, kappa = {abs_sum / abs(val):.3e}")

    result = {
        "metric": "loop hafnians/s and subset-terms/s at N=50 complex128; % FP64 vector peak"
                  if args.precision == "fp64" else f"loop hafnians/s at N={N}, {args.precision} path",
        "value": lhaf_per_s,
        "unit": "lhaf/s",
        "n_gpus": 1,
        "steps": args.steps,
        "warmup": args.warmup,
        "ms_per_step": gpu_ms / args.steps,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": {"fp64": "c128", "fp32comp": "c128 Hessenberg + c64 La Budde/series (compensated)",
                  "dd": "double-double complex (~106-bit significand)"}[args.precision],
        "data": "synthetic",
        "config": {
            "workload": f"loop hafnian N={N} of a 100-mode pure Gaussian state (Haar U, r=1.2, sigma=0.1), "
                        f"{N} distinct modes occupied",
            "N": N,
            "subset_terms_per_lhaf": int(terms),
            **({"lane_grid_per_subset_size": tuned} if tuned else {}),
        },
        "subset_terms_per_s": terms * lhaf_per_s,
        "yardstick_flops_per_lhaf": flops,
        # the yardstick is the paper's formulation; the operations are those of the kernels run
        "operations_per_lhaf": prof["charpoly_flops"] / args.steps,
        "pct_fp64_peak": 100.0 * prof["charpoly_flops"] / args.steps * lhaf_per_s / (FP64_PEAK_TFLOPS * 1e12),
        "roofline": {
            "bound": "alu",
            "kernel": prof["dominant_kernel"],
            "kernel_note": {"dd": "one include child of the subset tree; each dd multiply-add counts as one but takes 12 "
                                  "FP64 instructions per real product",
                            "fp64": "subtree of 5 pairs (32 subsets) per wavefront, series products in registers",
                            "fp32comp": "gather + Householder Hessenberg + La Budde of the subsets of one size "
                                        "class"}[args.precision],
            "achieved": achieved,
            "peak": FP64_PEAK_TFLOPS,
            "unit": "TFLOP/s",
            "frac": (achieved / FP64_PEAK_TFLOPS) if achieved else None,
            "traffic": traffic_entry(prof["dominant_kernel"]) if args.precision == "fp64" else None,
            "traffic_unit": "HBM bytes per launch of the dominant instance (rocprofv3 FETCH_SIZE and WRITE_SIZE, "
                            "scaled by a plain copy)",
            # the path's own HBM input and output per loop hafnian: the N x N complex128
            # matrix in, the complex result and sum |t_S| out (24 B)
            "algorithmic_bytes_per_lhaf": N * N * 16 + 24,
            "flops_per_launch": prof["dominant_flops"] / max(1, prof["dominant_launches"]),
            "avg_launch_ms": prof["dominant_ms"] / max(1, prof["dominant_launches"]),
            "launches_per_step": prof["dominant_launches"] / args.steps,
            "all_per_subset_kernels": {"achieved": achieved_all,
                                       "frac": (achieved_all / FP64_PEAK_TFLOPS) if achieved_all else None,
                                       "launches_per_step": prof["charpoly_launches"] / args.steps,
                                       "kernel_ms_per_step": prof["charpoly_ms"] / args.steps},
        },
        "lhaf": [val.real, val.imag],
        "kappa": abs_sum / abs(val) if val != 0 else None,
        "paper_context": {
            "note": "paper Fig. 3: dim 50 random complex symmetric (Re, Im ~ U[0,1)), long double, "
                    "96 vCPUs Azure D96a v4 @2.345 GHz; different input distribution, same work",
            "seconds_per_lhaf": 2499.40737938881,
            "lhaf_per_s": 1.0 / 2499.40737938881,
        },
    }
    if rank == 0 and not args.no_cpu_baseline:
        log(f"cpu baseline: oracle on a ~{args.cpu_seconds:.0f} s sample ...")
        result["cpu_baseline"] = cpu_baseline(A, N, args.cpu_seconds, args.cpu_one_thread_seconds)
        log(f"cpu baseline: {result['cpu_baseline']['subset_terms_per_s']:.1f} subset-terms/s on "
            f"{result['cpu_baseline']['cores']} threads")
    print(json.dumps(result), flush=True)


if __name__ == "__main__":
    main()
