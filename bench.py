"""Benchmark: tensor-train S_N steps/s on the 256^2 x 2048-ordinate crossing-beam
workload on one MI355X.

A step is one pass of the whole hot path: TT-format upwind transport
operator, absorption/emission, TT sum by concatenation, Gram-SVD rounding
(Gram contractions, eigensolves, truncation, core updates).  The workload is
the crossing-beam case: 256^2 cells, 32 x 64 ordinates, kappa = 1e-3, cold
medium, two inflow beams, tolerance 1e-6, rank cap 64, a 400-step run.  The
steps before the warmup (400 - warmup - steps, when positive) ramp the ranks
up untimed, so the timed steps are the run's last ones, at the rank plateau;
with the default flags the timed steps are 21-400 (the whole run after a
warmup).  Inputs are resident in HBM before timing, and only the roofline
kernel's HIP event pair is live in the timed region; the per-phase breakdown
and roofline fractions come from further, fully profiled steps of the same
context.  Then: the same protocol in the FP32-mixed form ("fp32_mixed"); the
rounding benchmark (a seeded synthetic state whose step concatenates to
(R1, R2) = (322, 62), 100 repeats per precision, "rounding_bench"); the
reverse sweep of the differentiation workload ("gradient"); the optically
thick 3-D workload in both precisions ("thick_3d"); machine peaks measured in
the same process ("measured_peaks"); the CPU oracle on the host's cores.

Prints one JSON line (see the keys below).  --gpus > 1 is not supported:
the hot path runs on one GPU.
"""
import argparse
import json
import os
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

METRIC = "TT steps/s at 256²×2048 angles; FP32-mixed vs FP64 speedup at rel err 1e-6"
FP64_PEAK_TFLOPS = 78.6
GRAM_ROWS_MAX = 384          # widest concatenated rank the row-slice Gram holds in LDS
R1CAP = 5 * 64 + 2 + 1       # crossing beams: B r1_cap + 2 inflow terms + emission slot
GRAM_KERNEL64 = "k_gram_rows<double> (left Gram X_cat^T X_cat, row slices staged in LDS, FP64 MFMA)"
GRAM_KERNEL32 = "k_gram_rows<float> (FP32 entries, FP64 MFMA)"
ROUNDING_PHASES = ("gram_tall", "gram_reduce", "eig_bond1", "eig_M1", "eig_bond2", "eig_M2",
                   "x_update", "small_gemm")
HBM_PEAK_GBS = 8000.0
RUN_STEPS = 400              # the crossing-beam run
BREAKDOWN_STEPS = 20         # fully profiled steps after the timed ones


TRAFFIC_FILE = os.path.join(ROOT, "profiles", "crossing_beams_256sq_fp64_gram_rows_traffic.md")


def gram_rows_digest():
    """Digest of the row-slice Gram kernel's source (its shape constants and
    body), to tell whether stored byte counters still describe it."""
    import hashlib
    s = open(os.path.join(ROOT, "paper_2503_18056_amd", "csrc", "k_gemm.hip")).read()
    a = s.index("// row-slice Gram (k_gram_rows) shape")
    b = s.index("\n", s.index("template <> struct GrShape<0>"))
    k0 = s.index("template <typename T, int S>\n__device__ __forceinline__ void gram_rows_body(")
    k1 = s.index("__global__ __launch_bounds__(256) void k_gram_rows_reduce")
    return hashlib.sha256((s[a:b] + s[k0:k1]).encode()).hexdigest()[:16]


def stored_traffic():
    """(bytes per launch, algorithmic bytes per launch) from the committed
    rocprofv3 FETCH_SIZE / WRITE_SIZE summary, or (None, None) if the kernel
    changed since the counters were taken."""
    try:
        kv = {}
        for line in open(TRAFFIC_FILE):
            if ":" in line and not line.startswith(("#", "|", " ", "`")):
                k, v = line.split(":", 1)
                kv[k.strip()] = v.strip()
        if kv.get("kernel_source_digest") != gram_rows_digest():
            return None, None
        return float(kv["traffic_bytes_per_launch"]), float(kv["algorithmic_bytes_per_launch"])
    except (OSError, KeyError, ValueError):
        return None, None


def gram_flops(ns, R1):
    """Algorithmic flops of the symmetric left Gram of an N_s x R1 core."""
    return float(ns) * R1 * (R1 + 1)


def tt_rel_diff(A, B):
    """||A - B|| / ||B|| of two three-core TTs without forming either tensor
    and without cancelling squared norms: with Q R = X_A (Cholesky QR; X_A
    has full column rank), A - B = Q (R C_A - M C_B) - E C_B where
    M = Q^T X_B and E = X_B - Q M is orthogonal to Q, so the two parts add
    in squares.  C = Theta x Phi is the r1 x (N_theta N_phi) unfolding.
    None when B is the zero tensor."""
    import numpy as np

    def unfold(Th, Ph):
        r1, nt, r2 = Th.shape
        return (Th.reshape(r1 * nt, r2) @ Ph).reshape(r1, -1)

    def gram_norm2(G, C):
        # ||X C||^2 = tr(C^T G C) with G = X^T X, as a sum of nonnegative terms
        w, V = np.linalg.eigh(G)
        return float(np.sum(np.clip(w, 0.0, None)[:, None] * (V.T @ C) ** 2))
    XA, XB = A[0], B[0]
    CA, CB = unfold(A[1], A[2]), unfold(B[1], B[2])
    nb2 = gram_norm2(XB.T @ XB, CB)
    if not nb2 > 0.0:
        return None
    R = np.linalg.cholesky(XA.T @ XA).T
    Q = np.linalg.solve(R.T, XA.T).T
    M = Q.T @ XB
    E = XB - Q @ M
    d2 = float(np.sum((R @ CA - M @ CB) ** 2)) + gram_norm2(E.T @ E, CB)
    return (d2 / nb2) ** 0.5


def progress(msg):
    print(f"[bench] {msg}", file=sys.stderr, flush=True)


def timed_run(p, ramp, W, K, precision, nbreak=BREAKDOWN_STEPS):
    """Steps 1..ramp+W untimed, the next K timed with only the Gram kernel's
    event pair live, then nbreak steps with every profiling class (the
    breakdown); inputs resident in HBM throughout."""
    import torch
    from paper_2503_18056_amd import TTState
    st = TTState(p, device=0, max_steps=ramp + W + K + nbreak, precision=precision)
    if ramp + W:
        st.step(ramp + W)
    torch.cuda.synchronize()
    warm = st.cores()
    r_start = st.ranks()
    st.tt_profile_enable(True, classes=["gram_tall"])
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    st.step(K)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    prof = st.tt_profile_read()
    st.tt_profile_enable(False)
    r_break = st.ranks()
    st.tt_profile_enable(True)
    st.step(nbreak)
    torch.cuda.synchronize()
    breakdown = st.tt_profile_read()
    st.tt_profile_enable(False)
    return st, t1 - t0, prof, warm, r_start, breakdown, r_break


def host_info():
    """CPU model, visible cores and the BLAS NumPy uses (for the oracle rows)."""
    info = {"cores_visible": len(os.sched_getaffinity(0))}
    try:
        for line in open("/proc/cpuinfo"):
            if line.startswith("model name"):
                info["cpu_model"] = line.split(":", 1)[1].strip()
                break
    except OSError:
        pass
    try:
        from threadpoolctl import threadpool_info
        blas = [i for i in threadpool_info() if i.get("user_api") == "blas"]
        if blas:
            info["blas"] = {"library": blas[0].get("internal_api"), "version": blas[0].get("version"),
                            "threads": blas[0].get("num_threads")}
    except Exception:
        pass
    return info


def measured_peaks():
    """HBM copy bandwidth and dense FP64 / FP32 MFMA rates of this GPU,
    measured in this process by the library's microbenchmarks."""
    import ctypes as C
    import torch
    from paper_2503_18056_amd import _ffi
    lib = _ffi.load()
    out = {}
    for which, name, nbytes, iters in ((0, "hbm_copy_GBs", 1 << 30, 10), (1, "fp64_mfma_TFLOPs", 0, 20000),
                                       (2, "fp32_mfma_TFLOPs", 0, 20000)):
        wsb = lib.tt_kernel_microbench_workspace(which, nbytes)
        ws = torch.empty(int(wsb), dtype=torch.uint8, device="cuda")
        r = C.c_double()
        st = lib.tt_kernel_microbench(which, nbytes, iters, C.c_void_p(ws.data_ptr()), int(wsb),
                                      C.byref(r), None)
        out[name] = r.value if st == 0 else None
        del ws
    out["note"] = ("HBM: streaming copy of 1 GiB, read + write bytes; MFMA: v_mfma_f64_16x16x4f64 / "
                   "v_mfma_f32_16x16x4f32 on register operands, 2048 blocks of 4 wavefronts")
    return out


def phase_roofline(prof, ranks, nsteps, ns, nbc, peaks):
    """Per-phase roofline of the crossing-beam step:
    concat HBM-bound (read X, write X_cat), Gram and X update max(MFMA,
    HBM), the rank-sized products and eigensolves latency-bound (their
    measured time is their roofline time).  ``ranks``: (r1, r2) entering
    each profiled step, and the r1' it rounded to."""
    def fp64_time(flops, nbytes, peak_tf, bw_gbs):
        return max(flops / (peak_tf * 1e12), nbytes / (bw_gbs * 1e9))
    out = {}
    for label, peak_tf, bw in (("vendor", FP64_PEAK_TFLOPS, HBM_PEAK_GBS),
                               ("measured", peaks.get("fp64_mfma_TFLOPs"), peaks.get("hbm_copy_GBs"))):
        if not peak_tf or not bw:
            continue
        roof = {"concat": 0.0, "gram_tall": 0.0, "x_update": 0.0}
        for (r1, r2, r1n) in ranks:
            R1 = 5 * r1 + nbc
            roof["concat"] += fp64_time(0.0, ns * (r1 + R1) * 8.0, peak_tf, bw)
            roof["gram_tall"] += fp64_time(ns * R1 * (R1 + 1.0), ns * R1 * 8.0, peak_tf, bw)
            roof["x_update"] += fp64_time(2.0 * ns * R1 * r1n, ns * (R1 + r1n) * 8.0, peak_tf, bw)
        phases = {}
        tot_meas = prof.get("step", (0.0, 0))[0]
        tot_roof = 0.0
        for k, (ms, n) in prof.items():
            if k in ("step", "material_energy") or n == 0:
                continue
            if k in roof:
                r_ms = roof[k] * 1e3
                phases[k] = {"measured_ms_per_step": ms / nsteps, "roofline_ms_per_step": r_ms / nsteps,
                             "frac": r_ms / ms if ms > 0 else None}
                tot_roof += r_ms
            elif k == "gram_reduce":
                phases[k] = {"measured_ms_per_step": ms / nsteps, "roofline_ms_per_step": 0.0,
                             "frac": 0.0, "note": "no algorithmic work (sums the per-block Gram tiles)"}
            else:
                phases[k] = {"measured_ms_per_step": ms / nsteps, "bound": "latency",
                             "roofline_ms_per_step": ms / nsteps, "frac": 1.0}
                tot_roof += ms
        eig_ms = sum(prof.get(k, (0.0, 0))[0] for k in ("eig_bond1", "eig_M1", "eig_bond2", "eig_M2"))
        small_ms = prof.get("small_gemm", (0.0, 0))[0]
        bound_ms = tot_roof - eig_ms - small_ms
        out[label] = {"peaks": {"fp64_TFLOPs": peak_tf, "hbm_GBs": bw}, "phases": phases,
                      "step_frac_latency_phases_as_measured": tot_roof / tot_meas if tot_meas else None,
                      "step_frac_bandwidth_and_mfma_phases": (bound_ms / (tot_meas - eig_ms - small_ms)
                                                              if tot_meas > eig_ms + small_ms else None),
                      "step_measured_ms": tot_meas / nsteps,
                      "latency_bound_ms_per_step": (eig_ms + small_ms) / nsteps}
    return out


def cpu_baseline(p, start_cores, nsteps_target_s=15.0, max_steps=60):
    """The CPU oracle (FP64, NumPy) on a bounded sample of the same workload:
    steps from the GPU run's post-warmup state until ~15 s have elapsed."""
    import numpy as np
    from oracle import Setup, tt
    try:
        from threadpoolctl import threadpool_info
        threads = max([i.get("num_threads", 1) for i in threadpool_info()] or [1])
    except Exception:
        threads = os.cpu_count() or 1
    s = Setup(p)
    X, Th, Ph = start_cores
    T = s.T0.copy()
    t0 = time.perf_counter()
    n = 0
    while n < max_steps and time.perf_counter() - t0 < nsteps_target_s:
        (X, Th, Ph), T, _ = tt.step(X, Th, Ph, T, s, p["tol"], p["rmax"])
        n += 1
    dt = time.perf_counter() - t0
    if not all(np.isfinite(a).all() for a in (X, Th, Ph)):
        return {"value": None, "unit": "steps/s", "cores": int(threads), "kind": "oracle",
                "sample": f"oracle state became non-finite within {n} steps; no rate reported"}
    return {"value": n / dt, "unit": "steps/s", "cores": int(threads), "kind": "oracle",
            "sample": f"{n} consecutive steps of the same workload starting from the GPU "
                      f"state at the start of the timed steps (ranks {X.shape[1]},{Ph.shape[0]}), "
                      f"NumPy FP64, {len(os.sched_getaffinity(0))} host cores visible",
            "host": host_info()}


def cpu_oracle_extra(p, start_cores, budget_s=12.0):
    """More of the CPU oracle beside the GPU (bounded samples, host only):
    the TT oracle on the crossing-beam workload at one BLAS thread; the TT
    oracle's first five steps of the thick 3-D workload at all cores; and the
    full-grid S_N oracle on the 32^2 parity case, in the paper's unit
    (angle-updates/s; the paper's serial-Python S_N rates are 3.1-4.3e7)."""
    import numpy as np
    import workloads as wl
    from oracle import Setup, full, tt
    from threadpoolctl import threadpool_limits
    out = {}
    s = Setup(p)
    X, Th, Ph = start_cores
    T = s.T0.copy()
    with threadpool_limits(limits=1):
        t0 = time.perf_counter()
        n = 0
        while n < 40 and time.perf_counter() - t0 < budget_s:
            (X, Th, Ph), T, _ = tt.step(X, Th, Ph, T, s, p["tol"], p["rmax"])
            n += 1
        dt = time.perf_counter() - t0
    out["tt_crossing_beams_1thread"] = {"steps_per_s": n / dt, "steps": n,
                                        "sample": "consecutive steps from the GPU's post-warmup state"}
    p4 = wl.c4(steps=5)
    s4 = Setup(p4)
    t0 = time.perf_counter()
    tt.run(s4, 5)
    dt = time.perf_counter() - t0
    out["tt_thick3d_first5_allcores"] = {"steps_per_s": 5 / dt, "seconds": dt,
                                         "cores": len(os.sched_getaffinity(0))}
    p1 = wl.c1()
    s1 = Setup(p1)
    I = full.initial_intensity(s1)
    t0 = time.perf_counter()
    full.run(s1, p1["steps"], I=I)
    dt = time.perf_counter() - t0
    nang = p1["ntheta"] * p1["nphi"]
    ns1 = p1["nx"] * p1["ny"]
    out["full_grid_parity_case"] = {"steps_per_s": p1["steps"] / dt,
                                    "angle_updates_per_s": ns1 * nang * p1["steps"] / dt,
                                    "workload": "32x32 cells, 8x16 ordinates, 10 steps"}
    return out


def mixed_run(p, ramp, W, K, dt, hist, end64):
    """The FP32-mixed precision form on the same workload and protocol."""
    from paper_2503_18056_amd import TT_FP32_MIXED
    ns = p["nx"] * p["ny"]
    sm, dtm, profm, _, rm_start, bdm, _ = timed_run(p, ramp, W, K, TT_FP32_MIXED)
    histm = sm.tt_get_rank_history()
    endm = sm.cores()
    gm_ms, gm_n = profm.get("gram_tall", (0.0, 0))
    s0 = ramp + W
    rm_in = [rm_start] + histm[s0:s0 + K - 1]
    flops_m = sum(gram_flops(ns, 5 * r1 + 2) for (r1, _) in rm_in)
    mixed = {
        "steps_per_s": K / dtm,
        "ms_per_step": dtm * 1e3 / K,
        "speedup_vs_fp64": (K / dtm) / (K / dt),
        "rel_diff_vs_fp64_gpu_end": tt_rel_diff(endm, end64),
        "rank_history_equal_steps": sum(a == b for a, b in zip(histm, hist)),
        "ranks_end": list(sm.ranks()),
        "gram_kernel": {
            "kernel": GRAM_KERNEL32 if R1CAP <= GRAM_ROWS_MAX else "k_gram_wide<float>",
            "avg_launch_ms": gm_ms / gm_n if gm_n else None,
            "achieved_algorithmic_TFLOPs": flops_m / (gm_ms * 1e-3) / 1e12 if gm_ms > 0 else 0.0,
            "peak_fp64_mfma_TFLOPs": FP64_PEAK_TFLOPS,
        },
        "kernel_breakdown_ms": {k: {"ms_total": round(v[0], 3), "launches": v[1]}
                                for k, v in bdm.items()},
        "breakdown_steps": BREAKDOWN_STEPS,
    }
    sm.close()
    return mixed


def slice_sweep(p, nsteps, slices=(1, 2, 3, 4, 5, 6), prof_steps=20):
    """Slice count of the FP32-mixed Gram (tt_set_gram_slices) against the
    FP64 library on the same run: for each count, the whole run's steps/s,
    the rank history against FP64's, the end state's difference from FP64's,
    and the average Gram launch over ``prof_steps`` profiled steps after it.
    Counts 4 to 6 run one path, the entries on FP64 MFMA."""
    import torch
    from paper_2503_18056_amd import TT_FP32_MIXED, TT_FP64, TTState
    warm = TTState(p, device=0, max_steps=2, precision=TT_FP32_MIXED)
    for sl in slices:  # module load and first launch of every instance, untimed
        warm.tt_set_gram_slices(sl)
        warm.step(1)
    warm.close()

    def run(prec, sl=None):
        st = TTState(p, device=0, max_steps=nsteps + prof_steps, precision=prec)
        if sl is not None:
            st.tt_set_gram_slices(sl)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        st.step(nsteps)
        torch.cuda.synchronize()
        dt = time.perf_counter() - t0
        hist, end = st.tt_get_rank_history(), st.cores()
        st.tt_profile_enable(True, classes=["gram_tall"])
        st.step(prof_steps)
        torch.cuda.synchronize()
        gms, gn = st.tt_profile_read().get("gram_tall", (0.0, 0))
        st.close()
        return dt, hist, end, (gms / gn if gn else None)

    dt64, h64, e64, g64 = run(TT_FP64)
    out = {"workload": f"{p['name']}: the first {nsteps} steps (rank ramp included), then "
                       f"{prof_steps} steps with the Gram timed",
           "fp64": {"steps_per_s": nsteps / dt64, "gram_avg_launch_ms": g64,
                    "ranks_end": list(h64[-1]) if h64 else None},
           "slices": {}}
    for sl in slices:
        progress(f"Gram slice sweep: {sl} slices")
        dt, h, e, g = run(TT_FP32_MIXED, sl)
        out["slices"][str(sl)] = {
            "slice_products": sl * (sl + 1) // 2 if sl < 4 else None,  # None: FP64 products
            "steps_per_s": nsteps / dt,
            "gram_avg_launch_ms": g,
            "rank_history_equal_steps": sum(a == b for a, b in zip(h, h64)),
            "ranks_end": list(h[-1]) if h else None,
            "rel_diff_vs_fp64_end": tt_rel_diff(e, e64),
        }
    return out


def rounding_bench(p, reps=100):
    """Rounding throughput at the crossing-beam cap shape: a seeded
    synthetic state (orthonormal X and Phi rows, bond-1 spectrum 10^(-k/8),
    ranks (64, 12)) is installed and stepped once, which concatenates it to
    (R1, R2) = (322, 62) and rounds that; repeated ``reps`` times per
    precision with every profiling class on.  Reports the rounding phases
    per rounding and the whole step."""
    import torch
    import workloads as wl
    from paper_2503_18056_amd import TT_FP32_MIXED, TT_FP64, TTState
    X, Th, Ph = wl.rounding_bench_cores(p)
    ns = p["nx"] * p["ny"]
    out = {"workload": "seeded state on the crossing-beam shape (256^2, 32x64): orthonormal X "
                       "65536x64, Theta 64x32x12, Phi 12x64, bond-1 singular values 10^(-k/8); "
                       f"one step concatenates it to (R1, R2) = (322, 62); {reps} repeats"}
    for name, prec in (("fp64", TT_FP64), ("fp32_mixed", TT_FP32_MIXED)):
        st = TTState(p, device=0, max_steps=2, precision=prec, cores=(X, Th, Ph))
        st.step(1)  # first call: module load, not timed
        st.tt_profile_enable(True)
        for _ in range(reps):
            st.tt_set_cores(X, Th, Ph)
            st.step(1)
        torch.cuda.synchronize()
        prof = st.tt_profile_read()
        st.tt_profile_enable(False)
        info = st.tt_get_round_info()
        round_ms = sum(prof.get(k, (0.0, 0))[0] for k in ROUNDING_PHASES) / reps
        step_ms = prof.get("step", (0.0, 0))[0] / reps
        R1, r1n = int(info["R1"]), int(info["r1"])
        # Gram-SVD multiply-adds of the two N_s-long contractions (left Gram, X update)
        flops = gram_flops(ns, R1) + 2.0 * ns * R1 * r1n
        out[name] = {"ms_per_rounding": round_ms, "roundings_per_s": 1e3 / round_ms if round_ms else None,
                     "ms_per_step": step_ms, "R1": R1, "ranks_after": list(st.ranks()),
                     "ns_long_flops_per_rounding": flops,
                     "ns_long_TFLOPs": flops / (round_ms * 1e-3) / 1e12 if round_ms else None,
                     "phases_ms_per_rounding": {k: prof[k][0] / reps for k in ROUNDING_PHASES if k in prof}}
        st.close()
    return out


def randomized_rounding_bench(p, reps=10):
    """Gram-SVD rounding (tt_round, tolerance 1e-6, cap 64) against randomized
    rounding to fixed target ranks (tt_round_randomized, App. A.3) of one
    seeded state on the crossing-beam shape (256^2, 32x64): orthonormal X
    65536x192 and Phi rows 48x64, bond-1 singular values 10^(-k/8).  Each
    rounding starts from the same state (re-installed, untimed); host-timed
    median of ``reps`` calls, each ending in a synchronisation."""
    import time
    import numpy as np
    import torch
    import workloads as wl
    from paper_2503_18056_amd import TTState
    X, Th, Ph = wl.rounding_bench_cores(p, r1=192, r2=48)
    st = TTState(p, device=0, cores=(X, Th, Ph), r1_cap=192, r2_cap=48, max_steps=2)

    def timed(fn):
        ts, r = [], None
        for i in range(reps + 1):
            st.tt_set_cores(X, Th, Ph)
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            r = fn()
            torch.cuda.synchronize()
            if i:
                ts.append(time.perf_counter() - t0)
        return r, 1e3 * float(np.median(ts))

    out = {"workload": "seeded state on the crossing-beam shape (256^2, 32x64), ranks (192, 48), "
                       f"bond-1 singular values 10^(-k/8); median of {reps}"}
    r, ms = timed(lambda: st.tt_round(1e-6, 64))
    out["gram_svd"] = {"ms": ms, "ranks": list(r)}
    out["randomized"] = []
    for k1, k2 in ((64, 12), (72, 16), (64, 48), (128, 32)):
        om = wl.gaussian_test_matrices(p["ntheta"], p["nphi"], k1, k2, seed=3)
        r, ms = timed(lambda: st.tt_round_randomized(*om))
        out["randomized"].append({"target": [k1, k2], "ms": ms, "ranks": list(r)})
    st.close()
    return out


def thick_3d_run(W, K):
    """The optically thick 3-D workload (128^3 cells, 32 x 64 ordinates,
    kappa = 1e3 in the central 64^3 cube, coupled material, rank cap 128) in
    FP64 and in the FP32-mixed form: W untimed steps in which the ranks ramp
    to the cap, then K timed steps."""
    import workloads as wl
    from paper_2503_18056_amd import TT_FP32_MIXED, TT_FP64
    p = wl.c4(steps=W + K + 2)
    ns = p["nx"] * p["ny"] * p["nz"]
    blocks = 1 + 2 * p["dim"]
    out = {"workload": f"{p['name']}: 128^3 cells, 32x64 ordinates, kappa 1e3 in the central "
                       f"64^3 cube and 1 outside, coupled material, tol 1e-6, rank cap 128, "
                       f"steps {W + 1}-{W + K} of {W + K}"}
    ends = {}
    for name, prec in (("fp64", TT_FP64), ("fp32_mixed", TT_FP32_MIXED)):
        progress(f"thick 3-D, {name}: {W} warmup + {K} timed steps")
        st, dt, prof, _, r_start, bd, _ = timed_run(p, 0, W, K, prec, nbreak=2)
        hist = st.tt_get_rank_history()
        r_in = [r_start] + hist[W:W + K - 1]
        # concatenated rank at bond 1: (1 + 2 dim) r1 plus the emission slot
        flops = sum(gram_flops(ns, blocks * r1 + 1) for (r1, _) in r_in)
        gms, gn = prof.get("gram_tall", (0.0, 0))
        peak = FP64_PEAK_TFLOPS  # both precisions form the products on FP64 MFMA
        achieved = flops / (gms * 1e-3) / 1e12 if gms > 0 else 0.0
        round_ms = sum(bd.get(k, (0.0, 0))[0] for k in ROUNDING_PHASES) * K / 2.0
        out[name] = {
            "steps_per_s": K / dt,
            "ms_per_step": dt * 1e3 / K,
            "ranks_entering_timed_steps": [list(r) for r in r_in],
            "ranks_end": list(st.ranks()),
            "ms_per_rounding": round_ms / K,
            "gram": {"kernel": ("k_gram_wide (FP64 MFMA, 128x128 tile pairs, rows staged through LDS)"
                                if prec == TT_FP64 else
                                "k_gram_wide<float> (FP32 entries, FP64 MFMA, 128x128 tile pairs)"),
                     "avg_launch_ms": gms / gn if gn else None,
                     "achieved_algorithmic_TFLOPs": achieved,
                     "peak_TFLOPs": peak, "frac": achieved / peak},
            "kernel_breakdown_ms_2_steps": {k: {"ms_total": round(v[0], 3), "launches": v[1]}
                                            for k, v in bd.items()},
        }
        ends[name] = st.cores()
        st.close()
        progress(f"thick 3-D, {name}: {K / dt:.2f} steps/s, ranks {out[name]['ranks_end']}")
    out["speedup_mixed_vs_fp64"] = out["fp32_mixed"]["steps_per_s"] / out["fp64"]["steps_per_s"]
    out["rel_diff_mixed_vs_fp64_end"] = tt_rel_diff(ends["fp32_mixed"], ends["fp64"])
    return out


def gradient_run():
    """Taped forward and reverse sweep of the differentiation workload."""
    import numpy as np
    import torch
    import workloads as wl
    from paper_2503_18056_amd import TTState
    p = wl.c5()
    nsteps, K = p["steps"], p["ckpt_every"]
    st = TTState(p, device=0, max_steps=nsteps, ckpt_every=K)
    st.step(1)  # first call: module load and code upload, not timed
    st.tt_set_cores(p["X0"], p["Th0"], p["Ph0"])
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    st.step(nsteps)
    torch.cuda.synchronize()
    t1 = time.perf_counter()
    L, g = st.tt_grad(p["detector"])
    torch.cuda.synchronize()
    t2 = time.perf_counter()
    g = g.cpu().numpy()
    out = {
        "workload": f"{p['name']}: 128x128 cells, 16x32 ordinates, kappa = exp(GRF), pulse, "
                    f"tol 1e-6, rank cap 128, {nsteps} steps, checkpoint every {K}",
        "loss": L,
        "grad_finite": bool(np.isfinite(g).all()),
        "grad_max_abs": float(np.max(np.abs(g))),
        "ranks_end": list(st.ranks()),
        "forward_taped_s": t1 - t0,
        "grad_s": t2 - t1,
        "grad_over_forward": (t2 - t1) / (t1 - t0),
    }
    st.close()
    return out


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=380)
    ap.add_argument("--warmup", type=int, default=20)
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--no-mixed", action="store_true", help="skip the FP32-mixed run")
    ap.add_argument("--no-grad", action="store_true", help="skip the reverse-sweep run")
    ap.add_argument("--no-rounding-bench", action="store_true")
    ap.add_argument("--no-peaks", action="store_true", help="skip the peak microbenchmarks")
    ap.add_argument("--thick3d-steps", type=int, default=6,
                    help="timed steps of the thick 3-D workload in each precision (0 skips it)")
    ap.add_argument("--thick3d-warmup", type=int, default=6)
    ap.add_argument("--no-slice-sweep", action="store_true",
                    help="skip the FP32-mixed Gram slice-count sweep on the crossing beams")
    ap.add_argument("--slice-sweep-thick3d", type=int, default=0,
                    help="also sweep the slice count on the thick 3-D workload for this many steps")
    ap.add_argument("--calib-copy-mib", type=int, default=0,
                    help="run one plain device-to-device copy of this many MiB before the "
                         "warmup (a known-size kernel to scale hardware byte counters by)")
    ap.add_argument("--randomized-only", action="store_true",
                    help="only compare Gram-SVD and randomized rounding on one state (prints that JSON)")
    args = ap.parse_args()
    if args.gpus != 1:
        print(f"bench.py: --gpus {args.gpus} is not supported; the hot path runs on one GPU "
              "(sharding by spatial rows of X is designed, not built)", file=sys.stderr)
        sys.exit(2)
    import workloads as wl
    from paper_2503_18056_amd import TT_FP64

    if args.randomized_only:
        print(json.dumps({"randomized_rounding_bench": randomized_rounding_bench(wl.c2(steps=2))}))
        return
    W, K = args.warmup, args.steps
    ramp = max(0, RUN_STEPS - W - K)
    if args.calib_copy_mib > 0:
        import torch
        n = args.calib_copy_mib * (1 << 20) // 8
        src = torch.ones(n, dtype=torch.float64, device="cuda")
        dst = torch.empty_like(src)
        dst.copy_(src)
        torch.cuda.synchronize()
        del src, dst
    p = wl.c2(steps=ramp + W + K)
    progress(f"crossing beams, FP64: {ramp} ramp + {W} warmup + {K} timed steps")
    st, dt, prof, warm_cores, r_start, bd, r_break = timed_run(p, ramp, W, K, TT_FP64)
    progress(f"FP64 done: {K / dt:.1f} steps/s")
    hist = st.tt_get_rank_history()
    ns = p["nx"] * p["ny"]
    nang = p["ntheta"] * p["nphi"]
    nbc = len(p["inflow"])
    s0 = ramp + W
    # concatenated rank R1 entering each timed step: 5 r1 + 2 inflow terms
    r_in = [r_start] + hist[s0:s0 + K - 1]
    R1s = [5 * r1 + nbc for (r1, _) in r_in]
    gram_ms, gram_n = prof.get("gram_tall", (0.0, 0))
    flops = sum(gram_flops(ns, R) for R in R1s)
    achieved = flops / (gram_ms * 1e-3) / 1e12 if gram_ms > 0 else 0.0
    breakdown = {k: {"ms_total": round(v[0], 3), "launches": v[1]} for k, v in bd.items()}
    # ranks entering each breakdown step and the r1' each rounded to
    hb = [r_break] + hist[s0 + K:s0 + K + BREAKDOWN_STEPS]
    ranks_b = [(hb[i][0], hb[i][1], hb[i + 1][0]) for i in range(len(hb) - 1)]
    round_ms = sum(bd.get(k, (0.0, 0))[0] for k in ROUNDING_PHASES)
    traffic, alg_bytes = stored_traffic()
    end64 = st.cores()
    ranks64 = list(st.ranks())
    st.close()
    progress(f"FP64 end state: ranks {ranks64}, max |X| {abs(end64[0]).max():.3e}, "
             f"max |Phi| {abs(end64[2]).max():.3e}")
    peaks = {} if args.no_peaks else measured_peaks()
    if peaks:
        progress(f"measured peaks: {peaks}")
    if not args.no_mixed:
        progress("crossing beams, FP32-mixed")
    mixed = None if args.no_mixed else mixed_run(p, ramp, W, K, dt, hist, end64)
    out = {
        "metric": METRIC,
        "value": K / dt,
        "unit": "steps/s",
        "n_gpus": 1,
        "steps": K,
        "warmup": W,
        "ms_per_step": dt * 1e3 / K,
        "higher_is_better": True,
        "scaling": "weak",
        "vs_baseline": None,
        "dtype": "f64",
        "data": "synthetic",
        "config": {"workload": "crossing beams 256x256 cells, 32x64 ordinates, kappa 1e-3, "
                               "cold medium, 2 inflow beams, tol 1e-6, rank cap 64, timed steps "
                               f"{s0 + 1}-{s0 + K} of a {s0 + K}-step run",
                   "precision": "fp64", "nx": 256, "ny": 256, "ntheta": 32, "nphi": 64,
                   "tol": 1e-6, "rmax": 64},
        "ranks_timed_start": list(r_start),
        "ranks_end": ranks64,
        "zcps": ns * K / dt,
        "angle_updates_per_s": ns * nang * K / dt,
        "rounding": {
            "ms_per_rounding": round_ms / BREAKDOWN_STEPS,
            "roundings_per_s": BREAKDOWN_STEPS / (round_ms * 1e-3) if round_ms > 0 else None,
            "note": "Gram-SVD rounding phases (Grams, eigensolves, SVDs, truncation and core "
                    f"updates) of {BREAKDOWN_STEPS} fully profiled steps after the timed ones",
        },
        "roofline": {
            "kernel": GRAM_KERNEL64 if R1CAP <= GRAM_ROWS_MAX else "k_gram_wide + k_gram_wide_reduce",
            "bound": "mfma",
            "achieved": achieved,
            "peak": FP64_PEAK_TFLOPS,
            "unit": "TFLOP/s",
            "frac": achieved / FP64_PEAK_TFLOPS,
            "frac_of_measured_peak": (achieved / peaks["fp64_mfma_TFLOPs"]
                                      if peaks.get("fp64_mfma_TFLOPs") else None),
            "traffic": traffic,
            "traffic_unit": "bytes per launch (rocprofv3 FETCH_SIZE + WRITE_SIZE, copy-calibrated; "
                            "profiles/crossing_beams_256sq_fp64_gram_rows_traffic.md)",
            "algorithmic_bytes_per_launch": alg_bytes,
            "avg_launch_ms": gram_ms / gram_n if gram_n else None,
            "algorithmic_flops_per_launch_avg": flops / max(1, gram_n),
            "timing": "HIP events on the library's stream around each launch in the timed steps "
                      "(the only events live there)",
        },
        "phase_roofline": phase_roofline(bd, ranks_b, BREAKDOWN_STEPS, ns, nbc, peaks),
        "kernel_breakdown_ms": breakdown,
        "breakdown_steps": f"{BREAKDOWN_STEPS} fully profiled steps after the timed ones",
        "measured_peaks": peaks or None,
        "fp32_mixed": mixed,
    }
    if not args.no_slice_sweep:
        out["gram_slice_sweep"] = slice_sweep(wl.c2(steps=RUN_STEPS + 20), RUN_STEPS)
    if args.slice_sweep_thick3d > 0:
        out["gram_slice_sweep_thick3d"] = slice_sweep(wl.c4(steps=args.slice_sweep_thick3d + 2),
                                                      args.slice_sweep_thick3d, prof_steps=2)
    if not args.no_rounding_bench:
        progress("rounding benchmark at (R1, R2) = (322, 62)")
        out["rounding_bench"] = rounding_bench(wl.c2(steps=2))
    if not args.no_rounding_bench:
        progress("Gram-SVD against randomized rounding at ranks (192, 48)")
        out["randomized_rounding_bench"] = randomized_rounding_bench(wl.c2(steps=2))
    if not args.no_grad:
        progress("differentiation workload: taped forward and reverse sweep")
        out["gradient"] = gradient_run()
    if args.thick3d_steps > 0:
        out["thick_3d"] = thick_3d_run(args.thick3d_warmup, args.thick3d_steps)
    if not args.no_cpu_baseline:
        progress("CPU oracle baseline (about 15 s)")
        out["cpu_baseline"] = cpu_baseline(p, warm_cores)
        progress("more of the CPU oracle (one thread; thick 3-D first steps; full grid)")
        out["cpu_oracle_extra"] = cpu_oracle_extra(p, warm_cores)
    print(json.dumps(out), flush=True)


if __name__ == "__main__":
    main()
