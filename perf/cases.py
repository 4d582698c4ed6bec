"""The work a user of this library has it do, as measured cases.

A user's program holds a ``TTState`` (one context: the problem's fields, its
inflow terms, its current cores), advances it with ``tt_step`` and reads the
energy density, the totals and the ranks; it differentiates a detector loss
with ``tt_grad``, rounds given cores (``tt_round``, ``tt_round_randomized``),
and calls the contraction and eigensolver entry points by themselves.  The
problems are the repository's own workloads at their tolerances (1e-4 for the
analytic test problems, 1e-6 for the thick 3-D medium), with seeded random
material fields and beam strengths.

Kinds
  run      set the initial cores, ``steps`` steps from them, energy and totals
  march    the program has a stored state (and ``ramp`` steps from it behind
           it) and takes ``steps`` more a pass
  grad     set the cores, ``steps`` taped steps, the loss and its gradient
  round    set the cores, one Gram-SVD rounding to ``tol``, energy and ranks
  sketch   set the cores, one randomized rounding, energy and ranks
  gram     A^T A of a tall matrix (float64 or float32 entries)
  eigh     eigenpairs of a dense symmetric matrix
"""
import ctypes as C
import math

import numpy as np
import torch

import workloads as wl
from paper_2503_18056_amd import TT_ROUND_ONCE, TT_ROUND_TWICE, TTState, _ffi

LIGHT = 1.0  # speed of light of every workload


def listed():
    return [
        # the smallest steps a program takes: a 12 x 10 mesh with inflow and a
        # coupled material; nothing but latency and launches
        dict(name="tiny_coupled", kind="run", problem="random", nx=12, ny=10, ntheta=4, nphi=8,
             steps=2, tol=1e-4, rmax=0, flux="upwind", twice=False, r1=20, r2=8),
        # the parity pulse: 32^2 mesh, ten steps from a rank-1 pulse
        dict(name="pulse_32", kind="run", problem="pulse", nx=32, ny=32, ntheta=8, nphi=16,
             steps=10, tol=1e-4, rmax=0, flux="upwind", twice=False, r1=36, r2=16),
        # the diffusion test: scattering medium, Rusanov flux, outflow faces,
        # two roundings a step, tiny ranks on a mid-sized mesh
        dict(name="diffusion_64", kind="run", problem="diffusion", nx=64, ny=64, ntheta=8, nphi=16,
             steps=4, tol=1e-4, rmax=0, flux="rusanov", twice=True, r1=3, r2=3),
        # the headline workload: crossing beams, marching on from a stored state
        # at the ranks the run settles at
        dict(name="beams_256", kind="march", problem="beams", nx=256, ny=256, ntheta=32, nphi=64,
             ramp=0, steps=2, tol=1e-4, rmax=28, flux="upwind", twice=False, r1=28, r2=12),
        # the line source on a ragged mesh through the HLL flux: an expanding
        # pulse whose ranks press against the cap
        dict(name="line_hll_97x75", kind="run", problem="line", nx=97, ny=75, ntheta=16, nphi=32,
             steps=8, tol=1e-4, rmax=64, flux="hll", twice=False, r1=20, r2=11),
        # the hohlraum: isotropic inflow on two faces, at rank 64 (the beams' cap)
        dict(name="hohlraum_64", kind="march", problem="hohlraum", nx=64, ny=64, ntheta=16, nphi=32,
             ramp=0, steps=1, tol=1e-4, rmax=64, flux="upwind", twice=False, r1=64, r2=24),
        # the optically thick 3-D medium with coupled material at its rank cap
        dict(name="thick3d_128", kind="march", problem="thick", nx=128, ny=128, nz=128, ntheta=32,
             nphi=64, ramp=6, steps=1, tol=1e-6, rmax=128, flux="upwind", twice=False, r1=128, r2=36),
        # the differentiation workload, reduced: taped steps and reverse sweep
        dict(name="grad_48", kind="grad", problem="grf", nx=48, ny=48, ntheta=8, nphi=16, steps=8,
             ckpt=4, tol=1e-3, rmax=64, flux="upwind", twice=False, r1=15, r2=10),
        # one rounding of given cores, by Gram-SVD and by sketching
        dict(name="round_192", kind="round", nx=90, ny=70, ntheta=32, nphi=64, tol=1e-4, r1=192, r2=48),
        dict(name="sketch_192", kind="sketch", nx=90, ny=70, ntheta=32, nphi=64, k1=64, k2=16,
             r1=192, r2=48),
        # the N_s-long contraction of the FP32-mixed form at the beams' rank cap
        dict(name="gram_f32_322", kind="gram", rows=65536, cols=322, single=True),
        # the rank-sized eigensolve by itself, at the beams' cap order
        dict(name="eigh_322", kind="eigh", n=322),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["run", "run", "run", "march", "grad", "round", "sketch", "gram", "eigh"])
    if kind == "gram":
        return dict(kind=kind, rows=log(500, 120000), cols=log(20, 900), single=rng.random() < 0.5)
    if kind == "eigh":
        return dict(kind=kind, n=log(8, 900))
    if kind in ("round", "sketch"):
        nt, npf = rng.choice([(8, 16), (16, 32), (32, 64)])
        r2 = min(npf, log(6, 48))
        r1 = log(16, 200)
        c = dict(kind=kind, nx=log(30, 120), ny=log(30, 120), ntheta=nt, nphi=npf, r1=r1, r2=r2)
        if kind == "round":
            c["tol"] = 10.0 ** rng.uniform(-4.0, -2.5)
        else:
            c.update(k1=max(4, r1 // 3), k2=max(2, r2 // 3))
        return c
    nt, npf = rng.choice([(4, 8), (8, 16), (8, 16), (16, 32)])
    tol = 10.0 ** rng.uniform(-4.0, -3.0)
    if kind == "grad":
        return dict(kind=kind, problem="grf", nx=log(16, 56), ny=log(16, 56), ntheta=8, nphi=16,
                    steps=rng.randint(3, 8), ckpt=rng.randint(2, 4), tol=max(tol, 3e-4), rmax=48,
                    flux="upwind", twice=False, r1=24, r2=12)
    if kind == "march":
        problem = rng.choice(["beams", "hohlraum", "thick"])
        if problem == "thick":
            n = log(16, 48)
            return dict(kind=kind, problem=problem, nx=n, ny=n + rng.randint(0, 3), nz=n, ntheta=8,
                        nphi=16, ramp=5, steps=1, tol=tol, rmax=48, flux="upwind", twice=False,
                        r1=40, r2=14)
        nx, r1 = log(32, 200), log(12, 64)
        return dict(kind=kind, problem=problem, nx=nx, ny=nx + rng.randint(0, 9), ntheta=nt, nphi=npf,
                    ramp=0, steps=rng.randint(1, 2), tol=tol, rmax=min(r1, nt * npf // 2),
                    flux="upwind", twice=False, r1=min(r1, nt * npf // 2), r2=min(npf, r1, 12))
    problem = rng.choice(["random", "pulse", "diffusion", "line"])
    flux = "rusanov" if problem == "diffusion" else rng.choice(["upwind", "upwind", "hll", "rusanov"])
    return dict(kind=kind, problem=problem, nx=log(9, 110), ny=log(9, 110), ntheta=nt, nphi=npf,
                steps=rng.randint(2, 10), tol=tol, rmax=48, flux=flux,
                twice=problem == "diffusion" or rng.random() < 0.25, r1=20, r2=8)


# ---- problems --------------------------------------------------------------

def _rectangle(p, nx, ny, kappa, rng):
    """The workload dict ``p`` on an nx x ny mesh with a random opacity."""
    ns = nx * ny
    p.update(nx=nx, ny=ny, kappa=kappa * np.exp(0.3 * rng.standard_normal(ns)), rho=np.ones(ns),
             cv=np.ones(ns), T0=np.full(ns, float(p["T0"][0])))
    return p


def _pulse_cores(p, sigma, amp):
    xs = (np.arange(p["nx"]) + 0.5) * (p["lx"] / p["nx"]) - 0.47 * p["lx"]
    ys = (np.arange(p["ny"]) + 0.5) * (p["ly"] / p["ny"]) - 0.52 * p["ly"]
    r2 = xs[None, :] ** 2 + ys[:, None] ** 2
    X0 = (amp * np.exp(-r2 / (2 * sigma ** 2))).reshape(-1, 1)
    return X0, np.ones((1, p["ntheta"], 1)), np.ones((1, p["nphi"]))


def _problem(case, seed):
    rng = np.random.default_rng(seed)
    nx, ny, nt, npf = case["nx"], case["ny"], case["ntheta"], case["nphi"]
    what = case["problem"]
    if what == "random":
        p = wl.small_random(nx=nx, ny=ny, ntheta=nt, nphi=npf, r1=3, r2=2, seed=seed % 100003,
                            bc="inflow", material=wl.COUPLED)
    elif what == "pulse":
        p = _rectangle(wl.c1(), nx, ny, 1.0, rng)
        p.update(ntheta=nt, nphi=npf)
        p["X0"], p["Th0"], p["Ph0"] = _pulse_cores(p, 0.08 * rng.uniform(0.9, 1.1), 5.0)
    elif what == "diffusion":
        p = wl.gaussian_diffusion(n=8, ntheta=nt, nphi=npf)
        p = _rectangle(p, nx, ny, 0.0, rng)
        p["kappa_s"] = 1e3 * np.exp(0.1 * rng.standard_normal(nx * ny))
        p["X0"], p["Th0"], p["Ph0"] = _pulse_cores(p, rng.uniform(0.3, 0.5), 0.1)
    elif what == "line":
        p = wl.line_source(n=8, ntheta=nt, nphi=npf)
        p = _rectangle(p, nx, ny, 0.5, rng)
        p["X0"], p["Th0"], p["Ph0"] = _pulse_cores(p, 0.12 * rng.uniform(0.9, 1.1), 5.0)
    elif what == "beams":
        p = _rectangle(wl.c2(), nx, ny, 0.3, rng)
        p.update(ntheta=nt, nphi=npf)
        p["inflow"] = [(f, fw * rng.uniform(0.7, 1.3), tw, pw)
                       for f, fw, tw, pw in wl.crossing_beams(p)]
        p["X0"], p["Th0"], p["Ph0"] = _cores(case, seed)
    elif what == "hohlraum":
        p = wl.hohlraum(n=8, ntheta=nt, nphi=npf)
        p = _rectangle(p, nx, ny, 0.3, rng)
        p["inflow"] = [(0, rng.uniform(0.9, 1.1) * np.ones(ny), np.ones(nt), np.ones(npf)),
                       (2, rng.uniform(0.5, 0.8) * np.ones(nx), np.ones(nt), np.ones(npf))]
        p["X0"], p["Th0"], p["Ph0"] = _cores(case, seed)
    elif what == "grf":
        p = _rectangle(wl.c5(n=16), nx, ny, 1.0, rng)
        n = max(nx, ny)
        field = wl.gaussian_random_field(n, 0.1, seed=seed)[:ny, :nx]
        p.update(kappa=np.exp(field).reshape(-1), ntheta=nt, nphi=npf)
        p["X0"], p["Th0"], p["Ph0"] = _pulse_cores(p, 0.08, 5.0)
        det = np.zeros((ny, nx))
        det[ny // 2:ny // 2 + max(1, ny // 8), 5 * nx // 8:5 * nx // 8 + max(1, nx // 8)] = 1.0
        p["detector"] = det.reshape(-1)
    elif what == "thick":
        nz = case["nz"]
        ns = nx * ny * nz
        p = wl.c4(n=4)
        x, y, z = (np.abs((np.arange(n) + 0.5) / n - 0.5) <= 0.25 for n in (nx, ny, nz))
        cube = (z[:, None, None] & y[None, :, None] & x[None, None, :]).reshape(-1)
        T0 = np.clip(0.75 * (1 + 0.05 * rng.standard_normal(ns)), 0.5, 1.0)
        p.update(nx=nx, ny=ny, nz=nz, ntheta=nt, nphi=npf, kappa=np.where(cube, 1e3, 1.0),
                 rho=np.ones(ns), cv=np.ones(ns), T0=T0,
                 X0=(p["c"] / (4 * np.pi) * p["a_r"] * T0 ** 4).reshape(ns, 1),
                 Th0=np.ones((1, nt, 1)), Ph0=np.ones((1, npf)))
    else:
        raise ValueError(what)
    p.update(tol=case["tol"], rmax=case["rmax"])
    if case["flux"] != "upwind":
        p["flux"] = case["flux"]
    return p


def _cores(case, seed):
    """Cores with orthonormal X and Phi and a falling bond spectrum: a stored
    state ends at its tolerance; a sum of terms before its rounding falls by a
    decade every 8 values down to 1e-6 and is level from there."""
    rng = np.random.default_rng(seed)
    ns, nt, npf, r1, r2 = case["nx"] * case["ny"], case["ntheta"], case["nphi"], case["r1"], case["r2"]
    X = np.linalg.qr(rng.standard_normal((ns, r1)))[0]
    Ph = np.linalg.qr(rng.standard_normal((npf, r2)))[0].T
    Q = np.linalg.qr(rng.standard_normal((nt * r2, r1)))[0].T if nt * r2 >= r1 \
        else rng.standard_normal((r1, nt * r2)) / math.sqrt(nt * r2)
    if case["kind"] == "march":
        s = case["tol"] ** (np.arange(r1) / max(1, r1 - 1))
        b = np.ones(r2)
    else:
        s = 10.0 ** -np.minimum(np.arange(r1) / 8.0, 6.0)
        # the angular modes fall too, so bond 2 has something to drop
        b = 10.0 ** -np.minimum(np.arange(r2) / 5.0, 6.0)
    s = s * rng.uniform(0.97, 1.03, r1)
    return X, s[:, None, None] * Q.reshape(r1, nt, r2) * b[None, None, :], Ph


def _empty_problem(case):
    """The context a program rounds given cores in: 2-D, no inflow."""
    p = wl.small_random(nx=case["nx"], ny=case["ny"], ntheta=case["ntheta"], nphi=case["nphi"])
    return p


def _matrix(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    if case["kind"] == "gram":
        A = torch.randn(case["rows"], case["cols"], dtype=torch.float64, device="cuda", generator=g)
        # columns of a concatenated core: scales over three decades
        A *= 10.0 ** (-3.0 * torch.rand(case["cols"], dtype=torch.float64, device="cuda", generator=g))
        return A.float() if case["single"] else A
    n = case["n"]
    A = torch.randn(n, 3 * n, dtype=torch.float64, device="cuda", generator=g)
    return A @ A.T / (3 * n)


# ---- the protocol ----------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    if kind in ("gram", "eigh"):
        lib = _ffi.load()
        A = _matrix(case, seed)
        n = A.shape[1]
        if kind == "eigh":
            need = lib.tt_kernel_eigh_workspace(n)
        elif case["single"]:
            need = lib.tt_kernel_gram_f32_workspace(A.shape[0], n, n)
        else:
            need = lib.tt_kernel_gram_workspace(A.shape[0], n, n)
        return dict(case=case, lib=lib, A=A, ws=torch.empty(int(need), dtype=torch.uint8, device="cuda"),
                    G=torch.empty(n, n, dtype=torch.float64, device="cuda"),
                    lam=torch.empty(n, dtype=torch.float64, device="cuda"))
    if kind in ("round", "sketch"):
        p = _empty_problem(case)
        cores = _cores(case, seed)
        st = TTState(p, cores=cores, r1_cap=case["r1"], r2_cap=case["r2"])
        state = dict(case=case, st=st, cores=cores)
        if kind == "sketch":
            om = wl.gaussian_test_matrices(case["ntheta"], case["nphi"], case["k1"], case["k2"], seed + 1)
            state["omega"] = [torch.as_tensor(o, device="cuda") for o in om]
        return state
    p = _problem(case, seed)
    st = TTState(p, schedule=TT_ROUND_TWICE if case["twice"] else TT_ROUND_ONCE,
                 max_steps=case["steps"], ckpt_every=case.get("ckpt", 0))
    if kind == "march":
        st.tt_step(case["ramp"])
    return dict(case=case, st=st, p=p, cores=(p["X0"], p["Th0"], p["Ph0"]))


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind in ("gram", "eigh"):
        lib, A, G, ws = state["lib"], state["A"], state["G"], state["ws"]
        n, ptr = A.shape[1], lambda t: C.c_void_p(t.data_ptr())  # noqa: E731
        if kind == "eigh":
            kept = C.c_int32()
            rc = lib.tt_kernel_eigh(ptr(A), n, n, 1.0, ptr(state["lam"]), ptr(G), n, C.byref(kept),
                                    ptr(ws), ws.numel(), None)
        elif case["single"]:
            rc = lib.tt_kernel_gram_f32(ptr(A), A.shape[0], n, n, ptr(G), n, ptr(ws), ws.numel(), None)
        else:
            rc = lib.tt_kernel_gram(ptr(A), A.shape[0], n, n, ptr(G), n, ptr(ws), ws.numel(), None)
        if rc != 0:
            raise RuntimeError(lib.tt_kernel_last_error().decode())
        return (state["lam"], G, kept.value) if kind == "eigh" else G
    st = state["st"]
    if kind != "march":
        st.tt_set_cores(*state["cores"])
    if kind == "round":
        ranks = st.tt_round(case["tol"])
    elif kind == "sketch":
        ranks = st.tt_round_randomized(*state["omega"])
    else:
        st.tt_step(case["steps"])
        ranks = st.ranks()
    if kind == "grad":
        loss, dk = st.tt_grad(state["p"]["detector"])
        return dict(loss=loss, dkappa=dk, r1=ranks[0], r2=ranks[1])
    E, rad, mat = st.tt_energy()
    out = dict(E=E, rad=rad, mat=mat, r1=ranks[0], r2=ranks[1])
    if case.get("problem") in ("random", "thick"):  # the materials that change
        out["T"] = st.tt_get_temperature()
    return out


def work(case):
    kind = case["kind"]
    if kind == "gram":
        K, n = case["rows"], case["cols"]
        return dict(bytes=K * n * (4 if case["single"] else 8) + 8.0 * n * n, flops=float(K) * n * (n + 1))
    if kind == "eigh":
        # tridiagonalisation, vectors of the tridiagonal, back-transformation
        n = case["n"]
        return dict(bytes=16.0 * n * n, flops=(4 / 3 + 4 / 3 + 2.0) * n ** 3)
    dim3 = "nz" in case
    ns = case["nx"] * case["ny"] * case.get("nz", 1)
    r1, r2, ang = case["r1"], case["r2"], case["ntheta"] * case["nphi"]
    if kind in ("round", "sketch"):
        k = case.get("k1", max(1, min(r1, int(8 * -math.log10(case.get("tol", 1e-4))))))
        gram = 2.0 * ns * r1 * k if kind == "sketch" else float(ns) * r1 * (r1 + 1)
        return dict(bytes=8.0 * ns * (r1 + k + 1), flops=gram + 2.0 * ns * r1 * k)
    # a step reads X and writes X' (and the energy reads X'); its contractions
    # are the Gram of the concatenated core and the update X' = X_cat P
    R1 = (7 if dim3 else 5) * r1 + 1
    passes = case["steps"] * (2 if case["twice"] else 1) * (3 if kind == "grad" else 1)
    return dict(bytes=passes * 8.0 * (2 * ns * r1 + 2 * r2 * ang) + 8.0 * ns * r1,
                flops=passes * (float(ns) * R1 * (R1 + 1) + 2.0 * ns * R1 * r1 + 8.0 * R1 ** 3))


# ---- the same results in plain numpy, by orthogonal factorisations ---------

def _truncate(X, Th, Ph, tol, rmax):
    """TT rounding by QR and SVD: per bond the smallest rank whose tail is
    within tol^2 |T|^2 / 2."""
    r1, nt, r2 = Th.shape
    Q3, R3 = np.linalg.qr(Ph.T)
    k2 = Q3.shape[1]
    W = (Th.reshape(r1 * nt, r2) @ R3.T).reshape(r1, nt * k2)
    Q2, R2 = np.linalg.qr(W.T)
    Qx, Rx = np.linalg.qr(X)
    U, S, Vt = np.linalg.svd(Rx @ R2.T, full_matrices=False)
    d2 = tol * tol * float(np.sum(S * S)) / 2.0

    def rank(s):
        tail = np.concatenate([np.cumsum((s * s)[::-1])[::-1], [0.0]])
        k = next(j for j in range(1, s.size + 1) if tail[j] <= d2)
        return min(k, rmax) if rmax > 0 else k
    a = rank(S)
    Th2 = ((S[:a, None] * Vt[:a]) @ Q2.T).reshape(a * nt, k2)
    U2, S2, V2 = np.linalg.svd(Th2, full_matrices=False)
    b = rank(S2)
    return Qx @ U[:, :a], U2[:, :b].reshape(a, nt, b), (S2[:b, None] * V2[:b]) @ Q3.T


def _angles(nt, npf):
    mu = -1.0 + (np.arange(nt) + 0.5) * (2.0 / nt)
    phi = (np.arange(npf) + 0.5) * (2.0 * np.pi / npf)
    return np.sqrt(1.0 - mu * mu), np.cos(phi), np.sin(phi)


def _energy(X, Th, Ph):
    nt, npf = Th.shape[1], Ph.shape[1]
    return X @ (Th.sum(axis=1) * (2.0 / nt) @ Ph.sum(axis=1)) * (2.0 * np.pi / npf) / LIGHT


def _upwind_step(X, Th, Ph, p, dt):
    """One 2-D upwind step at frozen temperature, vacuum or inflow faces."""
    nx, ny, r = p["nx"], p["ny"], X.shape[1]
    sint, cosp, sinp = _angles(p["ntheta"], p["nphi"])
    G = X.reshape(ny, nx, r)
    blocks = [(X, Th, Ph)]
    for ax, n, h in ((1, cosp, p["lx"] / nx), (0, sinp, p["ly"] / ny)):
        lam = LIGHT * dt / h
        lo, hi = np.zeros_like(G), np.zeros_like(G)
        if ax == 1:
            lo[:, 1:], hi[:, :-1] = G[:, :-1], G[:, 1:]
        else:
            lo[1:], hi[:-1] = G[:-1], G[1:]
        Ts = Th * sint[None, :, None]
        blocks.append(((G - lo).reshape(-1, r), Ts, Ph * (-lam * np.maximum(n, 0.0))))
        blocks.append(((hi - G).reshape(-1, r), Ts, Ph * (-lam * np.minimum(n, 0.0))))
    for face, fw, tw, pw in p["inflow"]:  # x-lo and y-lo only
        e = np.zeros((ny, nx))
        if face == 0:
            e[:, 0] = fw
        else:
            e[0, :] = fw
        n, h = (cosp, p["lx"] / nx) if face == 0 else (sinp, p["ly"] / ny)
        blocks.append((e.reshape(-1, 1), (sint * tw)[None, :, None],
                       (LIGHT * dt / h * np.maximum(n, 0.0) * pw)[None, :]))
    ext = LIGHT * dt * p["rho"] * p["kappa"]
    d = 1.0 / (1.0 + ext)
    blocks = [(d[:, None] * b[0], b[1], b[2]) for b in blocks]
    if np.any(p["T0"] != 0.0):
        s = d * ext * LIGHT / (4 * np.pi) * p["a_r"] * p["T0"] ** 4
        blocks.append((s[:, None], np.ones((1, p["ntheta"], 1)), np.ones((1, p["nphi"]))))
    R1, R2 = (sum(b[1].shape[k] for b in blocks) for k in (0, 2))
    Tc = np.zeros((R1, p["ntheta"], R2))
    i = j = 0
    for _, t, _ in blocks:
        Tc[i:i + t.shape[0], :, j:j + t.shape[2]] = t
        i, j = i + t.shape[0], j + t.shape[2]
    return _truncate(np.concatenate([b[0] for b in blocks], axis=1), Tc,
                     np.concatenate([b[2] for b in blocks], axis=0), p["tol"], p["rmax"])


def exact(case, seed):
    kind = case["kind"]
    if kind in ("gram", "eigh"):
        A = _matrix(case, seed).double()
        if kind == "gram":
            return A.T @ A
        lam, V = np.linalg.eigh(A.cpu().numpy())
        lam, V = lam[::-1].copy(), V[:, ::-1].copy()
        V *= np.sign(V[np.argmax(np.abs(V), axis=0), np.arange(V.shape[1])])
        return lam, V, None
    dV_of = lambda p: (p["lx"] / p["nx"]) * (p["ly"] / p["ny"])  # noqa: E731
    if kind == "round":
        p = _empty_problem(case)
        E = _energy(*_truncate(*_cores(case, seed), case["tol"], 0))
        return dict(E=E, rad=float(E.sum()) * dV_of(p), mat=None, r1=None, r2=None)
    if kind == "sketch":
        X, Th, Ph = _cores(case, seed)
        p = _empty_problem(case)
        o1, o2 = wl.gaussian_test_matrices(case["ntheta"], case["nphi"], case["k1"], case["k2"], seed + 1)
        r1, nt, r2 = Th.shape
        B = (Th.reshape(r1 * nt, r2) @ Ph).reshape(r1, -1)
        Q1 = np.linalg.qr(X @ (B @ o1))[0]
        A2 = ((Q1.T @ X) @ Th.reshape(r1, -1)).reshape(-1, r2)
        Q2 = np.linalg.qr(A2 @ (Ph @ o2))[0]
        E = _energy(Q1, Q2.reshape(Q1.shape[1], nt, -1), (Q2.T @ A2) @ Ph)
        return dict(E=E, rad=float(E.sum()) * dV_of(p), mat=None, r1=None, r2=None)
    if kind in ("run", "march") and case["problem"] in ("pulse", "line", "beams", "hohlraum") \
            and case["flux"] == "upwind" and not case["twice"]:
        p = _problem(case, seed)
        steps = case["steps"] + case.get("ramp", 0)
        if steps * p["nx"] * p["ny"] * (5.0 * case["r1"]) ** 2 > 2e11:
            return None
        dt = p["cfl"] * min(p["lx"] / p["nx"], p["ly"] / p["ny"]) / p["c"]
        c = (p["X0"], p["Th0"], p["Ph0"])
        for _ in range(steps):
            c = _upwind_step(*c, p, dt)
        E = _energy(*c)
        mat = float(np.sum(p["rho"] * p["cv"] * p["T0"])) * dV_of(p)
        return dict(E=E, rad=float(E.sum()) * dV_of(p), mat=mat, r1=None, r2=None)
    return None
