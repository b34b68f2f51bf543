"""Performance cases of the MRS filament library: what a program that uses it
spends its time on, through the public entry points.

`listed()` gives the standing cases, `draw(rng)` one more of the same ranges;
`prepare(case, seed)` makes the inputs and handles a program holds before the
call, `run(state)` is one pass, `work(case)` the bytes and operations a pass
cannot do without, and `exact(case, seed)` the results in float64 from plain
torch.

Kinds of case
  eval    mrs_eval_device on caller arrays: one mobility evaluation
  steps   a resident ensemble: state in (mrs_ensemble_set_state), a run of
          time steps, state and velocities out (mrs_ensemble_get)
  swim    the same for swimmers (waveform and Lennard-Jones repulsion)
  batch   new loads for many ensembles of different sizes, one batched
          evaluation (what a serving tick does), results out
  slices  perturbed copies of one ensemble stepped together from a HIP graph
          (the fine propagators of a Parareal iteration)
  rods    mrs_rod_forces_device: elastic loads of filaments on caller arrays

Results of MRS_FP32C runs are kept in single precision, which is what that
mode computes the velocities to; MRS_FP64 results stay in double.
"""
import math

import numpy as np
import torch

import paper_2604_12083_amd as mrs

_PREC = {"fp64": mrs.MRS_FP64, "fp32c": mrs.MRS_FP32C}
_INTEG = {"euler": mrs.MRS_EULER, "rk2": mrs.MRS_RK2, "rk4": mrs.MRS_RK4}
_STAGES = {"euler": 1, "rk2": 2, "rk4": 4}
_PAIR_FLOPS = 92  # of one (target, source) pair, FMA = 2
_EXACT_MOST = 2.5e10  # pairs of all evaluations above which exact() gives none


def listed():
    return [
        # the smallest call: one 64-point filament, where launches count
        {"name": "eval_64_fp64", "kind": "eval", "n": 64, "prec": "fp64"},
        # an odd mid-size one-shot evaluation
        {"name": "eval_5003_fp32c", "kind": "eval", "n": 5003, "prec": "fp32c"},
        # large one-shot evaluations in both precisions: throughput
        {"name": "eval_51200_fp64", "kind": "eval", "n": 51200, "prec": "fp64"},
        {"name": "eval_256000_fp32c", "kind": "eval", "n": 256000, "prec": "fp32c"},
        # a single relaxing filament, 100 Euler steps per call
        {"name": "rod64_fp64", "kind": "steps", "fil": 1, "pts": 64, "prec": "fp64", "integ": "euler", "dt": 1e-6,
         "nsteps": 100},
        # the benchmark ensemble, both precisions
        {"name": "ens12800_fp32c", "kind": "steps", "fil": 100, "pts": 128, "prec": "fp32c", "integ": "euler",
         "dt": 2e-7, "nsteps": 20},
        {"name": "ens12800_fp64", "kind": "steps", "fil": 100, "pts": 128, "prec": "fp64", "integ": "euler",
         "dt": 2e-7, "nsteps": 20},
        # swimmers: the paper's timing case and a large school
        {"name": "swim25_fp32c", "kind": "swim", "fil": 25, "box": 4.0, "prec": "fp32c", "integ": "rk2", "dt": 1e-6,
         "nsteps": 20},
        {"name": "swim1000_fp32c", "kind": "swim", "fil": 1000, "box": 40.0, "prec": "fp32c", "integ": "rk2",
         "dt": 1e-6, "nsteps": 4},
        # requests of different sizes in one launch sequence
        {"name": "batch12_fp32c", "kind": "batch", "ens": 12, "fil_lo": 4, "fil_hi": 64, "layout": 7,
         "prec": "fp32c"},
        # 16 fine slices of 3,200 points, RK4 from a graph
        {"name": "slices16_fp32c", "kind": "slices", "ens": 16, "fil": 32, "pts": 100, "prec": "fp32c",
         "integ": "rk4", "dt": 1e-6, "nsteps": 10},
        # the elastic loads alone (half-angle frames, forces, torques)
        {"name": "rods_25600_fp64", "kind": "rods", "fil": 200, "pts": 128, "prec": "fp64"},
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["eval", "eval", "steps", "swim", "batch", "slices", "rods"])
    prec = rng.choice(["fp64", "fp32c"])
    if kind == "eval":
        return {"kind": kind, "n": log_int(48, 100000), "prec": prec}
    if kind == "steps":
        return {"kind": kind, "fil": log_int(1, 150), "pts": rng.randint(40, 200), "prec": prec,
                "integ": rng.choice(["euler", "rk2", "rk4"]), "dt": 2e-7, "nsteps": rng.randint(5, 30)}
    if kind == "swim":
        fil = log_int(6, 500)
        return {"kind": kind, "fil": fil, "box": round(rng.uniform(0.9, 1.3) * math.sqrt(fil), 3), "prec": prec,
                "integ": rng.choice(["euler", "rk2", "rk4"]), "dt": 1e-6, "nsteps": rng.randint(2, 10)}
    if kind == "batch":
        return {"kind": kind, "ens": rng.randint(2, 20), "fil_lo": 2, "fil_hi": log_int(8, 80),
                "layout": rng.randrange(1 << 20), "prec": prec}
    if kind == "slices":
        return {"kind": kind, "ens": rng.randint(3, 16), "fil": log_int(4, 32), "pts": rng.randint(50, 140),
                "prec": prec, "integ": rng.choice(["rk2", "rk4"]), "dt": 1e-6, "nsteps": rng.randint(4, 12)}
    return {"kind": kind, "fil": log_int(1, 400), "pts": rng.randint(2, 300), "prec": "fp64"}


# ------------------------------------------------------------------- inputs

_SWIM_POINTS = 51  # points of a swimmer


def _unit(v):
    return v / np.linalg.norm(v, axis=-1, keepdims=True)


def _filaments(rng, counts, box, ds):
    """Sinusoidal filaments (amplitude 0.1, wavelength 1) of counts[i] points
    at spacing ds, bases uniform in [0, box]^3, any direction and plane, with
    random point loads: (offsets, X, D, f, n)."""
    F = len(counts)
    base = rng.uniform(0.0, box, size=(F, 3))
    d = _unit(rng.normal(size=(F, 3)))
    a = np.where(np.abs(d[:, :1]) > 0.9, [[0.0, 1.0, 0.0]], [[1.0, 0.0, 0.0]])
    p0 = _unit(np.cross(d, a))
    psi = rng.uniform(0.0, 2.0 * math.pi, size=(F, 1))
    p = np.cos(psi) * p0 + np.sin(psi) * np.cross(d, p0)
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    fil = np.repeat(np.arange(F), counts)
    s = ((np.arange(off[-1]) - off[fil]) * ds)[:, None]
    w = 2.0 * math.pi
    X = base[fil] + s * d[fil] + 0.1 * np.sin(w * s) * p[fil]
    tangent = _unit(d[fil] + 0.1 * w * np.cos(w * s) * p[fil])
    normal = np.cross(d, p)[fil]
    D = np.concatenate([np.cross(normal, tangent), normal, tangent], axis=1)
    return off, X, D, rng.normal(size=X.shape), rng.normal(size=X.shape)


def _box(n):
    """Side of the box that keeps the density of 12,800 points in side 10."""
    return 10.0 * (n / 12800.0) ** (1.0 / 3.0)


def _swimmers(rng, F, box):
    """F straight rods of length 1 near the plane z = 1, no two points of
    different rods closer than 0.2 (a candidate that is too close is drawn
    again): (offsets, X, D)."""
    M = _SWIM_POINTS
    s = np.arange(M) / (M - 1) - 0.5
    cells, Xs, ds = {}, [], []
    while len(Xs) < F:
        c = np.array([*rng.uniform(0.0, box, size=2), rng.uniform(0.9, 1.1)])
        ang = rng.uniform(0.0, 2.0 * math.pi)
        d = np.array([math.cos(ang), math.sin(ang), 0.0])
        X = c + s[:, None] * d
        key = (int(c[0] // 1.2), int(c[1] // 1.2))
        close = [j for i in (-1, 0, 1) for k in (-1, 0, 1) for j in cells.get((key[0] + i, key[1] + k), [])]
        if any(np.min(((X[:, None] - Xs[j][None]) ** 2).sum(-1)) < 0.04 for j in close):
            continue
        cells.setdefault(key, []).append(len(Xs))
        Xs.append(X)
        ds.append(d)
    d = np.repeat(np.array(ds), M, axis=0)
    z = np.broadcast_to([0.0, 0.0, 1.0], d.shape)
    return (np.arange(F + 1) * M).astype(np.int32), np.concatenate(Xs), np.concatenate([np.cross(z, d), z, d], axis=1)


def _rotate_rows(D, v):
    """Frames D (n x 9) with every director rotated by the rotation vector v."""
    th = np.linalg.norm(v, axis=1)[:, None, None]
    k = (v / np.maximum(np.linalg.norm(v, axis=1, keepdims=True), 1e-300))[:, None, :]
    d = D.reshape(-1, 3, 3)
    out = d * np.cos(th) + np.cross(k, d) * np.sin(th) + k * (k * d).sum(-1, keepdims=True) * (1 - np.cos(th))
    return np.ascontiguousarray(out.reshape(-1, 9))


def _batch_counts(case):
    r = np.random.default_rng(case["layout"])
    out = []
    for _ in range(case["ens"]):
        F = int(round(math.exp(r.uniform(math.log(case["fil_lo"]), math.log(case["fil_hi"])))))
        out.append([int(r.integers(64, 257))] * F)
    return out


def _inputs(case, seed):
    """The ensembles of a case, each a dict of host arrays and parameters."""
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    if kind == "eval":
        n, ds = case["n"], 1.0 / 128
        off, X, D, f, t = _filaments(rng, [128] * ((n + 127) // 128), _box(n), ds)
        return [dict(X=X[:n].copy(), f=f[:n].copy(), n=t[:n].copy(), eps=1.5 * ds, mu=1.0)]
    if kind == "swim":
        off, X, D = _swimmers(rng, case["fil"], case["box"])
        ds = 1.0 / (_SWIM_POINTS - 1)
        return [dict(off=off, X=X, D=D, f=None, n=None, eps=4.0 * ds, mu=1.0, ds=ds, a=1e-3,
                     wave=(0.05, 2.0 * math.pi, 20.0 * math.pi), lj=(12.0 * ds, 1e-4))]
    if kind == "batch":
        counts = _batch_counts(case)
    else:
        counts = [[case["pts"]] * case["fil"]]
    ens = []
    for c in counts:
        ds = 1.0 / c[0]
        off, X, D, f, t = _filaments(rng, c, _box(sum(c)), ds)
        ens.append(dict(off=off, X=X, D=D, f=f, n=t, eps=1.5 * ds, mu=1.0, ds=ds, a=1e-4, wave=None, lj=None))
    if kind == "slices":
        base, ens = ens[0], []
        for _ in range(case["ens"]):
            e = dict(base)
            e["X"] = base["X"] + rng.normal(scale=1e-3, size=base["X"].shape)
            e["D"] = _rotate_rows(base["D"], rng.normal(scale=1e-3, size=base["X"].shape))
            ens.append(e)
    elif kind == "rods":  # strained and twisted filaments
        e = ens[0]
        e["X"] = e["X"] + rng.normal(scale=2e-3, size=e["X"].shape)
        e["D"] = _rotate_rows(e["D"], rng.normal(scale=0.05, size=e["X"].shape))
    return ens


class _Ens:
    """A resident ensemble that is freed with its state."""

    def __init__(self, ctx, e):
        rod = mrs.rod_params((e["a"],) * 3, (1.0,) * 3, (0.0,) * 3, e["ds"])
        self.h = mrs.mrs_ensemble_create(ctx, e["off"], e["X"], e["D"], e["f"], e["n"], e["eps"], e["mu"], rod)
        if e["wave"] is not None:
            mrs.mrs_ensemble_set_swimming(ctx, self.h, e["wave"], e["lj"])

    def __del__(self):
        mrs.mrs_ensemble_destroy(self.h)


_ctx = []


def _context():
    if not _ctx:
        _ctx.append(mrs.mrs_context_create(0))
    return _ctx[0]


def prepare(case, seed):
    ctx = _context()
    ens = _inputs(case, seed)
    st = {"case": case, "ctx": ctx, "prec": _PREC[case["prec"]]}
    if case["kind"] in ("eval", "rods"):
        e = ens[0]
        st["stream"] = torch.cuda.Stream()
        for k in ("X", "D", "f", "n"):
            if k in e:
                st[k] = torch.from_numpy(e[k]).cuda()
        st["eps"], st["mu"] = e["eps"], e["mu"]
        st["U"], st["W"] = torch.empty_like(st["X"]), torch.empty_like(st["X"])
        if case["kind"] == "rods":
            st["off"] = e["off"]
            st["rod"] = mrs.rod_params((e["a"],) * 3, (1.0,) * 3, (0.0,) * 3, e["ds"])
        torch.cuda.synchronize()
    else:
        st["host"] = ens
        st["ens"] = [_Ens(ctx, e) for e in ens]
    return st


# ------------------------------------------------------------------- passes


def _kept(st, arrays):
    return [a.astype(np.float32) for a in arrays] if st["prec"] == mrs.MRS_FP32C else list(arrays)


def run(st):
    case, ctx, prec = st["case"], st["ctx"], st["prec"]
    kind = case["kind"]
    if kind == "eval":
        with torch.cuda.stream(st["stream"]):
            mrs.mrs_eval_device(ctx, case["n"], st["X"], st["f"], st["n"], st["eps"], st["mu"], prec, st["U"],
                                st["W"], st["stream"])
            return (st["U"].float(), st["W"].float()) if prec == mrs.MRS_FP32C else (st["U"], st["W"])
    if kind == "rods":
        mrs.mrs_rod_forces_device(ctx, st["off"], st["X"], st["D"], st["rod"], st["f"], st["n"], st["U"], st["W"],
                                  st["stream"])
        return st["U"], st["W"]
    hs = [e.h for e in st["ens"]]
    if kind == "batch":
        for h, e in zip(hs, st["host"]):
            mrs.mrs_ensemble_set_external(ctx, h, e["f"], e["n"])
        mrs.mrs_batch_eval(ctx, hs, prec, True)
        return [_kept(st, mrs.mrs_ensemble_get(ctx, h)[2:]) for h in hs]
    for h, e in zip(hs, st["host"]):
        mrs.mrs_ensemble_set_state(ctx, h, e["X"], e["D"])
        if e["wave"] is not None:
            mrs.mrs_ensemble_set_time(ctx, h, 0.0)
    integ = _INTEG[case["integ"]]
    if kind == "slices":
        mrs.mrs_batch_step(ctx, hs, integ, case["dt"], case["nsteps"], prec, True, True)
    else:
        mrs.mrs_ensemble_step(ctx, hs[0], integ, case["dt"], case["nsteps"], prec, True)
    got = [_kept(st, mrs.mrs_ensemble_get(ctx, h)) for h in hs]
    # 16 slices of X, D, U, Omega: one array per slice and quantity, joined per slice
    return [np.concatenate(g, axis=1) for g in got] if kind == "slices" else got[0]


def _sizes(case):
    kind = case["kind"]
    if kind == "eval":
        return [case["n"]]
    if kind == "swim":
        return [case["fil"] * _SWIM_POINTS]
    if kind == "batch":
        return [sum(c) for c in _batch_counts(case)]
    return [case["fil"] * case["pts"]] * case.get("ens", 1)


def _evals(case):
    return _STAGES[case["integ"]] * case["nsteps"] if "integ" in case else 1


def work(case):
    kind, n = case["kind"], _sizes(case)
    if kind == "rods":  # X, D, f, n in, g, m out; about 300 operations per segment
        return {"bytes": 8.0 * 24 * n[0], "flops": 300.0 * n[0]}
    per = {"eval": 15, "batch": 12, "steps": 30, "swim": 30, "slices": 30}[kind]  # doubles in and out per point
    return {"bytes": 8.0 * per * sum(n), "flops": float(_PAIR_FLOPS) * _evals(case) * sum(k * k for k in n)}


# ----------------------------------------------- the same in plain float64


def _mobility(X, f, n, eps, mu):
    """U, Omega of all points (regularised Stokeslet, rotlet and dipole sums
    of the blob 15 eps^4 / (8 pi (r^2 + eps^2)^(7/2)))."""
    N = X.shape[0]
    U, W = torch.empty_like(X), torch.empty_like(X)
    e2 = eps * eps
    step = max(1, int(2 ** 24 // max(N, 1)))
    src = [X[:, c][None] for c in range(3)]
    fs = [f[:, c][None] for c in range(3)]
    ns = [n[:, c][None] for c in range(3)]
    for a in range(0, N, step):
        r = [X[a:a + step, c][:, None] - src[c] for c in range(3)]
        R2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2] + e2
        q = 1.0 / torch.sqrt(R2)
        i2 = 1.0 / R2
        q3 = q * i2
        q5 = q3 * i2
        q7 = q5 * i2
        fr = r[0] * fs[0] + r[1] * fs[1] + r[2] * fs[2]
        nr = r[0] * ns[0] + r[1] * ns[1] + r[2] * ns[2]
        A = q3 * fr
        B = (1.5 * q5 + 3.75 * e2 * q7) * nr
        h3 = q3 + 1.5 * e2 * q5
        g = [h3 * r[c] for c in range(3)]
        u = (q + e2 * q3) @ f
        w = (3.75 * e2 * e2 * q7 - 0.75 * e2 * q5 - 0.5 * q3) @ n
        gn = [[g[c] @ n[:, k] for k in range(3)] for c in range(3)]
        gf = [[g[c] @ f[:, k] for k in range(3)] for c in range(3)]
        for c in range(3):
            i, j = (c + 1) % 3, (c + 2) % 3
            u[:, c] += (A * r[c]).sum(1) + gn[j][i] - gn[i][j]
            w[:, c] += (B * r[c]).sum(1) + gf[j][i] - gf[i][j]
        U[a:a + step], W[a:a + step] = u, w
    k = 1.0 / (8.0 * math.pi * mu)
    return k * U, k * W


def _loads(e, X, D, t):
    """Point forces and torques on the fluid: external, elastic (half-angle
    mid frames) and Lennard-Jones."""
    off = torch.from_numpy(np.asarray(e["off"], dtype=np.int64)).to(X.device)
    N, F = X.shape[0], off.numel() - 1
    fil = torch.repeat_interleave(torch.arange(F, device=X.device), off[1:] - off[:-1])
    g = torch.zeros_like(X) if e["f"] is None else torch.from_numpy(e["f"]).to(X)
    m = torch.zeros_like(X) if e["n"] is None else torch.from_numpy(e["n"]).to(X)
    g, m = g.clone(), m.clone()
    k = torch.nonzero(fil[1:] == fil[:-1])[:, 0]  # segment between nodes k and k + 1
    if k.numel():
        ds = e["ds"]
        Da, Db = D[k].view(-1, 3, 3), D[k + 1].view(-1, 3, 3)  # [segment, director, component]
        R = (Db[:, :, :, None] * Da[:, :, None, :]).sum(1)
        tr = R[:, 0, 0] + R[:, 1, 1] + R[:, 2, 2]
        w = 0.5 * torch.sqrt(1.0 + tr)
        V = (R - R.transpose(1, 2)) / (4.0 * w)[:, None, None]
        V2 = (V[:, :, :, None] * V[:, None, :, :]).sum(2)
        S = torch.eye(3, dtype=X.dtype, device=X.device) + V + V2 / (1.0 + w)[:, None, None]
        Dh = (S[:, None, :, :] * Da[:, :, None, :]).sum(3)
        dX = X[k + 1] - X[k]
        stretch = (dX[:, None, :] * Dh).sum(2) / ds
        stretch[:, 2] -= 1.0
        Fs = (stretch[:, :, None] * Dh).sum(1)
        om = torch.zeros(k.numel(), 3, dtype=X.dtype, device=X.device)
        if e["wave"] is not None:
            A, kw, fw = e["wave"]
            s = ((k - off[fil[k]]).to(X.dtype) + 0.5) * ds
            om[:, 1] -= kw * kw * A * torch.sin(kw * s + fw * t)
        kap = torch.stack([((Db[:, (i + 1) % 3] - Da[:, (i + 1) % 3]) * Dh[:, (i + 2) % 3]).sum(1)
                           for i in range(3)], 1) / ds - om
        Ns = e["a"] * (kap[:, :, None] * Dh).sum(1)
        cr = 0.5 * torch.linalg.cross(dX, Fs)
        g.index_add_(0, k, Fs)
        g.index_add_(0, k + 1, -Fs)
        m.index_add_(0, k, Ns + cr)
        m.index_add_(0, k + 1, cr - Ns)
    if e["lj"] is not None:
        sig, en = e["lj"]
        rc2 = 2.0 ** (1.0 / 3.0) * sig * sig
        step = max(1, int(2 ** 24 // N))
        for a in range(0, N, step):
            r = X[a:a + step, None, :] - X[None, :, :]
            r2 = (r * r).sum(2)
            near = (r2 < rc2) & (fil[a:a + step, None] != fil[None, :])
            r2 = torch.where(near, r2, torch.ones_like(r2))
            s6 = (sig * sig / r2) ** 3
            c = torch.where(near, 24.0 * en * (2.0 * s6 * s6 - s6) / r2, torch.zeros_like(r2))
            g[a:a + step] += (c[:, :, None] * r).sum(1)
    return g, m


def _rotated(D, v, clean):
    """Frames rotated by the rotation vectors v; clean: made orthonormal again."""
    th = torch.linalg.norm(v, dim=1)[:, None, None]
    half = torch.sinc(0.5 * th / math.pi)  # sin(th / 2) / (th / 2)
    x = v[:, None, :].expand(-1, 3, -1)
    d = D.view(-1, 3, 3)
    c1 = torch.linalg.cross(x, d)
    d = d + torch.sinc(th / math.pi) * c1 + 0.5 * half * half * torch.linalg.cross(x, c1)
    if clean:
        d3 = d[:, 2] / torch.linalg.norm(d[:, 2], dim=1, keepdim=True)
        d1 = d[:, 0] - (d[:, 0] * d3).sum(1, keepdim=True) * d3
        d1 = d1 / torch.linalg.norm(d1, dim=1, keepdim=True)
        d = torch.stack([d1, torch.linalg.cross(d3, d1), d3], 1)
    return d.reshape(-1, 9)


def _exact_steps(case, e):
    X, D = torch.from_numpy(e["X"]).cuda(), torch.from_numpy(np.ascontiguousarray(e["D"])).cuda()
    dt, integ, t = case["dt"], case["integ"], 0.0
    node = {"euler": [0.0], "rk2": [0.0, 0.5], "rk4": [0.0, 0.5, 0.5, 1.0]}[integ]
    weight = {"euler": [1.0], "rk2": [0.0, 1.0], "rk4": [1 / 6, 1 / 3, 1 / 3, 1 / 6]}[integ]
    for _ in range(case["nsteps"]):
        su, sw, Xs, Ds, k = 0.0, 0.0, X, D, None
        for s, (c, w) in enumerate(zip(node, weight)):
            if s:
                Xs, Ds = X + c * dt * Us, _rotated(D, c * dt * k, False)
            g, m = _loads(e, Xs, Ds, t + c * dt)
            Us, Ws = _mobility(Xs, g, m, e["eps"], e["mu"])
            if s == 0:
                U, W = Us, Ws
            if integ == "rk4" and s:  # the inverse derivative of the exponential map, to the order needed
                th = c * dt * k
                t1 = torch.linalg.cross(th, Ws)
                k = Ws - 0.5 * t1 + torch.linalg.cross(th, t1) / 12.0
            else:
                k = Ws
            su, sw = su + w * Us, sw + w * k
        X, D, t = X + dt * su, _rotated(D, dt * sw, True), t + dt
    return [X, D, U, W]


def exact(case, seed):
    if case["kind"] != "rods" and _evals(case) * sum(k * k for k in _sizes(case)) > _EXACT_MOST:
        return None
    ens = _inputs(case, seed)
    kind = case["kind"]
    if kind == "eval":
        e = ens[0]
        X, f, n = (torch.from_numpy(e[k]).cuda() for k in ("X", "f", "n"))
        return _mobility(X, f, n, e["eps"], e["mu"])
    if kind in ("rods", "batch"):
        out = []
        for e in ens:
            X, D = torch.from_numpy(e["X"]).cuda(), torch.from_numpy(np.ascontiguousarray(e["D"])).cuda()
            g, m = _loads(e, X, D, 0.0)
            out.append((g, m) if kind == "rods" else _mobility(X, g, m, e["eps"], e["mu"]))
        return out[0] if kind == "rods" else out
    if kind == "slices":
        return [torch.cat(_exact_steps(case, e), 1) for e in ens]
    return _exact_steps(case, ens[0])
