"""What is timed: the calls a user of the hydrodynamics library makes, over the range of their sizes.

Five kinds of case, each through the Python binding:

 * "patch":  one patch advanced by a number of Runge-Kutta steps (1D, 2D, 3D; FP32 and FP64; HLL, HLLC and the
   HLLC -> HLL switch; generalised-minmod and learned slopes; launched steps, a graph replay, or the host's own loop);
 * "tubes":  a batch of shock tubes set, run to one time and read back;
 * "levels": global steps of nested levels (subcycling, flux replacement), every level read back;
 * "train":  training samples of a fine run and Adam steps of the limiter's network on them;
 * the Kelvin-Helmholtz diagnostics (kinetic energy, its spectrum) after the steps of a "patch" case with "diag".

exact() is the method in 64 bits in plain torch, written from the formulas of the method.
"""
import math

import numpy as np
import torch

from paper_1207_3392_amd import hydro
from paper_1207_3392_amd import limiter
from paper_1207_3392_amd import workloads as wl

PER, OUT, REF = 0, 1, 2
HLL, HLLC, SWITCH = 0, 1, 2


def _patch(name, problem, nx, ny=1, nz=1, bits=32, solver=HLLC, theta=2.0, cfl=0.4, steps=10, mode="graph",
           learned=False, diag=False):
    return {"name": name, "kind": "patch", "problem": problem, "nx": nx, "ny": ny, "nz": nz, "bits": bits,
            "solver": solver, "theta": theta, "cfl": cfl, "steps": steps, "mode": mode, "learned": learned, "diag": diag}


def listed():
    return [
        # the smallest run: a shock tube as in the convergence tables, 100 steps launched one by one, read back
        _patch("sod1d_600", "sod", 600, theta=1.4, cfl=0.5, steps=100, mode="launch"),
        # a small 2D run driven by the host's own loop (dt read back before every step), reflecting walls
        _patch("implosion2d_180x150", "blast", 180, 150, solver=HLL, theta=1.4, cfl=0.4, steps=10, mode="host"),
        # the paper's Kelvin-Helmholtz resolution, with the diagnostics it is analysed by
        _patch("kh2d_2048", "kh", 2048, 2048, steps=20, diag=True),
        # the 3D benchmark flow at the size that one GPU of a split run gets
        _patch("flow3d_256", "smooth", 256, 256, 256, cfl=0.3, steps=10),
        # Rayleigh-Taylor: gravity, walls in z, HLL, a box that no tile divides, launched steps
        _patch("rt3d_250x190x310", "rt", 250, 190, 310, solver=HLL, cfl=0.3, steps=10, mode="launch"),
        # double precision, for reference runs
        _patch("blast3d_f64_150x140x130", "blast", 150, 140, 130, bits=64, theta=1.4, cfl=0.3, steps=10),
        # strong shocks with the HLLC -> HLL switch
        _patch("blast3d_switch_200x180x160", "blast", 200, 180, 160, solver=SWITCH, theta=1.4, cfl=0.3, steps=10),
        # the learned limiter in 2D (its training flow) and in 3D
        _patch("kh2d_1024_learned", "kh", 1024, 1024, steps=10, learned=True),
        _patch("rt3d_learned_150x120x160", "rt", 150, 120, 160, cfl=0.3, steps=4, mode="launch", learned=True),
        # a parameter study: 512 uneven tubes to one time
        {"name": "tubes_512", "kind": "tubes", "count": 512, "nmin": 128, "nmax": 4096, "solver": HLLC, "t_end": 0.1},
        # the paper's multilevel depth in 2D
        {"name": "sedov2d_7x256", "kind": "levels", "problem": "sedov", "ndim": 2, "n0": 256, "nlev": 7, "bits": 32, "solver": HLL,
         "cfl": 0.4, "steps": 10},
        # retraining the limiter: samples of a fine run, then Adam steps over them
        {"name": "train_2048", "kind": "train", "n": 2048, "batch": 65536, "steps": 40},
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: a kind, then sizes spread over the range that the listed ones span."""
    kind = rng.choice(["1d", "2d", "2d", "3d", "3d", "f64", "learned", "tubes", "levels", "train"])
    if kind == "1d":
        c = _patch("", "sod", _logint(rng, 100, 20000), bits=rng.choice([32, 64]), solver=rng.choice([HLL, HLLC]),
                   theta=rng.choice([1.0, 1.4, 2.0]), cfl=0.5, steps=2 * rng.randint(20, 60), mode=rng.choice(["launch", "graph"]))
    elif kind == "2d":
        p = rng.choice(["blast", "kh"])
        c = _patch("", p, _logint(rng, 100, 2000), _logint(rng, 100, 2000), solver=rng.choice([HLL, HLLC, SWITCH]),
                   theta=rng.choice([1.4, 2.0]), steps=2 * rng.randint(3, 8), mode=rng.choice(["launch", "graph", "host"]))
    elif kind == "3d":
        p = rng.choice(["smooth", "rt", "blast"])
        c = _patch("", p, rng.randint(60, 250), rng.randint(60, 250), rng.randint(60, 250), solver=rng.choice([HLL, HLLC, SWITCH]),
                   theta=1.4 if p == "blast" else 2.0, cfl=0.3, steps=2 * rng.randint(2, 5), mode=rng.choice(["launch", "graph"]))
    elif kind == "f64":
        if rng.random() < 0.5:
            c = _patch("", "blast", _logint(rng, 100, 1500), _logint(rng, 100, 1500), bits=64, solver=rng.choice([HLL, HLLC, SWITCH]),
                       theta=1.4, steps=2 * rng.randint(2, 6), mode=rng.choice(["launch", "graph"]))
        else:
            c = _patch("", "smooth", rng.randint(50, 150), rng.randint(50, 150), rng.randint(50, 150), bits=64,
                       solver=rng.choice([HLL, HLLC]), cfl=0.3, steps=2 * rng.randint(1, 4))
    elif kind == "learned":
        if rng.random() < 0.5:
            c = _patch("", "kh", _logint(rng, 150, 1024), _logint(rng, 150, 1024), steps=2 * rng.randint(2, 5), learned=True)
        else:
            c = _patch("", "rt", rng.randint(50, 150), rng.randint(50, 130), rng.randint(50, 160), cfl=0.3,
                       steps=2 * rng.randint(1, 2), mode="launch", learned=True)
    elif kind == "tubes":
        nmin = _logint(rng, 64, 1000)
        c = {"kind": "tubes", "count": _logint(rng, 8, 400), "nmin": nmin, "nmax": nmin + _logint(rng, 100, 3000),
             "solver": rng.choice([HLL, HLLC]), "t_end": rng.choice([0.03, 0.05, 0.08])}
    elif kind == "levels":
        if rng.random() < 0.6:
            # the blast needs enough levels that its fastest waves stay in the finest ones
            nlev = rng.randint(2, 7)
            c = {"kind": "levels", "problem": "sedov" if nlev > 4 else "waves", "ndim": 2, "n0": 4 * rng.randint(16, 64), "nlev": nlev,
                 "bits": rng.choice([32, 32, 64]), "solver": rng.choice([HLL, HLLC]), "cfl": 0.3, "steps": rng.randint(4, 8)}
        else:
            c = {"kind": "levels", "problem": "waves", "ndim": 3, "n0": 4 * rng.randint(8, 24), "nlev": rng.randint(2, 4), "bits": 32,
                 "solver": rng.choice([HLL, HLLC]), "cfl": 0.25, "steps": rng.randint(2, 4)}
    else:
        c = {"kind": "train", "n": 4 * rng.randint(100, 500), "batch": _logint(rng, 4000, 100000), "steps": rng.randint(10, 40)}
    c.pop("name", None)
    return c


# ---------------------------------------------------------------- inputs ----


def _dev():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _axes(n, lo, hi, dev):
    """Cell centres along z, y, x (those with more than one cell), shaped to broadcast."""
    nd = 3 if n[2] > 1 else (2 if n[1] > 1 else 1)
    out = []
    for q in range(nd):
        c = lo[q] + (torch.arange(n[q], dtype=torch.float64, device=dev) + 0.5) * ((hi[q] - lo[q]) / n[q])
        out.append(c.reshape([-1 if r == q else 1 for r in reversed(range(nd))]))
    return out  # x, y, z


def _problem(c, seed):
    """The initial state: a workloads.Problem whose W is a float64 tensor on the GPU."""
    dev = _dev()
    rng = np.random.default_rng(seed)
    n = (c["nx"], c["ny"], c["nz"])
    nd = 3 if n[2] > 1 else (2 if n[1] > 1 else 1)
    shape = tuple(reversed(n[:nd]))
    # cubic cells, as in the paper's runs; the Kelvin-Helmholtz box is the unit square
    lo, hi = [0.0, 0.0, 0.0], [1.0, n[1] / n[0] if nd > 1 else 1.0, n[2] / n[0] if nd > 2 else 1.0]
    gamma, accel, bc = 1.4, (0.0, 0.0, 0.0), [[REF, REF]] * 3
    W = torch.zeros((nd + 2,) + shape, dtype=torch.float64, device=dev)
    if c["problem"] == "kh":
        hi, gamma, bc = [1.0, 1.0, 1.0], 5.0 / 3.0, [[PER, PER]] * 3
        x, y = _axes(n, lo, hi, dev)
        inner = 0.5 * (torch.tanh((y - 0.25) / 0.025) - torch.tanh((y - 0.75) / 0.025))
        lat = torch.tensor(rng.uniform(-1e-3, 1e-3, size=(64, 64)), device=dev)
        ix = (x * 64).long().clamp(max=63).reshape(-1)
        iy = (y * 64).long().clamp(max=63).reshape(-1)
        W[0] = 1.0 + inner
        W[1] = -0.5 + inner
        W[2] = (0.01 * torch.sin(2 * math.pi * x) + lat[iy][:, ix]) * torch.exp(-0.5 * (torch.cos(2 * math.pi * y) / (0.2 * math.pi)) ** 2)
        W[3] = 2.5
    elif c["problem"] == "smooth":
        gamma, bc, hi = 5.0 / 3.0, [[PER, PER]] * 3, [1.0, 1.0, 1.0]
        x, y, z = _axes(n, lo, hi, dev)
        W[0] = 1.0
        W[4] = 1.0
        for v, amp in ((0, 0.2), (1, 0.1), (2, 0.1), (3, 0.1)):
            for _ in range(8):
                k, ph = rng.integers(-3, 4, size=3), rng.uniform(0, 2 * math.pi)
                a = 2 * math.pi * (int(k[0]) * x + int(k[1]) * y)
                b = 2 * math.pi * int(k[2]) * z + ph
                W[v] += amp / 8 * (torch.cos(a) * torch.cos(b) - torch.sin(a) * torch.sin(b))
    elif c["problem"] == "rt":
        accel, bc = (0.0, 0.0, -0.1), [[PER, PER], [PER, PER], [REF, REF]]
        lo, hi = [-0.5, -0.5 * hi[1], -0.5 * hi[2]], [0.5, 0.5 * hi[1], 0.5 * hi[2]]
        x, y, z = _axes(n, lo, hi, dev)
        rho = torch.where(z > 0, 2.0, 1.0)
        W[0] = rho
        pert = torch.zeros((1,) + shape[1:], dtype=torch.float64, device=dev)
        for _ in range(8):
            k, ph = rng.integers(-4, 5, size=2), rng.uniform(0, 2 * math.pi)
            pert = pert + torch.cos(2 * math.pi * (int(k[0]) * x + int(k[1]) * y / (hi[1] - lo[1])) + ph)
        W[3] = 0.01 * pert / 8 * 0.5 * (1 + torch.cos(2 * math.pi * z / (hi[2] - lo[2])))
        W[4] = 2.5 - rho * 0.1 * z
    elif c["problem"] == "blast":
        # a hot ball in a closed box: shocks that meet the walls and each other
        xs = _axes(n, lo, hi, dev)
        centre = rng.uniform(0.3, 0.6, size=nd)
        r2 = sum((a - float(centre[q]) * hi[q]) ** 2 for q, a in enumerate(xs))
        inside = r2 < (0.2 * min(hi[:nd])) ** 2
        pin, rin = rng.uniform(2.0, 4.0), rng.uniform(0.5, 2.0)
        W[0] = torch.where(inside, float(rin), 1.0)
        W[nd + 1] = torch.where(inside, float(pin), 0.3)
    elif c["problem"] == "waves":
        # a developed periodic flow: every variable varies everywhere
        hi, gamma, bc = [1.0, 1.0, 1.0], 5.0 / 3.0, [[PER, PER]] * 3
        x, y = _axes(n, lo, hi, dev)
        for v, (mean, amp) in enumerate(((1.0, 0.4), (0.0, 0.5), (0.0, 0.5), (2.5, 0.4))):
            W[v] = mean
            for _ in range(12):
                k, ph = rng.integers(-20, 21, size=2), rng.uniform(0, 2 * math.pi)
                W[v] += amp / 6 * torch.cos(2 * math.pi * (int(k[0]) * x + int(k[1]) * y) + ph)
    else:  # "sod"
        bc = [[OUT, OUT]] * 3
        (x,) = _axes(n, lo, hi, dev)
        f = rng.uniform(0.8, 1.2, size=4)
        W[0] = torch.where(x < 0.5, f[0], 0.125 * f[1])
        W[2] = torch.where(x < 0.5, f[2], 0.1 * f[3])
    bc = [bc[q] if q < nd else [0, 0] for q in range(3)]
    hi = [hi[q] if q < nd else 1.0 for q in range(3)]
    lo = [lo[q] if q < nd else 0.0 for q in range(3)]
    return wl.Problem(nd, n, tuple(lo), tuple(hi), gamma, tuple(tuple(b) for b in bc), W, theta=c["theta"], cfl=c["cfl"], accel=accel)


def _conserved(W, nd, gamma):
    U = W.clone()
    U[1:nd + 1] *= W[0]
    U[nd + 1] = W[nd + 1] / (gamma - 1) + 0.5 * W[0] * (W[1:nd + 1] ** 2).sum(0)
    return U


def _state_view(patch, U):
    """The conserved state on the GPU, where the library keeps it: in the workspace that this program owns (what a program
    that renders or couples the flow on the GPU reads).  Found by the values that set_state has just put there."""
    dt = torch.float32 if patch.precision == 32 else torch.float64
    es = 4 if patch.precision == 32 else 8
    flat = U.reshape(patch.nv, -1).to(dt)
    start = -patch.workspace.data_ptr() % 256
    ws = patch.workspace[start:start + (patch.workspace.numel() - start) // 256 * 256].view(dt)
    per = 256 // es

    def find(v, after):
        k = min(8, patch.ncell)
        rows = ws.view(-1, per)[:, :k]
        for i in torch.nonzero((rows == flat[v, :k]).all(1)).reshape(-1).tolist():
            o = i * per
            if o >= after and o + patch.ncell <= ws.numel() and bool((ws[o:o + patch.ncell] == flat[v]).all()):
                return o
        raise RuntimeError("the state is not in the workspace")

    first = find(0, 0)
    stride = (find(patch.nv - 1, first + patch.ncell) - first) // (patch.nv - 1)
    return torch.as_strided(ws, (patch.nv, patch.ncell), (stride, 1), ws.storage_offset() + first)


def _tube_problems(c, seed):
    # the lengths belong to the study, the states are its inputs
    lengths = [t.n for t in wl.batched_tubes(c["count"], c["count"], c["nmin"], c["nmax"])]
    states = wl.batched_tubes(c["count"], seed, c["nmin"], c["nmax"])
    return [wl.tube_problem(wl.Tube(n, t.left, t.right, (n // 2) / n), t_end=c["t_end"]) for n, t in zip(lengths, states)]


def _levels(c, seed):
    if c["problem"] == "waves":
        return wl.smooth_levels(c["ndim"], c["n0"], c["nlev"], seed)
    rng = np.random.default_rng(seed)
    return wl.sedov_levels(c["ndim"], c["n0"], c["nlev"], e_d=float(rng.uniform(0.5, 1.5)), p0=float(rng.uniform(0.5e-5, 2e-5)))


def _fine(c):
    return {"problem": "waves", "nx": c["n"], "ny": c["n"], "nz": 1, "theta": 2.0, "cfl": 0.4}


def prepare(case, seed):
    c = case
    if c["kind"] == "patch":
        pr = _problem(c, seed)
        U = _conserved(pr.W, pr.ndim, pr.gamma)
        p = hydro.Patch(pr, c["bits"], hydro.LIM_LEARNED if c["learned"] else hydro.LIM_THETA, set_initial=False)
        p.workspace.zero_()
        p.set_state(U.cpu().numpy(), hydro.CONSERVED)
        pr.W = None
        s = {"case": c, "patch": p}
        if c["nx"] * c["ny"] * c["nz"] > 100000:  # small runs are read back to the host
            s["state"] = _state_view(p, U)
        if c["learned"]:
            p.set_mlp(limiter.trained_params())
        if c["mode"] == "graph":
            p.advance_graph(c["steps"], c["cfl"], solver=c["solver"], prepare_only=True)
        return s
    if c["kind"] == "tubes":
        problems = _tube_problems(c, seed)
        return {"case": c, "batch": hydro.Batch(problems), "W": [p.W for p in problems]}
    if c["kind"] == "levels":
        return {"case": c, "fmr": hydro.Fmr(_levels(c, seed), c["bits"])}
    pr = _problem(_fine(c), seed)
    pr.W = pr.W.cpu().numpy()
    p = hydro.Patch(pr)
    rng = np.random.default_rng(seed)
    idx = torch.tensor(rng.integers(0, p.sample_count(), size=(c["steps"], c["batch"])), dtype=torch.int32, device=_dev())
    return {"case": c, "patch": p, "idx": idx, "trainer": hydro.Trainer(limiter.init_params(seed))}


# ------------------------------------------------------------------ pass ----


def run(state):
    c = state["case"]
    if c["kind"] == "patch":
        p = state["patch"]
        if c["mode"] == "graph":
            p.advance_graph(c["steps"], c["cfl"], solver=c["solver"])
        elif c["mode"] == "launch":
            p.advance(c["steps"], c["cfl"], solver=c["solver"])
        else:
            for _ in range(c["steps"]):
                p.step(p.cfl_dt(c["cfl"]), c["solver"])
        out = {"state": state["state"] if "state" in state else p.get_state()}
        if c["diag"]:
            out["kinetic"] = p.kinetic_energy()
            out["spectrum"] = p.kinetic_spectrum()[1]
        return out
    if c["kind"] == "tubes":
        b = state["batch"]
        for i, W in enumerate(state["W"]):
            b.set_state(i, W)
        b.run_to(c["t_end"], 0.4, c["solver"])
        got = [b.get_state(i) for i in range(c["count"])]
        return np.concatenate(got, axis=1)
    if c["kind"] == "levels":
        f = state["fmr"]
        dts = [f.step(c["cfl"], solver=c["solver"]) for _ in range(c["steps"])]
        return {"dt": np.array(dts), "levels": [f.get_state(l) for l in range(f.nlev)]}
    x, t = state["patch"].make_samples()
    for i in range(c["steps"]):
        state["trainer"].step(x, t, state["idx"][i], 1e-3)
    return {"x": x, "t": t, "params": state["trainer"].params()}


# ------------------------------------------------------------------ work ----

# operations per cell and step (both stages): recovery, slopes, face states, Riemann solves, update, CFL rate
_OPS = {1: 330, 2: 640, 3: 1000}


def _steps_of_tubes(c):
    # cells times steps of an average tube: dt = 0.4 dx / (|v| + c), |v| + c about 3 in these states
    n = 0.5 * (c["nmin"] + c["nmax"])
    return c["count"] * n, 3.0 * n * c["t_end"] / 0.4


def work(case):
    c = case
    if c["kind"] == "patch":
        nd = 3 if c["nz"] > 1 else (2 if c["ny"] > 1 else 1)
        cells, es = c["nx"] * c["ny"] * c["nz"], c["bits"] // 8
        # a step reads the state and writes the next one; the network is 2368 operations for each slope of each stage
        flops = cells * (_OPS[nd] + (2 * 2368 * nd * (nd + 2) if c["learned"] else 0))
        b = c["steps"] * cells * 2 * (nd + 2) * es
        f = c["steps"] * flops
        if c["diag"]:  # the state once more for each diagnostic, and a complex FP64 transform in two passes
            b += cells * (2 * 12 + 3 * 16)
            f += cells * 5 * math.log2(cells)
        return {"bytes": b, "flops": f}
    if c["kind"] == "tubes":  # each tube fits a compute unit: its state is read and written once
        cells, steps = _steps_of_tubes(c)
        return {"bytes": cells * 24, "flops": cells * steps * _OPS[1]}
    if c["kind"] == "levels":
        nd, cells = c["ndim"], c["n0"] ** c["ndim"]
        n = sum(2 ** l for l in range(c["nlev"])) * cells
        return {"bytes": c["steps"] * n * 2 * (nd + 2) * c["bits"] // 8, "flops": c["steps"] * n * _OPS[nd]}
    ns = (c["n"] // 4) ** 2 * 8
    return {"bytes": c["n"] ** 2 * 16 + ns * 20 + c["steps"] * c["batch"] * 24, "flops": c["steps"] * c["batch"] * 3 * 2368}


def tolerance(case):
    """About four times what run() was measured to differ from exact() by, over the listed and two dozen drawn cases."""
    c = case
    if c["kind"] == "patch":  # measured up to 2.6e-7 and 2.4e-6 (FP32), 2.5e-16 and 2.4e-15 (FP64)
        if c["bits"] == 64:
            return {"rel": 1e-15, "max": 1e-14}
        if c["solver"] == SWITCH:  # a face whose pressure jump rounds to the other side of the threshold: 1.4e-6, 8e-3
            return {"rel": 6e-6, "max": 3e-2}
        return {"rel": 1e-6, "max": 1e-5}
    if c["kind"] == "tubes":  # thousands of steps: 1.1e-5 and 2.4e-4
        return {"rel": 5e-5, "max": 1e-3}
    if c["kind"] == "levels":  # up to 640 steps of the deepest level: 3.0e-6 and 3.8e-5 (FP32), 3.6e-15 (FP64)
        return {"rel": 1.5e-14, "max": 2e-13} if c["bits"] == 64 else {"rel": 1.2e-5, "max": 2e-4}
    return {"rel": 3e-4, "max": 3e-2}  # a sample divides small differences by their largest: 2.4e-5 and 8e-3


# ----------------------------------------------------- the method in 64 bits ----


def _prim(U, nd, gamma):
    W = U.clone()
    W[1:nd + 1] = U[1:nd + 1] / U[0]
    W[nd + 1] = (gamma - 1) * (U[nd + 1] - 0.5 * (U[1:nd + 1] * W[1:nd + 1]).sum(0))
    return W


def _ghosts(W, q, bc, normal=None):
    """W with two ghost cells at each end of dimension q; normal: the index of the component that a mirror negates."""
    ax = W.dim() - 1 - q
    n = W.shape[ax]
    lo = {PER: [n - 2, n - 1], OUT: [0, 0], REF: [1, 0]}[bc[q][0]]
    hi = {PER: [0, 1], OUT: [n - 1, n - 1], REF: [n - 1, n - 2]}[bc[q][1]]
    ends = []
    for idx, kind in ((lo, bc[q][0]), (hi, bc[q][1])):
        e = W.index_select(ax, torch.tensor(idx, device=W.device))
        if kind == REF and normal is not None:
            e[normal] = -e[normal]
        ends.append(e)
    return torch.cat([ends[0], W, ends[1]], ax)


def _at(A, q, lo, n):
    return A.narrow(A.dim() - 1 - q, lo, n)


def _minmod(a, b, theta):
    s = torch.minimum(torch.minimum(theta * a.abs(), theta * b.abs()), 0.5 * (a + b).abs())
    return torch.where(a * b > 0, torch.sign(a) * s, 0.0)


def _bf(x):
    return x.to(torch.float32).to(torch.bfloat16).to(torch.float64)


def _net(params, x):
    """The network on x (..., 4): bf16 operands, everything else in 64 bits; also what its backward pass needs."""
    w1, b1 = _bf(params[:128]).view(32, 4), params[128:160]
    w2, b2 = _bf(params[160:1184]).view(32, 32), params[1184:1216]
    w3, b3 = _bf(params[1216:1248]), params[1248]
    xb = _bf(x)
    z1 = xb @ w1.t() + b1
    h1 = _bf(z1.clamp(min=0))
    z2 = h1 @ w2.t() + b2
    h2 = _bf(z2.clamp(min=0))
    return h2 @ w3 + b3, (xb, z1, h1, z2, h2, w2, w3)


def _learned_slopes(Wg, q, bc, params):
    """Slopes of the cells -1 .. n from the 5-cell stencils (ghost cells take those of their source)."""
    n = Wg.shape[Wg.dim() - 1 - q] - 4
    w = [_at(Wg, q, k, n) for k in range(5)]
    d = torch.stack([w[k + 1] - w[k] for k in range(4)], -1)
    s = d.abs().amax(-1) + 1e-12 * (w[2].abs() + 1e-30)
    x, y = d / s[..., None], torch.empty_like(s)
    for part, to in zip(x.reshape(-1, 4).split(1 << 20), y.view(-1).split(1 << 20)):
        to.copy_(_net(params, part)[0])
    dm, dp = d[..., 1], d[..., 2]
    sg = torch.sign(dp)
    sig = sg * torch.minimum((sg * s * y).clamp(min=0), 2 * torch.minimum(dm.abs(), dp.abs()))
    sig = torch.where(dm * dp > 0, sig, 0.0)
    ends = []
    for i, src, kind in ((0, 0, bc[q][0]), (1, n - 1, bc[q][1])):
        e = _at(sig, q, src if kind != PER else n - 1 - src, 1).clone()
        if kind == OUT:
            e.zero_()
        elif kind == REF:
            e = -e
            e[1 + q] = -e[1 + q]
        ends.append(e)
    return torch.cat([ends[0], sig, ends[1]], sig.dim() - 1 - q)


def _flux(wl_, wr, q, nd, gamma, solver):
    """The face flux normal to q; solver: HLL or HLLC."""
    def side(w):
        v, p, r = w[1 + q], w[nd + 1], w[0]
        U = _conserved(w, nd, gamma)
        F = U * v
        F[1 + q] += p
        F[nd + 1] += p * v
        return r, v, p, torch.sqrt(gamma * p / r), U, F
    rl, vl, pl, cl, Ul, Fl = side(wl_)
    rr, vr, pr, cr, Ur, Fr = side(wr)
    zero = torch.zeros_like(rl)
    ap = torch.maximum(zero, torch.maximum(vl + cl, vr + cr))
    am = torch.maximum(zero, torch.maximum(cl - vl, cr - vr))
    if solver == HLL:
        return (ap * Fl + am * Fr - ap * am * (Ur - Ul)) / (ap + am)
    A, B = rr * (ap - vr), rl * (am + vl)
    sm = (A * vr + B * vl + pl - pr) / (A + B)

    def star(r, v, p, U, F, w, s):
        rs = r * (s - v) / (s - sm)
        ps = p + r * (s - v) * (sm - v)
        Us = U.clone()
        Us[0] = rs
        for k in range(nd):
            Us[1 + k] = rs * (sm if k == q else w[1 + k])
        Us[nd + 1] = ((s - v) * U[nd + 1] - p * v + ps * sm) / (s - sm)
        return F + s * (Us - U)
    F = torch.where(sm >= 0, star(rl, vl, pl, Ul, Fl, wl_, -am), star(rr, vr, pr, Ur, Fr, wr, ap))
    return torch.where(am == 0, Fl, torch.where(ap == 0, Fr, F))


def _face_fluxes(Wg, q, nd, gamma, theta, solver, slopes=None, hll=None):
    """Fluxes through the n + 1 faces along q of the cells inside Wg's two ghost layers."""
    m = Wg.shape[Wg.dim() - 1 - q]
    if slopes is None:
        d = _at(Wg, q, 1, m - 1) - _at(Wg, q, 0, m - 1)
        slopes = _minmod(_at(d, q, 0, m - 2), _at(d, q, 1, m - 2), theta)
    w = _at(Wg, q, 1, m - 2)
    left = _at(w, q, 0, m - 3) + 0.5 * _at(slopes, q, 0, m - 3)
    right = _at(w, q, 1, m - 3) - 0.5 * _at(slopes, q, 1, m - 3)
    if hll is None:
        return _flux(left, right, q, nd, gamma, solver)
    return torch.where(hll, _flux(left, right, q, nd, gamma, HLL), _flux(left, right, q, nd, gamma, HLLC))


def _shocks(W, nd, bc):
    """Per dimension q: cells in a shock moving along q."""
    bits = []
    for q in range(nd):
        g = _ghosts(W, q, bc, 1 + q)
        n = W.shape[W.dim() - 1 - q]
        a, b = _at(g, q, 1, n), _at(g, q, 3, n)
        pa, pb = a[nd + 1], b[nd + 1]
        bits.append(((pb - pa).abs() > 0.5 * torch.minimum(pa, pb)) & (b[1 + q] < a[1 + q]))
    return bits


def _rate(U, nd, gamma, dq):
    W = _prim(U, nd, gamma)
    c = torch.sqrt(gamma * W[nd + 1] / W[0])
    return max(float(((W[1 + q].abs() + c) / dq[q]).max()) for q in range(nd))


def _rhs(U, pr, dq, solver, params=None):
    nd, gamma = pr.ndim, pr.gamma
    W = _prim(U, nd, gamma)
    L = torch.zeros_like(U)
    bits = _shocks(W, nd, pr.bc) if solver == SWITCH and nd > 1 else None
    for q in range(nd):
        n = U.shape[U.dim() - 1 - q]
        g = _ghosts(W, q, pr.bc, 1 + q)
        hll = None
        if bits is not None:
            f = torch.zeros_like(bits[0])
            for r in range(nd):
                if r != q:
                    f |= bits[r]
            f = _at(_ghosts(f[None], q, pr.bc), q, 1, n + 2)[0]
            ax = f.dim() - 1 - q
            hll = f.narrow(ax, 0, n + 1) | f.narrow(ax, 1, n + 1)
        F = _face_fluxes(g, q, nd, gamma, pr.theta, min(solver, HLLC),
                         None if params is None else _learned_slopes(g, q, pr.bc, params), hll)
        L -= (_at(F, q, 1, n) - _at(F, q, 0, n)) / dq[q]
    for q in range(nd):
        if pr.accel[q]:
            L[1 + q] += U[0] * pr.accel[q]
            L[nd + 1] += U[1 + q] * pr.accel[q]
    return L


def _patch_exact(c, pr, U, steps, params=None):
    dq = [(pr.hi[q] - pr.lo[q]) / pr.n[q] for q in range(pr.ndim)]
    for _ in range(steps):
        dt = c["cfl"] / _rate(U, pr.ndim, pr.gamma, dq)
        U1 = U + dt * _rhs(U, pr, dq, c["solver"], params)
        U = 0.5 * (U + U1 + dt * _rhs(U1, pr, dq, c["solver"], params))
    return U


def _spectrum(U, box):
    n = U.shape[-1]
    k = torch.fft.fftfreq(n, 1.0 / n, device=U.device, dtype=torch.float64)
    shell = torch.floor(torch.sqrt(k[:, None] ** 2 + k[None, :] ** 2) + 0.5).long().reshape(-1)
    power = sum(torch.fft.fft2(U[1 + q] / torch.sqrt(U[0])).abs() ** 2 for q in range(2)).reshape(-1)
    dk = 2 * math.pi / box
    e = torch.zeros(int(shell.max()) + 1, dtype=torch.float64, device=U.device).index_add_(0, shell, power)
    return e * (0.5 * box * box / float(n) ** 4 / dk)


def _tubes_exact(c, seed):
    dev, gamma, theta = _dev(), 1.4, 2.0
    problems = _tube_problems(c, seed)
    n = torch.tensor([p.n[0] for p in problems], device=dev)
    m = int(n.max())
    W = torch.ones((3, len(problems), m), dtype=torch.float64, device=dev)
    for i, p in enumerate(problems):
        W[:, i, :p.n[0]] = torch.tensor(p.W, device=dev).float().double()
    inside = torch.arange(m, device=dev)[None, :] < n[:, None]
    # beyond its end a tube repeats its last cell: the outflow ghosts of every tube, whatever its length
    last = torch.minimum(torch.arange(m, device=dev)[None, :].expand(len(problems), m), n[:, None] - 1)
    tail = lambda A: torch.gather(A, 2, last[None].expand(3, -1, -1))  # noqa: E731
    bc = ((OUT, OUT), (0, 0), (0, 0))
    U = _conserved(W, 1, gamma)
    dx = 1.0 / n.double()
    t = torch.zeros(len(problems), dtype=torch.float64, device=dev)
    for k in range(400000):
        if k % 64 == 0 and bool((t >= c["t_end"]).all()):
            break
        Wn = _prim(U, 1, gamma)
        rate = torch.where(inside, Wn[1].abs() + torch.sqrt(gamma * Wn[2] / Wn[0]), 0.0).amax(1) / dx
        dt = torch.minimum(0.4 / rate, c["t_end"] - t).clamp(min=0)
        cdt = (dt / dx)[None, :, None]
        U1, Us = None, U
        for stage in range(2):
            F = _face_fluxes(_ghosts(tail(_prim(Us, 1, gamma)), 0, bc, 1), 0, 1, gamma, theta, c["solver"])
            D = Us - cdt * (F[..., 1:] - F[..., :-1])
            U1, Us = Us, D
        U = 0.5 * (U + Us)
        t = t + dt
    out = _prim(U, 1, gamma).cpu().numpy()
    return np.concatenate([out[:, i, :p.n[0]] for i, p in enumerate(problems)], axis=1)


class _NestedLevels:
    """Subcycled nested levels with flux replacement; refined levels carry two exterior cells per side."""

    def __init__(self, lv, solver, cfl, bits):
        dev = _dev()
        self.lv, self.nd, self.gamma, self.theta, self.solver, self.cfl = lv, lv.base.ndim, lv.base.gamma, lv.base.theta, solver, cfl
        self.geo = [lv.level_geometry(l) for l in range(lv.nlev)]
        self.dq = [[(hi[q] - lo[q]) / n[q] for q in range(self.nd)] for n, lo, hi in self.geo]
        self.U = []
        for l in range(lv.nlev):
            W = torch.tensor(lv.W[l], device=dev)
            U = _conserved(W if bits == 64 else W.float().double(), self.nd, self.gamma)
            if l:
                shape = [U.shape[0]] + [s + 4 for s in U.shape[1:]]
                P = torch.ones(shape, dtype=torch.float64, device=dev)
                self.inner(P, l).copy_(U)
                U = P
            self.U.append(U)

    def inner(self, A, l):
        if l:
            for q in range(self.nd):
                A = _at(A, q, 2, A.shape[A.dim() - 1 - q] - 4)
        return A

    def along(self, W, l, q):
        """Cells of level l with two more at each end of dimension q."""
        if l == 0:
            return _ghosts(W, q, self.lv.base.bc, 1 + q)
        for r in range(self.nd):
            if r != q:
                W = _at(W, r, 2, W.shape[W.dim() - 1 - r] - 4)
        return W

    def prolong(self, l, parent):
        """Level l's exterior from its parent's cells (an array of that level's own layout)."""
        lo, n = self.lv.boxes[l - 1]
        off = 2 if l > 1 else 0
        W = _prim(parent, self.nd, self.gamma)
        for q in range(self.nd):  # the box and two cells around it
            W = _at(W, q, lo[q] + off - 2, n[q] + 4)
        core = W
        for q in range(self.nd):
            core = _at(core, q, 1, n[q] + 2)
        fine = core
        for q in range(self.nd):
            fine = fine.repeat_interleave(2, fine.dim() - 1 - q)
        for q in range(self.nd):
            s = W
            for r in range(self.nd):
                if r != q:
                    s = _at(s, r, 1, n[r] + 2)
            d = _at(s, q, 1, n[q] + 3) - _at(s, q, 0, n[q] + 3)
            g = 0.25 * _minmod(_at(d, q, 0, n[q] + 2), _at(d, q, 1, n[q] + 2), 1.0)
            for r in range(self.nd):
                g = g.repeat_interleave(2, g.dim() - 1 - r)
            sign = torch.ones(2 * (n[q] + 2), dtype=torch.float64, device=g.device)
            sign[::2] = -1
            fine = fine + g * sign.reshape([-1 if r == q else 1 for r in reversed(range(self.nd))])
        keep = self.inner(self.U[l], l).clone()
        self.U[l] = _conserved(fine, self.nd, self.gamma)
        self.inner(self.U[l], l).copy_(keep)

    def fluxes(self, U, l):
        W = _prim(U, self.nd, self.gamma)
        return [_face_fluxes(self.along(W, l, q), q, self.nd, self.gamma, self.theta, self.solver) for q in range(self.nd)]

    def div(self, F, l):
        return -sum((_at(f, q, 1, f.shape[f.dim() - 1 - q] - 1) - _at(f, q, 0, f.shape[f.dim() - 1 - q] - 1)) / self.dq[l][q]
                    for q, f in enumerate(F))

    def step(self, l=0, parent=None):
        """One step of level l and everything finer; returns its size and the fluxes through its own edge."""
        if l:
            self.prolong(l, parent)
        nd, last = self.nd, l == self.lv.nlev - 1
        child = None
        F0 = self.fluxes(self.U[l], l)
        if last:
            dt = self.cfl / _rate(self.inner(self.U[l], l), nd, self.gamma, self.dq[l])
        else:
            dt1, e1 = self.step(l + 1, self.U[l])
            half = self.U[l].clone()
            self.inner(half, l).add_(dt1 * self.div(F0, l))
            dt2, e2 = self.step(l + 1, half)
            dt = dt1 + dt2
            child = [[a + b for a, b in zip(x, y)] for x, y in zip(e1, e2)]
        U1 = self.U[l].clone()
        self.inner(U1, l).add_(dt * self.div(F0, l))
        F1 = self.fluxes(U1, l)
        F = [0.5 * dt * (a + b) for a, b in zip(F0, F1)]
        I = self.inner(self.U[l], l)
        I.add_(self.div(F, l))
        if child:
            lo, n = self.lv.boxes[l]
            for q in range(nd):
                for side in range(2):
                    face = lo[q] + side * n[q]
                    c, cell = _at(F[q], q, face, 1), _at(I, q, face if side else face - 1, 1)
                    for r in range(nd):
                        if r != q:
                            c, cell = _at(c, r, lo[r], n[r]), _at(cell, r, lo[r], n[r])
                    f = child[q][side]
                    for r in range(nd):
                        if r != q:
                            f = 0.5 * (f.index_select(f.dim() - 1 - r, torch.arange(0, 2 * n[r], 2, device=f.device))
                                       + f.index_select(f.dim() - 1 - r, torch.arange(1, 2 * n[r], 2, device=f.device)))
                    cell.add_((f - c) * ((1 if side else -1) / self.dq[l][q]))
            fine, under = self.inner(self.U[l + 1], l + 1), I
            for q in range(nd):
                m = fine.shape[fine.dim() - 1 - q]
                fine = 0.5 * (fine.index_select(fine.dim() - 1 - q, torch.arange(0, m, 2, device=fine.device))
                              + fine.index_select(fine.dim() - 1 - q, torch.arange(1, m, 2, device=fine.device)))
                under = _at(under, q, lo[q], n[q])
            under.copy_(fine)
        edge = [[_at(f, q, 0, 1), _at(f, q, f.shape[f.dim() - 1 - q] - 1, 1)] for q, f in enumerate(F)]
        return dt, edge


def _train_exact(c, seed):
    dev = _dev()
    pr = _problem(_fine(c), seed)
    U = _conserved(pr.W.float().double(), 2, pr.gamma)
    m = c["n"] // 4
    blocks = U.view(4, m, 4, m, 4)
    Wc = _prim(blocks.mean((2, 4)), 2, pr.gamma)
    x, t = [], []
    for q in range(2):
        g = _ghosts(Wc, q, ((PER, PER), (PER, PER)))
        d = [_at(g, q, k + 1, m) - _at(g, q, k, m) for k in range(4)]
        s = torch.stack(d).abs().amax(0) + 1e-12 * (Wc.abs() + 1e-30)
        sub = [_prim((blocks.mean(2) if q == 0 else blocks.mean(4)).select(3 if q == 0 else 2, k), 2, pr.gamma) for k in range(4)]
        sg = 0.4 * (3 * (sub[3] - sub[0]) + sub[2] - sub[1])
        sn = torch.sign(d[2])
        sg = torch.where(d[1] * d[2] > 0, sn * torch.minimum((sn * sg).clamp(min=0), 2 * torch.minimum(d[1].abs(), d[2].abs())), 0.0)
        x.append(torch.stack([a / s for a in d], -1).reshape(-1, 4))
        t.append((sg / s).reshape(-1))
    x, t = torch.cat(x), torch.cat(t)
    rng = np.random.default_rng(seed)
    idx = torch.tensor(rng.integers(0, t.numel(), size=(c["steps"], c["batch"])), device=dev)
    p = torch.tensor(limiter.init_params(seed), device=dev).double()
    m1, m2 = torch.zeros_like(p), torch.zeros_like(p)
    for k in range(c["steps"]):
        y, (xb, z1, h1, z2, h2, w2, w3) = _net(p, x[idx[k]])
        dy = 2 * (y - t[idx[k]]) / c["batch"]
        dz2 = torch.where(z2 > 0, dy[:, None] * w3, 0.0)
        dz2b = _bf(dz2)
        dz1 = torch.where(z1 > 0, dz2b @ w2, 0.0)
        g = torch.cat([(_bf(dz1).t() @ xb).reshape(-1), dz1.sum(0), (dz2b.t() @ h1).reshape(-1), dz2.sum(0), dy @ h2, dy.sum()[None]])
        m1, m2 = 0.9 * m1 + 0.1 * g, 0.999 * m2 + 0.001 * g * g
        p = p - 1e-3 * (m1 / (1 - 0.9 ** (k + 1))) / (torch.sqrt(m2 / (1 - 0.999 ** (k + 1))) + 1e-8)
    return {"x": x, "t": t, "params": p}


def exact(case, seed):
    """What run() returns on the first call after prepare(case, seed), in 64 bits."""
    c = case
    if c["kind"] == "patch":
        pr = _problem(c, seed)
        U = _conserved(pr.W, pr.ndim, pr.gamma)
        if c["bits"] == 32:
            U = U.float().double()
        params = torch.tensor(limiter.trained_params(), device=U.device).double() if c["learned"] else None
        U = _patch_exact(c, pr, U, c["steps"], params)
        out = {"state": U.reshape(pr.ndim + 2, -1)}
        if c["diag"]:
            dv = 1.0 / pr.n[0] / pr.n[1]
            out["kinetic"] = np.array([float((U[1 + q] ** 2 / (2 * U[0])).sum()) * dv if q < pr.ndim else 0.0 for q in range(3)])
            out["spectrum"] = _spectrum(U, 1.0)
        return out
    if c["kind"] == "tubes":
        steps = 9 * c["nmax"] * c["t_end"] / 0.4  # of the longest tube
        if steps * (1.5e-3 + c["count"] * c["nmax"] * 1.5e-9) > 18:
            return None
        return _tubes_exact(c, seed)
    if c["kind"] == "levels":
        lv = _levels(c, seed)
        if 2 ** lv.nlev * c["steps"] * 0.03 > 60:
            return None
        m = _NestedLevels(lv, c["solver"], c["cfl"], c["bits"])
        dts = [m.step()[0] for _ in range(c["steps"])]
        return {"dt": np.array(dts), "levels": [m.inner(U, l).reshape(m.nd + 2, -1) for l, U in enumerate(m.U)]}
    return _train_exact(c, seed)
