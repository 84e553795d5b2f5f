"""The work that users of the library have it do, as cases that can be timed.

A case is a whole call as a program makes it: initial data handed over as host
arrays, a number of time steps, the moments (and for small grids the
distribution) read back; or a stretch of closure training.  The solver, its
device workspace and the network stand before the call, as a program keeps
them over many calls; every pass starts from the same initial data.

``exact`` states the scheme again in plain FP64 torch: eager correction,
literal limiter and WENO weights, every value stored in the Eulerian frame.
"""
import math

import numpy as np
import torch

from paper_1212_0204_amd import Batch, Solver
from paper_1212_0204_amd.mlp import ClosureNet

DEV = "cuda" if torch.cuda.is_available() else "cpu"


def _grid(name, n, nv, dv, tau, steps, init, length=1.0, bc="periodic", precision=0, scheme=0,
          cfl=0.0, strang=False, read_f=False):
    n = tuple(n) + (1,) * (3 - len(n))
    c = {"kind": "grid", "d": sum(1 for m in n if m > 1), "nx": n[0], "ny": n[1], "nz": n[2],
         "length": length, "nv": nv, "dv": dv, "tau": tau, "steps": steps, "init": init, "bc": bc,
         "precision": precision, "scheme": scheme, "cfl": cfl, "strang": strang, "read_f": read_f}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the 1D Sod tube of the paper's section 5 as a whole run: every step
        # is a chain of small dependent pieces of work
        _grid("sod1d_200x64_fp64", (200,), 64, 0.25, 1e-2, 100, "sod", bc="outflow", read_f=True),
        # a finer tube of odd length in the precision form, on many blocks
        _grid("sod1d_3001x48_fp32", (3001,), 48, 0.25, 1e-3, 40, "sod", bc="outflow", precision=1),
        # a small ragged 2D box, as parameter studies run them
        _grid("gas2d_70x37x16sq_fp64", (70, 37), 16, 0.5, 1e-3, 40, "gas", read_f=True),
        # the 2D gas of the benchmark
        _grid("gas2d_256sq_x_32sq_fp64", (256, 256), 32, 0.5, 1e-3, 40, "gas"),
        # the 2D disk in the precision form
        _grid("disk2d_512sq_x_32sq_fp32", (512, 512), 32, 0.5, 1e-4, 20, "disk", length=2.0,
              precision=1),
        # the WENO Euler solve on the 2D gas
        _grid("weno2d_256sq_x_32sq_fp64", (256, 256), 32, 0.5, 1e-3, 20, "gas", scheme=3),
        # a free time step at kinetic CFL 1: many short steps, one sub-step each
        _grid("offlattice2d_256sq_fp64", (256, 256), 32, 0.5, 1e-3, 40, "gas", cfl=1.0),
        # the 3D gas of the benchmark in the precision form: the largest grid
        _grid("gas3d_64cube_x_24cube_fp32", (64, 64, 64), 24, 0.5, 1e-3, 12, "gas", precision=1),
        # a ragged 3D box in FP64 with an outflow axis
        _grid("gas3d_50x36x28x16cube_fp64", (50, 36, 28), 16, 0.75, 2e-3, 8, "gas", bc="mixed"),
        # a study of many independent shock tubes
        {"name": "batch_512_tubes_fp32", "kind": "batch", "tubes": 512, "nx_lo": 200, "nx_hi": 4000,
         "steps": 128},
        # closure steps on the disk: nearly every cell in equilibrium
        {"name": "closure2d_512sq_x_32sq", "kind": "closure", "n": 512, "length": 2.0, "nv": 32,
         "dv": 0.5, "tau": 1e-4, "sigma": 0.01, "threshold": 1e-3, "steps": 20},
        # minibatch training of the closure network
        {"name": "train_4096", "kind": "train", "rows": 200000, "batch": 4096, "steps": 10},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges."""
    what = rng.choice(["1d", "1d", "2d", "2d", "2d", "2d_small", "weno", "free", "3d", "3d", "batch",
                       "closure", "train"])
    rel = 10.0 ** rng.uniform(-2.0, -0.4)  # tau / dt: steps near equilibrium stay physical
    prec = rng.choice([0, 0, 1])
    if what == "1d":
        nx = _log_int(rng, 100, 4000)
        return _grid(None, (nx,), rng.choice([32, 40, 48, 64, 65]), 0.25, rel / (0.25 * nx), rng.randint(20, 80),
                     rng.choice(["sod", "gas"]), bc=rng.choice(["outflow", "outflow", "periodic"]),
                     precision=prec, scheme=rng.choice([0, 0, 0, 1]))
    if what == "2d_small":
        n = (rng.randint(20, 120), rng.randint(20, 120))
        return _grid(None, n, rng.choice([16, 20, 24]), 0.5, rel / (0.5 * n[0]), rng.randint(20, 50), "gas",
                     bc=rng.choice(["periodic", "outflow", "mixed"]), precision=prec,
                     scheme=rng.choice([0, 0, 0, 1, 2, 3]), read_f=True)
    if what == "3d":
        n = (rng.randint(24, 66), rng.randint(20, 50), rng.randint(20, 50))
        return _grid(None, n, rng.choice([12, 16, 20]), 0.75, rel / (0.75 * n[0]), rng.randint(6, 14), "gas",
                     bc=rng.choice(["periodic", "mixed", "outflow"]), precision=prec)
    if what == "batch":
        return {"kind": "batch", "tubes": _log_int(rng, 32, 512), "nx_lo": rng.randint(150, 400),
                "nx_hi": rng.randint(1500, 4000), "steps": 16 * rng.randint(3, 8)}
    if what == "closure":
        n = rng.randint(160, 512)
        return {"kind": "closure", "n": n, "length": n / 256, "nv": rng.choice([16, 24, 32]),
                "dv": 0.5, "tau": 10.0 ** rng.uniform(-4.0, -3.6), "sigma": 0.01, "threshold": 1e-3,
                "steps": rng.randint(8, 20)}
    if what == "train":
        return {"kind": "train", "rows": _log_int(rng, 20000, 400000),
                "batch": _log_int(rng, 512, 8192), "steps": rng.randint(6, 12)}
    n = (rng.randint(150, 400), rng.randint(150, 400))
    tau = rel / (0.5 * n[0])
    cfl, scheme = 0.0, rng.choice([0, 0, 0, 0, 1, 2])
    if what == "weno":
        scheme, prec = 3, 0
    if what == "free":
        cfl, scheme = rng.uniform(0.8, 4.0), 0
    return _grid(None, n, rng.choice([16, 20, 24, 32]), 0.5, tau, rng.randint(16, 40), "gas",
                 bc=rng.choice(["periodic", "periodic", "outflow", "mixed"]), precision=prec,
                 scheme=scheme, cfl=cfl, strang=rng.random() < 0.2)


# ------------------------------------------------------------------ inputs
def _cells(c):
    return [c["nx"], c["ny"], c["nz"]][:c["d"]]


def _bc(c):
    d = c["d"]
    return {"periodic": (0,) * d, "outflow": (1,) * d, "mixed": (1,) + (0,) * (d - 1)}[c["bc"]]


def _dt(c):
    """time step of a free-velocity case at its kinetic CFL number, else None"""
    if not c["cfl"]:
        return None
    dx = c["length"] / c["nx"]
    return min(1.0, 2.0 * c["cfl"] / c["nv"]) * dx / c["dv"]


def _wave(rng, n, modes):
    """a smooth periodic field of a dozen random Fourier modes, |g| <= 1"""
    d = len(n)
    x = np.meshgrid(*[(np.arange(m) + 0.5) / m for m in reversed(n)], indexing="ij")
    g = np.zeros(tuple(reversed(n)))
    norm = 0.0
    for _ in range(12):
        m = rng.integers(-modes, modes + 1, d)
        if not m.any():
            m[0] = 1
        amp = rng.uniform(0.3, 1.0) / np.linalg.norm(m)
        g += amp * np.cos(2 * np.pi * sum(mi * xi for mi, xi in zip(m, x)) + rng.uniform(0, 2 * np.pi))
        norm += amp
    return (g * (2.0 / norm)).clip(-1.0, 1.0).reshape(-1)


def _disk(rng, n, length):
    x = (np.arange(n) + 0.5) * (length / n)
    cx, cy = length * rng.uniform(0.45, 0.55, 2)
    r = 0.1 * length * rng.uniform(0.9, 1.1)
    ins = ((x[None, :] - cx) ** 2 + (x[:, None] - cy) ** 2 <= r * r).reshape(-1)
    rho = np.where(ins, 1.0, 0.125)
    return rho, np.zeros((2, n * n)), np.where(ins, 1.0, 0.1) / rho


def _fields(c, seed):
    """(rho, u, theta) host arrays of a grid case"""
    rng = np.random.default_rng(seed)
    n, d = _cells(c), c["d"]
    if c["init"] == "sod":
        left = (np.arange(n[0]) + 0.5) / n[0] < rng.uniform(0.4, 0.6)
        rho = np.where(left, 1.0, rng.uniform(0.12, 0.2))
        p = np.where(left, 1.0, rng.uniform(0.1, 0.16))
        return rho, np.zeros((1, n[0])), p / rho
    if c["init"] == "disk":
        return _disk(rng, n[0], c["length"])
    modes = {1: 6, 2: 8, 3: 4}[d]
    rho = 1.0 + 0.15 * _wave(rng, n, modes)
    u = np.stack([0.05 * _wave(rng, n, modes) for _ in range(d)])
    theta = 1.0 + 0.1 * _wave(rng, n, modes)
    return rho, u, theta


def _tubes(c, seed):
    """(n_cells, dx, n_vel, dv, tau) of each tube and the concatenated fields;
    dv is the smallest power of two whose grid spans six thermal widths"""
    # the study's tubes come with the case, their states with the seed
    shape = np.random.default_rng(4 + c["tubes"])
    rng = np.random.default_rng(seed)
    tubes, fields = [], []
    for _ in range(c["tubes"]):
        nx = int(shape.integers(c["nx_lo"], c["nx_hi"] + 1))
        nv = int(shape.choice((32, 64, 128)))
        rel = float(10.0 ** shape.uniform(-2.0, -0.4))  # tau / dt: steps that stay physical
        rl, pl, rr, pr = rng.uniform(0.7, 1.0, 4)
        dv = 2.0 ** math.ceil(math.log2(6.0 * math.sqrt(2.0) / (nv / 2)))
        left = (np.arange(nx) + 0.5) / nx < 0.5
        rho = np.where(left, rl, rr)
        tubes.append((nx, 1.0 / nx, nv, dv, rel / (nx * dv)))
        fields.append((rho, np.zeros(nx), np.where(left, pl, pr) / rho))
    return tubes, [np.concatenate(a) for a in zip(*fields)]


def _samples(c, seed):
    """stencil inputs and targets of the size that closure snapshots have"""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    x = 0.1 * torch.randn(c["rows"], 37, device=DEV, generator=g)
    x[:, 36] = torch.rand(c["rows"], device=DEV, generator=g) * 1.5 - 1.4
    w = torch.randn(37, 4, device=DEV, generator=g)
    t = torch.sin(2.0 * x @ w) + 0.3 * x[:, 36:37] + 0.05 * torch.randn(
        c["rows"], 4, device=DEV, generator=g)
    return x.contiguous(), t.contiguous()


# -------------------------------------------------------------- preparation
def prepare(case, seed):
    c = case
    if c["kind"] == "grid":
        s = Solver(c["d"], _cells(c), c["length"] / c["nx"], c["nv"], c["dv"], bc=_bc(c),
                   precision=c["precision"], scheme=c["scheme"], tau=c["tau"], dt=_dt(c),
                   strang=c["strang"])
        return {"case": c, "solver": s, "fields": _fields(c, seed)}
    if c["kind"] == "batch":
        tubes, fields = _tubes(c, seed)
        return {"case": c, "solver": Batch(tubes), "fields": fields}
    if c["kind"] == "closure":
        s = Solver(2, (c["n"], c["n"]), c["length"] / c["n"], c["nv"], c["dv"], precision=1,
                   tau=c["tau"])
        net = ClosureNet(seed=seed % 1000, sigma=c["sigma"])
        fields = _disk(np.random.default_rng(seed), c["n"], c["length"])
        return {"case": c, "solver": s, "net": net, "fields": fields}
    x, t = _samples(c, seed)
    return {"case": c, "net": ClosureNet(seed=seed % 1000), "x": x, "t": t, "seed": seed}


def run(state):
    c = state["case"]
    if c["kind"] == "train":
        net = state["net"]
        net.train(state["x"], state["t"], c["steps"], batch=c["batch"], seed=state["seed"])
        return {"params": net.params, "m": net.m, "v": net.v, "grad": net.grad, "loss": net.loss}
    s = state["solver"]
    s.set_state_macro(*state["fields"])
    if c["kind"] == "closure":
        s.closure_enable(state["net"], threshold=c["threshold"])
    s.step(c["steps"])
    if c["kind"] == "batch":
        # the per-tube arrays are views of one array, returned as that
        return {"U": s.read_moments()[0].base, "flags": s.tube_flags()}
    out = {"U": s.read_moments()}
    if c["kind"] == "grid" and c["read_f"]:
        out["f"] = s.read_f()
    return out


def work(case):
    c = case
    if c["kind"] == "train":
        # forward, gradients of the inputs and of the weights
        n = 11012
        return {"bytes": c["steps"] * (c["batch"] * (41 * 4 + 4) + 8 * 4 * n),
                "flops": c["steps"] * 6 * c["batch"] * n}
    if c["kind"] == "closure":
        nc = c["n"] ** 2
        # no pieces in closure cells: the first step writes and reads them once
        return {"bytes": c["steps"] * nc * 64 + 2 * 4 * nc * c["nv"] ** 2 + 64 * nc,
                "flops": c["steps"] * nc * (2 * 11012 + 20 * c["nv"] ** 2)}
    if c["kind"] == "batch":
        tubes, _ = _tubes(c, 0)
        cv = sum(t[0] * t[2] for t in tubes)
        nc = sum(t[0] for t in tubes)
        return {"bytes": c["steps"] * (8 * cv + 48 * nc) + 4 * cv + 48 * nc,
                "flops": c["steps"] * 20 * cv}
    nc, nvel, nm = int(np.prod(_cells(c))), c["nv"] ** c["d"], c["d"] + 2
    piece = 4 if c["precision"] else 8
    cv = nc * nvel
    return {"bytes": c["steps"] * (2 * piece * cv + 16 * nm * nc) + piece * cv + 16 * nm * nc
            + (8 + piece) * cv * c["read_f"],
            "flops": c["steps"] * cv * (12 + 2 * nm)}


# ------------------------------------------------- the scheme in plain FP64
def _t(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


def _shifted(a, axis, off, bc):
    """a at the cells `off` further along `axis` (periodic or zero gradient)"""
    n = a.shape[axis]
    i = torch.arange(n, device=DEV) + off
    i = i % n if bc == 0 else i.clamp(0, n - 1)
    return a.index_select(axis, i)


def _prims(U, d):
    rho, u = U[0], U[1:1 + d] / U[0]
    usq = (u * u).sum(0)
    return rho, u, (2 * U[d + 1] - rho * usq) / (d * rho)


def _flux(U, a, d):
    rho, u, th = _prims(U, d)
    p = rho * th
    F = U * u[a]
    F[0] = U[1 + a]
    F[1 + a] += p
    F[d + 1] += p * u[a]
    return F


def _speeds(U, d):
    rho, u, th = _prims(U, d)
    c = torch.sqrt((d + 2.0) / d * th)
    return [(u[a].abs() + c) for a in range(d)]


def _limited(num, den, unlimited):
    if unlimited:
        return den
    chi = num / torch.where(den == 0, torch.ones_like(den), den)
    phi = (chi.abs() + chi) / (1 + chi)
    return torch.where((den == 0) | ~(chi > 0), torch.zeros_like(den), den * phi)


def _muscl_rhs(U, alpha, d, bcs, unlimited, shift=_shifted):
    """sum over the axes of the flux difference of every cell"""
    div = torch.zeros_like(U)
    for a in range(d):
        ax = U.dim() - 1 - a
        F = _flux(U, a, d)
        Wp, Wm = F + alpha[a] * U, F - alpha[a] * U
        at = lambda w, o: shift(w, ax, o, bcs[a])  # noqa: E731

        def face(o):  # between the cells j + o and j + o + 1
            sp = _limited(at(Wp, o) - at(Wp, o - 1), at(Wp, o + 1) - at(Wp, o), unlimited)
            sm = _limited(at(Wm, o + 1) - at(Wm, o), at(Wm, o + 2) - at(Wm, o + 1), unlimited)
            return (0.5 * (at(F, o) + at(F, o + 1)) - 0.5 * alpha[a] * (at(U, o + 1) - at(U, o))
                    + 0.25 * (sp - sm))
        div += face(0) - face(-1)
    return div


def _weno5(v):
    q = [(2 * v[0] - 7 * v[1] + 11 * v[2]) / 6, (-v[1] + 5 * v[2] + 2 * v[3]) / 6,
         (2 * v[2] + 5 * v[3] - v[4]) / 6]
    b = [13 / 12 * (v[0] - 2 * v[1] + v[2]) ** 2 + 0.25 * (v[0] - 4 * v[1] + 3 * v[2]) ** 2,
         13 / 12 * (v[1] - 2 * v[2] + v[3]) ** 2 + 0.25 * (v[1] - v[3]) ** 2,
         13 / 12 * (v[2] - 2 * v[3] + v[4]) ** 2 + 0.25 * (3 * v[2] - 4 * v[3] + v[4]) ** 2]
    w = [g / (1e-6 + x) ** 2 for g, x in zip((0.1, 0.6, 0.3), b)]
    return sum(wi * qi for wi, qi in zip(w, q)) / sum(w)


def _weno_rhs(U, alpha, d, bcs):
    div = torch.zeros_like(U)
    for a in range(d):
        ax = U.dim() - 1 - a
        F = _flux(U, a, d)
        hp, hm = 0.5 * (F + alpha[a] * U), 0.5 * (F - alpha[a] * U)

        def face(o):
            return (_weno5([_shifted(hp, ax, o + q, bcs[a]) for q in (-2, -1, 0, 1, 2)])
                    + _weno5([_shifted(hm, ax, o + q, bcs[a]) for q in (3, 2, 1, 0, -1)]))
        div += face(0) - face(-1)
    return div


def _euler(U, c, dt, dx):
    d, bcs = c["d"], _bc(c)
    weno = c["scheme"] == 3
    alpha = [float(x.max()) for x in _speeds(U, d)]
    s = max(1, math.ceil((2.5 if weno else 2.0) * dt * sum(alpha) / dx))
    h = dt / s / dx
    for i in range(s):
        if i:
            alpha = [float(x.max()) for x in _speeds(U, d)]
        if not weno:
            U = U - h * _muscl_rhs(U, alpha, d, bcs, c["scheme"] == 2)
            continue
        U1 = U - h * _weno_rhs(U, alpha, d, bcs)
        U2 = 0.75 * U + 0.25 * (U1 - h * _weno_rhs(U1, alpha, d, bcs))
        U = U / 3 + 2 / 3 * (U2 - h * _weno_rhs(U2, alpha, d, bcs))
    return U


def _exact_grid(c, seed):
    d, nv, dv, bcs = c["d"], c["nv"], c["dv"], _bc(c)
    shape = tuple(reversed(_cells(c)))
    dx = c["length"] / c["nx"]
    dt = _dt(c) or dx / dv
    w = dv ** d
    k = np.arange(nv) - nv // 2
    v = torch.as_tensor(k * dv, dtype=torch.float64, device=DEV)
    one = (1,) * d
    vx = v.view(nv, *one)
    rows = [(0.0, 0.0)] if d == 1 else ([(0.0, y * dv) for y in k.tolist()] if d == 2 else
                                       [(z * dv, y * dv) for z in k.tolist() for y in k.tolist()])

    def invariants(row):
        """m_r(v) over the nodes of one velocity row, as numbers or (nv, 1..)"""
        trans = [row[1], row[0]][:d - 1]
        return [1.0, vx] + trans + [0.5 * (vx * vx + sum(t * t for t in trans))]

    M = torch.zeros(d + 2, d + 2, dtype=torch.float64, device=DEV)
    for row in rows:
        m = [torch.as_tensor(x, dtype=torch.float64, device=DEV).reshape(-1).expand(nv)
             for x in invariants(row)]
        m = torch.stack(m)
        M += w * w * (m @ m.T)
    A = torch.linalg.inv(M)

    def maxwellian(P, row):
        rho, u, th = P
        q = (vx - u[0]) ** 2
        for t, ua in zip([row[1], row[0]][:d - 1], u[1:]):
            q = q + (t - ua) ** 2
        return rho / (2 * math.pi * th) ** (0.5 * d) * torch.exp(-q / (2 * th))

    def moments_of(get):
        S = torch.zeros((d + 2,) + shape, dtype=torch.float64, device=DEV)
        for r, row in enumerate(rows):
            g = get(r, row)
            for q, m in enumerate(invariants(row)):
                S[q] += (m * g).sum(0) if torch.is_tensor(m) else m * g.sum(0)
        return w * S

    def corrected(cf, g, row):
        for q, m in enumerate(invariants(row)):
            g = g + w * m * cf[q]
        return g

    def equilibrium(U):
        P = _prims(U, d)
        cE = torch.tensordot(A, U - moments_of(lambda r, row: maxwellian(P, row)), 1)
        return lambda row: corrected(cE, maxwellian(P, row), row)

    rho, u, th = (_t(a) for a in _fields(c, seed))
    rho, u, th = rho.view(shape), u.view((d,) + shape), th.view(shape)
    U = torch.stack([rho, *(rho * u), 0.5 * rho * (u * u).sum(0) + 0.5 * d * rho * th])
    E = equilibrium(U)
    f = torch.stack([E(row) for row in rows])
    for n in range(c["steps"]):
        e = dt / c["tau"] if not c["strang"] or n else 0.5 * dt / c["tau"]
        lam, mu = math.exp(-e), -math.expm1(-e)
        if _dt(c):
            cc = [(kk * dv) * dt / dx for kk in k.tolist()]
            sh = [math.ceil(x * (n + 1) - 0.5) - math.ceil(x * n - 0.5) for x in cc]
        else:
            sh = k.tolist()
        ix = torch.arange(shape[-1], device=DEV)[None] - torch.tensor(sh, device=DEV)[:, None]
        ix = ix % shape[-1] if bcs[0] == 0 else ix.clamp(0, shape[-1] - 1)
        ix = ix.view((nv,) + (1,) * (d - 1) + (shape[-1],)).expand((nv,) + shape)
        E = equilibrium(U)
        fn = torch.empty_like(f)
        sF, sE = torch.zeros_like(U), torch.zeros_like(U)
        for r, row in enumerate(rows):
            def moved(g):
                g = torch.gather(g, g.dim() - 1, ix)
                if d > 1:
                    g = _shifted(g, g.dim() - 2, -sh[r % nv], bcs[1])
                if d > 2:
                    g = _shifted(g, 1, -sh[r // nv], bcs[2])
                return g
            F, Er = moved(f[r]), moved(E(row))
            fn[r] = lam * F + mu * Er
            for q, m in enumerate(invariants(row)):
                sF[q] += (m * F).sum(0) if torch.is_tensor(m) else m * F.sum(0)
                sE[q] += (m * Er).sum(0) if torch.is_tensor(m) else m * Er.sum(0)
        Us, UM = lam * w * sF, mu * w * sE
        if c["scheme"] == 1:
            UE = UM
        else:
            UE = mu * _euler(U, c, dt, dx)
            cf = torch.tensordot(A, UE - UM, 1)
            for r, row in enumerate(rows):
                fn[r] = corrected(cf, fn[r], row)
        f, U = fn, Us + UE
    out = {"U": U.reshape(d + 2, -1).cpu().numpy()}
    if c["read_f"]:
        out["f"] = f.reshape(nv ** d, -1).cpu().numpy()
    return out


def _exact_batch(c, seed):
    """all tubes side by side, padded to the longest with their last cell"""
    tubes, (rho, u, th) = _tubes(c, seed)
    nx = np.array([t[0] for t in tubes])
    col = lambda q: _t([float(t[q]) for t in tubes])[:, None]  # noqa: E731
    dx, dv, tau, nvs = col(1), col(3), col(4), [t[2] for t in tubes]
    n_t, nxs, nvm = len(tubes), int(nx.max()), max(nvs)
    last = torch.as_tensor(nx - 1, device=DEV)[:, None]
    start = torch.as_tensor(np.cumsum(nx) - nx, device=DEV)[:, None]
    pos = torch.arange(nxs, device=DEV)[None]
    real = pos <= last

    def cells(off):  # cell pos + off of each tube, zero gradient outside
        return (pos + off).clamp(min=0).minimum(last)

    def shift(a, _axis, off, _bc):
        return torch.gather(a, 2, cells(off)[None].expand(a.shape[0], -1, -1))

    pad = lambda a: _t(a)[start + cells(0)]  # noqa: E731
    rho, u, th = pad(rho), pad(u), pad(th)
    U = torch.stack([rho, rho * u, 0.5 * rho * u * u + 0.5 * rho * th])
    half = torch.as_tensor(nvs, device=DEV)[:, None] // 2
    on = [torch.as_tensor([float(i < nv) for nv in nvs], dtype=torch.float64, device=DEV)[:, None]
          for i in range(nvm)]
    vel = [(i - half) * dv for i in range(nvm)]
    m = [torch.stack([o, o * x, 0.5 * o * x * x]) for o, x in zip(on, vel)]  # (3, tubes, 1)
    M = sum(dv[:, :, None] ** 2 * torch.einsum("rt,st->trs", q[:, :, 0], q[:, :, 0]) for q in m)
    A = torch.linalg.inv(M).permute(1, 2, 0)[..., None]  # (3, 3, tubes, 1)
    speed = lambda U: (_speeds(U, 1)[0] * real).amax(1, keepdim=True)  # noqa: E731
    solve = lambda D: (A * D[None]).sum(1)  # noqa: E731

    def equilibrium(U):
        r, (uu,), t = _prims(U, 1)
        mx = lambda x: r / torch.sqrt(2 * math.pi * t) * torch.exp(-(x - uu) ** 2 / (2 * t))  # noqa: E731
        CM = sum(dv * q * mx(x) for q, x in zip(m, vel))
        cE = solve(U - CM)
        return lambda i: on[i] * mx(vel[i]) + dv * (m[i] * cE).sum(0)

    E = equilibrium(U)
    f = torch.stack([E(i) for i in range(nvm)])
    dt = dx / dv
    lam, mu = torch.exp(-dt / tau), -torch.expm1(-dt / tau)
    for _ in range(c["steps"]):
        E = equilibrium(U)
        sF, sE, fn = torch.zeros_like(U), torch.zeros_like(U), torch.empty_like(f)
        for i in range(nvm):
            at = cells(half - i)
            F, Ei = torch.gather(f[i], 1, at), torch.gather(E(i), 1, at)
            fn[i] = lam * F + mu * Ei
            sF += m[i] * F
            sE += m[i] * Ei
        alpha = speed(U)
        s = torch.ceil(2.0 * dt * alpha / dx).clamp(min=1.0)
        h = dt / s / dx
        V = U
        for it in range(int(s.max())):
            if it:
                alpha = speed(V)
            V = torch.where(it < s, V - h * _muscl_rhs(V, [alpha], 1, [1], False, shift), V)
        UE, UM = mu * V, mu * dv * sE
        cf = solve(UE - UM)
        for i in range(nvm):
            fn[i] += dv * (m[i] * cf).sum(0)
        f, U = fn, lam * dv * sF + UE
    U = U.cpu().numpy()
    real = real.cpu().numpy()
    return {"U": np.concatenate([U[:, t, real[t]].reshape(-1) for t in range(n_t)]), "flags": None}


def _exact_train(c, seed):
    """the same steps with FP64 weights, activations and moments"""
    x, t = _samples(c, seed)
    x, t = x.double(), t.double()
    flat = _t(ClosureNet(seed=seed % 1000).params.cpu().numpy())
    m, v = torch.zeros_like(flat), torch.zeros_like(flat)
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    sizes = [(64, 37), (64,), (64, 64), (64,), (64, 64), (64,), (4, 64), (4,)]
    for it in range(c["steps"]):
        i = torch.randint(0, c["rows"], (c["batch"],), device=DEV, generator=g, dtype=torch.int32)
        lr = 2e-3 * (2e-4 / 2e-3) ** (it / max(c["steps"] - 1, 1))
        p = flat.clone().requires_grad_()
        W, o = [], 0
        for s in sizes:
            W.append(p[o:o + math.prod(s)].view(s))
            o += math.prod(s)
        a = x[i.long()]
        for q in range(3):
            a = torch.tanh(a @ W[2 * q].T + W[2 * q + 1])
        loss = ((a @ W[6].T + W[7] - t[i.long()]) ** 2).mean()
        grad, = torch.autograd.grad(loss, p)
        m, v = 0.9 * m + 0.1 * grad, 0.999 * v + 0.001 * grad * grad
        flat = flat - lr * (m / (1 - 0.9 ** (it + 1))) / ((v / (1 - 0.999 ** (it + 1))).sqrt() + 1e-8)
    return {"params": flat, "m": m, "v": v, "grad": grad, "loss": loss.detach().reshape(1)}


def exact(case, seed):
    c = case
    if c["kind"] == "batch":
        return _exact_batch(c, seed)
    if c["kind"] == "train":
        return _exact_train(c, seed)
    if c["kind"] == "closure":
        dx = c["length"] / c["n"]
        if math.exp(-dx / c["dv"] / c["tau"]) > 1e-18:
            return None  # the network's estimate counts: not a number of the scheme
        g = _grid(None, (c["n"], c["n"]), c["nv"], c["dv"], c["tau"], c["steps"], "disk",
                  length=c["length"], precision=1)
        return _exact_grid(g, seed)
    return _exact_grid(c, seed)
