"""The work that users of the framework have it do, as cases that can be timed.

Kinds of work:

* ``uniform``  one periodic grid stepped by hand: band fill, CFL reduction and
  advance, the band refilled every second step (two steps a pass, so the state
  is back in its first buffer);
* ``amr``      coarse steps of a refined hierarchy (two a pass: level 0 changes
  buffer every coarse step), eager or replayed from HIP graphs;
* ``adjoint``  the gradient of a loss after a number of steps with respect to
  the initial density and velocity, through torch.autograd (forward with
  checkpoints, then the reverse sweep);
* ``regrid``   the refinement flags of level 1, a new hierarchy (another seeded
  grid list stands for the clustered one, so every pass returns one layout) and
  the (O)verlap of every level into it.

Each case names its launch configuration as a user's program does: the default
or what the autotuner keeps on such a workload.  ``exact`` is the same scheme
in plain torch at 64 bits: unsplit MUSCL-Hancock on primitives with minmod
slopes, HLLD fluxes (Miyoshi & Kusano 2005), constrained transport with the
arithmetic (Balsara & Spicer 1999) or the upwinded (Gardiner & Stone 2005)
edge EMF, on a periodic box; its gradients come from torch's autograd.
"""

import math

import numpy as np
import torch
from torch.utils.checkpoint import checkpoint

from paper_1110_1616_amd import amr as A
from paper_1110_1616_amd import autodiff as AD
from paper_1110_1616_amd import inputs as I

GAMMA = 5.0 / 3.0
CFL = 0.4
TWO_PI = 2.0 * math.pi

# What the autotuner keeps (bench.py): fused persistent launches on
# hierarchies, XCD chunks on one large grid; "" is the library's default.
FUSED = "1,32,12"
FUSED_XCD = "1,32,14"
FUSED_ONE = "1,32,10"


# ---------------------------------------------------------------- the cases
def _uniform(ndim, n, dtype="f64", emf=0, launch=""):
    nx, ny, nz = tuple(n) + (1,) * (3 - len(n))
    return {"kind": "uniform", "ndim": ndim, "nx": nx, "ny": ny, "nz": nz, "dtype": dtype, "emf": emf,
            "launch": launch}


def _amr(ndim, n0, levels, ext, tree, dtype="f64", graph=False, launch="", log_uniform=False, kind="amr"):
    return {"kind": kind, "ndim": ndim, "n0": n0, "levels": levels, "ext_lo": ext[0], "ext_hi": ext[1],
            "tree": tree, "dtype": dtype, "graph": graph, "launch": launch, "log_uniform": log_uniform}


def _adjoint(ndim, n, steps, every):
    nx, ny, nz = tuple(n) + (1,) * (3 - len(n))
    return {"kind": "adjoint", "ndim": ndim, "nx": nx, "ny": ny, "nz": nz, "steps": steps, "every": every}


def listed():
    return [
        # a small 2-D run: what a step costs when the launches are most of it
        dict(_uniform(2, (64, 64)), name="grid2d_64_f64"),
        # a 2-D production grid of odd extents, in single precision
        dict(_uniform(2, (1021, 517), "f32"), name="grid2d_odd_f32"),
        # an odd little 3-D grid in the library's default configuration
        dict(_uniform(3, (37, 33, 35), "f32"), name="grid3d_odd_f32"),
        # one large 3-D grid, tuned: the single-grid benchmark
        dict(_uniform(3, (128, 128, 128), launch=FUSED_ONE), name="grid3d_128_f64"),
        # the upwinded edge EMF (always the two-kernel path)
        dict(_uniform(3, (72, 72, 72), emf=1), name="upwind3d_72_f64"),
        # small hierarchies, eager and untuned: many short launches a step
        dict(_amr(2, 64, 3, (8, 32), 4), name="amr2d_64_f64"),
        dict(_amr(3, 24, 3, (8, 16), 11), name="amr3d_24_f64"),
        # the headline: 3 levels on a base of 112^3, 549 grids, from graphs
        dict(_amr(3, 112, 3, (8, 32), 3, graph=True, launch=FUSED), name="amr3d_112_f64"),
        # the deep hierarchy's 1/8-volume subvolume: 6 levels, FP32
        dict(_amr(3, 100, 6, (8, 48), 5, "f32", True, FUSED_XCD, True), name="deep6_100_f32"),
        # gradients: the differentiation benchmark's grid and step count ...
        dict(_adjoint(3, (64, 64, 64), 20, 5), name="adjoint3d_64_f64"),
        # ... and a small 2-D one, where launches count
        dict(_adjoint(2, (96, 80), 10, 5), name="adjoint2d_f64"),
        # the adaptive part of a run: a new finest level and its transfer
        dict(_amr(3, 48, 3, (8, 32), 3, kind="regrid"), name="regrid3d_48_f64"),
    ]


def _size(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["uniform2", "uniform3", "uniform3", "amr2", "amr3", "amr3", "adjoint2", "adjoint3"])
    if kind == "uniform2":
        n = (_size(rng, 33, 1100), _size(rng, 33, 1100))
        return _uniform(2, n, rng.choice(["f64", "f32"]), rng.choice([0, 0, 1]), rng.choice(["", FUSED]))
    if kind == "uniform3":
        n = (_size(rng, 20, 128), _size(rng, 20, 128), _size(rng, 20, 128))
        return _uniform(3, n, rng.choice(["f64", "f32"]), rng.choice([0, 0, 1]), rng.choice(["", FUSED, FUSED_ONE]))
    if kind == "amr2":
        return _amr(2, 2 * _size(rng, 16, 96), 3, (8, 32), rng.randrange(100), rng.choice(["f64", "f32"]),
                    rng.choice([False, True]), rng.choice(["", FUSED]))
    if kind == "amr3":
        return _amr(3, 4 * _size(rng, 6, 20), rng.choice([2, 3]), (8, rng.choice([16, 32])), rng.randrange(100),
                    rng.choice(["f64", "f32"]), rng.choice([False, True]), rng.choice(["", FUSED, FUSED_XCD]))
    if kind == "adjoint2":
        return _adjoint(2, (_size(rng, 24, 256), _size(rng, 24, 256)), rng.choice([4, 7, 10]), rng.choice([2, 5]))
    return _adjoint(3, (_size(rng, 16, 64), _size(rng, 16, 64), _size(rng, 16, 64)), rng.choice([4, 7, 10]),
                    rng.choice([2, 5]))


# ---------------------------------------------------------------- inputs
class _Modes:
    """Eight Fourier modes each for density, velocity, vector potential and
    pressure on the unit box (the framework's smooth seeded fields)."""

    def __init__(self, seed, ndim, b_rms):
        rng = np.random.default_rng(seed)

        def modes():
            k = np.zeros((8, 3))
            for m in range(8):
                while not k[m].any():
                    k[m, :ndim] = rng.integers(-4, 5, size=ndim)
            return k, rng.uniform(0.0, TWO_PI, size=8)

        def unit():
            a = rng.normal(size=(8, 3))
            return a / np.linalg.norm(a, axis=1, keepdims=True)

        self.rho, self.p = modes(), modes()
        self.psi, self.pot = modes(), modes()
        a_psi, self.a_pot = unit(), unit()
        self.v = -np.cross(TWO_PI * self.psi[0], a_psi)  # curl of the stream function: times sin
        self.v *= 0.1 / math.sqrt(0.5 * float((self.v ** 2).sum()))
        b = np.cross(TWO_PI * self.pot[0], self.a_pot)
        self.a_pot = self.a_pot * (b_rms / math.sqrt(0.5 * float((b ** 2).sum())))


def _mode_sum(modes, amp, axes, quarter=0.0):
    """sum_m amp[m] cos(2 pi k_m . x + phi_m - quarter turn), shape (z, y, x)."""
    k, phi = modes
    dev = axes[0].device
    kt = torch.as_tensor(k, device=dev)
    ph = [TWO_PI * kt[:, a, None] * axes[a][None, :] for a in range(3)]
    ph[2] = ph[2] + torch.as_tensor(phi - quarter * 0.5 * math.pi, device=dev)[:, None]
    yx = (ph[1][:, :, None] + ph[0][:, None, :]).reshape(8, -1)
    am = torch.as_tensor(amp, device=dev)[:, None]
    out = (am * torch.cos(ph[2])).t() @ torch.cos(yx) - (am * torch.sin(ph[2])).t() @ torch.sin(yx)
    return out.reshape(len(axes[2]), len(axes[1]), len(axes[0]))


def _edge_factor(k, h, r):
    """Mean of the r finest samples of a mode along a coarse edge, over its
    value at the middle."""
    d = TWO_PI * np.asarray(k) * h
    s = np.sin(0.5 * d)
    return np.where(np.abs(s) < 1e-14, 1.0, np.sin(0.5 * r * d) / (r * np.where(np.abs(s) < 1e-14, 1.0, s)))


def _grid_fields(F, ndim, lo, hi, n_level, n_fine, ratio, jump, p_amp, dev):
    """Primitives and face B of the box [lo, hi) of a level with n_level cells
    per axis; the potential is averaged over `ratio` finest samples an edge."""
    h = [1.0 / n_level[a] if a < ndim else 1.0 for a in range(3)]

    def axis(a, off, more=0):
        if a >= ndim:
            return torch.zeros(1, dtype=torch.float64, device=dev)
        idx = torch.arange(lo[a], hi[a] + more, device=dev) % n_level[a]
        return (idx.double() + off) * h[a]

    c = [axis(a, 0.5) for a in range(3)]
    rho = 1.0 + 0.1 * _mode_sum(F.rho, np.ones(8), c)
    if jump:
        rho = torch.where(((c[0] >= 0.25) & (c[0] < 0.75))[None, None, :], 4.0 * rho, rho)
    p = 1.0 + p_amp * _mode_sum(F.p, np.ones(8), c) if p_amp else torch.ones_like(rho)
    prim = [rho] + [_mode_sum(F.psi, F.v[:, a].copy(), c, 1.0) for a in range(3)] + [p]

    pot = []
    for a in range(3):
        amp = F.a_pot[:, a].copy()
        if a < ndim:
            amp = amp * _edge_factor(F.pot[0][:, a], 1.0 / n_fine[a], ratio)
        pot.append(_mode_sum(F.pot, amp, [axis(b, 0.5) if b == a else axis(b, 0.0, 1) for b in range(3)]))

    def diff(f, a):
        return torch.diff(f, dim=2 - a) / h[a] if a < ndim else 0.0

    b = [diff(pot[(a + 2) % 3], (a + 1) % 3) - diff(pot[(a + 1) % 3], (a + 2) % 3) for a in range(3)]
    return [t.contiguous() for t in prim], [t.contiguous() for t in b]


def _single(case, seed, p_amp=0.0):
    """Seeded state of one periodic grid (the 4:1 density jump where the
    pressure is smooth: gradients are taken of smooth states)."""
    ndim, n = case["ndim"], (case["nx"], case["ny"], case["nz"])
    dev = "cuda" if torch.cuda.is_available() else "cpu"
    F = _Modes(seed, ndim, 0.1 if ndim == 2 else 0.3)
    return _grid_fields(F, ndim, (0, 0, 0), n, n, n, 1, not p_amp, p_amp, dev)


def _launch(H, text):
    if text:
        H.set_launch_config(*[int(v) for v in text.split(",")])


def _views(H, U):
    """Interior views of grid 0's pools: cells, then faces along x, y, z."""
    g, n = H.ghost, H.grid_shape(0)
    P = [n[a] + 2 * g + 1 if a < H.ndim else 1 for a in range(3)]
    lo = [g if a < H.ndim else 0 for a in range(3)]
    out = []
    for q, f in enumerate(U.fields):
        e = [n[a] + (1 if q == 5 + a and a < H.ndim else 0) for a in range(3)]
        box = f[H.offsets[0]:H.offsets[0] + P[0] * P[1] * P[2]].view(P[2], P[1], P[0])
        out.append(box[lo[2]:lo[2] + e[2], lo[1]:lo[1] + e[1], lo[0]:lo[0] + e[0]])
    return out


def prepare(case, seed):
    return {"uniform": _prepare_uniform, "amr": _prepare_amr, "regrid": _prepare_amr,
            "adjoint": _prepare_adjoint}[case["kind"]](case, seed)


def _prepare_uniform(case, seed):
    ndim = case["ndim"]
    n = (case["nx"], case["ny"], case["nz"])[:ndim]
    prim, b = _single(case, seed)
    H = A.Hierarchy(ndim, n, [(0, (0,) * ndim, n)], ghost=4, dtype=case["dtype"], gamma=GAMMA, cfl=CFL,
                    emf=case["emf"])
    _launch(H, case["launch"])
    U, V = H.new_state(), H.new_state()
    A.amr_load_primitive(H.h, 0, prim, b, U.c)
    return {"kind": "uniform", "H": H, "U": U, "V": V, "out": _views(H, U)}


def _tree(case):
    return I.amr_hierarchy(case["ndim"], (case["n0"],) * case["ndim"], case["levels"], seed=case["tree"],
                           ext=(case["ext_lo"], case["ext_hi"]), log_uniform=case["log_uniform"])


def _prepare_amr(case, seed):
    ndim, L = case["ndim"], case["levels"]
    N0 = (case["n0"],) * ndim
    grids = _tree(case)
    H = A.Hierarchy(ndim, N0, grids, nlevels=L, ghost=4, dtype=case["dtype"], gamma=GAMMA, cfl=CFL)
    _launch(H, case["launch"])
    Ua, Ub = H.new_state(), H.new_state()
    F = _Modes(seed, ndim, 0.1 if ndim == 2 else 0.3)
    fine = [n * 2 ** (L - 1) for n in N0]
    for gi, (l, lo, hi) in enumerate(grids):
        lo, hi = tuple(lo) + (0,) * (3 - ndim), tuple(hi) + (1,) * (3 - ndim)
        prim, b = _grid_fields(F, ndim, lo, hi, [n * 2 ** l for n in N0], fine, 2 ** (L - 1 - l), False, 0.0, "cuda")
        A.amr_load_primitive(H.h, gi, prim, b, Ua.c)
    st = {"kind": case["kind"], "H": H, "Ua": Ua, "Ub": Ub, "par": 0, "stream": None}
    if case["graph"]:
        st["stream"] = torch.cuda.Stream()
        torch.cuda.synchronize()
        with torch.cuda.stream(st["stream"]):
            H.graph_capture(Ua, Ub, 0)
    if case["kind"] == "regrid":
        st["case"], st["new"] = case, _tree(dict(case, tree=case["tree"] + 1))
        H.fill(0, A.AMR_FILL_SAME_LEVEL, Ua)
        for l in range(1, L):
            H.fill(l, A.AMR_FILL_FULL, Ua, Ua)
    return st


def _prepare_adjoint(case, seed):
    ndim = case["ndim"]
    n = (case["nx"], case["ny"], case["nz"])[:ndim]
    prim, b = _single(case, seed, p_amp=0.1)
    H = A.Hierarchy(ndim, n, [(0, (0,) * ndim, n)], ghost=2, gamma=GAMMA)
    ctl = [t.requires_grad_(True) for t in prim[:4]]
    return {"kind": "adjoint", "H": H, "ctl": ctl, "p": prim[4], "b": b, "dts": _steps(case), "every": case["every"]}


def _steps(case):
    """Frozen step sizes of the differentiated run, a little under the CFL
    limit of these states."""
    ndim = case["ndim"]
    h = min(1.0 / v for v in (case["nx"], case["ny"], case["nz"])[:ndim])
    return [(0.08 if ndim == 2 else 0.05) * h] * case["steps"]


# ---------------------------------------------------------------- one pass
def run(state):
    return {"uniform": _run_uniform, "amr": _run_amr, "regrid": _run_regrid,
            "adjoint": _run_adjoint}[state["kind"]](state)


def _run_uniform(s):
    H, U, V = s["H"], s["U"], s["V"]
    H.fill(0, A.AMR_FILL_SAME_LEVEL, U)
    H.compute_dt(U)
    H.advance(U, V, cycle=0, band=4)
    H.compute_dt(V)
    H.advance(V, U, cycle=0, band=2)
    return s["out"]


def _run_amr(s):
    H = s["H"]
    if s["stream"] is None:
        for _ in range(2):
            s["par"] = H.coarse_step(s["Ua"], s["Ub"], s["par"])
    else:
        with torch.cuda.stream(s["stream"]):
            for _ in range(2):
                s["par"] = H.graph_launch(s["par"])
    return s["Ua"].fields


def _run_regrid(s):
    H, U, c = s["H"], s["Ua"], s["case"]
    flags = H.flags(1, U, U, 0.03)
    new = A.Hierarchy(c["ndim"], H.domain[:c["ndim"]], s["new"], nlevels=H.nlevels, ghost=H.ghost, dtype=c["dtype"],
                      gamma=GAMMA, cfl=CFL)
    V = new.overlap_from(H, [U] * H.nlevels)
    return {"flags": flags, "state": V.fields}


def _loss(rho, mx, my, mz):
    """Kinetic energy in the low corner box of (at most) 16 cells an axis,
    per cell of the grid."""
    s = tuple(slice(0, min(16, e)) for e in rho.shape)
    return ((mx[s] ** 2 + my[s] ** 2 + mz[s] ** 2) / (2.0 * rho[s])).sum() / rho.numel()


def _run_adjoint(s):
    H = s["H"]
    U = AD.LoadPrimitive.apply(H, 0, *s["ctl"], s["p"], *s["b"])
    out = AD.StoreInterior.apply(H, 0, *AD.advance(H, 0, s["dts"], U, every=s["every"]))
    J = _loss(*out[:4])
    grads = torch.autograd.grad(J, s["ctl"])
    return {"loss": J.detach(), "grad": list(grads), "state": [t.detach() for t in out]}


# ---------------------------------------------------------------- the floor
# Operations of the scheme (each +, -, *, /, sqrt one): per cell with
# predicted states, per Riemann problem, per updated cell, face and edge EMF.
_PRED, _HLLD = {2: 612, 3: 912}, 367
_CELL, _FACE, _EDGE = {2: 48, 3: 55}, {2: 5, 3: 8}, 4


def _step_flops(ndim, cells):
    return cells * (_PRED[ndim] + ndim * _HLLD + _CELL[ndim] + ndim * _FACE[ndim] + (3 if ndim == 3 else 1) * _EDGE)


def work(case):
    es = 4 if case.get("dtype") == "f32" else 8
    ndim = case["ndim"]
    if case["kind"] in ("uniform", "adjoint"):
        cells = case["nx"] * case["ny"] * case["nz"]
        if case["kind"] == "uniform":
            return {"bytes": 2 * 16 * es * cells, "flops": 2 * _step_flops(ndim, cells)}
        # forward: the state read and written a step; reverse: the step's
        # input and the adjoint read, the adjoint written, and about three
        # times the forward step's operations (values and derivatives)
        k = case["steps"]
        return {"bytes": k * (16 + 24) * es * cells, "flops": 4 * k * _step_flops(ndim, cells)}
    cells = [0] * case["levels"]
    for l, lo, hi in _tree(case):
        cells[l] += int(np.prod([hi[a] - lo[a] for a in range(ndim)]))
    if case["kind"] == "regrid":
        # the old state read once, the new one written once
        return {"bytes": 16 * es * sum(cells), "flops": 0}
    updates = sum(c * 2 ** l for l, c in enumerate(cells))
    return {"bytes": 2 * 16 * es * updates, "flops": 2 * _step_flops(ndim, updates)}


# ------------------------------------------------------- the same in 64 bits
class _Plain:
    """The scheme on one periodic grid in plain torch, float64.  Fields have
    shape (z, y, x); face arrays hold each cell's low face.  Lab components:
    conserved (rho, mx, my, mz, E, Bx, By, Bz), primitive (rho, v, p, B)."""

    def __init__(self, case):
        self.nd = case["ndim"]
        self.emf = case.get("emf", 0)
        n = (case["nx"], case["ny"], case["nz"])
        self.h = [1.0 / n[a] for a in range(self.nd)]

    @staticmethod
    def up(f, a):  # value at c + e_a
        return torch.roll(f, -1, 2 - a)

    @staticmethod
    def dn(f, a):  # value at c - e_a
        return torch.roll(f, 1, 2 - a)

    def load(self, prim, b):
        rho, vx, vy, vz, p = prim
        low = [b[a].narrow(2 - a, 0, b[a].shape[2 - a] - 1) if a < self.nd else b[a] for a in range(3)]
        B = self.centred(low)
        E = p / (GAMMA - 1.0) + 0.5 * rho * (vx * vx + vy * vy + vz * vz) + 0.5 * (B[0] ** 2 + B[1] ** 2 + B[2] ** 2)
        return [rho, rho * vx, rho * vy, rho * vz, E] + low

    def store(self, U):
        out = list(U)
        for a in range(self.nd):
            f = U[5 + a]
            out[5 + a] = torch.cat([f, f.narrow(2 - a, 0, 1)], 2 - a)
        return out

    def centred(self, low):
        return [0.5 * (low[a] + self.up(low[a], a)) if a < self.nd else low[a] for a in range(3)]

    def primitive(self, U, B):
        v = [U[1 + a] / U[0] for a in range(3)]
        p = (GAMMA - 1.0) * (U[4] - 0.5 * U[0] * sum(x * x for x in v) - 0.5 * sum(x * x for x in B))
        return [U[0]] + v + [p] + list(B)

    @staticmethod
    def conserved(w):
        k = 0.5 * w[0] * (w[1] ** 2 + w[2] ** 2 + w[3] ** 2) + 0.5 * (w[5] ** 2 + w[6] ** 2 + w[7] ** 2)
        return [w[0], w[0] * w[1], w[0] * w[2], w[0] * w[3], w[4] / (GAMMA - 1.0) + k] + list(w[5:])

    @staticmethod
    def fast(r, p, b2, bn):
        a = (GAMMA * p + b2) / r
        d = a * a - 4.0 * GAMMA * p * bn * bn / (r * r)
        return torch.sqrt(0.5 * (a + torch.sqrt(torch.clamp(d, min=1e-300))))

    def dt(self, U):
        w = self.primitive(U, self.centred(U[5:]))
        b2 = w[5] ** 2 + w[6] ** 2 + w[7] ** 2
        s = sum((w[1 + a].abs() + self.fast(w[0], w[4], b2, w[5 + a])) / self.h[a] for a in range(self.nd))
        return CFL / s.max()

    @staticmethod
    def flux(w, d):
        v2 = w[1] ** 2 + w[2] ** 2 + w[3] ** 2
        b2 = w[5] ** 2 + w[6] ** 2 + w[7] ** 2
        pt = w[4] + 0.5 * b2
        e = w[4] / (GAMMA - 1.0) + 0.5 * w[0] * v2 + 0.5 * b2
        vn, bn = w[1 + d], w[5 + d]
        f = [w[0] * vn]
        f += [w[0] * vn * w[1 + a] - bn * w[5 + a] + (pt if a == d else 0.0) for a in range(3)]
        f.append((e + pt) * vn - bn * (w[1] * w[5] + w[2] * w[6] + w[3] * w[7]))
        f += [w[5 + a] * vn - bn * w[1 + a] if a != d else torch.zeros_like(vn) for a in range(3)]
        return f

    @staticmethod
    def minmod(a, b):
        zero = torch.zeros_like(a)
        return torch.where(a * b > 0, torch.where(b.abs() < a.abs(), b, a), zero)

    def hlld(self, L, R, bn):
        """L, R: (rho, u, v, w, p, by, bz) with the normal first."""
        def side(q):
            b2 = bn * bn + q[5] ** 2 + q[6] ** 2
            e = q[4] / (GAMMA - 1.0) + 0.5 * q[0] * (q[1] ** 2 + q[2] ** 2 + q[3] ** 2) + 0.5 * b2
            return e, q[4] + 0.5 * b2, self.fast(q[0], q[4], b2, bn)

        el, ptl, cl = side(L)
        er, ptr, cr = side(R)
        c = torch.where(cl > cr, cl, cr)
        sl = torch.where(L[1] < R[1], L[1], R[1]) - c
        sr = torch.where(L[1] > R[1], L[1], R[1]) + c
        rl, rr = L[0] * (sl - L[1]), R[0] * (sr - R[1])
        sm = (rr * R[1] - rl * L[1] - ptr + ptl) / (rr - rl)
        pts = ptl + rl * (sm - L[1])
        tiny = 1e-12 * pts
        one = torch.ones_like(bn)

        def star(q, s, rd, e, pt):
            rs = rd / (s - sm)
            den = rd * (s - sm) - bn * bn
            deg = den.abs() <= tiny
            den = torch.where(deg, one, den)
            fv = torch.where(deg, 0.0 * one, bn * (sm - q[1]) / den)
            fb = torch.where(deg, one, (rd * (s - q[1]) - bn * bn) / den)
            v, w = q[2] - q[5] * fv, q[3] - q[6] * fv
            by, bz = q[5] * fb, q[6] * fb
            vb = q[1] * bn + q[2] * q[5] + q[3] * q[6]
            es = ((s - q[1]) * e - pt * q[1] + pts * sm + bn * (vb - sm * bn - v * by - w * bz)) / (s - sm)
            return [rs, sm, v, w, es, by, bz]

        SL, SR = star(L, sl, rl, el, ptl), star(R, sr, rr, er, ptr)
        ql, qr = torch.sqrt(SL[0]), torch.sqrt(SR[0])
        ssl, ssr = sm - bn.abs() / ql, sm + bn.abs() / qr
        sg = torch.where(bn > 0, one, -one)
        mean = [(ql * SL[a] + qr * SR[a] + (SR[a + 3] - SL[a + 3]) * sg) / (ql + qr) for a in (2, 3)]
        mean += [(ql * SR[a + 3] + qr * SL[a + 3] + ql * qr * (SR[a] - SL[a]) * sg) / (ql + qr) for a in (2, 3)]
        vbm = sm * bn + mean[0] * mean[2] + mean[1] * mean[3]
        ddeg = 0.5 * bn * bn <= tiny

        def double(S, q, sign):
            vb = sm * bn + S[2] * S[5] + S[3] * S[6]
            e = S[4] - sign * q * (vb - vbm) * sg
            new = [S[0], sm, mean[0], mean[1], e, mean[2], mean[3]]
            return [torch.where(ddeg, a, b) for a, b in zip(S, new)]

        DL, DR = double(SL, ql, 1.0), double(SR, qr, -1.0)

        def cons(q, e):
            return [q[0], q[0] * q[1], q[0] * q[2], q[0] * q[3], e, q[5], q[6]]

        def phys(q, e, pt):
            vb = q[1] * bn + q[2] * q[5] + q[3] * q[6]
            return [q[0] * q[1], q[0] * q[1] ** 2 + pt - bn * bn, q[0] * q[1] * q[2] - bn * q[5],
                    q[0] * q[1] * q[3] - bn * q[6], (e + pt) * q[1] - bn * vb, q[5] * q[1] - bn * q[2],
                    q[6] * q[1] - bn * q[3]]

        fl, fr = phys(L, el, ptl), phys(R, er, ptr)
        ul, ur = cons(L, el), cons(R, er)
        usl, usr = cons(SL, SL[4]), cons(SR, SR[4])
        udl, udr = cons(DL, DL[4]), cons(DR, DR[4])
        out = []
        for q in range(7):
            a = fl[q] + sl * (usl[q] - ul[q])
            b = fr[q] + sr * (usr[q] - ur[q])
            x = torch.where(sr >= 0, b, fr[q])
            x = torch.where(ssr >= 0, b + ssr * (udr[q] - usr[q]), x)
            x = torch.where(sm >= 0, a + ssl * (udl[q] - usl[q]), x)
            x = torch.where(ssl >= 0, a, x)
            out.append(torch.where(sl > 0, fl[q], x))
        return out

    def step(self, dt, *U):
        nd, up, dn = self.nd, self.up, self.dn
        low = U[5:]
        W = self.primitive(U, self.centred(low))
        states, du = [], [0.0] * 8
        for d in range(nd):
            s = [self.minmod(w - dn(w, d), up(w, d) - w) for w in W]
            lo, hi = [w - 0.5 * x for w, x in zip(W, s)], [w + 0.5 * x for w, x in zip(W, s)]
            lo[5 + d], hi[5 + d] = low[d], up(low[d], d)
            states.append((lo, hi))
            du = [a - 0.5 * dt / self.h[d] * (y - x) for a, x, y in zip(du, self.flux(lo, d), self.flux(hi, d))]
        F = []
        for d in range(nd):
            order = [0, 1 + d, 1 + (d + 1) % 3, 1 + (d + 2) % 3, 4, 5 + (d + 1) % 3, 5 + (d + 2) % 3]
            half = []
            for w in states[d]:
                u = [a + b for a, b in zip(self.conserved(w), du)]
                q = self.primitive(u, u[5:])
                half.append([q[i] for i in order])
            F.append(self.hlld([dn(x, d) for x in half[1]], half[0], low[d]))

        def slot(s, d):  # rotated flux component that carries lab slot s
            return s if s in (0, 4) else 1 + (s - 1 - d) % 3 if s < 4 else 5 + (s - 6 - d) % 3

        new = list(U)
        for s in range(5) if nd == 3 else (0, 1, 2, 3, 4, 7):
            new[s] = U[s] - sum(dt / self.h[d] * (up(F[d][slot(s, d)], d) - F[d][slot(s, d)]) for d in range(nd))
        E = {}
        if self.emf:
            m = [a + b for a, b in zip(self.conserved(W), du)]
            v = [m[1 + a] / m[0] for a in range(3)]
        for a in range(3) if nd == 3 else (2,):
            b, c = (a + 1) % 3, (a + 2) % 3
            bS, bN, cW, cE = -dn(F[b][5], c), -F[b][5], dn(F[c][6], b), F[c][6]
            E[a] = 0.25 * ((bS + bN) + (cW + cE))
            if self.emf:
                ne = v[c] * W[5 + b] - v[b] * W[5 + c]
                nw, se = dn(ne, b), dn(ne, c)
                sw = dn(nw, c)
                mb, mc = F[b][0], F[c][0]

                def upw(f, lo, hi):
                    return torch.where(f > 0, lo, torch.where(f < 0, hi, 0.5 * (lo + hi)))

                E[a] = E[a] + 0.25 * ((upw(dn(mb, c), cW - sw, cE - se) - upw(mb, nw - cW, ne - cE)) +
                                      (upw(dn(mc, b), bS - sw, bN - nw) - upw(mc, se - bS, ne - bN)))
        for a in range(nd):
            b, c = (a + 1) % 3, (a + 2) % 3
            curl = 0.0
            if b < nd:
                curl = curl + (up(E[c], b) - E[c]) / self.h[b]
            if c < nd:
                curl = curl - (up(E[b], c) - E[b]) / self.h[c]
            new[5 + a] = U[5 + a] - dt * curl
        return tuple(new)


def exact(case, seed):
    """What run() returns for a new state, in 64 bits; None for hierarchies
    (hundreds of grids of every shape: minutes in plain torch)."""
    if case["kind"] == "uniform":
        P = _Plain(case)
        U = P.load(*_single(case, seed))
        for _ in range(2):
            U = P.step(P.dt(U), *U)
        return P.store(U)
    if case["kind"] == "adjoint":
        P = _Plain(case)
        prim, b = _single(case, seed, p_amp=0.1)
        ctl = [t.requires_grad_(True) for t in prim[:4]]
        U = P.load(ctl + [prim[4]], b)
        for dt in _steps(case):
            U = checkpoint(P.step, dt, *U, use_reentrant=False)
        out = P.store(U)
        J = _loss(*out[:4])
        grads = torch.autograd.grad(J, ctl)
        return {"loss": J.detach(), "grad": list(grads), "state": [t.detach() for t in out]}
    return None
