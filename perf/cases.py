"""The calls whose time matters to a program that runs real-time TDDFT on this
library, over the sizes such programs use.

Every case is one call (or the pair of calls that a step makes) of a public
entry point on a mesh recipe of this repository: the harmonic trap, the
pseudopotential-like molecule on box cells, the graded molecule and the
all-electron-like molecule on trilinear cells.  Meshes keep the recipes' cell
sizes, so a mesh of fewer cells is a smaller box around fewer atoms.

A case's inputs (orbitals, well depths) come from its seed; the mesh comes
from the case.  ``exact`` evaluates the same quantity in plain torch FP64 with
a finite-element code of its own.
"""
import math

import numpy as np
import torch

from paper_1810_13130_amd import tdfe

MIXED = tdfe.MIXED_FP32


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def _case(call, mesh, p, ncell, n_orb, precision="f64", **kw):
    c = dict(call=call, mesh=mesh, p=p, nx=ncell[0], ny=ncell[1], nz=ncell[2], n_orb=n_orb, precision=precision,
             dt=0.05, tol=1e-10, steps=1, k_max=128, proj=0)
    c.update(kw)
    return c


def listed():
    return [
        # one Magnus step of one orbital in a trap: the smallest run, where
        # launches and the adaptive loop's host side are all there is
        dict(name="trap_step", **_case("step", "trap", 4, (4, 4, 4), 1)),
        # one application of H to the orbital block of the box workload, as a
        # program's own eigensolver or propagator calls it
        dict(name="box_apply_f64", **_case("apply", "box", 5, (16, 16, 16), 8)),
        # the FP32 operator on an odd mesh and an odd block
        dict(name="box_apply_f32_odd", **_case("apply", "box", 4, (13, 17, 11), 5, "mixed")),
        # H with the Kleinman-Bylander term of four atoms
        dict(name="box_nonlocal_f64", **_case("apply", "box", 5, (16, 16, 16), 8, proj=16)),
        # one exponential of a fixed Hamiltonian (frozen potential dynamics) in
        # the mixed precision that long runs use
        dict(name="box_expm_mixed", **_case("expm", "box", 5, (16, 16, 16), 8, "mixed")),
        # whole predictor-corrector steps with Hartree and exchange: a run's loop
        dict(name="box_propagate_f64", **_case("propagate", "box", 5, (16, 16, 16), 8, steps=2)),
        # the operator on the graded molecule, FP64 in the block of 8 orbitals
        # a Krylov chunk holds, and FP32 in its block of 16
        dict(name="graded_apply_f64", **_case("apply", "graded", 6, (31, 31, 31), 8)),
        dict(name="graded_apply_f32", **_case("apply", "graded", 6, (31, 31, 31), 16, "mixed")),
        # a full-step exponential on the graded molecule: where its runs spend
        # their time
        dict(name="graded_expm_f64", **_case("expm", "graded", 6, (24, 24, 24), 8, k_max=160)),
        # the same for all-electron wells: order 7, cells down to 0.02, short steps
        dict(name="ae_expm_mixed", **_case("expm", "ae", 7, (19, 20, 21), 8, "mixed", dt=0.005)),
        # the two evaluations of the density-dependent potential that a step
        # makes (midpoint, end of step), warm-started from each other
        dict(name="graded_scf_f64", **_case("scf", "graded", 6, (24, 24, 24), 16)),
        # field gradient of the dipole: a run forward and back
        dict(name="box_gradient_f64", **_case("gradient", "box", 5, (8, 8, 8), 4, steps=5, tol=1e-12, k_max=64)),
    ]


def _dim(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _mesh_dims(rng, lo, hi, most):
    while True:
        d = tuple(_dim(rng, lo, hi) for _ in range(3))
        if d[0] * d[1] * d[2] <= most:
            return d


def draw(rng):
    kind = rng.choice(["trap", "box_apply", "box_apply", "box_nonlocal", "box_expm", "box_propagate", "graded_apply",
                       "graded_apply", "graded_expm", "ae_expm", "graded_scf", "box_gradient"])
    prec = rng.choice(["f64", "mixed"])
    if kind == "trap":
        n = rng.randint(3, 8)
        return _case("step", "trap", rng.randint(3, 6), (n, rng.randint(3, 8), n), 1, prec)
    if kind == "box_apply":
        return _case("apply", "box", rng.randint(3, 7), _mesh_dims(rng, 6, 20, 4096), _dim(rng, 1, 16), prec)
    if kind == "box_nonlocal":
        return _case("apply", "box", rng.randint(3, 6), _mesh_dims(rng, 8, 17, 4096), rng.randint(1, 9),
                     proj=4 * rng.randint(1, 4))
    if kind == "box_expm":
        return _case("expm", "box", rng.randint(3, 6), _mesh_dims(rng, 6, 18, 4096), rng.randint(1, 9), prec)
    if kind == "box_propagate":
        return _case("propagate", "box", rng.randint(4, 6), _mesh_dims(rng, 6, 16, 4096), rng.randint(1, 9), prec,
                     steps=rng.randint(1, 2))
    if kind == "graded_apply":
        return _case("apply", "graded", rng.randint(4, 7), _mesh_dims(rng, 8, 26, 15000), _dim(rng, 1, 16), prec)
    if kind == "graded_expm":
        return _case("expm", "graded", rng.randint(4, 6), _mesh_dims(rng, 8, 20, 8000), rng.randint(1, 8), prec,
                     k_max=160)
    if kind == "ae_expm":
        return _case("expm", "ae", 7, _mesh_dims(rng, 10, 19, 5000), rng.randint(1, 8), "mixed", dt=0.005)
    if kind == "graded_scf":
        return _case("scf", "graded", rng.randint(4, 6), _mesh_dims(rng, 8, 20, 8000), _dim(rng, 1, 16))
    return _case("gradient", "box", rng.randint(3, 5), _mesh_dims(rng, 4, 8, 512), rng.randint(1, 4),
                 steps=rng.randint(2, 5), tol=1e-12, k_max=64)


# ---------------------------------------------------------------------------
# recipes: mesh, atoms, potential, orbitals, projectors
# ---------------------------------------------------------------------------
_SPACING = {"trap": 4.0, "box": 1.25, "graded": 32.0 / 31.0, "ae": 32.0 / 39.0}
_WIDTH = {"trap": 1.0, "box": 2.5, "graded": 3.0, "ae": 2.0}


def _shape(c):
    return c["nx"], c["ny"], c["nz"]


def _atoms(c):
    """Positions [n_atom, 3] (fixed by the case) and charges."""
    if c["mesh"] == "trap":
        return np.zeros((0, 3)), np.zeros(0)
    if c["proj"]:
        want = c["proj"] // 4
    else:
        want = {"box": 4, "graded": 16, "ae": 6}[c["mesh"]]
    half = np.array([0.5 * n * _SPACING[c["mesh"]] for n in _shape(c)])
    room = np.minimum({"box": 4.0, "graded": 5.0, "ae": 3.0}[c["mesh"]], half - 2.5 * _SPACING[c["mesh"]])
    rng = np.random.default_rng(11)
    R = []
    for _ in range(400):
        x = rng.uniform(-1.0, 1.0, 3) * room
        if len(R) < want and all(np.linalg.norm(x - y) >= 1.8 for y in R):
            R.append(x)
    while c["proj"] and len(R) < want:  # a projector set per atom, however close
        R.append(rng.uniform(-1.0, 1.0, 3) * room)
    kinds = {"box": (1.0, 4.0), "graded": (1.0, 4.0, 6.0), "ae": (6.0, 7.0, 8.0)}[c["mesh"]]
    return np.array(R), rng.choice(np.array(kinds), size=len(R))


def _vertices(c):
    """Vertices [nz+1, ny+1, nx+1, 3]; graded ones are drawn towards the atoms
    until every cell keeps its orientation."""
    h = _SPACING[c["mesh"]]
    ax = [h * (np.arange(n + 1) - 0.5 * n) for n in _shape(c)]
    Z, Y, X = np.meshgrid(ax[2], ax[1], ax[0], indexing="ij")
    V = np.stack([X, Y, Z], axis=-1)
    if c["mesh"] not in ("graded", "ae"):
        return V
    s, h_min = (1.5, 0.25) if c["mesh"] == "graded" else (1.0, 0.02)
    a = 1.0 - h_min / h
    pull = np.zeros_like(V)
    for r in _atoms(c)[0]:
        d = V - r
        pull += d * np.exp(-np.sum(d * d, axis=-1, keepdims=True) / s ** 2)
    # a window of the domain's faces keeps the outer boundary where it is
    lim = np.array([ax[0][-1], ax[1][-1], ax[2][-1]])
    pull *= np.prod(np.clip((lim - np.abs(V)) / (1.5 * h), 0.0, 1.0), axis=-1, keepdims=True)
    while True:
        W = V - a * pull
        ok = True
        for oz in (0, 1):
            for oy in (0, 1):
                for ox in (0, 1):
                    ex = W[oz:oz + c["nz"], oy:oy + c["ny"], 1:] - W[oz:oz + c["nz"], oy:oy + c["ny"], :-1]
                    ey = W[oz:oz + c["nz"], 1:, ox:ox + c["nx"]] - W[oz:oz + c["nz"], :-1, ox:ox + c["nx"]]
                    ez = W[1:, oy:oy + c["ny"], ox:ox + c["nx"]] - W[:-1, oy:oy + c["ny"], ox:ox + c["nx"]]
                    ok = ok and bool(np.all(np.sum(np.cross(ex, ey) * ez, axis=-1) > 0))
        if ok:
            return W
        a *= 0.97


def _potential(c, xyz, seed):
    """External potential at xyz [..., 3] (torch); well depths vary by a few
    per cent with the seed."""
    if c["mesh"] == "trap":
        g = 1.0 + 0.02 * np.random.default_rng([7, seed]).uniform(-1, 1)
        return 0.5 * g * (xyz * xyz).sum(-1)
    R, Z = _atoms(c)
    depth = Z * (1.0 + 0.03 * np.random.default_rng([7, seed]).uniform(-1, 1, len(Z)))
    v = torch.zeros(xyz.shape[:-1], dtype=xyz.dtype, device=xyz.device)
    for r, z in zip(R, depth):
        d2 = ((xyz - torch.as_tensor(r, dtype=xyz.dtype, device=xyz.device)) ** 2).sum(-1)
        v -= z / torch.sqrt(d2 + 1e-4) if c["mesh"] == "ae" else z * torch.exp(-2.0 * d2)
    return v


def _orbitals(c, xyz, mass, seed):
    """Orthonormal Loewdin coefficients [n_dof, n_orb]: plane waves under a
    Gaussian, with the phase of a small kick along z."""
    rng = np.random.default_rng([13, seed])
    env = torch.exp(-(xyz * xyz).sum(-1) / (2.0 * _WIDTH[c["mesh"]] ** 2)) * torch.sqrt(mass)
    X = torch.empty((len(xyz), c["n_orb"]), dtype=torch.float64, device=xyz.device)
    for al in range(c["n_orb"]):
        f = torch.full_like(env, 1.0 if c["mesh"] == "trap" else 0.0)
        for _ in range(6):
            k = rng.normal(size=3) * 0.6
            a = rng.normal() * (0.05 if c["mesh"] == "trap" else 1.0)
            f += a * torch.cos(xyz @ torch.as_tensor(k, device=xyz.device) + rng.uniform(0, 2 * math.pi))
        X[:, al] = env * f
    for _ in range(2):
        L = torch.linalg.cholesky(X.T @ X)
        X = torch.linalg.solve_triangular(L, X.T, upper=False).T.contiguous()
    return X * torch.exp(-0.02j * xyz[:, 2])[:, None]


def _projectors(c, xyz):
    """u_p, dV_p at the Gauss points [n_proj, n_quad]: s and p channels of each atom."""
    us, dvs = [], []
    for r in _atoms(c)[0][:c["proj"] // 4]:
        d = xyz - torch.as_tensor(r, dtype=xyz.dtype, device=xyz.device)
        r2 = (d * d).sum(-1)
        env, well = torch.exp(-r2 / (2 * 0.9 ** 2)), torch.exp(-r2 / (2 * 0.75 ** 2))
        for ch in range(4):
            us.append(env if ch == 0 else d[..., ch - 1] * env)
            dvs.append((-1.5 if ch == 0 else 0.8) * well)
    return torch.stack(us).reshape(len(us), -1).contiguous(), torch.stack(dvs).reshape(len(us), -1).contiguous()


def _xc(c):
    return tdfe.XC_XC if c["mesh"] in ("graded", "ae") else tdfe.XC_X


def _fields(c, seed):
    return np.random.default_rng([5, seed]).uniform(-1e-3, 1e-3, c["steps"])


# ---------------------------------------------------------------------------
# what a program holds, and one pass
# ---------------------------------------------------------------------------
class State:
    pass


def prepare(case, seed):
    c, s = case, State()
    s.case = c
    k_max = c["k_max"] if c["call"] in ("step", "expm", "propagate", "gradient") else 8
    s.ctx = tdfe.Context(c["p"], _shape(c), _vertices(c), n_orb_max=c["n_orb"], k_max=k_max,
                         precision=MIXED if c["precision"] == "mixed" else tdfe.FP64)
    xq = s.ctx.quad_coords()
    s.ctx.set_potential(_potential(c, xq, seed).contiguous())
    if c["proj"]:
        s.ctx.set_projectors(*_projectors(c, xq))
    if c["call"] in ("propagate", "scf", "gradient"):
        R, Z = _atoms(c)
        s.ctx.set_scf(hartree=True, xc=_xc(c), Z=Z, R=R, n_orb=c["n_orb"])
    xyz, mass = s.ctx.dof_coords(), s.ctx.mass_diag()
    s.psi = _orbitals(c, xyz, mass, seed).contiguous()
    if c["call"] == "apply":
        s.psi = _krylov_block(c, s.psi, seed)
        s.out = torch.zeros_like(s.psi)
    elif c["call"] == "scf":
        s.psi2 = _midpoint_state(s.psi, xyz)
        s.ctx.scf_fields(s.psi2)  # the potential of the instant before, which a run has
    elif c["call"] == "gradient":
        s.E = _fields(c, seed)
    return s


def _krylov_block(c, psi, seed):
    """The block that the operator is applied to: as the vectors of a Krylov
    space from the second on, it has the orbitals' extent and is rough."""
    g = torch.Generator(device=psi.device)
    g.manual_seed(int(seed))
    x = psi * torch.randn(psi.shape, generator=g, dtype=torch.float64, device=psi.device)
    return (x if c["precision"] == "f64" else x.to(torch.complex64)).contiguous()


def _kept(c, v):
    """What a run stores of a result: the FP32 paths' states and records hold
    FP32-accurate values, so a mixed run's snapshots are single precision."""
    if c["precision"] == "f64":
        return v
    if isinstance(v, np.ndarray):
        return v.astype(np.float32)
    return v.to(torch.complex64 if v.is_complex() else torch.float32)


def _midpoint_state(psi, xyz):
    """A state of slightly different density, as half a step makes it."""
    return (psi * torch.exp(0.01 * torch.sin(xyz[:, :1] + 0.3 * xyz[:, 1:2]))).contiguous()


def run(state):
    c, ctx = state.case, state.ctx
    if c["call"] == "apply":
        if c["precision"] == "mixed":
            return ctx.apply_H_add_f32(state.psi, state.out)
        return ctx.apply_H(state.psi, state.out)
    if c["call"] == "expm":
        ctx.lanczos_expm(state.psi, c["dt"], c["tol"])
        return _kept(c, state.psi)
    if c["call"] == "step":
        rep = ctx.magnus_step(state.psi, c["dt"], 0.0, c["tol"])
        return {"psi": _kept(c, state.psi), "moments": _kept(c, np.append(rep["mu"], rep["charge"]))}
    if c["call"] == "propagate":
        records, _ = ctx.propagate(state.psi, c["steps"], c["dt"], tol=c["tol"])
        return {"psi": _kept(c, state.psi), "records": _kept(c, records)}
    if c["call"] == "scf":
        phi1, w1 = ctx.scf_fields(state.psi)
        phi2, w2 = ctx.scf_fields(state.psi2)
        return {"phi1": phi1, "w1": w1, "phi2": phi2, "w2": w2}
    L, g = ctx.dipole_gradient(state.psi, state.E, c["dt"], tol=c["tol"])
    return {"mu": L, "gradient": g}


# ---------------------------------------------------------------------------
# the bytes and operations a pass cannot do without
# ---------------------------------------------------------------------------
def _sizes(c):
    cells = c["nx"] * c["ny"] * c["nz"]
    dof = (c["nx"] * c["p"] - 1) * (c["ny"] * c["p"] - 1) * (c["nz"] * c["p"] - 1)
    return cells, dof, cells * (c["p"] + 1) ** 3


def _apply_work(c, n_orb, real):
    cells, dof, quad = _sizes(c)
    n = c["p"] + 1
    geometry = cells * (24 if c["mesh"] in ("graded", "ae") else 4) * 8
    cols = 2 * n_orb
    return (dof * cols * real * 2 + (quad + dof) * real + geometry,
            cells * cols * (12 * n ** 4 + 14 * n ** 3))


# Krylov dimensions of the recipes at dt (larger cells, coarser orders need fewer)
_KRYLOV = {("trap", "f64"): 10, ("trap", "mixed"): 9, ("box", "f64"): 17, ("box", "mixed"): 12,
           ("graded", "f64"): 115, ("graded", "mixed"): 80, ("ae", "mixed"): 38, ("ae", "f64"): 45}


def _expm_work(c, k, real):
    """k operator products; per step the three-term recurrence reads two more
    vectors and writes one, and the sum at the end reads every basis vector."""
    _, dof, _ = _sizes(c)
    b, f = _apply_work(c, c["n_orb"], real)
    vec = dof * 2 * c["n_orb"] * real
    return k * (b + 4 * vec), k * (f + 14 * dof * 2 * c["n_orb"])


def _scf_work(c):
    """Density from the orbitals, one Poisson solve, the potential at the points."""
    cells, dof, quad = _sizes(c)
    n = c["p"] + 1
    its = 25 if c["mesh"] in ("graded", "ae") else 1
    b = dof * 2 * c["n_orb"] * 8 + 3 * quad * 8 + its * 8 * dof * 8
    f = cells * 2 * c["n_orb"] * (3 * n ** 4 + 3 * n ** 3) + its * (cells * 12 * n ** 4 + 12 * dof * round(dof ** (1 / 3)))
    return b, f


def work(case):
    c = case
    real = 4 if c["precision"] == "mixed" else 8
    k = _KRYLOV[c["mesh"], c["precision"]]
    if c["call"] == "apply":
        b, f = _apply_work(c, c["n_orb"], real)
        return {"bytes": b, "flops": f}
    if c["call"] in ("expm", "step"):
        b, f = _expm_work(c, k, real)
        return {"bytes": b, "flops": f}
    if c["call"] == "scf":
        b, f = _scf_work(c)
        return {"bytes": 2 * b, "flops": 2 * f}
    eb, ef = _expm_work(c, k, real)
    sb, sf = _scf_work(c)
    each = (1.7 * eb + 2 * sb, 1.7 * ef + 2 * sf)  # predictor over dt/2, corrector over dt, two potentials
    back = 3 if c["call"] == "gradient" else 1
    return {"bytes": back * c["steps"] * each[0], "flops": back * c["steps"] * each[1]}


# ---------------------------------------------------------------------------
# the same quantities in plain torch FP64
# ---------------------------------------------------------------------------
def _lagrange(nodes, x):
    V = np.ones((len(x), len(nodes)))
    D = np.zeros((len(x), len(nodes)))
    for i, xi in enumerate(nodes):
        others = [xm for m, xm in enumerate(nodes) if m != i]
        V[:, i] = np.prod([(x - xm) / (xi - xm) for xm in others], axis=0)
        for l in range(len(others)):
            term = np.ones(len(x)) / (xi - others[l])
            for m in range(len(others)):
                if m != l:
                    term = term * (x - others[m]) / (xi - others[m])
            D[:, i] += term
    return V, D


def _rules(p):
    P = np.polynomial.legendre.Legendre.basis(p)
    inner = np.sort(P.deriv().roots().real)
    for _ in range(3):
        inner = inner - P.deriv()(inner) / P.deriv(2)(inner)
    gll = np.concatenate([[-1.0], inner, [1.0]])
    wl = 2.0 / (p * (p + 1) * P(gll) ** 2)
    xg, wg = np.polynomial.legendre.leggauss(p + 1)
    B, D = _lagrange(gll, xg)
    return gll, wl, xg, wg, B, D


def _con(T, U, axis):
    """Contraction of the axis of U [E, C, z, y, x] (or without C) with T [out, in]."""
    return (U.movedim(axis, -1) @ T.T).movedim(-1, axis)


class Fem:
    """Spectral elements on trilinear cells: nodes, overlap, H, density, Poisson."""

    def __init__(self, c):
        self.dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
        t = lambda a: torch.as_tensor(np.ascontiguousarray(a), device=self.dev)  # noqa: E731
        p = self.p = c["p"]
        n = self.n = p + 1
        nx, ny, nz = _shape(c)
        V = _vertices(c)
        self.axes = [V[..., d].mean(axis=tuple(a for a in range(3) if a != 2 - d)) for d in range(3)]
        gll, wl, xg, wg, B, D = _rules(p)
        self.rule = (gll, xg, wg, B, D)
        self.B, self.D = t(B), t(D)
        V = t(V)
        corners = torch.stack([V[dz:dz + nz, dy:dy + ny, dx:dx + nx].reshape(-1, 3)
                               for dz in (0, 1) for dy in (0, 1) for dx in (0, 1)], 1)  # [E, 8, 3]
        self.E = len(corners)
        self.full = (nz * p + 1, ny * p + 1, nx * p + 1)
        ez, ey, ex = torch.meshgrid(*(torch.arange(m, device=self.dev) for m in (nz, ny, nx)), indexing="ij")
        k, j, i = torch.meshgrid(*(torch.arange(n, device=self.dev),) * 3, indexing="ij")
        node = lambda e, q: e.reshape(-1, 1, 1, 1) * p + q  # noqa: E731
        self.idx = (node(ex, i) + self.full[2] * (node(ey, j) + self.full[1] * node(ez, k))).reshape(-1)
        inside = torch.zeros(self.full, dtype=torch.bool, device=self.dev)
        inside[1:-1, 1:-1, 1:-1] = True
        self.dof = inside.reshape(-1).nonzero()[:, 0]
        self.n_nodes = inside.numel()
        xq, self.J = self._map(corners, xg)
        det = torch.linalg.det(self.J)
        w = t(np.einsum("c,b,a->cba", wg, wg, wg))
        self.wdet = w * det  # [E, z, y, x]
        self.xq = xq
        Ji = torch.linalg.inv(self.J)
        self.G = Ji @ Ji.transpose(-1, -2)
        del Ji, det
        xn, Jn = self._map(corners, gll)
        m = t(np.einsum("c,b,a->cba", wl, wl, wl)) * torch.linalg.det(Jn)
        self.mass = torch.zeros(self.n_nodes, dtype=torch.float64, device=self.dev).index_add_(0, self.idx, m.reshape(-1))
        self.xyz = torch.empty((self.n_nodes, 3), dtype=torch.float64, device=self.dev)
        self.xyz[self.idx] = xn.reshape(-1, 3)
        self.minv = 1.0 / torch.sqrt(self.mass[self.dof])
        del self.J

    def _map(self, corners, s):
        """Points [E, z, y, x, 3] and Jacobians d x_d / d xi_r of the tensor grid s."""
        f = np.stack([(1 - s) / 2, (1 + s) / 2], 1)
        g = np.stack([np.full_like(s, -0.5), np.full_like(s, 0.5)], 1)
        val = lambda a, b, c: torch.as_tensor(np.einsum("zu,yv,xw->zyxuvw", a, b, c).reshape(-1, 8), device=self.dev)  # noqa: E731
        sh = (len(corners), len(s), len(s), len(s))
        x = (val(f, f, f) @ corners).reshape(*sh, 3)
        J = torch.stack([val(f, f, g) @ corners, val(f, g, f) @ corners, val(g, f, f) @ corners], -1).reshape(*sh, 3, 3)
        return x, J

    # nodes [n_nodes, C] <-> cells [E, C, z, y, x]
    def cells(self, u):
        n = self.n
        return u[self.idx].reshape(self.E, n, n, n, -1).movedim(-1, 1)

    def nodes(self, y):
        y = y.movedim(1, -1).reshape(self.E * self.n ** 3, -1)
        return torch.zeros((self.n_nodes, y.shape[1]), dtype=torch.float64, device=self.dev).index_add_(0, self.idx, y)

    def values(self, u):
        U = self.cells(u)
        for a in (-1, -2, -3):
            U = _con(self.B, U, a)
        return U

    def test(self, f):
        """Integrals of f [E, C, z, y, x] (weights included) against every node's function."""
        for a in (-1, -2, -3):
            f = _con(self.B.T, f, a)
        return self.nodes(f)

    def form(self, u, vq, kin):
        """kin grad.grad + vq applied to nodal columns u [n_nodes, C]."""
        out = []
        for cols in u.split(4, 1):
            U = self.cells(cols)
            bx, dx = _con(self.B, U, -1), _con(self.D, U, -1)
            byx, dyx, bydx = _con(self.B, bx, -2), _con(self.D, bx, -2), _con(self.B, dx, -2)
            g = [_con(self.B, bydx, -3), _con(self.B, dyx, -3), _con(self.D, byx, -3)]
            val = _con(self.B, byx, -3) if vq is not None else None
            w = (kin * self.wdet)[:, None]
            f = [w * sum(self.G[..., d, r][:, None] * g[r] for r in range(3)) for d in range(3)]
            del g
            zx = _con(self.B.T, f[0], -3)
            zy = _con(self.B.T, f[1], -3)
            zz = _con(self.D.T, f[2], -3)
            if vq is not None:
                zz = zz + _con(self.B.T, (self.wdet * vq)[:, None] * val, -3)
            y = _con(self.D.T, _con(self.B.T, zx, -2), -1)
            y = y + _con(self.B.T, _con(self.D.T, zy, -2) + _con(self.B.T, zz, -2), -1)
            out.append(self.nodes(y))
        return torch.cat(out, 1)

    def spread(self, x):
        u = torch.zeros((self.n_nodes, x.shape[1]), dtype=torch.float64, device=self.dev)
        u[self.dof] = x
        return u

    def hbar(self, vq, psi, nl=None):
        x = torch.view_as_real(psi).reshape(len(psi), -1)
        y = self.minv[:, None] * self.form(self.spread(self.minv[:, None] * x), vq, 0.5)[self.dof]
        if nl is not None:
            y = y + nl[0].T @ ((nl[0] @ x) / nl[1][:, None])
        return torch.view_as_complex(y.reshape(len(psi), -1, 2).contiguous())

    def kb(self, u, dv):
        """M^-1/2 int u dV N_j [n_proj, n_dof] and int u dV u."""
        sh = (-1, self.E, self.n, self.n, self.n)
        f = (self.wdet * (u * dv).reshape(sh)).movedim(0, 1)
        D = (f.movedim(1, 0) * u.reshape(sh)).reshape(len(u), -1).sum(1)
        return (self.test(f)[self.dof] * self.minv[:, None]).T.contiguous(), D

    def density(self, psi):
        x = torch.view_as_real(psi).reshape(len(psi), -1) * self.minv[:, None]
        return sum((self.values(self.spread(cols)) ** 2).sum(1) for cols in x.split(4, 1))

    def _poisson_setup(self, c):
        """Boundary values and the 1D eigenvectors of the axis-averaged mesh."""
        R, Z = _atoms(c)
        f = torch.zeros(self.n_nodes, dtype=torch.float64, device=self.dev)
        for r, z in zip(R, Z):
            f += z / (self.xyz - torch.as_tensor(r, device=self.dev)).norm(dim=1)
        f[self.dof] = 0.0
        self.fb = f
        self.lift = self.form(f[:, None], None, 1.0)[self.dof, 0]
        self.ev, self.lam = [], []
        gll, xg, wg, B, D = self.rule
        for ax in self.axes:
            N = (len(ax) - 1) * self.p + 1
            K, M = np.zeros((N, N)), np.zeros((N, N))
            for e in range(len(ax) - 1):
                h = 0.5 * (ax[e + 1] - ax[e])
                s = slice(e * self.p, e * self.p + self.n)
                K[s, s] += D.T @ (wg[:, None] * D) / h
                M[s, s] += B.T @ (wg[:, None] * B) * h
            L = np.linalg.cholesky(M[1:-1, 1:-1])
            Li = np.linalg.inv(L)
            lam, Q = np.linalg.eigh(Li @ K[1:-1, 1:-1] @ Li.T)
            self.ev.append(torch.as_tensor(Li.T @ Q, device=self.dev))
            self.lam.append(torch.as_tensor(lam, device=self.dev))

    def _precondition(self, r):
        z, y, x = (s - 2 for s in self.full)
        t = r.reshape(z, y, x)
        for a, Q in ((2, self.ev[0]), (1, self.ev[1]), (0, self.ev[2])):
            t = _con(Q.T, t, a)
        t = t / (self.lam[2][:, None, None] + self.lam[1][:, None] + self.lam[0])
        for a, Q in ((2, self.ev[0]), (1, self.ev[1]), (0, self.ev[2])):
            t = _con(Q, t, a)
        return t.reshape(-1)

    def hartree(self, c, rho):
        if not hasattr(self, "fb"):
            self._poisson_setup(c)
        A = lambda v: self.form(self.spread(v[:, None]), None, 1.0)[self.dof, 0]  # noqa: E731
        b = 4 * math.pi * self.test((self.wdet * rho)[:, None])[self.dof, 0] - self.lift
        x = self._precondition(b)
        r = b - A(x)
        d = z = self._precondition(r)
        rz = r @ z
        for _ in range(200):
            if r.norm() <= 1e-14 * b.norm():
                break
            Ad = A(d)
            al = rz / (d @ Ad)
            x, r = x + al * d, r - al * Ad
            z = self._precondition(r)
            rz, old = r @ z, rz
            d = z + rz / old * d
        phi = self.fb.clone()
        phi[self.dof] = x
        return phi

    def w(self, c, psi):
        rho = self.density(psi)
        phi = self.hartree(c, rho)
        v = self.values(phi[:, None])[:, 0] - (3 * rho / math.pi) ** (1 / 3)
        if _xc(c) == tdfe.XC_XC:
            v = v + _pz81(rho)
        return phi, v, rho

    def expm(self, vq, psi, tau, tol, k_max):
        """Lanczos of every column to an error estimate far below the call's."""
        C = psi.shape[1]
        norm = psi.norm(dim=0)
        Q = [psi / norm]
        al, be = [], []
        for k in range(k_max):
            w = self.hbar(vq, Q[-1])
            a = (Q[-1].conj() * w).sum(0).real
            w = w - a * Q[-1]
            if k:
                w = w - be[-1] * Q[-2]
            al.append(a)
            b = w.norm(dim=0)
            T = torch.diag_embed(torch.stack(al, -1))
            if k:
                off = torch.stack(be, -1)
                T = T + torch.diag_embed(off, 1) + torch.diag_embed(off, -1)
            if k % 4 == 3 or k == k_max - 1:
                lam, U = torch.linalg.eigh(T.cpu())
                y = (U * torch.exp(-1j * tau * lam)[:, None, :]) @ U[:, 0, :, None].to(torch.complex128)
                y = y[..., 0].to(self.dev)
                if float((abs(tau) * b * norm * y[:, -1].abs()).max()) < tol or k == k_max - 1:
                    break
            be.append(b)
            Q.append(w / b)
        out = torch.zeros_like(psi)
        for q, yk in zip(Q, y.T):
            out += q * (yk * norm)
        return out

    def moments(self, rho):
        f = self.wdet * rho
        return torch.cat([f.sum()[None], (f[..., None] * self.xq).reshape(-1, 3).sum(0)])


def _pz81(rho):
    rho = rho.clamp_min(1e-300)
    rs = (3.0 / (4.0 * math.pi * rho)) ** (1 / 3)
    sq, ln = rs.sqrt(), rs.log()
    den = 1 + 1.0529 * sq + 0.3334 * rs
    hi = -0.1423 / den * (1 + 1.0529 * sq * 7 / 6 + 0.3334 * rs * 4 / 3) / den
    lo = 0.0311 * ln - 0.048 - 0.0311 / 3 + (2 / 3) * 0.0020 * rs * ln + (2 * -0.0116 - 0.0020) / 3 * rs
    return torch.where(rs >= 1, hi, lo)


def exact(case, seed):
    c = case
    if c["call"] == "gradient":
        return None  # reverse-mode derivatives of whole runs: over the time a plain evaluation may take
    fem = Fem(c)
    vq = _potential(c, fem.xq, seed)
    xyz = fem.xyz[fem.dof]
    psi = _orbitals(c, xyz, fem.mass[fem.dof], seed).contiguous()
    if c["call"] == "apply":
        nl = None
        if c["proj"]:
            nl = fem.kb(*_projectors(c, fem.xq))
        return fem.hbar(vq, _krylov_block(c, psi, seed).to(torch.complex128), nl)
    if c["call"] == "scf":
        phi1, w1, _ = fem.w(c, psi)
        phi2, w2, _ = fem.w(c, _midpoint_state(psi, xyz))
        sh = (fem.E, -1)
        return {"phi1": phi1, "w1": w1.reshape(sh), "phi2": phi2, "w2": w2.reshape(sh)}
    if c["call"] in ("expm", "step"):
        out = fem.expm(vq, psi, c["dt"], 1e-13, c["k_max"])
        if c["call"] == "expm":
            return out
        m = fem.moments(fem.density(out))
        return {"psi": out, "moments": torch.roll(m, -1).cpu().numpy()}
    w1 = w2 = fem.w(c, psi)[1]
    records = []
    for _ in range(c["steps"]):
        mid = fem.expm(vq + 1.25 * w1 - 0.25 * w2, psi, 0.5 * c["dt"], 1e-13, c["k_max"])
        psi = fem.expm(vq + fem.w(c, mid)[1], psi, c["dt"], 1e-13, c["k_max"])
        w2 = w1
        _, w1, rho = fem.w(c, psi)
        records.append(fem.moments(rho))
    return {"psi": psi, "records": torch.stack(records)}
