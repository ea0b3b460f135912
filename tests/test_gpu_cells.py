"""The operator's two output forms and the four-lane kernel against the oracle.

Per-cell results (summed by their consumer) and the atomic scatter are the
same operator: TDFE_CELL_BUFFER_BYTES = 0 forces the scatter, a small value
makes a launch go through the cell buffer in slices of 16 columns.  Column
counts sit at and around the 16-column passes of the four-lane kernel (p = 6
FP64, p = 7) and below the 9 columns it starts at.  Bars: 1e-12 (FP64) and
2e-6 (FP32) relative, as for every operator kernel here; 1e-10 for the
exponential.
"""
import numpy as np
import pytest

import workloads as W
from gpu_util import gpu_context, oracle_mesh, rel
from oracle import lanczos, operators as op

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MESH = {"box": 2, "graded": 3}


def _cfg(mesh, p, n_orb, nc=(3, 2, 3)):
    return W.scaled(W.CONFIGS[MESH[mesh]], ncell=nc, p=p, n_orb=n_orb)


def _cap(monkeypatch, cfg, cap):
    """None: as shipped; "scatter": no buffer; "slices": 16 FP64 columns fit."""
    if cap == "scatter":
        monkeypatch.setenv("TDFE_CELL_BUFFER_BYTES", "0")
    elif cap == "slices":
        monkeypatch.setenv("TDFE_CELL_BUFFER_BYTES", str(int(np.prod(cfg.ncell)) * (cfg.p + 1) ** 3 * 16 * 8))


@pytest.mark.parametrize("cap", [None, "scatter", "slices"])
@pytest.mark.parametrize("mesh,p,n_orb", [("box", 6, 5), ("box", 7, 8), ("graded", 6, 8), ("graded", 6, 9),
                                          ("graded", 7, 17), ("box", 5, 19), ("graded", 4, 3), ("box", 1, 1),
                                          ("box", 2, 1), ("box", 4, 1), ("box", 4, 2), ("box", 6, 2)])
def test_operator_output_forms(mesh, p, n_orb, cap, monkeypatch):
    cfg = _cfg(mesh, p, n_orb)
    _cap(monkeypatch, cfg, cap)
    ctx = gpu_context(cfg, n_orb=n_orb, k_max=4)
    m, vq = oracle_mesh(cfg)
    x = W.random_block(m.n_dof, n_orb, 60 + p)
    ref = op.apply_Hbar(m, vq, x)
    xd = torch.from_numpy(x).cuda()
    assert rel(ctx.apply_H(xd).cpu().numpy(), ref) < 1e-12
    y0 = W.random_block(m.n_dof, n_orb, 61)
    y = torch.from_numpy(y0).cuda()
    ctx.apply_H_add(xd, y)
    assert np.abs(y.cpu().numpy() - y0 - ref).max() < 1e-12 * max(np.abs(ref).max(), np.abs(y0).max())
    ctx.close()


@pytest.mark.parametrize("cap", [None, "scatter"])
@pytest.mark.parametrize("mesh,p,n_orb", [("box", 7, 7), ("graded", 7, 9), ("graded", 6, 6), ("box", 5, 3),
                                          ("box", 3, 1), ("box", 5, 2)])
def test_fp32_operator_output_forms(mesh, p, n_orb, cap, monkeypatch):
    cfg = _cfg(mesh, p, n_orb)
    _cap(monkeypatch, cfg, cap)
    ctx = gpu_context(cfg, n_orb=n_orb, k_max=4, precision=1)
    m, vq = oracle_mesh(cfg)
    x = W.random_block(m.n_dof, n_orb, 70 + p)
    y = torch.zeros((m.n_dof, n_orb), dtype=torch.complex64, device="cuda")
    ctx.apply_H_add_f32(torch.from_numpy(x.astype(np.complex64)).cuda(), y)
    assert rel(y.cpu().numpy(), op.apply_Hbar(m, vq, x)) < 2e-6
    ctx.close()


@pytest.mark.parametrize("cap", [None, "scatter"])
@pytest.mark.parametrize("mesh,p,n_orb", [("box", 3, 1), ("box", 6, 6), ("graded", 6, 8), ("graded", 7, 5)])
def test_exponential_with_both_output_forms(mesh, p, n_orb, cap, monkeypatch):
    cfg = _cfg(mesh, p, n_orb, nc=(3, 3, 2))
    _cap(monkeypatch, cfg, cap)
    ctx = gpu_context(cfg, n_orb=n_orb, k_max=96)
    m, vq = oracle_mesh(cfg)
    x = W.random_block(m.n_dof, n_orb, 80 + p)
    x /= np.linalg.norm(x, axis=0)
    psi = torch.from_numpy(x).cuda()
    ctx.lanczos_expm(psi, 0.02, 1e-12)
    ref = lanczos.lanczos_expm(lambda z: op.apply_Hbar(m, vq, z), x, 0.02, 1e-12, 96)
    ref = ref[0] if isinstance(ref, tuple) else ref
    assert np.abs(psi.cpu().numpy() - ref).max() < 1e-10
    ctx.close()


@pytest.mark.parametrize("p", [1, 2, 4, 5, 7, 8])
def test_one_column_stiffness_on_curved_cells(p):
    """The Hartree solve's stiffness products (one column, full grid) at each
    order: CG to a relative residual of 1e-13 against the oracle's; the bar
    allows for a condition number of 1e3."""
    from oracle import scf
    cfg = _cfg("graded", p, 1)
    ctx = gpu_context(cfg, n_orb=1, k_max=4)
    Z, R = W.atoms(cfg)
    ctx.set_scf(hartree=True, Z=Z, R=R, n_orb=1, pcg_tol=1e-13)
    m, _ = oracle_mesh(cfg)
    x = W.random_block(m.n_dof, 1, 90 + p) * 1e-2
    phi, _ = ctx.scf_fields(torch.from_numpy(x).cuda(), w=False)
    ref, _ = scf.Hartree(m, Z, R, tol=1e-13).solve(scf.density(m, x))
    assert rel(phi.cpu().numpy(), ref) < 1e-10
    ctx.close()


@pytest.mark.parametrize("p,n_orb", [(2, 1), (3, 2), (4, 3), (5, 2), (6, 1), (6, 5), (7, 3), (7, 5)])
def test_fp32_exponential_of_smooth_orbitals(p, n_orb):
    """The rounding of the FP32 stiffness entries is the same on every cell, so
    a smooth orbital sums it up over the series; rounded together they must
    not add to the storage rounding: 2^-24 sqrt(k) of some 12 iterations, 2.1e-7
    in the 2-norm, with half as much again."""
    cfg = W.scaled(W.CONFIGS[2], ncell=(8, 8, 8), p=p, n_orb=n_orb)
    ctx = gpu_context(cfg, n_orb=n_orb, k_max=64, precision=1)
    m, vq = oracle_mesh(cfg)
    x = W.initial_psibar(cfg, m.dof_xyz, m.M)[:, :n_orb]
    psi = torch.from_numpy(np.ascontiguousarray(x)).cuda()
    ctx.lanczos_expm(psi, 0.05, 1e-12)
    ref = lanczos.lanczos_expm(lambda z: op.apply_Hbar(m, vq, z), x, 0.05, 1e-12, 64)[0]
    err = np.linalg.norm(psi.cpu().numpy() - ref) / np.linalg.norm(ref)
    print(f"[fp32 exponential] p={p} n_orb={n_orb} {err:.2e}", flush=True)
    assert err < 3.2e-7
    ctx.close()
