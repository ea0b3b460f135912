"""Launches that go through the cell buffer in column slices, with a last slice
narrower than its column block, against the oracle.

TDFE_CELL_BUFFER_BYTES leaves room for 16 columns, so 16 + 6, 16 + 10 and 16 +
14 columns end in blocks of 8 and 16 columns whose last lanes hold none.  Bars:
1e-12 (FP64) and 2e-6 (FP32) relative, as for every operator kernel here.
"""
import numpy as np
import pytest

import workloads as W
from gpu_util import gpu_context, oracle_mesh, rel
from oracle import operators as op

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

MESH = {"box": 2, "graded": 3}


def _context(monkeypatch, mesh, p, n_orb, size, **kw):
    cfg = W.scaled(W.CONFIGS[MESH[mesh]], ncell=(3, 2, 3), p=p, n_orb=n_orb)
    monkeypatch.setenv("TDFE_CELL_BUFFER_BYTES", str(int(np.prod(cfg.ncell)) * (p + 1) ** 3 * 16 * size))
    return gpu_context(cfg, n_orb=n_orb, k_max=4, **kw), *oracle_mesh(cfg)


@pytest.mark.parametrize("mesh,p,n_orb", [("graded", 4, 11), ("graded", 5, 13), ("graded", 3, 15), ("graded", 6, 13),
                                          ("box", 5, 13), ("box", 4, 15)])
def test_ragged_last_slice(mesh, p, n_orb, monkeypatch):
    ctx, m, vq = _context(monkeypatch, mesh, p, n_orb, 8)
    x = W.random_block(m.n_dof, n_orb, 40 + p)
    ref = op.apply_Hbar(m, vq, x)
    xd = torch.from_numpy(x).cuda()
    assert rel(ctx.apply_H(xd).cpu().numpy(), ref) < 1e-12
    y0 = W.random_block(m.n_dof, n_orb, 41)
    y = torch.from_numpy(y0).cuda()
    ctx.apply_H_add(xd, y)
    assert np.abs(y.cpu().numpy() - y0 - ref).max() < 1e-12 * max(np.abs(ref).max(), np.abs(y0).max())
    ctx.close()


@pytest.mark.parametrize("mesh,p,n_orb", [("box", 4, 11), ("box", 5, 10), ("graded", 6, 13), ("graded", 4, 10),
                                          ("graded", 7, 11)])
def test_fp32_slices(mesh, p, n_orb, monkeypatch):
    ctx, m, vq = _context(monkeypatch, mesh, p, n_orb, 4, precision=1)
    x = W.random_block(m.n_dof, n_orb, 50 + p)
    y0 = W.random_block(m.n_dof, n_orb, 51)
    y = torch.from_numpy(y0.astype(np.complex64)).cuda()
    ctx.apply_H_add_f32(torch.from_numpy(x.astype(np.complex64)).cuda(), y)
    assert rel(y.cpu().numpy(), y0 + op.apply_Hbar(m, vq, x)) < 2e-6
    ctx.close()
