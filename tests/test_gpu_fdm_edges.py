"""The fast diagonalisation's transforms at the edges of their tiles: axes of
1, of 16 m - 1, 16 m and 16 m + 1 interior nodes, lines that do not fill a
block, and the longest axis of the line kernel beside one that goes to the
library.  The exact solve on box meshes and the preconditioned CG on curved
ones against the oracle's CG at a relative residual of 1e-13; the bar allows
for a condition number of 1e3, as for every Hartree solve here.
"""
import numpy as np
import pytest

import workloads as W
from gpu_util import gpu_context, oracle_mesh, rel

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mesh,p,nc", [("box", 1, (16, 17, 18)), ("box", 2, (16, 17, 9)), ("box", 1, (2, 3, 33)),
                                       ("box", 1, (34, 2, 2)), ("box", 1, (129, 2, 4)), ("box", 1, (3, 130, 4)),
                                       ("box", 1, (4, 3, 130)), ("graded", 1, (18, 16, 17)),
                                       ("graded", 2, (8, 17, 16)), ("graded", 1, (3, 4, 130)),
                                       ("graded", 1, (130, 3, 4)), ("graded", 1, (4, 129, 3))])
def test_transform_edges(mesh, p, nc):
    from oracle import scf
    cfg = W.scaled(W.CONFIGS[2 if mesh == "box" else 3], ncell=nc, p=p, n_orb=1)
    ctx = gpu_context(cfg, n_orb=1, k_max=4)
    Z, R = W.atoms(cfg)
    ctx.set_scf(hartree=True, Z=Z, R=R, n_orb=1, pcg_tol=1e-13)
    m, _ = oracle_mesh(cfg)
    x = W.random_block(m.n_dof, 1, 90 + p) * 1e-2
    phi, _ = ctx.scf_fields(torch.from_numpy(x).cuda(), w=False)
    ref, _ = scf.Hartree(m, Z, R, tol=1e-13).solve(scf.density(m, x))
    print(f"[fdm edges] {mesh} p={p} {nc} {rel(phi.cpu().numpy(), ref):.2e}", flush=True)
    assert rel(phi.cpu().numpy(), ref) < 1e-10
    ctx.close()
