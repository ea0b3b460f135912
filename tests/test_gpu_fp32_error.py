"""How far one FP32 application of the operator is from the oracle.

A rounding errs by 0.41 x 2^-24 of its value in the root mean square.  What a
rough vector's values go through one after the other is some 17 of them in the
scales and sums of a cell and n / 2 + 2 in each of seven contractions; they add up
in squares, and rounded coefficients, the same on every cell, must not add to
them: 5% on top.
"""
import numpy as np
import pytest

import workloads as W
from gpu_util import gpu_context, oracle_mesh
from oracle import operators as op

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mesh,p,n_orb", [("box", 2, 3), ("box", 3, 4), ("box", 4, 5), ("box", 5, 2), ("box", 5, 6),
                                          ("box", 6, 1), ("box", 6, 9), ("box", 7, 3), ("box", 7, 8)])
def test_fp32_operator_error(mesh, p, n_orb):
    err = _error(mesh, p, n_orb)
    bar = 1.05 * 0.41 * 2.0 ** -24 * np.sqrt(17 + 7 * ((p + 1) // 2 + 2))
    print(f"[fp32 operator] {mesh} p={p} n_orb={n_orb} {err:.3e} of {bar:.3e}", flush=True)
    assert err < bar


@pytest.mark.parametrize("n_orb", [5, 7])
def test_fp32_four_lanes_as_exact_as_lane_pairs(n_orb, monkeypatch):
    """p = 7, trilinear cells, 9 to 15 columns: the same contractions of the
    same values by two kernels, so the same error, but for 5%."""
    err = _error("graded", 7, n_orb)
    monkeypatch.setenv("TDFE_APPLY_VARIANT", "pair")
    pairs = _error("graded", 7, n_orb)
    print(f"[fp32 operator] p=7 n_orb={n_orb} four lanes {err:.3e}, pairs {pairs:.3e}", flush=True)
    assert err < 1.05 * pairs


def _error(mesh, p, n_orb):
    cfg = W.scaled(W.CONFIGS[2 if mesh == "box" else 3], ncell=(9, 8, 10) if p < 6 else (7, 6, 7), p=p, n_orb=n_orb)
    ctx = gpu_context(cfg, n_orb=n_orb, k_max=4, precision=1)
    m, vq = oracle_mesh(cfg)
    x = W.random_block(m.n_dof, n_orb, 70 + p).astype(np.complex64)
    y = torch.zeros((m.n_dof, n_orb), dtype=torch.complex64, device="cuda")
    ctx.apply_H_add_f32(torch.from_numpy(x).cuda(), y)
    ref = op.apply_Hbar(m, vq, x.astype(np.complex128))
    ctx.close()
    return np.linalg.norm(y.cpu().numpy() - ref) / np.linalg.norm(ref)
