"""The small exponential at the edges of its table and of its row layouts.

|tau| r (r the Gershgorin half-width) runs over the smallest series (a start
of the backward recurrence that grows by 1e21 a step, and the limit below it
where J_1 = z / 2 is all there is), over 64 terms, over the start at 128 from
which the Bessel table lies in memory, and k over the rows per lane.  y has
unit norm; the series adds at most a few hundred rounded terms of size one, so
the bar is 1e-12 absolute.  The Lanczos iteration takes the same series beside
its update up to k = 256 and in a kernel of its own beyond: one call of tau
against two of tau / 2, whose Krylov dimensions lie in other ranges, to the
sum of their tolerances and of the rounding of some 300 iterations, 1e-9.
"""
import numpy as np
import pytest

import workloads as W
from gpu_util import gpu_context, oracle_mesh, rel
from oracle.lanczos import tridiag_expm_e1

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2, 63, 64, 65, 128, 129, 200, 256, 257])
@pytest.mark.parametrize("tau_r", [1e-30, 1.1e-20, 1e-8, 0.03, 1.0, 9.0, 17.3, 18.0, 55.0, 55.9, 57.0, 300.0])
def test_small_exponential_edges(k, tau_r):
    from paper_1810_13130_amd import tdfe
    rng = np.random.default_rng(k)
    a, b = rng.uniform(-1.0, 1.0, k), rng.uniform(0.05, 1.0, k - 1)
    rad = np.zeros(k)
    rad[:-1] += b
    rad[1:] += b
    r = 0.5 * ((a + rad).max() - (a - rad).min())
    tau = -0.05 if k % 2 else 0.05
    s = tau_r / (abs(tau) * (r if r > 0 else 1.0))
    y, terms = tdfe.tridiag_expm(a * s, b * s, tau)
    assert terms == (int(np.ceil(tau_r + 10 * np.cbrt(tau_r) + 20)) if k > 1 else 0)
    assert np.abs(y - tridiag_expm_e1(a * s, b * s, tau)).max() <= 1e-12


@pytest.mark.parametrize("tau,kmin,kmax", [(60.0, 65, 128), (160.0, 129, 256), (300.0, 257, 500)])
def test_lanczos_over_the_row_layouts(tau, kmin, kmax):
    cfg = W.scaled(W.CONFIGS[3], ncell=(3, 3, 3), p=4, n_orb=3)
    ctx = gpu_context(cfg, n_orb=3, k_max=500)
    m, _ = oracle_mesh(cfg)
    x = W.random_block(m.n_dof, 3, 5)
    one, two = torch.from_numpy(x).cuda(), torch.from_numpy(x).cuda()
    ks, _ = ctx.lanczos_expm(one, tau, 1e-10)
    for _ in range(2):
        kh, _ = ctx.lanczos_expm(two, tau / 2, 1e-10)
    print(f"[small-exp] tau={tau} k={ks} half={kh}", flush=True)
    assert kmin <= max(ks) <= kmax
    assert rel(one.cpu().numpy(), two.cpu().numpy()) < 1e-9
    ctx.close()
