"""The box kernels with 64-bit offsets (rows of thousands of columns, or layers
of millions of nodes) against the line kernel on the same inputs.  Each is
within 1e-12 (FP64) or 2e-6 (FP32) of the oracle at ordinary sizes, so they
agree to twice that."""
import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

FAR = 8


# p, cells, orbitals: just past the reach of 32 bits
@pytest.mark.parametrize("p,nc,n_orb,fp32", [(1, (182, 182, 2), 4096, False), (2, (66, 66, 2), 4000, False),
                                             (3, (40, 40, 1), 4096, False), (4, (24, 24, 1), 4091, False),
                                             (5, (18, 18, 1), 4096, False), (7, (316, 316, 1), 4, False),
                                             (2, (92, 92, 1), 4096, True), (4, (34, 34, 1), 4096, True),
                                             (5, (24, 24, 1), 4090, True), (6, (18, 18, 1), 4096, True)])
def test_far_offsets(p, nc, n_orb, fp32, monkeypatch):
    from paper_1810_13130_amd import tdfe
    V = W.box_vertices(-1.0, 1.0, nc) * (np.arange(3) * 0.3 + 1.0)
    g = torch.Generator(device="cuda")
    g.manual_seed(p)
    x = y = v = None
    for variant in (None, "line"):
        if variant:
            monkeypatch.setenv("TDFE_APPLY_VARIANT", variant)
        ctx = tdfe.Context(p, nc, V, n_orb_max=n_orb, k_max=2, precision=int(fp32))
        if not variant:
            assert ctx.lib.tdfe_operator_route(ctx.h, 2 * n_orb, int(fp32)) & FAR
            dt = torch.complex64 if fp32 else torch.complex128
            x = torch.randn((ctx.n_dof, n_orb), generator=g, dtype=dt, device="cuda")
            v = torch.randn((ctx.n_cell, (p + 1) ** 3), generator=g, dtype=torch.float64, device="cuda")
        ctx.set_potential(v)
        out = torch.zeros_like(x)
        ctx.apply_H_add_f32(x, out) if fp32 else ctx.apply_H_add(x, out)
        ctx.close()
        if variant:
            scale = float(out.abs().max())
            assert float((y - out).abs().max()) < (4e-6 if fp32 else 2e-12) * scale
        y = out
