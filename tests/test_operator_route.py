"""Which operator kernel a launch runs on wide meshes and long rows (host only),
and the span of a block's cells that the choice rests on, against a walk over
every position of the block."""
import ctypes
import itertools
import os
import shutil
import subprocess

import numpy as np
import pytest

import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LINE, PLANE, PAIR, QUAD, FAR = 0, 1, 3, 4, 8
ADD, REPLACE, KRYLOV = 16, 32, 64  # through the cell buffer


@pytest.fixture(scope="module")
def lib():
    from paper_1810_13130_amd import tdfe
    if not os.path.exists(tdfe.LIB_PATH):
        pytest.skip("libtdfe.so not built")
    return tdfe.load()


def _route(lib, mesh, p, nc, n_orb, fp32, variant=None, monkeypatch=None):
    from paper_1810_13130_amd import tdfe
    d = tdfe.MeshDesc()
    d.p, d.nq, d.n_orb_max, d.k_max, d.precision = p, p + 1, n_orb, 4, 1 if fp32 else 0
    d.ncell[0], d.ncell[1], d.ncell[2] = nc
    v = np.ascontiguousarray(W.box_vertices(-1.0, 1.0, nc))
    if mesh == "trilinear":
        v[1, 1, 1] += 0.1 / max(nc)
    d.vertices = v.ctypes.data_as(tdfe._DP)
    h = ctypes.c_void_p()
    assert lib.tdfe_fe_mesh_setup(ctypes.byref(d), None, ctypes.byref(h)) == 0
    r = lib.tdfe_operator_route(h, 2 * n_orb, int(fp32))
    lib.tdfe_destroy(h)
    return r


@pytest.mark.parametrize("mesh,p,nc,n_orb,fp32,want", [
    ("box", 5, (16, 16, 16), 8, False, PAIR + REPLACE + KRYLOV),
    # 32 columns of 20,000 rows and more across a block's z planes
    ("box", 5, (96, 96, 2), 32, False, PAIR), ("box", 5, (120, 120, 2), 32, False, PAIR),
    ("box", 5, (190, 190, 2), 32, False, PAIR + FAR), ("box", 4, (240, 240, 2), 32, True, PLANE),
    ("box", 4, (400, 400, 2), 32, True, PLANE + FAR),
    # rows of hundreds of orbitals
    ("box", 5, (24, 24, 24), 512, False, PAIR), ("box", 5, (48, 48, 4), 512, False, PAIR + FAR),
    ("box", 4, (24, 24, 2), 4096, False, PLANE + FAR), ("box", 6, (8, 8, 2), 4096, False, QUAD),
    # the four-lane kernel has an address per row of nodes
    ("box", 6, (160, 160, 2), 32, False, QUAD), ("trilinear", 6, (160, 160, 2), 32, False, QUAD),
    ("trilinear", 7, (120, 120, 2), 32, True, PAIR), ("trilinear", 7, (160, 160, 2), 32, True, QUAD),
    ("trilinear", 5, (100, 100, 2), 32, False, PAIR), ("trilinear", 5, (190, 190, 2), 32, False, LINE),
    ("trilinear", 6, (160, 160, 2), 32, True, PLANE), ("box", 8, (4, 4, 4), 8, False, LINE)])
def test_route(lib, mesh, p, nc, n_orb, fp32, want):
    assert _route(lib, mesh, p, nc, n_orb, fp32) == want


@pytest.mark.parametrize("p,pairs", [(1, 1), (2, 4), (3, 2), (4, 2), (5, 16), (6, 4), (7, 4)])
def test_trilinear_fp64_kernel_by_columns(lib, p, pairs):
    """Lane pairs up to so many orbitals; from nine columns on the four-lane
    kernel at p = 6 and 7, planes else."""
    for n_orb in (1, 2, 3, 4, 5, 9, 16):
        want = PAIR if n_orb <= pairs else QUAD if p > 5 else PLANE
        assert _route(lib, "trilinear", p, (7, 6, 5), n_orb, False) & 7 == want, n_orb


# where apply_H_add, apply_H and the Krylov update go through the cell buffer:
# not in launches of microseconds, nor where the atomics hide
@pytest.mark.parametrize("mesh,p,nc,n_orb,fp32,want", [
    ("box", 3, (6, 5, 7), 8, False, KRYLOV), ("box", 1, (17, 16, 18), 8, False, KRYLOV),
    ("box", 1, (98, 97, 99), 1, False, 0), ("box", 5, (20, 19, 21), 1, False, ADD + REPLACE + KRYLOV),
    ("box", 5, (20, 19, 21), 5, False, ADD + REPLACE + KRYLOV), ("box", 5, (16, 16, 16), 32, False, REPLACE),
    ("box", 6, (16, 15, 17), 8, False, KRYLOV), ("box", 6, (7, 6, 8), 16, False, REPLACE + KRYLOV),
    ("box", 7, (14, 13, 15), 8, False, REPLACE + KRYLOV), ("box", 5, (8, 7, 9), 8, True, KRYLOV),
    ("box", 4, (13, 17, 11), 5, True, ADD + KRYLOV), ("box", 5, (20, 19, 21), 8, True, ADD + KRYLOV),
    ("box", 5, (20, 19, 21), 16, True, KRYLOV), ("trilinear", 3, (6, 5, 7), 1, False, KRYLOV),
    ("trilinear", 5, (20, 19, 21), 1, False, ADD + REPLACE + KRYLOV), ("trilinear", 5, (20, 19, 21), 8, False, KRYLOV),
    ("trilinear", 2, (49, 48, 50), 1, False, 0), ("trilinear", 7, (14, 13, 15), 8, False, REPLACE + KRYLOV),
    ("trilinear", 4, (24, 23, 25), 9, True, ADD + KRYLOV), ("trilinear", 4, (24, 23, 25), 8, True, KRYLOV),
    ("box", 1, (40, 39, 41), 9, False, ADD + REPLACE + KRYLOV), ("box", 1, (40, 39, 41), 1, False, 0),
    ("trilinear", 1, (40, 39, 41), 13, True, KRYLOV), ("trilinear", 2, (20, 19, 21), 1, True, KRYLOV),
    ("trilinear", 2, (49, 48, 50), 1, True, 0), ("trilinear", 2, (49, 48, 50), 3, True, ADD),
    ("box", 2, (49, 48, 50), 13, True, ADD), ("box", 3, (22, 21, 23), 2, False, ADD + REPLACE + KRYLOV)])
def test_cell_buffer(lib, mesh, p, nc, n_orb, fp32, want):
    r = _route(lib, mesh, p, nc, n_orb, fp32)
    assert r & (ADD if fp32 else ADD + REPLACE) == want & (ADD + REPLACE)
    assert r & KRYLOV == want & KRYLOV


def test_trilinear_fp32_kernel_by_columns(lib):
    """p = 7: four lanes where a block of 16 columns is not full, else pairs;
    below planes."""
    for p in range(1, 8):
        for n_orb in (1, 4, 5, 7, 8, 9, 16, 32):
            want = PLANE if p < 7 else QUAD if 4 < n_orb < 8 else PAIR
            assert _route(lib, "trilinear", p, (7, 6, 5), n_orb, True) & 7 == want, (p, n_orb)


def test_block_span(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    src = tmp_path / "span.cpp"
    src.write_text('#include "tdfe_span.h"\n'
                   'extern "C" long long rows(int p, int x, int y, int z, int cells) {\n'
                   '  return tdfe_span::block_rows(p, x, y, z, cells);\n}\n')
    out = tmp_path / "span.so"
    subprocess.check_call(["g++", "-std=c++17", "-shared", "-fPIC", "-I",
                           os.path.join(ROOT, "paper_1810_13130_amd", "csrc"), str(src), "-o", str(out)])
    f = ctypes.CDLL(str(out)).rows
    f.restype = ctypes.c_longlong
    for p, (ncx, ncy, ncz) in itertools.product((1, 2, 5), itertools.product((1, 2, 3, 5), (1, 2, 4), (1, 2, 3, 7))):
        nx, ny = ncx * p - 1, ncy * p - 1
        c = np.arange(ncx * ncy * ncz)
        row = p * ((c % ncx) + nx * ((c // ncx) % ncy) + nx * ny * (c // (ncx * ncy)))
        for cells in (1, 2, 3, 7, 16, 32):
            most = max(int(row[i:i + cells].max() - row[i]) for i in c)
            got = f(p, ncx, ncy, ncz, cells)
            assert got == most + p * (nx * ny + nx + 1), (p, ncx, ncy, ncz, cells)
