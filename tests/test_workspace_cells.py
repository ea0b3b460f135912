"""Device memory that a context asks for (host only): the buffer of per-cell
operator results is there only where an operator kernel writes them."""
import ctypes
import os

import numpy as np
import pytest

import workloads as W


@pytest.fixture(scope="module")
def lib():
    from paper_1810_13130_amd import tdfe
    if not os.path.exists(tdfe.LIB_PATH):
        pytest.skip("libtdfe.so not built")
    return tdfe.load()


def _bytes(lib, p, precision):
    from paper_1810_13130_amd import tdfe
    d = tdfe.MeshDesc()
    nc = (6, 5, 4)
    d.p, d.nq, d.n_orb_max, d.k_max, d.precision = p, p + 1, 4, 8, precision
    d.ncell[0], d.ncell[1], d.ncell[2] = nc
    v = np.ascontiguousarray(W.box_vertices(-1.0, 1.0, nc))
    d.vertices = v.ctypes.data_as(tdfe._DP)
    h = ctypes.c_void_p()
    assert lib.tdfe_fe_mesh_setup(ctypes.byref(d), None, ctypes.byref(h)) == 0
    b = ctypes.c_size_t()
    q = [ctypes.c_int64() for _ in range(3)]
    assert lib.tdfe_query(h, *(ctypes.byref(x) for x in q), ctypes.byref(b)) == 0
    lib.tdfe_destroy(h)
    return b.value


# p, precision, variant of the operator, whether per-cell results are used
@pytest.mark.parametrize("p,precision,variant,used", [(5, 0, None, True), (5, 1, None, True), (5, 2, None, False),
                                                      (5, 3, None, False), (5, 4, None, False), (8, 0, None, False),
                                                      (5, 0, "line", False)])
def test_cell_buffer_only_where_used(lib, p, precision, variant, used, monkeypatch):
    if variant:
        monkeypatch.setenv("TDFE_APPLY_VARIANT", variant)
    full = _bytes(lib, p, precision)
    monkeypatch.setenv("TDFE_CELL_BUFFER_BYTES", "0")
    assert (full > _bytes(lib, p, precision)) == used
