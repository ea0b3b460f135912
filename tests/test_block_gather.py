"""Which bytes the operator's block kernels read, lane by lane, on the host.

The kernels gather through a buffer resource that ends with the last DoF row,
`ld` columns wide from where the launch's columns begin.  A launch on some
columns of a wider vector begins part of a row in, so the resource reaches past
the vector; the lanes of the last column block that hold no column must then
not read at all.
"""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1810_13130_amd", "csrc")


@pytest.fixture(scope="module")
def span(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("span")
    src = d / "span.cpp"
    src.write_text('#include "tdfe_span.h"\n'
                   'extern "C" long long gather_offset(int act, long long rows, int ld, int colg, int size) {\n'
                   '  return tdfe_span::gather_offset(act != 0, rows, ld, colg, size);\n}\n')
    lib = d / "span.so"
    subprocess.check_call(["g++", "-std=c++17", "-shared", "-fPIC", "-I", CSRC, str(src), "-o", str(lib)])
    f = ctypes.CDLL(str(lib)).gather_offset
    f.restype = ctypes.c_longlong
    f.argtypes = [ctypes.c_int, ctypes.c_longlong, ctypes.c_int, ctypes.c_int, ctypes.c_int]
    return f


# p, cells, columns of the vector, first column and columns of the launch, size of a value, cells per block
@pytest.mark.parametrize("p,nc,ld,col0,cols,size,cpb",
                         [(5, (3, 2, 3), 26, 16, 10, 8, 1), (4, (2, 3, 2), 22, 16, 6, 8, 2), (4, (3, 2, 2), 30, 16, 14, 4, 2),
                          (3, (2, 2, 3), 18, 16, 2, 8, 4), (2, (3, 3, 2), 28, 16, 12, 4, 8), (1, (4, 3, 3), 6, 0, 6, 8, 16),
                          (6, (2, 2, 2), 16, 0, 16, 8, 1)])
def test_lanes_read_inside_the_vector(span, p, nc, ld, col0, cols, size, cpb):
    n = p + 1
    ncx, ncy, ncz = nc
    nx, ny, nz = (m * p - 1 for m in nc)
    rows = nx * ny * nz
    cb = 2
    while cb < min(cols, 16):
        cb *= 2
    i = np.arange(n)
    reads = 0
    for c0 in range(0, ncx * ncy * ncz, cpb):
        def row(c):
            x, y, z = c % ncx, (c // ncx) % ncy, c // (ncx * ncy)
            return (x * p - 1) + nx * ((y * p - 1) + ny * (z * p - 1))
        base = max(row(c0), 0)
        nrec = min((rows - base) * ld * size, 0x7fffffff)
        end = ((rows - base) * ld - col0) * size  # where the vector ends, from the launch's first column in row `base`
        for slot in range(cpb):
            cell_ok = c0 + slot < ncx * ncy * ncz
            c = c0 + slot if cell_ok else c0
            for j in range(n):
                for colg in range(((cols + cb - 1) // cb) * cb):
                    act = cell_ok and colg < cols
                    o = span(act, row(c) + nx * j - base, ld, colg, size)
                    off = (o + (i[:, None] + nx * ny * i) * (ld * size)) % 2 ** 32
                    read = off + size <= nrec
                    reads += int(read.sum())
                    assert not np.any(read & (off + size > end)), (c0, slot, j, colg)
                    if not act:
                        assert not read.any()
    assert reads >= rows * cols  # every value of the launch is read at least once
