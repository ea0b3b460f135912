// Sums of per-cell results at the DoFs (the assembly of Eq. DiscreteHamiltonian),
// for kernels that read the per-cell output [n_cell][n^3][cols] of the plane,
// lane-pair and four-lane operators.
//
// A DoF on a cell face, edge or corner has 2, 4 or 8 contributions.  Along a row
// of DoFs (fixed y and z node) the y and z sharing is the row's own, so a block
// that works row by row has at most four base positions, the same for all its
// lanes; only the x sharing differs between lanes, and is one more load at the
// cell boundaries.  The contributions are added in a fixed order.
#pragma once
#include "tdfe_internal.h"

namespace {

struct CellMap {
  int ncx, ncy, ncz, p, NxI, NyI, NzI;  // cells, order, DoFs per axis
};

// base positions (in nodes) of row (J, K) of the node grid: its own cells, and
// those before along y (yb), z (zb) and both where the row is shared
struct CellRow {
  int64_t base, base_y, base_z, base_yz;
  bool yb, zb;
};

__device__ __forceinline__ CellRow cell_row(const CellMap& M, int J, int K) {
  const int n = M.p + 1;
  const int64_t vol = (int64_t)n * n * n;
  const int cy = J / M.p, j = J - cy * M.p, cz = K / M.p, k = K - cz * M.p;
  auto at = [&](int yy, int jj, int zz, int kk) {
    return ((int64_t)yy + (int64_t)M.ncy * zz) * M.ncx * vol + (int64_t)(kk * n + jj) * n;
  };
  CellRow R;
  R.yb = j == 0;
  R.zb = k == 0;
  R.base = at(cy, j, cz, k);
  R.base_y = R.yb ? at(cy - 1, M.p, cz, k) : 0;
  R.base_z = R.zb ? at(cy, j, cz - 1, M.p) : 0;
  R.base_yz = R.yb && R.zb ? at(cy - 1, M.p, cz - 1, M.p) : 0;
  return R;
}

// f(base) for every base position of the row, in that order
template <typename F>
__device__ __forceinline__ void for_bases(const CellRow& R, F f) {
  f(R.base);
  if (R.yb) f(R.base_y);
  if (R.zb) {
    f(R.base_z);
    if (R.yb) f(R.base_yz);
  }
}

// one lane's node of a row, W columns of it
template <typename T, int W>
struct CellLane {
  typedef T V __attribute__((ext_vector_type(W)));
  int64_t m1, m2;
  bool edge;

  // DoF I (0-based) of the row
  __device__ __forceinline__ void at(const CellMap& M, int I) {
    const int n = M.p + 1, vol = n * n * n;
    const int ex = (I + 1) / M.p, i = I + 1 - ex * M.p;
    edge = i == 0;
    m1 = (int64_t)ex * vol + i;
    m2 = edge ? m1 - vol + M.p : m1;  // the same node in the cell before
  }
  // sums of the contributions of W columns from column W o of C, in S
  template <typename S>
  __device__ __forceinline__ void sum(const T* __restrict__ e, const CellRow& R, int C, int o, S (&h)[W]) {
#pragma unroll
    for (int q = 0; q < W; ++q) h[q] = (S)0;
    for_bases(R, [&](int64_t base) {
      const V u = *((const V*)(e + (base + m1) * C) + o);
      const V v = *((const V*)(e + (base + m2) * C) + o);
#pragma unroll
      for (int q = 0; q < W; ++q) h[q] += edge ? (S)u[q] + (S)v[q] : (S)u[q];
    });
  }
};

}  // namespace
