// Matrix-free spectral-FE operator on MI355X (gfx950).
//
// One workgroup handles CPB cells x CB real columns.  Every thread owns one
// (line, column) of a cell and keeps a 1D line of N values in registers; the
// line orientation changes between phases through LDS.  Per cell and column
// the action of Eq. DiscreteHamiltonian is
//   y_e = B^T B^T B^T [ V w u_q + sum_d Dg_d^T ( kin G_d w Dg_d u_q ) ]
// with u_q = (B x B x B) u_e the values at the Gauss points and Dg the
// collocation derivative on the Gauss points (Dg B = D exactly because
// nq = p + 1).  Box cells have a diagonal metric G, so each direction's
// gradient term is finished by the thread owning that direction's line;
// curved (trilinear) cells compute J, det J and J^-1 J^-T per Gauss point
// from the 8 cell corners and couple the three gradient components.
// The element results are added into the output with FP64/FP32 atomics
// (hardware global_atomic_add), after the M^-1/2 scaling of the Loewdin
// form (Eq. TDKSMatVecStandard).  What bounds the one-column launches (the
// Hartree solve's): FP64 issue, of which the metric was two thirds, and the
// atomics' 64-byte segments.  24^3 trilinear cells, p = 6: 215 -> 96 us per
// product with the metric formed per line, folded tables and z as the last
// contraction.  The quadratic form u^T H u of every
// column is accumulated from the quadrature-point fluxes and reduced per
// workgroup; it equals Re<x, Hbar x> and feeds the Lanczos alpha.
#include "tdfe_cells.h"
#include "tdfe_fold.h"

namespace {

template <typename T>
__device__ __forceinline__ void atomic_add(T* p, T v) {
  unsafeAtomicAdd(p, v);
}

template <int N, int CB, int CPB, int GEOM>
struct ApplyShape {
  static constexpr int LINES = N * N;
  static constexpr int THREADS = CPB * LINES * CB;
  static constexpr int VOL = N * N * N;
  static constexpr int NARR = GEOM ? 4 : 2;
};

template <int N, int CB>
__device__ __forceinline__ int lidx(int slot, int z, int y, int x, int col) {
  return (((slot * N + z) * N + y) * N + x) * CB + col;
}

struct KParams {
  const void* x;
  void* y;
  int ld, cols, nchunks;
  const double* colscale;
  double kin;
  const void* vw;
  const double* minv;
  const double* cellgeo;
  const double* corners;
  const double* tab;
  double* energy;
  const int* done;
  int ncx, ncy, ncz, p, Nx, Ny, Nz;
  int64_t n_cell;
  int lowdin, fullgrid;
  int64_t* groups_out;  // host pointer, set by the launcher
};

// the 6 entries of w detJ J^-1 J^-T (w: the product Gauss weight) at the
// reference point (xa, xb, xc) of a trilinear cell with corners C[8][3]
// (z-corner slowest, x fastest)
__device__ __forceinline__ void metric_at(const double* C, double xa, double xb, double xc, double w, double g[6]) {
  const double f[2][3] = {{0.5 * (1 - xa), 0.5 * (1 - xb), 0.5 * (1 - xc)},
                          {0.5 * (1 + xa), 0.5 * (1 + xb), 0.5 * (1 + xc)}};
  double J[3][3] = {{0, 0, 0}, {0, 0, 0}, {0, 0, 0}};
  for (int vz = 0; vz < 2; ++vz)
    for (int vy = 0; vy < 2; ++vy)
      for (int vx = 0; vx < 2; ++vx) {
        const double* X3 = C + ((vz * 2 + vy) * 2 + vx) * 3;
        const double sx = vx ? 0.5 : -0.5, sy = vy ? 0.5 : -0.5, sz = vz ? 0.5 : -0.5;
        const double d0 = sx * f[vy][1] * f[vz][2];
        const double d1 = f[vx][0] * sy * f[vz][2];
        const double d2 = f[vx][0] * f[vy][1] * sz;
        for (int d = 0; d < 3; ++d) {
          J[d][0] += X3[d] * d0;
          J[d][1] += X3[d] * d1;
          J[d][2] += X3[d] * d2;
        }
      }
  // adjugate: J^-1 = adj / det ; det J^-1 J^-T = adj adj^T / det
  double A[3][3];
  A[0][0] = J[1][1] * J[2][2] - J[1][2] * J[2][1];
  A[0][1] = J[0][2] * J[2][1] - J[0][1] * J[2][2];
  A[0][2] = J[0][1] * J[1][2] - J[0][2] * J[1][1];
  A[1][0] = J[1][2] * J[2][0] - J[1][0] * J[2][2];
  A[1][1] = J[0][0] * J[2][2] - J[0][2] * J[2][0];
  A[1][2] = J[0][2] * J[1][0] - J[0][0] * J[1][2];
  A[2][0] = J[1][0] * J[2][1] - J[1][1] * J[2][0];
  A[2][1] = J[0][1] * J[2][0] - J[0][0] * J[2][1];
  A[2][2] = J[0][0] * J[1][1] - J[0][1] * J[1][0];
  const double det = J[0][0] * A[0][0] + J[0][1] * A[1][0] + J[0][2] * A[2][0];
  const double s = w / det;
  g[0] = s * (A[0][0] * A[0][0] + A[0][1] * A[0][1] + A[0][2] * A[0][2]);
  g[1] = s * (A[0][0] * A[1][0] + A[0][1] * A[1][1] + A[0][2] * A[1][2]);
  g[2] = s * (A[0][0] * A[2][0] + A[0][1] * A[2][1] + A[0][2] * A[2][2]);
  g[3] = s * (A[1][0] * A[1][0] + A[1][1] * A[1][1] + A[1][2] * A[1][2]);
  g[4] = s * (A[1][0] * A[2][0] + A[1][1] * A[2][1] + A[1][2] * A[2][2]);
  g[5] = s * (A[2][0] * A[2][0] + A[2][1] * A[2][1] + A[2][2] * A[2][2]);
}

// The Jacobian along an x line of a trilinear cell: its xi column is constant
// there, the eta and zeta columns are linear in xi.  A thread that owns the
// line forms these five vectors once and each point's columns by six
// multiply-adds (metric_at from the corners takes about 130 operations more).
struct LineJac {
  double x[3], y0[3], y1[3], z0[3], z1[3];
};
__device__ __forceinline__ LineJac line_jacobian(const double* C, double xb, double xc) {
  const double fy[2] = {0.5 * (1 - xb), 0.5 * (1 + xb)}, fz[2] = {0.5 * (1 - xc), 0.5 * (1 + xc)};
  LineJac L;
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    auto X = [&](int vx, int vy, int vz) { return C[((vz * 2 + vy) * 2 + vx) * 3 + d]; };
    double sx = 0.0, ey[2], ez[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      sx += fz[u] * (fy[0] * (X(1, 0, u) - X(0, 0, u)) + fy[1] * (X(1, 1, u) - X(0, 1, u)));
      ey[u] = 0.5 * (fz[0] * (X(u, 1, 0) - X(u, 0, 0)) + fz[1] * (X(u, 1, 1) - X(u, 0, 1)));
      ez[u] = 0.5 * (fy[0] * (X(u, 0, 1) - X(u, 0, 0)) + fy[1] * (X(u, 1, 1) - X(u, 1, 0)));
    }
    L.x[d] = 0.5 * sx;
    L.y0[d] = 0.5 * (ey[0] + ey[1]);
    L.y1[d] = 0.5 * (ey[1] - ey[0]);
    L.z0[d] = 0.5 * (ez[0] + ez[1]);
    L.z1[d] = 0.5 * (ez[1] - ez[0]);
  }
  return L;
}
// w detJ J^-1 J^-T at xi = xa of the line
__device__ __forceinline__ void line_metric(const LineJac& L, double xa, double w, double g[6]) {
  double y[3], z[3];
#pragma unroll
  for (int d = 0; d < 3; ++d) {
    y[d] = L.y0[d] + xa * L.y1[d];
    z[d] = L.z0[d] + xa * L.z1[d];
  }
  const double* x = L.x;
  // rows of the adjugate: cross products of the columns
  const double a0[3] = {y[1] * z[2] - y[2] * z[1], y[2] * z[0] - y[0] * z[2], y[0] * z[1] - y[1] * z[0]};
  const double a1[3] = {z[1] * x[2] - z[2] * x[1], z[2] * x[0] - z[0] * x[2], z[0] * x[1] - z[1] * x[0]};
  const double a2[3] = {x[1] * y[2] - x[2] * y[1], x[2] * y[0] - x[0] * y[2], x[0] * y[1] - x[1] * y[0]};
  const double s = w / (x[0] * a0[0] + x[1] * a0[1] + x[2] * a0[2]);
  g[0] = s * (a0[0] * a0[0] + a0[1] * a0[1] + a0[2] * a0[2]);
  g[1] = s * (a0[0] * a1[0] + a0[1] * a1[1] + a0[2] * a1[2]);
  g[2] = s * (a0[0] * a2[0] + a0[1] * a2[1] + a0[2] * a2[2]);
  g[3] = s * (a1[0] * a1[0] + a1[1] * a1[1] + a1[2] * a1[2]);
  g[4] = s * (a1[0] * a2[0] + a1[1] * a2[1] + a1[2] * a2[2]);
  g[5] = s * (a2[0] * a2[0] + a2[1] * a2[1] + a2[2] * a2[2]);
}

template <typename T, int N, int CB, int CPB, int GEOM>
__global__ void __launch_bounds__(CPB * N * N * CB)
    apply_kernel(KParams P) {
  using S = ApplyShape<N, CB, CPB, GEOM>;
  constexpr int VOL = S::VOL;
  __shared__ T sU[CPB * VOL * CB];
  __shared__ T sR[CPB * VOL * CB];
  __shared__ T sGY[GEOM ? CPB * VOL * CB : 1];
  __shared__ T sGZ[GEOM ? CPB * VOL * CB : 1];
  // one-column launches of curved cells (the Hartree solve's stiffness
  // products) form each Gauss point's metric in registers at the flux step,
  // where one thread owns the point: the LDS of the metric (48 KB for two
  // p = 7 cells) would otherwise hold a CU to one block of two waves
  constexpr bool GREG = GEOM && CB == 1;
  __shared__ T sGeo[(GEOM && !GREG) ? CPB * VOL * 6 : 1];
  __shared__ T sW3[VOL];
  __shared__ double sEta[N];
  __shared__ double sCor[GEOM ? CPB * 24 : 1];
  // 1D tables as compile-time constants (the weights and Gauss points, read
  // with per-thread indices, stay in LDS)
  constexpr tdfe1d::Rule R = tdfe1d::make_rule(N - 1);
  constexpr FoldSet<N> FS = make_foldset<N>();
  __shared__ double sRed[S::THREADS];

  if (P.done && *P.done) return;

  const int t = threadIdx.x;
  const int L = remap_block(blockIdx.x, gridDim.x);
  const int chunk = L % P.nchunks;
  const int group = L / P.nchunks;
  const int col = t % CB;
  const int line = (t / CB) % S::LINES;
  const int slot = t / (CB * S::LINES);
  const int64_t cell = (int64_t)group * CPB + slot;
  const bool cell_ok = cell < P.n_cell;
  const int colg = chunk * CB + col;
  const bool col_ok = colg < P.cols;
  const bool act = cell_ok && col_ok;

  for (int i = t; i < VOL; i += S::THREADS) sW3[i] = (T)P.tab[TAB_W3Q + i];
  if (t < N) sEta[t] = P.tab[TAB_ETA + t];

  int cx = 0, cy = 0, cz = 0;
  if (cell_ok) {
    cx = (int)(cell % P.ncx);
    cy = (int)((cell / P.ncx) % P.ncy);
    cz = (int)(cell / ((int64_t)P.ncx * P.ncy));
  }
  const T* __restrict__ X = (const T*)P.x;
  T* __restrict__ Y = (T*)P.y;
  const T* __restrict__ VW = (const T*)P.vw;
  T cs = (T)1;
  if (P.colscale && col_ok) cs = (T)P.colscale[colg >> 1];

  const int NxI = P.Nx - 2, NyI = P.Ny - 2;
  auto node_index = [&](int i, int j, int k, bool& inside) -> int64_t {
    const int I = cx * P.p + i, J = cy * P.p + j, K = cz * P.p + k;
    if (P.fullgrid) {
      inside = true;
      return (int64_t)I + (int64_t)P.Nx * ((int64_t)J + (int64_t)P.Ny * K);
    }
    inside = I > 0 && I < P.Nx - 1 && J > 0 && J < P.Ny - 1 && K > 0 && K < P.Nz - 1;
    return (int64_t)(I - 1) + (int64_t)NxI * ((int64_t)(J - 1) + (int64_t)NyI * (K - 1));
  };


  // prologue: the block's cell corners and this thread's z-line gather (values
  // and M^-1/2, from valid addresses, masked later) are issued together; the
  // metric is computed from LDS while the gather is in flight
  constexpr int NCR = GEOM ? (CPB * 24 + S::THREADS - 1) / S::THREADS : 1;
  double cr[NCR];
  if constexpr (GEOM) {
#pragma unroll
    for (int k = 0; k < NCR; ++k) {
      const int f = t + k * S::THREADS;
      const int64_t c0 = (int64_t)group * CPB;
      const bool ok = f < CPB * 24 && c0 + f / 24 < P.n_cell;
      const double val = P.corners[ok ? c0 * 24 + f : 0];
      cr[k] = ok ? val : 0.0;
    }
  }
  T gx1[N], gm1[N];
  unsigned gmask = 0;
  {
    const int i = line % N, j = line / N;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      bool inside;
      const int64_t id = node_index(i, j, k, inside);
      const bool ok = act && inside;
      if (ok) gmask |= 1u << k;
      const int64_t id0 = ok ? id : 0;
      gx1[k] = X[id0 * P.ld + (ok ? colg : 0)];
      gm1[k] = (T)P.minv[P.lowdin ? id0 : 0];
    }
  }
  if constexpr (GEOM) {
#pragma unroll
    for (int k = 0; k < NCR; ++k) {
      const int f = t + k * S::THREADS;
      if (f < CPB * 24) sCor[f] = cr[k];
    }
  }
  __syncthreads();
  // geometry of curved cells: 6 entries of detJ w J^-1 J^-T at every Gauss point
  if constexpr (GEOM && !GREG) {
    for (int it = t; it < CPB * VOL; it += S::THREADS) {
      const int sl = it / VOL, q = it % VOL;
      const int64_t ce = (int64_t)group * CPB + sl;
      if (ce >= P.n_cell) continue;
      const int a = q % N, b = (q / N) % N, c = q / (N * N);
      double gd[6];
      metric_at(sCor + sl * 24, sEta[a], sEta[b], sEta[c], (double)sW3[q], gd);
      T* g = sGeo + (sl * VOL + q) * 6;
#pragma unroll
      for (int w6 = 0; w6 < 6; ++w6) g[w6] = (T)gd[w6];
    }
  }
  __syncthreads();

  double energy = 0.0;
  T r1[N], r2[N];

  // ---- F1: gather z-lines, interpolate in z -----------------------------------
  {
    const int i = line % N, j = line / N;
#pragma unroll
    for (int k = 0; k < N; ++k)
      r1[k] = ((gmask >> k) & 1u) ? gx1[k] * (P.lowdin ? gm1[k] * cs : cs) : (T)0;
    eo<T, N, 1>(FS.B, r1, r2);
#pragma unroll
    for (int c = 0; c < N; ++c) sU[lidx<N, CB>(slot, c, j, i, col)] = r2[c];
  }
  __syncthreads();
  // ---- F2: interpolate in y -------------------------------------------------------
  {
    const int i = line % N, c = line / N;
#pragma unroll
    for (int j = 0; j < N; ++j) r1[j] = sU[lidx<N, CB>(slot, c, j, i, col)];
    eo<T, N, 1>(FS.B, r1, r2);
#pragma unroll
    for (int b = 0; b < N; ++b) sU[lidx<N, CB>(slot, c, b, i, col)] = r2[b];
  }
  __syncthreads();
  // ---- F3: interpolate in x; x-direction flux (box) or x-derivative (curved) -------------
  const T* vwc = (VW && cell_ok) ? VW + cell * VOL : nullptr;
  double gx = 0, gy = 0, gz = 0;
  if constexpr (!GEOM) {
    if (cell_ok) {
      gx = P.kin * P.cellgeo[cell * 4 + 0];
      gy = P.kin * P.cellgeo[cell * 4 + 1];
      gz = P.kin * P.cellgeo[cell * 4 + 2];
    }
  }
  {
    const int b = line % N, c = line / N;
#pragma unroll
    for (int i = 0; i < N; ++i) r1[i] = sU[lidx<N, CB>(slot, c, b, i, col)];
    T uq[N], du[N];
    eo<T, N, 1>(FS.B, r1, uq);
    eo<T, N, -1>(FS.G, uq, du);
    if constexpr (!GEOM) {
      T pot[N], f[N];
#pragma unroll
      for (int a = 0; a < N; ++a) {
        const int q = a + N * (b + N * c);
        pot[a] = vwc ? vwc[q] * uq[a] : (T)0;
        f[a] = (T)gx * sW3[q] * du[a];
        energy += (double)f[a] * (double)du[a] + (double)pot[a] * (double)uq[a];
      }
      eo<T, N, -1>(FS.Gt, f, r2);
#pragma unroll
      for (int a = 0; a < N; ++a) {
        sU[lidx<N, CB>(slot, c, b, a, col)] = uq[a];
        sR[lidx<N, CB>(slot, c, b, a, col)] = pot[a] + r2[a];
      }
      // The quadratic form is made final after each phase: left alone the compiler
      // keeps the products of all phases for the reduction at the end (FP64 n =
      // 9, 8 columns: 57 registers spilled; 16 orbitals on 12 x 11 x 13 cells 731
      // us a launch, 570 so, and 705 with unfolded tables, 34 spilled)
      asm volatile("" : "+v"(energy));
    } else {
#pragma unroll
      for (int a = 0; a < N; ++a) {
        sU[lidx<N, CB>(slot, c, b, a, col)] = uq[a];
        sR[lidx<N, CB>(slot, c, b, a, col)] = du[a];  // x-derivative
      }
    }
  }
  __syncthreads();

  if constexpr (!GEOM) {
    // ---- F4: z-direction flux -----------------------------------------------------
    {
      const int a = line % N, b = line / N;
#pragma unroll
      for (int c = 0; c < N; ++c) {
        r1[c] = sU[lidx<N, CB>(slot, c, b, a, col)];
        r2[c] = sR[lidx<N, CB>(slot, c, b, a, col)];
      }
      T f[N], d[N];
      eo<T, N, -1>(FS.G, r1, d);
#pragma unroll
      for (int c = 0; c < N; ++c) {
        f[c] = (T)gz * sW3[a + N * (b + N * c)] * d[c];
        energy += (double)f[c] * (double)d[c];
      }
      asm volatile("" : "+v"(energy));
      eo<T, N, -1>(FS.Gt, f, d);
#pragma unroll
      for (int c = 0; c < N; ++c) sR[lidx<N, CB>(slot, c, b, a, col)] = r2[c] + d[c];
    }
    __syncthreads();
    // ---- F5: y-direction flux, then B^T in y ------------------------------------------
    {
      const int a = line % N, c = line / N;
#pragma unroll
      for (int b = 0; b < N; ++b) {
        r1[b] = sU[lidx<N, CB>(slot, c, b, a, col)];
        r2[b] = sR[lidx<N, CB>(slot, c, b, a, col)];
      }
      T f[N], d[N];
      eo<T, N, -1>(FS.G, r1, d);
#pragma unroll
      for (int b = 0; b < N; ++b) {
        f[b] = (T)gy * sW3[a + N * (b + N * c)] * d[b];
        energy += (double)f[b] * (double)d[b];
      }
      asm volatile("" : "+v"(energy));
      eo<T, N, -1>(FS.Gt, f, d);
#pragma unroll
      for (int b = 0; b < N; ++b) r1[b] = r2[b] + d[b];
      eo<T, N, 1>(FS.Bt, r1, r2);
#pragma unroll
      for (int j = 0; j < N; ++j) sR[lidx<N, CB>(slot, c, j, a, col)] = r2[j];
    }
    __syncthreads();
  } else {
    // ---- F4/F5: y- and z-derivatives of u_q ------------------------------------------
    {
      const int a = line % N, c = line / N;
#pragma unroll
      for (int b = 0; b < N; ++b) r1[b] = sU[lidx<N, CB>(slot, c, b, a, col)];
      eo<T, N, -1>(FS.G, r1, r2);
#pragma unroll
      for (int b = 0; b < N; ++b) sGY[lidx<N, CB>(slot, c, b, a, col)] = r2[b];
    }
    {
      const int a = line % N, b = line / N;
#pragma unroll
      for (int c = 0; c < N; ++c) r1[c] = sU[lidx<N, CB>(slot, c, b, a, col)];
      eo<T, N, -1>(FS.G, r1, r2);
#pragma unroll
      for (int c = 0; c < N; ++c) sGZ[lidx<N, CB>(slot, c, b, a, col)] = r2[c];
    }
    __syncthreads();
    // ---- P: pointwise fluxes, x-part of the transposed derivative --------------------
    {
      const int b = line % N, c = line / N;
      T fx[N], pot[N];
      LineJac J;
      if constexpr (GREG) J = line_jacobian(sCor + slot * 24, sEta[b], sEta[c]);
#pragma unroll
      for (int a = 0; a < N; ++a) {
        const int q = a + N * (b + N * c);
        const int li = lidx<N, CB>(slot, c, b, a, col);
        const T u = sU[li], dx = sR[li], dy = sGY[li], dz = sGZ[li];
        T gr[6];
        const T* g = gr;
        if constexpr (GREG) {
          double gd[6] = {0, 0, 0, 0, 0, 0};
          if (cell_ok) line_metric(J, R.eta[a], (double)sW3[q], gd);
#pragma unroll
          for (int w6 = 0; w6 < 6; ++w6) gr[w6] = (T)gd[w6];
        } else {
          g = sGeo + (slot * VOL + q) * 6;
        }
        const T k = (T)P.kin;
        const T ffx = k * (g[0] * dx + g[1] * dy + g[2] * dz);
        const T ffy = k * (g[1] * dx + g[3] * dy + g[4] * dz);
        const T ffz = k * (g[2] * dx + g[4] * dy + g[5] * dz);
        pot[a] = vwc ? vwc[q] * u : (T)0;
        energy += (double)ffx * dx + (double)ffy * dy + (double)ffz * dz + (double)pot[a] * u;
        fx[a] = ffx;
        sGY[li] = ffy;
        sGZ[li] = ffz;
      }
      asm volatile("" : "+v"(energy));
      eo<T, N, -1>(FS.Gt, fx, r1);
#pragma unroll
      for (int a = 0; a < N; ++a) sU[lidx<N, CB>(slot, c, b, a, col)] = pot[a] + r1[a];
    }
    __syncthreads();
    // ---- B1: z-part of the transposed derivative -----------------------------------
    {
      const int a = line % N, b = line / N;
      T d[N];
#pragma unroll
      for (int c = 0; c < N; ++c) {
        r1[c] = sU[lidx<N, CB>(slot, c, b, a, col)];
        r2[c] = sGZ[lidx<N, CB>(slot, c, b, a, col)];
      }
      eo<T, N, -1>(FS.Gt, r2, d);
#pragma unroll
      for (int c = 0; c < N; ++c) sU[lidx<N, CB>(slot, c, b, a, col)] = r1[c] + d[c];
    }
    __syncthreads();
    // ---- B2: y-part of the transposed derivative, then B^T in y --------------------------
    {
      const int a = line % N, c = line / N;
      T d[N];
#pragma unroll
      for (int b = 0; b < N; ++b) {
        r1[b] = sU[lidx<N, CB>(slot, c, b, a, col)];
        r2[b] = sGY[lidx<N, CB>(slot, c, b, a, col)];
      }
      eo<T, N, -1>(FS.Gt, r2, d);
#pragma unroll
      for (int b = 0; b < N; ++b) r1[b] += d[b];
      eo<T, N, 1>(FS.Bt, r1, r2);
#pragma unroll
      for (int j = 0; j < N; ++j) sR[lidx<N, CB>(slot, c, j, a, col)] = r2[j];
    }
    __syncthreads();
  }
  // ---- B4: B^T in x ------------------------------------------------------------------------
  {
    const int j = line % N, c = line / N;
#pragma unroll
    for (int a = 0; a < N; ++a) r1[a] = sR[lidx<N, CB>(slot, c, j, a, col)];
    eo<T, N, 1>(FS.Bt, r1, r2);
#pragma unroll
    for (int i = 0; i < N; ++i) sR[lidx<N, CB>(slot, c, j, i, col)] = r2[i];
  }
  __syncthreads();
  // ---- B5: B^T in z and scatter-add: z last, so that neighbouring lanes write
  // neighbouring x nodes (an atomic costs per 64-byte segment, whatever it
  // carries: with x last a one-column launch was 343 segments per p = 6 cell) ----
  {
    const int i = line % N, j = line / N;
#pragma unroll
    for (int c = 0; c < N; ++c) r1[c] = sR[lidx<N, CB>(slot, c, j, i, col)];
    eo<T, N, 1>(FS.Bt, r1, r2);
    if (act) {
#pragma unroll
      for (int k = 0; k < N; ++k) {
        bool inside;
        const int64_t id = node_index(i, j, k, inside);
        if (inside) atomic_add(Y + id * P.ld + colg, P.lowdin ? r2[k] * (T)P.minv[id] : r2[k]);
      }
    }
  }

  // ---- per-column quadratic form --------------------------------------------------------------
  if (P.energy) {
    sRed[t] = act ? energy : 0.0;
    __syncthreads();
    if (t < CB) {
      double s = 0.0;
      for (int u = t; u < S::THREADS; u += CB) s += sRed[u];
      if (chunk * CB + t < P.cols) P.energy[(int64_t)group * P.cols + chunk * CB + t] = s;
    }
  }
}

// ---------------------------------------------------------------------------------------------
// dispatch
// ---------------------------------------------------------------------------------------------
template <int N, int CB, int GEOM>
constexpr int pick_cpb() {
  // aim for >= 128 threads per block and <= 64 KB of line arrays
  int cpb = 1;
  while (cpb * N * N * CB < 128 && cpb < 16) cpb *= 2;
  return cpb;
}

template <typename T, int N, int CB, int GEOM>
tdfe_status launch_t(tdfe_ctx* c, KParams& P, int nchunks) {
  constexpr int CPB = pick_cpb<N, CB, GEOM>();
  using S = ApplyShape<N, CB, CPB, GEOM>;
  static_assert(S::THREADS <= 1024, "block too large");
  const int64_t groups = (c->n_cell + CPB - 1) / CPB;
  P.nchunks = nchunks;
  if (P.groups_out) *P.groups_out = groups;
  const int64_t grid = groups * nchunks;
  hipLaunchKernelGGL((apply_kernel<T, N, CB, CPB, GEOM>), dim3((unsigned)grid), dim3(S::THREADS), 0,
                     c->stream, P);
  TDFE_HIP(c, hipGetLastError());
  return TDFE_OK;
}

template <typename T, int N>
tdfe_status launch_n(tdfe_ctx* c, KParams& P, bool geom) {
  // largest column block that keeps the workgroup within 1024 threads and the
  // line arrays within ~96 KB of LDS
  const int cols = P.cols;
  constexpr int VOLB = N * N * N * (int)sizeof(T);
  int cb;
  if (cols <= 1) cb = 1;
  else if (cols <= 2) cb = 2;
  else if (cols <= 4) cb = 4;
  else if (cols <= 8) cb = 8;
  else cb = 16;
  auto fits = [&](int b) {
    const int narr = geom ? 4 : 2;
    return N * N * b <= 1024 && narr * VOLB * b + (geom ? 6 * VOLB : 0) <= 96 * 1024;
  };
  while (cb > 1 && !fits(cb)) cb >>= 1;
  const int nchunks = (cols + cb - 1) / cb;
#define TDFE_CASE(CBV)                                                                   \
  case CBV:                                                                              \
    if constexpr (N * N * CBV <= 1024 && 2 * VOLB * CBV <= 96 * 1024) {                    \
      if (geom) {                                                                        \
        if constexpr (4 * VOLB * CBV + 6 * VOLB <= 96 * 1024) return launch_t<T, N, CBV, 1>(c, P, nchunks); \
      } else                                                                             \
        return launch_t<T, N, CBV, 0>(c, P, nchunks);                                    \
    }                                                                                    \
    break;
  switch (cb) {
    TDFE_CASE(1)
    TDFE_CASE(2)
    TDFE_CASE(4)
    TDFE_CASE(8)
    TDFE_CASE(16)
  }
#undef TDFE_CASE
  return tdfe_fail(c, TDFE_EINVAL, "no operator kernel for n=%d cols=%d", N, cols);
}

template <typename T>
tdfe_status launch_p(tdfe_ctx* c, KParams& P, bool geom) {
  switch (c->n) {
    case 2: return launch_n<T, 2>(c, P, geom);
    case 3: return launch_n<T, 3>(c, P, geom);
    case 4: return launch_n<T, 4>(c, P, geom);
    case 5: return launch_n<T, 5>(c, P, geom);
    case 6: return launch_n<T, 6>(c, P, geom);
    case 7: return launch_n<T, 7>(c, P, geom);
    case 8: return launch_n<T, 8>(c, P, geom);
    case 9: return launch_n<T, 9>(c, P, geom);
  }
  return tdfe_fail(c, TDFE_EINVAL, "unsupported order p=%d", c->p);
}

// y (+)= the sums of the per-cell results: one block per row of DoFs (fixed y
// and z), a lane per node and W columns (16 bytes where the columns allow it)
template <typename T, int W, bool ADD>
__global__ void __launch_bounds__(256)
    assemble_kernel(const T* __restrict__ e, T* __restrict__ y, CellMap M, int cols, int ld, const int* done) {
  if (done && *done) return;
  const int C2 = cols / W;
  const int Op = C2 <= 4 ? 4 : (C2 <= 8 ? 8 : (C2 <= 16 ? 16 : 32));
  const int XL = 256 / Op;
  const CellRow R = cell_row(M, 1 + (int)(blockIdx.x % (unsigned)M.NyI), 1 + (int)(blockIdx.x / (unsigned)M.NyI));
  T* const yr = y + (int64_t)blockIdx.x * M.NxI * ld;
  for (int o = (int)threadIdx.x % Op; o < C2; o += Op)
    for (int I = (int)threadIdx.x / Op; I < M.NxI; I += XL) {
      CellLane<T, W> L;
      L.at(M, I);
      T* const d = yr + (int64_t)I * ld + W * o;
      T h[W], y0[W];
      if constexpr (ADD) {
#pragma unroll
        for (int q = 0; q < W; ++q) y0[q] = d[q];
      }
      L.sum(e, R, cols, o, h);
#pragma unroll
      for (int q = 0; q < W; ++q) d[q] = ADD ? y0[q] + h[q] : h[q];
    }
}

}  // namespace

int64_t tdfe_blocks_apply(const tdfe_ctx* c, int cols) {
  // upper bound on the number of cell groups any launch uses (CPB >= 1)
  (void)cols;
  return c->n_cell;
}

// box cells: lane pairs for FP64 at even n (two waves per SIMD), planes otherwise
static bool box_pair(const tdfe_ctx* c, const ApplyArgs& a) {
  return (c->variant == TDFE_VARIANT_PAIR || (c->variant == 0 && !a.fp32)) && tdfe_pair_kernel_ok(c);
}

static tdfe_status launch_blocks(tdfe_ctx* c, const ApplyArgs& a) {
  // default policy, from measurements on the benchmark and graded workloads:
  // the four-lane kernel where tdfe_quad_kernel_ok says; box cells: see
  // box_pair; trilinear cells: see tdfe_curved_pair
  if (tdfe_quad_kernel_ok(c, a)) return tdfe_launch_apply_quad(c, a);
  if (!c->box) return tdfe_launch_apply_curved(c, a);
  return box_pair(c, a) ? tdfe_launch_apply_pair(c, a) : tdfe_launch_apply_box(c, a);
}

static size_t cell_bytes(const tdfe_ctx* c, int cols, bool fp32) {
  return (size_t)c->n_cell * c->n * c->n * c->n * cols * (fp32 ? 4 : 8);
}

// Whether 32-bit byte offsets reach every node of a block's cells: always in
// the four-lane kernel (a 64-bit address per row of nodes, and its own check),
// else a matter of the cells per block of the kernel that would run.
static bool offsets_near(const tdfe_ctx* c, const ApplyArgs& a) {
  if (tdfe_quad_kernel_ok(c, a)) return true;
  const int64_t row = (int64_t)a.ld * (a.fp32 ? 4 : 8), layer = (int64_t)c->Nx * c->Ny + c->Nx;
  if (130 * c->p * layer * row < (int64_t)1 << 31) return true;  // for any block (at most 128 cells)
  int64_t cells = 0;
  ApplyArgs q = a;
  q.query = true;
  q.n_blocks_out = &cells;
  return launch_blocks(const_cast<tdfe_ctx*>(c), q) == TDFE_OK &&
         tdfe_span::near(c->p, c->ncx, c->ncy, c->ncz, cells, row);
}

// Launches of the plane, lane-pair and four-lane kernels: Loewdin DoF vectors,
// p <= 7; two or more columns on trilinear cells (one column leaves n threads
// per cell with the metric staged for the whole cell: the line kernel is
// faster there, 0.64 ms against 2.2 ms for the Hartree solve's one-column
// products on the graded mesh).  Box cells have kernels with 64-bit offsets
// for rows so long or layers so large that 32 bits do not reach over a block;
// trilinear cells go to the line kernel there.
static bool block_kernels_ok(const tdfe_ctx* c, const ApplyArgs& a) {
  if (c->variant == TDFE_VARIANT_LINE || !a.lowdin || a.fullgrid || c->n_cell >= (int64_t)1 << 30) return false;
  if (c->box) return tdfe_box_kernel_ok(c);
  return tdfe_curved_kernel_ok(c, a.cols, a.fp32) && offsets_near(c, a);
}

// Columns of a launch whose per-cell results fit the cell buffer (0: none): all
// of them, or a multiple of 16.
static int cells_fit(const tdfe_ctx* c, const ApplyArgs& a) {
  if (!c->eloc_bytes || a.cols % 2 || !block_kernels_ok(c, a)) return 0;
  const int cap = (int)std::min<size_t>(c->eloc_bytes / cell_bytes(c, 1, a.fp32), 1 << 20);
  const int step = a.cols <= cap ? a.cols : cap / 16 * 16;
  // (64-bit offsets come with the scatter only)
  for (int cols : {step, step ? a.cols % step : 0}) {
    ApplyArgs s = a;
    s.cols = cols;
    if (cols && !offsets_near(c, s)) return 0;
  }
  return step;
}

// Atomics are performed per 64-byte segment: a row of columns of more than one
// segment that is no whole number of them costs up to twice its size.
static bool split_row(int cols, bool fp32) {
  const int row = cols * (fp32 ? 4 : 8);
  return row > 64 && row % 64 != 0;
}

// Per-cell results take plain stores where the scatter takes atomics, and leave
// n^3 / p^3 vectors to be summed.  Summed by the Krylov update, which then has no
// operator output to read, seed and clear, they pay wherever they fit from n^3 /
// p^3 = 3.4 on (n = 3), on trilinear cells 2.4 (n = 4).  Per iteration: 16^3 box
// cells, p = 5, 8 orbitals, FP64 (113 MB) 112 + 36 us scattered, 63 + 48 us per
// cell; FP32 (57 MB) 56 + 24 and 38 + 28.  Beyond the memory-side cache: 24^3
// trilinear cells, p = 6, FP64 (607 MB) 545 + 228 us scattered, 537 + 314 us per
// cell.  Below n = 3 or 4 they pay while the L2s hold them, or against split rows
// (p = 1, box, 13 orbitals, 250,000 DoFs FP32 1,546 us scattered, 1,138 per cell, 60,000
// DoFs FP64 711 and 632), but not for one orbital (p = 1, 60,000 DoFs FP64 168 and 196;
// trilinear p = 2, 900,000 DoFs FP32 334 and 434, 60,000 149 and 137).
bool tdfe_cells_ok(const tdfe_ctx* c, int cols, bool fp32) {
  ApplyArgs a{};
  a.cols = a.ld = cols;
  a.lowdin = true;
  a.fp32 = fp32;
  if (cells_fit(c, a) != cols) return false;
  if (c->cell_always || c->p >= (c->box ? 2 : 3)) return true;
  if (cols == 2) return c->p == 2 && c->n_dof < 200000;
  return cell_bytes(c, cols, fp32) <= (size_t)32 << 20 || split_row(cols, fp32);
}

// Whether a launch into a DoF vector goes through the cell buffer, `step` columns
// at a time, with a pass of its own that sums the cells.  The pass costs 3 to 5
// us and reading the buffer; what it saves are the atomics, which hide behind the
// arithmetic of the larger orders, and where the result replaces y the pass that
// clears it.  So, from 200,000 DoFs or a million values on:
//  * p = 1, eight values per DoF: split rows only (250,000 DoFs, box, 9 orbitals FP64
//    239 us per cell against 346, FP32 172 and 244);
//  * box cells, result replaces y: always (16^3 cells, p = 5, 8 orbitals 90 us
//    against 102, 64 orbitals in slices 642 and 714; 20 x 19 x 21 one orbital 42
//    and 84), except for the four-lane kernel at n = 7 beyond 64 MB, which hides its
//    atomics (16 x 15 x 17, 8 orbitals 161 and 148);
//  * box cells, added to y: less than a segment or split rows, not the FP64
//    four-lane kernel (p = 5, one orbital 42 and 80, 5 orbitals 140 and 163; 8
//    orbitals 177 and 161; p = 6, 5 orbitals 136 and 113); FP32 also whole segments,
//    from 200,000 DoFs and up to 128 MB (8 orbitals 97 us per cell and 101; 60,000
//    DoFs: 24 and 18), and split rows in slices (p = 2, 13 orbitals, 900,000 DoFs 314
//    and 497);
//  * trilinear cells, result replaces y: the four-lane kernel (n = 8: 14 x 13 x 15,
//    8 orbitals 205 and 216; n = 7 up to 64 MB), and up to three orbitals from p = 3 on (p =
//    5, one 89 and 118; 8 orbitals 253 and 230);
//  * trilinear cells, added to y, from 200,000 DoFs on, not the four-lane kernel:
//    less than a segment from p = 3 on (FP64 p = 5, one orbital 88 and 112), FP32 from
//    two orbitals also at p = 2 (3 orbitals 138 and 160, 5 183 and 231; one 86 and 75);
//    FP32 split rows from p = 3 on (p = 4, 9 orbitals 226 and 278; 8 orbitals 116 and
//    99), in the four-lane kernel too.
// A last slice of less than 8 columns is not worth a launch and a sum (p > 1).
static bool sum_pays(const tdfe_ctx* c, const ApplyArgs& a, int step) {
  if (c->cell_always) return true;
  const bool quad = tdfe_quad_kernel_ok(c, a), sliced = step < a.cols, large = c->n_dof >= 200000;
  const int row = a.cols * (a.fp32 ? 4 : 8);
  const size_t bytes = cell_bytes(c, a.cols, a.fp32);
  const bool split = split_row(a.cols, a.fp32);
  if (!large && c->n_dof * a.cols < 1000000) return false;
  if (c->p == 1) return split && (c->box || !a.fp32);
  if (sliced && a.cols % step != 0 && a.cols % step < 8) return false;
  if (a.overwrite) {
    if (quad) return c->n == 8 || bytes <= (size_t)64 << 20;
    return c->box || (c->p >= 3 && row < 64);
  }
  if (sliced) return c->box && a.fp32 && split;
  if (c->box) return row < 64 || split ? a.fp32 || !quad : a.fp32 && large && bytes <= (size_t)128 << 20;
  if (!large) return false;
  if (row < 64) return !quad && (c->p >= 3 || (a.fp32 && a.cols >= 4));
  return a.fp32 && split && c->p >= 3;
}

tdfe_status tdfe_launch_apply_cells(tdfe_ctx* c, const ApplyArgs& a0) {
  ApplyArgs a = a0;
  if (cells_fit(c, a) != a.cols) return tdfe_fail(c, TDFE_EINVAL, "apply: no per-cell results for this launch");
  if (a.fp32 && !tdfe_fp32(c)) return tdfe_fail(c, TDFE_EINVAL, "apply: FP32 launch in an FP64 context");
  a.y = c->eloc;
  a.eld = a.cols;
  a.cells = true;
  return launch_blocks(c, a);
}

// y (+)= H x through the cell buffer, `step` columns at a time
static tdfe_status launch_cells_sum(tdfe_ctx* c, const ApplyArgs& a0, int step) {
  const size_t eb = a0.fp32 ? 4 : 8;
  const CellMap M{c->ncx, c->ncy, c->ncz, c->p, c->Nx - 2, c->Ny - 2, c->Nz - 2};
  const dim3 grid((unsigned)(M.NyI * M.NzI));
  for (int col0 = 0; col0 < a0.cols; col0 += step) {
    ApplyArgs a = a0;
    a.cols = std::min(step, a0.cols - col0);
    a.eld = a.cols;
    a.cells = true;
    a.x = (const char*)a0.x + col0 * eb;
    a.y = c->eloc;
    if (a0.colscale) a.colscale = a0.colscale + col0 / 2;
    TDFE_TRY(launch_blocks(c, a));
    void* const y = (char*)a0.y + col0 * eb;
    auto assemble = [&](auto kernel, auto* e, auto* out) {
      hipLaunchKernelGGL(kernel, grid, dim3(256), 0, c->stream, e, out, M, a.cols, a.ld, a.done_flag);
    };
    auto* const e64 = (const double*)c->eloc;
    auto* const e32 = (const float*)c->eloc;
    if (!a.fp32 && a.overwrite) assemble(assemble_kernel<double, 2, false>, e64, (double*)y);
    if (!a.fp32 && !a.overwrite) assemble(assemble_kernel<double, 2, true>, e64, (double*)y);
    if (a.fp32 && a.cols % 4 == 0) assemble(assemble_kernel<float, 4, true>, e32, (float*)y);
    if (a.fp32 && a.cols % 4 != 0) assemble(assemble_kernel<float, 2, true>, e32, (float*)y);
    TDFE_HIP(c, hipGetLastError());
  }
  return TDFE_OK;
}

bool tdfe_can_overwrite(const tdfe_ctx* c, const ApplyArgs& a0) {
  if (c->octree || a0.fp32 || a0.energy) return false;
  ApplyArgs a = a0;
  a.overwrite = true;
  const int step = cells_fit(c, a);
  return step > 0 && sum_pays(c, a, step);
}

static tdfe_status launch_local(tdfe_ctx* c, const ApplyArgs& a) {
  if (c->octree) return tdfe_launch_apply_octree(c, a);
  // the FP32 copy of the potential exists in mixed contexts only
  if (a.fp32 && !tdfe_fp32(c)) return tdfe_fail(c, TDFE_EINVAL, "apply: FP32 launch in an FP64 context");
  if (a.cols < 1) return tdfe_fail(c, TDFE_EINVAL, "apply: cols < 1");
  // M^-1/2 exists on the interior DoFs only
  if (a.lowdin && a.fullgrid) return tdfe_fail(c, TDFE_EINVAL, "apply: Loewdin scaling on the full node grid");
  if (c->mfma && tdfe_mfma_kernel_ok(c, a)) return tdfe_launch_apply_mfma(c, a);
  const int step = cells_fit(c, a);
  if ((step == a.cols || (step > 0 && !a.energy)) && (a.overwrite || sum_pays(c, a, step)))
    return launch_cells_sum(c, a, step);
  if (block_kernels_ok(c, a)) {
    ApplyArgs b = a;
    b.eld = a.cols;
    b.far = !offsets_near(c, a);
    return launch_blocks(c, b);
  }
  // full-grid and one-column curved launches, p = 8, trilinear cells beyond
  // 32-bit offsets: the line kernel, which scatters by atomics
  KParams P{};
  P.x = a.x;
  P.y = a.y;
  P.ld = a.ld;
  P.cols = a.cols;
  P.colscale = a.colscale;
  P.kin = a.kin;
  P.vw = a.fp32 ? (const void*)a.vw32 : (const void*)a.vw;
  P.minv = c->minv;
  P.cellgeo = c->cellgeo;
  P.corners = c->corners;
  P.tab = c->tab;
  P.energy = a.energy;
  P.done = a.done_flag;
  P.ncx = c->ncx;
  P.ncy = c->ncy;
  P.ncz = c->ncz;
  P.p = c->p;
  P.Nx = c->Nx;
  P.Ny = c->Ny;
  P.Nz = c->Nz;
  P.n_cell = c->n_cell;
  P.lowdin = a.lowdin;
  P.fullgrid = a.fullgrid;
  P.groups_out = a.n_blocks_out;
  const bool geom = !c->box;
  if (a.fp32) return launch_p<float>(c, P, geom);
  return launch_p<double>(c, P, geom);
}

int tdfe_operator_route(const tdfe_ctx* c, int cols, int fp32) {
  ApplyArgs a{};
  a.cols = a.ld = cols;
  a.lowdin = true;
  a.fp32 = fp32 != 0;
  if (c->octree || (c->mfma && tdfe_mfma_kernel_ok(c, a)) || !block_kernels_ok(c, a)) return 0;
  const bool pair = c->box ? box_pair(c, a) : tdfe_curved_pair(c, a.cols, a.fp32);
  const int step = cells_fit(c, a);
  return (tdfe_quad_kernel_ok(c, a) ? 4 : (pair ? 3 : 1)) + (offsets_near(c, a) ? 0 : 8) +
         (step && sum_pays(c, a, step) ? 16 : 0) + (tdfe_can_overwrite(c, a) ? 32 : 0) +
         (tdfe_cells_ok(c, cols, a.fp32) ? 64 : 0);
}

tdfe_status tdfe_launch_apply(tdfe_ctx* c, const ApplyArgs& a) {
  TDFE_TRY(launch_local(c, a));
  if (a.nonlocal) TDFE_TRY(tdfe_launch_nonlocal(c, a));
  return TDFE_OK;
}
