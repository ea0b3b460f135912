// Operator kernel for rectilinear (box) cells: "plane" sum factorisation.
//
// Same operator as tdfe_apply.hip (Eq. DiscreteHamiltonian in the Loewdin
// form, Eq. TDKSMatVecStandard), organised for the register file of CDNA4:
// each thread owns one column and an n x n plane of a cell's values.
//
//   A  (plane at fixed y node j):  gather u(i,k); z: B u; x: B and S B on it
//   -- LDS transpose of the two arrays -->
//   B  (plane at fixed x point a): y: B on both -> u_q and the x stiffness term;
//      in registers the y and z stiffness terms S u_q, the potential term, all
//      weighted and summed, and the transposed y interpolation of the sum
//   -- LDS transpose of the one array -->
//   C  (plane at fixed y node j):  x: B^T; z: B^T; results x M^-1/2 (CellOut).
//
// The metric of a box cell is one diagonal per cell, so a direction's
// derivative, flux and transposed derivative are one contraction with the 1D
// stiffness S of the Gauss-point basis (make_gauss_stiff): ten 1D contractions
// per cell and three arrays through LDS, where separate derivatives took
// fifteen and four.  What bounds the kernel is instruction issue and latency,
// so the shorter chain shows directly: FP32, 13 x 17 x 11 cells, p = 4, 5
// orbitals 48.0 -> 31.6 us (the lane-pair kernel, FP64, 16^3 cells, p = 5, 8
// orbitals: 139 -> 112 us).
//
// Only the y direction crosses threads.  Every 1D contraction uses the
// reflection symmetry of the GLL nodes and Gauss points
// (B[n-1-a][n-1-i] = B[a][i], S and S B likewise): even/odd folding halves the
// multiply-adds.  The folded tables are evaluated at compile time for the
// kernel's order (make_foldset), so each coefficient is an instruction
// constant: no table loads, and no scalar-memory waits that would also wait
// for the LDS transposes.
#include "tdfe_fold.h"

namespace {

template <typename T>
struct PlaneParams {
  const void* x;
  void* y;  // CELLS: per-cell results [n_cell][n^3][cols]; else the DoF vector, added to
  int ld, cols, nchunks, eld;
  const double* colscale;
  double kin;
  const void* vw;
  const double* minv;
  const double* m1x;  // separable M^-1/2 factors of a box mesh: minv(I,J,K) = m1x[I] m1y[J] m1z[K]
  const double* m1y;
  const double* m1z;
  const double* cellgeo;
  double* energy;
  const int* done;
  int ncx, ncy, ncz, p, Nx, Ny, Nz;
  int64_t n_cell;
  bool cells;
  bool far;    // offsets of 64 bits (host)
  bool query;  // report the cells per block only (host)
  double wq[TDFE_MAXN];  // Gauss weights (indexed by the thread's plane)
};

// occupancy target: FP64 planes of n >= 6 need more than 256 registers per
// lane, so they run one wave per SIMD and use the accumulation registers
template <typename T, int N>
constexpr int plane_wpe() {
  return sizeof(T) == 4 ? (N == 5 || N == 6 ? 3 : 2) : (N >= 6 ? 1 : 2);
}

template <typename T, int N, int CB, int CPB, bool CELLS, bool FAR>
__global__ void __launch_bounds__(CPB * N * CB) __attribute__((amdgpu_waves_per_eu(plane_wpe<T, N>())))
    plane_kernel(PlaneParams<T> P) {
  constexpr int VOL = N * N * N;
  constexpr int THREADS = CPB * N * CB;
  // 1D tables of order N, folded, as compile-time constants
  constexpr BoxFoldSet<N> FS = make_box_foldset<N, sizeof(T) == 4>();
  auto wprod = [&](int b, int c) { return (T)(FS.wq[b] * FS.wq[c]); };
  // FP32 at n = 2, 4, 6 and 7: phase A takes x first, on the nodes (one contraction
  // more), and at n = 4 interpolates by eo1: S multiplies the rounding of what it
  // is applied to, and an exponential of smooth orbitals shows it.  In a model of
  // this arithmetic (p = 3, 5, 6; 12 to 20 iterations) errors of 9.7e-8, 1.46e-7
  // and 1.78e-7 become 7.0e-8, 1.26e-7 and 1.70e-7, where derivatives on either
  // side of the flux give 8.0e-8, 1.30e-7 and 1.78e-7.
  constexpr bool F32 = sizeof(T) == 4;
  constexpr bool XFIRST = F32 && (N == 2 || N == 4 || N == 6 || N == 7), MID = F32 && N == 4;
  auto interp = [&](const T* in, T* out) {
    if constexpr (MID)
      eo1<T, N>(FS.B, FS.b, in, out);
    else
      eo<T, N, 1>(FS.B, in, out);
  };
  __shared__ T sX[CPB * VOL * CB];
  __shared__ T sV[CPB * VOL];  // weighted potential of the block's cells
  __shared__ double sRed[THREADS];
  if (P.done && *P.done) return;

  const int t = threadIdx.x;
  const int L = remap_block(blockIdx.x, gridDim.x);
  const int chunk = L % P.nchunks;
  const int group = L / P.nchunks;
  const int col = t % CB;
  const int pl = (t / CB) % N;
  const int slot = CPB == 1 ? 0 : t / (CB * N);
  const int64_t cell = (int64_t)group * CPB + slot;
  const bool cell_ok = cell < P.n_cell;
  const int colg = chunk * CB + col;
  const bool act = cell_ok && colg < P.cols;

  const int64_t c0 = (int64_t)group * CPB;
  const CellPos B0 = cell_pos(P, (int)c0);
  const CellPos cp = CPB == 1 ? B0 : cell_next(P, B0, cell_ok ? slot : 0);
  T* __restrict__ Y = (T*)P.y;
  double cs = 1.0;
  if (P.colscale && act) cs = P.colscale[colg >> 1];

  // block staging: the weighted potential of the block's cells, their M^-1/2
  // factors along x, y and z and their metric go to LDS.  The loads are issued
  // here, the phase A gather right after them, and the LDS stores follow both,
  // so that a wave waits for memory once rather than once per array.
  constexpr int NFC = 3 * N + 3;  // per cell: m_x[N], m_y[N], m_z[N], metric[3]
  constexpr int NV = (CPB * VOL + THREADS - 1) / THREADS;
  constexpr int NF = (CPB * NFC + THREADS - 1) / THREADS;
  __shared__ double sF[CPB * NFC];
  T vr[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int q = t + k * THREADS;
    const int64_t ce = c0 + q / VOL;
    const bool ok = P.vw && q < CPB * VOL && ce < P.n_cell;
    vr[k] = ok ? ((const T*)P.vw)[ce * VOL + q % VOL] : (T)0;
  }
  double fr[NF];
#pragma unroll
  for (int k = 0; k < NF; ++k) {
    const int f = t + k * THREADS;
    const int r = f % NFC;
    const int sl = f / NFC;
    const bool ok = f < CPB * NFC && c0 + sl < P.n_cell;
    const CellPos e = CPB == 1 ? B0 : cell_next(P, B0, ok ? sl : 0);
    const int64_t cv = c0 + (ok ? sl : 0);
    // one load from a selected (always valid) address: no branches
    const double* src = r < N ? P.m1x + (e.x * P.p + r)
                        : r < 2 * N ? P.m1y + (e.y * P.p + r - N)
                        : r < 3 * N ? P.m1z + (e.z * P.p + r - 2 * N)
                                    : P.cellgeo + (cv * 4 + r - 3 * N);
    const double val = *src;
    fr[k] = ok ? val : 0.0;
  }
  const double* sFc = sF + slot * NFC;  // this thread's cell
  // LDS index: slot, y index, x index, z index, column
  auto sidx = [&](int y, int x, int z) { return (((slot * N + y) * N + x) * N + z) * CB + col; };
  const int NxI = P.Nx - 2, NyI = P.Ny - 2;

  // ---------------- A: plane j = pl, values (i, k) -------------------------------------
  T u[N][N];  // [i][k] gathered, then [i][c], then S B u at [x point][z point]
  {
    const int j = pl;
    typedef CellIn<T, FAR> In;
    typedef typename In::Off Off;
    const In X(P, B0);
    const Off ldb = (Off)P.ld * (Off)sizeof(T), kst = (Off)(NxI * NyI) * ldb;
    Off o0 = (Off)(cp.row(P) - X.first + NxI * j) * ldb + (Off)colg * (Off)sizeof(T);
    if (!act || (j == 0 && cp.y == 0) || (j == N - 1 && cp.y == P.ncy - 1)) o0 = In::NONE;
#pragma unroll
    for (int k = 0; k < N; ++k) {
      Off ok = o0 + k * kst;
      if (k == 0 && cp.z == 0) ok = In::NONE;
      if (k == N - 1 && cp.z == P.ncz - 1) ok = In::NONE;
#pragma unroll
      for (int i = 0; i < N; ++i) {
        Off o = ok + i * ldb;
        if (i == 0 && cp.x == 0) o = In::NONE;
        if (i == N - 1 && cp.x == P.ncx - 1) o = In::NONE;
        u[i][k] = X.load(o);
      }
    }
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const int q = t + k * THREADS;
      if (q < CPB * VOL) sV[q] = vr[k];
    }
#pragma unroll
    for (int k = 0; k < NF; ++k) {
      const int f = t + k * THREADS;
      if (f < CPB * NFC) sF[f] = fr[k];
    }
    __syncthreads();
    // (the y factor goes into the z factors in FP64: two roundings fewer per
    // value in FP32)
    const double my = sFc[N + j] * (cs * FS.in);
    T fx[N], fz[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
      fx[q] = (T)sFc[q];
      fz[q] = (T)(sFc[2 * N + q] * my);
    }
#pragma unroll
    for (int k = 0; k < N; ++k)
#pragma unroll
      for (int i = 0; i < N; ++i) u[i][k] *= fx[i] * fz[k];
    if constexpr (XFIRST) {
      // x, per z node: interpolation and S B; z of both, per x point: the first
      // into the transpose buffer
      T v[N][N];
#pragma unroll
      for (int k = 0; k < N; ++k) {
        T line[N], o1[N], o2[N];
#pragma unroll
        for (int i = 0; i < N; ++i) line[i] = u[i][k];
        interp(line, o1);
        eo0<T, N>(FS.SB, line, o2);
#pragma unroll
        for (int a = 0; a < N; ++a) {
          v[a][k] = o1[a];
          u[a][k] = o2[a];
        }
      }
#pragma unroll
      for (int a = 0; a < N; ++a) {
        T o1[N], o2[N];
        interp(v[a], o1);
        eo<T, N, 1>(FS.B, u[a], o2);
#pragma unroll
        for (int c = 0; c < N; ++c) {
          sX[sidx(pl, a, c)] = o1[c];
          u[a][c] = o2[c];
        }
      }
    } else {
      // z: interpolation, per x node
#pragma unroll
      for (int i = 0; i < N; ++i) {
        T o[N];
        interp(u[i], o);
#pragma unroll
        for (int c = 0; c < N; ++c) u[i][c] = o[c];
      }
      // x, per z point: interpolation into the transpose buffer, S B kept
#pragma unroll
      for (int c = 0; c < N; ++c) {
        T line[N], o1[N], o2[N];
#pragma unroll
        for (int i = 0; i < N; ++i) line[i] = u[i][c];
        interp(line, o1);
        eo0<T, N>(FS.SB, line, o2);
#pragma unroll
        for (int a = 0; a < N; ++a) {
          sX[sidx(pl, a, c)] = o1[a];
          u[a][c] = o2[a];
        }
      }
    }
  }
  __syncthreads();
  // ---------------- transposes (j; a, c) -> (a; j, c), y interpolation of u ----------------
  T uq[N][N];  // [b][c] at x point a = pl
#pragma unroll
  for (int c = 0; c < N; ++c) {
    T l[N], o[N];
#pragma unroll
    for (int j = 0; j < N; ++j) l[j] = sX[sidx(j, pl, c)];
    interp(l, o);
#pragma unroll
    for (int b = 0; b < N; ++b) uq[b][c] = o[b];
  }
  __syncthreads();
#pragma unroll
  for (int a = 0; a < N; ++a)
#pragma unroll
    for (int c = 0; c < N; ++c) sX[sidx(pl, a, c)] = u[a][c];
  __syncthreads();

  // ---------------- B: plane a = pl, quadrature values (b, c) --------------------------------
  double energy = 0.0;
  T gx = 0, gy = 0, gz = 0;
  if (cell_ok) {
    // Gauss weight of this thread's x point, selected from the constants (an
    // array indexed per lane would be a memory load and a wait)
    double wa = FS.wq[0];
#pragma unroll
    for (int q = 1; q < N; ++q) wa = pl == q ? FS.wq[q] : wa;
    gx = (T)(P.kin * FS.gx * sFc[3 * N + 0]);  // S B carries the x weights
    gy = (T)(P.kin * FS.gs * sFc[3 * N + 1] * wa);
    gz = (T)(P.kin * FS.gs * sFc[3 * N + 2] * wa);
  }
  // x stiffness term and the potential, per z point
  T acc[N][N];
#pragma unroll
  for (int c = 0; c < N; ++c) {
    T l[N], o[N];
#pragma unroll
    for (int j = 0; j < N; ++j) l[j] = sX[sidx(j, pl, c)];
    eo<T, N, 1>(FS.B, l, o);
#pragma unroll
    for (int b = 0; b < N; ++b) {
      const T f = gx * wprod(b, c) * o[b];
      acc[b][c] = sV[slot * VOL + pl + N * (b + N * c)] * uq[b][c] + f;  // (0 without a potential)
    }
    // keep the potential reads of later lines from being hoisted here
    __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
  // z stiffness term, per y point
#pragma unroll
  for (int b = 0; b < N; ++b) {
    T d[N];
    eo0<T, N>(FS.S, uq[b], d);
    const T g = gz * (T)FS.wq[b];
#pragma unroll
    for (int c = 0; c < N; ++c) acc[b][c] += g * d[c];
  }
  // y stiffness term, the quadratic form u_q . (sum) and the transposed y
  // interpolation into the transpose buffer, per z point
#pragma unroll
  for (int c = 0; c < N; ++c) {
    T l[N], d[N];
#pragma unroll
    for (int b = 0; b < N; ++b) l[b] = uq[b][c];
    eo0<T, N>(FS.S, l, d);
    const T g = gy * (T)FS.wq[c];
    T le = 0;
#pragma unroll
    for (int b = 0; b < N; ++b) {
      d[b] = g * d[b] + acc[b][c];
      acc_energy<T>(energy, le, d[b] * l[b]);
    }
    flush_energy<T>(energy, le);
    eo<T, N, 1>(FS.Bt, d, l);
#pragma unroll
    for (int j = 0; j < N; ++j) sX[sidx(j, pl, c)] = l[j];
  }
  // the quadratic form is parked in LDS here, unconditionally: otherwise the
  // compiler sinks its whole accumulation chain into the final reduction and
  // keeps every partial product alive across phase C
  sRed[t] = act ? energy : 0.0;
  __syncthreads();

  // ---------------- C: plane j = pl: x then z transposed, scatter ------------------------------
  {
    const int j = pl;
    T h[N][N];  // [i][c]
#pragma unroll
    for (int c = 0; c < N; ++c) {
      T l[N], o[N];
#pragma unroll
      for (int a = 0; a < N; ++a) l[a] = sX[sidx(pl, a, c)];
      eo<T, N, 1>(FS.Bt, l, o);
#pragma unroll
      for (int i = 0; i < N; ++i) h[i][c] = o[i];
    }
    T fx[N], fz[N];
    const double my = sFc[N + j] * FS.out;
#pragma unroll
    for (int q = 0; q < N; ++q) {
      fx[q] = (T)sFc[q];
      fz[q] = (T)(sFc[2 * N + q] * my);
    }
    const CellOut<T, N, CELLS, FAR> E(Y, P, B0, cp, c0, slot, j, colg, act);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      T o[N];
      eo<T, N, 1>(FS.Bt, h[i], o);
      if (E.jok && E.xok(i)) {
#pragma unroll
        for (int k = 0; k < N; ++k)
          if (E.zok(k)) E.put(i, k, E.off, o[k] * (fx[i] * fz[k]));
      }
    }
  }
  // ---------------- per-column quadratic form -------------------------------------------------
  if (P.energy) {
    __syncthreads();
    if (t < CB) {
      double acc = 0.0;
      for (int u = t; u < THREADS; u += CB) acc += sRed[u];
      if (chunk * CB + t < P.cols) P.energy[(int64_t)group * P.eld + chunk * CB + t] = acc;
    }
  }
}

// ----------------------------------------------------------------------------------------------
// host side
// ----------------------------------------------------------------------------------------------

// LDS bytes of one block of cpb cells
template <typename T, int N, int CB>
constexpr int plane_lds(int cpb) {
  constexpr int VOL = N * N * N;
  return cpb * VOL * CB * (int)sizeof(T) + cpb * VOL * (int)sizeof(T) +
         cpb * N * CB * 8 + cpb * (3 * N + 3) * 8;
}

// cells per block: at most 512 threads, and LDS small enough for the
// occupancy plane_wpe asks for (an FP64 block must also fit one CU at one wave
// per SIMD: at most four waves).  Up to four columns a block is one wavefront:
// barriers cost nothing, few cells spread over more of the chip, and the
// per-column sums over the block stay short (a complex FP64 column at p = 4
// on 4^3 cells 12.7 -> 11.7 us and on 28^3 57.8 -> 57.0, two FP64 columns
// there 81.7 -> 76.0, an FP32 one at p = 3 on 4^3 12.9 -> 10.4; no size or
// order was slower by more than 2%)
template <typename T, int N, int CB>
constexpr int plane_cpb() {
  constexpr int budget = sizeof(T) == 8 ? 64 * 1024 : 40 * 1024;
  if (CB <= 4) return 64 / (N * CB);
  int cpb = 1;
  while (cpb * 2 * N * CB <= 512 && plane_lds<T, N, CB>(cpb * 2) <= budget) cpb *= 2;
  return cpb;
}

template <typename T, int N, int CB>
tdfe_status launch_plane(tdfe_ctx* c, PlaneParams<T>& P, int64_t* groups_out) {
  constexpr int CPB = plane_cpb<T, N, CB>();
  if (P.query) {
    *groups_out = CPB;
    return TDFE_OK;
  }
  const int64_t groups = (c->n_cell + CPB - 1) / CPB;
  P.nchunks = (P.cols + CB - 1) / CB;
  if (groups_out) *groups_out = groups;
  const dim3 grid((unsigned)(groups * P.nchunks)), block(CPB * N * CB);
  if (P.cells)
    hipLaunchKernelGGL((plane_kernel<T, N, CB, CPB, true, false>), grid, block, 0, c->stream, P);
  else if (P.far)
    hipLaunchKernelGGL((plane_kernel<T, N, CB, CPB, false, true>), grid, block, 0, c->stream, P);
  else
    hipLaunchKernelGGL((plane_kernel<T, N, CB, CPB, false, false>), grid, block, 0, c->stream, P);
  TDFE_HIP(c, hipGetLastError());
  return TDFE_OK;
}

template <typename T, int N>
tdfe_status launch_plane_n(tdfe_ctx* c, PlaneParams<T>& P, int64_t* g) {
  if (P.cols <= 1) return launch_plane<T, N, 1>(c, P, g);
  if (P.cols <= 2) return launch_plane<T, N, 2>(c, P, g);
  if (P.cols <= 4) return launch_plane<T, N, 4>(c, P, g);
  if (P.cols <= 8) return launch_plane<T, N, 8>(c, P, g);
  return launch_plane<T, N, 16>(c, P, g);
}

template <typename T>
tdfe_status launch_plane_p(tdfe_ctx* c, PlaneParams<T>& P, int64_t* g) {
  switch (c->n) {
    case 2: return launch_plane_n<T, 2>(c, P, g);
    case 3: return launch_plane_n<T, 3>(c, P, g);
    case 4: return launch_plane_n<T, 4>(c, P, g);
    case 5: return launch_plane_n<T, 5>(c, P, g);
    case 6: return launch_plane_n<T, 6>(c, P, g);
    case 7: return launch_plane_n<T, 7>(c, P, g);
    case 8: return launch_plane_n<T, 8>(c, P, g);
  }
  return tdfe_fail(c, TDFE_EINVAL, "box operator: unsupported order p=%d", c->p);
}


template <typename T>
tdfe_status launch_box(tdfe_ctx* c, const ApplyArgs& a) {
  static_assert(sizeof(PlaneParams<T>) <= 4096, "kernel arguments exceed 4 KB");
  PlaneParams<T> P{};
  P.x = a.x;
  P.y = a.y;
  P.ld = a.ld;
  P.cols = a.cols;
  P.colscale = a.colscale;
  P.kin = a.kin;
  P.vw = a.fp32 ? (const void*)a.vw32 : (const void*)a.vw;
  P.minv = c->minv;
  P.m1x = c->m1x;
  P.m1y = c->m1y;
  P.m1z = c->m1z;
  P.cellgeo = c->cellgeo;
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
  P.eld = a.eld;
  P.cells = a.cells;
  P.far = a.far;
  P.query = a.query;
  const int N = c->n;
  for (int i = 0; i < N; ++i) P.wq[i] = c->wq[i];
  return launch_plane_p<T>(c, P, a.n_blocks_out);
}

}  // namespace

// true if the box kernel handles this context (rectilinear mesh, p <= 7)
bool tdfe_box_kernel_ok(const tdfe_ctx* c) { return c->box && c->n <= 8; }

tdfe_status tdfe_launch_apply_box(tdfe_ctx* c, const ApplyArgs& a) {
  if (a.cols < 1) return tdfe_fail(c, TDFE_EINVAL, "apply: cols < 1");
  return a.fp32 ? launch_box<float>(c, a) : launch_box<double>(c, a);
}
