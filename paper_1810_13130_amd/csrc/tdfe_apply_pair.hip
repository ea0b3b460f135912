// Operator kernel for rectilinear (box) cells, even n: two lanes per plane.
//
// The same operator and phase order as the plane kernel (Eq. DiscreteHamiltonian
// in the Loewdin form, Eq. TDKSMatVecStandard), but the n x n plane of one
// column is shared by an adjacent lane pair: each lane holds the half of the z
// index range that is its own, lane 0 the indices 0..n/2-1 and lane 1 their
// mirror images n-1..n/2, both in local order.  Contractions along x and y stay
// inside a lane (even/odd folded, as in the plane kernel); a contraction along
// z forms, in each lane, the partial sums over its own inputs for its own
// outputs and for the partner's, and swaps the latter with the partner by a DPP
// quad permutation.  The mirror symmetry of the 1D tables
// (A[n-1-c][n-1-k] = A[c][k] for B, S and S B, see the plane kernel) makes the
// two lanes run identical code with identical coefficients.  All tables are
// compile-time constants (make_pairset).  A lane then keeps half the registers
// of a plane-owning thread, which lets FP64 run two waves per SIMD.
#include "tdfe_fold.h"

namespace {

constexpr int PH = 4;  // largest half order (n = 8)

// folded table of an even-order matrix (no middle row or column)
template <typename T>
struct FoldE {
  T E[PH * PH];  // (A[a][i] + A[a][n-1-i]) / 2, a, i < n/2
  T O[PH * PH];  // (A[a][i] - A[a][n-1-i]) / 2
};

// split table of a matrix for a contraction along the paired direction:
// own[cc][kk] = A[cc][kk], oth[cc][kk] = A[n-1-cc][kk]
template <typename T>
struct SplitT {
  T own[PH * PH];
  T oth[PH * PH];
};

template <typename T>
struct PairParams {
  const void* x;
  void* y;  // CELLS: per-cell results [n_cell][n^3][cols]; else the DoF vector, added to
  int ld, cols, nchunks, eld;
  const double* colscale;
  double kin;
  const void* vw;
  const double* m1x;  // separable M^-1/2 factors: minv(I,J,K) = m1x[I] m1y[J] m1z[K]
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
  double wq[TDFE_MAXN];
};

// the kernel's tables for order N, evaluated at compile time
struct PairSet {
  FoldE<double> fB, fBt, fS, fSB;  // B, B^T, S, S B (x and y directions)
  SplitT<double> zB, zBt, zS;      // B, B^T, S along z
  double wq[TDFE_MAXN];
  double in = 1.0, out = 1.0, gx = 1.0, gy = 1.0, gz = 1.0;  // as in BoxFoldSet
};

constexpr void fold_even(const double* A, int N, bool transpose, FoldE<double>& F) {
  const int H = N / 2;
  for (int a = 0; a < H; ++a)
    for (int i = 0; i < H; ++i) {
      const double ai = transpose ? A[i * TDFE_MAXN + a] : A[a * TDFE_MAXN + i];
      const double aj = transpose ? A[(N - 1 - i) * TDFE_MAXN + a] : A[a * TDFE_MAXN + N - 1 - i];
      F.E[a * PH + i] = 0.5 * (ai + aj);
      F.O[a * PH + i] = 0.5 * (ai - aj);
    }
}

constexpr void split_tab(const double* A, int N, bool transpose, SplitT<double>& F) {
  const int H = N / 2;
  for (int c = 0; c < H; ++c)
    for (int k = 0; k < H; ++k) {
      F.own[c * PH + k] = transpose ? A[k * TDFE_MAXN + c] : A[c * TDFE_MAXN + k];
      F.oth[c * PH + k] = transpose ? A[k * TDFE_MAXN + N - 1 - c] : A[(N - 1 - c) * TDFE_MAXN + k];
    }
}

template <int N, bool F32>
constexpr PairSet make_pairset() {
  const tdfe1d::Rule R = tdfe1d::make_rule(N - 1);
  const GaussStiff K = make_gauss_stiff(R);
  PairSet F{};
  fold_even(R.B, N, false, F.fB);
  fold_even(R.B, N, true, F.fBt);
  fold_even(K.S, N, false, F.fS);
  fold_even(K.SB, N, false, F.fSB);
  split_tab(R.B, N, false, F.zB);
  split_tab(R.B, N, true, F.zBt);
  split_tab(K.S, N, false, F.zS);
  if (F32) {
    constexpr F32Factors f = f32_factors(N);
    for (int i = 0; i < PH * PH; ++i) {
      F.fB.E[i] *= f.B;
      F.fB.O[i] *= f.B;
      F.fBt.E[i] *= f.Bt;
      F.fBt.O[i] *= f.Bt;
      F.fS.E[i] *= f.S;
      F.fS.O[i] *= f.S;
      F.fSB.E[i] *= f.SB;
      F.fSB.O[i] *= f.SB;
      F.zB.own[i] *= f.zB;
      F.zB.oth[i] *= f.zB;
      F.zBt.own[i] *= f.zB;
      F.zBt.oth[i] *= f.zB;
      F.zS.own[i] *= f.zS;
      F.zS.oth[i] *= f.zS;
    }
    F.in = 1.0 / (f.B * f.B * f.zB);
    F.out = 1.0 / (f.Bt * f.Bt * f.zB);
    F.gx = f.B / f.SB;
    F.gy = 1.0 / f.S;
    F.gz = 1.0 / f.zS;
  }
  for (int i = 0; i < TDFE_MAXN; ++i) F.wq[i] = R.wq[i];
  return F;
}

// out[a] = sum_i A[a][i] in[i], A folded with A[n-1-a][n-1-i] = A[a][i] (even N)
// ZERO: A sends a constant to zero (as eo0)
template <typename T, int N, bool ZERO = false>
__device__ __forceinline__ void eoe(const FoldE<double>& F, const T* in, T* out) {
  constexpr int H = N / 2, HE = ZERO ? H - 1 : H;
  T e[H], o[H];
#pragma unroll
  for (int i = 0; i < H; ++i) {
    e[i] = in[i] + in[N - 1 - i];
    o[i] = in[i] - in[N - 1 - i];
  }
  if constexpr (ZERO)
#pragma unroll
    for (int i = 0; i < HE; ++i) e[i] -= e[H - 1];
#pragma unroll
  for (int a = 0; a < H; ++a) {
    T Pv = 0, Qv = 0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      if (i < HE) Pv += (T)F.E[a * PH + i] * e[i];
      Qv += (T)F.O[a * PH + i] * o[i];
    }
    out[a] = Pv + Qv;
    out[N - 1 - a] = Pv - Qv;
  }
}

// value of the partner lane (lane ^ 1)
template <typename T>
__device__ __forceinline__ T pair_swap(T v) {
  if constexpr (sizeof(T) == 8) {
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0xB1, 0xf, 0xf, false);  // quad_perm 1,0,3,2
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0xB1, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
  } else {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xf, 0xf, false));
  }
}

// contraction along the paired direction: in/out hold this lane's H local
// entries
template <typename T, int N>
__device__ __forceinline__ void zsplit(const SplitT<double>& F, const T* x, T* out) {
  constexpr int H = N / 2;
  T own[H], oth[H];
#pragma unroll
  for (int c = 0; c < H; ++c) {
    T a = 0, b = 0;
#pragma unroll
    for (int k = 0; k < H; ++k) {
      a += (T)F.own[c * PH + k] * x[k];
      b += (T)F.oth[c * PH + k] * x[k];
    }
    own[c] = a;
    oth[c] = b;
  }
#pragma unroll
  for (int c = 0; c < H; ++c) out[c] = own[c] + pair_swap(oth[c]);
}

template <typename T, int N>
constexpr int pair_wpe() {
  return sizeof(T) == 8 ? 2 : 3;
}

template <typename T, int N, int CB, int CPB, bool CELLS, bool FAR>
__global__ void __launch_bounds__(2 * CPB * N * CB) __attribute__((amdgpu_waves_per_eu(pair_wpe<T, N>())))
    pair_kernel(PairParams<T> P) {
  static_assert(N % 2 == 0 && N / 2 <= PH, "even n <= 8");
  constexpr int H = N / 2;
  constexpr int VOL = N * N * N;
  constexpr int THREADS = 2 * CPB * N * CB;
  constexpr PairSet FS = make_pairset<N, sizeof(T) == 4>();
  __shared__ T sX[CPB * VOL * CB];
  __shared__ T sV[CPB * VOL];
  __shared__ double sRed[THREADS];
  if (P.done && *P.done) return;

  const int t = threadIdx.x;
  const int h = t & 1;  // half of the z range
  const int r = t >> 1;
  const int L = remap_block(blockIdx.x, gridDim.x);
  const int chunk = L % P.nchunks;
  const int group = L / P.nchunks;
  const int col = r % CB;
  const int pl = (r / CB) % N;
  const int slot = CPB == 1 ? 0 : r / (CB * N);
  const int64_t cell = (int64_t)group * CPB + slot;
  const bool cell_ok = cell < P.n_cell;
  const int colg = chunk * CB + col;
  const bool act = cell_ok && colg < P.cols;
  // global z index of local entry q
  auto zg = [&](int q) { return h ? N - 1 - q : q; };

  const int64_t c0 = (int64_t)group * CPB;
  const CellPos B0 = cell_pos(P, (int)c0);
  const CellPos cp = CPB == 1 ? B0 : cell_next(P, B0, cell_ok ? slot : 0);
  T* __restrict__ Y = (T*)P.y;
  double cs = 1.0;
  if (P.colscale && act) cs = P.colscale[colg >> 1];

  // block staging (as in the plane kernel): potential, M^-1/2 factors along
  // x, y, z and the metric of the block's cells; loads issued before the
  // phase A gather, LDS stores after it, one wait for memory per wave
  constexpr int NFC = 3 * N + 3;
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
    const double* src = r < N ? P.m1x + (e.x * P.p + r)
                        : r < 2 * N ? P.m1y + (e.y * P.p + r - N)
                        : r < 3 * N ? P.m1z + (e.z * P.p + r - 2 * N)
                                    : P.cellgeo + (cv * 4 + r - 3 * N);
    const double val = *src;
    fr[k] = ok ? val : 0.0;
  }
  const double* sFc = sF + slot * NFC;
  auto sidx = [&](int y, int x, int z) { return (((slot * N + y) * N + x) * N + z) * CB + col; };
  const int NxI = P.Nx - 2, NyI = P.Ny - 2;

  // Loewdin factors of node plane j = pl (phases A and C; read again in C
  // rather than held through B)
  struct PlaneFactors {
    T fx[N], fz[H];
  };
  auto plane_factors = [&](PlaneFactors& Q, double s) {
    const double my = sFc[N + pl] * s;
#pragma unroll
    for (int q = 0; q < N; ++q) Q.fx[q] = (T)sFc[q];
#pragma unroll
    for (int q = 0; q < H; ++q) Q.fz[q] = (T)(sFc[2 * N + zg(q)] * my);
  };

  // ---------------- A: plane j = pl, values (i, local k) ---------------------------------
  T u[N][H];  // [i][local k] gathered, then [i][c], then S B u at [x point][local z point]
  {
    typedef CellIn<T, FAR> In;
    typedef typename In::Off Off;
    const In X(P, B0);
    const Off ldb = (Off)P.ld * (Off)sizeof(T), kst = (Off)(NxI * NyI) * ldb;
    Off o0 = (Off)(cp.row(P) - X.first + NxI * pl) * ldb + (Off)colg * (Off)sizeof(T);
    if (!act || (pl == 0 && cp.y == 0) || (pl == N - 1 && cp.y == P.ncy - 1)) o0 = In::NONE;
#pragma unroll
    for (int k = 0; k < H; ++k) {
      Off ok = o0 + (Off)zg(k) * kst;
      if (k == 0 && (h ? cp.z == P.ncz - 1 : cp.z == 0)) ok = In::NONE;
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
    PlaneFactors Q;
    plane_factors(Q, cs * FS.in);
#pragma unroll
    for (int k = 0; k < H; ++k)
#pragma unroll
      for (int i = 0; i < N; ++i) u[i][k] *= Q.fx[i] * Q.fz[k];
    if constexpr (sizeof(T) == 4) {
      // FP32: x first, on the nodes (see the plane kernel)
      T v[N][H];
#pragma unroll
      for (int k = 0; k < H; ++k) {
        T line[N], o1[N], o2[N];
#pragma unroll
        for (int i = 0; i < N; ++i) line[i] = u[i][k];
        eoe<T, N>(FS.fB, line, o1);
        eoe<T, N, true>(FS.fSB, line, o2);
#pragma unroll
        for (int a = 0; a < N; ++a) {
          v[a][k] = o1[a];
          u[a][k] = o2[a];
        }
      }
#pragma unroll
      for (int a = 0; a < N; ++a) {
        T o1[H], o2[H];
        zsplit<T, N>(FS.zB, v[a], o1);
        zsplit<T, N>(FS.zB, u[a], o2);
#pragma unroll
        for (int c = 0; c < H; ++c) {
          sX[sidx(pl, a, zg(c))] = o1[c];
          u[a][c] = o2[c];
        }
      }
    } else {
      // z: interpolation (paired), per x node
#pragma unroll
      for (int i = 0; i < N; ++i) {
        T o[H];
        zsplit<T, N>(FS.zB, u[i], o);
#pragma unroll
        for (int c = 0; c < H; ++c) u[i][c] = o[c];
      }
      // x, per local z point: interpolation into the transpose buffer, S B kept
#pragma unroll
      for (int c = 0; c < H; ++c) {
        T line[N], o1[N], o2[N];
#pragma unroll
        for (int i = 0; i < N; ++i) line[i] = u[i][c];
        eoe<T, N>(FS.fB, line, o1);
        eoe<T, N, true>(FS.fSB, line, o2);
#pragma unroll
        for (int a = 0; a < N; ++a) {
          sX[sidx(pl, a, zg(c))] = o1[a];
          u[a][c] = o2[a];
        }
      }
    }
  }
  __syncthreads();
  // ---------------- transposes (j; a, c) -> (a; j, c), y interpolation of u ----------------
  T uq[N][H];  // [b][local c] at x point a = pl
#pragma unroll
  for (int c = 0; c < H; ++c) {
    T l[N], o[N];
#pragma unroll
    for (int j = 0; j < N; ++j) l[j] = sX[sidx(j, pl, zg(c))];
    eoe<T, N>(FS.fB, l, o);
#pragma unroll
    for (int b = 0; b < N; ++b) uq[b][c] = o[b];
  }
  __syncthreads();
#pragma unroll
  for (int a = 0; a < N; ++a)
#pragma unroll
    for (int c = 0; c < H; ++c) sX[sidx(pl, a, zg(c))] = u[a][c];
  __syncthreads();

  // ---------------- B: plane a = pl, Gauss points (b, local c) ---------------------------------
  double energy = 0.0;
  T gx = 0, gy = 0, gz = 0;
  if (cell_ok) {
    double wa = FS.wq[0];  // selected from the constants: no per-lane memory load
#pragma unroll
    for (int q = 1; q < N; ++q) wa = pl == q ? FS.wq[q] : wa;
    gx = (T)(P.kin * FS.gx * sFc[3 * N + 0]);  // S B carries the x weights
    gy = (T)(P.kin * FS.gy * sFc[3 * N + 1] * wa);
    gz = (T)(P.kin * FS.gz * sFc[3 * N + 2] * wa);
  }
  // z Gauss weights of this lane's points: the rule's weights are symmetric
  // (bitwise, for every order), so the mirror point's weight is wq[c] itself
  T wc[H];
#pragma unroll
  for (int c = 0; c < H; ++c) wc[c] = (T)FS.wq[c];
  // x stiffness term and the potential, per local z point
  T acc[N][H];
#pragma unroll
  for (int c = 0; c < H; ++c) {
    T l[N], o[N];
#pragma unroll
    for (int j = 0; j < N; ++j) l[j] = sX[sidx(j, pl, zg(c))];
    eoe<T, N>(FS.fB, l, o);
#pragma unroll
    for (int b = 0; b < N; ++b) {
      const T f = gx * ((T)FS.wq[b] * wc[c]) * o[b];
      acc[b][c] = sV[slot * VOL + pl + N * (b + N * zg(c))] * uq[b][c] + f;  // (0 without a potential)
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  __syncthreads();
  // z stiffness term, per y point (paired contraction)
#pragma unroll
  for (int b = 0; b < N; ++b) {
    T d[H];
    zsplit<T, N>(FS.zS, uq[b], d);
    const T g = gz * (T)FS.wq[b];
#pragma unroll
    for (int c = 0; c < H; ++c) acc[b][c] += g * d[c];
  }
  // y stiffness term, the quadratic form u_q . (sum) and the transposed y
  // interpolation into the transpose buffer, per local z point
#pragma unroll
  for (int c = 0; c < H; ++c) {
    T l[N], d[N];
#pragma unroll
    for (int b = 0; b < N; ++b) l[b] = uq[b][c];
    eoe<T, N, true>(FS.fS, l, d);
    const T g = gy * wc[c];
    T le = 0;
#pragma unroll
    for (int b = 0; b < N; ++b) {
      d[b] = g * d[b] + acc[b][c];
      acc_energy<T>(energy, le, d[b] * l[b]);
    }
    flush_energy<T>(energy, le);
    eoe<T, N>(FS.fBt, d, l);
#pragma unroll
    for (int j = 0; j < N; ++j) sX[sidx(j, pl, zg(c))] = l[j];
  }
  sRed[t] = act ? energy : 0.0;
  __syncthreads();

  // ---------------- C: plane j = pl: x transposed, z transposed (paired), scatter -------------------
  {
    T hh[N][H];  // [x node][local z point]
#pragma unroll
    for (int c = 0; c < H; ++c) {
      T l[N], o[N];
#pragma unroll
      for (int a = 0; a < N; ++a) l[a] = sX[sidx(pl, a, zg(c))];
      eoe<T, N>(FS.fBt, l, o);
#pragma unroll
      for (int i = 0; i < N; ++i) hh[i][c] = o[i];
    }
    PlaneFactors Q;
    plane_factors(Q, FS.out);
    const CellOut<T, N, CELLS, FAR> E(Y, P, B0, cp, c0, slot, pl, colg, act);
    typedef typename CellOut<T, N, CELLS, FAR>::Off Off;
    Off oz[H];  // this lane's z entries
#pragma unroll
    for (int k = 0; k < H; ++k) oz[k] = E.off + (Off)zg(k) * (Off)E.sz;
    const bool z0 = h ? E.hiz : E.loz;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      T o[H];
      zsplit<T, N>(FS.zBt, hh[i], o);
      if (E.jok && E.xok(i)) {
#pragma unroll
        for (int k = 0; k < H; ++k)
          if (k > 0 || z0) E.put(i, 0, oz[k], o[k] * (Q.fx[i] * Q.fz[k]));
      }
    }
  }
  // ---------------- per-column quadratic form ----------------------------------------------------
  if (P.energy) {
    __syncthreads();
    if (t < CB) {
      double acc = 0.0;
      for (int u = 2 * t; u < THREADS; u += 2 * CB) acc += sRed[u] + sRed[u + 1];
      if (chunk * CB + t < P.cols) P.energy[(int64_t)group * P.eld + chunk * CB + t] = acc;
    }
  }
}

// ----------------------------------------------------------------------------------------------
// host side
// ----------------------------------------------------------------------------------------------

template <typename T, int N, int CB>
constexpr int pair_lds(int cpb) {
  constexpr int VOL = N * N * N;
  return cpb * VOL * CB * (int)sizeof(T) + cpb * VOL * (int)sizeof(T) + 2 * cpb * N * CB * 8 + cpb * (3 * N + 3) * 8;
}

// cells per block: at most 256 threads (blocks of a few waves pack the CUs
// at two or more waves per SIMD) and LDS for the occupancy pair_wpe asks for
template <typename T, int N, int CB>
constexpr int pair_cpb() {
  constexpr int budget = sizeof(T) == 8 ? 64 * 1024 : 40 * 1024;
  int cpb = 1;
  while (2 * cpb * 2 * N * CB <= 256 && pair_lds<T, N, CB>(cpb * 2) <= budget) cpb *= 2;
  return cpb;
}

template <typename T, int N, int CB>
tdfe_status launch_pair(tdfe_ctx* c, PairParams<T>& P, int64_t* groups_out) {
  constexpr int CPB = pair_cpb<T, N, CB>();
  static_assert(pair_lds<T, N, CB>(CPB) <= 160 * 1024, "LDS");
  if (P.query) {
    *groups_out = CPB;
    return TDFE_OK;
  }
  const int64_t groups = (c->n_cell + CPB - 1) / CPB;
  P.nchunks = (P.cols + CB - 1) / CB;
  if (groups_out) *groups_out = groups;
  const dim3 grid((unsigned)(groups * P.nchunks)), block(2 * CPB * N * CB);
  if (P.cells)
    hipLaunchKernelGGL((pair_kernel<T, N, CB, CPB, true, false>), grid, block, 0, c->stream, P);
  else if (P.far)
    hipLaunchKernelGGL((pair_kernel<T, N, CB, CPB, false, true>), grid, block, 0, c->stream, P);
  else
    hipLaunchKernelGGL((pair_kernel<T, N, CB, CPB, false, false>), grid, block, 0, c->stream, P);
  TDFE_HIP(c, hipGetLastError());
  return TDFE_OK;
}

template <typename T, int N>
tdfe_status launch_pair_n(tdfe_ctx* c, PairParams<T>& P, int64_t* g) {
  if (P.cols <= 1) return launch_pair<T, N, 1>(c, P, g);
  if (P.cols <= 2) return launch_pair<T, N, 2>(c, P, g);
  if (P.cols <= 4) return launch_pair<T, N, 4>(c, P, g);
  if (P.cols <= 8) return launch_pair<T, N, 8>(c, P, g);
  return launch_pair<T, N, 16>(c, P, g);
}

template <typename T>
tdfe_status launch_pair_box(tdfe_ctx* c, const ApplyArgs& a) {
  static_assert(sizeof(PairParams<T>) <= 4096, "kernel arguments exceed 4 KB");
  PairParams<T> P{};
  P.x = a.x;
  P.y = a.y;
  P.ld = a.ld;
  P.cols = a.cols;
  P.colscale = a.colscale;
  P.kin = a.kin;
  P.vw = a.fp32 ? (const void*)a.vw32 : (const void*)a.vw;
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
  switch (N) {
    case 2: return launch_pair_n<T, 2>(c, P, a.n_blocks_out);
    case 4: return launch_pair_n<T, 4>(c, P, a.n_blocks_out);
    case 6: return launch_pair_n<T, 6>(c, P, a.n_blocks_out);
    case 8: return launch_pair_n<T, 8>(c, P, a.n_blocks_out);
  }
  return tdfe_fail(c, TDFE_EINVAL, "paired box operator: order p=%d is not odd", c->p);
}

}  // namespace

// true if the lane-pair box kernel can handle this context (rectilinear mesh, odd p <= 7)
bool tdfe_pair_kernel_ok(const tdfe_ctx* c) { return c->box && c->n % 2 == 0 && c->n <= 8; }

tdfe_status tdfe_launch_apply_pair(tdfe_ctx* c, const ApplyArgs& a) {
  if (a.cols < 1) return tdfe_fail(c, TDFE_EINVAL, "apply: cols < 1");
  if (!tdfe_pair_kernel_ok(c)) return tdfe_fail(c, TDFE_EINVAL, "paired box operator: unsupported mesh or order");
  return a.fp32 ? launch_pair_box<float>(c, a) : launch_pair_box<double>(c, a);
}
