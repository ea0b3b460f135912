// Even/odd folded 1D tables and the small-matvec helpers shared by the
// plane-ownership operator kernels (box and trilinear cells).  The GLL nodes
// and Gauss points are symmetric about 0, so B[n-1-a][n-1-i] = B[a][i] and D,
// Dg are antisymmetric: a 1D contraction splits into an even and an odd half
// of size n/2 each.
#pragma once
#include <type_traits>

#include "tdfe_internal.h"
#include "tdfe_rule1d.h"
#include "tdfe_span.h"

namespace {

constexpr int EO_MAX_H = 5;  // (9 + 1) / 2

// folded form of one N x N matrix with reflection symmetry S (+1 or -1), in the
// kernel's working precision (no conversions at the point of use)
template <typename T>
struct Folded {
  T E[EO_MAX_H * EO_MAX_H];  // (A[a][i] + A[a][N-1-i]) / 2, a, i < H
  T O[EO_MAX_H * EO_MAX_H];  // (A[a][i] - A[a][N-1-i]) / 2
  T mc[EO_MAX_H];            // A[a][H] (odd N)
  T mr[EO_MAX_H + 1];        // A[H][i], i <= H (odd N)
};

// the six folded tables of order N (B, B^T, D, D^T, Dg, Dg^T) and the Gauss
// weights, evaluated at compile time: a kernel declares
//   constexpr FoldSet<N> FS = make_foldset<N>();
// and every coefficient becomes a constant of the instruction stream
template <int N>
struct FoldSet {
  Folded<double> B, Bt, D, Dt, G, Gt;
  double wq[TDFE_MAXN];
};

// The 1D stiffness of the Gauss-point Lagrange basis, S = Dg^T diag(w) Dg, and
// S B (nodes to points).  On box cells, whose metric is one diagonal per
// cell, a direction's derivative, flux and transposed derivative are S along
// it times the other two directions' weights: one contraction instead of two.
// S is symmetric under reflection of both indices, so it folds as B does.
struct GaussStiff {
  double S[TDFE_MAXN * TDFE_MAXN];
  double SB[TDFE_MAXN * TDFE_MAXN];
};
constexpr GaussStiff make_gauss_stiff(const tdfe1d::Rule& R) {
  GaussStiff G{};
  const int n = R.n;
  for (int a = 0; a < n; ++a)
    for (int b = 0; b < n; ++b) {
      double v = 0.0;
      for (int q = 0; q < n; ++q) v += R.wq[q] * R.Dg[q * TDFE_MAXN + a] * R.Dg[q * TDFE_MAXN + b];
      G.S[a * TDFE_MAXN + b] = v;
    }
  for (int a = 0; a < n; ++a)
    for (int i = 0; i < n; ++i) {
      double v = 0.0;
      for (int q = 0; q < n; ++q) v += G.S[a * TDFE_MAXN + q] * R.B[q * TDFE_MAXN + i];
      G.SB[a * TDFE_MAXN + i] = v;
    }
  return G;
}

// FP32 entries of the box kernels' tables.  Rounded as they are they err by
// some 2e-8 of the table's norm, the same on every cell, and that is a quarter
// of an FP32 operator's whole error on rough vectors; on smooth ones, where S
// multiplies little more than 1 and x, it adds up over the terms of an
// exponential.  So each table is stored times a factor in [1, 2), and the
// factor is divided out of the scales that a cell's values and stiffness terms
// are multiplied by anyway.  The factors are the best of 8 million tried for
// n: least error of the rounded entries in the Frobenius norm, with that of the
// images of 1 and x (for S and S B of the columns' sums and of x, four times
// weighted).  They leave 1e-12 to 1e-8 (n = 2 .. 8) of the norm.
// Relative error of one application in the 2-norm, rough vectors, p = 3 to 7:
// 2.1, 1.8, 3.1, 2.1 and 2.6e-7 without them (entries of S and S B rounded so that
// 1 and x keep their images), 1.5, 1.4, 1.6, 1.7 and 1.8e-7 so, and 1.6, 1.7, 3.2,
// 1.8 and 2.0e-7 for a kernel with derivatives on either side of the flux.  (n =
// 4: B itself is kept, eo1 takes half of the middle pair exactly.)
// zB, zS: the lane pairs' tables along z, which are not folded.
struct F32Factors {
  double B = 1.0, Bt = 1.0, S = 1.0, SB = 1.0, zB = 1.0, zS = 1.0;
  double D = 1.0, G = 1.0;  // trilinear cells, four-lane kernel
};
constexpr F32Factors f32_factors(int N) {
  switch (N) {
    case 2: return {1.46140062809200, 1.46140062809200, 1.0, 1.65737457274267, 1.61684665082995, 1.0};
    case 3: return {1.03040337562240, 1.03040337562240, 1.92209072113039, 1.47100592848871};
    case 4: return {1.0, 1.07268476539059, 1.33175274484762, 1.99836685462980, 1.67130209418044, 1.37747953557320};
    case 5: return {1.86699926960131, 1.86699926960131, 1.80610855435722, 1.38926094107585};
    case 6: return {1.55907900878783, 1.55907900878783, 1.79760520503759, 1.89983373788399, 1.71932972875035,
                    1.09584027715945};
    case 7: return {1.59642291522439, 1.59642291522439, 1.23522284087879, 1.48919430297576};
    case 8: return {1.98078020932613, 1.98078020932613, 1.60004636661610, 1.15822634604022, 1.05413327285020,
                    1.87712638329818,
                    1.56014991319470, 1.03100566826716};
  }
  return {};
}

constexpr void fold_c(const double* A, int N, int S, bool transpose, Folded<double>& F) {
  const int H = N / 2;
  for (int a = 0; a < H; ++a)
    for (int i = 0; i < H; ++i) {
      const double ai = transpose ? A[i * TDFE_MAXN + a] : A[a * TDFE_MAXN + i];
      const double aj = transpose ? A[(N - 1 - i) * TDFE_MAXN + a] : A[a * TDFE_MAXN + N - 1 - i];
      F.E[a * EO_MAX_H + i] = 0.5 * (ai + aj);
      F.O[a * EO_MAX_H + i] = 0.5 * (ai - aj);
    }
  if (N & 1) {
    for (int a = 0; a < H; ++a) F.mc[a] = transpose ? A[H * TDFE_MAXN + a] : A[a * TDFE_MAXN + H];
    for (int i = 0; i <= H; ++i) F.mr[i] = transpose ? A[i * TDFE_MAXN + H] : A[H * TDFE_MAXN + i];
    if (S < 0) F.mr[H] = 0.0;
  }
}

constexpr void scale_c(Folded<double>& F, double f) {
  for (double& v : F.E) v *= f;
  for (double& v : F.O) v *= f;
  for (double& v : F.mc) v *= f;
  for (double& v : F.mr) v *= f;
}

// g: factor of Dg and Dg^T
template <int N>
constexpr FoldSet<N> make_foldset(double g = 1.0) {
  const tdfe1d::Rule R = tdfe1d::make_rule(N - 1);
  FoldSet<N> F{};
  fold_c(R.B, N, 1, false, F.B);
  fold_c(R.B, N, 1, true, F.Bt);
  fold_c(R.D, N, -1, false, F.D);
  fold_c(R.D, N, -1, true, F.Dt);
  fold_c(R.Dg, N, -1, false, F.G);
  fold_c(R.Dg, N, -1, true, F.Gt);
  scale_c(F.G, g);
  scale_c(F.Gt, g);
  for (int i = 0; i < TDFE_MAXN; ++i) F.wq[i] = R.wq[i];
  return F;
}

// the folded tables of the box kernels: B, B^T, S and S B, for FP32 times their
// factors (b: B's), and what takes those out again: `in` for a cell's gathered values,
// `out` for its results, gx for the x stiffness term (S B along x, B along y and z),
// gs for the y and z terms
template <int N>
struct BoxFoldSet {
  Folded<double> B, Bt, S, SB;
  double wq[TDFE_MAXN];
  double b = 1.0, in = 1.0, out = 1.0, gx = 1.0, gs = 1.0;
};
template <int N, bool F32>
constexpr BoxFoldSet<N> make_box_foldset() {
  const tdfe1d::Rule R = tdfe1d::make_rule(N - 1);
  const GaussStiff K = make_gauss_stiff(R);
  BoxFoldSet<N> F{};
  fold_c(R.B, N, 1, false, F.B);
  fold_c(R.B, N, 1, true, F.Bt);
  fold_c(K.S, N, 1, false, F.S);
  fold_c(K.SB, N, 1, false, F.SB);
  if (F32) {
    constexpr F32Factors f = f32_factors(N);
    scale_c(F.B, f.B);
    scale_c(F.Bt, f.Bt);
    scale_c(F.S, f.S);
    scale_c(F.SB, f.SB);
    F.b = f.B;
    F.in = 1.0 / (f.B * f.B * f.B);
    F.out = 1.0 / (f.Bt * f.Bt * f.Bt);
    F.gx = f.B / f.SB;
    F.gs = 1.0 / f.S;
  }
  for (int i = 0; i < TDFE_MAXN; ++i) F.wq[i] = R.wq[i];
  return F;
}

// quadratic form: FP32 kernels sum each line in FP32 and promote the line
// sums; FP64 kernels accumulate directly
template <typename T>
__device__ __forceinline__ void acc_energy(double& e, T& line, T v) {
  if constexpr (sizeof(T) == 4)
    line += v;
  else
    e += v;
}
template <typename T>
__device__ __forceinline__ void flush_energy(double& e, T line) {
  if constexpr (sizeof(T) == 4) e += (double)line;
}

// logical block of physical block p in a grid of G: the dispatcher hands
// blocks to the 8 XCDs round robin (block p to XCD p mod 8), and XCD x takes
// the contiguous logical range starting at x q + min(x, r) (q = G / 8,
// r = G mod 8; q + 1 blocks for x < r), so that neighbouring cells, which
// share nodes, run under one L2
__device__ __forceinline__ int remap_block(int p, int G) {
  const int q = G >> 3, r = G & 7, x = p & 7;
  return x * q + min(x, r) + (p >> 3);
}

// position of a cell on the grid of cells
struct CellPos {
  int x, y, z;
  // DoF row of its node (0, 0, 0) (before the first DoF on the domain's faces)
  template <typename Params>
  __device__ __forceinline__ int64_t row(const Params& P) const {
    return (int64_t)(x * P.p - 1) + (int64_t)(P.Nx - 2) * ((int64_t)(y * P.p - 1) + (int64_t)(P.Ny - 2) * (z * P.p - 1));
  }
};
// of the block's first cell (uniform: scalar arithmetic), and of the cell
// `slot` cells further on
template <typename Params>
__device__ __forceinline__ CellPos cell_pos(const Params& P, int c0) {
  const int yz = c0 / P.ncx;
  return {c0 % P.ncx, yz % P.ncy, yz / P.ncy};
}
template <typename Params>
__device__ __forceinline__ CellPos cell_next(const Params& P, CellPos c, int slot) {
  c.x += slot;
  while (c.x >= P.ncx) {
    c.x -= P.ncx;
    if (++c.y == P.ncy) {
      c.y = 0;
      ++c.z;
    }
  }
  return c;
}

// Where a cell's results go.  CELLS: to the cell's own n^3 rows of y, every node
// (plain stores; the consumer sums the cells, tdfe_cells.h).  Otherwise added
// to the DoF vector y by hardware atomics, DoF nodes only.  Atomics on this
// chip are performed beyond the per-XCD L2s at about 1.3 TB/s of values, plain
// stores run at 5.5; see sum_pays and tdfe_cells_ok for when the cell rows pay.
//
// Addresses are a block-uniform 64-bit base per node row (scalar arithmetic)
// plus a byte offset per lane, of 32 bits where that reaches every node of the
// block's cells (tdfe_span::near) and of 64 (FAR) where rows are so long, or
// layers of nodes so large, that it does not.
template <typename T, int N, bool CELLS, bool FAR = false>
struct CellOut {
  typedef std::conditional_t<FAR, int64_t, uint32_t> Off;
  char* base;        // the block's first cell, node (0, 0, 0)
  Off off;           // this lane's cell, node (0, j, 0) and column from there
  int64_t sx, sz;    // bytes
  bool lox, hix, loz, hiz, jok;
  template <typename Params>
  __device__ __forceinline__ CellOut(T* Y, const Params& P, const CellPos& B, const CellPos& c, int64_t c0, int slot,
                                     int j, int colg, bool act) {
    lox = CELLS || c.x > 0;
    hix = CELLS || c.x < P.ncx - 1;
    loz = CELLS || c.z > 0;
    hiz = CELLS || c.z < P.ncz - 1;
    jok = act && (CELLS || ((j > 0 || c.y > 0) && (j < N - 1 || c.y < P.ncy - 1)));
    if constexpr (CELLS) {
      sx = (int64_t)P.cols * (int)sizeof(T);
      sz = N * N * sx;
      base = (char*)Y + c0 * N * sz;
      off = (Off)((slot * (N * N * N) + N * j) * P.cols + colg) * (Off)sizeof(T);
    } else {
      const int64_t NxI = P.Nx - 2, NyI = P.Ny - 2;
      sx = (int64_t)P.ld * (int)sizeof(T);
      sz = NxI * NyI * sx;
      base = (char*)Y + B.row(P) * sx;
      off = (Off)(c.row(P) - B.row(P) + NxI * j) * (Off)sx + (Off)colg * (Off)sizeof(T);
    }
  }
  // x node i, z node k are written (i, k compile-time constants after unrolling)
  __device__ __forceinline__ bool xok(int i) const { return (i > 0 || lox) && (i < N - 1 || hix); }
  __device__ __forceinline__ bool zok(int k) const { return (k > 0 || loz) && (k < N - 1 || hiz); }
  // node (i, j, k) with k uniform, or i uniform and the z offset part of o
  __device__ __forceinline__ void put(int i, int k, Off o, T v) const {
    T* const d = (T*)(base + (i * sx + k * sz) + o);
    if constexpr (CELLS)
      *d = v;
    else
      unsafeAtomicAdd(d, v);
  }
};

// The gather of a box cell's plane, by byte offsets per lane from the block's
// first row (FAR: from the vector's).  Entries that are not read (the Dirichlet
// planes, columns past the last) carry NONE, to which the offsets of a cell's
// nodes may be added, and give 0.
template <typename T, bool FAR>
struct CellIn {
  typedef uint32_t Off;
  static constexpr Off NONE = tdfe_span::NO_READ;
  __amdgpu_buffer_rsrc_t r;  // from the block's first row to the vector's end
  int64_t first;
  template <typename Params>
  __device__ __forceinline__ CellIn(const Params& P, const CellPos& B) : first(B.row(P)) {
    const int64_t rows = (int64_t)(P.Nx - 2) * (P.Ny - 2) * (P.Nz - 2);
    const int64_t bytes = (rows - first) * P.ld * (int)sizeof(T);
    const uint64_t ad = (uint64_t)(uintptr_t)P.x + (uint64_t)(first * P.ld * (int)sizeof(T));
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)ad);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(ad >> 32));
    const int nrec = __builtin_amdgcn_readfirstlane((int)(bytes < 0x7fffffff ? bytes : 0x7fffffff));
    r = __builtin_amdgcn_make_buffer_rsrc((void*)(uintptr_t)(((uint64_t)hi << 32) | lo), 0, nrec, 0x00020000);
  }
  __device__ __forceinline__ T load(Off o) const {
    if constexpr (sizeof(T) == 8)
      return __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, (int)o, 0, 0));
    else
      return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, (int)o, 0, 0));
  }
};
template <typename T>
struct CellIn<T, true> {
  typedef int64_t Off;
  static constexpr Off NONE = INT64_MIN;
  const char* x;
  static constexpr int64_t first = 0;
  template <typename Params>
  __device__ __forceinline__ CellIn(const Params& P, const CellPos&) : x((const char*)P.x) {}
  // one load from a selected (always valid) address: no branches
  __device__ __forceinline__ T load(Off o) const {
    const T v = *(const T*)(x + (o < 0 ? 0 : o));
    return o < 0 ? (T)0 : v;
  }
};

// out[a] = sum_i A[a][i] in[i] by even/odd folding; A given folded (in any
// precision, converted to T), symmetry S
template <typename T, int N, int S, typename FT>
__device__ __forceinline__ void eo(const Folded<FT>& F, const T* in, T* out) {
  constexpr int H = N / 2;
  T e[H > 0 ? H : 1], o[H > 0 ? H : 1];
#pragma unroll
  for (int i = 0; i < H; ++i) {
    e[i] = in[i] + in[N - 1 - i];
    o[i] = in[i] - in[N - 1 - i];
  }
  // coefficients that are exactly zero (for odd N the middle row of B, whose
  // middle Gauss point is a GLL node, and the middle column of B^T) are
  // skipped: the tables are compile-time constants, so the tests fold away
#pragma unroll
  for (int a = 0; a < H; ++a) {
    T Pv = 0, Qv = 0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      if (F.E[a * EO_MAX_H + i] != 0) Pv += (T)F.E[a * EO_MAX_H + i] * e[i];
      if (F.O[a * EO_MAX_H + i] != 0) Qv += (T)F.O[a * EO_MAX_H + i] * o[i];
    }
    if constexpr (N & 1)
      if (F.mc[a] != 0) Pv += (T)F.mc[a] * in[H];
    out[a] = Pv + Qv;
    out[N - 1 - a] = S > 0 ? Pv - Qv : Qv - Pv;
  }
  if constexpr (N & 1) {
    T m = 0;
    if constexpr (S > 0) {
#pragma unroll
      for (int i = 0; i < H; ++i)
        if (F.mr[i] != 0) m += (T)F.mr[i] * e[i];
      if (F.mr[H] != 0) m += (T)F.mr[H] * in[H];
    } else {
#pragma unroll
      for (int i = 0; i < H; ++i)
        if (F.mr[i] != 0) m += (T)F.mr[i] * o[i];
    }
    out[H] = m;
  }
}

// two matrices on the same input line share the fold
template <typename T, int N, int S1, int S2, typename FT>
__device__ __forceinline__ void eo2(const Folded<FT>& F1, const Folded<FT>& F2, const T* in, T* out1, T* out2) {
  eo<T, N, S1>(F1, in, out1);
  eo<T, N, S2>(F2, in, out2);
}

// eo for a matrix that sends a constant to zero (S, S B): the middle value, or
// the middle pair's sum, is taken off the folded sums first, and its column is
// left out.  As many operations, and the rounding of the entries acts on the
// differences along the line, not on the values: with eo and entries rounded
// as they are an FP32 exponential of smooth orbitals on box cells was off by
// 4.5e-7 at p = 6, with eo0 and the tables' factors by 1.5e-7.
template <typename T, int N, typename FT>
__device__ __forceinline__ void eo0(const Folded<FT>& F, const T* in, T* out) {
  constexpr int H = N / 2, HE = (N & 1) ? H : H - 1;
  const T mid = (N & 1) ? 2 * in[H] : in[H - 1] + in[H];
  T e[HE > 0 ? HE : 1], o[H];
#pragma unroll
  for (int i = 0; i < H; ++i) {
    if (i < HE) e[i] = in[i] + in[N - 1 - i] - mid;
    o[i] = in[i] - in[N - 1 - i];
  }
#pragma unroll
  for (int a = 0; a < H; ++a) {
    T Pv = 0, Qv = 0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      if (i < HE) Pv += (T)F.E[a * EO_MAX_H + i] * e[i];
      Qv += (T)F.O[a * EO_MAX_H + i] * o[i];
    }
    out[a] = Pv + Qv;
    out[N - 1 - a] = Pv - Qv;
  }
  if constexpr (N & 1) {
    T m = 0;
#pragma unroll
    for (int i = 0; i < H; ++i) m += (T)F.mr[i] * e[i];
    out[H] = m;
  }
}

// eo for B (b times B), whose rows sum to one, in the same way: the middle
// value, or the middle pair's, is put back with the last multiply-add, so that
// what is rounded before it are differences along the line
template <typename T, int N, typename FT>
__device__ __forceinline__ void eo1(const Folded<FT>& F, double b, const T* in, T* out) {
  constexpr int H = N / 2, HE = (N & 1) ? H : H - 1;
  const T mid = (N & 1) ? in[H] : in[H - 1] + in[H];
  const T mf = (N & 1) ? (T)b : (T)(0.5 * b);
  T e[HE > 0 ? HE : 1], o[H];
#pragma unroll
  for (int i = 0; i < H; ++i) {
    if (i < HE) e[i] = in[i] + in[N - 1 - i] - ((N & 1) ? 2 * mid : mid);
    o[i] = in[i] - in[N - 1 - i];
  }
#pragma unroll
  for (int a = 0; a < H; ++a) {
    T Pv = 0, Qv = 0;
#pragma unroll
    for (int i = 0; i < H; ++i) {
      if (i < HE) Pv += (T)F.E[a * EO_MAX_H + i] * e[i];
      Qv += (T)F.O[a * EO_MAX_H + i] * o[i];
    }
    Pv += mf * mid;
    out[a] = Pv + Qv;
    out[N - 1 - a] = Pv - Qv;
  }
  if constexpr (N & 1) out[H] = mf * mid;  // the middle Gauss point is a node
}

// host: fold an N x N table (row-major, stride TDFE_MAXN) with symmetry S
template <typename T>
void fold(const double* A, int N, int S, bool transpose, Folded<T>& F) {
  auto at = [&](int a, int i) { return transpose ? A[i * TDFE_MAXN + a] : A[a * TDFE_MAXN + i]; };
  const int H = N / 2;
  for (int a = 0; a < H; ++a)
    for (int i = 0; i < H; ++i) {
      F.E[a * EO_MAX_H + i] = (T)(0.5 * (at(a, i) + at(a, N - 1 - i)));
      F.O[a * EO_MAX_H + i] = (T)(0.5 * (at(a, i) - at(a, N - 1 - i)));
    }
  if (N & 1) {
    for (int a = 0; a < H; ++a) F.mc[a] = (T)at(a, H);
    for (int i = 0; i <= H; ++i) F.mr[i] = (T)at(H, i);
    if (S < 0) F.mr[H] = (T)0;
  }
}

}  // namespace
