// Operator kernel for blocks of more than 8 real columns, n = 8 and FP64 n = 7: four lanes
// per plane line, one wavefront per plane (Eq. DiscreteHamiltonian in the
// Loewdin form, Eq. TDKSMatVecStandard), for box and trilinear cells.
//
// A cell of 16 columns is n wavefronts.  In phases A and C wavefront w holds
// node plane y = w, in phase B point plane x = w; its 64 lanes are 16 columns x
// 4 positions q of the axis the phase contracts most (x in A and C, y in B), a
// lane holding that axis's entries q and n-1-q, and the n z entries in its
// registers:
//   A  gather; x: B, z: B, x: Dg (FP32: x: B and D, z: B on both; box: z: B, x: B
//      and S B)
//   -- LDS transpose of the two arrays -->
//   B  y: B on both; y and z derivatives, the six-entry metric, the potential,
//      transposed derivatives (box: the stiffness S along y and z, weights,
//      potential); y: B^T
//   -- LDS transpose (box: of the one array) -->
//   C  x: Dg^T and B^T (FP32: B^T and D^T; box: B^T), z: B^T; results x M^-1/2 (as
//      CellOut).
// A lane's two entries are folded into their even and odd parts, and every 1D
// table into a 4 x 4 even and a 4 x 4 odd half, so a contraction across the
// four lanes is two 4 x 4 products: FP64 by v_mfma_f64_4x4x4 (lane = 16 q +
// column, the instruction's own layout for input and output, so contractions
// along one axis chain without unfolding), FP32 by eight DPP quad broadcasts
// (lane = 4 column + q).  Contractions along z are folded constants within
// the lane, on the parts directly.
//
// Why: the FP64 rate of the matrix and vector units is the same on this chip
// and they share it (8 MFMA and 16 FMA take the sum of their times), so what
// this layout buys is not rate but registers and addresses: 2 n values per
// array and lane instead of 4 n (lane pairs) or n^2 (planes), so four waves
// per SIMD (FP64 at n = 8 two: its cell takes 117 KB of LDS) hide each other's
// gathers, transposes and barriers, and cell, plane and z row are uniform per
// wave, so masks and 64-bit addresses are scalar.
// What bounds it: FP64 at n = 7, 31^3 trilinear cells of 16 columns: vector and
// matrix units are busy half of the 1.20 ms (45k cycles of them per cell, 0.63
// ms at full use); waits at the ten barriers and the transposes' latency take
// the rest.  1.39 -> 1.20 ms against the lane pairs there; 20^3 cells at n = 8:
// FP64 815 -> 588 us, FP32 406 -> 389 us (FP32's DPP steps issue at half the
// rate of plain FP32, so at n = 7 the plane kernel stays ahead: 370 against
// 430 us).
// FP32 takes the x derivative from the nodes and every table with a factor
// (F32Factors): one application on rough vectors is off by 1.55e-7 (lane pairs
// 1.67e-7; with Dg on the interpolated values and plain tables 2.02e-7), an
// exponential of 40 iterations by 1.05e-7 (1.15e-7; 1.40e-7), for 3% of the
// launch (13 x 14 x 15 cells, 32 columns 220 -> 227 us).
#include "tdfe_fold.h"

namespace {

constexpr int QC = 16;  // columns per pass

// one 4 x 4 even and odd half, [out][in], zero padded; from folded inputs
// (u_i + u_{n-1-i}, u_i - u_{n-1-i}: twice the even and odd parts) to f times
// the parts of the result
struct QHalf {
  double E[16];
  double O[16];
};
// tables in the order a kernel stages them
struct QuadTables {
  QHalf t[6];
};

constexpr QHalf quad_half(const double* A, int N, int S, bool transpose, double f) {
  QHalf Q{};
  const int H = N / 2, HZ = (N + 1) / 2;
  for (int a = 0; a < HZ; ++a)
    for (int i = 0; i < HZ; ++i) {
      const double ai = transpose ? A[i * TDFE_MAXN + a] : A[a * TDFE_MAXN + i];
      const double aj = transpose ? A[(N - 1 - i) * TDFE_MAXN + a] : A[a * TDFE_MAXN + N - 1 - i];
      const bool midrow = (N & 1) && a == H, midcol = (N & 1) && i == H;
      // the middle entry is its own mirror: folded it is counted twice, and
      // its odd part is 0; the middle result is all even (S > 0) or comes
      // from the odd half alone (S < 0)
      Q.E[a * 4 + i] = (midrow && S < 0) ? 0.0 : (midcol ? 0.5 : 1.0) * 0.5 * f * (ai + aj);
      Q.O[a * 4 + i] = ((midrow && S > 0) || midcol) ? 0.0 : 0.5 * f * (ai - aj);
    }
  return Q;
}

// trilinear cells: B (folded -> parts), Dg (parts -> parts), Dg^T (folded ->
// folded), B^T (folded -> parts), FP32 also D, D^T (folded -> parts); box
// cells: B, S B (folded -> parts), S (parts -> folded), B^T
template <int N, bool BOX, bool F32>
constexpr QuadTables make_quad_tables() {
  const tdfe1d::Rule R = tdfe1d::make_rule(N - 1);
  const F32Factors f = F32 ? f32_factors(N) : F32Factors{};
  QuadTables Q{};
  Q.t[0] = quad_half(R.B, N, 1, false, f.B);
  if (BOX) {
    const GaussStiff K = make_gauss_stiff(R);
    Q.t[1] = quad_half(K.SB, N, 1, false, f.SB);
    Q.t[2] = quad_half(K.S, N, 1, false, 4.0 * f.S);
  } else {
    Q.t[1] = quad_half(R.Dg, N, -1, false, 2.0 * f.G);
    Q.t[2] = quad_half(R.Dg, N, -1, true, 2.0 * f.G);
    Q.t[4] = quad_half(R.D, N, -1, false, f.D);
    Q.t[5] = quad_half(R.D, N, -1, true, f.D);
  }
  Q.t[3] = quad_half(R.B, N, 1, true, f.Bt);  // (Bt = B at n = 8: one scale for gather and results)
  return Q;
}

template <int N, bool BOX, bool F32>
__device__ const QuadTables quad_tables = make_quad_tables<N, BOX, F32>();

template <typename T>
struct QuadParams {
  const void* x;
  T* y;  // as in CellOut
  int ld, cols, nchunks;
  int eld;  // columns of the quadratic-form rows
  const double* colscale;
  double kin;
  const void* vw;
  const double* minv;     // trilinear cells: M^-1/2 per DoF
  const double* corners;  // trilinear cells: [n_cell][2][2][2][3]
  const double* m1x;      // box cells: separable M^-1/2 factors
  const double* m1y;
  const double* m1z;
  const double* cellgeo;
  double* energy;
  const int* done;
  int ncx, ncy, ncz, p, Nx, Ny, Nz;
};

// a lane's share of one table: the A operand of the matrix instruction, or
// its row of coefficients
template <typename T>
struct QTab;
template <>
struct QTab<double> {
  double e, o;
};
template <>
struct QTab<float> {
  float e[4], o[4];
};

__device__ __forceinline__ QTab<double> qtab(const double* sT, int k, int lane) {
  const int i = (lane & 3) * 4 + (lane >> 4);
  return {sT[k * 32 + i], sT[k * 32 + 16 + i]};
}
__device__ __forceinline__ QTab<float> qtab(const float* sT, int k, int lane) {
  QTab<float> t;
  const int i = (lane & 3) * 4;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    t.e[j] = sT[k * 32 + i + j];
    t.o[j] = sT[k * 32 + 16 + i + j];
  }
  return t;
}

// (p, q) = (ce, co) + (E e, O o) across the four lanes of each column
__device__ __forceinline__ void qmul(const QTab<double>& t, double e, double o, double ce, double co, double& p,
                                     double& q) {
  p = __builtin_amdgcn_mfma_f64_4x4x4f64(t.e, e, ce, 0, 0, 0);
  q = __builtin_amdgcn_mfma_f64_4x4x4f64(t.o, o, co, 0, 0, 0);
}
// FP32: each step broadcasts one lane of the quad into a multiply-add.  The
// compiler does not fold DPP moves into multiply-adds, so the steps are written
// out; the leading s_nop covers the two wait states between a vector write of
// e or o and its first DPP read
#define TDFE_QSTEP(OP, K, ACC, V, C) \
  #OP "_dpp " ACC ", " V ", " C " quad_perm:[" #K "," #K "," #K "," #K "] row_mask:0xf bank_mask:0xf\n"
__device__ __forceinline__ void qmul(const QTab<float>& t, float e, float o, float ce, float co, float& p, float& q) {
  float a = ce, b = co;
  asm("s_nop 1\n"
      TDFE_QSTEP(v_fmac_f32, 0, "%0", "%2", "%4") TDFE_QSTEP(v_fmac_f32, 0, "%1", "%3", "%8")
      TDFE_QSTEP(v_fmac_f32, 1, "%0", "%2", "%5") TDFE_QSTEP(v_fmac_f32, 1, "%1", "%3", "%9")
      TDFE_QSTEP(v_fmac_f32, 2, "%0", "%2", "%6") TDFE_QSTEP(v_fmac_f32, 2, "%1", "%3", "%10")
      TDFE_QSTEP(v_fmac_f32, 3, "%0", "%2", "%7") TDFE_QSTEP(v_fmac_f32, 3, "%1", "%3", "%11")
      : "+&v"(a), "+&v"(b)
      : "v"(e), "v"(o), "v"(t.e[0]), "v"(t.e[1]), "v"(t.e[2]), "v"(t.e[3]), "v"(t.o[0]), "v"(t.o[1]), "v"(t.o[2]),
        "v"(t.o[3]));
  p = a;
  q = b;
}
// the same from zero
__device__ __forceinline__ void qmul0(const QTab<float>& t, float e, float o, float& p, float& q) {
  float a, b;
  asm("s_nop 1\n"
      TDFE_QSTEP(v_mul_f32, 0, "%0", "%2", "%4") TDFE_QSTEP(v_mul_f32, 0, "%1", "%3", "%8")
      TDFE_QSTEP(v_fmac_f32, 1, "%0", "%2", "%5") TDFE_QSTEP(v_fmac_f32, 1, "%1", "%3", "%9")
      TDFE_QSTEP(v_fmac_f32, 2, "%0", "%2", "%6") TDFE_QSTEP(v_fmac_f32, 2, "%1", "%3", "%10")
      TDFE_QSTEP(v_fmac_f32, 3, "%0", "%2", "%7") TDFE_QSTEP(v_fmac_f32, 3, "%1", "%3", "%11")
      : "=&v"(a), "=&v"(b)
      : "v"(e), "v"(o), "v"(t.e[0]), "v"(t.e[1]), "v"(t.e[2]), "v"(t.e[3]), "v"(t.o[0]), "v"(t.o[1]), "v"(t.o[2]),
        "v"(t.o[3]));
  p = a;
  q = b;
}
__device__ __forceinline__ void qmul0(const QTab<double>& t, double e, double o, double& p, double& q) {
  qmul(t, e, o, 0.0, 0.0, p, q);
}

// what a table whose rows sum to zero (S, S B) is applied to: FP32 less the
// value of the quad's last lane (see eo0), FP64 as it is
__device__ __forceinline__ double off_quad(double v) { return v; }
__device__ __forceinline__ float off_quad(float v) {
  return v - __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xFF, 0xf, 0xf, false));
}

// The Jacobian of a trilinear cell: its column along one reference axis is
// bilinear in the other two coordinates, so the 3 n^2 columns of a cell are
// formed once (entry [axis][u + n v], u and v the Gauss points of the other
// two axes in x, y, z order) and shared by its n^3 points.
template <int N>
__device__ __forceinline__ void quad_jacobian_column(double* sJ, const double* C, const double* sEW, int e) {
  const int d = e / (N * N), u = e % N, v = (e / N) % N;
  const int sd = 1 << d, s1 = d == 0 ? 2 : 1, s2 = d == 2 ? 2 : 4;
  const double wu = 0.5 * (1 + sEW[u]), wv = 0.5 * (1 + sEW[v]);
  const double w[4] = {0.5 * (1 - wu) * (1 - wv), 0.5 * wu * (1 - wv), 0.5 * (1 - wu) * wv, 0.5 * wu * wv};
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    double s = 0.0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int v0 = (q & 1) * s1 + (q >> 1) * s2;
      s += w[q] * (C[3 * (v0 + sd) + k] - C[3 * v0 + k]);
    }
    sJ[3 * e + k] = s;
  }
}

// kin w detJ J^-1 J^-T at Gauss point (a, b, c), for derivatives that carry the
// factors 1 / fx along x and 1 / fy along y and z
template <typename T, int N>
__device__ __forceinline__ void quad_metric(T* g, const double* sJ, const double* sEW, int a, int b, int c,
                                            double kin, double fx, double fy) {
  double Jm[3][3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    Jm[k][0] = sJ[3 * (b + N * c) + k];
    Jm[k][1] = sJ[3 * (N * N + a + N * c) + k];
    Jm[k][2] = sJ[3 * (2 * N * N + a + N * b) + k];
  }
  double A[3][3];  // adjugate: J^-1 = A / det
  A[0][0] = Jm[1][1] * Jm[2][2] - Jm[1][2] * Jm[2][1];
  A[0][1] = Jm[0][2] * Jm[2][1] - Jm[0][1] * Jm[2][2];
  A[0][2] = Jm[0][1] * Jm[1][2] - Jm[0][2] * Jm[1][1];
  A[1][0] = Jm[1][2] * Jm[2][0] - Jm[1][0] * Jm[2][2];
  A[1][1] = Jm[0][0] * Jm[2][2] - Jm[0][2] * Jm[2][0];
  A[1][2] = Jm[0][2] * Jm[1][0] - Jm[0][0] * Jm[1][2];
  A[2][0] = Jm[1][0] * Jm[2][1] - Jm[1][1] * Jm[2][0];
  A[2][1] = Jm[0][1] * Jm[2][0] - Jm[0][0] * Jm[2][1];
  A[2][2] = Jm[0][0] * Jm[1][1] - Jm[0][1] * Jm[1][0];
  const double det = Jm[0][0] * A[0][0] + Jm[0][1] * A[1][0] + Jm[0][2] * A[2][0];
  const double s = kin * sEW[N + a] * sEW[N + b] * sEW[N + c] / det;
  const double xx = s * (fx * fx), xy = s * (fx * fy), yy = s * (fy * fy);
  g[0] = (T)(xx * (A[0][0] * A[0][0] + A[0][1] * A[0][1] + A[0][2] * A[0][2]));
  g[1] = (T)(xy * (A[0][0] * A[1][0] + A[0][1] * A[1][1] + A[0][2] * A[1][2]));
  g[2] = (T)(xy * (A[0][0] * A[2][0] + A[0][1] * A[2][1] + A[0][2] * A[2][2]));
  g[3] = (T)(yy * (A[1][0] * A[1][0] + A[1][1] * A[1][1] + A[1][2] * A[1][2]));
  g[4] = (T)(yy * (A[1][0] * A[2][0] + A[1][1] * A[2][1] + A[1][2] * A[2][2]));
  g[5] = (T)(yy * (A[2][0] * A[2][0] + A[2][1] * A[2][1] + A[2][2] * A[2][2]));
}

template <typename T, int N, bool BOX, bool CELLS>
__global__ void __launch_bounds__(64 * N) __attribute__((amdgpu_waves_per_eu(4)))
    quad_kernel(QuadParams<T> P) {
  constexpr int H = N / 2;
  static_assert(N == 7 || N == 8);  // every lane of a quad holds entries
  constexpr bool ODD = (N & 1) != 0;
  constexpr int VOL = N * N * N;
  constexpr int THREADS = 64 * N;
  constexpr bool F32 = sizeof(T) == 4;
  // LDS strides of the transpose buffer [y][x][z][column]: for even n padded so
  // that the four positions q fall into different bank groups
  constexpr int PAD = ODD ? 0 : QC;
  constexpr int LX = N * QC + PAD, LY = N * LX + PAD;
  constexpr FoldSet<N> FS = make_foldset<N>(F32 ? f32_factors(N).G : 1.0);
  constexpr BoxFoldSet<N> FB = make_box_foldset<N, sizeof(T) == 4>();
  // FP64 on trilinear cells at n = 7: two blocks per CU (14 waves) need 128
  // registers per lane, and the flux phase holds 158 (26 spilled values of it
  // made scratch traffic of 2.8 GB per launch): half of its arrays wait in LDS
  constexpr bool PARK = !F32 && !BOX && N == 7;
  // what takes the tables' factors out of the x and of the y and z derivatives
  constexpr double GX = F32 ? f32_factors(N).B / f32_factors(N).D : 1.0, GY = F32 ? 1.0 / f32_factors(N).G : 1.0;
  constexpr int NX = PARK && 2 * N * THREADS > N * LY ? 2 * N * THREADS : N * LY;
  __shared__ T sX[NX];
  __shared__ T sV[VOL];
  __shared__ T sG[BOX ? 1 : VOL * 6];
  __shared__ T sM[BOX ? 1 : VOL];
  __shared__ double sRed[THREADS];
  constexpr int NTAB = F32 && !BOX ? 192 : 128;
  __shared__ T sT[NTAB];
  __shared__ double sC[BOX ? 1 : 24];
  __shared__ double sJ[BOX ? 1 : 9 * N * N];
  __shared__ double sEW[2 * N];
  if (P.done && *P.done) return;

  const int t = threadIdx.x;
  const int lane = t & 63;
  const int w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int q = F32 ? lane & 3 : lane >> 4;
  const int col = F32 ? lane >> 2 : lane & 15;
  const int L = remap_block(blockIdx.x, gridDim.x);
  const int ch = L % P.nchunks;
  const int cell = L / P.nchunks;
  const int cx = cell % P.ncx, cyz = cell / P.ncx;
  const int cy = cyz % P.ncy, cz = cyz / P.ncy;

  // ---- block staging: loads here, LDS stores after the first gather is issued ----
  constexpr int NV = (VOL + THREADS - 1) / THREADS;
  const int NxI = P.Nx - 2, NyI = P.Ny - 2;
  T vr[NV], mr[NV];
#pragma unroll
  for (int k = 0; k < NV; ++k) {
    const int r = t + k * THREADS;
    vr[k] = (P.vw && r < VOL) ? ((const T*)P.vw)[(int64_t)cell * VOL + r] : (T)0;
    if constexpr (!BOX) {
      // Dirichlet nodes: any value (their gathered values are 0 and their
      // results are not scattered)
      const int I = cx * P.p + r % N, J = cy * P.p + (r / N) % N, K = cz * P.p + r / (N * N);
      const bool in = r < VOL && I > 0 && I < P.Nx - 1 && J > 0 && J < P.Ny - 1 && K > 0 && K < P.Nz - 1;
      mr[k] = (T)(FB.in * P.minv[in ? (int64_t)(I - 1) + (int64_t)NxI * ((int64_t)(J - 1) + (int64_t)NyI * (K - 1)) : 0]);
    }
  }
  T tr = 0;
  if (t < NTAB) tr = (T)((const double*)&quad_tables<N, BOX, sizeof(T) == 4>)[t];
  double cr = 0.0;
  if constexpr (!BOX)
    if (t < 24) cr = P.corners[(int64_t)cell * 24 + t];
  if (t < 2 * N) {
    constexpr tdfe1d::Rule R = tdfe1d::make_rule(N - 1);
    double v = R.eta[0];
#pragma unroll
    for (int i = 0; i < N; ++i) {
      v = t == i ? R.eta[i] : v;
      v = t == N + i ? R.wq[i] : v;
    }
    sEW[t] = v;
  }

  // lane masks along x: node q and node n-1-q are DoFs (cell faces on the
  // domain boundary hold Dirichlet nodes)
  const bool x1ok = !(q == 0 && cx == 0);
  const bool x2ok = !(q == 0 && cx == P.ncx - 1);
  const bool jok = !(w == 0 && cy == 0) && !(w == N - 1 && cy == P.ncy - 1);
  auto kok = [&](int k) { return !(k == 0 && cz == 0) && !(k == N - 1 && cz == P.ncz - 1); };
  // row of node (0, w, k) among the DoFs (-1 relative to the first DoF of the
  // row on the domain's x face)
  auto row0 = [&](int k) {
    return (int64_t)(cx * P.p - 1) + (int64_t)NxI * ((int64_t)(cy * P.p + w - 1) + (int64_t)NyI * (cz * P.p + k - 1));
  };
  const int ldb = P.ld * (int)sizeof(T);

  // positions of a lane's two entries, recomputed by each phase from the lane
  // number (held through the kernel they would cost a dozen registers):
  // a1, a2 in the transpose buffer in node plane y = w (x entries q, n-1-q),
  // b1, b2 in point plane x = w (y entries), g1, g2 + N^2 c its Gauss points,
  // n1, n2 + N^2 k its nodes
  struct Pos {
    int a1, a2, b1, b2, g1, g2, n1, n2;
  };
  auto pos = [&]() {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int qq = F32 ? ln & 3 : ln >> 4, cc = F32 ? ln >> 2 : ln & 15;
    const int qm = N - 1 - qq;
    return Pos{w * LY + qq * LX + cc, w * LY + qm * LX + cc, qq * LY + w * LX + cc, qm * LY + w * LX + cc,
               w + N * qq,            w + N * qm,            qq + N * w,            qm + N * w};
  };

  // the quadratic form of a lane's points; the middle entry is held twice
  auto park_energy = [&](double e) {
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int qq = F32 ? ln & 3 : ln >> 4, cc = F32 ? ln >> 2 : ln & 15;
    const double ew = ODD && qq == H ? 0.5 : 1.0;
    sRed[w * 64 + ln] = ch * QC + cc < P.cols ? e * ew : 0.0;
  };
  {
    const int colg = ch * QC + col;
    const bool cok = colg < P.cols;
    double cs = cok ? 1.0 : 0.0;
    if (P.colscale && cok) cs = P.colscale[colg >> 1];

    // ---------------- A: node plane y = w ----------------------------------------------
    T r1[N], r2[N];
    {
      // one buffer resource per z row, exactly the cell's n nodes: masked lanes
      // carry an offset past its end and read 0, masked rows have no records
      const uint32_t o1 = x1ok && cok ? (uint32_t)(q * ldb + colg * (int)sizeof(T)) : 0x80000000u;
      const uint32_t o2 = x2ok && cok ? (uint32_t)((N - 1 - q) * ldb + colg * (int)sizeof(T)) : 0x80000000u;
#pragma unroll
      for (int k = 0; k < N; ++k) {
        const uint64_t ad = (uint64_t)(uintptr_t)P.x + (uint64_t)(row0(k) * ldb);
        const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)ad);
        const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(ad >> 32));
        const int nrec = __builtin_amdgcn_readfirstlane(jok && kok(k) ? N * ldb : 0);
        const __amdgpu_buffer_rsrc_t rx =
            __builtin_amdgcn_make_buffer_rsrc((void*)(uintptr_t)(((uint64_t)hi << 32) | lo), 0, nrec, 0x00020000);
        if constexpr (F32) {
          r1[k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rx, (int)o1, 0, 0));
          r2[k] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(rx, (int)o2, 0, 0));
        } else {
          r1[k] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rx, (int)o1, 0, 0));
          r2[k] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(rx, (int)o2, 0, 0));
        }
      }
    }
    // box cells: M^-1/2 factors of the lane's two x entries and of the z rows,
    // the y factor in the latter
    T mx1 = 0, mx2 = 0, mi1 = 0, mi2 = 0, mz[N];
    if constexpr (BOX) {
      const double x1 = P.m1x[cx * P.p + q], x2 = P.m1x[cx * P.p + N - 1 - q];
      const double my = P.m1y[cy * P.p + w] * FB.in;
      mx1 = (T)x1;
      mx2 = (T)x2;
      mi1 = (T)(x1 * cs);
      mi2 = (T)(x2 * cs);
#pragma unroll
      for (int k = 0; k < N; ++k) mz[k] = (T)(P.m1z[cz * P.p + k] * my);
    }
    __builtin_amdgcn_sched_barrier(0);
    {
#pragma unroll
      for (int k = 0; k < NV; ++k) {
        const int r = t + k * THREADS;
        if (r < VOL) {
          sV[r] = vr[k];
          if constexpr (!BOX) sM[r] = mr[k];
        }
      }
      if (t < NTAB) sT[t] = tr;
      if constexpr (!BOX)
        if (t < 24) sC[t] = cr;
      __syncthreads();
      if constexpr (!BOX) {
        if (t < 3 * N * N) quad_jacobian_column<N>(sJ, sC, sEW, t);
        __syncthreads();
        for (int r = t; r < VOL; r += THREADS)
          quad_metric<T, N>(sG + r * 6, sJ, sEW, r % N, (r / N) % N, r / (N * N), P.kin, GX, GY);
      }
    }
    const Pos PA = pos();
    T t1[N], t2[N];  // second array: x derivative (box: S B u) at the x points
    {
#pragma unroll
      for (int k = 0; k < N; ++k) {
        T m1, m2;
        if constexpr (BOX) {
          m1 = mi1 * mz[k];
          m2 = mi2 * mz[k];
        } else {
          m1 = sM[PA.n1 + N * N * k] * (T)cs;
          m2 = sM[PA.n2 + N * N * k] * (T)cs;
        }
        const T u1 = r1[k] * m1, u2 = r2[k] * m2;
        r1[k] = u1 + u2;
        r2[k] = u1 - u2;
      }
      const QTab<T> tb = qtab(sT, 0, lane), td = qtab(sT, F32 && !BOX ? 4 : 1, lane);
      T o[N];
      if constexpr (F32 && !BOX) {
        // the x derivative from the nodes (D = Dg B)
#pragma unroll
        for (int k = 0; k < N; ++k) {
          qmul0(td, r1[k], r2[k], t2[k], t1[k]);  // (antisymmetric: the odd part first)
          qmul0(tb, r1[k], r2[k], r1[k], r2[k]);
        }
        auto along_z = [&](T* v) {
          eo<T, N, 1>(FB.B, v, o);
#pragma unroll
          for (int c = 0; c < N; ++c) v[c] = o[c];
        };
        along_z(r1);
        along_z(r2);
        along_z(t1);
        along_z(t2);
#pragma unroll
        for (int c = 0; c < N; ++c) {
          const T u1 = r1[c] + r2[c], u2 = r1[c] - r2[c];
          r1[c] = u1;
          r2[c] = u2;
          const T v1 = t1[c] + t2[c], v2 = t1[c] - t2[c];
          t1[c] = v1;
          t2[c] = v2;
        }
      } else if constexpr (BOX) {
        eo<T, N, 1>(FB.B, r1, o);
#pragma unroll
        for (int c = 0; c < N; ++c) r1[c] = o[c];
        eo<T, N, 1>(FB.B, r2, o);
#pragma unroll
        for (int c = 0; c < N; ++c) r2[c] = o[c];
#pragma unroll
        for (int c = 0; c < N; ++c) {
          T p1, q1;
          qmul0(td, off_quad(r1[c]), r2[c], p1, q1);
          t1[c] = p1 + q1;
          t2[c] = p1 - q1;
          qmul0(tb, r1[c], r2[c], p1, q1);
          r1[c] = p1 + q1;
          r2[c] = p1 - q1;
        }
      } else {
#pragma unroll
        for (int k = 0; k < N; ++k) qmul0(tb, r1[k], r2[k], r1[k], r2[k]);
        eo<T, N, 1>(FB.B, r1, o);
#pragma unroll
        for (int c = 0; c < N; ++c) r1[c] = o[c];
        eo<T, N, 1>(FB.B, r2, o);
#pragma unroll
        for (int c = 0; c < N; ++c) r2[c] = o[c];
#pragma unroll
        for (int c = 0; c < N; ++c) {
          T p1, q1;  // antisymmetric table: p is the odd part of the result, q the even one
          qmul0(td, r1[c], r2[c], p1, q1);
          t1[c] = q1 + p1;
          t2[c] = q1 - p1;
          const T u1 = r1[c] + r2[c], u2 = r1[c] - r2[c];
          r1[c] = u1;
          r2[c] = u2;
        }
      }
    }
    // ---------------- transposes (y = w; x lanes) -> (x = w; y lanes) ----------------------
    auto put = [&](int i1, int i2, const T* v1, const T* v2) {
#pragma unroll
      for (int c = 0; c < N; ++c) {
        sX[i1 + c * QC] = v1[c];
        sX[i2 + c * QC] = v2[c];
      }
    };
    // reads an array folded: sums in v1, differences in v2
    auto get_folded = [&](int i1, int i2, T* v1, T* v2) {
#pragma unroll
      for (int c = 0; c < N; ++c) {
        const T u1 = sX[i1 + c * QC], u2 = sX[i2 + c * QC];
        v1[c] = u1 + u2;
        v2[c] = u1 - u2;
      }
    };
    put(PA.a1, PA.a2, r1, r2);
    __syncthreads();
    const Pos PB = pos();
    T ue[N], uo[N];  // even and odd parts (along y) of u at the Gauss points
    {
      const QTab<T> tb = qtab(sT, 0, lane);
      get_folded(PB.b1, PB.b2, ue, uo);
#pragma unroll
      for (int c = 0; c < N; ++c) qmul0(tb, ue[c], uo[c], ue[c], uo[c]);
    }
    __syncthreads();
    {
      const Pos Q = pos();
      put(Q.a1, Q.a2, t1, t2);
    }
    __syncthreads();
    const Pos PC = pos();

    // ---------------- B: point plane x = w ---------------------------------------------------
    double energy = 0.0;
    if constexpr (BOX) {
      const QTab<T> tb = qtab(sT, 0, lane), ts = qtab(sT, 2, lane);
      double wa = FB.wq[0], wb = FB.wq[0];
#pragma unroll
      for (int i = 1; i < N; ++i) {
        wa = w == i ? FB.wq[i] : wa;
        wb = q == i ? FB.wq[i] : wb;
      }
      // twice: the sums below are folded values
      const T gx = (T)(2.0 * P.kin * FB.gx * P.cellgeo[(int64_t)cell * 4 + 0] * wb);
      const T gy = (T)(P.kin * FB.gs * P.cellgeo[(int64_t)cell * 4 + 1] * wa);
      const T gz = (T)(2.0 * P.kin * FB.gs * P.cellgeo[(int64_t)cell * 4 + 2] * (wa * wb));
      T se[N], so[N];
      get_folded(PC.b1, PC.b2, se, so);
      // x stiffness term and the potential
#pragma unroll
      for (int c = 0; c < N; ++c) {
        const T g = gx * (T)FB.wq[c];
        T p1, q1;
        qmul0(tb, se[c], so[c], p1, q1);
        const T v1 = sV[PC.g1 + N * N * c] * (ue[c] + uo[c]), v2 = sV[PC.g2 + N * N * c] * (ue[c] - uo[c]);
        se[c] = g * p1 + (v1 + v2);
        so[c] = g * q1 + (v1 - v2);
      }
      // z and y stiffness terms, the quadratic form
      T d[N];
      eo0<T, N>(FB.S, ue, d);
#pragma unroll
      for (int c = 0; c < N; ++c) se[c] += gz * d[c];
      eo0<T, N>(FB.S, uo, d);
#pragma unroll
      for (int c = 0; c < N; ++c) so[c] += gz * d[c];
      T le = 0;
#pragma unroll
      for (int c = 0; c < N; ++c) {
        const T g = gy * (T)FB.wq[c];
        T p1, q1;
        qmul0(ts, off_quad(ue[c]), uo[c], p1, q1);
        se[c] += g * p1;
        so[c] += g * q1;
        acc_energy<T>(energy, le, ue[c] * se[c] + uo[c] * so[c]);
      }
      flush_energy<T>(energy, le);
      const QTab<T> tt = qtab(sT, 3, lane);
#pragma unroll
      for (int c = 0; c < N; ++c) {
        T p1, q1;
        qmul0(tt, se[c], so[c], p1, q1);
        se[c] = p1 + q1;
        so[c] = p1 - q1;
      }
      park_energy(energy);
      __syncthreads();
      put(PC.b1, PC.b2, se, so);
      __syncthreads();
      // -------------- C: node plane y = w ----------------------------------------------------
      const Pos PD = pos();
      get_folded(PD.a1, PD.a2, r1, r2);
    } else {
      T d1[N], d2[N], e1[N], e2[N];  // x and y derivatives at the lane's two y points
      {
        const QTab<T> tb = qtab(sT, 0, lane), tg = qtab(sT, 1, lane);
        get_folded(PC.b1, PC.b2, d1, d2);
#pragma unroll
        for (int c = 0; c < N; ++c) {
          T p1, q1;
          qmul0(tb, d1[c], d2[c], p1, q1);
          d1[c] = p1 + q1;
          d2[c] = p1 - q1;
        }
        if constexpr (!F32) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < N; ++c) {
          T p1, q1;
          qmul0(tg, ue[c], uo[c], p1, q1);
          e1[c] = q1 + p1;
          e2[c] = q1 - p1;
          const T u1 = ue[c] + uo[c], u2 = ue[c] - uo[c];
          ue[c] = u1;
          uo[c] = u2;
        }
      }
      // per y point: z derivative, fluxes, potential, transposed z derivative;
      // d <- f_x, e <- f_y, u <- V u + Dg_z^T f_z
      auto fluxes = [&](int gp, T* u, T* dx, T* dy) {
        T dz[N], rz[N];
        eo<T, N, -1>(FS.G, u, dz);
        if constexpr (!F32) __builtin_amdgcn_sched_barrier(0);
        T le = 0;
#pragma unroll
        for (int c = 0; c < N; ++c) {
          const T* g = sG + (gp + N * N * c) * 6;
          const T ux = dx[c], uy = dy[c], uz = dz[c];
          const T fx = g[0] * ux + g[1] * uy + g[2] * uz;
          const T fy = g[1] * ux + g[3] * uy + g[4] * uz;
          const T fz = g[2] * ux + g[4] * uy + g[5] * uz;
          const T pot = sV[gp + N * N * c] * u[c];
          acc_energy<T>(energy, le, fx * ux + fy * uy + fz * uz + pot * u[c]);
          dx[c] = fx;
          dy[c] = fy;
          dz[c] = fz;
          u[c] = pot;
          if constexpr (!F32)
            if (c & 1) __builtin_amdgcn_sched_barrier(0);
        }
        flush_energy<T>(energy, le);
        if constexpr (!F32) __builtin_amdgcn_sched_barrier(0);
        eo<T, N, -1>(FS.Gt, dz, rz);
#pragma unroll
        for (int c = 0; c < N; ++c) u[c] += rz[c];
        __builtin_amdgcn_sched_barrier(0);
      };
      // the derivatives, then fluxes, of the row that is not being worked on
      // wait in slots of the transpose buffer of the lane's own
      auto park = [&](const T* v1, const T* v2) {
        int tt = lane;
        asm volatile("" : "+v"(tt));
        tt += 64 * w;
#pragma unroll
        for (int c = 0; c < N; ++c) {
          sX[c * THREADS + tt] = v1[c];
          sX[(N + c) * THREADS + tt] = v2[c];
        }
      };
      auto unpark = [&](T* v1, T* v2) {
        int tt = lane;
        asm volatile("" : "+v"(tt));
        tt += 64 * w;
#pragma unroll
        for (int c = 0; c < N; ++c) {
          v1[c] = sX[c * THREADS + tt];
          v2[c] = sX[(N + c) * THREADS + tt];
        }
      };
      if constexpr (PARK) {
        __syncthreads();
        park(d2, e2);
        __builtin_amdgcn_sched_barrier(0);
      }
      fluxes(pos().g1, ue, d1, e1);
      if constexpr (PARK) {
        unpark(d2, e2);
        park(d1, e1);
        __builtin_amdgcn_sched_barrier(0);
      }
      fluxes(pos().g2, uo, d2, e2);
      if constexpr (PARK) unpark(d1, e1);
      if constexpr (!F32) __builtin_amdgcn_sched_barrier(0);
      {
        const QTab<T> tg = qtab(sT, 2, lane), tt = qtab(sT, 3, lane);
#pragma unroll
        for (int c = 0; c < N; ++c) {
          T p1, q1;
          qmul0(tt, d1[c] + d2[c], d1[c] - d2[c], p1, q1);
          d1[c] = p1 + q1;
          d2[c] = p1 - q1;
        }
        if constexpr (!F32) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int c = 0; c < N; ++c) {
          T p1, q1;
          // s + Dg_y^T f_y, folded (the antisymmetric table swaps the parts)
          qmul(tg, e1[c] + e2[c], e1[c] - e2[c], ue[c] - uo[c], ue[c] + uo[c], p1, q1);
          qmul0(tt, q1, p1, p1, q1);
          ue[c] = p1 + q1;
          uo[c] = p1 - q1;
        }
      }
      park_energy(energy);
      __syncthreads();
      const Pos PD = pos();
      put(PD.b1, PD.b2, d1, d2);
      __syncthreads();
      // -------------- C: node plane y = w ----------------------------------------------------
      get_folded(PD.a1, PD.a2, d1, d2);
      __syncthreads();
      put(PD.b1, PD.b2, ue, uo);
      __syncthreads();
      get_folded(PD.a1, PD.a2, r1, r2);
      const QTab<T> tg = qtab(sT, F32 ? 5 : 2, lane);
      if constexpr (F32) {
        // B^T s + D^T f_x
        const QTab<T> tt = qtab(sT, 3, lane);
#pragma unroll
        for (int c = 0; c < N; ++c) qmul0(tt, r1[c], r2[c], r1[c], r2[c]);
      }
#pragma unroll
      for (int c = 0; c < N; ++c) {
        T p1, q1;
        qmul(tg, d1[c], d2[c], r2[c], r1[c], p1, q1);
        r1[c] = q1;
        r2[c] = p1;
      }
    }
    const Pos PE = pos();
    {
      if constexpr (!F32 || BOX) {
        const QTab<T> tt = qtab(sT, 3, lane);
#pragma unroll
        for (int c = 0; c < N; ++c) qmul0(tt, r1[c], r2[c], r1[c], r2[c]);
      }
      T o[N];
      eo<T, N, 1>(FB.Bt, r1, o);
#pragma unroll
      for (int k = 0; k < N; ++k) r1[k] = o[k];
      eo<T, N, 1>(FB.Bt, r2, o);
#pragma unroll
      for (int k = 0; k < N; ++k) {
        const T u1 = r1[k] + o[k], u2 = r1[k] - o[k];
        if constexpr (BOX) {
          r1[k] = u1 * (mx1 * mz[k]);
          r2[k] = u2 * (mx2 * mz[k]);
        } else {
          r1[k] = u1 * sM[PE.n1 + N * N * k];
          r2[k] = u2 * sM[PE.n2 + N * N * k];
        }
      }
    }
    {
      int ln = lane;
      asm volatile("" : "+v"(ln));
      const int qq = F32 ? ln & 3 : ln >> 4, cc = ch * QC + (F32 ? ln >> 2 : ln & 15);
      if (cc < P.cols) {
        if constexpr (CELLS) {
          T* const E = P.y + ((int64_t)cell * VOL + N * w) * P.cols;
          const uint32_t o1 = (uint32_t)(qq * P.cols + cc), o2 = (uint32_t)((N - 1 - qq) * P.cols + cc);
#pragma unroll
          for (int k = 0; k < N; ++k) {
            T* const row = E + (int64_t)(N * N * k) * P.cols;
            row[o1] = r1[k];
            if (!ODD || qq != H) row[o2] = r2[k];
          }
        } else if (jok) {
          const uint32_t o1 = (uint32_t)(qq * P.ld + cc), o2 = (uint32_t)((N - 1 - qq) * P.ld + cc);
          if (!(qq == 0 && cx == 0)) {
#pragma unroll
            for (int k = 0; k < N; ++k)
              if (kok(k)) unsafeAtomicAdd(P.y + row0(k) * P.ld + o1, r1[k]);
          }
          if (!(qq == 0 && cx == P.ncx - 1) && !(ODD && qq == H)) {
#pragma unroll
            for (int k = 0; k < N; ++k)
              if (kok(k)) unsafeAtomicAdd(P.y + row0(k) * P.ld + o2, r2[k]);
          }
        }
      }
    }
    // per-column quadratic form, in a fixed order
    if (P.energy && t < QC && ch * QC + t < P.cols) {
      double acc = 0.0;
      for (int u = 0; u < N; ++u)
#pragma unroll
        for (int v = 0; v < 4; ++v) acc += sRed[u * 64 + (F32 ? t * 4 + v : v * 16 + t)];
      P.energy[(int64_t)cell * P.eld + ch * QC + t] = acc;
    }
  }
}

// ----------------------------------------------------------------------------------------------
// host side
// ----------------------------------------------------------------------------------------------
template <typename T, int N, bool BOX>
tdfe_status launch_quad(tdfe_ctx* c, const QuadParams<T>& P, bool cells) {
  const dim3 grid((unsigned)(c->n_cell * P.nchunks)), block(64 * N);
  if (cells)
    hipLaunchKernelGGL((quad_kernel<T, N, BOX, true>), grid, block, 0, c->stream, P);
  else
    hipLaunchKernelGGL((quad_kernel<T, N, BOX, false>), grid, block, 0, c->stream, P);
  TDFE_HIP(c, hipGetLastError());
  return TDFE_OK;
}

template <typename T>
tdfe_status launch_quad_t(tdfe_ctx* c, const ApplyArgs& a) {
  QuadParams<T> P{};
  P.x = a.x;
  P.y = (T*)a.y;
  P.ld = a.ld;
  P.cols = a.cols;
  P.nchunks = (a.cols + QC - 1) / QC;
  P.eld = a.eld;
  P.colscale = a.colscale;
  P.kin = a.kin;
  P.vw = a.fp32 ? (const void*)a.vw32 : (const void*)a.vw;
  P.minv = c->minv;
  P.corners = c->corners;
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
  if (a.n_blocks_out) *a.n_blocks_out = c->n_cell;
  if (c->n == 8) return c->box ? launch_quad<T, 8, true>(c, P, a.cells) : launch_quad<T, 8, false>(c, P, a.cells);
  if constexpr (sizeof(T) == 8)
    if (c->n == 7) return c->box ? launch_quad<T, 7, true>(c, P, a.cells) : launch_quad<T, 7, false>(c, P, a.cells);
  return tdfe_fail(c, TDFE_EINVAL, "four-lane operator: unsupported order p=%d", c->p);
}

}  // namespace

// Where the four lanes of a line are used: n = 8 (all four hold entries) and
// FP64 at n = 7.  Measured per launch of 8 orbitals against the better of the
// other kernels: FP64 n = 8 588 : 815 (trilinear) and 123 : 127 us (box),
// n = 7 626 : 718 and 122 : 132; FP32 n = 8 389 : 406 and 59 : 64.  Below, a
// quarter of the lanes idle or the FP32 planes win: FP64 n = 6 644 : 554 and
// 121 : 106, n = 5 385 : 295, FP32 n = 7 530 : 470.  FP32 on trilinear cells: only
// where a block of 16 columns is not full, and where 32-bit offsets do not reach
// over a cell, which lane pairs need (14 x 13 x 15 cells, four lanes and pairs: 5
// orbitals 92 and 104 us, 8 104 and 94, 16 226 and 167, 32 427 and 340; 9 x 10 x
// 8: 5 32 and 40, 16 63 and 55).
bool tdfe_quad_kernel_ok(const tdfe_ctx* c, const ApplyArgs& a) {
  if (!c->box && a.fp32 && a.cols >= 16 &&
      tdfe_span::near(c->p, c->ncx, c->ncy, c->ncz, 1, (int64_t)a.ld * (int)sizeof(float)))
    return false;
  return c->variant == 0 && (c->n == 8 || (c->n == 7 && !a.fp32)) && a.cols > 8 &&
         c->n_cell * ((a.cols + QC - 1) / QC) < (int64_t)1 << 31 &&
         (int64_t)c->n * a.ld * (a.fp32 ? 4 : 8) < (int64_t)1 << 31;
}

tdfe_status tdfe_launch_apply_quad(tdfe_ctx* c, const ApplyArgs& a) {
  if (!tdfe_quad_kernel_ok(c, a)) return tdfe_fail(c, TDFE_EINVAL, "four-lane operator: unsupported launch");
  return a.fp32 ? launch_quad_t<float>(c, a) : launch_quad_t<double>(c, a);
}
