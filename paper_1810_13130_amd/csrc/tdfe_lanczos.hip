// Adaptive Lanczos exponential exp(-i tau Hbar) psibar on MI355X.
//
// Eqs. KrylovSubspace, zk, AdaptiveLanczos: for every orbital its own
// Lanczos recurrence on the real symmetric Hbar (run on the real and
// imaginary columns together, the scalars taken as pair sums), the small
// exponential y = exp(-i tau T_k) e_1 and the a-posteriori error
// eps_k = |tau| beta_k ||psibar|| |y_k|, checked after every iteration; an
// orbital is frozen once eps_k <= tol (or on happy breakdown), and the
// result is z = ||psibar|| sum_j y_j q_j.
//
// Device design:
//  * basis vectors are stored unnormalised (w_j) together with per-orbital
//    scale factors s_j = 1/beta_{j-1}; every consumer applies s_j on the fly,
//    which removes the normalisation pass;
//  * alpha_k = Re<q_k, Hbar q_k> comes from the operator kernel's own
//    quadrature-point quadratic form (no extra pass over the vectors);
//  * the three-term update and the norm partials are one streaming kernel,
//    which also sums the operator's per-cell results (update_cells_kernel) or,
//    where they do not pay, clears the operator output (update_kernel);
//  * all reductions are two-level with a fixed summation order
//    (deterministic);
//  * the small exponential is evaluated on the device by the Chebyshev
//    expansion of exp(-i tau x) on the Gershgorin interval of T_k
//    (Jacobi-Anger coefficients 2 (-i)^m J_m(tau r), Bessel values by
//    Miller's backward recurrence), one wavefront per orbital, rows across
//    lanes.  It gives the same y as an eigendecomposition of T_k to ~1e-15.
//    For k <= 256 it runs in leading blocks of the same iteration's update
//    kernel (T_k is complete once alpha_k is known), so the stop test after
//    the update is only a reduction and a comparison;
//  * the host enqueues iterations ahead, paced by a progress word the update
//    kernels store into pinned memory (no event per iteration: its queue
//    marker would drain the device before every operator launch), and stops
//    at a device "all converged" flag; iterations enqueued past convergence
//    exit at their first instruction.
#include <chrono>
#include <cmath>
#include <type_traits>

#include "tdfe_cells.h"
#include "tdfe_cheb.h"
#include "tdfe_internal.h"

namespace {

constexpr int RED_BLOCKS = 1024;  // blocks of the streaming reductions
constexpr int RED_THREADS = 256;
constexpr int CHK_THREADS = TDFE_CHEB_THREADS;

// scalar block layout per chunk (doubles), Nc = orbitals in the chunk
struct Scal {
  double* alpha;  // [k_max][Nc]
  double* beta;   // [k_max][Nc]
  double* scale;  // [k_max+2][Nc]  s_j applied to basis vector j (q_j = s_j w_j)
  double* cs;     // [k_max+2][Nc]  input scale of operator pass j: s_0, then s_j^2
  double* nrm;    // [Nc]
  double* err;    // [Nc]
  double* y;      // [Nc][k_max][2]
  double* ext;    // [Nc][2] max |alpha_j| and the term count of the last small exponential
  int* kconv;     // [Nc]
  int* status;    // [Nc] 0 active, 1 converged, 2 not converged at k_max, 3 Chebyshev too long
  int* nconv;     // [1]
  int* done;      // [1]
};

Scal carve_scal(tdfe_ctx* c, int Nc) {
  Scal s;
  double* p = c->scal;
  const int K = c->k_max;
  s.alpha = p;
  p += (size_t)K * Nc;
  s.beta = p;
  p += (size_t)K * Nc;
  s.scale = p;
  p += (size_t)(K + 2) * Nc;
  s.cs = p;
  p += (size_t)(K + 2) * Nc;
  s.nrm = p;
  p += Nc;
  s.err = p;
  p += Nc;
  s.y = p;
  p += (size_t)2 * K * Nc;
  s.ext = p;
  p += (size_t)2 * Nc;
  int* ip = (int*)c->counters;
  s.kconv = ip;
  s.status = ip + 64;
  s.nconv = ip + 128;
  s.done = ip + 129;
  return s;
}

// ---------------------------------------------------------------------------------------------
// block reduction helper: sums v over threads that share (t % C) -> out[col]
// ---------------------------------------------------------------------------------------------
__device__ void block_col_sum(double v, int C, double* sred, double* out) {
  const int t = threadIdx.x;
  sred[t] = v;
  __syncthreads();
  for (int s = blockDim.x / 2; s >= C; s >>= 1) {
    if (t < s) sred[t] += sred[t + s];
    __syncthreads();
  }
  if (t < C) out[t] = sred[t];
}

// sum of v over the block of RED_THREADS lanes, in thread 0: DPP adds within
// each wavefront (no LDS round trip, no barrier), one exchange of the four
// wavefronts' sums; fixed order.  The reductions between two operator passes
// are pure latency: with a tree of eight barriers and their scalars loaded
// after it they took 3.5 and 4.8 us of a 27 us iteration on a small box (a
// step of ten of these 336 -> 319 us with the reductions, the update's
// coefficients and its grid as they are here).
__device__ __forceinline__ double block_sum(double v, double* swave) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 63) swave[threadIdx.x >> 6] = v;
  __syncthreads();
  double s = swave[0];
#pragma unroll
  for (int w = 1; w < RED_THREADS / 64; ++w) s += swave[w];
  return s;
}

// copy one orbital chunk of the complex128 input into basis slot 0 (type T)
// and per-column sum of squares partials
template <typename T>
__global__ void __launch_bounds__(RED_THREADS)
    copy_in_kernel(const double* __restrict__ in, int ld_in, int col0, T* __restrict__ w0, int C, int64_t nrows,
                   double* __restrict__ partial) {
  __shared__ double sred[RED_THREADS];
  const int Cp = (C <= 1) ? 1 : (C <= 2 ? 2 : (C <= 4 ? 4 : (C <= 8 ? 8 : (C <= 16 ? 16 : (C <= 32 ? 32 : 64)))));
  const int col = threadIdx.x % Cp;
  const int rlane = threadIdx.x / Cp;
  const int rstride = (RED_THREADS / Cp) * gridDim.x;
  double acc = 0.0;
  if (col < C) {
    for (int64_t r = (int64_t)blockIdx.x * (RED_THREADS / Cp) + rlane; r < nrows; r += rstride) {
      const double v = in[r * ld_in + col0 + col];
      w0[r * C + col] = (T)v;
      acc += v * v;
    }
  }
  block_col_sum(acc, Cp, sred, sred);
  __syncthreads();
  if (threadIdx.x < C) partial[(int64_t)blockIdx.x * C + threadIdx.x] = sred[threadIdx.x];
}

// progress of the recurrence for the host's look-ahead: (generation, k) in
// one pinned word, stored without ordering (the host only uses it to pace
// its launches; results travel through the done flag and the readbacks).
// The update kernel of iteration k posts k - 1 when it starts, that is once
// iteration k - 1 has passed its stop test without finishing the set: after
// the set is done nothing is posted, and the host, waiting for a word that
// does not come, is already polling the done flag when it is raised.
constexpr int PROGRESS_KBITS = 11;  // k <= 1024
__device__ __forceinline__ void post_progress(unsigned* progress, int gen, int k) {
  if (progress)
    __hip_atomic_store(progress, ((unsigned)gen << PROGRESS_KBITS) | (unsigned)k, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

// The small exponential of iteration k rides on the update kernel of the same
// iteration: T_k needs alpha_1..alpha_k and beta_1..beta_{k-1}, all known when
// the update starts, and only the stop test waits for beta_k.  The first nblk blocks of the update grid each take
// one active orbital: y = exp(-i tau T_k) e_1 into its result slot (kept
// there when the orbital stops), and max |alpha| and the term count into ext.
struct SmallExp {
  Scal S;
  int Nc;
  int k;
  int k_max;
  int nblk;  // leading blocks that evaluate the small exponential (0: none)
  double tau;
  double* jtab;  // [Nc][TDFE_JTAB_STRIDE] Bessel tables
  unsigned* progress;  // pinned progress word (may be null)
  int gen;
  // alpha_k still as the operator's block partials [groups][2 Nc] (0: it is in
  // S.alpha), to be multiplied by mult^2 (may be null)
  const double* apart;
  int groups;
  const double* mult;
};

// alpha_k of orbital o from the operator's block partials, on one wavefront;
// every wavefront that asks forms the same sum in the same order
__device__ __forceinline__ double alpha_of(const SmallExp& e, int o) {
  const int C = 2 * e.Nc;
  const double m = e.mult ? e.mult[o] : 1.0;
  double acc = 0.0;
  sum_rows(e.groups, (int)threadIdx.x & 63, 64, [&](int64_t b) {
    const double2 p2 = *(const double2*)(e.apart + b * C + 2 * o);
    return p2.x + p2.y;
  }, acc);
  return lane_read(wave_sum(acc), 63) * (m * m);
}

//
// Up to SMALL_ROWS rows of T_k per lane, that is k <= 256 (chosen per launch
// as 1, 2 or 4, so that the common k <= 64 leaves the streaming blocks their
// registers).  In a kernel of its own after the update (as still beyond 256,
// where 8 or 16 rows take over 200 registers) the series cost 75 us of every
// iteration past 64 of a 1.26M-DoF FP64 exponential: 102.7 -> 100.0 ms over
// its 115 iterations.
constexpr int SMALL_ROWS = 4;
// R rows of T_k per lane; every load is issued before the first is waited for
template <int R, bool OWN>
__device__ void small_exp_block(const SmallExp& e, const int* done) {
  const int o = blockIdx.x;
  const int t = threadIdx.x;
  if (t >= CHK_THREADS) return;
  const int k = e.k, Nc = e.Nc;
  const int dn = *done, st = e.S.status[o];
  double a[R], bl[R], br[R], yr[R], yi[R], amax = 0.0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j = R * t + r;
    const bool row = j < k;
    a[r] = row ? e.S.alpha[(size_t)j * Nc + o] : 0.0;
    bl[r] = (row && j > 0) ? e.S.beta[(size_t)(j - 1) * Nc + o] : 0.0;
    br[r] = (row && j < k - 1) ? e.S.beta[(size_t)j * Nc + o] : 0.0;
  }
  double ak = 0.0;
  if constexpr (OWN) {
    ak = alpha_of(e, o);
#pragma unroll
    for (int r = 0; r < R; ++r) a[r] = R * t + r == k - 1 ? ak : a[r];
  }
  if (dn) return;
  if (o == 0 && t == 0) post_progress(e.progress, e.gen, k - 1);
  if (OWN && t == 0) e.S.alpha[(size_t)(k - 1) * Nc + o] = ak;
  if (st != 0) return;
  const int M = cheb_series<R>(k, a, bl, br, e.tau, e.jtab + (size_t)o * TDFE_JTAB_STRIDE, yr, yi, &amax);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j = R * t + r;
    if (j < k) {
      e.S.y[((size_t)o * e.k_max + j) * 2 + 0] = yr[r];
      e.S.y[((size_t)o * e.k_max + j) * 2 + 1] = yi[r];
    }
  }
  if (t == 0) {
    e.S.ext[2 * o + 0] = amax;
    e.S.ext[2 * o + 1] = (double)M;
  }
}

// Coefficients of the three-term step of one orbital (zero once it has
// stopped): every value is loaded before any is used, and before the kernel
// looks at its done flag, so that a short step waits for memory once.
struct Coef {
  double s, ca, cm;
  __device__ __forceinline__ Coef(const int* status, const double* alpha_j, const double* s_j, const double* m_j,
                                  int o) {
    const int st = status[o];
    const double sj = s_j[o], aj = alpha_j[o], mj = m_j ? m_j[o] : 1.0;
    s = st == 0 ? sj : 0.0;
    ca = st == 0 ? aj * sj : 0.0;
    cm = st == 0 ? mj : 0.0;
  }
};

// Three-term step in two reads.  The operator pass of vector j accumulates
// s_j^2 Hbar w_j (s_0 Hbar w_0 for j = 0) onto a buffer that this kernel
// seeded with -q_{j-1}, so that on entry Hq = (Hbar q_j - beta_{j-1} q_{j-1}) / m_j
// with m_j = beta_{j-1} (m_0 = 1).  Then
//   w_{j+1} = m_j Hq - alpha_j s_j w_j,   Hq <- -q_j = -s_j w_j,   partial ||w_{j+1}||^2.
template <typename T, int SR>
__global__ void __launch_bounds__(RED_THREADS)
    update_kernel(T* __restrict__ hq, const T* __restrict__ wa, T* __restrict__ wn, int C, int64_t nrows,
                  const double* alpha_j, const double* s_j, const double* m_j, const int* status,
                  double* __restrict__ partial, const int* done, SmallExp se) {
  __shared__ double sred[RED_THREADS];
  if ((int)blockIdx.x < se.nblk) {
    small_exp_block<SR, false>(se, done);
    return;
  }
  const int dn = *done;
  if (blockIdx.x == 0 && threadIdx.x == 0 && !dn) post_progress(se.progress, se.gen, se.k - 1);
  const int bid = (int)blockIdx.x - se.nblk;  // streaming block index, 0..RED_BLOCKS-1
  if constexpr (sizeof(T) == 4) {
    // FP32: a lane moves one orbital's (re, im) pair as one 8-byte access
    // (496 us per graded chunk of 16 orbitals, 6.5 TB/s; 4-byte accesses
    // 586 us); the orbital's sum of squares goes to its even column, 0 to
    // the odd one (the consumers sum column pairs)
    const int Nc2 = C >> 1;
    const int Op = (Nc2 <= 1) ? 1 : (Nc2 <= 2 ? 2 : (Nc2 <= 4 ? 4 : (Nc2 <= 8 ? 8 : (Nc2 <= 16 ? 16 : 32))));
    const int o = threadIdx.x % Op;
    const int rlane = threadIdx.x / Op;
    const int rstride = (RED_THREADS / Op) * (gridDim.x - se.nblk);
    double acc = 0.0;
    if (o < Nc2) {
      const Coef cf(status, alpha_j, s_j, m_j, o);
      if (dn) return;
      const double sd = cf.s, ca = cf.ca, cm = cf.cm;
      typedef float f2 __attribute__((ext_vector_type(2)));
      f2* __restrict__ h2 = (f2*)hq;
      const f2* __restrict__ a2 = (const f2*)wa;
      f2* __restrict__ n2 = (f2*)wn;
      for (int64_t r = (int64_t)bid * (RED_THREADS / Op) + rlane; r < nrows; r += rstride) {
        const int64_t i = r * Nc2 + o;
        const f2 a = __builtin_nontemporal_load(&a2[i]);
        const f2 h = __builtin_nontemporal_load(&h2[i]);
        f2 v, z;
        v.x = (float)(cm * (double)h.x - ca * (double)a.x);
        v.y = (float)(cm * (double)h.y - ca * (double)a.y);
        z.x = (float)(-sd * (double)a.x);
        z.y = (float)(-sd * (double)a.y);
        __builtin_nontemporal_store(z, &h2[i]);
        __builtin_nontemporal_store(v, &n2[i]);
        acc += (double)v.x * (double)v.x + (double)v.y * (double)v.y;
      }
    }
    if (dn) return;
    block_col_sum(acc, Op, sred, sred);
    __syncthreads();
    if (threadIdx.x < C) partial[(int64_t)bid * C + threadIdx.x] = (threadIdx.x & 1) ? 0.0 : sred[threadIdx.x >> 1];
    return;
  }
  const int Cp = (C <= 1) ? 1 : (C <= 2 ? 2 : (C <= 4 ? 4 : (C <= 8 ? 8 : (C <= 16 ? 16 : (C <= 32 ? 32 : 64)))));
  const int col = threadIdx.x % Cp;
  const int rlane = threadIdx.x / Cp;
  const int rstride = (RED_THREADS / Cp) * (gridDim.x - se.nblk);
  double acc = 0.0;
  if (col < C) {
    const int o = col >> 1;
    const Coef cf(status, alpha_j, s_j, m_j, o);
    if (dn) return;
    const double s = cf.s, ca = cf.ca, cm = cf.cm;
    for (int64_t r = (int64_t)bid * (RED_THREADS / Cp) + rlane; r < nrows; r += rstride) {
      const int64_t i = r * C + col;
      // non-temporal: each element is touched once here, and the vectors
      // (0.8 GB per chunk on the graded workload) are far larger than the
      // caches; measured 520 -> 502 us per FP64 update there
      const double a = (double)__builtin_nontemporal_load(&wa[i]);
      const double v = cm * (double)__builtin_nontemporal_load(&hq[i]) - ca * a;
      __builtin_nontemporal_store((T)(-s * a), &hq[i]);
      const T vt = (T)v;
      __builtin_nontemporal_store(vt, &wn[i]);
      acc += (double)vt * (double)vt;
    }
  }
  if (dn) return;
  block_col_sum(acc, Cp, sred, sred);
  __syncthreads();
  if (threadIdx.x < C) partial[(int64_t)bid * C + threadIdx.x] = sred[threadIdx.x];
}

// The three-term step after an operator that leaves per-cell results: one pass
// sums a DoF's contributions and takes the step,
//   w_{j+1} = m_j (sum of the cells' s_j^2 Hbar w_j) - alpha_j s_j w_j
//             - m_j s_{j-1} w_{j-1},      m_j = beta_{j-1} (1 and no last term for j = 0).
// Blocks work row by row of DoFs (see tdfe_cells.h), a lane moves 16 bytes of a
// row (one FP64 or two FP32 orbitals).  Reads the cell results once (n^3 / p^3
// vectors), w_j and w_{j-1}, writes w_{j+1}; no operator output vector is kept,
// seeded or cleared.
constexpr int CELL_BLOCKS = 2048;  // at most: one block per row of DoFs up to this
template <typename T, int W, int SR, bool OWN>
__global__ void __launch_bounds__(RED_THREADS)
    update_cells_kernel(const T* __restrict__ e, const T* __restrict__ wa, const T* __restrict__ wp,
                        T* __restrict__ wn, int C, CellMap M, const double* alpha_j, const double* s_j,
                        const double* m_j, const double* s_p, const int* status, double* __restrict__ partial,
                        const int* done, SmallExp se) {
  typedef typename CellLane<T, W>::V V;
  constexpr int NO = W / 2;  // orbitals per lane
  __shared__ double sred[RED_THREADS];
  __shared__ double sorb[2 * RED_THREADS / 4];
  __shared__ double salpha[TDFE_MAX_COLS / 2];
  if ((int)blockIdx.x < se.nblk) {
    small_exp_block<SR, OWN>(se, done);
    return;
  }
  const int dn = *done;
  if (blockIdx.x == 0 && threadIdx.x == 0 && !dn) post_progress(se.progress, se.gen, se.k - 1);
  const int bid = (int)blockIdx.x - se.nblk;
  const int C2 = C / W;
  const int Op = C2 <= 4 ? 4 : (C2 <= 8 ? 8 : (C2 <= 16 ? 16 : 32));
  const int XL = RED_THREADS / Op;
  const int o = (int)threadIdx.x % Op;
  const int xl = (int)threadIdx.x / Op;
  double acc[NO], ca[NO], cm[NO], cb[NO];
#pragma unroll
  for (int q = 0; q < NO; ++q) {
    const int oo = min(o, C2 - 1) * NO + q;
    const Coef cf(status, alpha_j, s_j, m_j, oo);
    const double sp = s_p[oo];
    ca[q] = OWN ? cf.s : cf.ca;
    cm[q] = cf.cm;
    cb[q] = wp ? cf.cm * sp : 0.0;
    acc[q] = 0.0;
  }
  if constexpr (OWN) {
    // few operator blocks: every block sums their partials itself (see run_chunk)
    for (int oo = (int)threadIdx.x >> 6; oo < se.Nc; oo += RED_THREADS / 64) {
      const double al = alpha_of(se, oo);
      if ((threadIdx.x & 63) == 0) salpha[oo] = al;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NO; ++q) ca[q] = ca[q] != 0.0 ? ca[q] * salpha[min(o, C2 - 1) * NO + q] : 0.0;
  }
  if (o < C2) {
    if (dn) return;
    const int nrows = M.NyI * M.NzI;
    for (int r = bid; r < nrows; r += (int)gridDim.x - se.nblk) {
      const CellRow R = cell_row(M, 1 + r % M.NyI, 1 + r / M.NyI);
      for (int I = xl; I < M.NxI; I += XL) {
        CellLane<T, W> L;
        L.at(M, I);
        const int64_t d = ((int64_t)r * M.NxI + I) * C2 + o;
        const V a = __builtin_nontemporal_load((const V*)wa + d);
        V b = (V)0;
        if (wp) b = __builtin_nontemporal_load((const V*)wp + d);
        double h[W];
        L.sum(e, R, C, o, h);
        V w;
#pragma unroll
        for (int q = 0; q < W; ++q) {
          w[q] = (T)(cm[q / 2] * h[q] - ca[q / 2] * (double)a[q] - cb[q / 2] * (double)b[q]);
          acc[q / 2] += (double)w[q] * (double)w[q];
        }
        __builtin_nontemporal_store(w, (V*)wn + d);
      }
    }
  }
  if (dn) return;
#pragma unroll
  for (int q = 0; q < NO; ++q) {
    block_col_sum(acc[q], Op, sred, sred);
    __syncthreads();
    if (threadIdx.x < C2) sorb[threadIdx.x * NO + q] = sred[threadIdx.x];
    __syncthreads();
  }
  // the consumers sum column pairs: the orbital's sum in its even column
  if (threadIdx.x < C) partial[(int64_t)bid * C + threadIdx.x] = (threadIdx.x & 1) ? 0.0 : sorb[threadIdx.x >> 1];
}

// out[o] = f( sum_b partial[b][2o] + partial[b][2o+1] ), one block per orbital, fixed order.
// mode 0: plain sum, times mult[o]^2 if mult is given (alpha from the quadratic form of the
//         scaled operator input); 2: sqrt, scale0[o] = 1/sqrt and cs0[o] = scale0[o] (0 if
//         zero); 3: as 2 with cs0[o] = scale0[o]^2
__global__ void __launch_bounds__(RED_THREADS)
    finalize_pairs_kernel(const double* __restrict__ partial, int64_t nblocks, int C, double* out, int mode,
                          double* scale0, double* cs0, const double* mult, const int* done) {
  __shared__ double swave[RED_THREADS / 64];
  const int o = blockIdx.x;
  const int dn = done ? *done : 0;
  const double mo = mult ? mult[o] : 1.0;
  double acc = 0.0;
  sum_rows(nblocks, (int)threadIdx.x, RED_THREADS, [&](int64_t b) {
    const double2 p2 = *(const double2*)(partial + b * C + 2 * o);
    return p2.x + p2.y;
  }, acc);
  double v = block_sum(acc, swave);
  if (threadIdx.x == 0 && !dn) {
    if (mode == 0 && mult) v *= mo * mo;
    if (mode >= 1) v = sqrt(v);
    out[o] = v;
    if (mode >= 2) {
      const double sc = v > 0.0 ? 1.0 / v : 0.0;
      scale0[o] = sc;
      if (cs0) cs0[o] = mode == 3 ? sc * sc : sc;
    }
  }
}

// first level of a two-level fixed-order sum of [nrows][C] partials: block b
// sums its contiguous share of rows for every column into out[b][C] (the
// second level is finalize_pairs_kernel over the ALPHA_SLICES rows of out)
constexpr int ALPHA_SLICES = 128;
// up to this many partials every block of the update sums them itself
constexpr int ALPHA_OWN = 2048;
__global__ void __launch_bounds__(RED_THREADS)
    slice_sums_kernel(const double* __restrict__ partial, int64_t nrows, int C, double* __restrict__ out,
                      const int* done) {
  __shared__ double sred[RED_THREADS];
  if (done && *done) return;
  const int Cp = (C <= 1) ? 1 : (C <= 2 ? 2 : (C <= 4 ? 4 : (C <= 8 ? 8 : (C <= 16 ? 16 : (C <= 32 ? 32 : 64)))));
  const int col = threadIdx.x % Cp;
  const int rl = threadIdx.x / Cp;
  const int nl = RED_THREADS / Cp;
  const int64_t per = (nrows + ALPHA_SLICES - 1) / ALPHA_SLICES;
  const int64_t r0 = (int64_t)blockIdx.x * per;
  const int64_t r1 = r0 + per < nrows ? r0 + per : nrows;
  double acc = 0.0;
  if (col < C)
    sum_rows(r1 - r0, rl, nl, [&](int64_t r) { return partial[(r0 + r) * C + col]; }, acc);
  sred[threadIdx.x] = acc;
  __syncthreads();
  if (rl == 0 && col < C) {
    double s = 0.0;
    for (int l = 0; l < nl; ++l) s += sred[l * Cp + col];
    out[(int64_t)blockIdx.x * C + col] = s;
  }
}

// ---------------------------------------------------------------------------------------------
// small exponential and adaptive stop, one wavefront per orbital
// ---------------------------------------------------------------------------------------------
// stop decision of orbital o after the small exponential: error estimate, y at
// convergence (from Lyr / Lyi, or already in its result slot if these are
// null), status; called by nthreads lanes
__device__ void stop_test(Scal S, int o, int Nc, int k, int k_max, int kcap, double tau, double tol, double tol_rel,
                          int M, double amax, double nrm, double bk, double ylr, double yli, const double* Lyr,
                          const double* Lyi, int nthreads, int* err_flag, int* host_flag, int gen) {
  const int t = threadIdx.x;
  int fin = 0;
  if (M < 0) {
    if (t == 0) {
      // 3: |tau| ||T_k|| beyond the Bessel table (TDFE_EINVAL); 4: T_k not finite
      const bool nf = M == TDFE_CHEB_NONFINITE;
      S.status[o] = nf ? 4 : 3;
      if (!nf) atomicOr(err_flag, 1);
      if (atomicAdd(S.nconv, 1) + 1 == Nc) {
        *S.done = 1;
        fin = 1;
      }
    }
  } else {
    const double eps = fabs(tau) * bk * nrm * sqrt(ylr * ylr + yli * yli);
    const bool happy = bk <= 1e-14 * amax;
    // mixed precision: no tighter than the storage precision of the basis allows
    const bool conv = (eps <= fmax(tol, tol_rel * nrm)) || happy;
    // a NaN or Inf in beta_k or in the small exponential ends the orbital at
    // once (status 4, reported as TDFE_ENONFINITE) instead of running to k_max
    const bool nonfinite = !isfinite(eps);
    // kcap: the chunk's Krylov dimension limit (k_max, or a soft cap)
    const bool stop = conv || nonfinite || k >= kcap;
    if (stop && Lyr) {
      for (int j = t; j < k; j += nthreads) {
        S.y[((size_t)o * k_max + j) * 2 + 0] = Lyr[j];
        S.y[((size_t)o * k_max + j) * 2 + 1] = Lyi[j];
      }
    }
    if (t == 0) {
      S.err[o] = eps;
      if (stop) {
        S.kconv[o] = k;
        S.status[o] = nonfinite ? 4 : (conv ? 1 : 2);
        S.scale[(size_t)k * Nc + o] = 0.0;  // freezes the orbital in later operator passes
        S.cs[(size_t)k * Nc + o] = 0.0;
        if (atomicAdd(S.nconv, 1) + 1 == Nc) {
          *S.done = 1;
          fin = 1;
        }
      }
    }
  }
  // the orbital that completes the set raises the host-visible flag (pinned
  // memory) to this run's generation number: a write left over from an
  // earlier run cannot be mistaken for this one, so the host needs no
  // synchronisation between runs; the host reads it once an iteration's
  // event has completed
  if (fin && host_flag) {
    *host_flag = gen;
    __threadfence_system();
  }
}

__global__ void __launch_bounds__(CHK_THREADS)
    check_kernel(Scal S, int Nc, int k, int k_max, int kcap, double tau, double tol, double tol_rel, int* err_flag,
                 int* host_flag, int gen, double* jtab) {
  __shared__ ChebLds L;
  __shared__ double sa[TDFE_KCAP], sb[TDFE_KCAP];
  const int o = blockIdx.x;
  const int t = threadIdx.x;
  if (*S.done || S.status[o] != 0) return;
  for (int j = t; j < k; j += CHK_THREADS) {
    sa[j] = S.alpha[(size_t)j * Nc + o];
    sb[j] = S.beta[(size_t)j * Nc + o];  // sb[k-1] = beta_k (not part of T_k)
  }
  __syncthreads();
  double amax = 0.0;
  const int M = cheb_expm_e1(k, sa, sb, tau, L, jtab + (size_t)o * TDFE_JTAB_STRIDE, &amax);
  stop_test(S, o, Nc, k, k_max, kcap, tau, tol, tol_rel, M, amax, S.nrm[o], sb[k - 1], L.yr[k - 1], L.yi[k - 1], L.yr, L.yi,
            CHK_THREADS, err_flag, host_flag, gen);
}

// beta_k = ||w_k|| from the update partials, the scale 1/beta_k of the next
// basis vector, and the stop test of the same orbital, on the small
// exponential the update kernel has left in its result slot and ext
__global__ void __launch_bounds__(RED_THREADS)
    beta_check_kernel(const double* __restrict__ partial, int64_t nblocks, int C, Scal S, int Nc, int k, int k_max,
                      int kcap, double tau, double tol, double tol_rel, int* err_flag, int* host_flag, int gen) {
  __shared__ double swave[RED_THREADS / 64];
  const int o = blockIdx.x;
  const int dn = *S.done, st = S.status[o];
  const double amax = S.ext[2 * o + 0], terms = S.ext[2 * o + 1], nrm = S.nrm[o];
  const double2 yl = *(const double2*)(S.y + ((size_t)o * k_max + k - 1) * 2);
  double acc = 0.0;
  sum_rows(nblocks, (int)threadIdx.x, RED_THREADS, [&](int64_t b) {
    const double2 p2 = *(const double2*)(partial + b * C + 2 * o);
    return p2.x + p2.y;
  }, acc);
  const double bk = sqrt(block_sum(acc, swave));
  if (threadIdx.x != 0 || dn) return;
  const double sc = bk > 0.0 ? 1.0 / bk : 0.0;
  S.beta[(size_t)(k - 1) * Nc + o] = bk;
  S.scale[(size_t)k * Nc + o] = sc;
  S.cs[(size_t)k * Nc + o] = sc * sc;
  if (st != 0) return;
  stop_test(S, o, Nc, k, k_max, kcap, tau, tol, tol_rel, (int)terms, amax, nrm, bk, yl.x, yl.y, nullptr, nullptr, 1,
            err_flag, host_flag, gen);
}

// z = ||psi|| sum_j y_j s_j w_j, written into the complex128 output chunk.
// A lane keeps one orbital and takes RPT rows; the coefficients y_j s_j of the
// block's orbitals are staged in LDS in tiles of COMB_JT iterations (kcap: an
// upper bound of every orbital's k, the iterations enqueued), and 8 values
// are loaded per round so that several loads are in flight per lane.  Reads
// the whole basis once, so memory bounds it; four rows per lane (from 2^18
// values on) spread a block's start, two dependent reads and the staging,
// over four times the data
// (one row each: 209 us for 18 FP64 vectors of 63 MB, 89 us for 12 FP32 ones,
// 7.6 ms for 115 of 374 MB; so 189 us, 80 us and 7.3 ms, 6.0 TB/s).
constexpr int COMB_JT = 32;
template <typename T, int RPT>
__global__ void __launch_bounds__(256)
    combine_kernel(const T* __restrict__ W, int64_t stride_vec, int C, int64_t nrows, Scal S, int Nc, int k_max,
                   int kcap, double* __restrict__ out, int ld_out, int col0) {
  typedef T V2 __attribute__((ext_vector_type(2)));
  constexpr int JU = 8 / RPT;  // iterations per round
  __shared__ double2 sa[COMB_JT * (TDFE_MAX_COLS / 2)];
  const int rpb = 256 / Nc;  // rows side by side in a block
  const int o = (int)threadIdx.x % Nc, rl = (int)threadIdx.x / Nc;
  const int64_t r0 = (int64_t)blockIdx.x * RPT * rpb + rl;
  const int kc = rl < rpb && r0 < nrows ? S.kconv[o] : 0;
  const V2* __restrict__ w[RPT];
#pragma unroll
  for (int u = 0; u < RPT; ++u) {
    const int64_t r = r0 + u * rpb;
    w[u] = (const V2*)W + (r < nrows ? r : 0) * Nc + o;
  }
  const int64_t sv = stride_vec >> 1;
  double zr[RPT], zi[RPT];
#pragma unroll
  for (int u = 0; u < RPT; ++u) zr[u] = zi[u] = 0.0;
  for (int j0 = 0; j0 < kcap; j0 += COMB_JT) {
    const int jt = min(COMB_JT, kcap - j0);
    __syncthreads();
    for (int i = threadIdx.x; i < jt * Nc; i += blockDim.x) {
      const int jj = j0 + i / Nc, oo = i % Nc;
      const double sc = S.scale[(size_t)jj * Nc + oo];
      sa[i] = make_double2(S.y[((size_t)oo * k_max + jj) * 2 + 0] * sc, S.y[((size_t)oo * k_max + jj) * 2 + 1] * sc);
    }
    __syncthreads();
    const int je = min(kc - j0, jt);  // this orbital's iterations in the tile (none if <= 0)
    auto round = [&](int jj, auto count) {
      constexpr int J = decltype(count)::value;
      V2 q[J][RPT];
#pragma unroll
      for (int v = 0; v < J; ++v)
#pragma unroll
        for (int u = 0; u < RPT; ++u) q[v][u] = __builtin_nontemporal_load(w[u] + (j0 + jj + v) * sv);
#pragma unroll
      for (int v = 0; v < J; ++v) {
        const double2 a = sa[(jj + v) * Nc + o];
#pragma unroll
        for (int u = 0; u < RPT; ++u) {
          const double qr = (double)q[v][u].x, qi = (double)q[v][u].y;
          zr[u] += a.x * qr - a.y * qi;
          zi[u] += a.x * qi + a.y * qr;
        }
      }
    };
    int jj = 0;
    for (; jj + JU <= je; jj += JU) round(jj, std::integral_constant<int, JU>{});
    for (; jj < je; ++jj) round(jj, std::integral_constant<int, 1>{});
  }
  if (rl >= rpb) return;
  const double nr = S.nrm[o];
#pragma unroll
  for (int u = 0; u < RPT; ++u) {
    const int64_t r = r0 + u * rpb;
    if (r < nrows) {
      out[r * ld_out + col0 + 2 * o] = nr * zr[u];
      out[r * ld_out + col0 + 2 * o + 1] = nr * zi[u];
    }
  }
}

__global__ void init_scal_kernel(Scal S, int Nc) {
  const int o = threadIdx.x;
  if (o < Nc) {
    S.status[o] = 0;
    S.kconv[o] = 0;
    S.err[o] = 0.0;
  }
  if (o == 0) {
    *S.nconv = 0;
    *S.done = 0;
  }
}

// orbitals with zero norm are finished before the first iteration; a
// non-finite norm (a NaN or Inf entry in the orbital) finishes the orbital
// with status 4, which the host reports as TDFE_ENONFINITE
__global__ void zero_norm_kernel(Scal S, int Nc, int* host_flag, int gen) {
  const int o = threadIdx.x;
  const double nr = o < Nc ? S.nrm[o] : 1.0;
  const bool bad = !isfinite(nr);
  if (o < Nc && (bad || !(nr > 0.0))) {
    S.status[o] = bad ? 4 : 1;
    S.kconv[o] = 0;
    if (atomicAdd(S.nconv, 1) + 1 == Nc) {
      *S.done = 1;
      *host_flag = gen;
      __threadfence_system();
    }
  }
}

// per-orbital results of one chunk into a deferred-result slot:
// [n_max] k, [n_max] status, [n_max] error estimate, [1] Chebyshev-table flag
__global__ void stash_results_kernel(const int* kconv, const int* status, const double* err, const int* err_flag,
                                     int Nc, int o0, int n_max, double* slot) {
  for (int o = threadIdx.x; o < Nc; o += blockDim.x) {
    slot[o0 + o] = (double)kconv[o];
    slot[n_max + o0 + o] = (double)status[o];
    slot[2 * n_max + o0 + o] = err[o];
  }
  if (threadIdx.x == 0 && *err_flag) slot[3 * n_max] = 1.0;
}

// One chunk of Nc orbitals.  Kc < k_max runs a soft-capped chunk (wider than
// the basis memory holds at k_max): if an orbital reaches Kc unconverged, the
// chunk ends before its combination (the input is untouched) with *restart
// set, and the caller runs those orbitals again at k_max.
template <typename T>
tdfe_status run_chunk(tdfe_ctx* c, const void* vw, const double* in, double* out, int ld, int o0, int Nc,
                      double tau, double tol, int* k_out, double* err_out, int* status_out, LanczosHook* hook,
                      double* defer_slot, int Kc, bool* restart) {
  const int C = 2 * Nc;
  const int64_t nd = c->n_dof;
  const int64_t vstride = nd * C;
  T* W = (T*)c->krylov;
  T* Hq = (T*)c->hq;
  Scal S = carve_scal(c, Nc);
  const int K = c->k_max;
  *restart = false;
  // the basis holds (k_max + 1) vectors of 2 chunk_orb columns; the operator
  // output and the Bessel tables max(chunk_orb, wide_orb) orbitals
  if (Kc < 1 || Kc > K || (int64_t)(Kc + 1) * C > (int64_t)(K + 1) * 2 * c->chunk_orb ||
      Nc > std::max(c->chunk_orb, c->wide_orb) || (Kc < K && hook))
    return tdfe_fail(c, TDFE_EINVAL, "Lanczos chunk of %d orbitals with cap %d does not fit the workspace", Nc, Kc);
  int* err_flag = (int*)c->counters + 140;
  // FP32 basis vectors carry rounding of 2^-24 relative: a Krylov error
  // estimate below a small multiple of that (times ||psibar||) buys nothing
  const double tol_rel = sizeof(T) == 4 ? TDFE_MIXED_TOL_FLOOR : 0.0;

  // per-cell operator output summed by the update itself (the nonlocal term
  // adds to an assembled vector)
  const bool cells = c->n_proj == 0 && tdfe_cells_ok(c, C, sizeof(T) == 4);
  const CellMap map{c->ncx, c->ncy, c->ncz, c->p, c->Nx - 2, c->Ny - 2, c->Nz - 2};
  // streaming blocks of the update, and rows of its norm partials
  const int red_blocks = cells ? std::min(CELL_BLOCKS, map.NyI * map.NzI) : RED_BLOCKS;
  hipLaunchKernelGGL(init_scal_kernel, dim3(1), dim3(64), 0, c->stream, S, Nc);
  if (!cells) TDFE_TRY(tdfe_zero(c, Hq, (size_t)vstride * sizeof(T)));
  TDFE_TRY(tdfe_zero(c, err_flag, sizeof(int)));
  hipLaunchKernelGGL((copy_in_kernel<T>), dim3(RED_BLOCKS), dim3(RED_THREADS), 0, c->stream, in, ld, 2 * o0, W, C, nd,
                     c->partial);
  hipLaunchKernelGGL(finalize_pairs_kernel, dim3(Nc), dim3(RED_THREADS), 0, c->stream, c->partial,
                     (int64_t)RED_BLOCKS, C, S.nrm, 2, S.scale, S.cs, (const double*)nullptr, (const int*)nullptr);
  // host-visible copy of the done flag (pinned memory), tagged with this
  // run's generation number
  volatile int* hflag = c->poll + 32;
  const int gen = ++c->flag_gen;
  int* dflag = nullptr;
  TDFE_HIP(c, hipHostGetDevicePointer((void**)&dflag, (void*)(c->poll + 32), 0));
  hipLaunchKernelGGL(zero_norm_kernel, dim3(1), dim3(64), 0, c->stream, S, Nc, dflag, gen);
  TDFE_HIP(c, hipGetLastError());
  // the recurrence's progress word (pinned, posted by the update kernels):
  // read by the host to stay LOOK iterations ahead of the device.  An event recorded per iteration would do
  // the same but drains the queue before the next operator launch (about
  // 5 us per iteration on this device).
  volatile unsigned* hprog = (volatile unsigned*)(c->poll + 34);
  unsigned* dprog = nullptr;
  TDFE_HIP(c, hipHostGetDevicePointer((void**)&dprog, (void*)(c->poll + 34), 0));
  const unsigned gtag = (unsigned)gen & ((1u << (32 - PROGRESS_KBITS)) - 1u);

  const int LOOK = 2;
  int k_enq = 0;
  for (int k = 1; k <= Kc; ++k) {
    k_enq = k;
    T* wk = W + (int64_t)(k - 1) * vstride;
    ApplyArgs a{};
    a.x = wk;
    a.y = Hq;
    a.ld = C;
    a.cols = C;
    a.colscale = S.cs + (size_t)(k - 1) * Nc;
    a.kin = 0.5;
    a.vw = (const double*)vw;
    a.vw32 = (const float*)vw;
    a.lowdin = true;
    a.fullgrid = false;
    a.nonlocal = true;
    a.energy = c->partial;
    int64_t groups = 0;
    a.n_blocks_out = &groups;
    a.done_flag = S.done;
    a.fp32 = sizeof(T) == 4;
    TDFE_TRY(cells ? tdfe_launch_apply_cells(c, a) : tdfe_launch_apply(c, a));
    // m = beta_{k-2} for k >= 2 (the operator input was scaled by s^2, not s), 1 for k = 1
    const double* m = k >= 2 ? S.beta + (size_t)(k - 2) * Nc : (const double*)nullptr;
    const bool ride = k <= SMALL_ROWS * CHK_THREADS;  // small exponential on the update's leading blocks
    // Few operator blocks: alpha is summed by the update's own blocks, each for
    // itself, and left in S.alpha by the blocks of the small exponential; the
    // update's norm partials then lie behind the operator's.  A launch of 2 to 3
    // us less in iterations of 19 (one orbital on 4^3 cells, 11 blocks: a step
    // of ten 290 -> 264 us) to 27 us (4 orbitals on 8^3 cells, 256 blocks: 28.6
    // -> 27.7 ms in 680); beyond, every block's reads of all partials grow past
    // what the launch costs.  Up to k = 64 only: its registers (80 instead of
    // 44) are not worth having in the kernels of long iterations.
    const bool own_alpha = cells && k <= CHK_THREADS && groups * C <= ALPHA_OWN;
    double* const norms = own_alpha ? c->partial + ALPHA_OWN : c->partial;
    if (!own_alpha && groups > 64 * ALPHA_SLICES) {
      // many operator blocks: a first level over slices of rows (all columns
      // at once), then the per-orbital sums over the slices (29,791 blocks:
      // 13 us against 45 us in one level; 4,096 blocks: 9.5 us against 6.8 us)
      hipLaunchKernelGGL(slice_sums_kernel, dim3(ALPHA_SLICES), dim3(RED_THREADS), 0, c->stream,
                         (const double*)c->partial, groups, C, c->partial2, (const int*)S.done);
      hipLaunchKernelGGL(finalize_pairs_kernel, dim3(Nc), dim3(RED_THREADS), 0, c->stream, (const double*)c->partial2,
                         (int64_t)ALPHA_SLICES, C, S.alpha + (size_t)(k - 1) * Nc, 0, (double*)nullptr, (double*)nullptr,
                         m, (const int*)S.done);
    } else if (!own_alpha) {
      hipLaunchKernelGGL(finalize_pairs_kernel, dim3(Nc), dim3(RED_THREADS), 0, c->stream, c->partial, groups, C,
                         S.alpha + (size_t)(k - 1) * Nc, 0, (double*)nullptr, (double*)nullptr, m, (const int*)S.done);
    }
    SmallExp se{S, Nc, k, K, ride ? Nc : 0, tau, c->jtab, dprog, gen, c->partial, own_alpha ? (int)groups : 0, m};
    auto update = [&](auto rows) {
      constexpr int R = decltype(rows)::value;
      if (!cells) {
        hipLaunchKernelGGL((update_kernel<T, R>), dim3(red_blocks + se.nblk), dim3(RED_THREADS), 0, c->stream, Hq,
                           (const T*)wk, W + (int64_t)k * vstride, C, nd,
                           (const double*)(S.alpha + (size_t)(k - 1) * Nc),
                           (const double*)(S.scale + (size_t)(k - 1) * Nc), m, (const int*)S.status, c->partial,
                           (const int*)S.done, se);
        return;
      }
      auto run = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(red_blocks + se.nblk), dim3(RED_THREADS), 0, c->stream, (const T*)c->eloc,
                           (const T*)wk, k >= 2 ? (const T*)(wk - vstride) : (const T*)nullptr,
                           W + (int64_t)k * vstride, C, map, (const double*)(S.alpha + (size_t)(k - 1) * Nc),
                           (const double*)(S.scale + (size_t)(k - 1) * Nc), m,
                           (const double*)(S.scale + (size_t)(k >= 2 ? k - 2 : 0) * Nc), (const int*)S.status,
                           norms, (const int*)S.done, se);
      };
      // 16 bytes per lane where the columns allow it
      constexpr int WIDE = sizeof(T) == 4 ? 4 : 2;
      constexpr bool CAN_OWN = R == 1;
      if (CAN_OWN && own_alpha)
        C % WIDE == 0 ? run(update_cells_kernel<T, WIDE, R, CAN_OWN>) : run(update_cells_kernel<T, 2, R, CAN_OWN>);
      else
        C % WIDE == 0 ? run(update_cells_kernel<T, WIDE, R, false>) : run(update_cells_kernel<T, 2, R, false>);
    };
    if (k <= CHK_THREADS || !ride)
      update(std::integral_constant<int, 1>{});
    else if (k <= 2 * CHK_THREADS)
      update(std::integral_constant<int, 2>{});
    else
      update(std::integral_constant<int, SMALL_ROWS>{});
    // beta_k, the scale 1/beta_k of the next basis vector and the stop test
    if (ride) {
      hipLaunchKernelGGL(beta_check_kernel, dim3(Nc), dim3(RED_THREADS), 0, c->stream, (const double*)norms,
                         (int64_t)red_blocks, C, S, Nc, k, K, Kc, tau, tol, tol_rel, err_flag, dflag, gen);
    } else {
      hipLaunchKernelGGL(finalize_pairs_kernel, dim3(Nc), dim3(RED_THREADS), 0, c->stream, c->partial,
                         (int64_t)red_blocks, C, S.beta + (size_t)(k - 1) * Nc, 3, S.scale + (size_t)k * Nc,
                         S.cs + (size_t)k * Nc, (const double*)nullptr, (const int*)S.done);
      hipLaunchKernelGGL(check_kernel, dim3(Nc), dim3(CHK_THREADS), 0, c->stream, S, Nc, k, K, Kc, tau, tol, tol_rel,
                         err_flag, dflag, gen, c->jtab);
    }
    TDFE_HIP(c, hipGetLastError());
    if (k > LOOK) {
      // wait until iteration k - LOOK has passed its stop test (posted when
      // the next update starts) or the set is done.  The progress word only
      // paces the launches: after every 2 ms without it the stream is queried
      // (a query puts a marker into the queue, which costs the device a
      // drain, so it is kept off the normal path), and if the stream has
      // drained the loop goes on
      const unsigned want = (unsigned)(k - LOOK);
      auto t_last = std::chrono::steady_clock::now();
      for (int spin = 1;; ++spin) {
        if (*hflag == gen) break;
        const unsigned v = *hprog;
        if ((v >> PROGRESS_KBITS) == gtag && (v & ((1u << PROGRESS_KBITS) - 1u)) >= want) break;
        if ((spin & 255) == 0) {
          const auto now = std::chrono::steady_clock::now();
          if (now - t_last > std::chrono::milliseconds(2)) {
            const hipError_t q = hipStreamQuery(c->stream);
            if (q == hipSuccess) break;
            if (q != hipErrorNotReady) return tdfe_fail(c, TDFE_EDEVICE, "Lanczos: %s", hipGetErrorString(q));
            t_last = now;
          }
        }
        __builtin_ia32_pause();
      }
      if (*hflag == gen) break;
    }
  }
  if (hook)
    TDFE_TRY(hook->after_loop(c, W, vstride, Nc, o0, S.scale, S.kconv, S.alpha, S.beta, S.nrm, k_enq, sizeof(T) == 4));
  if (Kc < K) {
    // soft cap: the states decide between the combination and a restart
    const void* hs = nullptr;
    TDFE_TRY(tdfe_readback(c, S.status, Nc * sizeof(int), 256, &hs));
    TDFE_HIP(c, hipStreamSynchronize(c->stream));
    for (int o = 0; o < Nc; ++o)
      if (((const volatile int*)hs)[o] == 2) *restart = true;
    if (*restart) return TDFE_OK;
  }
  // combination
  {
    auto combine = [&](auto kernel, int rows) {
      hipLaunchKernelGGL(kernel, dim3((unsigned)((nd + rows - 1) / rows)), dim3(256), 0, c->stream, (const T*)W, vstride,
                         C, nd, S, Nc, K, std::min(k_enq, K), out, ld, 2 * o0);
    };
    if (nd * C >= 1 << 18)
      combine(combine_kernel<T, 4>, 4 * (256 / Nc));
    else
      combine(combine_kernel<T, 1>, 256 / Nc);
    TDFE_HIP(c, hipGetLastError());
  }
  if (defer_slot) {
    // results stay on the device until the caller's single readback
    hipLaunchKernelGGL(stash_results_kernel, dim3(1), dim3(64), 0, c->stream, (const int*)S.kconv,
                       (const int*)S.status, (const double*)S.err, (const int*)err_flag, Nc, o0, c->n_orb_max,
                       defer_slot);
    TDFE_HIP(c, hipGetLastError());
    return TDFE_OK;
  }
  // results through the pinned readback area (Nc <= 32: 128 + 128 + 256 + 4 bytes)
  const void *hk = nullptr, *hs = nullptr, *he = nullptr, *hf = nullptr;
  TDFE_TRY(tdfe_readback(c, S.kconv, Nc * sizeof(int), 0, &hk));
  TDFE_TRY(tdfe_readback(c, S.status, Nc * sizeof(int), 256, &hs));
  TDFE_TRY(tdfe_readback(c, S.err, Nc * sizeof(double), 512, &he));
  TDFE_TRY(tdfe_readback(c, err_flag, sizeof(int), 1024, &hf));
  TDFE_HIP(c, hipStreamSynchronize(c->stream));
  for (int o = 0; o < Nc; ++o) {
    k_out[o] = ((const volatile int*)hk)[o];
    err_out[o] = ((const volatile double*)he)[o];
    status_out[o] = ((const volatile int*)hs)[o];
  }
  const int ef = *(const volatile int*)hf;
  if (ef) return tdfe_fail(c, TDFE_EINVAL, "small exponential: |tau| ||T|| too large for the Chebyshev table");
  return TDFE_OK;
}

}  // namespace

tdfe_status tdfe_poll_events(tdfe_ctx* c) {
  if (c->evs) return TDFE_OK;
  c->evs = new hipEvent_t[TDFE_N_EVENTS];
  c->n_evs = 0;
  for (int i = 0; i < TDFE_N_EVENTS; ++i) {
    // host-side completion only: the flags the host reads are written by the
    // kernels themselves with a system-scope fence
    TDFE_HIP(c, hipEventCreateWithFlags(&c->evs[i], hipEventDisableTiming | hipEventDisableSystemFence));
    c->n_evs = i + 1;
  }
  return TDFE_OK;
}

// zero fill by a kernel: hipMemsetAsync costs tens of microseconds of stream
// idle time around its own fill launch, more than the fill itself here
__global__ void zero_kernel(unsigned* p, int64_t nwords) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  const int64_t n4 = ((uintptr_t)p % 16 == 0) ? nwords / 4 : 0;
  uint4* q = (uint4*)p;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4; i += stride) q[i] = make_uint4(0, 0, 0, 0);
  for (int64_t i = 4 * n4 + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nwords; i += stride) p[i] = 0u;
}

tdfe_status tdfe_zero(tdfe_ctx* c, void* p, size_t bytes) {
  if (bytes == 0) return TDFE_OK;
  if (bytes % 4 != 0 || (uintptr_t)p % 4 != 0) return tdfe_fail(c, TDFE_EINVAL, "zero fill: size or address not word aligned");
  const int64_t nw = (int64_t)(bytes / 4);
  const int64_t blocks = std::min<int64_t>((nw / 4 + 255) / 256 + 1, 4096);
  hipLaunchKernelGGL(zero_kernel, dim3((unsigned)blocks), dim3(256), 0, c->stream, (unsigned*)p, nw);
  TDFE_HIP(c, hipGetLastError());
  return TDFE_OK;
}

// copy of a few device words into the pinned readback area; the kernel's
// stores reach host memory before the stream completes, so one stream
// synchronisation makes all readbacks of a call visible
__global__ void readback_kernel(const unsigned* src, unsigned* dst, int nwords) {
  for (int i = threadIdx.x; i < nwords; i += blockDim.x) dst[i] = src[i];
  __threadfence_system();
}

tdfe_status tdfe_readback(tdfe_ctx* c, const void* dev_src, size_t bytes, size_t off, const void** host) {
  if (bytes % 4 != 0 || off % 8 != 0 || off + bytes > TDFE_READBACK_BYTES)
    return tdfe_fail(c, TDFE_EINVAL, "readback: %zu bytes at offset %zu", bytes, off);
  char* h = (char*)(c->poll + TDFE_READBACK_OFFSET_INTS) + off;
  void* d = nullptr;
  TDFE_HIP(c, hipHostGetDevicePointer(&d, (void*)h, 0));
  hipLaunchKernelGGL(readback_kernel, dim3(1), dim3(256), 0, c->stream, (const unsigned*)dev_src, (unsigned*)d,
                     (int)(bytes / 4));
  TDFE_HIP(c, hipGetLastError());
  *host = h;
  return TDFE_OK;
}

// Orbitals per Krylov chunk for a call on n_orb orbitals: at most the
// workspace's chunk_orb, chosen to minimise the operator's padded column work
// (a launch on `cols` real columns costs about the next power of two up to 16,
// then whole blocks of 16), with a small charge per chunk so that ties go to
// fewer chunks.  32 orbitals with room for 9 run as 4 x 8, not 9 + 9 + 9 + 5.
static int chunk_size_upto(int n_orb, int cap) {
  if (n_orb <= cap) return n_orb;
  auto padded = [](int cols) {
    if (cols > 16) return (cols + 15) / 16 * 16;
    int q = 1;
    while (q < cols) q <<= 1;
    return q;
  };
  int best = cap;
  double best_cost = 1e300;
  for (int sz = cap; sz >= 1; --sz) {
    const int n = (n_orb + sz - 1) / sz;
    const int last = n_orb - (n - 1) * sz;
    const double cost = (double)(n - 1) * padded(2 * sz) + padded(2 * last) + 4.0 * n;
    if (cost < best_cost) {
      best_cost = cost;
      best = sz;
    }
  }
  return best;
}

static int chunk_size(const tdfe_ctx* c, int n_orb) { return chunk_size_upto(n_orb, c->chunk_orb); }

// chunk and Krylov cap of the next exponential on n_orb orbitals: chunks wider
// than the basis memory holds at k_max once an earlier exponential has shown
// a Krylov dimension k_seen with a cap of at least 2 k_seen (and
// TDFE_SOFT_CAP_MIN); otherwise the chunk at k_max
static void soft_chunk(const tdfe_ctx* c, int n_orb, bool hooked, int* chunk, int* kcap) {
  *chunk = chunk_size(c, n_orb);
  *kcap = c->k_max;
  if (hooked || c->k_seen <= 0 || n_orb <= c->chunk_orb || c->wide_orb <= c->chunk_orb) return;
  const int need = std::max(2 * c->k_seen, TDFE_SOFT_CAP_MIN);
  int wmax = c->chunk_orb;
  for (int w = c->chunk_orb + 1; w <= std::min(n_orb, c->wide_orb); ++w)
    if (tdfe_soft_cap(c, w) >= need) wmax = w;
  if (wmax <= c->chunk_orb) return;
  *chunk = chunk_size_upto(n_orb, wmax);
  if (*chunk > c->chunk_orb) *kcap = tdfe_soft_cap(c, *chunk);
}

// y = exp(-i tau T) e_1 for one tridiagonal T given on the device (the small
// exponential of the Lanczos stop test, on its own): one wavefront, the same
// series and Bessel table as check_kernel
__global__ void __launch_bounds__(CHK_THREADS)
    tridiag_expm_kernel(const double* alpha, const double* beta, int k, double tau, double* y, double* jtab,
                        int* status) {
  __shared__ ChebLds L;
  __shared__ double sa[TDFE_KCAP], sb[TDFE_KCAP];
  const int t = threadIdx.x;
  for (int j = t; j < k; j += CHK_THREADS) {
    sa[j] = alpha[j];
    sb[j] = j < k - 1 ? beta[j] : 0.0;
  }
  __syncthreads();
  double amax = 0.0;
  int M;
  if (k <= CHK_THREADS) {
    double yr[1], yi[1];
    M = cheb_expm_e1_rows<1>(k, sa, sb, tau, jtab, yr, yi, &amax);
    if (M >= 0 && t < k) {
      y[2 * t] = yr[0];
      y[2 * t + 1] = yi[0];
    }
  } else {
    M = cheb_expm_e1(k, sa, sb, tau, L, jtab, &amax);
    if (M >= 0)
      for (int j = t; j < k; j += CHK_THREADS) {
        y[2 * j] = L.yr[j];
        y[2 * j + 1] = L.yi[j];
      }
  }
  if (t == 0) *status = M;
}

extern "C" tdfe_status tdfe_tridiag_expm_query(int k, size_t* bytes) {
  if (!bytes || k < 1 || k > TDFE_KCAP) return TDFE_EINVAL;
  *bytes = (size_t)(TDFE_JTAB_STRIDE + 8) * sizeof(double);
  return TDFE_OK;
}

extern "C" tdfe_status tdfe_tridiag_expm(const double* dev_alpha, const double* dev_beta, int k, double tau,
                                         double* dev_y, void* dev_scratch, size_t scratch_bytes, void* hip_stream,
                                         int* host_terms) {
  if (!dev_alpha || !dev_y || !dev_scratch || k < 1 || k > TDFE_KCAP || (k > 1 && !dev_beta) || !std::isfinite(tau))
    return TDFE_EINVAL;
  size_t need = 0;
  TDFE_TRY(tdfe_tridiag_expm_query(k, &need));
  if (scratch_bytes < need || (uintptr_t)dev_scratch % 256 != 0) return TDFE_ENOMEM;
  hipStream_t st = (hipStream_t)hip_stream;
  double* jtab = (double*)dev_scratch;
  int* dstatus = (int*)(jtab + TDFE_JTAB_STRIDE);
  hipLaunchKernelGGL(tridiag_expm_kernel, dim3(1), dim3(CHK_THREADS), 0, st, dev_alpha, dev_beta, k, tau, dev_y, jtab,
                     dstatus);
  if (hipGetLastError() != hipSuccess) return TDFE_EDEVICE;
  int M = 0;
  if (hipMemcpyAsync(&M, dstatus, sizeof(int), hipMemcpyDeviceToHost, st) != hipSuccess ||
      hipStreamSynchronize(st) != hipSuccess)
    return TDFE_EDEVICE;
  if (host_terms) *host_terms = M;
  if (M == TDFE_CHEB_NONFINITE) return TDFE_ENONFINITE;
  if (M < 0) return TDFE_EINVAL;
  return TDFE_OK;
}

extern "C" tdfe_status tdfe_krylov_chunk(const tdfe_ctx* c, int n_orb, int* chunk) {
  if (!c || !chunk || n_orb < 1 || n_orb > c->n_orb_max) return TDFE_EINVAL;
  *chunk = chunk_size(c, n_orb);
  return TDFE_OK;
}

extern "C" tdfe_status tdfe_krylov_soft_chunk(const tdfe_ctx* c, int n_orb, int* chunk, int* kcap) {
  if (!c || !chunk || !kcap || n_orb < 1 || n_orb > c->n_orb_max) return TDFE_EINVAL;
  soft_chunk(c, n_orb, false, chunk, kcap);
  return TDFE_OK;
}

// deferred-result slot `slot` (0 or 1) in the scalar block, past the Lanczos
// scalars of a full chunk and before the occupations
static double* result_slot(tdfe_ctx* c, int slot) {
  const size_t base = (size_t)(6 * c->k_max + 8) * c->n_orb_max;  // carve_scal takes 6 k_max + 8 per orbital
  return c->scal + base + (size_t)slot * (3 * c->n_orb_max + 1);
}

double* tdfe_lanczos_result_slot(tdfe_ctx* c, int slot) { return result_slot(c, slot); }

bool tdfe_lanczos_can_defer(const tdfe_ctx* c) { return (size_t)(3 * c->n_orb_max + 1) * 8 <= 4096; }

tdfe_status tdfe_lanczos_enqueue_results(tdfe_ctx* c, int slot, const void** host) {
  return tdfe_readback(c, result_slot(c, slot), (size_t)(3 * c->n_orb_max + 1) * 8, 4096 + (size_t)slot * 4096,
                       host);
}

tdfe_status tdfe_lanczos_results(tdfe_ctx* c, const void* host, int n_orb, double tol, int* kmax_out,
                                 int* ksum_out, double* errmax_out) {
  const volatile double* h = (const volatile double*)host;
  const int nm = c->n_orb_max;
  int kmax = 0, ksum = 0, bad = 0, nonfinite = 0;
  double emax = 0.0;
  for (int o = 0; o < n_orb; ++o) {
    const int k = (int)h[o];
    kmax = std::max(kmax, k);
    ksum += k;
    emax = std::max(emax, (double)h[2 * nm + o]);
    if ((int)h[nm + o] == 2) bad = 1;
    if ((int)h[nm + o] == 4) nonfinite = 1;
  }
  if (kmax_out) *kmax_out = kmax;
  if (ksum_out) *ksum_out = ksum;
  if (errmax_out) *errmax_out = emax;
  if (!bad && !nonfinite) c->k_seen = kmax;
  if (nonfinite) return tdfe_fail(c, TDFE_ENONFINITE, "Lanczos: non-finite norm or recurrence coefficient");
  if (h[3 * nm] != 0.0) return tdfe_fail(c, TDFE_EINVAL, "small exponential: |tau| ||T|| too large for the Chebyshev table");
  if (bad) return tdfe_fail(c, TDFE_ENOCONV, "Lanczos reached k_max=%d without eps <= %g", c->k_max, tol);
  return TDFE_OK;
}

tdfe_status tdfe_lanczos_run(tdfe_ctx* c, const double* vw, const void* in, void* out, int n_orb, double tau,
                             double tol, int* k_out, double* err_out, int* kmax_out, int* ksum_out,
                             double* errmax_out, LanczosHook* hook, int defer) {
  const int ld = 2 * n_orb;
  double* slot = nullptr;
  if (defer >= 0) {
    if (defer > 1 || hook || k_out || err_out || kmax_out || ksum_out || errmax_out || !tdfe_lanczos_can_defer(c))
      return tdfe_fail(c, TDFE_EINVAL, "lanczos: deferred results need slot 0/1 and no host outputs");
    slot = result_slot(c, defer);
    TDFE_TRY(tdfe_zero(c, slot + 3 * c->n_orb_max, sizeof(double)));
  }
  std::vector<int> ks(n_orb), st(n_orb);
  std::vector<double> es(n_orb);
  const void* v = !tdfe_fp32(c) ? (const void*)vw : (const void*)c->vw32;
  // when the input is also the output, every chunk must read the input before
  // any chunk writes: the combination of a chunk only writes that chunk's
  // columns, and copy_in of a chunk only reads them, so chunk order is safe
  // (a soft-capped chunk that restarts has not written its columns either).
  auto run = [&](int o0, int Nc, int kc, bool* restart) {
    if (!tdfe_fp32(c))
      return run_chunk<double>(c, v, (const double*)in, (double*)out, ld, o0, Nc, tau, tol, ks.data() + o0,
                               es.data() + o0, st.data() + o0, hook, slot, kc, restart);
    return run_chunk<float>(c, v, (const double*)in, (double*)out, ld, o0, Nc, tau, tol, ks.data() + o0,
                            es.data() + o0, st.data() + o0, hook, slot, kc, restart);
  };
  int csz = 0, kcap = 0;
  soft_chunk(c, n_orb, hook != nullptr, &csz, &kcap);
  for (int o0 = 0; o0 < n_orb; o0 += csz) {
    const int Nc = std::min(csz, n_orb - o0);
    bool restart = false;
    TDFE_TRY(run(o0, Nc, Nc > c->chunk_orb ? kcap : c->k_max, &restart));
    if (!restart) continue;
    // an orbital needs more than the soft cap: these orbitals again at k_max
    // in chunks the basis holds, and no more soft caps below that dimension
    c->k_seen = std::max(c->k_seen, kcap + 1);
    const int sub = chunk_size(c, Nc);
    for (int q0 = o0; q0 < o0 + Nc; q0 += sub) {
      bool again = false;
      TDFE_TRY(run(q0, std::min(sub, o0 + Nc - q0), c->k_max, &again));
    }
  }
  if (slot) {
    // the first exponential of a context: read its Krylov dimensions back
    // now (one wait on the device, once), so that the next exponential -- the
    // same step's corrector -- may already run soft-capped chunks
    if (c->k_seen == 0 && c->wide_orb > c->chunk_orb && n_orb > c->chunk_orb) {
      const void* h = nullptr;
      TDFE_TRY(tdfe_lanczos_enqueue_results(c, defer, &h));
      TDFE_HIP(c, hipStreamSynchronize(c->stream));
      const volatile double* hv = (const volatile double*)h;
      const int nm = c->n_orb_max;
      int kmax = 0, ok = 1;
      for (int o = 0; o < n_orb; ++o) {
        kmax = std::max(kmax, (int)hv[o]);
        if ((int)hv[nm + o] != 1) ok = 0;  // only a set that converged informs the cap
      }
      if (ok) c->k_seen = kmax;
    }
    return TDFE_OK;
  }
  int kmax = 0, ksum = 0, bad = 0, nonfinite = 0;
  double emax = 0.0;
  for (int o = 0; o < n_orb; ++o) {
    kmax = std::max(kmax, ks[o]);
    ksum += ks[o];
    emax = std::max(emax, es[o]);
    if (st[o] == 2) bad = 1;
    if (st[o] == 4) nonfinite = 1;
    if (k_out) k_out[o] = ks[o];
    if (err_out) err_out[o] = es[o];
  }
  if (kmax_out) *kmax_out = kmax;
  if (ksum_out) *ksum_out = ksum;
  if (errmax_out) *errmax_out = emax;
  if (!bad && !nonfinite) c->k_seen = kmax;
  if (nonfinite) return tdfe_fail(c, TDFE_ENONFINITE, "Lanczos: non-finite norm or recurrence coefficient");
  if (bad) return tdfe_fail(c, TDFE_ENOCONV, "Lanczos reached k_max=%d without eps <= %g", c->k_max, tol);
  return TDFE_OK;
}

extern "C" {

static tdfe_status apply_checked(tdfe_ctx* c, const void* dev_psibar, void* dev_out, int n_orb, bool zero) {
  if (!c || !dev_psibar || !dev_out) return TDFE_EINVAL;
  if (n_orb < 1 || n_orb > c->n_orb_max) return tdfe_fail(c, TDFE_EINVAL, "apply_H: n_orb out of range");
  if (dev_psibar == dev_out) return tdfe_fail(c, TDFE_EINVAL, "apply_H: output aliases input");
  if (!c->bound) return tdfe_fail(c, TDFE_ESTATE, "apply_H before bind_workspace");
  if (!c->have_potential) return tdfe_fail(c, TDFE_ESTATE, "apply_H before set_potential");
  const int cols = 2 * n_orb;
  ApplyArgs a{};
  a.x = dev_psibar;
  a.y = dev_out;
  a.ld = cols;
  a.cols = cols;
  a.kin = 0.5;
  a.vw = c->vw;
  a.lowdin = true;
  a.nonlocal = true;
  a.fp32 = false;
  a.overwrite = zero && tdfe_can_overwrite(c, a);
  if (zero && !a.overwrite) TDFE_TRY(tdfe_zero(c, dev_out, (size_t)c->n_dof * cols * sizeof(double)));
  return tdfe_launch_apply(c, a);
}

tdfe_status tdfe_apply_H(tdfe_ctx* c, const void* dev_psibar, void* dev_out, int n_orb) {
  return apply_checked(c, dev_psibar, dev_out, n_orb, true);
}

tdfe_status tdfe_apply_H_add(tdfe_ctx* c, const void* dev_psibar, void* dev_out, int n_orb) {
  return apply_checked(c, dev_psibar, dev_out, n_orb, false);
}

tdfe_status tdfe_apply_H_add_f32(tdfe_ctx* c, const void* dev_psibar, void* dev_out, int n_orb) {
  if (!c || !dev_psibar || !dev_out) return TDFE_EINVAL;
  if (n_orb < 1 || n_orb > c->n_orb_max) return tdfe_fail(c, TDFE_EINVAL, "apply_H_f32: n_orb out of range");
  if (dev_psibar == dev_out) return tdfe_fail(c, TDFE_EINVAL, "apply_H_f32: output aliases input");
  if (!tdfe_fp32(c)) return tdfe_fail(c, TDFE_EINVAL, "apply_H_f32 needs a mixed-precision context");
  if (!c->bound) return tdfe_fail(c, TDFE_ESTATE, "apply_H_f32 before bind_workspace");
  if (!c->have_potential) return tdfe_fail(c, TDFE_ESTATE, "apply_H_f32 before set_potential");
  ApplyArgs a{};
  a.x = dev_psibar;
  a.y = dev_out;
  a.ld = 2 * n_orb;
  a.cols = 2 * n_orb;
  a.kin = 0.5;
  a.vw32 = c->vw32;
  a.lowdin = true;
  a.nonlocal = true;
  a.fp32 = true;
  return tdfe_launch_apply(c, a);
}

tdfe_status tdfe_lanczos_expm(tdfe_ctx* c, void* dev_psibar, int n_orb, double tau, double tol, int* host_k,
                              double* host_err) {
  if (!c || !dev_psibar) return TDFE_EINVAL;
  if (n_orb < 1 || n_orb > c->n_orb_max) return tdfe_fail(c, TDFE_EINVAL, "lanczos_expm: n_orb out of range");
  if (!(tol > 0.0) || !std::isfinite(tau)) return tdfe_fail(c, TDFE_EINVAL, "lanczos_expm: bad tau/tol");
  if (!c->bound) return tdfe_fail(c, TDFE_ESTATE, "lanczos_expm before bind_workspace");
  if (!c->have_potential) return tdfe_fail(c, TDFE_ESTATE, "lanczos_expm before set_potential");
  return tdfe_lanczos_run(c, c->vw, dev_psibar, dev_psibar, n_orb, tau, tol, host_k, host_err, nullptr, nullptr,
                          nullptr);
}

}  // extern "C"
