// Chebyshev evaluation of y = exp(-i s T) e_1 for a real symmetric tridiagonal
// T (k x k; diagonal sa[0..k), off-diagonal sb[0..k-1)), on one wavefront of
// TDFE_CHEB_THREADS lanes: Gershgorin interval [c - r, c + r], Jacobi-Anger
// coefficients 2 (-i sgn(s))^m J_m(|s| r), Bessel values by Miller's backward
// recurrence normalised with J_0 + 2 sum J_2m = 1, and the three-term
// recurrence v_{m+1} = 2 X v_m - v_{m-1}, X = (T - c)/r, v_0 = e_1, rows across
// lanes.  Nothing here synchronises with another wavefront, except that
// cheb_expm_e1 ends on a barrier of its one-wavefront workgroup.
//
// What bounds it is one chain of dependent FP64 operations (Miller's steps,
// then the terms), so it is kept short: every lane runs Miller's recurrence
// on the same values and keeps its own entry of each 64, so that up to 128
// values never leave the registers, a longer table is written and read back
// by the same lanes without a fence, and a term is three dependent FMAs on
// coefficients scaled beforehand.  With one lane running the recurrence into
// global memory and terms of six dependent operations a step of ten short
// iterations on a small box took 404 us, with this 336 us.
#pragma once
#include <hip/hip_runtime.h>

#define TDFE_CHEB_THREADS 64
// largest Bessel table: |s| r up to about 6.5e4 (the all-electron-like
// workload's smallest cells reach a few 1e4 at its dt)
#define TDFE_MAX_BESSEL 65536
#define TDFE_KCAP 1024
// per-orbital Bessel table in global memory (every evaluation path): the
// table plus two register chunks of padding for the look-ahead load
#define TDFE_JTAB_STRIDE (TDFE_MAX_BESSEL + 2 + 2 * TDFE_CHEB_THREADS)

struct ChebLds {
  double yr[TDFE_KCAP], yi[TDFE_KCAP];
};

// whole-wavefront neighbour exchange by DPP row shifts (the value of lane t-1,
// resp. t+1; 0 at the ends): no LDS traffic
__device__ __forceinline__ double lane_prev(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x138, 0xf, 0xf, false);  // wave_shr:1
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x138, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double lane_next(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x130, 0xf, 0xf, false);  // wave_shl:1
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x130, 0xf, 0xf, false);
  return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double lane_read(double v, int lane) {
  const int lo = __builtin_amdgcn_readlane(__double2loint(v), lane);
  const int hi = __builtin_amdgcn_readlane(__double2hiint(v), lane);
  return __hiloint2double(hi, lo);
}

// largest value over the wavefront by DPP exchanges (fmax: a NaN is passed over)
template <int CTRL>
__device__ __forceinline__ double lane_fmax(double v) {
  const int lo = __double2loint(v), hi = __double2hiint(v);
  return fmax(v, __hiloint2double(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false),
                                  __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false)));
}
__device__ __forceinline__ double wave_fmax(double v) {
  v = lane_fmax<0xB1>(v);   // quad_perm [1,0,3,2]
  v = lane_fmax<0x4E>(v);   // quad_perm [2,3,0,1]
  v = lane_fmax<0x141>(v);  // row_half_mirror
  v = lane_fmax<0x140>(v);  // row_mirror: each row of 16 holds its largest
  v = lane_fmax<0x142>(v);  // row_bcast:15
  v = lane_fmax<0x143>(v);  // row_bcast:31: the last row holds the largest of all
  return lane_read(v, TDFE_CHEB_THREADS - 1);
}

// Bessel values J_0..J_M(z), z the same on every lane: entry 64 q + t of the
// table in lane t.  The first 128 entries are returned in j0 and j1; a table
// that starts beyond them is written to Jg as well (whole chunks of 64, every
// lane its own entries, which only that lane reads back) and sets *big.
// Returns M, -1 if z exceeds the table, or TDFE_CHEB_NONFINITE if z is not
// finite (an Inf in T).  z is bounded before it is converted to an integer,
// so no term count can overflow.  The values are left unnormalised; *inv
// receives 1 / (J_0 + 2 sum J_2m).  Entries M+1.. of the last chunk are small
// or zero, never undefined.
//
// The recurrence starts at ms: a start with J_{ms+1} = 0 leaves a relative
// error at M of about exp(-2 (ms - M) acosh(M / z)); with acosh(1 + x) about
// sqrt(2 x) the start below keeps that under exp(-20), at an entry that is
// itself below 1e-15 of the sum.
#define TDFE_CHEB_NONFINITE (-2)
__device__ __forceinline__ int cheb_bessel(double z, double* Jg, double& j0, double& j1, bool& big, double* inv) {
  const int t = threadIdx.x;
  *inv = 1.0;
  big = false;
  j0 = t == 0 ? 1.0 : 0.0;
  j1 = 0.0;
  if (isnan(z) || isinf(z)) return TDFE_CHEB_NONFINITE;
  if (z > 2.0 * TDFE_MAX_BESSEL) return -1;
  if (!(z > 1e-300)) return 0;
  const int M = __builtin_amdgcn_readfirstlane((int)ceil(z + 10.0 * cbrt(z) + 20.0));
  // the table's limit, with the room of the widest start
  if (((M + 21 + (int)(2.0 * sqrt((double)M))) | 1) > TDFE_MAX_BESSEL) return -1;
  if (z < 1e-20) {  // J_1 = z / 2, the rest below 1e-41
    j0 = t == 1 ? 0.5 * z : j0;
    return M;
  }
  const int ms = __builtin_amdgcn_readfirstlane(M + 7 + (int)(7.1 * sqrt(z / (M - z)))) | 3;
  big = ms >= 2 * TDFE_CHEB_THREADS;
  const double tz = 2.0 / z;
  double jp = 0.0, jc = 1e-300, even = 0.0;  // J_{m+1}, J_m, sum of J_2m
  int m = ms;
  for (int q = ms / TDFE_CHEB_THREADS; q >= 0; --q) {
    double cur = 0.0;
    const int m0 = q * TDFE_CHEB_THREADS;
    for (; m > m0; m -= 4) {  // m = 3 mod 4
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        cur = t == m - u - m0 ? jc : cur;
        if (u & 1) even += jc;
        const double jn = ((m - u) * tz) * jc - jp;
        jp = jc;
        jc = jn;
      }
      // a step grows by at most 2 m / z < 1e22, so four stay in range
      if (fabs(jc) > 1e200) {
        jp *= 1e-200;
        jc *= 1e-200;
        even *= 1e-200;
        cur *= 1e-200;
        j1 *= 1e-200;
        for (int c = q + 1; big && c <= ms / TDFE_CHEB_THREADS; ++c) Jg[c * TDFE_CHEB_THREADS + t] *= 1e-200;
      }
    }
    if (big) Jg[m0 + t] = cur;
    j1 = q == 1 ? cur : j1;
    j0 = cur;  // q = 0 comes last
  }
  *inv = 1.0 / (2.0 * even - jp);  // jp = J_0
  return M;
}

// y = exp(-i s T) e_1 for k <= R TDFE_CHEB_THREADS, called by one full
// wavefront (lanes 0..63 of the workgroup, all active): R consecutive rows per
// lane (lane t holds rows R t .. R t + R - 1; a, bl, br: diagonal, left and
// right off-diagonal, zero past k), the Chebyshev vectors in registers, the
// neighbours across lanes by DPP shifts, so that a term costs no LDS round
// trip or barrier.  Every lane keeps 64 consecutive coefficients in one
// register (the next 64 loaded one chunk ahead) and each term takes its own by
// a lane read.  Jg: TDFE_JTAB_STRIDE doubles of the calling wavefront's own.
// Row R t + r of y is returned in yr[r], yi[r] (zero past k); the result is M,
// -1 if |s| r exceeds the table, or TDFE_CHEB_NONFINITE.
template <int R>
__device__ __forceinline__ int cheb_series(int k, const double (&a)[R], const double (&bl)[R], const double (&br)[R],
                                  double s, double* Jg, double (&yr)[R], double (&yi)[R], double* amax) {
  const int t = threadIdx.x;
  double nlo = -1e300, hi = -1e300, am = 0.0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (R * t + r < k) {
      nlo = fmax(nlo, fabs(bl[r]) + fabs(br[r]) - a[r]);
      hi = fmax(hi, a[r] + fabs(bl[r]) + fabs(br[r]));
      am = fmax(am, fabs(a[r]));
    }
    yr[r] = 0.0;
    yi[r] = 0.0;
  }
  const double lo = -wave_fmax(nlo);
  hi = wave_fmax(hi);
  *amax = wave_fmax(am);
  const double cc = 0.5 * (lo + hi), rr = 0.5 * (hi - lo);
  const double z = fabs(s) * rr;
  double jr, jnx, jn;
  bool big;
  const int M = cheb_bessel(z, Jg, jr, jnx, big, &jn);
  if (M < 0) return M;
  const double inv2 = rr > 0.0 ? 2.0 / rr : 0.0;
  double A[R], L[R], U[R], vp[R], vc[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    A[r] = (R * t + r < k) ? (a[r] - cc) * inv2 : 0.0;
    L[r] = bl[r] * inv2;
    U[r] = br[r] * inv2;
    vp[r] = (t == 0 && r == 0) ? 1.0 : 0.0;
  }
  // v <- 2 X w - v
  auto step = [&](double(&v)[R], const double(&w)[R]) {
    const double left = lane_prev(w[R - 1]), right = lane_next(w[0]);
#pragma unroll
    for (int r = 0; r < R; ++r)
      v[r] = U[r] * (r < R - 1 ? w[r + 1] : right) + (L[r] * (r > 0 ? w[r - 1] : left) + (A[r] * w[r] - v[r]));
  };
  // 2 jn (-i sgn)^m by lane (m = t mod 4): 1, -i sgn, -1, +i sgn
  const double sgn = s >= 0.0 ? 1.0 : -1.0;
  const double cf = 2.0 * jn * ((t & 1) ? ((t & 2) ? sgn : -sgn) : ((t & 2) ? -1.0 : 1.0));
  double cj = cf * jr;
  yr[0] = 0.5 * lane_read(cj, 0) * vp[0];
  if (M >= 1) {
#pragma unroll
    for (int r = 0; r < R; ++r) vc[r] = 0.0;
    step(vc, vp);
    const double c1 = lane_read(cj, 1);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      vc[r] *= 0.5;
      yi[r] = c1 * vc[r];
    }
    // terms mm and mm + 1 (the one past M, if M is even, is in the table too)
    for (int mm = 2; mm <= M; mm += 2) {
      if ((mm & (TDFE_CHEB_THREADS - 1)) == 0) {
        cj = cf * jnx;
        if (big) jnx = Jg[mm + TDFE_CHEB_THREADS + t];  // < TDFE_JTAB_STRIDE since mm <= M < TDFE_MAX_BESSEL
      }
      const double ce = lane_read(cj, mm & (TDFE_CHEB_THREADS - 1));
      const double co = lane_read(cj, (mm + 1) & (TDFE_CHEB_THREADS - 1));
      step(vp, vc);
#pragma unroll
      for (int r = 0; r < R; ++r) yr[r] += ce * vp[r];
      step(vc, vp);
#pragma unroll
      for (int r = 0; r < R; ++r) yi[r] += co * vc[r];
    }
  }
  const double pr = cos(s * cc), pim = -sin(s * cc);
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const double a0 = yr[r], b0 = yi[r];
    yr[r] = a0 * pr - b0 * pim;
    yi[r] = a0 * pim + b0 * pr;
  }
  return M;
}

// the same with T read from sa / sb (any memory the wavefront can read)
template <int R>
__device__ inline int cheb_expm_e1_rows(int k, const double* sa, const double* sb, double s, double* Jg,
                                        double (&yr)[R], double (&yi)[R], double* amax) {
  const int t = threadIdx.x;
  double a[R], bl[R], br[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j = R * t + r;
    const bool row = j < k;
    a[r] = row ? sa[j] : 0.0;
    bl[r] = (row && j > 0) ? sb[j - 1] : 0.0;
    br[r] = (row && j < k - 1) ? sb[j] : 0.0;
  }
  return cheb_series<R>(k, a, bl, br, s, Jg, yr, yi, amax);
}

template <int R>
__device__ inline int cheb_rows_lds(int k, const double* sa, const double* sb, double s, ChebLds& L, double* Jg,
                                    double* amax) {
  double yr[R], yi[R];
  const int M = cheb_expm_e1_rows<R>(k, sa, sb, s, Jg, yr, yi, amax);
  const int t = threadIdx.x;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int j = R * t + r;
    if (j < k) {
      L.yr[j] = yr[r];
      L.yi[j] = yi[r];
    }
  }
  __syncthreads();
  return M;
}

// y = exp(-i s T) e_1 for TDFE_CHEB_THREADS < k <= TDFE_KCAP on one
// wavefront, left in L.yr / L.yi (rows per lane by k: 2, 3, 4, 8 or 16)
__device__ inline int cheb_expm_e1(int k, const double* sa, const double* sb, double s, ChebLds& L, double* Jg,
                                   double* amax) {
  if (k <= 2 * TDFE_CHEB_THREADS) return cheb_rows_lds<2>(k, sa, sb, s, L, Jg, amax);
  if (k <= 3 * TDFE_CHEB_THREADS) return cheb_rows_lds<3>(k, sa, sb, s, L, Jg, amax);
  if (k <= 4 * TDFE_CHEB_THREADS) return cheb_rows_lds<4>(k, sa, sb, s, L, Jg, amax);
  if (k <= 8 * TDFE_CHEB_THREADS) return cheb_rows_lds<8>(k, sa, sb, s, L, Jg, amax);
  return cheb_rows_lds<16>(k, sa, sb, s, L, Jg, amax);
}
