// Pieces shared by the eigensolve kernels (paper Sec. II-A, Eq. 4): the
// Jacobi rotation of a pair, the round-robin pairing, fixed-order dot
// products and the per-iteration control step.
#pragma once

#include "common.h"

namespace rpca {
namespace eigk {

constexpr double kTiny2 = 1.0e-300;
constexpr int kMaxSweeps = 40;

// Simultaneous rotation steps (see eig_core.h).
constexpr int kMaxSteps = 12;          // per launch; then sweeps only
constexpr int kMaxPasses = 100;        // steps and sweeps together
constexpr float kOrthMax = 0.25f;      // largest |V^T V - I| entry that a step starts from
constexpr float kRowSumMax = 0.9f;     // largest row sum of |K| (a bound of its norm) of a step
constexpr double kTangentMax = 0.5;    // tangents are clipped here
constexpr float kColdTangent = 0.25f;  // first launch: steps only once every tangent is below
constexpr float kWideFourth = 0.02f;   // wide solves: above this tangent, U to fourth order

// Bound on the second-order error of an entry of P: for FP32 solves half the
// rounding of P's own entries (over the iterations of 20-frame windows the error
// itself stays below 2e-9, that of the diagonal Z this replaces, whose
// off-diagonals were left out up to 1e-8 sigma_i sigma_j, below 5e-9), for FP64
// solves at the rounding of the products.
template <typename T>
struct PTarget;
template <>
struct PTarget<double> {
  static constexpr float value = 2.0e-15f;
};
template <>
struct PTarget<float> {
  static constexpr float value = 3.0e-8f;
};
// Entries of |V^T V - I| below which V counts as orthogonal.
template <typename T>
struct OrthGoal;
template <>
struct OrthGoal<double> {
  static constexpr float skip = 2.0e-15f;
};
template <>
struct OrthGoal<float> {
  static constexpr float skip = 1.0e-11f;
};

// Column j of packed upper index idx = j (j + 1) / 2 + i, i <= j (idx < 2^22:
// the float square root is exact enough to be off by at most one).
__device__ inline int packed_col(int idx) {
  int j = static_cast<int>(fmaf(__builtin_sqrtf(fmaf(8.0f, static_cast<float>(idx), 1.0f)), 0.5f, -0.5f));
  if (j * (j + 1) / 2 > idx) --j;
  else if ((j + 1) * (j + 2) / 2 <= idx) ++j;
  return j;
}

template <typename T>
struct RotEps;
template <>
struct RotEps<double> {
  static constexpr double eps2 = 1.0e-30;
};
template <>
struct RotEps<float> {
  static constexpr double eps2 = 1.0e-16;
};

template <typename T>
__device__ inline bool off_diag_large(double gij, double gii, double gjj) {
  const double a2 = gij * gij;
  return a2 > kTiny2 && a2 > RotEps<T>::eps2 * fabs(gii * gjj);
}

// Round-robin pairing of round r (0 <= r < N2-1) over N2 (even) indices:
// pair 0 is (N2-1, r), pair k >= 1 is ((r+k) mod M, (r-k) mod M), M = N2-1.
__device__ inline void pair_indices(int r, int k, int N2, int& p, int& q) {
  const int M = N2 - 1;
  int a, b;
  if (k == 0) {
    a = N2 - 1;
    b = r;
  } else {
    a = r + k;
    if (a >= M) a -= M;
    b = r - k;
    if (b < 0) b += M;
  }
  p = a < b ? a : b;
  q = a < b ? b : a;
}

// Per-round column table of J, written by the threads that compute the
// round's rotations: for index i, column i of J is a_i e_u + b_i e_v with
// (u, v) the pair containing i, packed as u | v << 8 | rotated << 16, (a_i,
// b_i) stored together (one 16-byte read), and dg_i the exact shift of the
// diagonal entry g_ii (-t g_pq for p, +t g_pq for q).  An index paired with
// the padding index gets the identity column.
__device__ inline void set_pair_columns(int p, int q, int n, double c, double s, double dt,
                                        int* cu, double2* cab, double* cd) {
  if (q >= n) {
    cu[p] = p | (p << 8);
    cab[p] = make_double2(1.0, 0.0);
    cd[p] = 0.0;
    return;
  }
  const int packed = p | (q << 8) | (s != 0.0 ? (1 << 16) : 0);
  cu[p] = packed;
  cab[p] = make_double2(c, -s);
  cd[p] = -dt;
  cu[q] = packed;
  cab[q] = make_double2(s, c);
  cd[q] = dt;
}

// Entry (i, j) of J^T G J from the column table (G with leading dimension LD).
template <int LD>
__device__ inline double rotated_entry(int i, int j, const double* G, const int* cu,
                                       const double2* cab, const double* cd) {
  const int pi = cu[i], pj = cu[j];
  const int ui = pi & 0xff, vi = (pi >> 8) & 0xff;
  const int uj = pj & 0xff, vj = (pj >> 8) & 0xff;
  const double2 abi = cab[i], abj = cab[j];
  const double ai = abi.x, bi = abi.y, aj = abj.x, bj = abj.y;
  double gen = ai * aj * G[ui * LD + uj];
  gen = fma(ai * bj, G[ui * LD + vj], gen);
  gen = fma(bi * aj, G[vi * LD + uj], gen);
  gen = fma(bi * bj, G[vi * LD + vj], gen);
  const double diag = G[i * LD + i] + cd[i];
  const bool same_rotated_pair = (pi >> 16) != 0 && (pi & 0xffff) == (pj & 0xffff);
  return i == j ? diag : (same_rotated_pair ? 0.0 : gen);
}

// 1/x and 1/sqrt(x) for positive normal x: the hardware estimate refined by
// two Newton steps (each doubles the number of correct bits).
__device__ inline double rcp_pos(double x) {
  double r = __builtin_amdgcn_rcp(x);
  r = r * fma(-x, r, 2.0);
  r = r * fma(-x, r, 2.0);
  return r;
}
__device__ inline double rsqrt_pos(double x) {
  double y = __builtin_amdgcn_rsq(x);
  const double hx = 0.5 * x;
  y = y * fma(-hx * y, y, 1.5);
  y = y * fma(-hx * y, y, 1.5);
  return y;
}

// Rotation of one pair from the entries of G.
template <typename T>
__device__ inline void make_rotation(double gpp, double gqq, double gpq, double& c, double& s,
                                     double& dt) {
  if (off_diag_large<T>(gpq, gpp, gqq)) {
    const double d = gqq - gpp;
    const double h2 = fma(d, d, 4.0 * gpq * gpq);   // > 0 since gpq != 0
    double t = 2.0 * gpq * rcp_pos(fma(h2, rsqrt_pos(h2), fabs(d)));
    if (d < 0.0) t = -t;
    c = rsqrt_pos(fma(t, t, 1.0));
    s = t * c;
    dt = t * gpq;
  } else {
    c = 1.0;
    s = 0.0;
    dt = 0.0;
  }
}

// What one pair (i, j) of G~ (diagonal entries di, dj, off-diagonal e) gives:
// the first-order entry z = w[di, dj] e of the thresholded function, the two
// factors mz, kappa of its error bound, the clipped tangent t of the rotation,
// and whether the sweeps would rotate the pair.
//
// The second-order terms of P are products e_ij e_jk of two pairs with a second
// divided difference of w, which is a difference of two first ones (slopes of w,
// w'(d) where two indices agree) over a gap.  mz is |e| times the largest slope
// that the pair can bring: w[di, dj], w' = tau / (2 d^1.5) of a kept value, and
// w' = 1/(2 tau^2) at the threshold where a value may lie on either side of it
// (w[di, dj] alone is nearly zero for a value just above the threshold, and a
// window with one column there was taken for converged, with P = 0).  kappa is
// |e| over the gap: |di - dj|; for two kept values, where w is smooth, min(di, dj)
// when that is larger; for two dropped values, whose own term vanishes but which
// pass on what a kept value couples to one of them, the distance of the larger
// from the threshold.  The last two hold only while the pair's values stay on
// their side of the threshold tau^2 whatever the off-diagonals do: by Gershgorin
// when n |e| is at most their distance from it (if that holds for every pair of a
// row, the row's radius is within the distance).  Pairs far below the threshold
// that are safe in this sense are not rotated at all: they are the rounding noise
// of rank-deficient windows.
struct PairTerms {
  double z, t;
  float mz, kappa;
  int rotate;
};
// ri, rj: 1/si and 1/sj (0 for a value of 0).
template <typename T>
__device__ inline PairTerms pair_terms(double e, double di, double dj, double si, double sj, double ri,
                                       double rj, double wi, double wj, double tau, int n) {
  PairTerms o;
  const double g = dj - di, ag = fabs(g), ae = fabs(e), tau2 = tau * tau;
  const bool ki = si > tau, kj = sj > tau;
  const bool safe = n * ae <= fmin(fabs(di - tau2), fabs(dj - tau2));
  const double smax = fmax(si, sj);
  o.rotate = off_diag_large<T>(e, di, dj) ? 1 : 0;
  o.z = 0.0;
  o.t = 0.0;
  o.mz = 0.0f;
  o.kappa = 0.0f;
  if (ae == 0.0) return o;
  // (the bound's factors from the hardware's estimates of the reciprocals)
  double q, mz = 0.0;  // 1 / gap, |e| times the largest slope
  if (ki != kj) {
    q = rcp_pos(ag);  // one above, one not: g != 0
    const double rk = ki ? ri : rj;
    o.z = e * ((ki ? wi : wj) * q);
    mz = 0.5 * (tau * rk) * (ae * rk * rk);
  } else if (ki) {
    const double rm = fmax(ri, rj);
    o.z = e * (ri * rj) * (tau * rcp_pos(si + sj));
    mz = 0.5 * (tau * rm) * (ae * rm * rm);
    q = __builtin_amdgcn_rcp(safe ? fmax(ag, fmin(di, dj)) : ag);
  } else {
    q = __builtin_amdgcn_rcp(safe ? tau2 - fmax(di, dj) : ag);
  }
  if (!safe) mz = 0.5 * ae * __builtin_amdgcn_rcp(tau2);  // no slope is larger
  o.mz = fmaxf(fabsf(static_cast<float>(o.z)), static_cast<float>(mz));
  o.kappa = static_cast<float>(ae * q);  // (infinite for equal values that are not safe)
  if (ki || kj || !safe || smax > 0.125 * tau) {
    const double h2 = fma(g, g, 4.0 * e * e);
    if (h2 > kTiny2) {
      const double t = 2.0 * e * rcp_pos(fma(h2, rsqrt_pos(h2), ag));
      o.t = fmin(fmax(g < 0.0 ? -t : t, -kTangentMax), kTangentMax);
    }
  }
  return o;
}

// Maximum of v >= 0 over the wave (DPP within rows of 16 lanes, then the four
// rows), added to *cell by one lane: float bits of non-negative values order
// as integers, and a maximum does not depend on the order of its terms.  NaN
// orders above every number.  Every lane of the wave must be active.
template <int CTRL>
__device__ inline unsigned dpp_max(unsigned v) {
  const unsigned o = static_cast<unsigned>(
      __builtin_amdgcn_update_dpp(0, static_cast<int>(v), CTRL, 0xF, 0xF, false));
  return v > o ? v : o;
}
__device__ inline void wave_max_to(float x, unsigned* cell) {
  unsigned v = __float_as_uint(x);
  v = dpp_max<0xB1>(v);   // lanes [1,0,3,2] of each quad
  v = dpp_max<0x4E>(v);   // lanes [2,3,0,1]
  v = dpp_max<0x141>(v);  // mirror of each half row
  v = dpp_max<0x140>(v);  // mirror of each row
  unsigned a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 16);
  const unsigned c = __builtin_amdgcn_readlane(v, 32), e = __builtin_amdgcn_readlane(v, 48);
  a = a > b ? a : b;
  b = c > e ? c : e;
  a = a > b ? a : b;
  if ((threadIdx.x & 63) == 0 && a != 0u) atomicMax(cell, a);
}

// 1/sqrt(d), or 0 for d <= 0 (the rounding of a zero eigenvalue); NaN for infinity.
__device__ inline double rsqrt_or_zero(double d) { return d <= kTiny2 ? 0.0 : rsqrt_pos(d); }

// View of a wide solve's workspace (see common.h).  cls is the class of the
// Jacobi kernel, whose scratch comes first.
struct WideEig {
  WideCtl* ctl;
  double *G, *W, *S, *K, *T, *U, *C, *Z;
  double* VT0;  // V^T of the even steps, then of the odd ones
  double* V0;   // the solve's V buffer
  double* V12;  // the two others
  size_t q;     // nb x nb
  __device__ explicit WideEig(const SolveDesc& d) {
    const int c = d.n <= kEigWideMaxN ? kEigWideMaxN : kEigHugeMaxN;
    double* p = d.escratch + static_cast<size_t>(c) * c;
    ctl = reinterpret_cast<WideCtl*>(p);
    p += kWideCtlDoubles;
    q = static_cast<size_t>(d.nb) * d.nb;
    G = p;
    W = p + q;
    S = p + 2 * q;
    K = p + 3 * q;
    T = p + 4 * q;
    U = p + 5 * q;
    C = p + 6 * q;
    Z = p + 7 * q;
    V12 = p + 8 * q;
    VT0 = p + 10 * q;
    V0 = d.V;
  }
  // V after s steps from buffer v0: the previous iteration's V stays where it
  // is (the Jacobi kernel starts from it if the steps fail), the steps
  // alternate between the other two buffers.
  __device__ static int vsel(int v0, int s) { return s == 0 ? v0 : (v0 + (s & 1 ? 1 : 2)) % 3; }
  __device__ double* vt(int b) const { return VT0 + b * q; }
  __device__ double* v(int b) const { return b == 0 ? V0 : V12 + (b - 1) * q; }
};

// Dot product over the zero-padded length NMAX with four independent
// partial sums (fixed trip count, so every load can be in flight at once).
template <int NMAX, typename F>
__device__ inline double dot4(F&& term) {
  double s0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0;
#pragma unroll 4
  for (int k = 0; k < NMAX; k += 4) {
    s0 = term(k + 0, s0);
    s1 = term(k + 1, s1);
    s2 = term(k + 2, s2);
    s3 = term(k + 3, s3);
  }
  return (s0 + s1) + (s2 + s3);
}

// The eigensolve runs on A / 2^e (the Gram / 2^2e, tau / 2^e), whose projector is
// the same: e = 0 unless ||X||_F^2 lies so far from 1 that squares of the Gram's
// entries, which rotations and their tests form, would leave the range of a
// double.  No FP32 input needs it (||X||_F^2 between 2^-298 and 2^286).
__device__ inline int eig_shift(double nXF2) {
  const int e = __builtin_amdgcn_frexp_exp(nXF2);  // 0 for 0 and infinity
  return e >= -300 && e <= 300 ? 0 : __builtin_amdgcn_readfirstlane(max(-1000, min(1000, e)) / 2);
}

// Control step of an eigensolve launch, run by one thread after the
// reduction has put the pass's scalars in scal (r2, sum|X|, sum X^2,
// non-finite count).  At the first step it records the norms of X and fixes
// mu and lambda (Sec. II-A); afterwards it applies the stopping test of the
// pass that just ran, ||X - L - S||_F < tol ||X||_F, and the iteration cap.
// A solve with a given start (S0, Y0) stops after fixing mu (the Gram of its
// first iterate needs mu) and eigensolves at its next launch.
// nXF2_prev and tau_prev are the state's ||X||_F^2 and tau as the previous
// launch left them (read early by the caller); tau_out receives this launch's
// threshold tau = 1/mu.
// Returns 1 when the eigensolve of this launch goes ahead.
__device__ inline int control_step(const SolveDesc& d, SolveState* st, const double* scal, int kd,
                                   double nXF2_prev, double tau_prev, double& tau_out) {
  int go = 0;
  tau_out = tau_prev;
  if (kd == 0 && d.warm && st->warm_stage == 1) {
    // given start: the reduced Gram is that of A_1 = X - S0 + Y0/mu (the
    // norms and mu were fixed by the previous launch)
    st->warm_stage = 2;
    go = 1;
  } else if (kd == 0) {
    st->nX1 = scal[1];
    st->nXF2 = scal[2];
    st->nonfinite = scal[3] > 0.0 ? 1 : 0;
    if (st->nonfinite) {
      st->status = kErrNonfinite;
      st->done = 1;
    } else if (st->nX1 == 0.0) {
      st->status = kOk;
      st->resid = 0.0;
      st->done = 1;
    } else {
      const double mu = d.mu_in > 0.0
                            ? d.mu_in
                            : static_cast<double>(d.m) * static_cast<double>(d.n) / (4.0 * st->nX1);
      const double lam = d.lam_in > 0.0
                             ? d.lam_in
                             : 1.0 / sqrt(static_cast<double>(d.m > d.n ? d.m : d.n));
      st->mu = mu;
      st->imu = 1.0 / mu;
      st->tau = 1.0 / mu;
      tau_out = 1.0 / mu;
      st->lam = lam;
      st->gamma = lam / mu;
      // a given start needs one more pass for the Gram of A_1 before the
      // first eigensolve
      st->warm_stage = d.warm ? 1 : 0;
      go = d.warm ? 0 : 1;
    }
  } else {
    st->r2 = scal[0];
    const double rel = sqrt(scal[0]) / sqrt(nXF2_prev);
    st->resid = rel;
    if (!__builtin_isfinite(st->r2)) {
      st->status = kErrNonfinite;
      st->done = 1;
    } else if (d.tol > 0.0 && rel < d.tol) {
      st->status = kOk;
      st->done = 1;
    } else if (kd >= d.maxit) {
      st->status = kNotConverged;
      st->done = 1;
    } else {
      go = 1;
    }
  }
  return go;
}

}  // namespace eigk
}  // namespace rpca
