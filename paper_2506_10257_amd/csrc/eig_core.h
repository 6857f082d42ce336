// Core of the FP64 eigensolver of the n x n Gram matrix (up to 64 frames) and the singular value
// thresholding weights (paper Sec. II-A, Eq. 4).
//
// For A = X - S + Y/mu (m x n, m pixels, n frames) the thresholded SVD
// D_tau(A) = U max(Lambda - tau, 0) V^T equals A P with
//     P = V diag(w) V^T,   w_i = max(sigma_i - tau, 0) / sigma_i,
// where A^T A = V diag(sigma^2) V^T.  One workgroup per solve:
//
//   0. (k_eig) reduction: add the streaming pass's group partials (Gram, residual,
//      and at the first step sum|X|, sum X^2, non-finite count) in order;
//   1. (k_eig) control: decide whether the solve continues (stopping test of the
//      previous pass, iteration cap, mu and lambda at the first iteration);
//   2. warm start: G~ = V_prev^T G V_prev with the previous eigenvectors,
//      which is nearly diagonal once the iteration settles.  V_prev is
//      brought back to orthogonality by one Newton-Schulz step of the polar
//      iteration, V <- V (3I - V^T V) / 2, every kOrthPeriod launches, so the
//      rounding of the products does not build up over hundreds of them;
//   3. until P is accurate (step 4): one simultaneous step, or one sweep.
//      * Simultaneous step: every pair's rotation at once, through the
//        antisymmetric K of the pairs' rotation tangents.  U = I + K + K^2/2
//        is made orthogonal by Newton-Schulz steps (as many as max|U^T U - I|
//        asks for), then G~ <- U^T G~ U and V <- V U.  These are n x n
//        products on the f64 matrix cores: about 0.3 us each at 20 frames,
//        against 13 us for the 19 dependent rounds of a sweep (0.7 us each:
//        the rotation's square roots and the LDS round trips).  Like a sweep
//        it reduces the off-diagonals quadratically once they are small
//        against the gaps; the few pairs that are not are clipped.  When U is
//        too far from orthogonal (strongly rotated, dense clusters) a sweep
//        runs instead.
//      * Sweep (the first launch of a solve, whose V starts from the
//        identity): cyclic two-sided Jacobi in LDS with the round-robin
//        parallel ordering
//        (each index meets every other once per sweep, n/2 disjoint pairs per
//        round).  G and V are double-buffered: a round reads one copy and
//        writes J^T G J and V J into the other, and the threads that own the
//        next round's pairs compute that round's rotations (and the column
//        table of its J) in the same phase, so a round costs one barrier;
//   4. P = V Z V^T in the storage precision, with Z the first-order expansion
//      of the thresholding function at the diagonal D of G~ (Daleckii-Krein:
//      Z_ii = w(d_i), Z_ij = w[d_i, d_j] G~_ij with the divided difference
//      w[,] of w).  It needs no gaps inside the kept or the dropped part of
//      the spectrum, and its error is second order, so step 3 stops one step
//      or sweep earlier than for a diagonal Z.  The second-order term is
//      bounded by n max|Z_ij| max(kappa_ij), kappa in essence the pair's
//      tangent (pair_terms); step 3 ends when that is below PTarget (or, as before, when
//      no pair needs a rotation).
//
// The rotation of a pair is the symmetric 2x2 Schur decomposition with the
// smaller angle (Golub & Van Loan, Matrix Computations, Sec. 8.5), written
// with one division: t = sgn(d) 2 g_pq / (|d| + sqrt(d^2 + 4 g_pq^2)),
// d = g_qq - g_pp, c = 1/sqrt(1 + t^2), s = t c.  A pair is rotated while
// g_pq^2 > eps^2 |g_pp g_qq| (relative off-diagonal test); eps is 1e-15 for
// FP64 solves and 1e-8 for FP32 solves, whose Gram entries carry the data's
// 6e-8 rounding (6x above the off-diagonals left unrotated).
#pragma once

#include <type_traits>

#include "common.h"
#include "eig_common.h"

namespace rpca {
namespace {

using namespace eigk;

// Row stride of the LDS matrices: 17 (mod 32) doubles where it fits, so both
// operand patterns of the matrix products (16 rows x 4 columns and 4 x 16)
// spread over the banks.
constexpr int eig_ld(int nmax) { return nmax == 32 ? 49 : nmax + 1; }

// LDS of one eigensolve.  Entries of the matrices outside n x n are zero for
// the whole step, so fixed-length products need no guards.
template <int NMAX>
struct EigLds {
  double G[2][NMAX * eig_ld(NMAX)];  // two copies of G
  double V[2][NMAX * eig_ld(NMAX)];  // two copies of V
  int cu[2][NMAX];
  double2 cab[2][NMAX];
  double cd[2][NMAX];
  double w[NMAX], dg[NMAX], sg[NMAX];  // w(d), d and sigma = sqrt(d)
  unsigned mx[2][4];                   // maxima of a pass (float bits), by parity of the pass
};

// Steps 2 to 4 for the Gram in copy 0 of G and V_prev (warm; else the identity)
// in copy 0 of V.  orth: bring V_prev back to orthogonality first.  Calls
// out(i, j, P_ij) for every i <= j of the 16 x 16 blocks that cover n (zero
// outside n x n).  Returns the copy that holds V; sweeps is set.  Every thread
// of the workgroup (NT) calls it, after a barrier; the results do not depend on
// NT.  mark(i) is called at the phase boundaries.
template <typename T, int NMAX, int NT, typename Out, typename Mark>
__device__ __forceinline__ int eig_core(EigLds<NMAX>& sh, int n, bool warm, bool orth, double tau,
                                        int& sweeps, Out&& out, Mark&& mark) {
  constexpr int LD = eig_ld(NMAX);
  constexpr int MU = (NMAX * (NMAX + 1) / 2 + NT - 1) / NT;  // upper entries per thread
  constexpr int MF = (NMAX * NMAX + NT - 1) / NT;            // full entries per thread
  typedef double d4 __attribute__((ext_vector_type(4)));
  constexpr int NWV = NT / 64;
  constexpr int NB16 = NMAX / 16;
  constexpr int MBK = (NB16 * NB16 + NWV - 1) / NWV;  // blocks per wave
  double* const G0s = sh.G[0];
  double* const G1s = sh.G[1];
  double* const V0s = sh.V[0];
  double* const V1s = sh.V[1];
  double* const w = sh.w;
  double* const dg = sh.dg;
  double* const sg = sh.sg;
  auto& cu = sh.cu;
  auto& cab = sh.cab;
  auto& cd = sh.cd;
  auto& mx = sh.mx;
  // (unknown to the compiler, so that a caller's loop does not keep every
  // address derived from it in registers across its other phases)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int nup = n * (n + 1) / 2;
  const int nfull = n * n;
  const int nk = (n + 3) >> 2;    // matrix-core steps of a product: entries past n are zero
  const int n16 = (n + 15) >> 4;  // 16 x 16 blocks per side
  int cur = 0;                    // which copy (0 or 1) holds the current G and V
  sweeps = 0;

  // Owned entries: upper-triangle (i <= j, column-packed) and full (row-major).
  int ui[MU], uj[MU], fr[MF], fc[MF];
#pragma unroll
  for (int q = 0; q < MU; ++q) {
    const int idx = tid + q * NT;
    const int j = idx < nup ? packed_col(idx) : 0;
    uj[q] = j;
    ui[q] = idx < nup ? idx - j * (j + 1) / 2 : 0;
  }
#pragma unroll
  for (int q = 0; q < MF; ++q) {
    const int idx = tid + q * NT;
    fr[q] = idx < nfull ? idx / n : 0;
    fc[q] = idx < nfull ? idx - fr[q] * n : 0;
  }

  // n x n products on the f64 matrix cores, one 16 x 16 output block per wave
  // and step: A operand lane l = entry (l % 16, l / 16), B operand lane l =
  // entry (l / 16, l % 16), result lane l, register r = entry (l / 16 + 4r,
  // l % 16).  A block's sum runs over its four-column steps in order, so the
  // result does not depend on which wave forms it.
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the lane, unknown to the compiler at each product: its operand addresses
  // are formed there instead of being kept in registers for the whole step
  auto lane = [&]() {
    int l = tid & 63;
    asm volatile("" : "+v"(l));
    return l;
  };
  // acc = block (bi, bj) of A B, with A (and B) read transposed on request
  auto block = [&](int l, const double* A, bool ta, const double* B, bool tb, int bi, int bj) {
    const int lr = l >> 4, lc = l & 15;
    d4 acc = {0.0, 0.0, 0.0, 0.0};
    const double* pa = ta ? A + lr * LD + 16 * bi + lc : A + (16 * bi + lc) * LD + lr;
    const double* pb = tb ? B + (16 * bj + lc) * LD + lr : B + lr * LD + 16 * bj + lc;
    const int sa = ta ? 4 * LD : 4, sb = tb ? 4 : 4 * LD;
#pragma unroll 4
    for (int kk = 0; kk < nk; ++kk)
      acc = __builtin_amdgcn_mfma_f64_16x16x4f64(pa[kk * sa], pb[kk * sb], acc, 0, 0, 0);
    return acc;
  };
  // every block (SYM: the upper ones), waves w0, w0 + 1, ... taking them in turn;
  // out(i, j, value) for the entries of n x n (SYM: those with i <= j)
  auto product = [&](auto sym, const double* A, bool ta, const double* B, bool tb, auto&& out) {
    constexpr bool SYM = decltype(sym)::value;
    const int nt = SYM ? n16 * (n16 + 1) / 2 : n16 * n16;
    const int l = lane(), lr = l >> 4, lc = l & 15;
    for (int t = wv; t < nt; t += NWV) {
      const int bj = SYM ? packed_col(t) : t % n16;
      const int bi = SYM ? t - bj * (bj + 1) / 2 : t / n16;
      const d4 acc = block(l, A, ta, B, tb, bi, bj);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * bi + lr + 4 * r, j = 16 * bj + lc;
        if (i < n && j < n && (!SYM || i <= j)) out(i, j, acc[r]);
      }
    }
  };
  // D <- D-shaped product in place: the blocks stay in registers until every
  // wave has read the operands; fix(i, j, value) gives the stored entry
  auto product_in_place = [&](const double* A, bool ta, const double* B, double* D, auto&& fix) {
    d4 acc[MBK];
    const int l = lane(), lr = l >> 4, lc = l & 15;
#pragma unroll
    for (int q = 0; q < MBK; ++q) {
      const int t = wv + q * NWV;
      acc[q] = d4{0.0, 0.0, 0.0, 0.0};
      if (t < n16 * n16) acc[q] = block(l, A, ta, B, false, t / n16, t % n16);
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < MBK; ++q) {
      const int t = wv + q * NWV;
      if (t < n16 * n16) {
        const int bi = t / n16, bj = t % n16;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = 16 * bi + lr + 4 * r, j = 16 * bj + lc;
          if (i < n && j < n) D[i * LD + j] = fix(i, j, acc[q][r]);
        }
      }
    }
  };
  const std::integral_constant<bool, true> kSym{};
  const std::integral_constant<bool, false> kAll{};

  // 2. Warm start: G~ = V^T G V (ends in copy 0, with V)
  if (warm) {
    if (orth) {
      product(kSym, V0s, true, V0s, false, [&](int i, int j, double v) {  // C = V^T V
        G1s[i * LD + j] = v;
        G1s[j * LD + i] = v;
      });
      __syncthreads();
      product_in_place(V0s, false, G1s, V0s,
                       [&](int i, int j, double v) { return fma(-0.5, v, 1.5 * V0s[i * LD + j]); });
      __syncthreads();
    }
    product(kAll, G0s, false, V0s, false, [&](int i, int j, double v) { G1s[i * LD + j] = v; });
    __syncthreads();
    product(kSym, V0s, true, G1s, false, [&](int i, int j, double v) {
      G0s[i * LD + j] = v;
      G0s[j * LD + i] = v;
    });
    __syncthreads();
  }
  mark(1);

  // 3. Simultaneous steps and Jacobi sweeps.
  const int N2 = n + (n & 1);
  const int M = N2 - 1;
  const int NP = N2 / 2;
  // One round: read copy SRC and the round's column table, write J^T G J and
  // V J into the other copy; the last wavefront builds the next round's
  // rotations and column table.
  auto round = [&](auto src_tag, int r) {
    constexpr int SRC = decltype(src_tag)::value;
    const double* Gc = SRC ? G1s : G0s;
    double* Gn = SRC ? G0s : G1s;
    const double* Vc = SRC ? V1s : V0s;
    double* Vn = SRC ? V0s : V1s;
    const int rb = r & 1;
    const int* tu_ = cu[rb];
    const double2* tab = cab[rb];
    const double* td = cd[rb];
#pragma unroll
    for (int q = 0; q < MU; ++q) {
      if (tid + q * NT < nup) {  // slots past n(n+1)/2 are skipped by whole waves
        const double v = rotated_entry<LD>(ui[q], uj[q], Gc, tu_, tab, td);
        Gn[ui[q] * LD + uj[q]] = v;
        Gn[uj[q] * LD + ui[q]] = v;
      }
    }
#pragma unroll
    for (int q = 0; q < MF; ++q) {
      if (tid + q * NT < nfull) {
        const int j = fc[q], i = fr[q];
        const int pj = tu_[j];
        const double2 abj = tab[j];
        Vn[i * LD + j] = fma(abj.x, Vc[i * LD + (pj & 0xff)], abj.y * Vc[i * LD + ((pj >> 8) & 0xff)]);
      }
    }
    const int kp = tid - (NT - 64);
    if (r + 1 < M && kp >= 0 && kp < NP) {
      int p, q;
      pair_indices(r + 1, kp, N2, p, q);
      double c = 1.0, s = 0.0, dt = 0.0;
      if (q < n) {
        const double gpp = rotated_entry<LD>(p, p, Gc, tu_, tab, td);
        const double gqq = rotated_entry<LD>(q, q, Gc, tu_, tab, td);
        const double gpq = rotated_entry<LD>(p, q, Gc, tu_, tab, td);
        make_rotation<T>(gpp, gqq, gpq, c, s, dt);
      }
      set_pair_columns(p, q, n, c, s, dt, cu[rb ^ 1], cab[rb ^ 1], cd[rb ^ 1]);
    }
    __syncthreads();
  };
  int steps = 0, pass = 0;
  if (tid < 8) mx[tid >> 2][tid & 3] = 0u;
  double zr[MU];  // Z of the owned pairs
  for (;;) {
    double* G = cur ? G1s : G0s;
    double* V = cur ? V1s : V0s;
    double* A = cur ? G0s : G1s;  // the other copies are free between rounds
    double* B = cur ? V0s : V1s;
    unsigned* mp = mx[pass & 1];
    if (tid < n) {
      const double di = G[tid * LD + tid];
      const double s = sqrt(fmax(di, 0.0));
      dg[tid] = di;
      sg[tid] = s;
      w[tid] = s > tau ? (s - tau) / s : 0.0;
    }
    __syncthreads();
    // Pairs: Z_ij, the tangent of the rotation (into K = A), the maxima of
    // |Z_ij| and of kappa_ij, and whether any pair is left to rotate.
    int need = 0;
    float mz = 0.0f, mk = 0.0f, mt = 0.0f;
#pragma unroll
    for (int q = 0; q < MU; ++q) {
      zr[q] = 0.0;
      if (tid + q * NT < nup && ui[q] < uj[q]) {
        const int i = ui[q], j = uj[q];
        const double e = G[i * LD + j];
        const PairTerms pt = pair_terms<T>(e, dg[i], dg[j], sg[i], sg[j], w[i], w[j], tau, n);
        zr[q] = pt.z;
        need |= pt.rotate;
        mz = fmaxf(mz, pt.mz);
        mk = fmaxf(mk, pt.kappa);
        mt = fmaxf(mt, fabsf(static_cast<float>(pt.t)));
        A[i * LD + j] = pt.t;
        A[j * LD + i] = -pt.t;
      } else if (tid + q * NT < nup) {
        A[ui[q] * LD + ui[q]] = 0.0;
      }
    }
    wave_max_to(mz, &mp[0]);
    wave_max_to(mk, &mp[1]);
    wave_max_to(mt, &mp[2]);
    if (!__syncthreads_or(need)) break;
    const float est = static_cast<float>(n) * __uint_as_float(mp[0]) * __uint_as_float(mp[1]);
    const float tmax = __uint_as_float(mp[2]);
    if (est < PTarget<T>::value) break;
    ++pass;
    if (tid < 4) mx[pass & 1][tid] = 0u;  // last read before the barrier above
    bool stepped = false;
    if (steps < kMaxSteps && (warm || tmax < kColdTangent)) {
      // U = I + K + K^2/2 into B (K^2 is symmetric, K antisymmetric)
      product(kSym, A, false, A, false, [&](int i, int j, double v) {
        const double k = A[i * LD + j], h = fma(0.5, v, i == j ? 1.0 : 0.0);
        B[i * LD + j] = h + k;
        if (i != j) B[j * LD + i] = h - k;
      });
      __syncthreads();
      stepped = true;
      for (int it = 0; it < kMaxOrth; ++it) {
        // C = U^T U into A, with max |C - I|
        float md = 0.0f;
        product(kSym, B, true, B, false, [&](int i, int j, double v) {
          A[i * LD + j] = v;
          A[j * LD + i] = v;
          md = fmaxf(md, fabsf(static_cast<float>(i == j ? v - 1.0 : v)));
        });
        unsigned* mo = mx[pass & 1];
        wave_max_to(md, &mo[0]);
        __syncthreads();
        const float off = __uint_as_float(mo[0]);
        ++pass;
        if (tid < 4) mx[pass & 1][tid] = 0u;
        if (!(off < kOrthMax)) {
          stepped = false;
          break;
        }
        if (off < OrthGoal<T>::skip) break;
        product_in_place(B, false, A, B,
                         [&](int i, int j, double v) { return fma(-0.5, v, 1.5 * B[i * LD + j]); });
        __syncthreads();
        if (0.75f * off * off * static_cast<float>(n) < OrthGoal<T>::skip) break;
      }
      if (stepped) {
        // W = G~ U into A and V U, then G~ <- U^T W
        product(kAll, G, false, B, false, [&](int i, int j, double v) { A[i * LD + j] = v; });
        product_in_place(V, false, B, V, [&](int, int, double v) { return v; });
        product(kSym, B, true, A, false, [&](int i, int j, double v) {
          G[i * LD + j] = v;
          G[j * LD + i] = v;
        });
        ++steps;
      }
      __syncthreads();
    }
    if (stepped) continue;
    if (sweeps >= kMaxSweeps) break;
    ++sweeps;
    if (tid < NP) {  // rotations of round 0
      int p, q;
      pair_indices(0, tid, N2, p, q);
      double c = 1.0, s = 0.0, dt = 0.0;
      if (q < n) make_rotation<T>(G[p * LD + p], G[q * LD + q], G[p * LD + q], c, s, dt);
      set_pair_columns(p, q, n, c, s, dt, cu[0], cab[0], cd[0]);
    }
    __syncthreads();
    for (int r = 0; r < M; ++r) {
      if (cur) round(std::integral_constant<int, 1>{}, r);
      else round(std::integral_constant<int, 0>{}, r);
      cur ^= 1;
    }
  }
  mark(2);

  // 4. P = V Z V^T (exactly symmetric).
  const double* Vf = cur ? V1s : V0s;
  double* Zs = cur ? G0s : G1s;
  double* Ys = cur ? V0s : V1s;
  __syncthreads();  // every thread is past its reads of the maxima and of A
#pragma unroll
  for (int q = 0; q < MU; ++q) {
    if (tid + q * NT < nup) {
      const int i = ui[q], j = uj[q];
      const double z = i == j ? w[i] : zr[q];
      Zs[i * LD + j] = z;
      Zs[j * LD + i] = z;
    }
  }
  __syncthreads();
  product(kAll, Vf, false, Zs, false, [&](int i, int j, double v) { Ys[i * LD + j] = v; });
  __syncthreads();
  const int l = lane(), lr = l >> 4, lc = l & 15;
  for (int t = wv; t < n16 * (n16 + 1) / 2; t += NWV) {  // zero outside n x n
    const int bj = packed_col(t), bi = t - bj * (bj + 1) / 2;
    const d4 acc = block(l, Ys, false, Vf, true, bi, bj);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * bi + lr + 4 * r, j = 16 * bj + lc;
      if (i <= j) out(i, j, acc[r]);
    }
  }
  return cur;
}

}  // namespace
}  // namespace rpca
