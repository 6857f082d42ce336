// Core of the FP64 eigensolver of the n x n Gram matrix (up to 64 frames) and
// the singular value thresholding weights (paper Sec. II-A, Eq. 4).
//
// For A = X - S + Y/mu (m x n, m pixels, n frames) the thresholded SVD
// D_tau(A) = U max(Lambda - tau, 0) V^T equals A P with
//     P = V diag(w) V^T,   w_i = max(sigma_i - tau, 0) / sigma_i,
// where A^T A = V diag(sigma^2) V^T.  One workgroup per solve:
//
//   1. warm start: S = V^T G V with the previous eigenvectors, which is nearly
//      diagonal once the iteration settles, and C = V^T V;
//   2. until P is accurate (step 3): one simultaneous step, or one sweep.
//      * Simultaneous step: every pair's rotation at once, U = I + R + R^2/2
//        with R = K - M/2, K the antisymmetric matrix of the pairs' rotation
//        tangents and M = C - I.  Then V <- V U, S <- U^T S U, C = V^T V.  V
//        need not be orthogonal to full precision: M is taken out to first
//        order wherever S, Z and U are formed (as in the iterative refinement
//        of Ogita & Aishima, Japan J. Indust. Appl. Math. 35, 2018), so it
//        converges with the off-diagonals.  These are n x n products on the
//        f64 matrix cores, 0.4-0.5 us each at 20 frames, against 13 us for the
//        19 dependent rounds of a sweep (0.7 us each: the rotation's square
//        roots and the LDS round trips).  Like a sweep a step reduces the
//        off-diagonals quadratically once they are small against the gaps; the
//        few pairs that are not are clipped.  Where the tangents are large and
//        dense (their row sums above kRowSumMax) a sweep runs instead.
//      * Sweep (the first launch of a solve, whose V starts from the
//        identity): cyclic two-sided Jacobi with the round-robin parallel
//        ordering (each index meets every other once per sweep, n/2 disjoint
//        pairs per round).  G and V are double-buffered: a round reads one copy
//        and writes J^T G J and V J into the other, and the threads that own
//        the next round's pairs compute that round's rotations (and the column
//        table of its J) in the same phase, so a round costs one barrier;
//   3. P = V Z V^T in the storage precision, with Z the first-order expansion
//      of the thresholding function at the diagonal D of S (Daleckii-Krein:
//      Z_ii = w(d_i), Z_ij = w[d_i, d_j] S_ij with the divided difference
//      w[,] of w).  It needs no gaps inside the kept or the dropped part of the
//      spectrum, and its error is second order, so step 2 stops one step or
//      sweep earlier than for a diagonal Z.  The second-order term is bounded
//      by n max(mz_ij, |M_ij|) max(kappa_ij, |M_ij|), with mz the pair's
//      off-diagonal times the largest slope of w it can bring and kappa in
//      essence the pair's tangent (pair_terms); step 2 ends when that is below
//      PTarget (or when no pair needs a rotation).
//
// The rotation of a pair is the symmetric 2x2 Schur decomposition with the
// smaller angle (Golub & Van Loan, Matrix Computations, Sec. 8.5), written
// with one division: t = sgn(d) 2 g_pq / (|d| + sqrt(d^2 + 4 g_pq^2)),
// d = g_qq - g_pp, c = 1/sqrt(1 + t^2), s = t c.  A sweep rotates a pair while
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
  double w[NMAX];                // w(d)
  double sd[NMAX], md[NMAX];     // diagonals of S and of M
  unsigned mx[2][8];             // maxima of a pass (float bits), by parity of the pass
};

// Steps 1 to 3 for the Gram in copy 0 of G and V_prev (warm; else the identity)
// in copy 0 of V.  Calls out(i, j, P_ij) for every i <= j of the 16 x 16 blocks
// that cover n (zero outside n x n).  Returns the copy that holds V; sweeps is
// set.  Every thread of the workgroup (NT) calls it, after a barrier; the
// results do not depend on NT.  mark(i) is called at the phase boundaries.
template <typename T, int NMAX, int NT, typename Out, typename Mark>
__device__ __forceinline__ int eig_core(EigLds<NMAX>& sh, int n, bool warm, double tau, int& sweeps,
                                        Out&& out, Mark&& mark) {
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
  auto& cu = sh.cu;
  auto& cab = sh.cab;
  auto& cd = sh.cd;
  // (unknown to the compiler, so that a caller's loop does not keep every
  // address derived from it in registers across its other phases)
  int tid = threadIdx.x;
  asm volatile("" : "+v"(tid));
  const int nup = n * (n + 1) / 2;
  const int nfull = n * n;
  const int nk = (n + 3) >> 2;  // matrix-core steps of a product: entries past n are zero
  // 16 x 16 blocks per side (fixed below 64 frames: a class of 32 has 17 to 32)
  const int n16 = NMAX <= 32 ? NB16 : (n + 15) >> 4;
  int cur = 0;  // which copy (0 or 1) holds the current S and V
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

  // n x n products on the f64 matrix cores, one 16 x 16 output block per wave:
  // A operand lane l = entry (l % 16, l / 16), B operand lane l = entry (l / 16,
  // l % 16), result lane l, register r = entry (l / 16 + 4r, l % 16).  A block's
  // sum runs over its four-column steps in order, so the result does not depend
  // on which wave forms it.
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  // the lane, unknown to the compiler at each product: its operand addresses
  // are formed there instead of being kept in registers for the whole step
  auto lane = [&]() {
    int l = tid & 63;
    asm volatile("" : "+v"(l));
    return l;
  };
  // block (bi, bj) of A B, with A (and B) read transposed on request; all of
  // its operands are read before the first product
  auto block = [&](int l, const double* A, bool ta, const double* B, bool tb, int bi, int bj) {
    const int lr = l >> 4, lc = l & 15;
    d4 acc = {0.0, 0.0, 0.0, 0.0};
    const double* pa = ta ? A + lr * LD + 16 * bi + lc : A + (16 * bi + lc) * LD + lr;
    const double* pb = tb ? B + (16 * bj + lc) * LD + lr : B + lr * LD + 16 * bj + lc;
    const int sa = ta ? 4 * LD : 4, sb = tb ? 4 : 4 * LD;
    // K steps [k, k + K): the columns past nk are zeros, so a few steps too many
    // cost less than branches between the products
    auto steps = [&](auto count, int k) {
      constexpr int K = decltype(count)::value;
      double a[K], b[K];
#pragma unroll
      for (int i = 0; i < K; ++i) {
        a[i] = pa[(k + i) * sa];
        b[i] = pb[(k + i) * sb];
      }
#pragma unroll
      for (int i = 0; i < K; ++i) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a[i], b[i], acc, 0, 0, 0);
    };
    if constexpr (NMAX == 16) {
      steps(std::integral_constant<int, 4>{}, 0);
    } else if constexpr (NMAX == 32) {  // 17 to 20 frames: 5; else 8
      steps(std::integral_constant<int, 5>{}, 0);
      if (nk > 5) steps(std::integral_constant<int, 3>{}, 5);
    } else {  // 33 to 64 frames: 9 to 16
      steps(std::integral_constant<int, 8>{}, 0);
#pragma unroll 1
      for (int k = 8; k < nk; k += 4) steps(std::integral_constant<int, 4>{}, k);
    }
    return acc;
  };
  // The output blocks of this wave, with the blocks dealt to the waves from
  // wave `from` on (two products in one phase: the second starts where the
  // first one's waves end).  f(q, bi, bj): the wave's q-th block.
  auto blocks = [&](auto sym, int from, auto&& f) {
    constexpr bool SYM = decltype(sym)::value;
    const int nt = SYM ? n16 * (n16 + 1) / 2 : n16 * n16;
    int t = (wv - from) & (NWV - 1);
#pragma unroll
    for (int q = 0; q < MBK; ++q, t += NWV)
      if (t < nt) {
        const int bj = SYM ? (NB16 <= 2 ? (t + 1) >> 1 : packed_col(t)) : t % n16;
        f(q, SYM ? t - bj * (bj + 1) / 2 : t / n16, bj);
      }
  };
  // g(i, j, value) for the entries of a block (SYM: those with i <= j); outside
  // n x n the operands, and so the values, are zero
  auto entries = [&](auto sym, int l, const d4& v, int bi, int bj, auto&& g) {
    constexpr bool SYM = decltype(sym)::value;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * bi + (l >> 4) + 4 * r, j = 16 * bj + (l & 15);
      if (!SYM || i <= j) g(i, j, v[r]);
    }
  };
  const std::integral_constant<bool, true> kSym{};
  const std::integral_constant<bool, false> kAll{};
  // D = A B (every block), D no operand of the phase
  auto product = [&](int from, const double* A, bool ta, const double* B, bool tb, double* D) {
    const int l = lane();
    blocks(kAll, from, [&](int, int bi, int bj) {
      entries(kAll, l, block(l, A, ta, B, tb, bi, bj), bi, bj, [&](int i, int j, double v) { D[i * LD + j] = v; });
    });
  };
  // S = A^T B (symmetric), with its diagonal in sd
  auto form_s = [&](const double* A, const double* B, double* D) {
    const int l = lane();
    blocks(kSym, 0, [&](int, int bi, int bj) {
      entries(kSym, l, block(l, A, true, B, false, bi, bj), bi, bj, [&](int i, int j, double v) {
        D[i * LD + j] = v;
        D[j * LD + i] = v;
        if (i == j) sh.sd[i] = v;
      });
    });
  };
  // C = V^T V (its upper half), with the diagonal of M = C - I in md
  auto form_c = [&](int from, const double* V, double* D) {
    const int l = lane();
    blocks(kSym, from, [&](int, int bi, int bj) {
      entries(kSym, l, block(l, V, true, V, false, bi, bj), bi, bj, [&](int i, int j, double v) {
        D[i * LD + j] = v;
        if (i == j) sh.md[i] = v - 1.0;
      });
    });
  };

  // 1. Warm start (S and V in copy 0, C in copy 1 of V)
  bool have_c = warm;
  if (tid < 16) sh.mx[tid >> 3][tid & 7] = 0u;
  if (warm) {
    product(0, G0s, false, V0s, false, G1s);
    __syncthreads();
    form_s(V0s, G1s, G0s);
    form_c(n16 * (n16 + 1) / 2, V0s, V1s);
    __syncthreads();
  }
  mark(1);

  // 2. Simultaneous steps and Jacobi sweeps.
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
  for (;;) {
    double* const G = cur ? G1s : G0s;
    double* const V = cur ? V1s : V0s;
    double* const A = cur ? G0s : G1s;  // the other copies are free between rounds
    double* const B = cur ? V0s : V1s;
    unsigned* const mp = sh.mx[pass & 1];
    if (!have_c) {
      if (tid < n) {
        sh.sd[tid] = G[tid * LD + tid];
        sh.md[tid] = 0.0;
      }
      __syncthreads();
    }
    // Pairs: Z (into B, over C: an entry's reader writes it), R (into A), the
    // maxima of the error bound's factors and of the tangents, and whether any
    // pair is left to rotate.
    int need = 0;
    float mz = 0.0f, mk = 0.0f, mm = 0.0f, mt = 0.0f;
#pragma unroll
    for (int q = 0; q < MU; ++q) {
      if (tid + q * NT < nup) {
        const int i = ui[q], j = uj[q];
        const double sii = sh.sd[i], sjj = sh.sd[j], mii = sh.md[i], mjj = sh.md[j];
        const double di = fma(-mii, sii, sii), dj = fma(-mjj, sjj, sjj);
        // (the Gram overflowed: NaN from here into P, and the solve says so)
        const double ri = rsqrt_or_zero(di), rj = rsqrt_or_zero(dj);
        const double si = di * ri, sj = dj * rj;
        const double wi = si <= tau ? 0.0 : fma(-tau, ri, 1.0), wj = sj <= tau ? 0.0 : fma(-tau, rj, 1.0);
        if (i == j) {
          w[i] = wi;
          B[i * LD + i] = fma(-mii, wi, wi);
          A[i * LD + i] = -0.5 * mii;
          mm = fmaxf(mm, fabsf(static_cast<float>(mii)));
        } else {
          const double m = have_c ? B[i * LD + j] : 0.0;
          const double e = fma(-0.5 * m, sii + sjj, G[i * LD + j]);
          const PairTerms pt = pair_terms<T>(e, di, dj, si, sj, ri, rj, wi, wj, tau, n);
          const double z = fma(-0.5 * m, wi + wj, pt.z);
          B[i * LD + j] = z;
          B[j * LD + i] = z;
          A[i * LD + j] = fma(-0.5, m, pt.t);
          A[j * LD + i] = fma(-0.5, m, -pt.t);
          need |= pt.rotate;
          mz = fmaxf(mz, pt.mz);
          mk = fmaxf(mk, pt.kappa);
          mt = fmaxf(mt, fabsf(static_cast<float>(pt.t)));
          mm = fmaxf(mm, fabsf(static_cast<float>(m)));
        }
      }
    }
    wave_max_to(mz, &mp[0]);
    wave_max_to(mk, &mp[1]);
    wave_max_to(mm, &mp[2]);
    wave_max_to(mt, &mp[3]);
    need = __syncthreads_or(need);
    mz = __uint_as_float(mp[0]);
    mk = __uint_as_float(mp[1]);
    mm = __uint_as_float(mp[2]);
    mt = __uint_as_float(mp[3]);
    const float nf = static_cast<float>(n);
    const bool ortho = mm < OrthGoal<T>::skip;
    if ((!need && ortho) || nf * fmaxf(mz, mm) * fmaxf(mk, mm) < PTarget<T>::value) break;
    if (++pass > kMaxPasses) break;
    if (tid < 8) sh.mx[pass & 1][tid] = 0u;  // last read before the barrier above
    bool step = steps < kMaxSteps && mm < kOrthMax && (warm || mt < kColdTangent);
    if (step && nf * mt > kRowSumMax) {
      // the row sums bound the norm of K (zero at most pairs): taken in order
      if (tid < n) {
        float s = 0.0f;
        for (int k = 0; k < n; ++k) s += fabsf(static_cast<float>(A[tid * LD + k]));
        atomicMax(&mp[4], __float_as_uint(s));
      }
      __syncthreads();
      step = __uint_as_float(mp[4]) < kRowSumMax;
    }
    if (!step && !ortho) {
      // V to full orthogonality first: the step with K = 0
#pragma unroll
      for (int q = 0; q < MU; ++q)
        if (tid + q * NT < nup && ui[q] < uj[q]) {
          const int i = ui[q], j = uj[q];
          const double h = 0.5 * (A[i * LD + j] + A[j * LD + i]);
          A[i * LD + j] = h;
          A[j * LD + i] = h;
        }
      __syncthreads();
      step = true;
    }
    if (step) {
      ++steps;
      {  // U = I + R + R^2/2 into B
        const int l = lane();
        blocks(kAll, 0, [&](int, int bi, int bj) {
          d4 r;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int i = 16 * bi + (l >> 4) + 4 * e, j = 16 * bj + (l & 15);
            r[e] = A[i * LD + j] + (i == j ? 1.0 : 0.0);
          }
          const d4 rr = block(l, A, false, A, false, bi, bj);
#pragma unroll
          for (int e = 0; e < 4; ++e) r[e] = fma(0.5, rr[e], r[e]);
          entries(kAll, l, r, bi, bj, [&](int i, int j, double v) { B[i * LD + j] = v; });
        });
      }
      __syncthreads();
      // W = S U into A; V U
      product(0, G, false, B, false, A);
      d4 vu[MBK];
      const int from = n16 * n16, lv = lane();
      blocks(kAll, from, [&](int q, int bi, int bj) { vu[q] = block(lv, V, false, B, false, bi, bj); });
      __syncthreads();
      blocks(kAll, from, [&](int q, int bi, int bj) {
        entries(kAll, lv, vu[q], bi, bj, [&](int i, int j, double v) { V[i * LD + j] = v; });
      });
      form_s(B, A, G);  // S = U^T W
      __syncthreads();
      form_c(0, V, B);
      have_c = true;
      __syncthreads();
      continue;
    }
    if (sweeps >= kMaxSweeps) break;
    ++sweeps;
    have_c = false;
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

  // 3. P = V Z V^T (exactly symmetric); Z is in the other copy of V.
  const double* Vf = cur ? V1s : V0s;
  const double* Zs = cur ? V0s : V1s;
  double* Ys = cur ? G0s : G1s;
  product(0, Vf, false, Zs, false, Ys);
  __syncthreads();
  const int l = lane();
  blocks(kSym, 0, [&](int, int bi, int bj) {
    const d4 acc = block(l, Ys, false, Vf, true, bi, bj);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * bi + (l >> 4) + 4 * r, j = 16 * bj + (l & 15);
      if (i <= j) out(i, j, acc[r]);
    }
  });
  return cur;
}

}  // namespace
}  // namespace rpca
