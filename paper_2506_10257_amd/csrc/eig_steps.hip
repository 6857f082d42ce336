// Warm-started eigensolve of windows of 65 to 144 frames by simultaneous
// rotation steps, one workgroup per solve.
//
// The method is that of the simultaneous steps in eig.hip: all pairs of the
// nearly diagonal G~ = V^T G V are rotated at once through matrix products, and
// P = V Z V^T with Z the first-order expansion of the thresholding function at
// the diagonal of G~.  Here the matrices (up to 166 KB each) stay in the
// solve's workspace, that is in the L2, and every product runs on the f64
// matrix cores, two 16 x 16 blocks of a row of blocks per wave at a time:
//
//   reduce   G = sum of the group partials, control step (stopping test)
//   W = G V;  S = V^T W, C = V^T V
//   step s = 0, 1, ...:
//     pairs   M = C - I; D and E of S - (M D + D M)/2; Z, K, error bound
//     T = K^2;  U = I + K + T/2 - M/2 (+ K^3/6 + T^2/24 for large rotations)
//     W = S U, V' = V U;  S = U^T W, C = V'^T V'
//   Y = Z V^T, P = V Y
//
// V need not be orthogonal to full precision: M = V^T V - I is carried and
// taken out to first order (in D and E, in Z, and in the next U, as in the
// iterative refinement of Ogita & Aishima, Japan J. Indust. Appl. Math. 35,
// 2018), so it converges with E.  Where the steps do not converge (strongly
// rotated dense clusters, or more than kWideSteps steps) the Jacobi kernel
// (eig_wide.hip), launched next, runs sweeps from the previous iteration's V.
//
// Bound: a product is 2 nb^3 FP64 operations on one CU (307 GFLOP/s: 19 us at
// 144 frames, 9 us at 112), and a solve takes about 15 of them per iteration;
// a Jacobi sweep is 131 (99) dependent rounds, 500 (230) us at 132 (100).
#include "common.h"
#include "eig_common.h"
#include "launch.h"

namespace rpca {
namespace {

using namespace eigk;

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kStepThreads = 1024;
constexpr int kStepWaves = kStepThreads / 64;

// Blocks (bi, bj) and (bi, bj + 1) of X^T Y (TA: of X Y; TB: of X^T Y^T), the
// second one only when `two`.  A operand lane l = entry (l % 16, l / 16) of the
// left factor, B operand lane l = entry (l / 16, l % 16) of the right one;
// result lane l, register r = entry (l / 16 + 4r, l % 16).
template <bool TA, bool TB>
__device__ inline void blocks2(const double* Xp, const double* Yp, int nb, int bi, int bj, bool two,
                               d4& s0, d4& s1) {
  const int l = threadIdx.x & 63, lr = l >> 4, lc = l & 15;
  const int bj1 = two ? bj + 1 : bj;
  gptr<const double> x = as_global<double>(
      static_cast<const void*>(TA ? Xp + (16 * bi + lc) * nb + lr : Xp + lr * nb + 16 * bi + lc));
  gptr<const double> y0 = as_global<double>(
      static_cast<const void*>(TB ? Yp + (16 * bj + lc) * nb + lr : Yp + lr * nb + 16 * bj + lc));
  gptr<const double> y1 = as_global<double>(
      static_cast<const void*>(TB ? Yp + (16 * bj1 + lc) * nb + lr : Yp + lr * nb + 16 * bj1 + lc));
  const int dx = TA ? 4 : 4 * nb, dy = TB ? 4 : 4 * nb;
  s0 = d4{0.0, 0.0, 0.0, 0.0};
  s1 = d4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 1
  for (int k0 = 0; k0 < nb; k0 += 16) {
    double a[4], b[4], c[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      a[k] = x[k * dx];
      b[k] = y0[k * dy];
      c[k] = y1[k * dy];
    }
    x += 4 * dx;
    y0 += 4 * dy;
    y1 += 4 * dy;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      s0 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[k], b[k], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f64_16x16x4f64(a[k], c[k], s1, 0, 0, 0);
    }
  }
}

// Every block of a product (SYM: the upper ones), as pairs of blocks of one
// block row, units u, u + kStepWaves, ... of this wave.  `u` is advanced past
// the product's units, so that two products with no barrier between them share
// the waves evenly.  out(i, j, value) is called for each entry (SYM: i <= j).
template <bool SYM, bool TA = false, bool TB = false, typename Out>
__device__ inline void product(int& u, const double* X, const double* Y, int nb, Out&& out) {
  const int nt = nb >> 4, l = threadIdx.x & 63, lr = l >> 4, lc = l & 15;
  int units = 0;
  for (int b = 0; b < nt; ++b) units += ((SYM ? nt - b : nt) + 1) >> 1;
  for (; u < units; u += kStepWaves) {
    int bi = 0, v = u;
    for (;; ++bi) {
      const int row = ((SYM ? nt - bi : nt) + 1) >> 1;
      if (v < row) break;
      v -= row;
    }
    const int bj = (SYM ? bi : 0) + 2 * v;
    const bool two = bj + 1 < nt;
    d4 s0, s1;
    blocks2<TA, TB>(X, Y, nb, bi, bj, two, s0, s1);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = 16 * bi + lr + 4 * r, j = 16 * bj + lc;
      if (!SYM || i <= j) out(i, j, s0[r]);
      if (two) out(i, j + 16, s1[r]);
    }
  }
  u -= units;
}

template <typename T>
__global__ void __launch_bounds__(kStepThreads)
k_eig_steps(const SolveDesc* __restrict__ descs, const int32_t* __restrict__ ids) {
  __shared__ double dg[kEigHugeMaxN], sg[kEigHugeMaxN], w[kEigHugeMaxN], sd[kEigHugeMaxN];
  __shared__ double scal[kScalars];
  __shared__ unsigned mx[2][4];
  __shared__ int s_go;
  __shared__ double s_tau;
  const int tid = threadIdx.x;
  const SolveDesc& d = descs[ids[blockIdx.x]];
  SolveState* st = d.st;
  // a solve's first eigensolve is the Jacobi kernel's
  if (st->done || st->iter == 0) return;
  const WideEig e(d);
  const int n = d.n, nb = d.nb, kd = st->iter;
  double pf_nXF2 = 0.0, pf_tau = 0.0;
  if (tid == 0) {
    pf_nXF2 = st->nXF2;
    pf_tau = st->tau;
    e.ctl->booked = 0;
  }

  // Sum of the group partials in group order; the Gram into both halves of G.
  {
    const int nent = kScalars + gram_blocks((n + 3) >> 2) * 16;
    constexpr int kChunk = 16;
    for (int idx = tid; idx < nent; idx += kStepThreads) {
      double sum = 0.0;
      for (int q0 = 0; q0 < d.groups; q0 += kChunk) {
        const int c = min(kChunk, d.groups - q0);
        double v[kChunk];
#pragma unroll
        for (int q = 0; q < kChunk; ++q)
          v[q] = q < c ? d.gpartials[static_cast<size_t>(q0 + q) * d.pstride + idx] : 0.0;
#pragma unroll
        for (int q = 0; q < kChunk; ++q)
          if (q < c) sum += v[q];
      }
      if (idx < kScalars) {
        scal[idx] = sum;
      } else {
        const int g = idx - kScalars, blk = g >> 4, el = g & 15;
        const int bj = packed_col(blk), bi = blk - bj * (bj + 1) / 2;
        const int i = 4 * bi + (el >> 2), j = 4 * bj + (el & 3);
        if (i <= j && j < n) {
          e.G[i * nb + j] = sum;
          e.G[j * nb + i] = sum;
        }
      }
    }
  }
  if (tid < 8) mx[tid >> 2][tid & 3] = 0u;
  __syncthreads();
  if (tid == 0) {
    double t = 0.0;
    s_go = control_step(d, st, scal, kd, pf_nXF2, pf_tau, t);
    s_tau = t;
  }
  __syncthreads();
  if (!s_go) return;
  const double tau = s_tau;
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto put = [&](double* M) { return [M, nb](int i, int j, double v) { M[i * nb + j] = v; }; };
  auto put_sym = [&](double* M) {
    return [M, nb](int i, int j, double v) {
      M[i * nb + j] = v;
      M[j * nb + i] = v;
    };
  };

  // W = G V (G symmetric), S = V^T W, C = V^T V
  const int v0 = e.ctl->vsel;
  double* V = e.v(v0);
  int u = wv;
  product<false>(u, e.G, V, nb, put(e.W));
  __syncthreads();
  u = wv;
  product<true>(u, V, e.W, nb, put_sym(e.S));
  product<true>(u, V, V, nb, put_sym(e.C));
  __syncthreads();

  int s = 0;
  bool ok = false;
  for (;; ++s) {
    unsigned* mp = mx[s & 1];
    if (tid < n) {
      const double sii = e.S[tid * nb + tid], m = e.C[tid * nb + tid] - 1.0;
      const double di = fma(-m, sii, sii), si = sqrt_or_zero(di);
      const double wi = si > tau ? 1.0 - tau * rcp_pos(si) : 0.0;
      sd[tid] = sii;
      dg[tid] = di;
      sg[tid] = si;
      w[tid] = wi;
      e.Z[tid * nb + tid] = fma(-m, wi, wi);
      e.K[tid * nb + tid] = 0.0;
    }
    __syncthreads();
    float mz = 0.0f, mk = 0.0f, mm = 0.0f, mt = 0.0f;
    for (int idx = tid; idx < n * (n + 1) / 2; idx += kStepThreads) {
      const int j = packed_col(idx), i = idx - j * (j + 1) / 2;
      const double c = e.C[i * nb + j];
      if (i == j) {
        mm = fmaxf(mm, fabsf(static_cast<float>(c - 1.0)));
        if (!(c == c)) mm = INFINITY;
        continue;
      }
      const double el = fma(-0.5 * c, sd[i] + sd[j], e.S[i * nb + j]);
      const PairTerms pt = pair_terms<T>(el, dg[i], dg[j], sg[i], sg[j], w[i], w[j], tau, n);
      const double z = fma(-0.5 * c, w[i] + w[j], pt.z);
      e.Z[i * nb + j] = z;
      e.Z[j * nb + i] = z;
      e.K[i * nb + j] = pt.t;
      e.K[j * nb + i] = -pt.t;
      mz = fmaxf(mz, pt.mz);
      mk = fmaxf(mk, pt.kappa);
      mt = fmaxf(mt, fabsf(static_cast<float>(pt.t)));
      mm = fmaxf(mm, fabsf(static_cast<float>(c)));
    }
    wave_max_to(mz, &mp[0]);
    wave_max_to(mk, &mp[1]);
    wave_max_to(mm, &mp[2]);
    wave_max_to(mt, &mp[3]);
    __syncthreads();
    mz = __uint_as_float(mp[0]);
    mk = __uint_as_float(mp[1]);
    mm = __uint_as_float(mp[2]);
    mt = __uint_as_float(mp[3]);
    if (tid < 4) mx[(s + 1) & 1][tid] = 0u;  // last read before the barrier above
    if (!(mm < kOrthMax)) break;
    ok = static_cast<float>(n) * fmaxf(mz, mm) * fmaxf(mk, mm) < PTarget<T>::value;
    if (ok || s == kWideSteps) break;

    // U = I + K + T/2 - M/2, T = K^2 = -K^T K (to fourth order for large K)
    const bool fourth = mt > kWideFourth;
    u = wv;
    if (!fourth) {
      product<true>(u, e.K, e.K, nb, [&](int i, int j, double v) {
        const double id = i == j ? 1.0 : 0.0, k = e.K[i * nb + j];
        const double m = j < n ? e.C[i * nb + j] - id : 0.0;
        const double h = id - 0.5 * (v + m);
        e.U[i * nb + j] = h + k;
        if (i != j) e.U[j * nb + i] = h - k;
      });
    } else {
      product<true>(u, e.K, e.K, nb, [&](int i, int j, double v) {
        e.T[i * nb + j] = -v;
        e.T[j * nb + i] = -v;
      });
      __syncthreads();
      // (K T into W, T^2 straight into U; an entry of both has one owner)
      u = wv;
      product<true>(u, e.K, e.T, nb, [&](int i, int j, double v) { e.W[i * nb + j] = -v; });
      u = wv;
      product<true>(u, e.T, e.T, nb, [&](int i, int j, double v) {
        const double id = i == j ? 1.0 : 0.0;
        const double m = j < n ? e.C[i * nb + j] - id : 0.0;
        const double h = id + 0.5 * (e.T[i * nb + j] - m) + v * (1.0 / 24.0);
        const double a = i == j ? 0.0 : fma(e.W[i * nb + j], 1.0 / 6.0, e.K[i * nb + j]);
        e.U[i * nb + j] = h + a;
        if (i != j) e.U[j * nb + i] = h - a;
      });
    }
    __syncthreads();
    // W = S U, V' = V U;  S = U^T W, C = V'^T V'
    double* Vn = e.v(WideEig::vsel(v0, s + 1));
    u = wv;
    product<false>(u, e.S, e.U, nb, put(e.W));
      product<false, true>(u, V, e.U, nb, put(Vn));
    V = Vn;
    __syncthreads();
    u = wv;
    product<true>(u, e.U, e.W, nb, put_sym(e.S));
      product<true>(u, V, V, nb, put_sym(e.C));
    __syncthreads();
  }
  if (!ok) return;  // the Jacobi kernel takes over, from V at v0

  // P = V (Z V^T) (exactly symmetric)
  u = wv;
  product<false, false, true>(u, e.Z, V, nb, put(e.W));
  __syncthreads();
  const gptr<T> P = as_global<T>(d.P);
  u = wv;
  product<true, true>(u, V, e.W, nb, [&](int i, int j, double v) {
    P[i * nb + j] = static_cast<T>(v);
    P[j * nb + i] = static_cast<T>(v);
  });
  const int rank = __syncthreads_count(tid < n && w[tid] != 0.0);
  if (tid == 0) {
    e.ctl->vsel = WideEig::vsel(v0, s);
    e.ctl->booked = kd + 1;
    st->rank = rank;
    st->sweeps = 0;
    st->iter = kd + 1;
  }
}

}  // namespace

hipError_t launch_eig_steps(int dtype, int grid, hipStream_t stream, const SolveDesc* descs,
                            const int32_t* ids) {
  if (grid <= 0) return hipSuccess;
  if (dtype == 1)
    RPCA_LAUNCH(k_eig_steps<float>, dim3(grid), dim3(kStepThreads), 0, stream, descs, ids);
  else
    RPCA_LAUNCH(k_eig_steps<double>, dim3(grid), dim3(kStepThreads), 0, stream, descs, ids);
  return hipGetLastError();
}

}  // namespace rpca
