// Eigensolve launch of solves of up to 64 frames: the final level of the
// streaming pass's reduction, the control step and the eigensolve and
// projector of eig_core.h, one workgroup per solve.
#include <atomic>
#include <type_traits>

#include "common.h"
#include "eig_common.h"
#include "eig_core.h"
#include "launch.h"

namespace rpca {
namespace {

using namespace eigk;

template <typename T, int NMAX, int NT>
__global__ void __launch_bounds__(NT)
k_eig(const SolveDesc* __restrict__ descs, const int32_t* __restrict__ ids) {
  constexpr int LD = eig_ld(NMAX);
  constexpr int MF = (NMAX * NMAX + NT - 1) / NT;  // full entries per thread
  __shared__ EigLds<NMAX> sh;
  __shared__ double scal[kScalars];
  __shared__ int s_go;
  __shared__ double s_tau;
  double* const G0s = sh.G[0];
  double* const V0s = sh.V[0];
  const int tid = threadIdx.x;
  const SolveDesc& d = descs[ids[blockIdx.x]];
  SolveState* st = d.st;
#ifdef RPCA_TRACE
  int64_t tprev = RPCA_NOW();
#define EIG_MARK(i)                               \
  do {                                            \
    if (tid == 0) {                               \
      const int64_t tnow_ = RPCA_NOW();           \
      st->trace[i] += tnow_ - tprev;              \
      tprev = tnow_;                              \
    }                                             \
  } while (0)
#else
#define EIG_MARK(i) \
  do {              \
  } while (0)
#endif

  if (st->done) return;
  const int n = d.n;
  const int nb = d.nb;
  const int kd = st->iter;
  // read now (thread 0 runs the control step), in flight during the reduction
  double pf_nXF2 = 0.0, pf_tau = 0.0;
  if (tid == 0) {
    pf_nXF2 = st->nXF2;
    pf_tau = st->tau;
  }
  int shift = eig_shift(st->nXF2);  // (0 before the first control step)
  const bool warm = kd > 0;
  const int nfull = n * n;

  int fr[MF], fc[MF];
#pragma unroll
  for (int q = 0; q < MF; ++q) {
    const int idx = tid + q * NT;
    fr[q] = idx < nfull ? idx / n : 0;
    fc[q] = idx < nfull ? idx - fr[q] * n : 0;
  }

  // Previous eigenvectors: issue the loads before the reduction.
  double vpre[MF];
#pragma unroll
  for (int q = 0; q < MF; ++q) {
    vpre[q] = 0.0;
    if (tid + q * NT < nfull) {
      vpre[q] = warm ? d.V[fr[q] * nb + fc[q]] : (fr[q] == fc[q] ? 1.0 : 0.0);
    }
  }

  // Zero the LDS matrices (they stay zero outside n x n).
  for (int idx = tid; idx < 2 * NMAX * LD; idx += NT) {
    (&sh.G[0][0])[idx] = 0.0;
    (&sh.V[0][0])[idx] = 0.0;
  }
  __syncthreads();

  // 0. Final level of the streaming pass's reduction, Gram straight into LDS.
  {
    const int nblk = gram_blocks((n + 3) >> 2);
    const int nent = kScalars + nblk * 16;
    constexpr int kChunk = 32;  // one batch of loads for up to 32 groups
    for (int idx = tid; idx < nent; idx += NT) {
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
        const int g = idx - kScalars;
        const int blk = g >> 4, e = g & 15;
        const int bj = packed_col(blk);
        const int bi = blk - bj * (bj + 1) / 2;
        const int i = 4 * bi + (e >> 2), j = 4 * bj + (e & 3);
        if (i <= j && j < n) {  // (split BF16: the other halves of the diagonal blocks differ)
          G0s[i * LD + j] = sum;
          G0s[j * LD + i] = sum;
        }
      }
    }
  }
#pragma unroll
  for (int q = 0; q < MF; ++q)
    if (tid + q * NT < nfull) V0s[fr[q] * LD + fc[q]] = vpre[q];
  __syncthreads();

  // 1. Control.
  if (tid == 0) {
    double t = 0.0;
    const int go = eigk::control_step(d, st, scal, kd, pf_nXF2, pf_tau, t);
    s_go = go;
    s_tau = t;
  }
  __syncthreads();
  if (!s_go) return;
  if (kd == 0 && !d.warm) shift = eig_shift(scal[2]);
  if (shift != 0) {
    for (int idx = tid; idx < NMAX * LD; idx += NT) G0s[idx] = ldexp(G0s[idx], -2 * shift);
    __syncthreads();
  }
  EIG_MARK(0);
  const double tau = ldexp(s_tau, -shift);
  int sweeps = 0;
  const gptr<T> Pd = as_global<T>(d.P);
  const int cur = eig_core<T, NMAX, NT>(
      sh, n, warm, tau, sweeps,
      [&](int i, int j, double v) {
        if (j < nb) {
          Pd[i * nb + j] = static_cast<T>(v);
          Pd[j * nb + i] = static_cast<T>(v);
        }
      },
      [&](int i) { (void)i; EIG_MARK(i); });
  const double* Vf = sh.V[cur];
#pragma unroll
  for (int q = 0; q < MF; ++q)
    if (tid + q * NT < nfull) d.V[fr[q] * nb + fc[q]] = Vf[fr[q] * LD + fc[q]];
  EIG_MARK(3);
  if (tid == 0) {
    int rank = 0;
    for (int k = 0; k < n; ++k) rank += sh.w[k] != 0.0 ? 1 : 0;
    st->rank = rank;
    st->sweeps = sweeps;
    st->sweeps_total += sweeps;
    st->iter = kd + 1;
  }
#undef EIG_MARK
}

}  // namespace

int eig_class(int n) {
  if (n <= kEigMaxN) return n <= 16 ? 16 : (n <= 32 ? 32 : 64);
  return n <= kEigWideMaxN ? kEigWideMaxN : (n <= kEigHugeMaxN ? kEigHugeMaxN : 0);
}

namespace {
// Threads per eigensolve workgroup, per [dtype][class 16/32/64].  Defaults
// from timing on MI355X: a round's work is spread over more waves as n grows.
std::atomic<int> g_eig_nt[2][3] = {{{256}, {512}, {1024}}, {{256}, {512}, {1024}}};
int cls_index(int ncls) { return ncls == 16 ? 0 : (ncls == 32 ? 1 : (ncls == 64 ? 2 : -1)); }
}  // namespace

bool eig_threads_valid(int ncls, int nt) {
  if (cls_index(ncls) < 0) return false;
  return nt == 256 || nt == 512 || (nt == 1024 && ncls >= 32);
}

int eig_threads(int dtype, int ncls) {
  const int c = cls_index(ncls);
  return c < 0 ? 0 : g_eig_nt[dtype == 0 ? 0 : 1][c].load(std::memory_order_relaxed);
}

bool set_eig_threads(int dtype, int ncls, int nt) {
  if (!eig_threads_valid(ncls, nt)) return false;
  g_eig_nt[dtype == 0 ? 0 : 1][cls_index(ncls)].store(nt, std::memory_order_relaxed);
  return true;
}

hipError_t launch_eig(int dtype, int ncls, int grid, hipStream_t stream, const SolveDesc* descs,
                      const int32_t* ids) {
  if (grid <= 0) return hipSuccess;
  const int nt = eig_threads(dtype, ncls);
  const dim3 g(grid), b(nt);
#define RPCA_EIG_CASE(N, NT)                                                  \
  if (ncls == N && nt == NT) {                                                \
    if (dtype == 0)                                                           \
      RPCA_LAUNCH((k_eig<double, N, NT>), g, b, 0, stream, descs, ids); \
    else                                                                      \
      RPCA_LAUNCH((k_eig<float, N, NT>), g, b, 0, stream, descs, ids);  \
    return hipGetLastError();                                                 \
  }
  RPCA_EIG_CASE(16, 256)
  RPCA_EIG_CASE(16, 512)
  RPCA_EIG_CASE(32, 256)
  RPCA_EIG_CASE(32, 512)
  RPCA_EIG_CASE(32, 1024)
  RPCA_EIG_CASE(64, 256)
  RPCA_EIG_CASE(64, 512)
  RPCA_EIG_CASE(64, 1024)
#undef RPCA_EIG_CASE
  return hipErrorInvalidValue;
}

}  // namespace rpca
