// Warm-started eigensolve of windows of 65 to 144 frames by simultaneous
// rotation steps, by a team of workgroups per solve.
//
// The method is that of the simultaneous steps in eig_core.h: all pairs of the
// nearly diagonal G~ = V^T G V are rotated at once through matrix products, and
// P = V Z V^T with Z the first-order expansion of the thresholding function at
// the diagonal of G~.  Here the matrices (up to 166 KB each) stay in the
// solve's workspace, that is in the L2, and every product runs on the f64
// matrix cores, 2 x 2 blocks of 16 x 16 per wave at a time:
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
// It also runs the first sweeps of a solve's first eigensolve.
//
// Bound: with one workgroup, by its CU's matrix cores: a product is 2 nb^3 FP64
// operations (307 GFLOP/s: 19 us at 144 frames, 9 us at 112), a launch has about
// ten, 220 (480) us at 100 (132) frames.  A team has one wave per 16 x 16 block
// of the widest phase: then a phase is one block's latency and the meeting after
// it, 6 to 8 us, and a launch 100 (125) us.  A launch of several solves divides
// kTeamGroups workgroups between them.  The blocks are computed alike however
// many workgroups there are, and products and sums are fused only where the code
// says so (the build's -ffp-contract=off), so the results have the same bits.
//
// A workgroup waits for its team at every meeting, for a bounded time (launch.h);
// then it gives up and the others follow at this meeting or a later one.  The
// Jacobi kernel, which runs after all of them have ended, advances the iteration
// and V where nobody gave up; else it ends the solve, and the host runs it again
// from its inputs with one workgroup (`alone`), which waits for nobody.
#include <algorithm>

#include "common.h"
#include "eig_common.h"
#include "launch.h"
#include "team.h"

namespace rpca {
namespace {

using namespace eigk;

typedef double d4 __attribute__((ext_vector_type(4)));

constexpr int kStepThreads = 512;
constexpr int kStepWaves = kStepThreads / 64;

// Workgroups of a team read what others of it wrote within the launch: such
// loads and stores go to the memory that all CUs share (relaxed atomics, agent
// scope), past the L2 of the CU's own XCD.
template <bool TEAM>
__device__ inline double ld(gptr<const double> p) {
  if constexpr (TEAM) return __hip_atomic_load((const double*)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else return *p;
}
template <bool TEAM, typename T>
__device__ inline void st_to(gptr<T> p, T v) {
  if constexpr (TEAM) __hip_atomic_store((T*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  else *p = v;
}

struct TeamCtl {  // one workgroup's view of its team (see team.h)
  WideCtl* ctl;
  int64_t until;
  __device__ void arrive() {
    __hip_atomic_fetch_add(&ctl->arrived, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ unsigned arrived() const {
    return __hip_atomic_load(&ctl->arrived, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __device__ bool lost() const {
    return __hip_atomic_load(&ctl->lost, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0u;
  }
  __device__ bool late() const { return wall_clock64() > until; }
  __device__ void lose() { __hip_atomic_store(&ctl->lost, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
};

// All workgroups of a team at a meeting, complete with `all` arrivals since the
// launch began: what any of them stored before is seen by all after.  False when
// one of them did not come in time (`ticks` of the 100 MHz wall clock).
template <bool TEAM>
__device__ inline bool meet(WideCtl* ctl, unsigned all, int64_t ticks, int* s_ok) {
  if constexpr (!TEAM) {
    __syncthreads();
    return true;
  } else {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's stores have left
    __syncthreads();
    if (threadIdx.x == 0) {
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      TeamCtl c{ctl, wall_clock64() + ticks};
      *s_ok = meet_team(c, all) ? 1 : 0;
    }
    __syncthreads();
    return *s_ok != 0;
  }
}

// Block (bi, bj) of X^T Y by one wave, every operand in flight at once (a
// team's waves have one block each; the loads' latency is paid once).
__device__ inline d4 block1(const double* Xp, const double* Yp, int nb, int bi, int bj) {
  constexpr int C = kEigHugeMaxN / 16;
  const int l = threadIdx.x & 63, lr = l >> 4, lc = l & 15, nt = nb >> 4;
  const gptr<const double> x = as_global<double>(static_cast<const void*>(Xp + lr * nb + 16 * bi + lc));
  const gptr<const double> y = as_global<double>(static_cast<const void*>(Yp + lr * nb + 16 * bj + lc));
  double a[C][4], b[C][4];
#pragma unroll
  for (int c = 0; c < C; ++c)
    if (c < nt) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        a[c][k] = ld<true>(x + (16 * c + 4 * k) * nb);
        b[c][k] = ld<true>(y + (16 * c + 4 * k) * nb);
      }
    }
  d4 s = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
  for (int c = 0; c < C; ++c)
    if (c < nt) {
#pragma unroll
      for (int k = 0; k < 4; ++k) s = __builtin_amdgcn_mfma_f64_16x16x4f64(a[c][k], b[c][k], s, 0, 0, 0);
    }
  return s;
}

// The 2 x 2 blocks (bi + p, bj + q) of X^T Y into s[p][q]; blocks past the last
// row or column (or, SYM, below the diagonal) are skipped.  A operand lane l =
// X entry (l / 16, l % 16), B operand lane l = Y entry (l / 16, l % 16) of a
// step's four rows; result lane l, register r = entry (l / 16 + 4r, l % 16).
// Both operands read 128 contiguous bytes per row, and four loads of 512 B feed
// four products of 64 cycles.
template <bool SYM>
__device__ inline void blocks4(const double* Xp, const double* Yp, int nb, int bi, int bj, d4 (&s)[2][2]) {
  const int l = threadIdx.x & 63, lr = l >> 4, lc = l & 15, last = (nb >> 4) - 1;
  gptr<const double> x[2], y[2];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    x[p] = as_global<double>(static_cast<const void*>(Xp + lr * nb + 16 * min(bi + p, last) + lc));
    y[p] = as_global<double>(static_cast<const void*>(Yp + lr * nb + 16 * min(bj + p, last) + lc));
#pragma unroll
    for (int q = 0; q < 2; ++q) s[p][q] = d4{0.0, 0.0, 0.0, 0.0};
  }
  const bool row1 = bi < last && !(SYM && bi + 1 > bj + 1), col1 = bj < last;
  const bool both = row1 && col1, low = row1 && !(SYM && bi + 1 > bj);
  const int dk = 4 * nb;
#pragma unroll 1
  for (int k0 = 0; k0 < nb; k0 += 16) {
    double a[2][4], b[2][4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
#pragma unroll
      for (int p = 0; p < 2; ++p) {
        a[p][k] = x[p][k * dk];
        b[p][k] = y[p][k * dk];
      }
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      x[p] += 4 * dk;
      y[p] += 4 * dk;
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) s[0][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[0][k], b[0][k], s[0][0], 0, 0, 0);
    if (col1) {
#pragma unroll
      for (int k = 0; k < 4; ++k) s[0][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[0][k], b[1][k], s[0][1], 0, 0, 0);
    }
    if (low) {
#pragma unroll
      for (int k = 0; k < 4; ++k) s[1][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[1][k], b[0][k], s[1][0], 0, 0, 0);
    }
    if (both) {
#pragma unroll
      for (int k = 0; k < 4; ++k) s[1][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[1][k], b[1][k], s[1][1], 0, 0, 0);
    }
  }
}

// Every block of X^T Y (SYM: the upper ones), in units of 2 x 2 blocks or, in a
// team, single ones: the units u, u + nw, ... of this wave (nw: waves of the
// solve).  `u` is advanced past the product's units, so that two products with
// no barrier between them share the waves evenly.  out(bi, bj, block) is called
// for each 16 x 16 block.
template <bool TEAM, bool SYM, typename Out>
__device__ inline void product(int& u, int nw, const double* X, const double* Y, int nb, Out&& out) {
  const int nt = nb >> 4, n2 = TEAM ? nt : (nt + 1) >> 1;
  const int units = SYM ? n2 * (n2 + 1) / 2 : n2 * n2;
  for (; u < units; u += nw) {
    const int uj = SYM ? packed_col(u) : u % n2, ui = SYM ? u - uj * (uj + 1) / 2 : u / n2;
    if constexpr (TEAM) {
      out(ui, uj, block1(X, Y, nb, ui, uj));
    } else {
      const int bi = 2 * ui, bj = 2 * uj;
      d4 s[2][2];
      blocks4<SYM>(X, Y, nb, bi, bj, s);
#pragma unroll
      for (int p = 0; p < 2; ++p)
#pragma unroll
        for (int q = 0; q < 2; ++q)
          if (bi + p < nt && bj + q < nt && !(SYM && bi + p > bj + q)) out(bi + p, bj + q, s[p][q]);
    }
  }
  u -= units;
}

// One lane's entries of a 16 x 16 block and their transposes, through the
// wave's own LDS buffer (16 rows of 17): a transposed block is then stored in
// rows of 128 bytes too, instead of 64 scattered entries per store.
constexpr int kTrLd = 17;
__device__ inline d4 transposed(const d4& v, double* tb) {
  const int l = threadIdx.x & 63, lr = l >> 4, lc = l & 15;
  d4 t;
#pragma unroll
  for (int r = 0; r < 4; ++r) tb[(lr + 4 * r) * kTrLd + lc] = v[r];
  __builtin_amdgcn_wave_barrier();  // LDS operations of a wave complete in order
#pragma unroll
  for (int r = 0; r < 4; ++r) t[r] = tb[lc * kTrLd + lr + 4 * r];
  __builtin_amdgcn_wave_barrier();
  return t;
}
template <bool TEAM, typename T>
__device__ inline void store_block(T* M, int nb, int bi, int bj, const d4& v) {
  const int l = threadIdx.x & 63, lr = l >> 4, lc = l & 15;
  const gptr<T> p = as_global<T>(static_cast<void*>(M + (16 * bi + lr) * nb + 16 * bj + lc));
#pragma unroll
  for (int r = 0; r < 4; ++r) st_to<TEAM>(p + 4 * r * nb, static_cast<T>(v[r]));
}
// Upper block (bi, bj) of a symmetric matrix h + k with h symmetric and k
// antisymmetric (entries of h, k; k may be zero), and its mirror image h - k.
// On the diagonal the entries above it decide both.
template <bool TEAM, typename T>
__device__ inline void store_mirrored(T* M, int nb, int bi, int bj, const d4& h, const d4& k, double* tb) {
  const d4 lo = transposed(h - k, tb);
  if (bi != bj) {
    store_block<TEAM>(M, nb, bi, bj, h + k);
    store_block<TEAM>(M, nb, bj, bi, lo);
  } else {
    const int l = threadIdx.x & 63, lr = l >> 4, lc = l & 15;
    d4 v;
#pragma unroll
    for (int r = 0; r < 4; ++r) v[r] = lr + 4 * r <= lc ? h[r] + k[r] : lo[r];
    store_block<TEAM>(M, nb, bi, bj, v);
  }
}
template <bool TEAM>
__device__ inline d4 load_block(const double* M, int nb, int bi, int bj) {
  const int l = threadIdx.x & 63, lr = l >> 4, lc = l & 15;
  const gptr<const double> p =
      as_global<double>(static_cast<const void*>(M + (16 * bi + lr) * nb + 16 * bj + lc));
  d4 v;
#pragma unroll
  for (int r = 0; r < 4; ++r) v[r] = ld<TEAM>(p + 4 * r * nb);
  return v;
}

template <typename T, bool TEAM>
__global__ void __launch_bounds__(kStepThreads)
k_eig_steps(const SolveDesc* __restrict__ descs, const int32_t* __restrict__ ids, int64_t ticks) {
  __shared__ double dg[kEigHugeMaxN], sg[kEigHugeMaxN], rg[kEigHugeMaxN], w[kEigHugeMaxN], sd[kEigHugeMaxN];
  __shared__ double tbuf[kStepWaves][16 * kTrLd];
  __shared__ double scal[kScalars];
  __shared__ unsigned mx[2][4];
  __shared__ int s_go, s_ok;
  __shared__ double s_tau;
  const int tid = threadIdx.x;
  const SolveDesc& d = descs[ids[blockIdx.y]];
  SolveState* st = d.st;
  // a solve's first eigensolve begins with the Jacobi kernel's sweeps
  if (st->done || (st->iter == 0 && WideEig(d).ctl->ready == 0u)) return;
#ifdef RPCA_TRACE
  int64_t tprev = RPCA_NOW();
#define STEP_MARK(i)                              \
  do {                                            \
    if (tid == 0 && blockIdx.x == 0) {            \
      const int64_t tnow_ = RPCA_NOW();           \
      st->trace[i] += tnow_ - tprev;              \
      tprev = tnow_;                              \
    }                                             \
  } while (0)
#else
#define STEP_MARK(i) \
  do {               \
  } while (0)
#endif
  const WideEig e(d);
  const int n = d.n, nb = d.nb, kd = st->iter;
  double pf_nXF2 = 0.0, pf_tau = 0.0;
  const int shift = eig_shift(st->nXF2);
  // workgroup g of the solve's team; thread and wave of the whole team
  const int g = TEAM ? blockIdx.x : 0;
  const int teams = TEAM && !d.alone ? gridDim.x : 1;
  if (g >= teams) return;
  const int nw = teams * kStepWaves, gtid = g * kStepThreads + tid;
  unsigned all = 0;  // arrivals that complete the next meeting
  if (tid == 0 && g == 0) {
    pf_nXF2 = st->nXF2;
    pf_tau = st->tau;
    e.ctl->booked = 0;
  }
  // read before the first meeting (workgroup 0 writes them after the last)
  const int v0 = e.ctl->vsel;

  // Sum of the group partials in group order; the Gram into both halves of G.
  {
    const int nent = kScalars + gram_blocks((n + 3) >> 2) * 16;
    constexpr int kChunk = 16;
    for (int idx = gtid; idx < nent; idx += teams * kStepThreads) {
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
        sum = ldexp(sum, -2 * shift);
        const int g = idx - kScalars, blk = g >> 4, el = g & 15;
        const int bj = packed_col(blk), bi = blk - bj * (bj + 1) / 2;
        const int i = 4 * bi + (el >> 2), j = 4 * bj + (el & 3);
        if (i <= j && j < n) {
          st_to<TEAM>(as_global<double>(static_cast<void*>(e.G + i * nb + j)), sum);
          st_to<TEAM>(as_global<double>(static_cast<void*>(e.G + j * nb + i)), sum);
        }
      }
    }
  }
  if (tid < 8) mx[tid >> 2][tid & 3] = 0u;
  if (!meet<TEAM>(e.ctl, all += teams, ticks, &s_ok)) return;
  if (tid == 0 && g == 0) {  // its scalars are this workgroup's own
    double t = pf_tau;
    s_go = kd == 0 ? 1 : control_step(d, st, scal, kd, pf_nXF2, pf_tau, t);  // kd = 0: done there
    s_tau = t;
    if constexpr (TEAM) {
      __hip_atomic_store(&e.ctl->tau, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&e.ctl->go, static_cast<uint32_t>(s_go), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  if constexpr (!TEAM) {
    __syncthreads();
    if (!s_go) return;
  }
  STEP_MARK(0);
  const int wv = __builtin_amdgcn_readfirstlane(tid >> 6), gw = g * kStepWaves + wv;
  const int l = tid & 63, lr = l >> 4, lc = l & 15, nt = nb >> 4;
  double* tb = tbuf[wv];
  const d4 zero = {0.0, 0.0, 0.0, 0.0};
  auto put = [&](double* M) { return [M, nb](int bi, int bj, const d4& v) { store_block<TEAM>(M, nb, bi, bj, v); }; };
  auto put_sym = [&](double* M) {
    return [=](int bi, int bj, const d4& v) { store_mirrored<TEAM>(M, nb, bi, bj, v, zero, tb); };
  };

  // W = G V (G symmetric), S = V^T W, C = V^T V (C: upper blocks only)
  const double* V = e.v(v0);
  int u = gw;
  product<TEAM, false>(u, nw, e.G, V, nb, put(e.W));
  if (!meet<TEAM>(e.ctl, all += teams, ticks, &s_ok)) return;
  if constexpr (TEAM) {
    if (tid == 0) {
      s_tau = __hip_atomic_load(&e.ctl->tau, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s_go = static_cast<int>(__hip_atomic_load(&e.ctl->go, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
    }
    __syncthreads();
    if (!s_go) return;
  }
  const double tau = ldexp(s_tau, -shift);
  u = gw;
  product<TEAM, true>(u, nw, V, e.W, nb, put_sym(e.S));
  product<TEAM, true>(u, nw, V, V, nb, put(e.C));
  // V^T, for the products with V as the left factor (or V^T as the right one)
  for (int t = gw; t < nt * nt; t += nw) {
    const int bi = t / nt, bj = t - bi * nt;
    store_block<TEAM>(e.vt(0), nb, bj, bi, transposed(load_block<TEAM>(V, nb, bi, bj), tb));
  }
  if (!meet<TEAM>(e.ctl, all += teams, ticks, &s_ok)) return;

  STEP_MARK(2);
  int s = 0;
  bool ok = false;
  for (;; ++s) {
    unsigned* mp = mx[s & 1];
    if (tid < n) {
      const double sii = ld<TEAM>(as_global<double>(static_cast<const void*>(e.S + tid * (nb + 1))));
      const double m = ld<TEAM>(as_global<double>(static_cast<const void*>(e.C + tid * (nb + 1)))) - 1.0;
      const double di = fma(-m, sii, sii), ri = rsqrt_or_zero(di), si = di * ri;
      const double wi = si <= tau ? 0.0 : fma(-tau, ri, 1.0);
      sd[tid] = sii;
      dg[tid] = di;
      sg[tid] = si;
      rg[tid] = ri;
      w[tid] = wi;
    }
    __syncthreads();
    float mz = 0.0f, mk = 0.0f, mm = 0.0f, mt = 0.0f;
    for (int t = gw; t < nt * (nt + 1) / 2; t += nw) {
      const int bj = packed_col(t), bi = t - bj * (bj + 1) / 2;
      const d4 cb = load_block<TEAM>(e.C, nb, bi, bj), sb = load_block<TEAM>(e.S, nb, bi, bj);
      const int j = 16 * bj + lc;
      d4 z = zero, k = zero;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int i = 16 * bi + lr + 4 * r;
        if (i > j || j >= n) continue;
        if (i == j) {
          const double m = cb[r] - 1.0;
          z[r] = fma(-m, w[i], w[i]);
          mm = fmaxf(mm, cb[r] == cb[r] ? fabsf(static_cast<float>(m)) : INFINITY);
        } else {
          const double el = fma(-0.5 * cb[r], sd[i] + sd[j], sb[r]);
          const PairTerms pt = pair_terms<T>(el, dg[i], dg[j], sg[i], sg[j], rg[i], rg[j], w[i], w[j], tau, n);
          z[r] = fma(-0.5 * cb[r], w[i] + w[j], pt.z);
          k[r] = pt.t;
          mz = fmaxf(mz, pt.mz);
          mk = fmaxf(mk, pt.kappa);
          mt = fmaxf(mt, fabsf(static_cast<float>(pt.t)));
          mm = fmaxf(mm, fabsf(static_cast<float>(cb[r])));
        }
      }
      store_mirrored<TEAM>(e.Z, nb, bi, bj, z, zero, tb);
      store_mirrored<TEAM>(e.K, nb, bi, bj, zero, k, tb);
    }
    wave_max_to(mz, &mp[0]);
    wave_max_to(mk, &mp[1]);
    wave_max_to(mm, &mp[2]);
    wave_max_to(mt, &mp[3]);
    if constexpr (TEAM) {
      __syncthreads();
      unsigned* top = e.ctl->mx[s];
      if (tid < 4 && mp[tid] != 0u)
        __hip_atomic_fetch_max(&top[tid], mp[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (!meet<TEAM>(e.ctl, all += teams, ticks, &s_ok)) return;
      if (tid < 4) mp[tid] = __hip_atomic_load(&top[tid], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    mz = __uint_as_float(mp[0]);
    mk = __uint_as_float(mp[1]);
    mm = __uint_as_float(mp[2]);
    mt = __uint_as_float(mp[3]);
    if (tid < 4) mx[(s + 1) & 1][tid] = 0u;  // last read before the barrier above
    STEP_MARK(1);
    if (!(mm < kOrthMax)) break;
    ok = static_cast<float>(n) * fmaxf(mz, mm) * fmaxf(mk, mm) < PTarget<T>::value;
    if (ok || s == kWideSteps) break;

    // U = I + K + T/2 - M/2, T = K^2 = -K^T K (to fourth order for large K)
    auto eye = [&](int bi, int bj) {  // I - M/2
      d4 h = zero;
      const d4 c = load_block<TEAM>(e.C, nb, bi, bj);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const double id = bi == bj && lr + 4 * r == lc ? 1.0 : 0.0;
        h[r] = 16 * bj + lc < n ? fma(-0.5, c[r] - id, id) : id;
      }
      return h;
    };
    u = gw;
    if (!(mt > kWideFourth)) {
      product<TEAM, true>(u, nw, e.K, e.K, nb, [&](int bi, int bj, const d4& v) {
        store_mirrored<TEAM>(e.U, nb, bi, bj, eye(bi, bj) - 0.5 * v, load_block<TEAM>(e.K, nb, bi, bj), tb);
      });
    } else {
      product<TEAM, true>(u, nw, e.K, e.K, nb,
                    [&](int bi, int bj, const d4& v) { store_mirrored<TEAM>(e.T, nb, bi, bj, -v, zero, tb); });
      if (!meet<TEAM>(e.ctl, all += teams, ticks, &s_ok)) return;
      // K T = -K^T T into W, then T^2 and U (a block of both has one owner)
      u = gw;
      product<TEAM, true>(u, nw, e.K, e.T, nb, [&](int bi, int bj, const d4& v) { store_block<TEAM>(e.W, nb, bi, bj, -v); });
      u = gw;
      product<TEAM, true>(u, nw, e.T, e.T, nb, [&](int bi, int bj, const d4& v) {
        const d4 h = eye(bi, bj) + 0.5 * load_block<TEAM>(e.T, nb, bi, bj) + v * (1.0 / 24.0);
        const d4 k = load_block<TEAM>(e.K, nb, bi, bj) + load_block<TEAM>(e.W, nb, bi, bj) * (1.0 / 6.0);
        store_mirrored<TEAM>(e.U, nb, bi, bj, h, k, tb);
      });
    }
    if (!meet<TEAM>(e.ctl, all += teams, ticks, &s_ok)) return;
    // W = S U, V' = V U (and its transpose);  S = U^T W, C = V'^T V'
    double* Vn = e.v(WideEig::vsel(v0, s + 1));
    u = gw;
    product<TEAM, false>(u, nw, e.S, e.U, nb, put(e.W));
    product<TEAM, false>(u, nw, e.vt(s & 1), e.U, nb, [&](int bi, int bj, const d4& v) {
      store_block<TEAM>(Vn, nb, bi, bj, v);
      store_block<TEAM>(e.vt((s + 1) & 1), nb, bj, bi, transposed(v, tb));
    });
    V = Vn;
    if (!meet<TEAM>(e.ctl, all += teams, ticks, &s_ok)) return;
    u = gw;
    product<TEAM, true>(u, nw, e.U, e.W, nb, put_sym(e.S));
    product<TEAM, true>(u, nw, V, V, nb, put(e.C));
    if (!meet<TEAM>(e.ctl, all += teams, ticks, &s_ok)) return;
    STEP_MARK(2);
  }
  if (!ok) return;  // the Jacobi kernel takes over, from V at v0

  // P = V (Z V^T) (exactly symmetric)
  const double* Vt = e.vt(s & 1);
  u = gw;
  product<TEAM, false>(u, nw, e.Z, Vt, nb, put(e.W));
  if (!meet<TEAM>(e.ctl, all += teams, ticks, &s_ok)) return;
  u = gw;
  product<TEAM, true>(u, nw, Vt, e.W, nb, [&](int bi, int bj, const d4& v) {
    store_mirrored<false>(static_cast<T*>(d.P), nb, bi, bj, v, zero, tb);
  });
  const int rank = __syncthreads_count(tid < n && w[tid] != 0.0);
  if (tid == 0 && g == 0) {
    // the Jacobi kernel makes it this iteration's, if it stands
    e.ctl->vnext = WideEig::vsel(v0, s);
    e.ctl->booked = kd + 1;
    st->rank = rank;
    st->sweeps = 0;
#ifdef RPCA_TRACE
    st->sweeps_total += s;
#endif
  }
  STEP_MARK(3);
#undef STEP_MARK
}

}  // namespace

// One wave per block of the widest phase (W and V', 2 (nb/16)^2 blocks), as long
// as the launch stays within kTeamGroups workgroups: a CU holds one of them, so
// the launches of six streams at once (the server's) are all resident or will
// be, whatever order their workgroups are placed in.  Fewer workgroups per
// solve are slower in step (100 frames, small images, us per iteration: 205 for
// one solve, 275 for 6, 342 for 16, 511 for 32 on four streams), one per solve
// is the least.
constexpr int kTeamGroups = 42;
int steps_team(int nb, int grid) {
  const int nt = nb / 16, most = (2 * nt * nt + kStepWaves - 1) / kStepWaves;
  return std::max(1, std::min(most, kTeamGroups / std::max(grid, 1)));
}

hipError_t launch_eig_steps(int dtype, int grid, int team, hipStream_t stream, const SolveDesc* descs,
                            const int32_t* ids) {
  if (grid <= 0) return hipSuccess;
  const dim3 g(team, grid), b(kStepThreads);
  if (dtype == 1 && team > 1)
    RPCA_LAUNCH((k_eig_steps<float, true>), g, b, 0, stream, descs, ids, t_limits.wait_ticks);
  else if (dtype == 1)
    RPCA_LAUNCH((k_eig_steps<float, false>), g, b, 0, stream, descs, ids, t_limits.wait_ticks);
  else if (team > 1)
    RPCA_LAUNCH((k_eig_steps<double, true>), g, b, 0, stream, descs, ids, t_limits.wait_ticks);
  else
    RPCA_LAUNCH((k_eig_steps<double, false>), g, b, 0, stream, descs, ids, t_limits.wait_ticks);
  return hipGetLastError();
}

}  // namespace rpca
