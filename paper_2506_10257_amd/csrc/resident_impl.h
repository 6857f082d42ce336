// One whole solve in one launch, its rows in registers.
//
// A window of up to 32 frames whose X, S and Y fit the register files of the
// chip (134 MB; 512 x 512 x 20 in FP32 takes 63 MB) needs no memory traffic
// between iterations but the reduction of its Gram partials.  Each workgroup
// (one per CU at most) keeps up to four 256-row tiles, one thread per row, and
// runs every iteration: eigensolve, update of its rows, Gram partial, all-to-all
// sum.  The eigensolve runs in every workgroup, on the same sums, so its
// projector needs no broadcast and V never leaves the LDS.  At 512 x 512 x 20
// an iteration of the launched path (eigensolve, update, reduction) is bound by
// the update's 105 MB (27 us), three launches and the eigensolve in series; here
// the update is the arithmetic of 1024 rows per CU.
//
// Sum across workgroups: two hops through memory, no fences.  Every 8-byte word
// carries 32 bits of a double and the sequence number of the exchange, is
// written by one relaxed agent-scope store (which goes through to memory) and
// polled by relaxed agent-scope loads, so a word is valid as soon as its number
// is right and nothing else has to be ordered:
//   1. workgroup w writes each entry of its partial (Gram blocks, residual);
//   2. workgroup e adds entry e (and e + grid, ...) over all workgroups, in the
//      order of k_reduce_groups and k_eig, and writes the sum;
//   3. every workgroup reads all sums.
// One buffer per hop is enough: a workgroup writes its next partial only after
// it has every sum, that is after every partial of this exchange was read, and
// writes a next sum only after every partial of the next exchange is there,
// that is after every workgroup has read the sums of this one.
//
// Every wait ends: the grid has at most one workgroup per CU, but nothing
// guarantees that all of them run at once (another process, other streams), so
// a wait is bounded by the wall clock.  A workgroup that gives up leaves the
// kernel; the others then give up as well, and the caller runs the launched
// path from the unchanged inputs.
//
// Bound by latency: at 512 x 512 x 20 FP32 an iteration takes 37 us (launched,
// with the same eigensolver, 49): eigensolve 9, update 6.0, Gram 8.2, partial
// 3.8, first hop and sum 6.4, second hop 2.7; at 128 x 128 x 20 FP64 25 us (39):
// 11.3, 3.1, 1.9, 1.5, 4.7, 2.6.
//
// The arithmetic is that of k_stream, k_reduce_groups and k_eig operation for
// operation, so the results are bitwise those of the launched path.
#pragma once

#include "common.h"
#include "eig_core.h"
#include "launch.h"
#include "stream_impl.h"

namespace rpca {
namespace {

__device__ inline void ll_store(uint64_t* cell, uint32_t seq, double v) {
  const uint64_t b = __builtin_bit_cast(uint64_t, v), s = static_cast<uint64_t>(seq) << 32;
  __hip_atomic_store(cell, s | (b & 0xffffffffu), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  __hip_atomic_store(cell + 1, s | (b >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// False when the time is over (ticks < 0: after one look).
__device__ inline bool ll_wait(const uint64_t* cell, uint32_t seq, int64_t ticks, double& v) {
  const int64_t until = wall_clock64() + ticks;
  const int most = ticks < 0 ? 1 : 64;
  for (;;) {
#pragma unroll 1
    for (int tries = 0; tries < most; ++tries) {
      const uint64_t a = __hip_atomic_load(cell, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const uint64_t b = __hip_atomic_load(cell + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if ((a >> 32) == seq && (b >> 32) == seq) {
        v = __builtin_bit_cast(double, (b << 32) | (a & 0xffffffffu));
        return true;
      }
    }
    if (wall_clock64() > until) return false;
  }
}

// l[k] += p_k a for k < BLK, where lane k of each row of 16 lanes of p holds
// p_k: a broadcast inside the FMA (DPP row_newbcast), so the projector costs no
// instruction beside the FMAs.  With scalar loads, as in k_stream, the scalar
// cache would have to be invalidated every iteration; through v_readlane the
// update took 10.4 us at 512 x 512 x 20.  (s_nop: two wait states between a
// write of p and its DPP use; the sums are written before the last read of p and a.)
template <int BLK, typename T>
__device__ inline void fma_row(T* l, T p, T a) {
  static_assert(BLK == 8 || BLK == 10, "columns per row of P");
  if constexpr (sizeof(T) == 4) {
    if constexpr (BLK == 8) {
      asm("s_nop 1\n\t"
          "v_fmac_f32_dpp %0, %8, %9 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f32_dpp %1, %8, %9 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f32_dpp %2, %8, %9 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f32_dpp %3, %8, %9 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f32_dpp %4, %8, %9 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f32_dpp %5, %8, %9 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f32_dpp %6, %8, %9 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f32_dpp %7, %8, %9 row_newbcast:7 row_mask:0xf bank_mask:0xf\n\t"
          : "+&v"(l[0]), "+&v"(l[1]), "+&v"(l[2]), "+&v"(l[3]), "+&v"(l[4]), "+&v"(l[5]), "+&v"(l[6]), "+&v"(l[7])
          : "v"(p), "v"(a));
    } else {
      asm("s_nop 1\n\t"
          "v_fmac_f32_dpp %0, %10, %11 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f32_dpp %1, %10, %11 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f32_dpp %2, %10, %11 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f32_dpp %3, %10, %11 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f32_dpp %4, %10, %11 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f32_dpp %5, %10, %11 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f32_dpp %6, %10, %11 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f32_dpp %7, %10, %11 row_newbcast:7 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f32_dpp %8, %10, %11 row_newbcast:8 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f32_dpp %9, %10, %11 row_newbcast:9 row_mask:0xf bank_mask:0xf\n\t"
          : "+&v"(l[0]), "+&v"(l[1]), "+&v"(l[2]), "+&v"(l[3]), "+&v"(l[4]), "+&v"(l[5]), "+&v"(l[6]), "+&v"(l[7]), "+&v"(l[8]), "+&v"(l[9])
          : "v"(p), "v"(a));
    }
  } else {
    if constexpr (BLK == 8) {
      asm("s_nop 1\n\t"
          "v_fmac_f64_dpp %0, %8, %9 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f64_dpp %1, %8, %9 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f64_dpp %2, %8, %9 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f64_dpp %3, %8, %9 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f64_dpp %4, %8, %9 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f64_dpp %5, %8, %9 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f64_dpp %6, %8, %9 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f64_dpp %7, %8, %9 row_newbcast:7 row_mask:0xf bank_mask:0xf\n\t"
          : "+&v"(l[0]), "+&v"(l[1]), "+&v"(l[2]), "+&v"(l[3]), "+&v"(l[4]), "+&v"(l[5]), "+&v"(l[6]), "+&v"(l[7])
          : "v"(p), "v"(a));
    } else {
      asm("s_nop 1\n\t"
          "v_fmac_f64_dpp %0, %10, %11 row_newbcast:0 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f64_dpp %1, %10, %11 row_newbcast:1 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f64_dpp %2, %10, %11 row_newbcast:2 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f64_dpp %3, %10, %11 row_newbcast:3 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f64_dpp %4, %10, %11 row_newbcast:4 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f64_dpp %5, %10, %11 row_newbcast:5 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f64_dpp %6, %10, %11 row_newbcast:6 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f64_dpp %7, %10, %11 row_newbcast:7 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f64_dpp %8, %10, %11 row_newbcast:8 row_mask:0xf bank_mask:0xf\n\t"
          "v_fmac_f64_dpp %9, %10, %11 row_newbcast:9 row_mask:0xf bank_mask:0xf\n\t"
          : "+&v"(l[0]), "+&v"(l[1]), "+&v"(l[2]), "+&v"(l[3]), "+&v"(l[4]), "+&v"(l[5]), "+&v"(l[6]), "+&v"(l[7]), "+&v"(l[8]), "+&v"(l[9])
          : "v"(p), "v"(a));
    }
  }
}

// NB: frames in registers (n <= NB); NT: threads, 256 per tile.
template <typename T, int NB, int NT>
__global__ void __launch_bounds__(NT)
k_resident(const SolveDesc d, const ResidentBuf rb) {
  constexpr int NMAX = NB <= 16 ? 16 : 32;
  constexpr int LD = eig_ld(NMAX);
  constexpr int TPW = NT / 256;
  constexpr int NB4 = (NB + 3) / 4 * 4;
  constexpr int LDT = kTile + 1;
  constexpr size_t kTileBytes = sizeof(T) * NB4 * LDT;
  constexpr size_t kRedBytes = sizeof(double) * gram_red_doubles(NB);
  constexpr size_t kQuarter = ((kTileBytes > kRedBytes ? kTileBytes : kRedBytes) + 15) / 16 * 16;
  constexpr int NENT = kScalars + gram_blocks(NB4 / 4) * 16;
  constexpr int BLK = NB % 10 == 0 ? 10 : 8;  // columns of P per row of 16 lanes
  constexpr int NBL = NB / BLK;
  // Where the registers do not hold X, Y, A and the eigensolve's working set,
  // Y waits in the tile's LDS during the eigensolve and X is read again after
  // it (from the L2 as a rule: 82 KB per CU, about 1 us).
  constexpr bool SLIM = NT == 1024 || NB * sizeof(T) >= 128;
  static_assert(kQuarter * TPW >= 2 * NT * sizeof(double), "exchange staging");
  __shared__ __align__(16) unsigned char smem[kQuarter * TPW];
  __shared__ EigLds<NMAX> eig;
  __shared__ double wred[NT / 64][kScalars];
  __shared__ double part[TPW][NENT];  // the tiles' partials
  __shared__ double sums[NENT];
  __shared__ T Ps[NB * NBL * 16];  // P(i, j) at ((i * NBL) + j / BLK) * 16 + j % BLK
  __shared__ SolveState st;
  __shared__ int s_go, s_lost;
  __shared__ double s_tau;

  const int tid = threadIdx.x, q = tid >> 8, t = tid & 255;
  const int n = d.n, grid = gridDim.x, tpw = rb.tpw;
  const int64_t m = d.m;
  const int tile = blockIdx.x * tpw + q;
  const bool act = q < tpw && tile < d.tiles;  // uniform over the 256 threads of a tile
  const uint32_t p = static_cast<uint32_t>(tile) * kTile + t;
  const bool valid = act && p < m;
  T* const tileA = reinterpret_cast<T*>(smem + kQuarter * q);
  double* const vals = reinterpret_cast<double*>(smem);
  double* const gsum = vals + NT;

#ifdef RPCA_TRACE
  int64_t tprev = RPCA_NOW();
#define RES_MARK(i)                       \
  do {                                    \
    if (threadIdx.x == 0) {               \
      const int64_t tnow_ = RPCA_NOW();   \
      if (i >= 0) st.trace[i] += tnow_ - tprev; \
      tprev = tnow_;                      \
    }                                     \
  } while (0)
#else
#define RES_MARK(i) \
  do {              \
  } while (0)
#endif
  // LDS matrices zero outside n x n, V the identity
  for (int i = tid; i < 2 * NMAX * LD; i += NT) {
    (&eig.G[0][0])[i] = 0.0;
    (&eig.V[0][0])[i] = 0.0;
  }
  if (tid == 0) {
    SolveState z{};
    st = z;
    s_lost = 0;
  }
  __syncthreads();
  if (tid < n) eig.V[0][tid * LD + tid] = 1.0;

  const int nblk = gram_blocks((n + 3) >> 2), nent = kScalars + nblk * 16;
  const int C = gram_chunks(nblk), Gq = gram_lane_group(C), Q = C / Gq;

  // The tile in LDS (A', frame-major) and the scalars -> sums over the solve
  // (false: gave up).
  uint32_t seq = 0;
  auto exchange = [&](auto norms, double r2, double s1, double s2, double nf) {
    ++seq;
    int tid = threadIdx.x;  // not hoisted out of the iterations, as in eig_core
    asm volatile("" : "+v"(tid));
    const int q = tid >> 8, t = tid & 255;
    const int gblk = t / C, gc = t - gblk * C;
    const bool gact = act && gblk < nblk;
    const int bj = gact ? packed_col(gblk) : 0, bi = gact ? gblk - bj * (bj + 1) / 2 : 0;
    T* const tileA = reinterpret_cast<T*>(smem + kQuarter * q);
    double* const red = reinterpret_cast<double*>(smem + kQuarter * q);
    double gacc[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) gacc[e] = 0.0;
    __syncthreads();
    if (gact) {
      const T* u = tileA + (4 * bi) * LDT;
      const T* v = tileA + (4 * bj) * LDT;
      for (int r = gc; r < kTile; r += C) {
        double ue[4], vf[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          ue[e] = static_cast<double>(u[e * LDT + r]);
          vf[e] = static_cast<double>(v[e * LDT + r]);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int f = 0; f < 4; ++f) gacc[e * 4 + f] = fma(ue[e], vf[f], gacc[e * 4 + f]);
      }
    }
    __syncthreads();
    RES_MARK(2);
    // r2 is zero in the first pass, the norms of X in all others
    double sc[kScalars] = {r2, s1, s2, nf};
    if constexpr (decltype(norms)::value) {
#pragma unroll
      for (int s = 1; s < kScalars; ++s) sc[s] = wave_sum(sc[s]);
    } else {
      sc[0] = wave_sum(sc[0]);
    }
    if ((tid & 63) == 0) {
#pragma unroll
      for (int s = 0; s < kScalars; ++s) wred[tid >> 6][s] = sc[s];
    }
    if (Gq >= 2) {
#pragma unroll
      for (int e = 0; e < 16; ++e) gacc[e] += quad_swap<kQuadXor1>(gacc[e]);
      if (Gq == 4) {
#pragma unroll
        for (int e = 0; e < 16; ++e) gacc[e] += quad_swap<kQuadXor2>(gacc[e]);
      }
    }
    if (gact && (gc & (Gq - 1)) == 0) {
      double* dst = red + (gblk * Q + gc / Gq) * kRedLd;
#pragma unroll
      for (int e = 0; e < 16; ++e) dst[e] = gacc[e];
    }
    __syncthreads();
    for (int idx = t; idx < nblk * 16; idx += 256) {
      double s = 0.0;
      if (act) {
        const double* src = red + (idx >> 4) * Q * kRedLd + (idx & 15);
#pragma unroll 4
        for (int c = 0; c < Q; ++c) s += src[c * kRedLd];
      }
      part[q][kScalars + idx] = s;
    }
    if (t < kScalars) {
      double s = wred[4 * q][t];
#pragma unroll
      for (int w = 1; w < 4; ++w) s += wred[4 * q + w][t];
      part[q][t] = act ? s : 0.0;
    }
    __syncthreads();
    // 1. this workgroup's tiles (missing ones are zero), summed as quads are
    for (int e = tid; e < nent; e += NT) {
      double v = part[0][e];
      if constexpr (TPW >= 2) {
        if (tpw >= 2) v += part[1][e];
      }
      if constexpr (TPW == 4) {
        if (tpw == 4) v += part[2][e] + part[3][e];
      }
      ll_store(rb.parts + 2 * (static_cast<size_t>(e) * grid + blockIdx.x), seq, v);
    }
    RES_MARK(3);
    // 2. entries blockIdx.x, blockIdx.x + grid, ...: `per` of them at a time
    const int64_t ticks = seq == 1 ? rb.arrive_ticks : rb.wait_ticks;
    const int per = NT >> rb.ushift, groups = (d.tiles + kGroup - 1) / kGroup, upad = 1 << rb.ushift;
    bool lost = false;
    for (int base = blockIdx.x; base < nent; base += grid * per) {
      const int el = tid >> rb.ushift, un = tid & (upad - 1);
      const int e = base + grid * el;
      double v = 0.0;
      if (e < nent && un < grid)
        lost = !ll_wait(rb.parts + 2 * (static_cast<size_t>(e) * grid + un), seq, ticks, v) || lost;
      // (the staging area's last reads: red before the barrier above, or this loop)
      if (base != static_cast<int>(blockIdx.x)) __syncthreads();
      vals[tid] = v;
      __syncthreads();
      for (int i = tid; i < per * groups; i += NT) {
        const int l = i / groups, g = i - l * groups;
        const double* uv = vals + (l << rb.ushift);
        const int cnt = min(kGroup, d.tiles - g * kGroup);  // slots of the group
        double quad[kGroup / 4];
#pragma unroll
        for (int k = 0; k < kGroup / 4; ++k) {  // every read before the first sum
          const int u0 = (g * kGroup + 4 * k) / tpw;
          auto unit = [&](int u) { return u < upad ? uv[u] : 0.0; };
          quad[k] = tpw == 4   ? unit(u0)
                    : tpw == 2 ? unit(u0) + unit(u0 + 1)
                               : (unit(u0) + unit(u0 + 1)) + (unit(u0 + 2) + unit(u0 + 3));
        }
        double s = quad[0];
#pragma unroll
        for (int k = 1; k < kGroup / 4; ++k)  // quads of slots, in order
          if (4 * k < cnt) s += quad[k];
        gsum[i] = s;
      }
      __syncthreads();
      if (tid < per && base + grid * tid < nent) {
        double s = 0.0;
        for (int g0 = 0; g0 < groups; g0 += 16) {  // sixteen reads in flight
          double v[16];
#pragma unroll
          for (int k = 0; k < 16; ++k) v[k] = g0 + k < groups ? gsum[tid * groups + g0 + k] : 0.0;
#pragma unroll
          for (int k = 0; k < 16; ++k)
            if (g0 + k < groups) s += v[k];
        }
        ll_store(rb.sums + 2 * (base + grid * tid), seq, s);
      }
    }
    RES_MARK(4);
    // 3. all sums
    for (int e = tid; e < nent; e += NT) {
      double v = 0.0;
      lost = !ll_wait(rb.sums + 2 * e, seq, ticks, v) || lost;
      sums[e] = v;
    }
    if (lost) s_lost = 1;
    __syncthreads();
    RES_MARK(5);
    return s_lost == 0;
  };
  // Control step on this workgroup's copy of the state; the Gram into LDS.
  auto control = [&](int kd) {
    for (int idx = tid; idx < nblk * 16; idx += NT) {
      const int blk = idx >> 4, e = idx & 15;
      const int cj = packed_col(blk), ci = blk - cj * (cj + 1) / 2;
      const int i = 4 * ci + (e >> 2), j = 4 * cj + (e & 3);
      if (i < n && j < n) {
        const double v = sums[kScalars + idx];
        eig.G[0][i * LD + j] = v;
        eig.G[0][j * LD + i] = v;
      }
    }
    if (tid == 0) {
      double tau = 0.0;
      s_go = control_step(d, &st, sums, kd, st.nXF2, st.tau, tau);
      s_tau = tau;
    }
    __syncthreads();
    return s_go != 0;
  };

  // Column by column through a running address (m is a scalar; the columns'
  // bases would take two scalar registers each).  Rows past m and frames past n
  // hold zeros, and zeros stay zeros through the update, so it needs no guards.
  auto columns = [&](auto base, auto&& f) __attribute__((always_inline)) {
    if (valid) {
      auto at = opaque(base) + p;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        if (j < n) {
          f(j, at);
          at += m;
        }
      }
    }
  };

  // Rows of X; norms and Gram of X (k_stream, init)
  const gptr<const T> X = as_global<T>(d.X);
  // (s goes out at the end only: the update needs x, y and a)
  T x[NB], s[NB], y[NB], a[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) {
    x[j] = 0;
    s[j] = 0;
    y[j] = 0;
  }
  columns(X, [&](int j, auto at) { x[j] = *at; });
  double s1 = 0.0, s2 = 0.0, nf = 0.0;
#pragma unroll
  for (int j = 0; j < NB4; ++j) {
    const T v = j < NB ? x[j] : T(0);
    const double xd = static_cast<double>(v);
    s1 += fabs(xd);
    s2 = fma(xd, xd, s2);
    nf += finite_val(v) ? 0.0 : 1.0;
    if (act) tileA[j * LDT + t] = v;
  }
  bool alive = exchange(std::true_type{}, 0.0, s1, s2, nf);
  bool go = false;
  if (alive) {
    go = control(0);
    if (!go && st.warm_stage == 1 && !st.done) {
      // given start: Gram of A_1 = X - S0 + Y0/mu (k_stream, warm)
      const T imu = static_cast<T>(st.imu);
      if (d.S0) columns(as_global<T>(d.S0), [&](int j, auto at) { s[j] = *at; });
      if (d.Y0) columns(as_global<T>(d.Y0), [&](int j, auto at) { y[j] = *at; });
      if (act) {
#pragma unroll
        for (int j = 0; j < NB4; ++j) tileA[j * LDT + t] = j < NB ? fma(y[j], imu, x[j] - s[j]) : T(0);
      }
      alive = exchange(std::false_type{}, 0.0, 0.0, 0.0, 0.0);
      if (alive) go = control(0);
    }
  }

  const gptr<T> L = as_global<T>(d.Lout);
  int kd = 0;
  {
    // A_1; later ones are what the update puts into the tile (same operations)
    const T imu = static_cast<T>(st.imu);
#pragma unroll
    for (int j = 0; j < NB; ++j) a[j] = fma(y[j], imu, x[j] - s[j]);
  }
  // Left to the launches, as for a lost wait: carried through the iterations
  // here, the shift took 4% of every solve (128 x 128 x 20 FP64: 12.3 to 12.7 ms).
  const int shift = __builtin_amdgcn_readfirstlane(eig_shift(st.nXF2));
  if (shift != 0) go = false;
  while (alive && go) {
    int sweeps = 0;
    RES_MARK(-1);
    if constexpr (SLIM) {
      if (act) {
#pragma unroll
        for (int j = 0; j < NB; ++j) tileA[j * LDT + t] = y[j];
      }
    }
    const int cur = eig_core<T, NMAX, NT>(
        eig, n, kd > 0, s_tau, sweeps,
        [&](int i, int j, double v) {
          if (j < NB) {
            Ps[(i * NBL + j / BLK) * 16 + j % BLK] = static_cast<T>(v);
            Ps[(j * NBL + i / BLK) * 16 + i % BLK] = static_cast<T>(v);
          }
        },
        [](int) {});
    __syncthreads();
    if (cur == 1) {  // V back to copy 0
      for (int i = tid; i < NMAX * LD; i += NT) eig.V[0][i] = eig.V[1][i];
    }
    if (tid == 0) {
      int rank = 0;
      for (int k = 0; k < n; ++k) rank += eig.w[k] != 0.0 ? 1 : 0;
      st.rank = rank;
      st.sweeps = sweeps;
      st.sweeps_total += sweeps;
      st.iter = kd + 1;
    }
    ++kd;
    RES_MARK(0);
    // Update of the rows (k_stream, update), all columns of L side by side.  L_k
    // goes out where this iteration may be the last.
    const T mu = static_cast<T>(st.mu), imu = static_cast<T>(st.imu), gam = static_cast<T>(st.gamma);
    const bool out = d.tol > 0.0 || kd >= d.maxit;
    double r2 = 0.0;
    if constexpr (SLIM) {
#pragma unroll
      for (int j = 0; j < NB; ++j) {  // (set by every thread: dead during the eigensolve)
        x[j] = 0;
        y[j] = 0;
      }
      columns(X, [&](int j, auto at) { x[j] = *at; });
      if (act) {
#pragma unroll
        for (int j = 0; j < NB; ++j) y[j] = tileA[j * LDT + t];
      }
    }
    if (act) {
      T l[NB], pr[2][NBL];  // a row of P is read while the one before it is used
      const T* const Pt = Ps + (t & 15);
#pragma unroll
      for (int j = 0; j < NB; ++j) l[j] = 0;
#pragma unroll
      for (int c = 0; c < NBL; ++c) pr[0][c] = Pt[c * 16];
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        if (i + 1 < NB) {
#pragma unroll
          for (int c = 0; c < NBL; ++c) pr[(i + 1) & 1][c] = Pt[((i + 1) * NBL + c) * 16];
        }
#pragma unroll
        for (int c = 0; c < NBL; ++c) fma_row<BLK>(l + c * BLK, pr[i & 1][c], a[i]);
        if constexpr (NT == 1024) __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        const T tt = fma(y[j], imu, x[j]) - l[j];
        const T sn = tt - clamp_sym(tt, gam);
        const T z = (x[j] - l[j]) - sn;
        const T yn = fma(mu, z, y[j]);
        const double zd = static_cast<double>(z);
        r2 = fma(zd, zd, r2);
        a[j] = fma(yn, imu, x[j] - sn);
        s[j] = sn;
        y[j] = yn;
        tileA[j * LDT + t] = a[j];
        // 128 registers: not more than two columns at a time
        if constexpr (NT == 1024)
          if (j & 1) __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int j = NB; j < NB4; ++j) tileA[j * LDT + t] = 0;
      // (written out: captured by a lambda, l becomes one 32-register tuple)
      if (out && valid) {
        gptr<T> at = opaque(L) + p;
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          if (j < n) {
            *at = l[j];
            at += m;
          }
        }
      }
    }
    RES_MARK(1);
    alive = exchange(std::false_type{}, r2, 0.0, 0.0, 0.0);
    if (alive) go = control(kd);
  }
#undef RES_MARK

  if (!alive || shift != 0) {
    if (tid == 0) __hip_atomic_store(rb.lost, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  if (st.status >= 0) {
    const bool none = kd == 0;  // sum|X| == 0: L = S = 0 (and Y = 0)
    if (none) columns(L, [&](int, auto at) { *at = T(0); });
    columns(as_global<T>(d.Sout), [&](int j, auto at) { *at = none ? T(0) : s[j]; });
    if (d.Yout) columns(as_global<T>(d.Yout), [&](int j, auto at) { *at = none ? T(0) : y[j]; });
  }
  if (blockIdx.x == 0 && tid == 0) *d.st = st;
}

template <typename T, int NB, int NT>
hipError_t launch_resident_class(int grid, hipStream_t stream, const SolveDesc& d, const ResidentBuf& rb) {
  hipLaunchKernelGGL((k_resident<T, NB, NT>), dim3(grid), dim3(NT), 0, stream, d, rb);
  return hipGetLastError();
}

}  // namespace
}  // namespace rpca
