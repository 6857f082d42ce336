// Processing steps around the RPCA solve, on the device (rpca_frame_* /
// rpca_moving_average / rpca_dice / rpca_rmse / rpca_masked_mean in
// include/rpca.h):
//
//   * consecutive-frame correlation, used to drop frames that correlate
//     poorly with their neighbours (the paper's in vivo reference, Sec. III);
//   * frame selection (copy of the kept frames into a new Casorati matrix);
//   * temporal moving average over W frames (same passage);
//   * binarisation and the Dice coefficient (Sec. II-F, Eq. 8), the RMSE
//     (Eq. 7) and the masked mean that gives the binarisation threshold.
//
// Every reduction is fixed-order: each workgroup writes a partial to its own
// slot and one more launch adds the slots in order, so results do not
// depend on scheduling.  Sums are FP64, counts are 64-bit integers.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>
#include <cstring>
#include <type_traits>
#include <vector>

#include "rpca.h"
#include "common.h"
#include "device_use.h"
#include "engine.h"

namespace rpca {
namespace {

constexpr int kPT = 256;        // threads per workgroup
constexpr int kMaxGrid = 2048;  // workgroups of a reduction pass
constexpr int kCorrMaxN = 160;  // frames handled by the correlation kernel
constexpr int kCorrFrames = 8;  // frames of a correlation workgroup

__device__ inline double wsum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}
__device__ inline long long wsum_i(long long v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// V consecutive values of one load (V = 1: any alignment).
template <typename T, int V>
struct Pack {
  typedef T type __attribute__((ext_vector_type(V)));
};
template <typename T>
struct Pack<T, 1> {
  typedef T type;
};
template <int V, typename P>
__device__ inline auto pick(const P& p, int k) {
  if constexpr (V == 1) return p;
  else return p[k];
}
// Sums of frame t, its square and its product with frame t+1 over one run of
// rows, for kCorrFrames frames: workgroup (rb, f) writes partial[rb][3t ..
// 3t+2] of its frames.  Bound by HBM: a workgroup reads its frames and the one
// after them once (1.13 reads per entry; with one frame per workgroup every
// frame was read twice), nine independent loads of V rows in flight per thread.
// Each thread accumulates over its rows in registers; one workgroup reduction at
// the end.  V > 1 needs m to be a multiple of V and X to be aligned to V
// entries.  1024 x 1024 x 132 FP32, call to host result: 379 us with one frame
// per workgroup, 346 with eight and V = 1, 168 with V = 4.
template <typename T, int V>
__global__ void __launch_bounds__(kPT)
k_frame_sums(const T* __restrict__ X, int64_t m, int n, double* __restrict__ partial) {
  constexpr int F = kCorrFrames;
  typedef typename Pack<T, V>::type P;
  __shared__ double red[kPT / 64][3 * F];
  const int t0 = blockIdx.y * F, nf = min(F, n - t0);
  const int64_t packs = m / V, per = (packs + gridDim.x - 1) / gridDim.x;
  const int64_t r0 = min(static_cast<int64_t>(blockIdx.x) * per, packs);
  const unsigned rows = static_cast<unsigned>(min(per, packs - r0));
  const P* base = reinterpret_cast<const P*>(X + static_cast<size_t>(t0) * m) + r0;
  double s[F], q[F], c[F];
#pragma unroll
  for (int k = 0; k < F; ++k) s[k] = q[k] = c[k] = 0.0;
  auto run = [&](auto full) {  // full: frame t0 + F exists
    for (unsigned i = threadIdx.x; i < rows; i += kPT) {
      P v[F + 1];
#pragma unroll
      for (int k = 0; k <= F; ++k)
        v[k] = full || t0 + k < n ? (base + static_cast<size_t>(k) * packs)[i] : P(0);
#pragma unroll
      for (int e = 0; e < V; ++e) {
        double x = static_cast<double>(pick<V>(v[0], e));
#pragma unroll
        for (int k = 0; k < F; ++k) {
          const double y = static_cast<double>(pick<V>(v[k + 1], e));
          s[k] += x;
          q[k] = fma(x, x, q[k]);
          c[k] = fma(x, y, c[k]);
          x = y;
        }
      }
    }
  };
  if (t0 + F < n) run(std::true_type{});
  else run(std::false_type{});
  const int wv = threadIdx.x >> 6;
#pragma unroll
  for (int k = 0; k < F; ++k) {
    const double a = wsum(s[k]), b = wsum(q[k]), e = wsum(c[k]);
    if ((threadIdx.x & 63) == 0) {
      red[wv][3 * k] = a;
      red[wv][3 * k + 1] = b;
      red[wv][3 * k + 2] = e;
    }
  }
  __syncthreads();
  if (threadIdx.x < 3 * nf) {
    double v = red[0][threadIdx.x];
#pragma unroll
    for (int w = 1; w < kPT / 64; ++w) v += red[w][threadIdx.x];
    partial[static_cast<size_t>(blockIdx.x) * 3 * n + 3 * t0 + threadIdx.x] = v;
  }
}

__device__ inline double wsum_any(double v) { return wsum(v); }
__device__ inline long long wsum_any(long long v) { return wsum_i(v); }

// Sum `slots` partials of `len` values into out[len], one workgroup per value:
// thread i adds slots i, i + kPT, ... in order, then lanes and waves in a fixed
// order: 6 us for 256 slots of 396 values.
template <typename V>
__global__ void __launch_bounds__(kPT)
k_sum_slots(const V* __restrict__ partial, int slots, int len, V* __restrict__ out) {
  __shared__ V red[kPT / 64];
  V v = 0;
#pragma unroll 4
  for (int s = threadIdx.x; s < slots; s += kPT) v += partial[static_cast<size_t>(s) * len + blockIdx.x];
  v = wsum_any(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  if (threadIdx.x == 0) {
    V t = red[0];
    for (int w = 1; w < kPT / 64; ++w) t += red[w];
    out[blockIdx.x] = t;
  }
}

// out[:, t] = mean of M[:, t .. t+W-1], t = 0 .. n-W.  One thread per pixel
// row keeps the last W values in an LDS ring and a running FP64 sum, so each
// input is read once and each output written once; eight frames are read ahead
// of the sum (one at a time a row's loads wait for each other: 264 us at 1024 x
// 1024 x 132 FP32 and W = 20, now 211, 5.2 TB/s).
constexpr int kMAT = 128;   // threads of the moving-average kernel (LDS ring W x 128)
constexpr int kMAhead = 8;  // frames read at a time

template <typename T>
__global__ void __launch_bounds__(kMAT)
k_moving_average(const T* __restrict__ X, int64_t m, int n, int W, T* __restrict__ out) {
  extern __shared__ __align__(16) unsigned char ring_raw[];
  T* ring = reinterpret_cast<T*>(ring_raw) + threadIdx.x;
  const int64_t p = static_cast<int64_t>(blockIdx.x) * kMAT + threadIdx.x;
  if (p >= m) return;
  const double inv = 1.0 / static_cast<double>(W);
  double sum = 0.0;
  int slot = 0;  // t % W
  const T* in = X + p;
  T* to = out + p;
  auto frame = [&](int t, T x) {
    T* const r = ring + static_cast<size_t>(slot) * kMAT;
    if (t >= W) sum -= static_cast<double>(*r);
    *r = x;
    sum += static_cast<double>(x);
    slot = slot + 1 == W ? 0 : slot + 1;
    if (t >= W - 1) {
      *to = static_cast<T>(sum * inv);
      to += m;
    }
  };
  int t = 0;
  for (; t + kMAhead <= n; t += kMAhead) {
    T x[kMAhead];
#pragma unroll
    for (int k = 0; k < kMAhead; ++k) x[k] = in[static_cast<size_t>(k) * m];
    in += static_cast<size_t>(kMAhead) * m;
#pragma unroll
    for (int k = 0; k < kMAhead; ++k) frame(t + k, x[k]);
  }
  for (; t < n; ++t, in += m) frame(t, *in);
}

// f(a, b) for every pair of entries of A and B that is this thread's: packs of
// V entries, four packs of each array in flight, then the count % V left over.
// Bound by HBM: RMSE of two 1024 x 1024 x 132 FP32 arrays, call to host result,
// 424 us with one entry in flight, now 279 (the pass itself 4.8 TB/s).
template <typename T, typename U, int V, typename F>
__device__ inline void for_pairs(const T* __restrict__ A, const U* __restrict__ B, int64_t count, F&& f) {
  typedef typename Pack<T, V>::type PA;
  typedef typename Pack<U, V>::type PB;
  const PA* pa = reinterpret_cast<const PA*>(A);
  const PB* pb = reinterpret_cast<const PB*>(B);
  const int64_t packs = count / V, id = blockIdx.x * static_cast<int64_t>(kPT) + threadIdx.x;
  const int64_t step = static_cast<int64_t>(gridDim.x) * kPT;
  constexpr int D = 4;
  int64_t i = id;
  for (; i + (D - 1) * step < packs; i += D * step) {
    PA a[D];
    PB b[D];
#pragma unroll
    for (int k = 0; k < D; ++k) {
      a[k] = pa[i + k * step];
      b[k] = pb[i + k * step];
    }
#pragma unroll
    for (int k = 0; k < D; ++k)
#pragma unroll
      for (int e = 0; e < V; ++e) f(pick<V>(a[k], e), pick<V>(b[k], e));
  }
  for (; i < packs; i += step) {
    const PA a = pa[i];
    const PB b = pb[i];
#pragma unroll
    for (int e = 0; e < V; ++e) f(pick<V>(a, e), pick<V>(b, e));
  }
  if (V > 1 && id < count - packs * V) f(A[packs * V + id], B[packs * V + id]);
}

// counts[slot][3] = |A >= ta & B >= tb|, |A >= ta|, |B >= tb| (compared in FP64)
template <typename T, int V>
__global__ void __launch_bounds__(kPT)
k_dice_counts(const T* __restrict__ A, double ta, const T* __restrict__ B, double tb, int64_t count,
              long long* __restrict__ partial) {
  __shared__ long long red[kPT / 64][3];
  long long both = 0, ca = 0, cb = 0;
  for_pairs<T, T, V>(A, B, count, [&](T x, T y) {
    const bool a = static_cast<double>(x) >= ta, b = static_cast<double>(y) >= tb;
    both += (a && b) ? 1 : 0;
    ca += a ? 1 : 0;
    cb += b ? 1 : 0;
  });
  both = wsum_i(both);
  ca = wsum_i(ca);
  cb = wsum_i(cb);
  const int wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    red[wv][0] = both;
    red[wv][1] = ca;
    red[wv][2] = cb;
  }
  __syncthreads();
  if (threadIdx.x < 3) {
    long long v = 0;
    for (int w = 0; w < kPT / 64; ++w) v += red[w][threadIdx.x];
    partial[static_cast<size_t>(blockIdx.x) * 3 + threadIdx.x] = v;
  }
}

// partial[slot][2] = sum over the slot of (A - B)^2 and of 1 (U = T), or of
// A * [mask != 0] and [mask != 0] (U = uint8_t).
template <typename T, typename U, int V>
__global__ void __launch_bounds__(kPT)
k_pair_sums(const T* __restrict__ A, const U* __restrict__ B, int64_t count, double* __restrict__ partial) {
  __shared__ double red[kPT / 64][2];
  double s = 0.0, c = 0.0;
  for_pairs<T, U, V>(A, B, count, [&](T x, U y) {
    const double a = static_cast<double>(x);
    if constexpr (std::is_same<T, U>::value) {
      const double dlt = a - static_cast<double>(y);
      s = fma(dlt, dlt, s);
      c += 1.0;
    } else {
      const bool on = y != 0;
      s += on ? a : 0.0;
      c += on ? 1.0 : 0.0;
    }
  });
  s = wsum(s);
  c = wsum(c);
  const int wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) {
    red[wv][0] = s;
    red[wv][1] = c;
  }
  __syncthreads();
  if (threadIdx.x < 2) {
    double v = red[0][threadIdx.x];
    for (int w = 1; w < kPT / 64; ++w) v += red[w][threadIdx.x];
    partial[static_cast<size_t>(blockIdx.x) * 2 + threadIdx.x] = v;
  }
}

// Frames from[0 .. gridDim.y) of src to consecutive frames of dst, in units of U
// (`len` of them per frame).  One launch for up to kCopyFrames frames: 130 frames
// of 1024 x 1024 FP32 took 399 us with a copy call each, now 196 (5.7 TB/s).
constexpr int kCopyFrames = 256;
constexpr int kCopyUnits = 8;  // units per thread
struct FrameList {
  int32_t from[kCopyFrames];
};
template <typename U>
__global__ void __launch_bounds__(kPT)
k_copy_frames(const U* __restrict__ src, U* __restrict__ dst, int64_t len, FrameList list) {
  const U* a = src + static_cast<size_t>(list.from[blockIdx.y]) * len;
  U* b = dst + static_cast<size_t>(blockIdx.y) * len;
  const int64_t i0 = static_cast<int64_t>(blockIdx.x) * kPT * kCopyUnits + threadIdx.x;
  if (i0 - threadIdx.x + kPT * kCopyUnits <= len) {
    U v[kCopyUnits];
#pragma unroll
    for (int k = 0; k < kCopyUnits; ++k) v[k] = a[i0 + k * kPT];
#pragma unroll
    for (int k = 0; k < kCopyUnits; ++k) b[i0 + k * kPT] = v[k];
  } else {
    for (int64_t i = i0; i < len; i += kPT) b[i] = a[i];
  }
}
template <typename U>
hipError_t copy_frames(const void* src, void* dst, int64_t len, const FrameList& list, int count,
                       hipStream_t s) {
  const int64_t per = static_cast<int64_t>(kPT) * kCopyUnits;
  hipLaunchKernelGGL(k_copy_frames<U>, dim3(static_cast<unsigned>((len + per - 1) / per), count), dim3(kPT), 0,
                     s, static_cast<const U*>(src), static_cast<U*>(dst), len, list);
  return hipGetLastError();
}

bool aligned(const void* p, size_t a) { return reinterpret_cast<uintptr_t>(p) % a == 0; }

int grid_for(int64_t count) {
  const int64_t g = (count + kPT * 16 - 1) / (kPT * 16);
  return static_cast<int>(g < 1 ? 1 : (g > kMaxGrid ? kMaxGrid : g));
}

// Run a partial-producing launch, sum its slots in order and copy `len`
// results to host memory `out` (stream-ordered, then synchronised).
template <typename V, typename Launch>
int reduce_to_host(hipStream_t s, int grid, int len, V* out, Launch&& launch) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) (void)hipGetLastError();
  const OtherCall other(dev);
  V* buf = nullptr;
  const size_t bytes = sizeof(V) * (static_cast<size_t>(grid) + 1) * len;
  hipError_t e = hipMallocAsync(reinterpret_cast<void**>(&buf), bytes, s);
  if (e != hipSuccess || !buf) {
    set_error("hipMallocAsync(reduction)", e);
    (void)hipGetLastError();
    return RPCA_ERR_NOMEM;
  }
  V* total = buf + static_cast<size_t>(grid) * len;
  launch(buf);
  e = hipGetLastError();
  if (e == hipSuccess) {
    hipLaunchKernelGGL(k_sum_slots<V>, dim3(len), dim3(kPT), 0, s, buf, grid, len, total);
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipMemcpyAsync(out, total, sizeof(V) * len, hipMemcpyDeviceToHost, s);
  const hipError_t ef = hipFreeAsync(buf, s);
  if (e == hipSuccess) e = ef;
  if (e == hipSuccess) e = hipStreamSynchronize(s);
  if (e != hipSuccess) {
    set_error("reduction", e);
    return RPCA_ERR_DEVICE;
  }
  return RPCA_OK;
}

bool dtype_ok(int32_t dtype) { return dtype == RPCA_F32 || dtype == RPCA_F64; }

}  // namespace
}  // namespace rpca

using namespace rpca;

extern "C" {

int rpca_frame_correlation(const void* M, int64_t m, int64_t n, int32_t dtype, double* rho,
                           void* stream) {
  if (!M || !rho || m < 2 || n < 2 || n > kCorrMaxN || !dtype_ok(dtype)) return RPCA_ERR_ARG;
  hipStream_t s = static_cast<hipStream_t>(stream);
  // row blocks per frame: enough workgroups in total to fill the device
  const int64_t rbs = (m + 16 * kPT - 1) / (16 * kPT);
  const int grid = static_cast<int>(rbs < 1 ? 1 : (rbs > 256 ? 256 : rbs));
  const int len = static_cast<int>(3 * n);
  std::vector<double> sums(len);
  const int rc = reduce_to_host(s, grid, len, sums.data(), [&](double* buf) {
    const dim3 g(grid, static_cast<unsigned>((n + kCorrFrames - 1) / kCorrFrames));
    const float* f = static_cast<const float*>(M);
    const double* d = static_cast<const double*>(M);
    const int nn = static_cast<int>(n);
    if (dtype == RPCA_F32 && m % 4 == 0 && aligned(M, 16))
      hipLaunchKernelGGL((k_frame_sums<float, 4>), g, dim3(kPT), 0, s, f, m, nn, buf);
    else if (dtype == RPCA_F32)
      hipLaunchKernelGGL((k_frame_sums<float, 1>), g, dim3(kPT), 0, s, f, m, nn, buf);
    else if (m % 2 == 0 && aligned(M, 16))
      hipLaunchKernelGGL((k_frame_sums<double, 2>), g, dim3(kPT), 0, s, d, m, nn, buf);
    else
      hipLaunchKernelGGL((k_frame_sums<double, 1>), g, dim3(kPT), 0, s, d, m, nn, buf);
  });
  if (rc != RPCA_OK) return rc;
  const double mm = static_cast<double>(m);
  for (int64_t t = 0; t + 1 < n; ++t) {
    const double sx = sums[3 * t], sxx = sums[3 * t + 1], sxy = sums[3 * t + 2];
    const double sy = sums[3 * (t + 1)], syy = sums[3 * (t + 1) + 1];
    const double cov = sxy - sx * sy / mm;
    const double vx = sxx - sx * sx / mm, vy = syy - sy * sy / mm;
    rho[t] = (vx > 0.0 && vy > 0.0) ? cov / std::sqrt(vx * vy) : 0.0;
  }
  return RPCA_OK;
}

int rpca_frame_keep(const double* rho, int64_t n, double threshold, int32_t* keep) {
  if (!rho || !keep || n < 1) return RPCA_ERR_ARG;
  int kept = 0;
  for (int64_t t = 0; t < n; ++t) {
    double best = -2.0;
    if (t > 0) best = std::fmax(best, rho[t - 1]);
    if (t + 1 < n) best = std::fmax(best, rho[t]);
    keep[t] = (n == 1 || best >= threshold) ? 1 : 0;
    kept += keep[t];
  }
  return kept;
}

int rpca_frame_select(const void* M, int64_t m, int64_t n, int32_t dtype, const int32_t* keep,
                      void* out, void* stream) {
  if (!M || !out || !keep || m < 1 || n < 1 || !dtype_ok(dtype)) return RPCA_ERR_ARG;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const size_t col = static_cast<size_t>(m) * (dtype == RPCA_F32 ? 4 : 8);
  // the widest unit that every frame's start and length allow
  const size_t es = dtype == RPCA_F32 ? 4 : 8;
  const size_t unit = col % 16 == 0 && aligned(M, 16) && aligned(out, 16) ? 16 : es;
  const int64_t len = static_cast<int64_t>(col / unit);
  int k = 0;  // frames written
  FrameList list;
  int held = 0;
  const char* base = static_cast<const char*>(M);  // frame indices in a list are relative to it
  // a result inside the input is built one frame after another
  const uintptr_t mi = reinterpret_cast<uintptr_t>(M), oi = reinterpret_cast<uintptr_t>(out);
  const bool apart = oi >= mi + col * static_cast<size_t>(n) || mi >= oi + col * static_cast<size_t>(n);
  const int limit = apart ? kCopyFrames : 1;
  int64_t t0 = 0;
  for (int64_t t = 0; t <= n; ++t) {
    if (held > 0 && (t == n || held == limit || t - t0 >= INT32_MAX)) {
      void* to = static_cast<char*>(out) + col * static_cast<size_t>(k);
      const hipError_t e = unit == 16  ? copy_frames<Pack<uint32_t, 4>::type>(base, to, len, list, held, s)
                           : unit == 8 ? copy_frames<uint64_t>(base, to, len, list, held, s)
                                       : copy_frames<uint32_t>(base, to, len, list, held, s);
      if (e != hipSuccess) {
        set_error("k_copy_frames", e);
        return RPCA_ERR_DEVICE;
      }
      k += held;
      held = 0;
    }
    if (t < n && keep[t]) {
      if (held == 0) {
        t0 = t;
        base = static_cast<const char*>(M) + col * static_cast<size_t>(t);
      }
      list.from[held++] = static_cast<int32_t>(t - t0);
    }
  }
  return k;
}

int rpca_moving_average(const void* M, int64_t m, int64_t n, int32_t W, int32_t dtype, void* out,
                        void* stream) {
  if (!M || !out || m < 1 || W < 1 || W > 32 || n < W || !dtype_ok(dtype)) return RPCA_ERR_ARG;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int grid = static_cast<int>((m + kMAT - 1) / kMAT);
  const size_t lds = static_cast<size_t>(W) * kMAT * (dtype == RPCA_F32 ? 4 : 8);
  if (dtype == RPCA_F32)
    hipLaunchKernelGGL(k_moving_average<float>, dim3(grid), dim3(kMAT), lds, s,
                       static_cast<const float*>(M), m, static_cast<int>(n), W, static_cast<float*>(out));
  else
    hipLaunchKernelGGL(k_moving_average<double>, dim3(grid), dim3(kMAT), lds, s,
                       static_cast<const double*>(M), m, static_cast<int>(n), W, static_cast<double*>(out));
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) {
    set_error("k_moving_average", e);
    return RPCA_ERR_DEVICE;
  }
  return RPCA_OK;
}

int rpca_dice(const void* A, double thr_a, const void* B, double thr_b, int64_t count, int32_t dtype,
              int64_t* counts, double* dice, void* stream) {
  if (!A || !B || count < 1 || !dtype_ok(dtype)) return RPCA_ERR_ARG;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int grid = grid_for(count);
  long long c[3] = {0, 0, 0};
  const bool packs = aligned(A, 16) && aligned(B, 16);
  const int rc = reduce_to_host(s, grid, 3, c, [&](long long* buf) {
    const float *fa = static_cast<const float*>(A), *fb = static_cast<const float*>(B);
    const double *da = static_cast<const double*>(A), *db = static_cast<const double*>(B);
    if (dtype == RPCA_F32 && packs)
      hipLaunchKernelGGL((k_dice_counts<float, 4>), dim3(grid), dim3(kPT), 0, s, fa, thr_a, fb, thr_b, count, buf);
    else if (dtype == RPCA_F32)
      hipLaunchKernelGGL((k_dice_counts<float, 1>), dim3(grid), dim3(kPT), 0, s, fa, thr_a, fb, thr_b, count, buf);
    else if (packs)
      hipLaunchKernelGGL((k_dice_counts<double, 2>), dim3(grid), dim3(kPT), 0, s, da, thr_a, db, thr_b, count, buf);
    else
      hipLaunchKernelGGL((k_dice_counts<double, 1>), dim3(grid), dim3(kPT), 0, s, da, thr_a, db, thr_b, count, buf);
  });
  if (rc != RPCA_OK) return rc;
  if (counts)
    for (int i = 0; i < 3; ++i) counts[i] = c[i];
  if (dice) {
    const long long den = c[1] + c[2];
    *dice = den == 0 ? 1.0 : 2.0 * static_cast<double>(c[0]) / static_cast<double>(den);
  }
  return RPCA_OK;
}

int rpca_rmse(const void* A, const void* B, int64_t count, int32_t dtype, double* out, void* stream) {
  if (!A || !B || !out || count < 1 || !dtype_ok(dtype)) return RPCA_ERR_ARG;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int grid = grid_for(count);
  double r[2] = {0, 0};
  const bool packs = aligned(A, 16) && aligned(B, 16);
  const int rc = reduce_to_host(s, grid, 2, r, [&](double* buf) {
    const float *fa = static_cast<const float*>(A), *fb = static_cast<const float*>(B);
    const double *da = static_cast<const double*>(A), *db = static_cast<const double*>(B);
    if (dtype == RPCA_F32 && packs)
      hipLaunchKernelGGL((k_pair_sums<float, float, 4>), dim3(grid), dim3(kPT), 0, s, fa, fb, count, buf);
    else if (dtype == RPCA_F32)
      hipLaunchKernelGGL((k_pair_sums<float, float, 1>), dim3(grid), dim3(kPT), 0, s, fa, fb, count, buf);
    else if (packs)
      hipLaunchKernelGGL((k_pair_sums<double, double, 2>), dim3(grid), dim3(kPT), 0, s, da, db, count, buf);
    else
      hipLaunchKernelGGL((k_pair_sums<double, double, 1>), dim3(grid), dim3(kPT), 0, s, da, db, count, buf);
  });
  if (rc != RPCA_OK) return rc;
  *out = std::sqrt(r[0] / static_cast<double>(count));
  return RPCA_OK;
}

int rpca_masked_mean(const void* A, const uint8_t* mask, int64_t count, int32_t dtype, double* out,
                     void* stream) {
  if (!A || !mask || !out || count < 1 || !dtype_ok(dtype)) return RPCA_ERR_ARG;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int grid = grid_for(count);
  double r[2] = {0, 0};
  const bool packs = aligned(A, 16) && aligned(mask, dtype == RPCA_F32 ? 4 : 2);
  const int rc = reduce_to_host(s, grid, 2, r, [&](double* buf) {
    const float* fa = static_cast<const float*>(A);
    const double* da = static_cast<const double*>(A);
    if (dtype == RPCA_F32 && packs)
      hipLaunchKernelGGL((k_pair_sums<float, uint8_t, 4>), dim3(grid), dim3(kPT), 0, s, fa, mask, count, buf);
    else if (dtype == RPCA_F32)
      hipLaunchKernelGGL((k_pair_sums<float, uint8_t, 1>), dim3(grid), dim3(kPT), 0, s, fa, mask, count, buf);
    else if (packs)
      hipLaunchKernelGGL((k_pair_sums<double, uint8_t, 2>), dim3(grid), dim3(kPT), 0, s, da, mask, count, buf);
    else
      hipLaunchKernelGGL((k_pair_sums<double, uint8_t, 1>), dim3(grid), dim3(kPT), 0, s, da, mask, count, buf);
  });
  if (rc != RPCA_OK) return rc;
  *out = r[1] > 0.0 ? r[0] / r[1] : std::nan("");
  return r[1] > 0.0 ? RPCA_OK : RPCA_ERR_ARG;
}

}  // extern "C"
