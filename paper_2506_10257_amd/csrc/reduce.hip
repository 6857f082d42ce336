// First level of the fixed-order reduction of the streaming pass's partial
// sums: one workgroup per (solve, group of kGroup slots, chunk of entries) adds
// the group's slots in slot order.  A window of 132 frames has 8980 entries per
// slot but, at 512 x 512 pixels, 8 groups only: with one workgroup per group
// its pass moved 18.4 MB through 8 CUs.  The eigensolve kernel adds the group sums in group
// order.  Running it as its own launch (instead of a last-arriving-workgroup
// scheme inside the streaming kernel) keeps device-scope fences, and the L2
// write-backs they imply, out of the streaming pass.
#include "common.h"
#include "launch.h"

namespace rpca {
namespace {

// A group's slots are added in quads, (v0 + v1) + (v2 + v3), and the quads in
// order: a workgroup of the whole-solve kernel (resident_impl.h) that holds four
// tiles can then hand on one sum.
constexpr int kChunkEntries = 2 * kThreads;  // entries of a workgroup

__global__ void __launch_bounds__(kThreads)
k_reduce_groups(const SolveDesc* __restrict__ descs, const GroupItem* __restrict__ items) {
  const GroupItem gi = items[blockIdx.x];
  const SolveDesc& d = descs[gi.solve];
  if (d.st->done) return;
  const int nent = kScalars + gram_blocks((d.n + 3) >> 2) * 16;
  const int e0 = blockIdx.y * kChunkEntries, e1 = min(nent, e0 + kChunkEntries);
  const int lo = gi.group * kGroup;
  const int cnt = min(kGroup, d.slots - lo);
  const double* src = d.partials + static_cast<size_t>(lo) * d.pstride;
  double* dst = d.gpartials + static_cast<size_t>(gi.group) * d.pstride;
  for (int idx = e0 + threadIdx.x; idx < e1; idx += kThreads) {
    double v[kGroup];
#pragma unroll
    for (int q = 0; q < kGroup; ++q)
      v[q] = q < cnt ? src[static_cast<size_t>(q) * d.pstride + idx] : 0.0;
    double sum = (v[0] + v[1]) + (v[2] + v[3]);
#pragma unroll
    for (int q = 4; q < kGroup; q += 4)
      if (q < cnt) sum += (v[q] + v[q + 1]) + (v[q + 2] + v[q + 3]);
    dst[idx] = sum;
  }
}

// Copy the state of every solve of a plan to one contiguous array (read back
// by the host with a single copy).
__global__ void __launch_bounds__(64)
k_gather_states(const SolveDesc* __restrict__ descs, int count, SolveState* __restrict__ out) {
  const int i = blockIdx.x * 64 + threadIdx.x;
  if (i < count) out[i] = *descs[i].st;
}

// Zero the state of every solve of a plan (done before its init pass).
__global__ void __launch_bounds__(64)
k_reset_states(const SolveDesc* __restrict__ descs, int count) {
  const int i = blockIdx.x * 64 + threadIdx.x;
  if (i < count) {
    SolveState z{};
    *descs[i].st = z;
  }
}

__global__ void __launch_bounds__(kThreads)
k_zero(uint64_t* __restrict__ p, size_t words) {
  const size_t stride = static_cast<size_t>(gridDim.x) * kThreads;
  for (size_t i = static_cast<size_t>(blockIdx.x) * kThreads + threadIdx.x; i < words; i += stride) p[i] = 0;
}

}  // namespace

hipError_t launch_zero(uint64_t* p, size_t words, hipStream_t stream) {
  const size_t g = (words + kThreads - 1) / kThreads;
  hipLaunchKernelGGL(k_zero, dim3(static_cast<unsigned>(g < 1024 ? g : 1024)), dim3(kThreads), 0, stream, p,
                     words);
  return hipGetLastError();
}

hipError_t launch_gather_states(int count, hipStream_t stream, const SolveDesc* descs,
                                SolveState* out) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_gather_states, dim3((count + 63) / 64), dim3(64), 0, stream, descs, count, out);
  return hipGetLastError();
}

hipError_t launch_reset_states(int count, hipStream_t stream, const SolveDesc* descs) {
  if (count <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_reset_states, dim3((count + 63) / 64), dim3(64), 0, stream, descs, count);
  return hipGetLastError();
}

int reduce_chunks(int nb) {
  return (kScalars + gram_blocks((nb + 3) >> 2) * 16 + kChunkEntries - 1) / kChunkEntries;
}

hipError_t launch_reduce(int grid, int chunks, hipStream_t stream, const SolveDesc* descs,
                         const GroupItem* items) {
  if (grid <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_reduce_groups, dim3(grid, chunks), dim3(kThreads), 0, stream, descs, items);
  return hipGetLastError();
}

}  // namespace rpca
