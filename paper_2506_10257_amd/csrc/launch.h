// Host-side launchers of the device kernels (internal to the library).
#pragma once

#include <hip/hip_ext.h>

#include "common.h"

namespace rpca {

// Kernel timing: while `start` is set, a solve-path launch on this thread
// records its own start and end timestamps into the pair (the dispatch packet
// carries them, so queue time between launches is not counted).  Either may be
// null, for a sequence of launches timed as one.  Both are null when timing is
// off: then the launch is a plain one.
struct LaunchEvents {
  hipEvent_t start = nullptr, stop = nullptr;
};
extern thread_local LaunchEvents t_launch_events;

// Bounds of the waits inside a launch, in ticks of the 100 MHz wall clock: at the
// whole-solve kernel's first exchange (workgroups still being placed), and at its
// later ones and the meetings of the eigensolver's teams (all are running).  Per
// host thread, so that a test can end its own calls' waits early
// (rpca_inject_wait).
struct RunLimits {
  int64_t arrive_ticks = 500000;   // 5 ms
  int64_t wait_ticks = 20000000;   // 200 ms
};
extern thread_local RunLimits t_limits;

#define RPCA_LAUNCH(K, G, B, SH, S, ...)                                                      \
  do {                                                                                       \
    if (::rpca::t_launch_events.start || ::rpca::t_launch_events.stop)                       \
      hipExtLaunchKernelGGL(K, G, B, SH, S, ::rpca::t_launch_events.start,                   \
                            ::rpca::t_launch_events.stop, 0, __VA_ARGS__);                   \
    else                                                                                     \
      hipLaunchKernelGGL(K, G, B, SH, S, __VA_ARGS__);                                       \
  } while (0)

// Frame classes compiled for the register-resident streaming kernels.  A solve
// with n frames runs on the smallest class >= n.
constexpr int kClassesF32[] = {4, 8, 10, 12, 16, 20, 24, 28, 32, 40, 48, 56, 60, 64};
constexpr int kClassesF64[] = {4, 8, 10, 12, 16, 20, 24, 28, 32};

// kModeWarm: for a solve started from a given S0 / Y0, the Gram of the first
// iterate A_1 = X - S0 + Y0/mu (after mu is fixed), copying S0 and Y0 into the
// iterate buffers that the first update pass reads.
enum StreamMode { kModeInit = 0, kModeUpdate = 1, kModeFinalize = 2, kModeWarm = 3 };

// dtype 0 = FP64, 1 = FP32 (as RPCA_F64 / RPCA_F32).
// mt: the multi-tile register kernel (work items of more than one tile).
hipError_t launch_stream_f32(int nb, int mode, bool mt, int grid, hipStream_t stream,
                             const SolveDesc* descs, const WorkItem* items);
hipError_t launch_stream_f64(int nb, int mode, bool mt, int grid, hipStream_t stream,
                             const SolveDesc* descs, const WorkItem* items);
// chunks: entry chunks of a group (reduce_chunks of the largest solve).
int reduce_chunks(int nb);
hipError_t launch_reduce(int grid, int chunks, hipStream_t stream, const SolveDesc* descs,
                         const GroupItem* items);
hipError_t launch_gather_states(int count, hipStream_t stream, const SolveDesc* descs,
                                SolveState* out);
hipError_t launch_reset_states(int count, hipStream_t stream, const SolveDesc* descs);

// Eigensolver classes 16, 32 and 64: the largest n each handles.  The
// workgroup size of each class (256, 512 or 1024 threads) is a tuning knob.
// ids lists the solves (indices into descs) of the launch.
// Returns 16, 32, 64, kEigWideMaxN or kEigHugeMaxN (0 if n is too large).
int eig_class(int n);
// Classes above 64 frames: the in-place eigensolver, ncls = kEigWideMaxN
// (V in LDS) or kEigHugeMaxN (V in global memory).  start: the solves' control
// step and the first sweeps of their first eigensolve, which the next
// launch_eig_steps goes on with.
hipError_t launch_eig_wide(int dtype, int ncls, int grid, bool start, hipStream_t stream,
                           const SolveDesc* descs, const int32_t* ids);
// Warm-started steps of the same solves, launched before launch_eig_wide
// (which returns at once where they converged).  `team` workgroups per solve.
int steps_team(int nb, int grid);
hipError_t launch_eig_steps(int dtype, int grid, int team, hipStream_t stream, const SolveDesc* descs,
                            const int32_t* ids);
// MFMA streaming kernel.  FP32 storage: nb a multiple of 16 up to 144;
// prec 0 = FP32 rebuild / FP64 Gram, 1 = split-BF16 (3 products) for both,
// 2 = split-BF16 (6 products).  FP64 storage: nb = 48, 64, ..., 128, both
// contractions in FP64.
hipError_t launch_wide_f32(int nb, int mode, int prec, int grid, hipStream_t stream,
                           const SolveDesc* descs, const WorkItem* items);
hipError_t launch_wide_f64(int nb, int mode, int grid, hipStream_t stream, const SolveDesc* descs,
                           const WorkItem* items);
bool eig_threads_valid(int ncls, int nt);
int eig_threads(int dtype, int ncls);
bool set_eig_threads(int dtype, int ncls, int nt);
hipError_t launch_eig(int dtype, int ncls, int grid, hipStream_t stream, const SolveDesc* descs,
                      const int32_t* ids);

// Whole-solve kernel (resident_impl.h): its exchange buffers.
struct ResidentBuf {
  uint64_t* parts;  // 2 words per (entry, workgroup)
  uint64_t* sums;   // 2 words per entry
  uint32_t* lost;   // set when a wait ran out of time
  int32_t tpw;      // 256-row tiles per workgroup (1, 2 or 4)
  int32_t ushift;   // log2 of the workgroup count, rounded up
  int64_t arrive_ticks, wait_ticks;  // bounds of a wait (RunLimits)
};
hipError_t launch_resident_f32(int nb, int threads, int grid, hipStream_t stream, const SolveDesc& d,
                               const ResidentBuf& rb);
hipError_t launch_resident_f64(int nb, int threads, int grid, hipStream_t stream, const SolveDesc& d,
                               const ResidentBuf& rb);
// Zero `words` 8-byte words.
hipError_t launch_zero(uint64_t* p, size_t words, hipStream_t stream);

}  // namespace rpca
