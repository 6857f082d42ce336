// Whole-solve kernels for float storage (see resident_impl.h): 512 threads (two
// tiles per workgroup), and 1024 (four tiles, 128 registers) for the windows of
// up to 20 frames that need them.
#include "resident_impl.h"

namespace rpca {

hipError_t launch_resident_f32(int nb, int threads, int grid, hipStream_t stream, const SolveDesc& d,
                               const ResidentBuf& rb) {
#define X(N, NT) \
  if (nb == N && threads == NT) return launch_resident_class<float, N, NT>(grid, stream, d, rb);
  X(10, 512) X(16, 512) X(20, 512) X(32, 512) X(10, 1024) X(16, 1024) X(20, 1024)
#undef X
  return hipErrorInvalidValue;
}

}  // namespace rpca
