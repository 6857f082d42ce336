// Whole-solve kernels for double storage (see resident_impl.h).
#include "resident_impl.h"

namespace rpca {

hipError_t launch_resident_f64(int nb, int threads, int grid, hipStream_t stream, const SolveDesc& d,
                               const ResidentBuf& rb) {
#define X(N, NT) \
  if (nb == N && threads == NT) return launch_resident_class<double, N, NT>(grid, stream, d, rb);
  X(10, 512) X(16, 512) X(20, 512)
#undef X
  return hipErrorInvalidValue;
}

}  // namespace rpca
