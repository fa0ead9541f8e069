// FP32 kernels of the resident solve (resident.h): the refinement loop with
// FP32 inner solves.
#include "resident.h"

namespace gabp {

namespace {

template <int LANES>
ResKernel kernel32(int K, int mode) {
  if (mode == kResOuterLoop) return k_resident<float, LANES, 8, kResOuterLoop>;
  if (mode == kResSerialOuter) {
    if (K == 4) return k_resident<float, LANES, 4, kResSerialOuter>;
    return K == 6 ? k_resident<float, LANES, 6, kResSerialOuter> : k_resident<float, LANES, 8, kResSerialOuter>;
  }
  if (mode == kResRefine) {
    if (K == 4) return k_resident<float, LANES, 4, kResRefine>;
    return K == 6 ? k_resident<float, LANES, 6, kResRefine> : k_resident<float, LANES, 8, kResRefine>;
  }
  if (K == 4) return k_resident<float, LANES, 4, kResOuter>;
  if (K == 6) return k_resident<float, LANES, 6, kResOuter>;
  return k_resident<float, LANES, 8, kResOuter>;
}

}  // namespace

ResKernel res_kernel32(int lanes, int K, int mode) {
  if (lanes == 256) return kernel32<256>(K, mode);
  if (lanes == 512) return kernel32<512>(K, mode);
  return kernel32<kRL>(K, mode);
}

}  // namespace gabp
