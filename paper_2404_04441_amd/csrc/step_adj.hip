// Instantiation unit: the float32 adjoint step kernels, without and with the imaging sums.
#include "step_kernels.h"

namespace wave {

hipError_t launch_variant_adj(int v, const StepArgs &a, hipStream_t s) {
  return a.img ? launch_variant<kF32, kImaging>(v, a, s) : launch_variant<kF32, kAdjoint>(v, a, s);
}

}  // namespace wave
