// Instantiation unit: the gradient's float32 step kernels (forward steps that
// also store the Laplacian, adjoint steps without and with the imaging sums).
#include "step_kernels.h"

namespace wave {

hipError_t launch_variant_lap(int v, const StepArgs &a, hipStream_t s) { return launch_variant<kF32, kStoreLap>(v, a, s); }

hipError_t launch_variant_adj(int v, const StepArgs &a, hipStream_t s) {
  return a.img ? launch_variant<kF32, kImaging>(v, a, s) : launch_variant<kF32, kAdjoint>(v, a, s);
}

}  // namespace wave
