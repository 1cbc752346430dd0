// Instantiation unit: the float32 forward step kernels that also store the Laplacian.
#include "step_kernels.h"

namespace wave {

hipError_t launch_variant_lap(int v, const StepArgs &a, hipStream_t s) { return launch_variant<kF32, kStoreLap>(v, a, s); }

}  // namespace wave
