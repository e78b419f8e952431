// Layers with too many channels for the other matrix-core kernels, with recorded membranes.
#include "tac_mfma_deep_kernel.h"

namespace tac {

hipError_t deep_launch_trace(const DeepParams& p, hipStream_t s) { return deep_launch_any<true>(p, s); }

}  // namespace tac
