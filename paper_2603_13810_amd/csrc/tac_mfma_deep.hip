// Layers with too many channels for the other matrix-core kernels: host side, and the kernels without recorded membranes.
#include "tac_mfma_deep_kernel.h"

namespace tac {

hipError_t deep_launch_plain(const DeepParams& p, hipStream_t s) { return deep_launch_any<false>(p, s); }

hipError_t deep_launch(const LayerParams& p, const DeepPlan& q, hipStream_t s) {
  DeepParams a;
  fill_params(a.m, p);
  a.q = q;
  a.K_last = p.K_last; a.n_lif_last = p.n_lif_last; a.decay_last = p.decay_last;
  return p.v_trace ? deep_launch_trace(a, s) : deep_launch_plain(a, s);
}

}  // namespace tac
