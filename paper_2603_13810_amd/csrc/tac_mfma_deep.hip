// Layers with too many channels for the other matrix-core kernels: host side, and the kernels without recorded membranes.
#include "tac_mfma_deep_kernel.h"

namespace tac {

hipError_t deep_launch_plain(const DeepParams& p, hipStream_t s) { return deep_launch_any<false>(p, s); }

hipError_t deep_launch(const LayerParams& p, const DeepPlan& q, hipStream_t s) {
  DeepParams a;
  MfmaParams& mp = a.m;
  mp.spikes = p.spikes; mp.w = static_cast<const uint8_t*>(p.w); mp.bias = p.bias; mp.v_inout = p.v_inout;
  mp.out = p.out; mp.v_trace = p.v_trace;
  mp.B = p.B; mp.Cin = p.Cin; mp.H = p.H; mp.W = p.W; mp.Ho = p.Ho; mp.Wo = p.Wo; mp.Cout = p.Cout; mp.stride = p.stride;
  mp.K = p.K; mp.G = p.G; mp.n_lif = p.n_lif; mp.row_tiles = 0; mp.maxpool = 0; mp.pool = 0; mp.out_pool = p.out_pool;
  mp.decay = p.decay; mp.theta = p.theta;
  for (int j = 0; j < TAC_MAX_K; ++j) {
    const double w = (double)p.wj[j] * (double)(1u << kFixShift);
    mp.wq[j] = j < p.K ? (uint32_t)(w + 0.5) : 0u;
  }
  a.q = q;
  a.K_last = p.K_last; a.n_lif_last = p.n_lif_last; a.decay_last = p.decay_last;
  return p.v_trace ? deep_launch_trace(a, s) : deep_launch_plain(a, s);
}

}  // namespace tac
