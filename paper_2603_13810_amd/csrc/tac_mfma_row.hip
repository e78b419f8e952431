// The row kernel: host side.
#include "tac_mfma_row_kernel.h"

namespace tac {

hipError_t row_launch(const LayerParams& p, const RowPlan& q, hipStream_t s) {
  RowParams a;
  MfmaParams& mp = a.m;
  mp.spikes = p.spikes; mp.w = static_cast<const uint8_t*>(p.w); mp.bias = p.bias; mp.v_inout = p.v_inout;
  mp.out = p.out; mp.v_trace = nullptr;
  mp.B = p.B; mp.Cin = p.Cin; mp.H = p.H; mp.W = p.W; mp.Ho = p.Ho; mp.Wo = p.Wo; mp.Cout = p.Cout; mp.stride = p.stride;
  mp.K = p.K; mp.G = p.G; mp.n_lif = p.n_lif; mp.row_tiles = 0; mp.maxpool = 0; mp.pool = 0; mp.out_pool = 0;
  mp.decay = p.decay; mp.theta = p.theta;
  for (int j = 0; j < TAC_MAX_K; ++j) {
    const double w = (double)p.wj[j] * (double)(1u << kFixShift);
    mp.wq[j] = j < p.K ? (uint32_t)(w + 0.5) : 0u;
  }
  a.q = q;
  a.K_last = p.K_last; a.n_lif_last = p.n_lif_last; a.decay_last = p.decay_last;
  return q.nnp == 1 ? row_launch_kp<1>(a, s) : row_launch_kp<2>(a, s);
}

}  // namespace tac
