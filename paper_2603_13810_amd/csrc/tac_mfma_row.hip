// The row kernel: host side.
#include "tac_mfma_row_kernel.h"

namespace tac {

hipError_t row_launch(const LayerParams& p, const RowPlan& q, hipStream_t s) {
  RowParams a;
  fill_params(a.m, p);
  a.q = q;
  a.K_last = p.K_last; a.n_lif_last = p.n_lif_last; a.decay_last = p.decay_last;
  return q.nnp == 1 ? row_launch_kp<1>(a, s) : row_launch_kp<2>(a, s);
}

}  // namespace tac
