// The in-between MFMA kernel, fp32 operands.
#include "tac_mfma_mid_kernel.h"

namespace tac {

hipError_t mid_launch_f32(const MidParams& p, int kp, int nnp, hipStream_t s) {
  if (kp == 1) return mid_launch_f32_kp<1, false>(p, nnp, s);
  if (kp == 2) return mid_launch_f32_kp<2, false>(p, nnp, s);
  if (kp == 4) return mid_launch_f32_kp<4, false>(p, nnp, s);
  return mid_launch_f32_kp<8, false>(p, nnp, s);
}

}  // namespace tac
