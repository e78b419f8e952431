// The in-between MFMA kernel, bf16 operands.
#include "tac_mfma_mid_kernel.h"

namespace tac {

hipError_t mid_launch_bf16(const MidParams& p, int kp, int nmc, int nnp, hipStream_t s) {
  if (kp == 1) return mid_launch_bf16_kp<1, false>(p, nmc, nnp, s);
  if (kp == 2) return mid_launch_bf16_kp<2, false>(p, nmc, nnp, s);
  if (kp == 4) return mid_launch_bf16_kp<4, false>(p, nmc, nnp, s);
  return mid_launch_bf16_kp<8, false>(p, nmc, nnp, s);
}

}  // namespace tac
