// The in-between MFMA kernel, bf16 operands, with the membrane trace.
#include "tac_mfma_mid_kernel.h"

namespace tac {

hipError_t mid_launch_bf16_trace(const MidParams& p, int kp, int nmc, int nnp, hipStream_t s) {
  if (kp == 1) return mid_launch_bf16_kp<1, true>(p, nmc, nnp, s);
  if (kp == 2) return mid_launch_bf16_kp<2, true>(p, nmc, nnp, s);
  if (kp == 4) return mid_launch_bf16_kp<4, true>(p, nmc, nnp, s);
  return mid_launch_bf16_kp<8, true>(p, nmc, nnp, s);
}

}  // namespace tac
