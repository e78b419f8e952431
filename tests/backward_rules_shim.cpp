// The host rules of the backward launch that choose between kernels, for the tests that hold them to what they are there for.
#include "tac_internal.h"

extern "C" int clear_in_recurrence(long long threads, long long floats) { return tac::backward_clear_in_recurrence((size_t)threads, (size_t)floats); }

extern "C" int input_gradient_on_matrix_cores(int G, int B, int Cin, int H, int W, int stride) {
  tac::BackwardParams p{};
  p.G = G; p.B = B; p.Cin = Cin; p.H = H; p.W = W; p.stride = stride;
  return tac::backward_dgrad_f32_supported(p);
}
