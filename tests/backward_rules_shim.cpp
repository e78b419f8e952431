// The host rules of the backward launch that choose between kernels, for the tests that hold them to what they are there for.
#include "tac_dgrad_plan.h"
#include "tac_wgrad_first_plan.h"

extern "C" int clear_in_recurrence(long long threads, long long floats) { return tac::backward_clear_in_recurrence((size_t)threads, (size_t)floats); }

// Its values per group (K = 0) or per frame of K (pool2: through that pool on load)
static void written_as(tac::BackwardParams& p, int K, int pool2) {
  p.grad_in_group = K == 0;
  p.K = std::max(1, K);
  p.pool2 = pool2;
}

extern "C" int input_gradient_on_matrix_cores(int G, int B, int Cin, int Cout, int H, int W, int stride, int K, int pool2) {
  tac::BackwardParams p{};
  written_as(p, K, pool2);
  p.G = G; p.B = B; p.Cin = Cin; p.Cout = Cout; p.H = H; p.W = W; p.stride = stride;
  return tac::backward_dgrad_f32_supported(p);
}

extern "C" void vector_kernel_tiles(int Cin, unsigned* out) { tac::dgrad_vector_tiles(Cin, out[0], out[1]); }

// Whether the four waves of a workgroup share the output channels (where the input gradient is formed on the matrix cores)
extern "C" int input_gradient_splits(int G, int B, int Cin, int Cout, int H, int W, int K, int pool2) {
  tac::BackwardParams p{};
  written_as(p, K, pool2);
  p.G = G; p.B = B; p.Cin = Cin; p.Cout = Cout; p.H = H; p.W = W; p.stride = 1;
  tac::DgradPlan q{};
  int np = 0;
  return tac::dgrad_f32_choose(p, q, np);
}

// out: groups of channels per workgroup, channel groups, slices, pairs per item, rows per item, strips, pair tiles, bytes of LDS.  0: not that kernel's layer.
extern "C" int first_weight_gradient(const tac_layer_desc_t* d, int* out) {
  tac::BackwardParams p{};
  p.B = d->B; p.Cin = d->Cin; p.H = d->H; p.W = d->W; p.Cout = d->Cout; p.stride = d->stride;
  p.Ho = (d->H - 1) / d->stride + 1;
  p.Wo = (d->W - 1) / d->stride + 1;
  p.pool2 = d->in_format == TAC_IN_BITS_POOL2 ? 1 : d->in_format == TAC_IN_BITS_MAXPOOL2 ? 2 : 0;
  p.dense = d->in_format == TAC_IN_F32;
  p.K = d->mode == TAC_PER_STEP ? 1 : std::min(d->K, d->T);
  p.K_last = d->T % p.K;
  p.G = (d->T + p.K - 1) / p.K;
  tac::FirstWgradPlan q{};
  if (!tac::first_wgrad_plan(p, q)) return 0;
  const int v[] = {q.ncg, q.co_groups, q.split, q.n_pairs, q.rows, q.n_strips, q.pair_tiles, q.total};
  std::copy(std::begin(v), std::end(v), out);
  return 1;
}
