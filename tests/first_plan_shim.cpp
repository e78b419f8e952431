// The host rules of the first layers' kernel, for the tests that hold them to what they are there for.
#include "tac_first_plan.h"

static tac::LayerParams params_of(const tac_layer_desc_t* d) {
  tac::LayerParams p{};
  p.B = d->B; p.Cin = d->Cin; p.H = d->H; p.W = d->W; p.Cout = d->Cout; p.stride = d->stride;
  p.Ho = (d->H - 1) / d->stride + 1;
  p.Wo = (d->W - 1) / d->stride + 1;
  p.Wwo = (p.Wo + 31) / 32;
  p.pool2 = d->in_format == TAC_IN_BITS_POOL2 ? 1 : d->in_format == TAC_IN_BITS_MAXPOOL2 ? 2 : 0;
  p.out_pool = d->out_format == TAC_OUT_BITS_MAXPOOL2;
  p.vector_only = d->kernel == TAC_KERNEL_DIRECT;
  p.bf16 = d->precision == TAC_BF16;
  return p;
}

// out: pairs, blocks, pair tiles, channel tiles, workgroups, bytes of LDS
extern "C" void first_plan_of(const tac_layer_desc_t* d, int with_trace, int with_state, long long* out) {
  tac::LayerParams p = params_of(d);
  float somewhere;
  p.v_trace = with_trace ? &somewhere : nullptr;
  p.v_inout = with_state ? &somewhere : nullptr;
  const tac::FirstPlan q = tac::first_plan(p);
  const long long v[] = {q.pairs, q.blocks, q.pair_tiles, q.co_tiles, q.workgroups, (long long)q.lds};
  for (int i = 0; i < 6; ++i) out[i] = v[i];
}

extern "C" int fp32_layer_on_matrix_cores(const tac_layer_desc_t* d) { return tac::first_f32_supported(params_of(d)); }
