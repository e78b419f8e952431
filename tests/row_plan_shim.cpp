// The plan of the row kernel, for the tests of what it takes and of whether its tiles cover the layer.
#include <cstring>
#include "tac_row_plan.h"

// out: kp, waves over the pixels, over the channels, blocks per wave, waves, rows counted through samples, segments per row, rows per tile, LDS rows, row tiles, channel tiles,
// blocks of 8 channels per job, jobs over the rows, rows per job, jobs, bytes of LDS, k-steps
extern "C" int row_plan_of(const tac_layer_desc_t* d, int traced, int nmc_w, int* out) {
  tac::LayerParams p;
  std::memset(&p, 0, sizeof(p));
  p.B = d->B; p.Cin = d->Cin; p.H = d->H; p.W = d->W; p.Cout = d->Cout; p.stride = d->stride;
  p.Ho = (d->H - 1) / d->stride + 1;
  p.Wo = (d->W - 1) / d->stride + 1;
  p.pool2 = d->in_format == TAC_IN_BITS_POOL2 ? 1 : d->in_format == TAC_IN_BITS_MAXPOOL2 ? 2 : 0;
  p.dense = d->in_format == TAC_IN_F32;
  p.out_pool = d->out_format == TAC_OUT_BITS_MAXPOOL2;
  p.Hs = p.pool2 ? 2 * d->H : d->H;
  p.Wwi = ((p.pool2 ? 2 * d->W : d->W) + 31) / 32;
  p.Wwo = (p.Wo + 31) / 32;
  p.K = d->mode == TAC_PER_STEP ? 1 : std::min(d->K, d->T);
  p.G = d->T / p.K;
  p.K_last = d->T % p.K;
  p.n_lif = d->mode == TAC_PRESERVE ? p.K : 1;
  p.bf16 = d->precision == TAC_BF16;
  float trace = 0.f;
  p.v_trace = traced ? &trace : nullptr;
  tac::RowPlan q;
  if (!tac::row_choose(p, q, nmc_w)) return 0;
  const int v[] = {q.kp, q.pw, q.nco, q.nnp, q.waves, q.flatten, q.spr, q.tr, q.lr, q.row_tiles, q.co_tiles, q.cb, q.parts, q.lrp, q.n_jobs, q.total, q.nks};
  std::copy(std::begin(v), std::end(v), out);
  return 1;
}
