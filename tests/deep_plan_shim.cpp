// The plan of the kernel for layers with too many channels for the other matrix-core kernels, for the tests that compare what it takes with what the
// vector kernel takes.
#include <cstring>
#include "tac_deep_plan.h"

static void layer_of(const tac_layer_desc_t* d, tac::LayerParams& p) {
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
}

// out: kp, pb, gb, flatten, rows per block, rows per tile, LDS rows, row tiles, channel tiles, segments, pixels per segment, bytes of LDS, bytes per group
extern "C" int deep_plan_of(const tac_layer_desc_t* d, int* out) {
  tac::LayerParams p;
  layer_of(d, p);
  tac::DeepPlan q;
  if (!tac::deep_choose(p, q)) return 0;
  const int v[] = {q.kp, q.pb, q.gb, q.flatten, q.rpb, q.tr, q.lr, q.row_tiles, q.co_tiles, q.nseg, q.xs, q.total, q.group};
  std::copy(std::begin(v), std::end(v), out);
  return 1;
}

// Frame loads of all rounds whose scalar offset is not inside the descriptor (of the last sample, whose descriptors are the shortest); -1: not the kernel's layer.
extern "C" long long deep_loads_outside(const tac_layer_desc_t* d) {
  tac::LayerParams p;
  layer_of(d, p);
  tac::DeepPlan q;
  if (!tac::deep_choose(p, q)) return -1;
  const long long chan = (long long)p.H * p.Wwi, frame = (long long)p.B * p.Cin * chan;
  const int n_groups = p.G + (p.K_last ? 1 : 0), channels = tac::deep_unit_channels(q.kp, tac::deep_wave_steps(q.nks));
  long long bad = 0;
  for (int g0 = 0; g0 < n_groups; g0 += q.gb) {
    const long long first = ((long long)g0 * p.K * p.B + p.B - 1) * p.Cin * chan;
    const long long bytes = std::min(((long long)(p.G * p.K + p.K_last) * frame - first) * 4, 0x7fffffffll);
    for (int j = 0; j < q.kp; ++j)
      for (int c = 0; c < channels; ++c)
        bad += tac::deep_scalar_offset(j, tac::deep_round_frames(g0, p.G, p.K, p.K_last), (uint32_t)frame, c, (uint32_t)chan) >= bytes;
  }
  return bad;
}
