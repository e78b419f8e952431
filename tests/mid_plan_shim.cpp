// The plan of the in-between kernel's launch for a layer, for the tests that say which of its variants a case takes: the host
// side of the kernel compiled into a library of its own, with the launches left out.
#include "tac_mfma_mid.hip"

namespace tac {
hipError_t mid_launch_bf16(const MidParams&, int, int, int, hipStream_t) { return hipSuccess; }
hipError_t mid_launch_bf16_trace(const MidParams&, int, int, int, hipStream_t) { return hipSuccess; }
hipError_t mid_launch_f32(const MidParams&, int, int, hipStream_t) { return hipSuccess; }
hipError_t mid_launch_f32_trace(const MidParams&, int, int, hipStream_t) { return hipSuccess; }
}  // namespace tac

// out (mid_plan_of): kp, nmc, nnp, direct, jobs, loaders, batches, flatten, rows per block, workgroups, bytes of LDS, split, nco.  0: the kernel does not
// take the layer, -1: no tile fits.
static tac::LayerParams params_of(const tac_layer_desc_t* d, float* trace) {
  tac::LayerParams p;
  std::memset(&p, 0, sizeof(p));
  p.v_trace = trace;
  p.B = d->B; p.Cin = d->Cin; p.H = d->H; p.W = d->W; p.Cout = d->Cout; p.stride = d->stride;
  p.Ho = (d->H - 1) / d->stride + 1;
  p.Wo = (d->W - 1) / d->stride + 1;
  p.pool2 = d->in_format == TAC_IN_BITS_POOL2 ? 1 : d->in_format == TAC_IN_BITS_MAXPOOL2 ? 2 : 0;
  p.out_pool = d->out_format == TAC_OUT_BITS_MAXPOOL2;
  p.Hs = p.pool2 ? 2 * d->H : d->H;
  p.Wwi = ((p.pool2 ? 2 * d->W : d->W) + 31) / 32;
  p.Wwo = (p.Wo + 31) / 32;
  p.K = d->mode == TAC_PER_STEP ? 1 : std::min(d->K, d->T);
  p.G = d->T / p.K;
  p.n_lif = d->mode == TAC_PRESERVE ? p.K : 1;
  p.bf16 = d->precision == TAC_BF16;
  return p;
}

extern "C" int mid_plan_of(const tac_layer_desc_t* d, int with_trace, int* out) {
  if (!tac::mfma_mid_supported(*d)) return 0;
  float trace;
  const tac::LayerParams p = params_of(d, with_trace ? &trace : nullptr);
  tac::MidParams a;
  int kp, nmc, nnp;
  if (!tac::mid_choose(p, a, kp, nmc, nnp)) return -1;
  const tac::MidPlan& q = a.q;
  const int v[] = {kp, nmc, nnp, q.direct, q.n_jobs, q.loaders, q.batches, q.flatten, q.rpb,
                   q.row_tiles * q.co_tiles * (q.flatten ? 1 : p.B), q.total, q.split, q.nco};
  std::copy(std::begin(v), std::end(v), out);
  return 1;
}

// Everything a launch does on the host, for timing it.
extern "C" int mid_launch_of(const tac_layer_desc_t* d) { return tac::mfma_mid_launch(params_of(d, nullptr), nullptr); }
