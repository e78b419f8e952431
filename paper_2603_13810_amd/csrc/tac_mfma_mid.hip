// Host side of the MFMA kernel for the layers in between (tac_mfma_mid_kernel.h has the kernel): which layers it takes,
// their prepared weights, and the tile a launch uses.
#include <algorithm>
#include <cmath>
#include "tac_mfma_mid_kernel.h"
#include "tac_plan_memo.h"

namespace tac {

namespace {

constexpr int kMidMaxW = 128, kMidMaxWo = 64, kMidMaxCin = 128;
constexpr int kMidLds = 160 * 1024;

// Which layers the kernel takes, and in tiles of how many 32-channel blocks their weights are laid out: four output rows
// of aggregates and the weights of a tile of output channels have to fit this much LDS together.
constexpr int kMidRows = 4;
constexpr int kMidLdsRule = 150 * 1024;

int mid_k_steps(int Cin, bool f32) { return f32 ? (9 * Cin + 1) / 2 : (9 * Cin + 15) / 16; }

int mid_rule_bytes(int Cin, int S, int W, int nmc, bool f32) {
  const int rows_in = (kMidRows - 1) * S + 3, nks = mid_k_steps(Cin, f32);
  const int a_bytes = ((rows_in * (W + 2) * Cin + 8) * (f32 ? 4 : 2) + 15) & ~15;
  return a_bytes + nks * nmc * 64 * (f32 ? 4 : 16) + ((nks * 2 * 4 + 15) & ~15) + nmc * 32 * 4;
}

// OIHW fp32 -> [cout tile][k-step][mc][lane][8] bf16: lane l of block mc holds cout
// 32 (tile nmc + mc) + l % 32 and the contraction slots kk = 16 ks + 8 (l / 32) + i with
// kk = tap * Cin + cin; slots beyond 9 Cin and channels beyond Cout are zero.
__global__ void mid_prepare_kernel(const float* __restrict__ w, uint32_t* __restrict__ out, int Cin, int Cout, int nmc,
                                   int nks, int total) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;                // one thread per bf16 pair
  if (i >= total) return;
  int t = i;
  const int e2 = t & 3; t >>= 2;
  const int l = t & 63; t >>= 6;
  const int mc = t % nmc; t /= nmc;
  const int ks = t % nks;
  const int tile = t / nks;
  const int co = (tile * nmc + mc) * 32 + (l & 31);
  float v[2];
  for (int u = 0; u < 2; ++u) {
    const int kk = 16 * ks + 8 * (l >> 5) + 2 * e2 + u;
    const int tap = kk / Cin, cin = kk - tap * Cin;
    v[u] = (tap < 9 && co < Cout) ? w[((size_t)co * Cin + cin) * 9 + tap] : 0.f;
  }
  out[i] = pack_bf16(v[0], v[1]);
}

// fp32: OIHW -> [cout tile][k-step][mc][lane] float32: lane l of block mc holds cout 32 (tile nmc + mc) + l % 32 and
// the contraction slot kk = 2 ks + l / 32 = tap * Cin + cin; slots beyond 9 Cin and channels beyond Cout are zero.
__global__ void mid_prepare_f32_kernel(const float* __restrict__ w, float* __restrict__ out, int Cin, int Cout, int nmc, int nks,
                                       int total) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= total) return;
  int t = i;
  const int l = t & 63; t >>= 6;
  const int mc = t % nmc; t /= nmc;
  const int ks = t % nks;
  const int tile = t / nks;
  const int co = (tile * nmc + mc) * 32 + (l & 31);
  const int kk = 2 * ks + (l >> 5);
  const int tap = kk / Cin, cin = kk - tap * Cin;
  out[i] = (tap < 9 && co < Cout) ? w[((size_t)co * Cin + cin) * 9 + tap] : 0.f;
}

// 64-channel tiles when the tile's weights and the aggregate tile fit the LDS together, else 32
int mid_nmc(int Cin, int S, int W, int Cout, bool f32) {
  return (!f32 && Cout > 32 && mid_rule_bytes(Cin, S, W, 2, f32) <= kMidLdsRule) ? 2 : 1;
}

size_t mid_tile_bytes(const tac_layer_desc_t& d, int nmc, bool f32) { return (size_t)mid_k_steps(d.Cin, f32) * nmc * 64 * (f32 ? 4 : 16); }

// Cycles of a wave's job: its chunks of words, then the passes over its pixels as build_job makes them (a last pass of 64 or
// fewer is a narrow one; sums take two at a time, single frames one; the mean pool goes over the four pixels of a block, the
// max pool reads all four first).
double mid_job_cycles(const MidPlan& q, const LayerParams& p) {
  const int n_px = q.cg * q.lrp * p.W;
  const bool sums = q.nb > 1 || p.pool2 == 1 || !p.bf16;
  const double corners = p.pool2 == 1 ? 4.0 : 1.0, reads = p.pool2 == 2 ? 300.0 : 0.0;
  double passes;
  if (sums && p.K == 1) passes = ((n_px + 63) / 64) * (300.0 + 400.0 * corners + reads);
  else if (sums) passes = ((n_px + 127) / 128) * q.nb * (600.0 * corners + reads);
  else if (p.K == 1) passes = n_px <= 64 ? 300.0 + reads : ((n_px + 127) / 128) * (450.0 + reads);
  else passes = (n_px / 256 + (n_px % 256 > 64)) * (700.0 + 2.0 * reads) + (n_px % 256 && n_px % 256 <= 64 ? 350.0 + reads : 0.0);
  // (a second batch of words is asked for when the first has been staged, and waited for)
  return 1000.0 + 500.0 * q.chunks + 600.0 * (q.batches - 1) + passes;
}

// The plan of one tile shape, or false when it does not fit the LDS.  pw_shift: lanes per row of a block (their log2),
// trg: row groups per tile.
bool mid_plan(MidPlan& q, const LayerParams& p, int kp, int nmc, int nnp, int pw_shift, int trg, bool flatten, int nmc_w, int split = 0, int nco = 1) {
  const bool f32 = !p.bf16;
  const int four = split ? 2 : nco, threads = four * kMidThreads;      // loaders counts waves of every four
  q.split = split;
  q.nco = nco;
  const int S = p.stride, C8 = p.Cin / 8;
  q.pw_shift = pw_shift;
  q.rpb = 32 >> q.pw_shift;
  q.wb = (p.Wo + 31) / 32;
  q.trg = trg;
  q.tr = trg * q.rpb;
  q.flatten = flatten;
  const long long rows = flatten ? (long long)p.B * p.Ho : p.Ho;
  q.tr = (int)std::min<long long>(q.tr, p.out_pool ? (rows + 1) / 2 * 2 : rows);
  const int samples = flatten ? std::min((q.tr + p.Ho - 2) / p.Ho + 1, p.B) : 1;        // a tile may touch
  q.lr = (q.tr - 1) * S + 3 + (samples - 1) * (3 - S);
  q.row_tiles = (int)((rows + q.tr - 1) / q.tr);
  q.co_tiles = (p.Cout + nco * nmc * 32 - 1) / (nco * nmc * 32);
  q.srows = p.pool2 ? 2 : 1;
  q.wws = p.Wwi;
  q.hs = p.Hs;
  q.nb = (p.K + kp - 1) / kp;
  q.rws = q.nb * kp * 8 + 4;                   // four unused dwords spread consecutive pairs over the LDS banks
  q.wpx = p.W + 2;
  q.xh = (q.wpx + 1) / 2;
  q.plane = q.lr * q.wpx * 16;
  q.plane += (128 - q.plane % 256 + 256) % 256;       // consecutive planes start half the banks apart (the two lane halves)
  q.nks = mid_k_steps(p.Cin, f32);
  q.nmc_w = nmc_w;
  auto up = [](int x) { return (x + 15) & ~15; };
  const int w_bytes = split ? 0 : q.nks * nco * nmc * (f32 ? 256 : 1024);
  const int ahead = split ? 0 : (2 * mid_depth(nmc, nnp) - 1) * nmc * 1024;    // the fetches ahead read past the weights
  const int parts_bytes = split ? 8 * 4096 : 0;                       // the waves' partial sums, behind everything else
  const bool sums = f32 || q.nb > 1 || p.pool2 == 1;
  const int lut_entries = sums ? q.nb << kp : (kp == 8 ? 256 : 1 << (2 * kp));
  q.off_w = q.plane * C8 * (f32 ? 2 : 1);
  q.off_tab = q.off_w + w_bytes;
  q.off_bias = up(q.off_tab + (q.nks * 2 + kMidTabPad) * 4);
  q.off_wq = q.off_bias + nco * nmc * 32 * 4;
  q.off_lut = q.off_wq + TAC_MAX_K * 4;
  q.off_unit = up(q.off_lut + lut_entries * 4);
  // groups of one or two frames on few channels: see the kernel's build_direct
  q.direct = nco == 1 && kp <= 2 && (kp == 1 || !p.pool2) && C8 * q.lr * p.W <= kMidDirect * threads;
  if (q.direct) {
    q.n_jobs = 0;
    q.loaders = 4;
    q.parts = 1;
    q.parts_shift = 0;
    q.lrp = q.lr;
    q.cg = C8;
    q.chunks = q.batches = q.rw = q.stage_wave = 0;
    q.off_px = q.off_stage = q.off_unit;
    q.off_part = up(std::max(q.off_unit, q.off_w + w_bytes + ahead));
    q.total = q.off_part + parts_bytes;
    return q.total <= kMidLds;
  }
  // Four waves form aggregates, each in as few jobs as the LDS has room to stage; fewer waves only where even the smallest
  // jobs of four do not fit (rows of 100 and more pixels in groups of 16 and more frames).
  bool found = false;
  double best = 0.0;
  MidPlan c = q;
  for (c.loaders = 4; c.loaders >= 1 && !found; c.loaders >>= 1)
    for (c.parts_shift = 0; c.parts_shift <= 6; ++c.parts_shift) {
      c.parts = 1 << c.parts_shift;
      c.lrp = (c.lr + c.parts - 1) / c.parts;
      if (c.parts > 1 && (c.lr + c.parts / 2 - 1) / (c.parts / 2) == 1) break;  // a row each already
      for (c.cg = C8; c.cg >= 1; --c.cg) {
        if (C8 % c.cg) continue;
        c.n_jobs = C8 / c.cg * c.parts;
        c.rw = c.lrp * c.srows * c.wws;
        const int n_units = 8 * c.cg * c.rw, n_px = c.cg * c.lrp * p.W;
        c.chunks = c.nb * ((n_units + 64 * mid_units(kp) - 1) / (64 * mid_units(kp)));
        c.batches = (c.chunks + kMidBatch - 1) / kMidBatch;
        c.off_px = up(c.off_unit + c.parts * n_units * 8);
        c.off_stage = up(c.off_px + c.parts * n_px * 8);
        c.stage_wave = up(c.cg * c.rw * c.rws * 4);
        c.off_part = up(std::max(c.off_stage + four * c.loaders * c.stage_wave, c.off_w + w_bytes + ahead));
        c.total = c.off_part + parts_bytes;
        if (c.total > kMidLds || c.stage_wave >= 1 << 24) continue;
        const double cost = (double)((c.n_jobs + four * c.loaders - 1) / (four * c.loaders)) * mid_job_cycles(c, p);
        // a second workgroup per compute unit is worth more than a job less
        const double scaled = cost * (c.total > kMidLds / 2 && c.off_px < kMidLds / 2 ? 1.3 : 1.0);
        if (found && scaled >= best) continue;
        found = true;
        best = scaled;
        q = c;
      }
    }
  return found;
}

// Estimated time of a launch in cycles: rounds of resident workgroups, each the sum of its phases (instructions of the
// loader; MFMAs, 32 cycles per 32x32x16 and 64 per fp32 32x32x2, or the LDS reads that feed them at 128 bytes per cycle;
// LIF steps).  Resident workgroups fill each other's gaps, but share the LDS and the matrix cores.  The figures are fitted to
// what the tiles of some hundred layers take; over 440 layers of all kinds the chosen tiles are 1.11 times as fast as with
// a coarser estimate (passes of 256 pixels whatever the job, two residents at most), which put single frames of few channels
// on one workgroup per compute unit.
double mid_cost(const MidPlan& q, const LayerParams& p, int nmc, int nnp) {
  const bool f32 = !p.bf16;
  const double build = q.direct ? 500.0 + 400.0 * ((p.Cin / 8 * q.lr * p.W + kMidThreads - 1) / kMidThreads) * (p.K == 2 || p.pool2 ? 2 : 1)
                                : (q.n_jobs + q.nco * q.loaders - 1) / (q.nco * q.loaders) * mid_job_cycles(q, p);
  // (an fp32 step waits for its operands: a wave alone takes about 90 cycles for one block)
  const double busy = q.nks * (f32 ? 64.0 * nnp : std::max(32.0 * nmc * nnp, 32.0 * (nmc + nnp))) + 300.0;
  const double mfma = f32 ? q.nks * 90.0 * nnp + 300.0 : busy;
  const double lif = p.n_lif * (nmc * nnp * (p.v_trace ? 1200.0 : 500.0) + 400.0 + 60.0 * q.rpb);
  const double wgs = (double)q.row_tiles * q.co_tiles * (q.flatten ? 1 : p.B);
  const double per_cu = std::ceil(wgs / 256.0);
  // workgroups that share a compute unit: as the LDS allows, and the registers (words of the threads' own and single frames leave
  // room for more than two with one or two accumulator blocks); 1003 workgroups of 8 -> 32 at 59 x 39, four a unit, take as
  // long as 502, two a unit
  const int blocks = nmc * nnp, by_registers = f32 || blocks > 2 || !(q.direct || p.K == 1) ? 2 : blocks == 1 ? 4 : 3;
  const int resident = std::min(q.nco == 1 ? by_registers : 1, kMidLds / q.total);
  const double together = std::min<double>(resident, per_cu) * q.nco;         // sets of four waves
  const double alone = 9000.0 + p.G * (build + mfma + lif + 500.0);
  const double shared = p.G * busy;                                     // what other workgroups cannot hide
  return std::ceil(per_cu / resident) * std::max(alone * (together > 1 ? 1.1 + 0.025 * together : 1.0), together * shared);
}

}  // namespace

bool mfma_mid_supported(const tac_layer_desc_t& d) {
  if (d.in_format == TAC_IN_F32) return false;
  const bool f32 = d.precision == TAC_FP32;
  if (d.Cin % 8 != 0 || d.Cin > kMidMaxCin) return false;
  if (d.W > kMidMaxW || (d.W + 2 - 3) / d.stride + 1 > kMidMaxWo) return false;
  return mid_rule_bytes(d.Cin, d.stride, d.W, mid_nmc(d.Cin, d.stride, d.W, d.Cout, f32), f32) <= kMidLdsRule;
}

int mfma_mid_weight_blocks(const LayerParams& p) { return mid_nmc(p.Cin, p.stride, p.W, p.Cout, !p.bf16); }

size_t mfma_mid_weight_bytes(const tac_layer_desc_t& d) {
  const bool f32 = d.precision == TAC_FP32;
  const int nmc = mid_nmc(d.Cin, d.stride, d.W, d.Cout, f32);
  const int tiles = (d.Cout + nmc * 32 - 1) / (nmc * 32);
  return (size_t)tiles * mid_tile_bytes(d, nmc, f32);
}

hipError_t mfma_mid_prepare(const tac_layer_desc_t& d, const float* w_oihw, void* w_prepared, hipStream_t s) {
  const bool f32 = d.precision == TAC_FP32;
  const int nmc = mid_nmc(d.Cin, d.stride, d.W, d.Cout, f32);
  const int tiles = (d.Cout + nmc * 32 - 1) / (nmc * 32);
  if (f32) {
    const int nks2 = (9 * d.Cin + 1) / 2;
    const int total = tiles * nks2 * nmc * 64;
    hipLaunchKernelGGL(mid_prepare_f32_kernel, dim3((total + 255) / 256), dim3(256), 0, s, w_oihw,
                       static_cast<float*>(w_prepared), d.Cin, d.Cout, nmc, nks2, total);
    return hipGetLastError();
  }
  const int nks = (9 * d.Cin + 15) / 16;
  const int total = tiles * nks * nmc * 64 * 4;
  hipLaunchKernelGGL(mid_prepare_kernel, dim3((total + 255) / 256), dim3(256), 0, s, w_oihw,
                     static_cast<uint32_t*>(w_prepared), d.Cin, d.Cout, nmc, nks, total);
  return hipGetLastError();
}

// Small images on many channels: eight waves share the pixel blocks of a workgroup (the kernel's SPLIT), as long as there are few of them:
// 512 blocks of 32 pixels x 32 channels.  Beyond that the four-wave tiles fill their waves and the exchange of partial sums costs more
// than it gives (us, split / not: 128 -> 128 at 16 x 16, K = 4, B = 16 (512) 23.5 / 33; B = 64 92 / 72; 64 -> 64 at 10 x 10, B = 128 (1280) 47 / 29).
// The two sum the products in different orders, so that a sample's last bits differ between the two sides of this line, the batch included.
static bool mid_split_rule(const LayerParams& p) {
  if (!p.bf16 || p.pool2 || p.Cin < 64 || p.Wo > 16) return false;
  const int rows = p.Wo > 8 ? 2 : p.Wo > 4 ? 4 : p.Wo > 2 ? 8 : 16;    // of a block
  return ((long long)p.B * p.Ho + rows - 1) / rows * ((p.Cout + 31) / 32) <= 512;
}

// Estimated time of such a launch, as mid_cost
static double mid_split_cost(const MidPlan& q, const LayerParams& p) {
  const int own = kMidRanges / q.split, regs = 16 / q.split, loaders = 2 * q.loaders;
  const double build = q.direct ? 500.0 + 400.0 * ((p.Cin / 8 * q.lr * p.W + 511) / 512) * (p.K == 2 ? 2 : 1)
                                : (q.n_jobs + loaders - 1) / loaders * mid_job_cycles(q, p);
  const double mfma = own * (400.0 + q.nks / 8.0 * 64.0) + 900.0;
  const double lif = p.n_lif * (200.0 + 40.0 * regs + 60.0 * q.rpb + (p.v_trace ? 20.0 * regs : 0.0));
  const double wgs = (double)q.row_tiles * q.co_tiles * (q.flatten ? 1 : p.B);
  const int resident = std::min(2, kMidLds / q.total);
  const double per_cu = std::ceil(wgs / 256.0), together = std::min<double>(resident, per_cu);
  return std::ceil(per_cu / resident) * (7000.0 + p.G * (build + mfma + lif + 300.0)) * (together > 1 ? 1.5 : 1.0);
}

static bool mid_choose(const LayerParams& p, MidParams& out, int& kp, int& nmc, int& nnp) {
  const bool f32 = !p.bf16;
  kp = p.K <= 2 ? p.K : p.K <= 4 ? 4 : 8;
  const int nmc_w = mid_nmc(p.Cin, p.stride, p.W, p.Cout, f32);
  const int wb = (p.Wo + 31) / 32;
  // a tile that straddles samples offsets its membranes by 32 bits and counts rows in fp32
  const bool may_flatten = (long long)p.B * p.Cout * p.Ho * p.Wo < (1ll << 30) && (long long)p.B * p.Ho < (1ll << 20) - 1024;
  double best = 0.0;
  bool found = false;
  if (mid_split_rule(p)) {
    const int pw = p.Wo > 8 ? 4 : p.Wo > 4 ? 3 : p.Wo > 2 ? 2 : 1;
    for (int split = 8; split >= 4; split /= 2)
      for (int fl = may_flatten ? 1 : 0; fl >= 0; --fl) {
        MidPlan q;
        if (!mid_plan(q, p, kp, 1, 1, pw, 8 / split, fl != 0, nmc_w, split)) continue;
        const double cost = mid_split_cost(q, p);
        if (found && cost >= best) continue;
        found = true;
        best = cost;
        out.q = q;
        nmc = nnp = 1;
      }
    if (found) return true;
  }
  const int max_nco = f32 && kp > 1 && p.Cin >= 16 && p.Cout > 32 ? 2 : 1;
  // as many rows per block as its lanes hold; fewer only where such a tile does not fit the LDS
  for (int pw = p.Wo > 16 ? 5 : p.Wo > 8 ? 4 : p.Wo > 4 ? 3 : p.Wo > 2 ? 2 : 1; pw <= 5 && !found; ++pw)
    for (int nco = 1; nco <= max_nco; ++nco)
      for (int c = 1; c <= (f32 || p.Cout <= 32 || nco > 1 ? 1 : 2); ++c)
        for (int x = 2; x >= 1; --x)
          for (int trg = 4 * x / wb; trg >= 1; trg >>= 1) {
            // pooled output, one row per block: the wave's two blocks are the two rows of a pooled row
            const bool pairs = p.out_pool && pw == 5;
            if (pairs && (x == 1 || trg < 2)) continue;
            if (f32 && x == 2 && (!pairs || nco > 1)) continue; // two blocks with four partial sums each: one wave per SIMD
            for (int fl = may_flatten ? 1 : 0; fl >= 0; --fl) {
              MidPlan q;
              if (!mid_plan(q, p, kp, c, x, pw, trg, fl != 0, nmc_w, 0, nco)) continue;
              const double cost = mid_cost(q, p, c, x) * (nco > 1 ? 1.05 : 1.0);     // (where the estimates are close it is not faster)
              // of equals the one that does not straddle samples, and of tiles that all have a compute unit to themselves the
              // smaller one, both of which are tried later
              const long long wgs = (long long)q.row_tiles * q.co_tiles * (q.flatten ? 1 : p.B);
              if (found && (cost > best || (cost == best && wgs > 256 && q.flatten))) continue;
              found = true;
              best = cost;
              out.q = q;
              nmc = c;
              nnp = x;
            }
          }
  return found;
}

hipError_t mfma_mid_launch(const LayerParams& p, hipStream_t s) {
  MidParams a;
  fill_params(a.m, p);
  a.K_last = p.K_last; a.n_lif_last = p.n_lif_last; a.decay_last = p.decay_last;
  // The choice looks at some hundred tiles (up to 18 us); the geometries a thread has asked for lately are remembered.
  struct Choice {
    MidPlan q;
    int kp, nmc, nnp;
  };
  static thread_local PlanMemo<14, Choice> known;
  const int key[14] = {p.B, p.Cin, p.H, p.W, p.Cout, p.stride, p.K, p.G, p.n_lif, p.pool2, p.out_pool, p.bf16, p.Wwi, p.v_trace != nullptr};
  const Choice* const e = known.of(key, [&](Choice& n) {
    if (!mid_choose(p, a, n.kp, n.nmc, n.nnp)) return false;
    n.q = a.q;
    return true;
  });
  if (!e) return hipErrorInvalidValue;
  a.q = e->q;
  const int kp = e->kp, nmc = e->nmc, nnp = e->nnp;
  if (!p.bf16) return p.v_trace ? mid_launch_f32_trace(a, kp, nnp, s) : mid_launch_f32(a, kp, nnp, s);
  return p.v_trace ? mid_launch_bf16_trace(a, kp, nmc, nnp, s) : mid_launch_bf16(a, kp, nmc, nnp, s);
}

}  // namespace tac
