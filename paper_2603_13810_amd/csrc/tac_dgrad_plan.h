// Host rules of the input gradient's fp32 kernels (tac_backward_dgrad_f32.hip; dgrad_kernel in tac_backward.hip).
#pragma once
#include <algorithm>
#include "tac_mfma_common.h"

namespace tac {

constexpr int kDgradThreads = 256;
constexpr int kDgradCo = 16;      // output channels per round
constexpr int kDgradM = 2;        // dY values per thread and channel
constexpr int kSplitCo = 32;      // output channels per round of the kernel whose waves share them, eight for each of the four
constexpr int kSplitPl = 112;     // dwords of dY per channel at most

struct DgradPlan {
  int rows, xw, n_pairs;          // a tile: rows x columns of n_pairs (group, sample) pairs
  int n_strips, n_segs, pair_tiles, ci_groups;
  int px, pl, cw;                 // pixels of a tile, dwords per channel of dY in LDS (with border), per row
  int vec_w;                      // the weights can be read 16 bytes at a time
  int off_dy, off_bad, total;
};

// Tiles of 32 input channels and up to `blocks` blocks of 32 pixels with up to pl_max positions of dY
inline bool dgrad_f32_tile(const BackwardParams& p, int blocks, int pl_max, DgradPlan& q) {
  const int px_max = blocks * 32;
  q.xw = std::min(p.W, std::min(64, px_max));
  q.n_segs = (p.W + q.xw - 1) / q.xw;
  q.cw = q.xw + 2;
  for (q.rows = std::min(p.H, px_max / q.xw); q.rows >= 1; --q.rows)
    if ((q.rows + 2) * q.cw <= pl_max) break;
  if (q.rows < 1) return false;
  q.n_strips = (p.H + q.rows - 1) / q.rows;
  q.rows = (p.H + q.n_strips - 1) / q.n_strips;
  q.n_pairs = 1;
  // several (group, sample) pairs while they fit the tile, with byte offsets below 2^30 between them
  if (q.n_strips == 1 && q.n_segs == 1)
    while (q.n_pairs * 2 * q.rows * q.xw <= px_max && q.n_pairs * 2 * (q.rows + 2) * q.cw <= pl_max &&
           (long long)q.n_pairs * 2 * p.Cout * p.H * p.W < (1ll << 28))
      q.n_pairs *= 2;
  q.pair_tiles = (p.G * p.B + q.n_pairs - 1) / q.n_pairs;
  q.ci_groups = (p.Cin + 31) / 32;
  q.px = q.n_pairs * q.rows * q.xw;
  q.pl = q.n_pairs * (q.rows + 2) * q.cw;
  return true;
}
inline long long dgrad_f32_tiles(const DgradPlan& q) { return (long long)q.pair_tiles * q.n_strips * q.n_segs * q.ci_groups; }

// What follows the products: a value per group, or one for each frame of it, or four through a pool (to_max: to one of four that is looked up).  A workgroup's stores are a
// chain, frame after frame, which outweighs the products of small layers: 64 <- 16 at 6 x 6, B = 3, one group of 8 through a max pool 18.4 us where the four waves share the
// output channels (and an eighth of the values each), 48.3 on the other kernel, which its products favour.  us: of a frame's values, of those of each workgroup
// of a compute unit in units of that; fitted to 570 random layers (10% rms).
struct DgradStores {
  double frame, pooled, to_max, per_workgroup;
};
inline double dgrad_store_us(const DgradStores& s, const BackwardParams& p, double per_cu) {
  if (p.grad_in_group && !p.pool2) return 0.0;
  const int K = std::max(1, (int)p.K);
  return (p.pool2 == 2 ? s.to_max * K : p.pool2 ? s.pooled * K : s.frame * (K - 0.5)) * std::max(1.0, s.per_workgroup * per_cu);
}

// Microseconds of the kernels without the frames' stores, fitted to 450 random layers with one value per group (1 to 128 channels on either side, 3 x 3 to 64 x 72 pixels, 1 to 768 pairs) to 6 or 7% rms, and 9% for
// the vector kernel.
// Rounds of 16 output channels (cycles at 2.5 GHz): a workgroup that has its compute unit to itself (two blocks a wave 10700, one 7500), or its part of several
// (7850, 4000); the stores.  Up to eight output channels take one shorter round (fitted to 174 layers, 7% rms).
inline double dgrad_thirds_us(const DgradPlan& q, int np, const BackwardParams& p) {
  const double per_cu = (double)((dgrad_f32_tiles(q) + kFittedUnits - 1) / kFittedUnits);
  const double cycles = p.Cout <= 8 ? std::max(np == 2 ? 6000.0 : 4300.0, per_cu * (np == 2 ? 5000.0 : 2300.0))
                                    : std::max(np == 2 ? 10700.0 : 7500.0, per_cu * (np == 2 ? 7850.0 : 4000.0));
  // (a lane stores 16 channels of 32, of fewer input channels at most four of eight)
  const int n = std::min(32, (int)p.Cin), stored = n / 8 * 4 + std::min(n % 8, 4);
  const double stores = dgrad_store_us(np == 2 ? DgradStores{5.46, 6.83, 11.97, 0.66} : DgradStores{2.75, 3.64, 6.38, 0.57}, p, per_cu);
  return 2.4 + (p.Cout + kDgradCo - 1) / kDgradCo * cycles / 2500.0 + 0.9 * per_cu * np + stores * stored / 16;
}
// Rounds of 32 output channels in products of fp32
inline double dgrad_split_us(const DgradPlan& q, const BackwardParams& p) {
  const double per_cu = (double)((dgrad_f32_tiles(q) + kFittedUnits - 1) / kFittedUnits);
  return 2.6 + (p.Cout + kSplitCo - 1) / kSplitCo * 3.55 * std::max(1.0, 0.64 * per_cu) + 2.7 * per_cu + dgrad_store_us({0.58, 0.72, 1.22, 0.67}, p, per_cu);
}
// A thread's chain over the output channels, or the pixels at the rate they go through; the stores
inline double dgrad_vector_us(const BackwardParams& p) {
  const double pairs = (double)p.G * p.B, pixels = (double)p.H * p.W, blocks = (double)(((int64_t)p.H * p.W + 255) / 256 * 256);
  return 3.4 + p.Cout * (0.34 + 0.054 * std::min(p.Cin, 4) + (p.Cin + 3) / 4 * pairs * blocks * 1.465e-6) + p.Cin * pairs * pixels * 3.4e-6 +
         dgrad_store_us({0.17, 0.32, 0.95, 0.0}, p, 0.0) * std::min(p.Cin, 4) / 4 + dgrad_store_us({0.51e-6, 1.72e-6, 2.04e-6, 0.0}, p, 0.0) * p.Cin * pairs * pixels;
}

// np: blocks of 32 pixels a wave (0: no tile).  True: dgrad_f32_split_kernel, whose four waves share the output channels of one block of pixels, for few tiles: of the 450
// layers 46 (128 -> 128 at 8 x 8, B = 16, one group 17.4 us, 28.1 on the other kernel; 16 -> 48 at 31 x 32, 16 pairs on 496 tiles 17.5 / 12.0: that one's); of 420 small layers, most
// of which store frames or pooled frames, 185: the chosen kernels take 0.4% longer than the best, 9% by estimates without the stores.
inline bool dgrad_f32_choose(const BackwardParams& p, DgradPlan& q, int& np) {
  np = 0;
  double best = 0.0;
  for (int n : {2, 1}) {
    DgradPlan c{};
    if (!dgrad_f32_tile(p, 4 * n, kDgradM * kDgradThreads, c)) continue;
    const double us = dgrad_thirds_us(c, n, p);
    if (np && us >= best) continue;
    np = n;
    best = us;
    q = c;
  }
  // Up to eight output channels are one short round of the other kernel, and less accurate here (8 channels 1.42e-7 of the norm, 1.10e-7 there); from nine on, on 22 layers that
  // this rule gives back to products of fp32, the error is 0.7 to 1.0 of that of thirds in one chain
  DgradPlan c{};
  if (!np || p.Cout <= 8 || !dgrad_f32_tile(p, 1, kSplitPl, c) || dgrad_f32_tiles(c) > 512 || dgrad_split_us(c, p) >= best) return false;
  q = c;
  return true;
}

// Tiles of four input channels of the vector kernel: `across` in y, where a grid has at most 65535 workgroups, `over` times.
inline void dgrad_vector_tiles(int Cin, unsigned& across, unsigned& over) {
  const long long tiles = ((long long)Cin + 3) / 4;
  over = (unsigned)((tiles + 65534) / 65535);
  across = (unsigned)((tiles + over - 1) / over);
}

// Which kernel forms an input gradient that is not the bf16 kernels': the matrix-core ones (true) take stride 1 and fill blocks of 32 input channels; the vector kernel takes
// any layer, four input channels per thread, and is the faster one for few input channels over many pixels, by both estimates (us on the vector kernel and on the other:
// 1 -> 64 at 64 x 64, B = 64, 8 groups 261 / 480, 4 -> 64 314 / 454, 8 -> 64 549 / 439; 1 -> 64 at 28 x 28, B = 64, 2 groups 34.6 / 28.1, 1 -> 8 8.8 / 9.2).  Its
// chains of products are less accurate than thirds.  So it takes no layer for which it would not be the faster one even against 32 input channels in products of fp32 (per output
// channel 0.23 us and the pixels at 0.184e6 a us, against 0.35 .. 0.63 and 0.55e6 for four), where thirds would be slower only with one to four output channels (2 -> 1 at 35 x 31, 64
// pairs 6.1 us, 5.0 there).
inline bool backward_dgrad_f32_supported(const BackwardParams& p) {
  if (p.stride != 1) return false;
  if (p.Cin >= (1 << 20)) return false;                  // 30-bit byte offsets within the weights of 16 output channels
  const double pairs = (double)p.G * p.B, pixels = (double)p.H * p.W;
  const double by_vectors = 0.35 + 0.07 * std::min(p.Cin, 4) + (p.Cin + 3) / 4 * pairs * (double)(((int64_t)p.H * p.W + 255) / 256 * 256) / 0.55e6;
  if (0.23 + (p.Cin + 31) / 32 * pairs * pixels / 0.184e6 <= by_vectors) return true;
  DgradPlan q{};
  int np = 0;
  return dgrad_f32_choose(p, q, np) || !np || dgrad_thirds_us(q, np, p) <= dgrad_vector_us(p);
}

}  // namespace tac
