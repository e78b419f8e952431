// Host rules of the weight gradient of first layers (tac_backward_wgrad_first.hip).
#pragma once
#include <algorithm>
#include "tac_mfma_common.h"

namespace tac {

constexpr int kFirstWgradThreads = 512;
constexpr int kFirstWgradChannels = 4;          // output channels of a wave: up to 72 sums in registers, beside 16 values of dY
constexpr int kFirstWgradSums = 8 * (72 + kFirstWgradChannels) * 8;     // LDS bytes of the waves' sums of dW and of the bias gradient
constexpr int kFirstWgradLds = 72 * 1024 + kFirstWgradSums;             // two workgroups per compute unit
// Products that a lane adds in a chain, as many as a chain of the other kernel's has MFMAs.  (More only where a strip of one row has more.)
constexpr int kFirstWgradChain = 64;

struct FirstWgradPlan {
  int ncg, co_groups, split;
  int n_pairs, rows, n_strips, pair_tiles;    // an item: (group, sample) pairs x output rows
  int quads, rows_in, cw;                     // quads per output row; aggregate rows per pair and channel, floats per row
  int flush;                                  // items after which a lane's chains of products end
  int off_w, off_sum, total;                  // LDS bytes
};

// False: a layer of the other kernel's (wgrad_f32_kernel).
inline bool first_wgrad_plan(const BackwardParams& p, FirstWgradPlan& q) {
  if (p.Cin > 2 || p.pool2) return false;
  const int S = p.stride, groups = (p.Cout + kFirstWgradChannels - 1) / kFirstWgradChannels;
  q.quads = (p.Wo + 3) / 4;
  q.cw = (q.quads * 4 * S + 3 + 7) & ~7;
  q.ncg = 1;
  // Workgroups of few channels need few slices to fill the chip (1 -> 32 at 28 x 28, B = 128: as fast with 64 slices as with 128, whose sums round twice as often), but
  // rebuild the aggregates once more each, which weighs with real-valued frames (2 -> 128 at 64 x 64, B = 16: 122 us a call, 132 the other way).
  const int most_groups = p.dense ? 4 : 8, most_slices = p.dense ? 128 : 64;
  while (q.ncg < 8 && groups / q.ncg > most_groups) q.ncg *= 2;
  q.co_groups = (groups + q.ncg - 1) / q.ncg;
  // frames whose values outweigh dY stay with the other kernel: 2 -> 48 stride 2 at 64 x 67, B = 33, groups of 8 (4 times) 45 / 53 us a call, 2 -> 32 stride 2 at
  // 32 x 32, B = 128, groups of 3 (3 times) 75 / 82; 1 -> 32 at 128 x 126, B = 64, groups of 16 (2 times) 174 / 168
  if (p.dense && p.K * S * S * p.Cin * q.co_groups > 2 * p.Cout) return false;
  const int lanes = kFirstWgradThreads / q.ncg, all_pairs = p.G * p.B;
  // rows of an item: two turns of the lanes, as far as the image and the LDS go; then pairs, while every slice gets an item
  const int slices = std::max(1, std::min(most_slices, 512 / q.co_groups));
  const int limit = kFirstWgradLds - kFirstWgradSums - 2 * TAC_MAX_K * 4;
  auto bytes = [&](int rows, int pairs) { return (long long)pairs * p.Cin * ((rows - 1) * S + 3) * q.cw * 4; };
  q.rows = std::min(p.Ho, std::max(1, 2 * lanes / q.quads));
  while (q.rows > 1 && bytes(q.rows, 1) > limit) q.rows = (q.rows + 1) / 2;
  if (bytes(q.rows, 1) > limit) return false;
  q.n_strips = (p.Ho + q.rows - 1) / q.rows;
  q.rows = (p.Ho + q.n_strips - 1) / q.n_strips;         // strips of the same height, as far as it goes
  q.n_pairs = 1;
  if (q.n_strips == 1)
    while (q.n_pairs * q.rows * q.quads < 2 * lanes && bytes(q.rows, q.n_pairs + 1) <= limit && (long long)slices * (q.n_pairs + 1) <= all_pairs) ++q.n_pairs;
  q.pair_tiles = (all_pairs + q.n_pairs - 1) / q.n_pairs;
  q.split = (int)std::min<long long>(slices, (long long)q.pair_tiles * q.n_strips);
  // few workgroups of real-valued frames have a long chain of loads each (2 -> 56 at 31 x 26, B = 2, three groups of 8 on 24 workgroups: 15.4 us, 9.4 on the other
  // kernel; of 25 layers below this line 3 lost more than 5% by it)
  if (p.dense && q.co_groups * q.split < 128) return false;
  // Few workgroups of one item each wait for its aggregates, a trip to memory for every four frames and turn of the threads: 2 -> 117 stride 2 at 55 x 68, B = 3,
  // groups of 16 on 48 workgroups of 12 trips 19.3 us, 15.5 on the other kernel; of 207 layers 16 are below this line, nine of them slower on this kernel (0.80 to 0.99 of the
  // speed) and seven faster (1.03 to 1.28).
  const int lines = q.n_pairs * p.Cin * ((q.rows - 1) * S + 3), trips = (lines * (q.cw / 8) + kFirstWgradThreads - 1) / kFirstWgradThreads * ((p.K + 3) / 4);
  if (!p.dense && p.Cin == 2 && q.co_groups * q.split < 64 && (long long)q.pair_tiles * q.n_strips <= q.split && trips >= 3) return false;
  // four products a quad and turn of the lanes
  q.flush = std::max(1, kFirstWgradChain / (4 * ((q.n_pairs * q.rows * q.quads + lanes - 1) / lanes)));
  q.rows_in = (q.rows - 1) * S + 3;
  q.off_w = (int)bytes(q.rows, q.n_pairs);
  q.off_sum = q.off_w + 2 * TAC_MAX_K * 4;
  q.total = q.off_sum + kFirstWgradSums;
  return (long long)q.pair_tiles * q.n_strips < (1ll << 31) && q.n_pairs * q.rows * q.quads < (1 << 20);
}

}  // namespace tac
