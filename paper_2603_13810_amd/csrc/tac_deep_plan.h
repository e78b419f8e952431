// Host rules of the kernel for layers with too many channels for the other matrix-core kernels (tac_mfma_deep_kernel.h).
#pragma once
#include <algorithm>
#include "tac_mfma_common.h"

namespace tac {

constexpr int kDeepThreads = 512;
constexpr int kDeepWaves = 8;                  // share the contraction
constexpr int kDeepSets = 4;                   // blocks of 32 pixels x 32 channels (of one group) in hand
constexpr int kDeepLds = 160 * 1024;
constexpr int kDeepMaxCin = 256;
constexpr int kDeepMaxK = 16;

// Geometry of one launch.  Byte offsets are from the start of the LDS.
struct DeepPlan {
  int kp;                       // frames per table index: 1, 2, 4, 8, or 16 (two tables of eight)
  int pb, gb;                   // pixel blocks per workgroup; groups in hand at a time
  int pw_shift, rpb, wb;        // lanes of a row within a block = 1 << pw_shift, rows per block, blocks per row
  int tr, lr, flatten;          // output rows per tile, LDS rows of the largest tile; rows are counted through all samples
  int row_tiles, co_tiles;
  int wpx, xh, plane, group;    // columns of an aggregate row, of its even half (stride 2); bytes per 8 channels, per group
  int nseg, xs;                 // a unit: xs pixels of a row, some channels (deep_unit_channels); segments per row
  int nks;                      // k-steps of 16
  int off_lut, lut_set, off_bias, off_tab, off_pair, total;
};

inline int deep_k_steps(int Cin) { return (9 * Cin + 15) / 16; }

// k-steps of a wave at most: 9 up to 128 input channels, else 18
__host__ __device__ constexpr int deep_wave_steps(int nks) { return nks <= 72 ? 9 : 18; }
// Channels of a unit: its words, twice (in hand and on their way), beside the weights and the sums in 256 registers
__host__ __device__ constexpr int deep_unit_channels(int kp, int wave_steps) {
  return kp <= 2 ? 8 : kp == 4 ? (wave_steps == 9 ? 8 : 4) : kp == 8 ? (wave_steps == 9 ? 4 : 2) : 2;
}

// Scalar byte offset of the words of frame j, channel c of a unit, in a load from a round's first word.  The range check of a buffer load compares the
// lane's offset with the descriptor's size less this one, which must not wrap below zero.
__host__ __device__ constexpr uint32_t deep_scalar_offset(int j, int frames, uint32_t frame_words, int c, uint32_t channel_words) {
  return ((uint32_t)(j < frames ? j : 0) * frame_words + (uint32_t)c * channel_words) * 4u;
}
// Frames of a round's first group, which no group of the round exceeds: a shorter last group alone in its round has only its own behind the descriptor's start.
__host__ __device__ constexpr int deep_round_frames(int g0, int G, int K, int K_last) { return g0 < G ? K : K_last; }

// False: the tile does not fit.
inline bool deep_plan(DeepPlan& q, const LayerParams& p, int pb, bool flatten) {
  const int S = p.stride, C8 = p.Cin / 8, n_groups = p.G + (p.K_last ? 1 : 0);
  q.kp = p.K <= 2 ? p.K : p.K <= 4 ? 4 : p.K <= 8 ? 8 : 16;
  q.pb = pb;
  q.pw_shift = p.Wo > 16 ? 5 : p.Wo > 8 ? 4 : p.Wo > 4 ? 3 : p.Wo > 2 ? 2 : 1;
  q.rpb = 32 >> q.pw_shift;
  q.wb = (p.Wo + 31) / 32;
  if (q.wb > pb) return false;
  q.flatten = flatten;
  const long long rows = flatten ? (long long)p.B * p.Ho : p.Ho;
  q.tr = (int)std::min<long long>(pb / q.wb * q.rpb, rows);
  const int samples = flatten ? std::min((q.tr + p.Ho - 2) / p.Ho + 1, p.B) : 1;        // a tile may touch
  q.lr = (q.tr - 1) * S + 3 + (samples - 1) * (3 - S);
  q.row_tiles = (int)((rows + q.tr - 1) / q.tr);
  q.co_tiles = (p.Cout + 31) / 32;
  q.wpx = p.W + 2;
  q.xh = (q.wpx + 1) / 2;
  q.plane = q.lr * q.wpx * 16;
  q.plane += (128 - q.plane % 256 + 256) % 256;         // consecutive planes start half the banks apart (the two lane halves)
  q.group = q.plane * C8;
  q.nks = deep_k_steps(p.Cin);
  q.lut_set = q.kp <= 2 ? 0 : q.kp == 16 ? 2048 : 1024;
  const int most_pairs = q.lr * ((p.W + 7) / 8);
  for (q.gb = std::min(kDeepSets / pb, n_groups); q.gb >= 1; --q.gb) {
    // the partial sums of the waves take the place of the aggregates they were made from
    q.off_lut = std::max(q.gb * q.group, kDeepWaves * 4096 * q.gb * pb);
    q.off_bias = q.off_lut + q.lut_set * (p.K_last ? 2 : 1);
    q.off_tab = q.off_bias + 128;
    q.off_pair = q.off_tab + q.nks * 8;
    q.total = q.off_pair + most_pairs * 8;
    if (q.total <= kDeepLds) break;
  }
  if (q.gb < 1) return false;
  // 32-bit byte offsets of a round's words
  if ((long long)q.gb * p.K * p.B * p.Cin * p.Hs * p.Wwi * 4 >= (1ll << 31)) return false;
  // how a row is cut: the fewest turns of the 512 threads, counted in words to load and pixels to form
  const int chans = deep_unit_channels(q.kp, deep_wave_steps(q.nks));
  double best = 0.0;
  for (int xs = 32; xs >= 8; xs /= 2) {
    if (xs / 2 >= p.W && xs > 8) continue;
    const int nseg = (p.W + xs - 1) / xs, units = p.Cin / chans * q.lr * nseg;
    const double turns = (q.gb * units + kDeepThreads - 1) / kDeepThreads;
    const double cost = turns * (100.0 + 4.0 * chans * q.kp + 25.0 * std::min(xs, p.W));
    if (best != 0.0 && cost >= best) continue;
    best = cost;
    q.nseg = nseg;
    q.xs = xs;
  }
  return true;
}

// The shapes the kernel reaches at all
inline bool deep_reaches(const LayerParams& p) {
  return p.bf16 && !p.dense && !p.pool2 && !p.out_pool && p.Cin % 8 == 0 && p.Cin >= 16 && p.Cin <= kDeepMaxCin && p.K <= kDeepMaxK && p.Wo <= 64 &&
         membranes_in_reach(p);
}

inline bool deep_choose(const LayerParams& p, DeepPlan& q) {
  if (!deep_reaches(p)) return false;
  // a tile that straddles samples offsets its membranes by 32 bits and counts rows in fp32
  const bool may_flatten = (long long)p.B * p.Cout * p.Ho * p.Wo < (1ll << 30) && (long long)p.B * p.Ho < (1ll << 20) - 1024;
  bool found = false;
  for (int fl = may_flatten ? 1 : 0; fl >= 0; --fl)
    for (int pb = 1; pb <= 2; ++pb) {
      DeepPlan c;
      if (!deep_plan(c, p, pb, fl != 0)) continue;
      const long long wgs = (long long)c.row_tiles * c.co_tiles * (c.flatten ? 1 : p.B);
      if (wgs * kDeepThreads >= (1ll << 32)) continue;                 // threads of a launch in one dimension
      // two blocks a workgroup where one block each is more than the chip takes in one go
      const long long old = found ? (long long)q.row_tiles * q.co_tiles * (q.flatten ? 1 : p.B) : 0;
      if (found && (c.flatten != q.flatten ? wgs >= old : old <= kFittedUnits)) continue;
      q = c;
      found = true;
    }
  return found;
}

}  // namespace tac
