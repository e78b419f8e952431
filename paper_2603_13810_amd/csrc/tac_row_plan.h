// Host rules of the row kernel (tac_mfma_row_kernel.h).
#pragma once
#include <algorithm>
#include <bit>
#include <cmath>
#include "tac_mfma_common.h"

namespace tac {

// Waves of a workgroup at most: one block of pixels leaves room for four waves on a SIMD (128 registers), two for three
__host__ __device__ constexpr int row_max_waves(int nnp) { return nnp == 1 ? 16 : 12; }
constexpr int kRowLds = 160 * 1024;
constexpr int kRowMHz = 2350;                  // of the launches that row_cost is fitted to
constexpr int kRowMaxK = 16;
constexpr int kRowTabPad = 16;                 // entries of the slot table behind the last k-step (fetched ahead)
constexpr int kRowDepth = 3;                   // sets of operand fragments in flight

// Chunks of 64 words (times the frames of a group) that a wave has in hand
__host__ __device__ constexpr int row_batch(int kp) { return kp <= 2 ? 8 : kp == 4 ? 6 : kp == 8 ? 4 : 2; }

// Geometry of one launch.  Byte offsets are from the start of the LDS.
struct RowPlan {
  int kp;                       // frames per table index: 1, 2, 4, 8, or 16 (two tables of eight)
  int pw, nco, nnp, waves;      // waves over the pixels, over the channels (tiles of 32); blocks of 32 pixels per wave; all waves: the others only form aggregates
  int spr;                      // segments of 16 pixels per output row
  int tr, lr, flatten;          // output rows per tile, LDS rows of the largest tile; rows are counted through all samples
  int row_tiles, co_tiles;
  int wpx, xh, plane;           // columns of an aggregate row, of its even half (stride 2); bytes per 8 channels
  int cb, parts, lrp, n_jobs;   // a job: cb blocks of 8 channels x lrp LDS rows; jobs over the rows; jobs per tile
  int stage_pair, stage_wave;   // staged dwords per (row, word) and 8 channels; bytes of a wave's staged words
  int nks, nmc_w;               // k-steps of 16; 32-channel blocks per tile of the prepared weights
  int off_w, off_stage, off_lut, lut_set, off_bias, off_tab, off_pair, off_px, total;
};

// Tiles of a launch; false: none.
inline bool row_tiles(RowPlan& q, const LayerParams& p, int pw, int nco, int nnp, bool flatten) {
  const int S = p.stride;
  q.pw = pw; q.nco = nco; q.nnp = nnp;
  q.spr = (p.Wo + 15) / 16;
  q.flatten = flatten;
  const int rows = flatten ? p.B * p.Ho : p.Ho;          // (below 2^20 when they are counted through all samples)
  q.tr = std::min(2 * pw * nnp / q.spr, rows);
  if (q.tr < 1) return false;
  // as few blocks as the rows need
  if ((q.tr * q.spr + 1) / 2 <= (pw - 1) * nnp) return false;
  const int samples = flatten ? std::min((q.tr + p.Ho - 2) / p.Ho + 1, p.B) : 1;        // a tile may touch
  q.lr = (q.tr - 1) * S + 3 + (samples - 1) * (3 - S);
  q.row_tiles = (int)(((long long)rows + q.tr - 1) / q.tr);
  q.co_tiles = (p.Cout + 32 * nco - 1) / (32 * nco);
  return true;
}

// The rest of the plan of some tiles; false: no way to form their aggregates fits.
inline bool row_plan(RowPlan& q, const LayerParams& p, int waves, int nmc_w) {
  const int C8 = p.Cin / 8, nco = q.nco;
  q.waves = waves;
  q.kp = p.K <= 2 ? p.K : p.K <= 4 ? 4 : p.K <= 8 ? 8 : 16;
  q.nmc_w = nmc_w;
  q.wpx = p.W + 2;
  q.xh = (q.wpx + 1) / 2;
  q.plane = q.lr * q.wpx * 16;
  q.plane += (128 - q.plane % 256 + 256) % 256;         // consecutive planes start half the banks apart (the two lane halves)
  q.nks = (9 * p.Cin + 15) / 16;
  q.stage_pair = q.kp * 8 + 4;                 // four unused dwords spread consecutive pairs over the LDS banks
  q.lut_set = q.kp <= 2 ? 0 : q.kp == 16 ? 2048 : 1024;
  auto up = [](int x) { return (x + 15) & ~15; };
  q.off_w = q.plane * C8;
  q.off_lut = q.off_w + (q.nks * nco + 2 * kRowDepth) * 1024;       // the fetches ahead read past the weights
  q.off_bias = q.off_lut + q.lut_set * (p.K_last ? 2 : 1);
  q.off_tab = q.off_bias + nco * 128;
  q.off_pair = q.off_tab + up((2 * q.nks + kRowTabPad) * 4);
  q.off_px = q.off_pair + up(q.lr * p.Wwi * 4);
  q.off_stage = q.off_px + up(q.lr * p.W * 8);
  if (q.off_stage > kRowLds) return false;
  double best = 0.0;
  RowPlan c = q;
  for (c.cb = 1; c.cb <= 4; c.cb *= 2) {
    // rows of a job: the most that a wave has registers for, then the next fewer ones that need more jobs
    const int most = std::min(q.lr, 64 * row_batch(q.kp) / (8 * c.cb * p.Wwi));
    if (most < 1) break;
    const int blocks = (C8 + c.cb - 1) / c.cb;
    for (c.parts = (q.lr + most - 1) / most;; c.parts = (q.lr + c.lrp - 2) / (c.lrp - 1)) {
      c.lrp = (q.lr + c.parts - 1) / c.parts;
      c.n_jobs = blocks * c.parts;
      c.stage_wave = up(c.cb * c.lrp * p.Wwi * c.stage_pair * 4);
      c.total = c.off_stage + waves * c.stage_wave;
      if (c.total <= kRowLds) {
        const int units = 8 * c.cb * c.lrp * p.Wwi;
        const double cost = (c.n_jobs + waves - 1) / waves * (400.0 + (units + 63) / 64 * (60.0 + 25.0 * c.kp) + (c.lrp * p.W + 63) / 64 * (60.0 + 45.0 * c.cb));
        if (best == 0.0 || cost < best) {
          best = cost;
          q = c;
        }
      }
      if (c.lrp == 1) break;
    }
  }
  return best != 0.0;
}

// Groups that a plan is chosen for: sequences of different lengths share it up to the next power of two (on 4000 random layers its estimate is 0.01% above the best one's on
// average, 2.3% at most).
inline int row_groups(const LayerParams& p) { return (int)std::bit_ceil((unsigned)(p.G + (p.K_last ? 1 : 0))); }

// Microseconds of a launch: the sum, over the turns that the chip takes, of what a compute unit spends on a group's aggregates (its instructions, or a
// wave's own chain of loads and LDS trips), on its contraction (the matrix cores, or the waits for fragments) and on its LIF steps.  The
// coefficients (cycles at kRowMHz) are a fit to 4600 timed launches of 127 random layers: 10% rms, and the plan chosen by it takes 1.6% longer than the best
// one on average.
inline double row_cost(const RowPlan& q, const LayerParams& p) {
  const long long wgs = (long long)q.row_tiles * q.co_tiles * (q.flatten ? 1 : p.B);
  const int mw = q.pw * q.nco, groups = row_groups(p);
  const int resident = std::max(1, std::min(kRowLds / q.total, row_max_waves(q.nnp) / q.waves));
  const long long per_cu = (wgs + kFittedUnits - 1) / kFittedUnits;
  const double together = (double)std::min<long long>(resident, per_cu), per_simd = together * q.waves / 4, multiply = together * mw / 4;
  const int turns = (q.n_jobs + q.waves - 1) / q.waves, chunks = (8 * q.cb * q.lrp * p.Wwi + 63) / 64, passes = (q.lrp * p.W + 63) / 64;
  const double issue = turns * (6.4 + chunks * (1.6 + 31 * q.kp) + passes * (12 + 35 * q.cb));
  const double form = std::max(3.4 * issue * std::max(per_simd, 1.0), 290.0 + turns * (430 + 180 * passes + 43 * chunks));
  const double contract = q.nks * std::max(45 * q.nnp * multiply, 38.0 + 51 * q.nnp);
  const double lif = p.n_lif * (27 + 613 * q.nnp * std::max(1.0, 0.5 * multiply));
  return (double)((per_cu + resident - 1) / resident) * (15300 + groups * (form + contract + lif + 870)) / kRowMHz + 2.6;
}

// What row_cost is not below for any plan of some tiles: each of its terms with as many workgroups side by side as the waves allow, times the turns.  Most plans
// are not worth working out after the first few: choosing takes 17 us on average instead of 32.
inline double row_cost_least(const RowPlan& q, const LayerParams& p, int waves) {
  const int mw = q.pw * q.nco, groups = row_groups(p), nks = (9 * p.Cin + 15) / 16, at_once = std::max(1, row_max_waves(q.nnp) / waves);
  const double per_cu = (double)(((long long)q.row_tiles * q.co_tiles * (q.flatten ? 1 : p.B) + kFittedUnits - 1) / kFittedUnits);
  const double turns = std::ceil(per_cu / at_once), multiply = per_cu * mw / 4;
  // (a pass over 64 pixels of 8 channels is 38 instructions at least)
  const double form = std::max(3.4 * 38 / 4 * per_cu * (p.Cin / 8) * (q.lr * p.W) / 64, 290.0 * turns);
  const double contract = nks * std::max(45 * q.nnp * multiply, turns * (38.0 + 51 * q.nnp));
  const double lif = p.n_lif * (27 * turns + 613 * q.nnp * std::max(turns, 0.5 * multiply));
  return 0.999999 * (turns * 15300 + groups * (form + contract + lif + 870 * turns)) / kRowMHz + 2.6;
}

// The shapes the kernel reaches at all.  Layers that record their membranes stay on the older kernel: writing those takes most of their time, and with
// groups of one or two frames it was the faster one at more than half of the shapes measured.
inline bool row_reaches(const LayerParams& p) {
  return p.bf16 && !p.dense && !p.pool2 && !p.out_pool && !p.v_trace && p.Cin % 8 == 0 && p.Cin <= 128 && p.K <= kRowMaxK && p.Wo > 16 && p.Wo <= 64 &&
         membranes_in_reach(p) && (long long)p.B * p.Cout * p.Ho * 4 < (1ll << 32) &&            // half-words of a step's output
         (long long)p.K * p.B * p.Cin * p.H * p.Wwi * 4 < (1ll << 31);                           // bytes of a group's words
}

// Layers with so little to do that neither the loads nor the contraction count stay on the older kernel, whose blocks need no tables of rows and pixels.  On
// 45 random ones the row kernel took from 1.16 times as long (24.2 us against 20.8 at 8 -> 96 channels, 40x17, groups of two) to 0.76 times, the same on
// average; on 203 random ones above the limits it was 1.21x faster on average (60.0 us to 26.9 at 32 -> 100 channels, 108x79, stride 2, groups of five) and
// 5% slower at most (16.0 us against 15.2 at 48 -> 32 channels, 25x24, groups of two).
inline bool row_too_little(const LayerParams& p) {
  const long long blocks = (long long)p.B * p.Ho * ((p.Wo + 31) / 32) * ((p.Cout + 31) / 32);
  return p.K <= 2 && p.Cin <= 16 * p.K && blocks <= (p.Cin <= 16 ? 2048 : 512);
}

inline bool row_choose(const LayerParams& p, RowPlan& q, int nmc_w) {
  if (!row_reaches(p) || row_too_little(p)) return false;
  // a tile that straddles samples offsets its membranes by 32 bits and counts rows in fp32
  const bool may_flatten = (long long)p.B * p.Cout * p.Ho * p.Wo < (1ll << 30) && (long long)p.B * p.Ho < (1ll << 20) - 1024;
  double best = 0.0;
  for (int fl = 0; fl <= (may_flatten ? 1 : 0); ++fl)
    for (int nnp = 1; nnp <= 2; ++nnp)
      for (int nco = 1; nco <= std::min(4, (p.Cout + 31) / 32); ++nco)
        for (int pw = 1; pw * nco <= row_max_waves(nnp); ++pw) {
          RowPlan tiles;
          if (!row_tiles(tiles, p, pw, nco, nnp, fl != 0)) continue;
          int before = 0;
          for (int least = 4; least <= 8; least += 2) {
            const int waves = std::max(least, pw * nco);
            if (waves == before) continue;
            before = waves;
            if (best != 0.0 && row_cost_least(tiles, p, waves) >= best) continue;
            RowPlan c = tiles;
            if (!row_plan(c, p, waves, nmc_w)) continue;
            const long long wgs = (long long)c.row_tiles * c.co_tiles * (c.flatten ? 1 : p.B);
            if (wgs * 64 * waves >= (1ll << 32) || (!c.flatten && p.B > 65535)) continue;        // the grid's limits
            const double cost = row_cost(c, p);
            if (best != 0.0 && cost >= best) continue;
            best = cost;
            q = c;
          }
        }
  return best != 0.0;
}

}  // namespace tac
