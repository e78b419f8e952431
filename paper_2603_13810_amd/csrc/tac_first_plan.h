// Host rules of the first layers' kernel (tac_mfma_small.hip).
#pragma once
#include "tac_mfma_common.h"

namespace tac {

constexpr int kFirstWaves = 8;                 // per workgroup at most
constexpr int kFirstMaxW = 128;                // input width limit (4 words per row)

// row of the aggregate tile: a padding column on either side, room for the last word's four pixels
__host__ __device__ constexpr int first_row_words(int W) { return ((W + 3) & ~3) + 2; }

// The tiles of a launch: `pairs` pairs of pixel blocks x `blocks` blocks of 32 channels, a wave each.
struct FirstPlan {
  int n_pairs, pair_tiles, co_tiles;           // block pairs per sample; tiles over them, over the channels
  int pairs, blocks, tile_words;               // per workgroup; 32-bit words of one aggregate tile
  long long workgroups;
  size_t lds;
};

inline FirstPlan first_plan(const LayerParams& l) {
  FirstPlan p;
  const int Wwo = l.Wwo;
  p.n_pairs = l.out_pool ? (l.Ho / 2) * Wwo : (int)(((long long)l.Ho * Wwo + 1) / 2);
  const int co_blocks = (l.Cout + 31) / 32;
  p.co_tiles = (co_blocks + 3) / 4;
  p.blocks = (co_blocks + p.co_tiles - 1) / p.co_tiles;
  p.pair_tiles = (p.n_pairs + kFirstWaves / p.blocks - 1) / (kFirstWaves / p.blocks);
  p.pairs = (p.n_pairs + p.pair_tiles - 1) / p.pair_tiles;
  // small grids: smaller workgroups, until there are two per compute unit
  while (p.pairs > 1 && (long long)p.pair_tiles * p.co_tiles * l.B < 512) {
    p.pairs = (p.pairs + 1) / 2;
    p.pair_tiles = (p.n_pairs + p.pairs - 1) / p.pairs;
  }
  p.workgroups = (long long)p.pair_tiles * p.co_tiles * l.B;
  // most output rows that a tile touches
  const int rows = l.out_pool ? 2 * ((p.pairs + Wwo - 2) / Wwo + 1) : (2 * p.pairs + Wwo - 2) / Wwo + 1;
  p.tile_words = (l.bf16 ? 1 : l.Cin) * ((rows - 1) * l.stride + 3) * first_row_words(l.W);
  p.lds = (size_t)2 * p.tile_words * 4 + (size_t)p.pairs * p.blocks * 4 * (l.v_trace ? 32 : l.v_inout ? kTurnFloats : 0);
  return p;
}

// fp32 layers of the same shapes, on the vector kernel's prepared weights ([cin][tap][cout padded to 32] fp32)
// Times against the vector kernel's (us): 1 -> 32 at 28 x 28, B = 128, 18 / 50 (see there), 2 -> 8 at 60 x 40, B = 128, one group 15.6 / 17.7, B = 8,
// four groups 10.7 / 17.1; with recorded membranes at 60 x 40, B = 128, one group, 2 -> 8 17.2 / 19.4, 2 -> 16 20.4 / 28.6, 2 -> 32 33.1 / 57.8 (a
// layer gives the same bits with and without recording: both take the same kernel).
inline bool first_f32_supported(const LayerParams& p) {
  if (p.vector_only || p.bf16 || p.pool2 || p.out_pool || p.Cin > 2 || p.W > kFirstMaxW) return false;
  if (!membranes_in_reach(p)) return false;    // (the vector kernel counts in 64 bits)
  // A launch has fewer than 2^32 threads in one dimension, and all workgroups are in one; the vector kernel's are in three (65535 times its 32
  // channels at most).
  const FirstPlan plan = first_plan(p);
  return plan.workgroups * plan.pairs * plan.blocks * 64 < (1ll << 32) && (p.Cout + 31) / 32 <= 65535;
}

}  // namespace tac
