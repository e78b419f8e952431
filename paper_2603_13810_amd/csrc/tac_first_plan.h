// Host rules of the first layers' kernel (tac_mfma_small.hip).
#pragma once
#include "tac_internal.h"

namespace tac {

constexpr int kFirstWaves = 8;                 // per workgroup at most
constexpr int kFirstMaxW = 128;                // input width limit (4 words per row)
constexpr int kFirstTileRows = 16;             // output rows per workgroup at most

// fp32 layers of the same shapes, on the vector kernel's prepared weights ([cin][tap][cout padded to 32] fp32)
// Times against the vector kernel's (us): 1 -> 32 at 28 x 28, B = 128, 18 / 50 (see there), 2 -> 8 at 60 x 40, B = 128, one group 15.6 / 17.7, B = 8,
// four groups 10.7 / 17.1.  With recorded membranes few channels are slower, 2 -> 8 at 60 x 40, B = 128, one group 31.8 / 18.8, 2 -> 16 32.3 / 28.7,
// 2 -> 32 33.0 / 57.8; they are taken all the same, since a layer gives the same bits with and without recording.
inline bool first_f32_supported(const LayerParams& p) {
  if (p.bf16 || p.pool2 || p.out_pool || p.Cin > 2 || p.W > kFirstMaxW) return false;
  // The upper lane half's membranes are four planes behind the lower one's, in 32-bit byte offsets from the tile's first row: planes of 2^28
  // neurons with channels there (more than 2 million rows) belong to the vector kernel, which counts in 64 bits.
  const long long plane = (long long)p.Ho * p.Wo;
  return p.Cout <= 4 || (4 * plane + kFirstTileRows * p.Wo) * 4 < (1ll << 32);
}

}  // namespace tac
