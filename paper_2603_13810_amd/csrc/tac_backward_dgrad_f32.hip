// Input gradient of the conv-LIF layer in fp32 on the matrix cores (v_mfma_f32_32x32x2_f32: operands, products and sums in
// fp32) for the stride-1 layers that the bf16 kernels do not take:
//   dA_k[ci][iy][ix] = sum over co, ky, kx of W[co][ci][ky][kx] * dY_k[co][iy + 1 - ky][ix + 1 - kx],
// written per group, per frame of the group (times beta^(Kg-1-j)), or through the pool on load.
//
// D[32 ci x 32 px] += W^T[32 ci x 2 co] . dY[2 co x 32 px], one pair of output channels and one tap per MFMA.  Workgroup =
// WI blocks of 32 input channels x a tile of pixels (rows of one or, in small images, of several (group, sample) pairs);
// four waves = WI channel blocks x WX = 4 / WI parts of the pixels, NP blocks of 32 pixels each.  Eight output channels at a
// time go through LDS: their weights as they lie in memory, [co][ci][9] (lanes nine floats apart: no bank conflict), and
// their dY rows with the zero border; the next eight are requested before the MFMAs (NP x 36 of 64 cycles each).
// Bound by the matrix cores on many channels, by the writes of the frames' gradients where those are per frame.
// Against one pixel x 4 channels per thread (us): 128 -> 128, B = 16, 4 groups, gradient per group, at 16 x 16 / 8 x 8 /
// 4 x 4 202 / 159 / 161 -> 68 / 45 / 46; 32 -> 64 at 14 x 14, B = 128, 7 groups, unpooled frames of the mean pool 98 -> 63.
//
// Few pixels (small images, small batches) leave that kernel with a few dozen workgroups that go through Cout / 8 rounds of two barriers
// each.  dgrad_f32_split_kernel shares a workgroup's 32 input channels x NP blocks of 32 pixels among four waves by output channel:
// 32 of them a round, a quarter of the rounds, four times the workgroups, and the waves' sums meet in LDS at the end.
#include <algorithm>
#include "tac_mfma_common.h"

namespace tac {

namespace {

constexpr int kThreads = 256;
constexpr int kCo = 8;            // output channels per round
constexpr int kM = 2;             // dY values per thread and channel
typedef __attribute__((ext_vector_type(4))) float f32x4;

struct DgradPlan {
  int rows, xw, n_pairs;          // a tile: rows x columns of n_pairs (group, sample) pairs
  int n_strips, n_segs, pair_tiles, ci_groups;
  int px, pl, cw;                 // pixels of a tile, dwords per channel of dY in LDS (with border), per row
  int vec_w;                      // the weights can be read 16 bytes at a time
  int off_dy, total;
};

__device__ __forceinline__ int group_frames(const BackwardParams& p, int k) {
  return (k == p.G - 1 && p.K_last) ? p.K_last : p.K;
}

template <int WI, int NP>
__global__ __launch_bounds__(kThreads, WI > 1 && NP == 4 ? 1 : 2) void dgrad_f32_kernel(const BackwardParams p, const DgradPlan q) {
  constexpr int kRow = 288 * WI;                         // floats of weights per output channel
  constexpr int NW = (kCo * kRow / 4 + kThreads - 1) / kThreads;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  float* const wl = reinterpret_cast<float*>(lds);
  float* const dyl = reinterpret_cast<float*>(lds + q.off_dy);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int wi = wave % WI, wx = wave / WI;
  uint32_t t = blockIdx.x;
  const int ci0 = (int)(t % (uint32_t)q.ci_groups) * (32 * WI); t /= (uint32_t)q.ci_groups;
  const int x0 = (int)(t % (uint32_t)q.n_segs) * q.xw; t /= (uint32_t)q.n_segs;
  const int y0 = (int)(t % (uint32_t)q.n_strips) * q.rows; t /= (uint32_t)q.n_strips;
  const int pair0 = (int)t * q.n_pairs, pairs = min(q.n_pairs, p.G * p.B - pair0);
  const size_t plane = (size_t)p.H * p.W;                // = Ho Wo (stride 1)

  // the lane's pixels: LDS offset of (pair, row, column) under tap (2, 2), the upper left of its window in dY
  int base[NP], px_pair[NP], px_y[NP], px_x[NP];
  bool ok[NP];
  const int per_pair = q.rows * q.xw;
#pragma unroll
  for (int b = 0; b < NP; ++b) {
    const int px = (wx * NP + b) * 32 + n;
    px_pair[b] = px / per_pair;
    const int rest = px - px_pair[b] * per_pair;
    px_y[b] = rest / q.xw;
    px_x[b] = rest - px_y[b] * q.xw;
    ok[b] = px_pair[b] < pairs && y0 + px_y[b] < p.H && x0 + px_x[b] < p.W;
    base[b] = ok[b] ? (px_pair[b] * (q.rows + 2) + px_y[b]) * q.cw + px_x[b] : 0;
  }
  // what the thread stages of every output channel's dY
  uint32_t off[kM];
  bool inside[kM];
#pragma unroll
  for (int m = 0; m < kM; ++m) {
    const int e = tid + m * kThreads;
    const int line = e / q.cw, c = e - line * q.cw, pr = line / (q.rows + 2), r = line - pr * (q.rows + 2);
    const int y = y0 + r - 1, x = x0 + c - 1;
    inside[m] = e < q.pl && pr < pairs && y >= 0 && y < p.H && x >= 0 && x < p.W;
    off[m] = inside[m] ? (uint32_t)((size_t)pr * p.Cout * plane + (size_t)y * p.W + x) : 0u;
  }
  const float* const dy0 = p.grad_y + (size_t)pair0 * p.Cout * plane;
  const int w_valid = min(32 * WI, p.Cin - ci0) * 9;     // floats of weights that exist per output channel
  f32x4 wr[NW];
  float dr[kCo][kM];
  auto request = [&](int co) {
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const int e = tid + i * kThreads, c = e / (kRow / 4), f = 4 * (e - c * (kRow / 4));
      const float* const src = p.w + ((size_t)min(co + c, p.Cout - 1) * p.Cin + ci0) * 9;
      if (q.vec_w) {
        wr[i] = *reinterpret_cast<const f32x4*>(src + min(f, w_valid - 4));
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) wr[i][u] = src[min(f + u, w_valid - 1)];
      }
    }
#pragma unroll
    for (int c = 0; c < kCo; ++c) {
      const float* const src = dy0 + (size_t)min(co + c, p.Cout - 1) * plane;
#pragma unroll
      for (int m = 0; m < kM; ++m) dr[c][m] = src[off[m]];
    }
  };
  f32x16 acc[NP];
#pragma unroll
  for (int b = 0; b < NP; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[b][r] = 0.f;
  const bool active = wx * NP * 32 < pairs * per_pair;   // wave-uniform

  request(0);
  for (int co = 0; co < p.Cout; co += kCo) {
    __syncthreads();                                     // the round before has been read
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const int e = tid + i * kThreads;
      // channels beyond Cout are zeros against zeros (the last channel's weights, read in their place, may be infinite); input
      // channels beyond Cin are not stored
      if (e < kCo * kRow / 4) *reinterpret_cast<f32x4*>(wl + 4 * e) = co + e / (kRow / 4) < p.Cout ? wr[i] : f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int m = 0; m < kM; ++m)
      if (tid + m * kThreads < q.pl) {
#pragma unroll
        for (int c = 0; c < kCo; ++c) dyl[c * q.pl + tid + m * kThreads] = inside[m] && co + c < p.Cout ? dr[c][m] : 0.f;
      }
    if (co + kCo < p.Cout) request(co + kCo);
    __syncthreads();
    if (!active) continue;
    const float* const w_lane = wl + h * kRow + (wi * 32 + n) * 9;
    const float* const d_half = dyl + h * q.pl;
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int shift = (2 - tap / 3) * q.cw + 2 - tap % 3;
#pragma unroll
      for (int i = 0; i < kCo / 2; ++i) {
        const float wv = w_lane[2 * i * kRow + tap];
#pragma unroll
        for (int b = 0; b < NP; ++b)
          acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv, d_half[2 * i * q.pl + base[b] + shift], acc[b], 0, 0, 0);
      }
    }
  }
  if (!active) return;
  // ---- register r of acc[b] on lane (n, h): input channel 8 (r / 4) + 4 h + r % 4 of the wave, pixel n of block b
  const int ci_w = ci0 + wi * 32 + 4 * h;
#pragma unroll
  for (int b = 0; b < NP; ++b) {
    if (!ok[b]) continue;
    const int pair = pair0 + px_pair[b], k = pair / p.B, sample = pair - k * p.B;
    const int iy = y0 + px_y[b], ix = x0 + px_x[b];
    const int Kg = group_frames(p, k);
    const float* const wj = Kg == p.K ? p.wj : p.wj_last;
    if (p.grad_in_group && !p.pool2) {
      float* const dst = p.grad_in + ((size_t)pair * p.Cin + ci_w) * plane + (size_t)iy * p.W + ix;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int c = 8 * (r >> 2) + (r & 3);
        if (ci_w + c < p.Cin) dst[(size_t)c * plane] = acc[b][r];
      }
      continue;
    }
    for (int j = 0; j < Kg; ++j) {
      const size_t chan0 = ((size_t)(k * p.K + j) * p.B + sample) * p.Cin + ci_w;
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int c = 8 * (r >> 2) + (r & 3);
        if (ci_w + c >= p.Cin) continue;
        const float g = wj[j] * acc[b][r];
        if (!p.pool2) {
          p.grad_in[(chan0 + c) * plane + (size_t)iy * p.W + ix] = g;
          continue;
        }
        // gradient of the unpooled frames [2H][2W]: a quarter to each input of the mean pool; all of it to the first
        // maximal input of the max pool's window in row-major order (the first set bit, or the first input when none is)
        float v[4] = {0.25f * g, 0.25f * g, 0.25f * g, 0.25f * g};
        if (p.pool2 == 2) {
          const uint32_t* const src = p.spikes + (chan0 + c) * 2 * p.H * p.Wwi + (size_t)(2 * iy) * p.Wwi + (ix >> 4);
          const uint32_t two = ((src[0] >> (2 * ix & 31)) & 3u) | (((src[p.Wwi] >> (2 * ix & 31)) & 3u) << 2);
          const int best = two ? __ffs(two) - 1 : 0;
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = e == best ? g : 0.f;
        }
        float* const dst = p.grad_in + (chan0 + c) * 4 * plane + (size_t)(2 * iy) * (2 * p.W) + 2 * ix;
        dst[0] = v[0]; dst[1] = v[1];
        dst[2 * p.W] = v[2]; dst[2 * p.W + 1] = v[3];
      }
    }
  }
}

constexpr int kSplitCo = 32;      // output channels per round, eight for each of the four waves
constexpr int kSplitPl = 112;     // dwords of dY per channel at most
template <int NP>
__global__ __launch_bounds__(kThreads, 2) void dgrad_f32_split_kernel(const BackwardParams p, const DgradPlan q) {
  constexpr int kRow = 288, NW = kSplitCo * kRow / 4 / kThreads, ND = kSplitCo * kSplitPl / kThreads;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  float* const wl = reinterpret_cast<float*>(lds);
  float* const dyl = reinterpret_cast<float*>(lds + q.off_dy);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  uint32_t t = blockIdx.x;
  const int ci0 = (int)(t % (uint32_t)q.ci_groups) * 32; t /= (uint32_t)q.ci_groups;
  const int x0 = (int)(t % (uint32_t)q.n_segs) * q.xw; t /= (uint32_t)q.n_segs;
  const int y0 = (int)(t % (uint32_t)q.n_strips) * q.rows; t /= (uint32_t)q.n_strips;
  const int pair0 = (int)t * q.n_pairs, pairs = min(q.n_pairs, p.G * p.B - pair0);
  const size_t plane = (size_t)p.H * p.W;

  int base[NP], px_pair[NP], px_y[NP], px_x[NP];
  bool ok[NP];
  const int per_pair = q.rows * q.xw;
#pragma unroll
  for (int b = 0; b < NP; ++b) {
    const int px = b * 32 + n;
    px_pair[b] = px / per_pair;
    const int rest = px - px_pair[b] * per_pair;
    px_y[b] = rest / q.xw;
    px_x[b] = rest - px_y[b] * q.xw;
    ok[b] = px_pair[b] < pairs && y0 + px_y[b] < p.H && x0 + px_x[b] < p.W;
    base[b] = ok[b] ? (px_pair[b] * (q.rows + 2) + px_y[b]) * q.cw + px_x[b] : 0;
  }
  // element e of a round's dY: channel e / pl, position e % pl (an offset of 2^32 - 1: outside the image, a zero)
  uint32_t off[ND];
  const int n_dy = kSplitCo * q.pl;
#pragma unroll
  for (int i = 0; i < ND; ++i) {
    const int e = tid + i * kThreads, c = e / q.pl, at = e - c * q.pl;
    const int line = at / q.cw, col = at - line * q.cw, pr = line / (q.rows + 2), r = line - pr * (q.rows + 2);
    const int y = y0 + r - 1, x = x0 + col - 1;
    const bool inside = e < n_dy && pr < pairs && y >= 0 && y < p.H && x >= 0 && x < p.W;
    off[i] = inside ? (uint32_t)(((size_t)pr * p.Cout + c) * plane + (size_t)y * p.W + x) : 0xffffffffu;
  }
  const float* const dy0 = p.grad_y + (size_t)pair0 * p.Cout * plane;
  const int w_valid = min(32, p.Cin - ci0) * 9;
  f32x4 wr[NW];
  float dr[ND];
  auto request = [&](int co) {
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const int e = tid + i * kThreads, c = e / (kRow / 4), f = 4 * (e - c * (kRow / 4));
      const float* const src = p.w + ((size_t)min(co + c, p.Cout - 1) * p.Cin + ci0) * 9;
      if (q.vec_w) {
        wr[i] = *reinterpret_cast<const f32x4*>(src + min(f, w_valid - 4));
      } else {
#pragma unroll
        for (int u = 0; u < 4; ++u) wr[i][u] = src[min(f + u, w_valid - 1)];
      }
    }
    const float* const src = dy0 + (size_t)co * plane;
    const int c_left = p.Cout - co;
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      if (i * kThreads >= n_dy) break;                   // (uniform)
      const bool there = off[i] != 0xffffffffu && (tid + i * kThreads) < c_left * q.pl;
      dr[i] = src[there ? off[i] : 0u];
      dr[i] = there ? dr[i] : 0.f;
    }
  };
  f32x16 acc[NP];
#pragma unroll
  for (int b = 0; b < NP; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[b][r] = 0.f;

  request(0);
  for (int co = 0; co < p.Cout; co += kSplitCo) {
    __syncthreads();                                     // the round before has been read
#pragma unroll
    for (int i = 0; i < NW; ++i) {
      const int e = tid + i * kThreads;
      // (channels beyond Cout: zeros against zeros, as above)
      *reinterpret_cast<f32x4*>(wl + 4 * e) = co + e / (kRow / 4) < p.Cout ? wr[i] : f32x4{0.f, 0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int i = 0; i < ND; ++i) {
      if (i * kThreads >= n_dy) break;
      if (tid + i * kThreads < n_dy) dyl[tid + i * kThreads] = dr[i];
    }
    if (co + kSplitCo < p.Cout) request(co + kSplitCo);
    __syncthreads();
    const float* const w_lane = wl + (8 * wave + h) * kRow + n * 9;
    const float* const d_half = dyl + (8 * wave + h) * q.pl;
#pragma unroll
    for (int tap = 0; tap < 9; ++tap) {
      const int shift = (2 - tap / 3) * q.cw + 2 - tap % 3;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float wv = w_lane[2 * i * kRow + tap];
#pragma unroll
        for (int b = 0; b < NP; ++b)
          acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv, d_half[2 * i * q.pl + base[b] + shift], acc[b], 0, 0, 0);
      }
    }
  }
  // ---- the four waves' sums: wave w finishes registers 4 w .. 4 w + 3, channels 8 w + 4 h + i
  __syncthreads();
  float* const part = reinterpret_cast<float*>(lds);
#pragma unroll
  for (int b = 0; b < NP; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) part[((wave * NP + b) * 16 + r) * 64 + lane] = acc[b][r];
  __syncthreads();
#pragma unroll
  for (int b = 0; b < NP; ++b) {
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      float a[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) a[w] = part[((w * NP + b) * 16 + 4 * wave + i) * 64 + lane];
      v[i] = (a[0] + a[1]) + (a[2] + a[3]);
    }
    if (!ok[b]) continue;
    const int pair = pair0 + px_pair[b], k = pair / p.B, sample = pair - k * p.B, ci = ci0 + 8 * wave + 4 * h;
    const int iy = y0 + px_y[b], ix = x0 + px_x[b];
    const int Kg = p.grad_in_group && !p.pool2 ? 1 : group_frames(p, k);
    for (int j = 0; j < Kg; ++j) {
      const float wj = p.grad_in_group && !p.pool2 ? 1.0f : group_frames(p, k) == p.K ? p.wj[j] : p.wj_last[j];
      const size_t chan0 = (p.grad_in_group && !p.pool2 ? (size_t)pair : (size_t)(k * p.K + j) * p.B + sample) * p.Cin + ci;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (ci + i >= p.Cin) continue;
        const float g = wj * v[i];
        if (!p.pool2) {
          p.grad_in[(chan0 + i) * plane + (size_t)iy * p.W + ix] = g;
          continue;
        }
        // through the pool on load, as above
        float u[4] = {0.25f * g, 0.25f * g, 0.25f * g, 0.25f * g};
        if (p.pool2 == 2) {
          const uint32_t* const src = p.spikes + (chan0 + i) * 2 * p.H * p.Wwi + (size_t)(2 * iy) * p.Wwi + (ix >> 4);
          const uint32_t two = ((src[0] >> (2 * ix & 31)) & 3u) | (((src[p.Wwi] >> (2 * ix & 31)) & 3u) << 2);
          const int best = two ? __ffs(two) - 1 : 0;
#pragma unroll
          for (int e = 0; e < 4; ++e) u[e] = e == best ? g : 0.f;
        }
        float* const dst = p.grad_in + (chan0 + i) * 4 * plane + (size_t)(2 * iy) * (2 * p.W) + 2 * ix;
        dst[0] = u[0]; dst[1] = u[1];
        dst[2 * p.W] = u[2]; dst[2 * p.W + 1] = u[3];
      }
    }
  }
}

// split: dgrad_f32_split_kernel's tile
bool dgrad_f32_tile(const BackwardParams& p, int wi, int np, DgradPlan& q, bool split = false) {
  const int px_max = (split ? 1 : 4 / wi) * np * 32, pl_max = split ? kSplitPl : kM * kThreads, co = split ? kSplitCo : kCo;
  q.xw = std::min(p.W, std::min(64, px_max));
  q.n_segs = (p.W + q.xw - 1) / q.xw;
  q.cw = q.xw + 2;
  for (q.rows = std::min(p.H, px_max / q.xw); q.rows >= 1; --q.rows)
    if ((q.rows + 2) * q.cw <= pl_max) break;
  if (q.rows < 1) return false;
  q.n_strips = (p.H + q.rows - 1) / q.rows;
  q.rows = (p.H + q.n_strips - 1) / q.n_strips;
  q.n_pairs = 1;
  // several (group, sample) pairs while they fit the tile, with 32-bit offsets between them
  if (q.n_strips == 1 && q.n_segs == 1)
    while (q.n_pairs * 2 * q.rows * q.xw <= px_max && q.n_pairs * 2 * (q.rows + 2) * q.cw <= pl_max &&
           (long long)q.n_pairs * 2 * p.Cout * p.H * p.W < (1ll << 31))
      q.n_pairs *= 2;
  q.pair_tiles = (p.G * p.B + q.n_pairs - 1) / q.n_pairs;
  q.ci_groups = (p.Cin + 32 * wi - 1) / (32 * wi);
  q.px = q.n_pairs * q.rows * q.xw;
  q.pl = q.n_pairs * (q.rows + 2) * q.cw;
  q.vec_w = p.Cin % 4 == 0 && ((uintptr_t)p.w & 15u) == 0;
  q.off_dy = co * 288 * wi * 4;
  q.total = std::max(q.off_dy + co * q.pl * 4, split ? np * 16384 : 0);
  return true;
}

}  // namespace

hipError_t backward_dgrad_f32_launch(const BackwardParams& p, hipStream_t s) {
  const int wi = p.Cin > 64 ? 4 : p.Cin > 32 ? 2 : 1;
  DgradPlan q{};
  int np = 0;
  double best = 0.0;
  long long grid = 0;
  for (int n : {4, 2, 1}) {
    DgradPlan c{};
    if (!dgrad_f32_tile(p, wi, n, c)) continue;
    // two resident workgroups share a compute unit's matrix cores: rounds of one workgroup's MFMAs, plus its staging
    const long long tiles = (long long)c.pair_tiles * c.n_strips * c.n_segs * c.ci_groups;
    const double cost = (double)((tiles + 255) / 256) * ((p.Cout + kCo - 1) / kCo) * (n * 36 * 64 + 1800.0);
    if (np && cost >= best) continue;
    np = n;
    best = cost;
    q = c;
    grid = tiles;
  }
  // Four waves that share the output channels, as long as two workgroups per compute unit hold all the tiles (us of the kernel, split / not:
  // 128 -> 128, 64 pairs at 8 x 8 (512 tiles) 31 / 51, at 4 x 4 (128) 25 / 53; at 16 x 16 (2048) the matrix cores are the bound and the weights
  // come four times as often: 115 / 72)
  bool split = false;
  DgradPlan c{};
  if (dgrad_f32_tile(p, 1, 1, c, true)) {
    const long long tiles = (long long)c.pair_tiles * c.n_strips * c.n_segs * c.ci_groups;
    const double cost = ((p.Cout + kSplitCo - 1) / kSplitCo) * (tiles > 256 ? 1.7 : 1.15) * (36 * 64 + 3000.0) + 4600.0;
    if (tiles <= 512 && (!np || cost < best)) {
      split = true;
      np = 1;
      q = c;
      grid = tiles;
    }
  }
  if (!np || grid >= (1ll << 31)) return hipErrorInvalidValue;
  auto launch = [&](auto kern) -> hipError_t {
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(kThreads), q.total, s, p, q);
    return hipGetLastError();
  };
  auto with_np = [&](auto wi_) -> hipError_t {
    constexpr int WI = decltype(wi_)::value;
    return np == 4 ? launch(&dgrad_f32_kernel<WI, 4>) : np == 2 ? launch(&dgrad_f32_kernel<WI, 2>) : launch(&dgrad_f32_kernel<WI, 1>);
  };
  if (split) return launch(&dgrad_f32_split_kernel<1>);
  switch (wi) {
    case 4: return with_np(std::integral_constant<int, 4>{});
    case 2: return with_np(std::integral_constant<int, 2>{});
    default: return with_np(std::integral_constant<int, 1>{});
  }
}

}  // namespace tac
