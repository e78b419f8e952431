// Input gradient of the conv-LIF layer on the matrix cores, as accurate as in fp32, for the stride-1 layers that the bf16 kernels do not take:
//   dA_k[ci][iy][ix] = sum over co, ky, kx of W[co][ci][ky][kx] * dY_k[co][iy + 1 - ky][ix + 1 - kx],
// written per group, per frame of the group (times beta^(Kg-1-j)), or through the pool on load.
//
// dgrad_f32_kernel: D[32 ci x 32 px] += W^T[32 ci x 16 co] . dY[16 co x 32 px].  v_mfma_f32_32x32x2_f32 takes 512 cycles for the 16 channels; here each fp32
// value is three bf16 values whose sum it is, and six products of v_mfma_f32_32x32x16_bf16 (192 cycles) are all that reach 2^-26 of the largest.
// The products of the first parts, once a tap and 16 channels, are one chain of sums; the five others, whose roundings are 2^-8 as large, are another, added at the end.
// Few roundings at full size make the result more accurate than products of fp32 are, whatever the number of channels: 96 <- 128 at 64 x 40, B = 16, three
// groups 2.2e-7 of the norm instead of 6.0e-7, 0.36 to 0.44 of the error on 30 layers of 8 to 128 output channels, 0.4 to 0.6 with 1 to 24 (in one chain
// two output channels were off by twice as much as products of fp32).  A round with an infinity, a NaN, or values that the subnormal numbers cut (below 2^-90) multiplies the
// values put together again on v_mfma_f32_32x32x2_f32.
// Workgroup = 32 input channels x a tile of pixels (rows of one or, in small images, of several (group, sample) pairs); four waves share the pixels,
// NP blocks of 32 each.  Sixteen output channels at a time go through LDS as thirds, [third][tap][half of the channels][ci] and [third][half][position];
// the next sixteen are requested before the MFMAs.  Two or three workgroups share a compute unit, so that one's splitting (400 vector instructions a round
// and wave, which bound it together with the MFMAs' 1728 NP cycles) runs under another's products.
// Products of fp32 and these (us): 96 <- 128 at 64 x 40, B = 16, three groups 537 -> 192; 32 <- 64 at 14 x 14, B = 128, seven groups 91 -> 59; 160 <- 96 at 41 x 33,
// 144 pairs 1290 -> 343.  Up to eight output channels (HALVES = 1): 64 <- 8 at 54 x 57, 144 pairs 91 -> 58, on fewer tiles than compute units 4.8 -> 5.0 (in full rounds 6.2).
//
// Few pixels (small images, small batches) leave that kernel with a few dozen workgroups that go through Cout / 16 rounds of two barriers
// each.  dgrad_f32_split_kernel shares a workgroup's 32 input channels x NP blocks of 32 pixels among four waves by output channel, in products of fp32:
// 32 of them a round, four times the workgroups, and the waves' sums meet in LDS at the end.
#include "tac_dgrad_plan.h"

namespace tac {

namespace {

constexpr int kThreads = kDgradThreads;
constexpr int kM = kDgradM;
typedef __attribute__((ext_vector_type(4))) float f32x4;

__device__ __forceinline__ int group_frames(const BackwardParams& p, int k) {
  return (k == p.G - 1 && p.K_last) ? p.K_last : p.K;
}

// x = hi + mid + lo, three bf16 values (8 bits each and their signs: all 24 bits of x) of eight values.  A set has none where its largest value is infinite, a NaN or rounds
// to an infinite hi, or lies (not being zero) below 2^-90, where the subnormal numbers begin to cut the lower parts off: then hi and mid are the two halves of
// the fp32 value and lo is kHalves, which is no third of anything.
struct Thirds {
  u32x4 hi, mid, lo;
};
constexpr uint32_t kThirdsFrom = (127u - 90u) << 23, kThirdsTo = 0x7f7f8000u, kHalves = 0x7fc1u;
__device__ __forceinline__ Thirds thirds(const float (&x)[8], bool& none) {
  Thirds o;
  uint32_t most = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) most = max(most, __float_as_uint(x[i]) & 0x7fffffffu);
  if (__builtin_expect(most - kThirdsFrom < kThirdsTo - kThirdsFrom || most == 0, 1)) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      o.hi[i] = pack_bf16(x[2 * i], x[2 * i + 1]);
      const float r0 = x[2 * i] - __uint_as_float(o.hi[i] << 16), r1 = x[2 * i + 1] - __uint_as_float(o.hi[i] & 0xffff0000u);
      o.mid[i] = pack_bf16(r0, r1);
      o.lo[i] = pack_bf16(r0 - __uint_as_float(o.mid[i] << 16), r1 - __uint_as_float(o.mid[i] & 0xffff0000u));
    }
  } else {
    none = true;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t u0 = __float_as_uint(x[2 * i]), u1 = __float_as_uint(x[2 * i + 1]);
      o.hi[i] = u0 >> 16 | (u1 & 0xffff0000u);
      o.mid[i] = (u0 & 0xffffu) | u1 << 16;
      o.lo[i] = kHalves | kHalves << 16;
    }
  }
  return o;
}
// The value again.  hi + (mid + lo) is exact.
__device__ __forceinline__ float whole(const uint8_t* hi, int term) {
  auto bits = [&](int part) { return (uint32_t)*reinterpret_cast<const uint16_t*>(hi + part * term) << 16; };
  const uint32_t h = bits(0), m = bits(1), l = bits(2);
  return l == kHalves << 16 ? __uint_as_float(h | m >> 16) : __uint_as_float(h) + (__uint_as_float(m) + __uint_as_float(l));
}

// LDS of a third of the weights: a tap's HALVES x 32 x 8 weights (16 bytes more spread the taps of an input channel over the banks), and with one half a tap of zeros
__host__ __device__ constexpr int tap_bytes(int halves) { return halves * 512 + 16; }
__host__ __device__ constexpr int w_bytes(int halves) { return (halves == 2 ? 9 : 10) * tap_bytes(halves); }

// FAR: planes of 2^23 pixels and more, whose channels have a buffer descriptor each.
// HALVES = 1: at most eight output channels, one round.  The 16 places of a product are eight channels of two taps: five products of two taps instead of nine of which half is
// zeros, and half of the splitting.
template <int NP, bool FAR, int HALVES>
__global__ __launch_bounds__(kThreads, NP == 1 ? 3 : 2) void dgrad_f32_kernel(const BackwardParams p, const DgradPlan q) {
  constexpr int kCo = 8 * HALVES, kTapBytes = tap_bytes(HALVES), kWBytes = w_bytes(HALVES), kW = HALVES * 288;
  constexpr int NW = (kW + kThreads - 1) / kThreads;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  uint8_t* const dyl = lds + q.off_dy;
  const int d_term = q.pl * 16 * HALVES;                 // bytes of one third of dY, [half of the channels][position]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wx = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  uint32_t t = blockIdx.x;
  const int ci0 = (int)(t % (uint32_t)q.ci_groups) * 32; t /= (uint32_t)q.ci_groups;
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
  // What the thread stages, as byte offsets (below 2^30) from the row above the tile's first in a channel of dY, from a channel's first weight of the tile; a load
  // at 2^30 or more gives zero
  constexpr uint32_t kOutside = 1u << 30;
  uint32_t off[kM], w_off[NW];
  int w_dst[NW];
#pragma unroll
  for (int m = 0; m < kM; ++m) {
    const int e = tid + m * kThreads;
    const int line = e / q.cw, c = e - line * q.cw, pr = line / (q.rows + 2), r = line - pr * (q.rows + 2);
    const int y = y0 + r - 1, x = x0 + c - 1;
    const bool inside = e < q.pl && pr < pairs && y >= 0 && y < p.H && x >= 0 && x < p.W;
    off[m] = inside ? (uint32_t)((size_t)pr * p.Cout * plane + (size_t)r * p.W + x) * 4u : kOutside;
  }
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const int e = tid + i * kThreads, half = e >= 288, f = e - 288 * half;
    w_off[i] = e < kW ? (uint32_t)(8 * half * p.Cin * 9 + f) * 4u : kOutside;
    w_dst[i] = f % 9 * kTapBytes + half * 512 + f / 9 * 16;          // (half 0 only with HALVES = 1)
  }
  const float* const dy0 = p.grad_y + (size_t)pair0 * p.Cout * plane + ((ptrdiff_t)y0 - 1) * p.W;      // (what lies in front of the array is never loaded)
  const float* const w0 = p.w + (size_t)ci0 * 9;
  auto source = [](const float* at, size_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(at), 0, (int)(bytes < kOutside ? bytes : kOutside), 0x00020000);
  };
  float wr[NW][8], dr[kM][kCo];
  auto request = [&](int co) {
    // output channels beyond the last are beyond the end; input channels beyond the last find other weights, and are not stored
    const size_t row = (size_t)co * p.Cin * 9, end = (size_t)p.Cout * p.Cin * 9 - (size_t)ci0 * 9;
    const auto w_src = source(w0 + row, row < end ? (end - row) * 4 : 0);
#pragma unroll
    for (int i = 0; i < NW; ++i)
#pragma unroll
      for (int c = 0; c < 8; ++c)
        wr[i][c] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(w_src, (int)(w_off[i] + (uint32_t)c * (uint32_t)p.Cin * 36u), 0, 0));
    const auto d_src = source(dy0 + (size_t)co * plane, kOutside);
#pragma unroll
    for (int c = 0; c < kCo; ++c) {
      const bool there = co + c < p.Cout;
      const auto own = FAR ? source(dy0 + (size_t)(co + c) * plane, there ? kOutside : 0) : d_src;
      const uint32_t chan = FAR ? 0u : there ? (uint32_t)c * (uint32_t)plane * 4u : kOutside;
#pragma unroll
      for (int m = 0; m < kM; ++m) dr[m][c] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(own, (int)(off[m] + chan), 0, 0));
    }
  };
  f32x16 acc[NP], small[NP];                             // the products of the first parts; the others, which start at 2^-8 of those
#pragma unroll
  for (int b = 0; b < NP; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[b][r] = small[b][r] = 0.f;
  const bool active = wx * NP * 32 < pairs * per_pair;   // wave-uniform

  int* const bad_round = reinterpret_cast<int*>(lds + q.off_bad);        // of this round and of the next
  if (tid < 2) bad_round[tid] = 0;
  if (HALVES == 1 && tid < 96) *reinterpret_cast<u32x4*>(lds + (tid >> 5) * kWBytes + 9 * kTapBytes + (tid & 31) * 16) = u32x4{0, 0, 0, 0};
  request(0);
  for (int co = 0, round = 0; co < p.Cout; co += kCo, round ^= 1) {
    __syncthreads();                                     // the round before has been read
    bool bad = false;
    if (tid == 0) bad_round[round ^ 1] = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i)
      if (tid + i * kThreads < kW) {
        const Thirds v = thirds(wr[i], bad);
        uint8_t* const dst = lds + w_dst[i];
        *reinterpret_cast<u32x4*>(dst) = v.hi;
        *reinterpret_cast<u32x4*>(dst + kWBytes) = v.mid;
        *reinterpret_cast<u32x4*>(dst + 2 * kWBytes) = v.lo;
      }
#pragma unroll
    for (int m = 0; m < kM; ++m)
      if (tid + m * kThreads < q.pl) {
#pragma unroll
        for (int half = 0; half < HALVES; ++half) {
          float x[8];
#pragma unroll
          for (int c = 0; c < 8; ++c) x[c] = dr[m][8 * half + c];
          const Thirds v = thirds(x, bad);
          uint8_t* const dst = dyl + (half * q.pl + tid + m * kThreads) * 16;
          *reinterpret_cast<u32x4*>(dst) = v.hi;
          *reinterpret_cast<u32x4*>(dst + d_term) = v.mid;
          *reinterpret_cast<u32x4*>(dst + 2 * d_term) = v.lo;
        }
      }
    if (co + kCo < p.Cout) request(co + kCo);
    if (bad) bad_round[round] = 1;
    __syncthreads();
    const bool any_bad = __builtin_amdgcn_readfirstlane(bad_round[round]) != 0;
    if (!active) continue;
    // a step: a tap of both halves of the channels, or two taps, one on either lane half (the tenth is zeros)
    constexpr int kSteps = HALVES == 2 ? 9 : 5;
    const uint8_t* const w_lane = HALVES == 2 ? lds + lane * 16 : lds + h * kTapBytes + n * 16;
    const uint8_t* const d_lane = HALVES == 2 ? dyl + h * q.pl * 16 : dyl;
    auto shift = [&](int step) {
      auto of = [&](int tap) { return (2 - tap / 3) * q.cw + 2 - tap % 3; };
      if constexpr (HALVES == 2) return of(step);
      else return h ? of(min(2 * step + 1, 8)) : of(2 * step);
    };
    constexpr int kStepBytes = HALVES == 2 ? kTapBytes : 2 * kTapBytes;
    if (__builtin_expect(any_bad, 0)) {
      // the round in products of fp32
#pragma clang loop unroll(disable)
      for (int step = 0; step < kSteps; ++step) {
        const int sh = shift(step);
#pragma clang loop unroll(disable)
        for (int i = 0; i < 8; ++i) {
          const float wv = whole(w_lane + step * kStepBytes + 2 * i, kWBytes);
#pragma unroll
          for (int b = 0; b < NP; ++b) {
            float dv = whole(d_lane + (base[b] + sh) * 16 + 2 * i, d_term);
            if (HALVES == 1 && step == 4 && h) dv = 0.f;             // (no infinity times the zeros of the tenth tap)
            acc[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(wv, dv, acc[b], 0, 0, 0);
          }
        }
      }
      continue;
    }
    auto load = [&](const uint8_t* at) { return *reinterpret_cast<const bf16x8*>(at); };
#pragma unroll
    for (int step = 0; step < kSteps; ++step) {
      const int sh = shift(step);
      bf16x8 w[3], d[NP][3];
#pragma unroll
      for (int e = 0; e < 3; ++e) w[e] = load(w_lane + step * kStepBytes + e * kWBytes);
#pragma unroll
      for (int b = 0; b < NP; ++b)
#pragma unroll
        for (int e = 0; e < 3; ++e) d[b][e] = load(d_lane + (base[b] + sh) * 16 + e * d_term);
      // the products of 2^-18 and more of the largest; the three left out are below 2^-26 of it
#pragma unroll
      for (int e = 0; e < 5; ++e) {
        constexpr int kFromW[5] = {0, 2, 1, 0, 1}, kFromD[5] = {2, 0, 1, 1, 0};
#pragma unroll
        for (int b = 0; b < NP; ++b) small[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[kFromW[e]], d[b][kFromD[e]], small[b], 0, 0, 0);
      }
#pragma unroll
      for (int b = 0; b < NP; ++b) acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w[0], d[b][0], acc[b], 0, 0, 0);
    }
  }
  if (!active) return;
#pragma unroll
  for (int b = 0; b < NP; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[b][r] += small[b][r];
  // ---- register r of acc[b] on lane (n, h): input channel 8 (r / 4) + 4 h + r % 4 of the wave, pixel n of block b
  const int ci_w = ci0 + 4 * h;
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

}  // namespace

hipError_t backward_dgrad_f32_launch(const BackwardParams& p, hipStream_t s) {
  DgradPlan q{};
  auto launch = [&](auto kern) -> hipError_t {
    const long long grid = dgrad_f32_tiles(q);
    if (grid >= (1ll << 31)) return hipErrorInvalidValue;
    if (q.total > 64 * 1024) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(kThreads), q.total, s, p, q);
    return hipGetLastError();
  };
  int np = 0;
  if (dgrad_f32_choose(p, q, np)) {
    q.vec_w = p.Cin % 4 == 0 && ((uintptr_t)p.w & 15u) == 0;
    q.off_dy = kSplitCo * 288 * 4;
    q.total = std::max(q.off_dy + kSplitCo * q.pl * 4, 16384);
    return launch(&dgrad_f32_split_kernel<1>);
  }
  if (!np) return hipErrorInvalidValue;
  const int halves = p.Cout <= 8 ? 1 : 2;
  q.off_dy = 3 * w_bytes(halves);
  q.off_bad = q.off_dy + 3 * 16 * halves * q.pl;
  q.total = q.off_bad + 16;
  const bool far = (long long)p.H * p.W >= (1ll << 23);
  auto with = [&](auto np_, auto halves_) {
    constexpr int NP = decltype(np_)::value, HALVES = decltype(halves_)::value;
    return far ? launch(&dgrad_f32_kernel<NP, true, HALVES>) : launch(&dgrad_f32_kernel<NP, false, HALVES>);
  };
  constexpr std::integral_constant<int, 1> one;
  constexpr std::integral_constant<int, 2> two;
  if (halves == 1) return np == 2 ? with(two, one) : with(one, one);
  return np == 2 ? with(two, two) : with(one, two);
}

}  // namespace tac
