// Weight and bias gradient of the conv-LIF layer in fp32 on the matrix cores (v_mfma_f32_32x32x2_f32: operands, products
// and sums in fp32), for every layer that the bf16 kernel does not take: fp32 layers, stride 2, real-valued frames, the
// mean pool on load, channel counts and widths of any kind.
//   dW[co][col] = sum over groups k, samples b, output pixels of dY_k[co][pixel] * A_k[ci][pixel's input under the tap],
// col = 9 ci + tap being the place of (ci, ky, kx) in dW[co], so that the 32 columns of an MFMA tile are 32 consecutive
// floats of dW whatever the number of input channels (one input channel fills 9 columns of a tile, 32 channels 9 tiles),
// and the atomics that combine the workgroups' sums hit consecutive addresses.
//
// Workgroup = WC blocks of 32 output channels x some column tiles x a slice of the list of items (group, sample, strip of
// output rows, segment of the row).  Per item the strip's dY values go to LDS as [channel][pixel] (rows padded to four
// pixels, requested one item ahead) and the aggregates of the columns' input channels as [channel][row][column], rebuilt
// from the packed words (a thread per 16 pixels).  An operand of four MFMAs is then one 16-byte read of dY (four pixels per
// lane half) and four 4-byte reads of the aggregates under the lane's own tap.  The four waves are WC channel blocks x WN
// blocks of NT column tiles x WP parts of the pixels.
//
// Against one thread per pixel with 8 x 9 accumulators, which rebuilt the aggregates once per eight output channels (the
// vector kernel before): see the figures at wgrad_f32_plan.
#include <algorithm>
#include "tac_mfma_common.h"

namespace tac {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

struct WgradPlan {
  int wn, wp;                     // waves over the column tiles, over the pixels
  int co_tiles, col_groups, split;
  int rows, xw, n_strips, n_segs; // output rows and columns of an item, strips and segments of the image
  int npx, nq, pxs;               // pixels (padded rows) and quads of an item, dwords per channel of dY in LDS
  int rows_in, cw, cp;            // aggregate rows, dwords per row and per channel
  int n_ch;                       // input channels of a column group, at most
  int off_a, off_q, total;        // LDS bytes
};

__device__ __forceinline__ int group_frames(const BackwardParams& p, int k) {
  return (k == p.G - 1 && p.K_last) ? p.K_last : p.K;
}

// i / d for a wave-uniform divisor and i below 2^20 (the quotient (i + 1/2) / d stays clear of integers by 1 / (2 d))
__device__ __forceinline__ int small_div(int i, float r) { return (int)(((float)i + 0.5f) * r); }

// blocks of 64 pixels of an item (dY values in registers per thread: times 32 WC / waves channels)
__host__ __device__ constexpr int wgrad_m(int wc, int nt, int waves) {
  return waves == 8 ? 4 : wc == 4 ? (nt >= 5 ? 1 : 2) : wc == 2 ? (nt >= 5 ? 2 : 4) : 4;
}

// DENSE: real-valued frames.  WV waves (4; 8 where dW has one column tile and there is nothing but pixels to share out).
template <int S, int WC, int NT, bool DENSE, int WV>
__global__ __launch_bounds__(64 * WV, 2) void wgrad_f32_kernel(const BackwardParams p, const WgradPlan q) {
  constexpr int kThreads = 64 * WV, M = wgrad_m(WC, NT, WV), C = 32 * WC / WV;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  float* const dyl = reinterpret_cast<float*>(lds);
  float* const agg = reinterpret_cast<float*>(lds + q.off_a);
  int32_t* const qoff = reinterpret_cast<int32_t*>(lds + q.off_q);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  uint32_t t0 = blockIdx.x;
  const int slice = (int)(t0 % (uint32_t)q.split); t0 /= (uint32_t)q.split;
  const int co0 = (int)(t0 % (uint32_t)q.co_tiles) * (32 * WC);
  const int col_first = (int)(t0 / (uint32_t)q.co_tiles) * (q.wn * NT * 32);
  const int n_cols = 9 * p.Cin;
  const int ci_first = col_first / 9;
  const int n_ch = min(min(col_first + q.wn * NT * 32, n_cols) - 1, n_cols - 1) / 9 - ci_first + 1;
  const int wc = wave % WC, rest = wave / WC;
  const int wn = rest % q.wn, wp = rest / q.wn;
  const size_t plane = (size_t)p.Ho * p.Wo;

  // columns of the lane: dword offset of (channel, ky, kx) in the aggregates
  int coff[NT];
  const int col_lane = col_first + wn * NT * 32 + n;
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int col = col_lane + 32 * t;
    const int ci = col / 9, tap = col - 9 * ci, ky = (tap * 11) >> 5, kx = tap - 3 * ky;
    coff[t] = col < n_cols ? (ci - ci_first) * q.cp + ky * q.cw + kx : 0;
  }
  // quads of the item: (row, four pixels) -> dword offset of the first one's input under tap (0, 0)
  const int quads_row = q.xw >> 2;
  for (int i = tid; i < q.nq + 2; i += kThreads) {
    const int yl = i / quads_row, xq = i - yl * quads_row;
    qoff[i] = i < q.nq ? yl * S * q.cw + xq * 4 * S : 0;
  }
  // the quad behind an odd number of them, and everything an aggregate is never written to, is zero
  for (int i = tid; i < 32 * WC; i += kThreads) *reinterpret_cast<f32x4*>(dyl + i * q.pxs + q.npx) = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int i = tid; i < q.n_ch * q.cp; i += kThreads) agg[i] = 0.f;

  // dY: wave w takes the channels w, w + WV, ..; lane + 64 m is a pixel of the item
  int px_y[M], px_x[M];
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int px = lane + 64 * m;
    px_y[m] = px < q.npx ? px / q.xw : 1 << 20;
    px_x[m] = px % q.xw;
  }
  float wd[C][M];
  const int items = p.G * p.B * q.n_strips * q.n_segs;
  struct Where { int k, b, y0, x0; };
  // the items of the slice are `split` apart: the step is taken apart once and added with carries
  struct Index { int seg, strip, b, k; };
  auto take_apart = [&](int it) {
    Index x;
    x.seg = it % q.n_segs; it /= q.n_segs;
    x.strip = it % q.n_strips; it /= q.n_strips;
    x.k = it / p.B; x.b = it - x.k * p.B;
    return x;
  };
  const Index by = take_apart(q.split);
  auto advance = [&](Index& x) {
    x.seg += by.seg; x.strip += by.strip; x.b += by.b; x.k += by.k;
    if (x.seg >= q.n_segs) { x.seg -= q.n_segs; ++x.strip; }
    if (x.strip >= q.n_strips) { x.strip -= q.n_strips; ++x.b; }
    if (x.b >= p.B) { x.b -= p.B; ++x.k; }
  };
  auto where = [&](const Index& x) { return Where{x.k, x.b, x.strip * q.rows, x.seg * q.xw}; };
  auto request = [&](const Where& w) {
    uint32_t off[M];
#pragma unroll
    for (int m = 0; m < M; ++m)
      off[m] = (uint32_t)(min(w.y0 + min(px_y[m], q.rows), p.Ho - 1) * p.Wo + min(w.x0 + px_x[m], p.Wo - 1));
    const float* const src = p.grad_y + ((size_t)w.k * p.B + w.b) * p.Cout * plane;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const float* const chan = src + (size_t)min(co0 + wave + WV * c, p.Cout - 1) * plane;     // (rows beyond Cout are not stored)
#pragma unroll
      for (int m = 0; m < M; ++m) wd[c][m] = chan[off[m]];
    }
  };

  const float inv_rows = 1.0f / (float)q.rows_in;
  f32x16 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
  float bias = 0.f;

  Index ahead = take_apart(min(slice, items - 1));
  Where w = where(ahead);
  if (slice < items) request(w);
  for (int it = slice; it < items; it += q.split) {
    const int Kg = group_frames(p, w.k);
    const float* const wj = Kg == p.K ? p.wj : p.wj_last;
    __syncthreads();                                     // the item before has been read
    // ---- dY to LDS, zeros where the item has no pixel
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const bool inside = w.y0 + px_y[m] < p.Ho && px_y[m] < q.rows && w.x0 + px_x[m] < p.Wo;
      if (lane + 64 * m < q.npx) {
        uint32_t at = (uint32_t)(wave * q.pxs + lane + 64 * m);
#pragma unroll
        for (int c = 0; c < C; ++c) {
          asm volatile("" : "+v"(at));                   // one address register, not one per channel kept across items
          dyl[at] = inside ? wd[c][m] : 0.f;
          at += WV * q.pxs;
        }
      }
    }
    // ---- aggregates of rows y0 S - 1 .., columns x0 S - 1 ..
    const int iy0 = w.y0 * S - 1, ix0 = w.x0 * S - 1;
    if constexpr (DENSE) {
      // real-valued frames [T][B][Cin][H][W] (the continuous-valued first layer, Sec. 4.2)
      const size_t fs = (size_t)p.B * p.Cin * p.H * p.W;
      const float* const x = reinterpret_cast<const float*>(p.spikes) + ((size_t)w.k * p.K * p.B + w.b) * p.Cin * p.H * p.W;
      const float inv_cw = 1.0f / (float)q.cw;
      for (int e = tid; e < n_ch * q.rows_in * q.cw; e += kThreads) {
        const int line = small_div(e, inv_cw), c = e - line * q.cw;
        const int ch = small_div(line, inv_rows), r = line - ch * q.rows_in;
        const int iy = iy0 + r, ix = ix0 + c;
        const bool inside = iy >= 0 && iy < p.H && ix >= 0 && ix < p.W;
        const float* const src = x + ((size_t)(ci_first + ch) * p.H + min(max(iy, 0), p.H - 1)) * p.W + min(max(ix, 0), p.W - 1);
        float a = 0.f;
        for (int j = 0; j < Kg; ++j) a = fmaf(wj[j], src[j * fs], a);
        agg[ch * q.cp + r * q.cw + c] = inside ? a : 0.f;
      }
    } else {
      const int hs = p.pool2 ? 2 * p.H : p.H;
      const size_t fs = (size_t)p.B * p.Cin * hs * p.Wwi;
      const uint32_t* const frames = p.spikes + ((size_t)w.k * p.K * p.B + w.b) * p.Cin * hs * p.Wwi;
      // a unit is 16 pixels of a row: half a stored word, or with a pool on load the whole word
      const int u_first = ix0 >> 4, n_uu = ((ix0 + q.cw - 1) >> 4) - u_first + 1;
      const float inv_uu = 1.0f / (float)n_uu;
      for (int e = tid; e < n_ch * q.rows_in * n_uu; e += kThreads) {
        const int line = small_div(e, inv_uu), unit = u_first + e - line * n_uu;
        const int ch = small_div(line, inv_rows), r = line - ch * q.rows_in;
        const int iy = iy0 + r, word = p.pool2 ? unit : unit >> 1;
        const bool inside = iy >= 0 && iy < p.H && word >= 0 && word < p.Wwi;
        const uint32_t* const src = frames + ((size_t)(ci_first + ch) * hs + (p.pool2 ? 2 : 1) * min(max(iy, 0), p.H - 1)) * p.Wwi +
                                    min(max(word, 0), p.Wwi - 1);
        float a[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) a[i] = 0.f;
        for (int j = 0; j < Kg; j += 4) {
          uint32_t f[4], f1[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) f[u] = f1[u] = src[(size_t)min(j + u, Kg - 1) * fs];
          if (p.pool2) {
#pragma unroll
            for (int u = 0; u < 4; ++u) f1[u] = src[(size_t)min(j + u, Kg - 1) * fs + p.Wwi];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            const float wt = j + u < Kg && inside ? wj[min(j + u, Kg - 1)] : 0.f;
            if (p.pool2 == 1) {
              // mean of the four bits: counts of 0..4 in nibbles, pixel i of the word in nibble i / 2 of lo (even) or hi
              const uint32_t t = (f[u] & 0x55555555u) + ((f[u] >> 1) & 0x55555555u), b = (f1[u] & 0x55555555u) + ((f1[u] >> 1) & 0x55555555u);
              const uint32_t lo = (t & 0x33333333u) + (b & 0x33333333u), hi = ((t >> 2) & 0x33333333u) + ((b >> 2) & 0x33333333u);
#pragma unroll
              for (int i = 0; i < 16; ++i)
                a[i] += (0.25f * (float)__builtin_amdgcn_ubfe(i & 1 ? hi : lo, 4 * (i >> 1), 4)) * wt;
            } else {
              // pixel i at bit i, or with the max pool the OR of its block at bit 2 i
              uint32_t o = f[u] | f1[u];
              o = p.pool2 ? pool_pairs(o) : o >> (16 * (unit & 1));
#pragma unroll
              for (int i = 0; i < 16; ++i) a[i] += (o >> i) & 1u ? wt : 0.f;
            }
            __builtin_amdgcn_sched_barrier(0);           // a frame after the other: the accumulators leave few registers
          }
        }
        float* const dst = agg + ch * q.cp + r * q.cw;
        const int c0 = unit * 16 - ix0;                  // column of the unit's first pixel
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (c0 + i >= 0 && c0 + i < q.cw) dst[c0 + i] = a[i];
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    advance(ahead);
    const Where next = where(ahead);
    if (it + q.split < items) request(next);
    __syncthreads();
    // ---- MFMAs: a step is two quads, one per lane half.  Pixels that only fill a quad have dY = 0; where their aggregates
    //      may be infinite (real-valued frames) those are replaced as well.
    const float* const dy_lane = dyl + (wc * 32 + n) * q.pxs;
    for (int i = wp; 2 * i < q.nq; i += q.wp) {
      const int quad = 2 * i + h;
      const f32x4 g = *reinterpret_cast<const f32x4*>(dy_lane + 4 * quad);
      const float* const a_quad = agg + qoff[quad];
      int real = 4;                                      // of the quad's pixels
      if constexpr (DENSE) {
        const int yl = quad / quads_row;
        real = quad < q.nq && w.y0 + yl < p.Ho ? p.Wo - w.x0 - 4 * (quad - yl * quads_row) : 0;
      }
      // the aggregates of tile t + 1 are requested in front of the MFMAs of tile t
      float a[2][4];
      auto fetch = [&](int t) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          a[t & 1][u] = a_quad[coff[t] + u * S];
          if (DENSE && u >= real) a[t & 1][u] = 0.f;
        }
      };
      fetch(0);
      bias += (g[0] + g[1]) + (g[2] + g[3]);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (t + 1 < NT) fetch(t + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(g[u], a[t & 1][u], acc[t], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    w = next;
  }
  // register r of acc[t] on lane (n, h): output channel 8 (r / 4) + 4 h + r % 4 of the wave, column n of tile t.  Waves that
  // share the pixels of a tile add up through LDS first: all workgroups end at about the same time, one address takes
  // an addition about every 0.1 us, and the chip some 200 a nanosecond (32 channels x 9 columns from 2048 waves: 190 us).
  auto add = [&](int t, int r, float v) {
    const int co = co0 + wc * 32 + 8 * (r >> 2) + 4 * h + (r & 3), col = col_lane + 32 * t;
    if (co < p.Cout && col < n_cols) atomicAdd(p.grad_w + (size_t)co * n_cols + col, v);
  };
  bias += __shfl_xor(bias, 32, 64);
  if (q.wp == 1) {
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int r = 0; r < 16; ++r) add(t, r, acc[t][r]);
  } else {
    float* const red = reinterpret_cast<float*>(lds);    // [wave][register][lane]
    const int stride = WC * q.wn * 16 * 64, first = (wave % (WC * q.wn)) * 16 * 64 + lane;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      __syncthreads();
#pragma unroll
      for (int r = 0; r < 16; ++r) red[(wave * 16 + r) * 64 + lane] = acc[t][r];
      __syncthreads();
      for (int r = wp; r < 16; r += q.wp) {
        float v = 0.f;
        for (int w = 0; w < q.wp; ++w) v += red[first + w * stride + r * 64];
        add(t, r, v);
      }
    }
    __syncthreads();
    red[wave * 64 + lane] = bias;
    __syncthreads();
    bias = 0.f;
    if (wp == 0)
      for (int w = 0; w < q.wp; ++w) bias += red[(wave + w * WC * q.wn) * 64 + lane];
  }
  if (p.grad_bias && col_first == 0 && wn == 0 && wp == 0) {
    const int co = co0 + wc * 32 + n;
    if (h == 0 && co < p.Cout) atomicAdd(p.grad_bias + co, bias);
  }
}

bool wgrad_f32_tile(const BackwardParams& p, int wc, int nt, int waves, WgradPlan& q) {
  const int S = p.stride, tiles = (9 * p.Cin + 31) / 32;
  q.wn = 1;
  while (q.wn < waves / wc && q.wn * nt < tiles) q.wn *= 2;
  q.wp = waves / wc / q.wn;
  q.co_tiles = (p.Cout + 32 * wc - 1) / (32 * wc);
  q.col_groups = (tiles + q.wn * nt - 1) / (q.wn * nt);
  q.n_ch = std::min(p.Cin, (q.wn * nt * 32 + 8) / 9 + 1);
  const int npx_max = 64 * wgrad_m(wc, nt, waves);
  for (q.xw = std::min(64, (p.Wo + 3) / 4 * 4); q.xw >= 4; q.xw = (q.xw / 2 + 3) / 4 * 4) {
    q.n_segs = (p.Wo + q.xw - 1) / q.xw;
    q.cw = ((q.xw - 1) * S + 3) | 1;                     // odd: rows of a channel start in different LDS banks
    for (q.rows = std::max(1, std::min(p.Ho, npx_max / q.xw)); q.rows >= 1; --q.rows) {
      q.n_strips = (p.Ho + q.rows - 1) / q.rows;
      q.rows = (p.Ho + q.n_strips - 1) / q.n_strips;     // strips of the same height, as far as it goes
      q.npx = q.rows * q.xw;
      q.nq = q.npx / 4;
      q.pxs = q.npx + 4;
      if (q.pxs / 4 % 2 == 0) q.pxs += 4;                // an odd number of 16-byte units: 16 channels cover the banks
      q.rows_in = (q.rows - 1) * S + 3;
      q.cp = q.rows_in * q.cw;
      q.off_a = 32 * wc * q.pxs * 4;
      q.off_q = q.off_a + (q.n_ch * q.cp + 4 * S) * 4;   // a quad beyond the image's last column reads a little further
      q.off_q = (q.off_q + 15) & ~15;
      q.total = std::max(q.off_q + (q.nq + 2) * 4, q.wp > 1 ? waves * 16 * 64 * 4 : 0);
      if (q.total <= (q.rows > 1 && waves == 4 ? 80 : 150) * 1024 && (long long)q.n_ch * q.cp < (1 << 20)) return true;
    }
    if (q.xw == 4) break;
  }
  return false;
}

}  // namespace

// Which tile: the column tiles per wave that leave the fewest MFMAs on columns that do not exist, a wave's time per item
// being its tiles (shared by the waves over the pixels) plus about one and a half tiles' worth of staging.
// Against the vector kernel: 32 -> 64 behind the mean pool at 14 x 14, B = 128, 7 groups of 4 frames 425 -> 71 us;
// 1 -> 32 at 28 x 28 of the same network 149 -> 79 us; 128 -> 128, B = 16, 4 groups of 4 frames at 8 x 8 / 4 x 4
// 368 / 378 -> 50 / 44 us; 2 -> 128 real-valued at 64 x 64 197 -> 66 us.
// One column tile (up to three input channels): eight waves share out the pixels.
hipError_t backward_wgrad_f32_launch(const BackwardParams& p, hipStream_t s) {
  const bool one_tile = 9 * p.Cin <= 32;
  const int waves = one_tile ? 8 : 4;
  const int wc = one_tile ? 1 : p.Cout > 64 ? 4 : p.Cout > 32 ? 2 : 1;
  WgradPlan q{};
  int nt = 0;
  double best = 0.0;
  for (int t : {6, 5, 3, 1}) {
    if ((p.dense && t > 3) || (one_tile && t > 1)) continue;           // (real-valued frames: first layers have few columns)
    WgradPlan c{};
    if (!wgrad_f32_tile(p, wc, t, waves, c)) continue;
    const double cost = c.col_groups * ((double)t / c.wp + 1.5);
    if (nt && cost >= best) continue;
    nt = t;
    best = cost;
    q = c;
  }
  if (!nt) return hipErrorInvalidValue;
  const long long items = (long long)p.G * p.B * q.n_strips * q.n_segs;
  const long long blocks = (long long)q.co_tiles * q.col_groups;
  // slices: up to two workgroups per compute unit, fewer where the additions of their sums would take longer than the
  // items that a slice more saves
  const long long fit = std::max(1ll, std::min(items, (512 + blocks - 1) / blocks));
  const double item_us = 2.5 + nt * q.nq / q.wp * 0.053, sum_us = std::max(0.1, 9.0 * p.Cin * p.Cout / 200e3);
  double least = 0.0;
  for (long long split = fit; split >= 1; split /= 2) {            // halves: 288 workgroups take as long as 512
    const double us = (double)((items + split - 1) / split) * item_us + (double)split * sum_us;
    if (split == fit || us < least) {
      least = us;
      q.split = (int)split;
    }
    if (split == 1) break;
  }
  const long long grid = blocks * q.split;
  if (grid >= (1ll << 31) || items >= (1ll << 31)) return hipErrorInvalidValue;
  auto launch = [&](auto kern) -> hipError_t {
    if (q.total > 64 * 1024) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * waves), q.total, s, p, q);
    return hipGetLastError();
  };
  if (one_tile) {
    if (p.stride == 1) return p.dense ? launch(&wgrad_f32_kernel<1, 1, 1, true, 8>) : launch(&wgrad_f32_kernel<1, 1, 1, false, 8>);
    return p.dense ? launch(&wgrad_f32_kernel<2, 1, 1, true, 8>) : launch(&wgrad_f32_kernel<2, 1, 1, false, 8>);
  }
  auto with_nt = [&](auto s_, auto wc_) -> hipError_t {
    constexpr int S = decltype(s_)::value, WC = decltype(wc_)::value;
    if (p.dense) return nt == 3 ? launch(&wgrad_f32_kernel<S, WC, 3, true, 4>) : launch(&wgrad_f32_kernel<S, WC, 1, true, 4>);
    switch (nt) {
      case 6: return launch(&wgrad_f32_kernel<S, WC, 6, false, 4>);
      case 5: return launch(&wgrad_f32_kernel<S, WC, 5, false, 4>);
      case 3: return launch(&wgrad_f32_kernel<S, WC, 3, false, 4>);
      default: return launch(&wgrad_f32_kernel<S, WC, 1, false, 4>);
    }
  };
  auto with_wc = [&](auto s_) -> hipError_t {
    switch (wc) {
      case 4: return with_nt(s_, std::integral_constant<int, 4>{});
      case 2: return with_nt(s_, std::integral_constant<int, 2>{});
      default: return with_nt(s_, std::integral_constant<int, 1>{});
    }
  };
  return p.stride == 1 ? with_wc(std::integral_constant<int, 1>{}) : with_wc(std::integral_constant<int, 2>{});
}

}  // namespace tac
