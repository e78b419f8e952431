// Weight and bias gradient of the conv-LIF layer in fp32 on the matrix cores (v_mfma_f32_32x32x2_f32: operands, products
// and sums in fp32), for every layer that the bf16 kernel does not take: fp32 layers, stride 2, real-valued frames, the
// mean pool on load, channel counts and widths of any kind.
//   dW[co][col] = sum over groups k, samples b, output pixels of dY_k[co][pixel] * A_k[ci][pixel's input under the tap],
// col = 9 ci + tap being the place of (ci, ky, kx) in dW[co], so that the 32 columns of an MFMA tile are 32 consecutive
// floats of dW whatever the number of input channels (one input channel fills 9 columns of a tile, 32 channels 9 tiles),
// and the atomics that combine the workgroups' sums hit consecutive addresses.
//
// Workgroup = 32 output channels x NT column tiles x a slice of the list of items (some (group, sample) pairs of a small
// image, or a strip of output rows and a segment of them).  Per item the dY values go to LDS as [channel][pixel] (rows
// padded to four pixels, requested one item ahead) and the aggregates of the columns' input channels as [channel][pair]
// [row][column], rebuilt from the packed words (a thread per 16 pixels).  An operand of four MFMAs is then one 16-byte read
// of dY (four pixels per lane half) and four 4-byte reads of the aggregates under the lane's own tap.  The eight waves share
// the pixels of the item.
//
// How the sums are cut decides their error, and with it the tile.  A one-signed sum of n terms that are added one after the
// other is off by about 2.5e-8 sqrt(n / 3) of itself; c such sums added up are off by 1 / sqrt(c) of that.
//   - An MFMA chain ends after some items and goes into a second set of sums: both chains have about the root of the length.
//   - The eight waves' sums meet in LDS.
//   - What is left is the chain of a dW element's additions in memory, one per slice.  Small tiles make many blocks and so
//     few slices: one of the compute units' 256 workgroups takes 32 channels x 32 to 160 columns.
#include <algorithm>
#include <cmath>
#include "tac_mfma_common.h"

namespace tac {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kWaves = 8, kThreads = 64 * kWaves;
constexpr int kChans = 32 / kWaves;     // output channels whose dY a wave brings to LDS
constexpr int kAhead = 2;               // units of 16 pixels whose first frames a thread requests one item ahead

struct WgradPlan {
  int co_tiles, col_groups, split;
  int flush;                      // items after which an MFMA chain ends
  int n_pairs, rows, xw;          // an item: (group, sample) pairs x output rows x columns; one pair unless a whole image fits
  int pair_tiles, n_strips, n_segs;
  int npx, nq, pxs;               // pixels (padded rows) and quads of an item, dwords per channel of dY in LDS
  int rows_in, cw, cp;            // aggregate rows per pair, dwords per row and per channel
  int n_ch;                       // input channels of a column group, at most
  int off_a, off_q, off_w, total; // LDS bytes
};

__device__ __forceinline__ int group_frames(const BackwardParams& p, int k) {
  return (k == p.G - 1 && p.K_last) ? p.K_last : p.K;
}

// Real-valued frames with one column tile: two workgroups per compute unit fill each other's waits for the frames (2 -> 128 at
// 64 x 64, B = 16, 4 groups of 4: 132 us a backward call, 149 with one); frames of bits ask for their words one item ahead.
__host__ __device__ constexpr bool wgrad_two_per_cu(int nt, bool dense) { return dense && nt == 1; }
__host__ __device__ constexpr int wgrad_resident(int nt, bool dense) { return wgrad_two_per_cu(nt, dense) ? 512 : 256; }
// blocks of 64 pixels of an item (dY values in registers per thread: times four channels)
__host__ __device__ constexpr int wgrad_m(int nt, bool dense) { return wgrad_two_per_cu(nt, dense) || nt > 3 ? 4 : 8; }

// DENSE: real-valued frames.
template <int S, int NT, bool DENSE>
__global__ __launch_bounds__(kThreads, wgrad_two_per_cu(NT, DENSE) ? 4 : 2) void wgrad_f32_kernel(const BackwardParams p, const WgradPlan q) {
  constexpr int M = wgrad_m(NT, DENSE);
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  float* const dyl = reinterpret_cast<float*>(lds);
  float* const agg = reinterpret_cast<float*>(lds + q.off_a);
  int32_t* const qoff = reinterpret_cast<int32_t*>(lds + q.off_q);
  float* const wl = reinterpret_cast<float*>(lds + q.off_w);           // frame weights: a whole group's, the last group's
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  uint32_t t0 = blockIdx.x;
  const int slice = (int)(t0 % (uint32_t)q.split); t0 /= (uint32_t)q.split;
  const int co0 = (int)(t0 % (uint32_t)q.co_tiles) * 32;
  const int col_first = (int)(t0 / (uint32_t)q.co_tiles) * (NT * 32);
  const int n_cols = 9 * p.Cin;
  const int ci_first = col_first / 9;
  const int n_ch = (min(col_first + NT * 32, n_cols) - 1) / 9 - ci_first + 1;
  const size_t plane = (size_t)p.Ho * p.Wo;
  const int n_rows = q.n_pairs * q.rows_in;              // aggregate rows per channel

  // columns of the lane: dword offset of (channel, ky, kx) in the aggregates
  int coff[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    const int col = col_first + n + 32 * t;
    const int ci = col / 9, tap = col - 9 * ci, ky = (tap * 11) >> 5, kx = tap - 3 * ky;
    coff[t] = col < n_cols ? (ci - ci_first) * q.cp + ky * q.cw + kx : 0;
  }
  // quads of the item: (pair, row, four pixels) -> dword offset of the first one's input under tap (0, 0)
  const int quads_row = q.xw >> 2;
  for (int i = tid; i < q.nq + 2; i += kThreads) {
    const int line = i / quads_row, xq = i - line * quads_row, pr = line / q.rows, yl = line - pr * q.rows;
    qoff[i] = i < q.nq ? (pr * q.rows_in + yl * S) * q.cw + xq * 4 * S : 0;
  }
  if (tid < 2 * TAC_MAX_K) {
    const int j = tid & (TAC_MAX_K - 1);
    wl[tid] = tid < TAC_MAX_K ? (j < p.K ? p.wj[j] : 0.f) : (j < p.K_last ? p.wj_last[j] : 0.f);
  }
  // the quad behind an odd number of them, and everything an aggregate is never written to, is zero
  if (tid < 32) *reinterpret_cast<f32x4*>(dyl + tid * q.pxs + q.npx) = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int i = tid; i < q.n_ch * q.cp; i += kThreads) agg[i] = 0.f;

  // dY: wave w takes the channels w, w + 8, ..; lane + 64 m is a pixel of the item
  constexpr int kNoPair = 1 << 14;
  int pos[M];                                            // pair << 16 | row << 8 | column
#pragma unroll
  for (int m = 0; m < M; ++m) {
    const int px = lane + 64 * m, line = px / q.xw, pr = line / q.rows;
    pos[m] = (px < q.npx ? pr : kNoPair) << 16 | (line - pr * q.rows) << 8 | (px - line * q.xw);
  }
  float wd[kChans][M];
  const int all_pairs = p.G * p.B;
  const int items = q.pair_tiles * q.n_strips * q.n_segs;
  // the items of the slice are `split` apart: the step is taken apart once and added with carries
  struct Index { int seg, strip, pt; };
  auto take_apart = [&](int it) {
    Index x;
    x.seg = it % q.n_segs; it /= q.n_segs;
    x.strip = it % q.n_strips;
    x.pt = it / q.n_strips;
    return x;
  };
  const Index by = take_apart(q.split);
  auto advance = [&](Index& x) {
    x.seg += by.seg; x.strip += by.strip; x.pt += by.pt;
    if (x.seg >= q.n_segs) { x.seg -= q.n_segs; ++x.strip; }
    if (x.strip >= q.n_strips) { x.strip -= q.n_strips; ++x.pt; }
  };
  struct Where { int pair0, pairs, k, b, y0, x0; };     // k, b: of the first pair
  auto where = [&](const Index& x) {
    const int pair0 = x.pt * q.n_pairs, k = pair0 / p.B;
    return Where{pair0, min(q.n_pairs, all_pairs - pair0), k, pair0 - k * p.B, x.strip * q.rows, x.seg * q.xw};
  };
  const uint32_t pair_floats = (uint32_t)(p.Cout * plane);               // (used with several pairs per item only)
  auto request = [&](const Where& w) {
    uint32_t off[M];
#pragma unroll
    for (int m = 0; m < M; ++m)
      off[m] = (uint32_t)min(pos[m] >> 16, w.pairs - 1) * pair_floats +
               (uint32_t)(min(w.y0 + (pos[m] >> 8 & 255), p.Ho - 1) * p.Wo + min(w.x0 + (pos[m] & 255), p.Wo - 1));
    const float* const src = p.grad_y + (size_t)w.pair0 * p.Cout * plane;
#pragma unroll
    for (int c = 0; c < kChans; ++c) {
      const float* const chan = src + (size_t)min(co0 + wave + kWaves * c, p.Cout - 1) * plane;     // (rows beyond Cout are not stored)
#pragma unroll
      for (int m = 0; m < M; ++m) wd[c][m] = chan[off[m]];
    }
  };

  const float inv_rows_in = 1.0f / (float)q.rows_in, inv_rows = 1.0f / (float)n_rows, inv_b = 1.0f / (float)p.B;
  // a line of the item's aggregates: channel, (group, sample) pair and row, and where its frames and weights are
  struct Line { int ch, iy, k, b, Kg; bool inside; const float* wj; };
  auto take_line = [&](const Where& w, int line) {
    Line l;
    l.ch = small_div(line, inv_rows);
    int rr = line - l.ch * n_rows, pr = 0;
    l.k = w.k;
    l.b = w.b;
    if (q.n_pairs > 1) {
      pr = small_div(rr, inv_rows_in);
      rr -= pr * q.rows_in;
      const int beyond = w.b + min(pr, w.pairs - 1), more = small_div(beyond, inv_b);
      l.k += more;
      l.b = beyond - more * p.B;
    }
    l.iy = w.y0 * S - 1 + rr;
    l.inside = pr < w.pairs && l.iy >= 0 && l.iy < p.H;
    l.Kg = group_frames(p, l.k);
    l.wj = wl + (l.Kg == p.K ? 0 : TAC_MAX_K);
    l.iy = min(max(l.iy, 0), p.H - 1);
    return l;
  };
  const int n_lines = n_ch * n_rows;
  const float inv_lines = 1.0f / (float)n_lines;
  // A unit is 16 pixels of a line: half a stored word, or with a pool on load the whole word.  `mask`: the bits of its word that
  // are pixels of the image.
  const int hs = p.pool2 ? 2 * p.H : p.H;
  const size_t fs = (size_t)p.B * p.Cin * hs * p.Wwi;    // words per frame
  struct Unit { Line l; int line, unit; uint32_t mask; const uint32_t* src; };
  auto first_unit = [&](const Where& w) { return (w.x0 * S - 1) >> 4; };
  auto units_of = [&](const Where& w) { return ((w.x0 * S + q.cw - 2) >> 4) - first_unit(w) + 1; };
  auto take_unit = [&](const Where& w, int e) {
    Unit x;
    const int nth = small_div(e, inv_lines);             // consecutive threads take consecutive lines: an odd number of dwords apart
    x.line = e - nth * n_lines;
    x.unit = first_unit(w) + nth;
    x.l = take_line(w, x.line);
    const int word = p.pool2 ? x.unit : x.unit >> 1;
    const int n_px = x.l.inside && x.unit >= 0 ? min(max(p.W - 16 * x.unit, 0), 16) : 0;
    x.mask = p.pool2 ? (n_px == 16 ? 0xffffffffu : (1u << 2 * n_px) - 1u) : ((1u << n_px) - 1u) << (16 * (x.unit & 1));
    x.src = p.spikes + ((((size_t)x.l.k * p.K * p.B + x.l.b) * p.Cin + ci_first + x.l.ch) * hs + (p.pool2 ? 2 : 1) * x.l.iy) * p.Wwi +
            min(max(word, 0), p.Wwi - 1);
    return x;
  };
  // four frames of a unit (with a pool on load both rows), from the first ones on
  auto load_frames = [&](const Unit& x, int j, uint32_t (&f)[4], uint32_t (&f1)[4]) {
#pragma unroll
    for (int u = 0; u < 4; ++u) f[u] = f1[u] = x.src[(size_t)min(j + u, x.l.Kg - 1) * fs];
    if (p.pool2) {
#pragma unroll
      for (int u = 0; u < 4; ++u) f1[u] = x.src[(size_t)min(j + u, x.l.Kg - 1) * fs + p.Wwi];
    }
  };
  constexpr bool AHEAD = !DENSE && NT <= 3;              // (two workgroups of one tile fill each other's waits)
  uint32_t pf[AHEAD ? kAhead : 1][4], pf1[AHEAD ? kAhead : 1][4];
  auto request_units = [&](const Where& w) {
    if constexpr (AHEAD) {
      const int n_units = n_lines * units_of(w);
#pragma unroll
      for (int a = 0; a < kAhead; ++a) {
        if (a > 0 && a * kThreads >= n_units) break;     // (uniform)
        load_frames(take_unit(w, min(tid + a * kThreads, n_units - 1)), 0, pf[a], pf1[a]);
      }
    }
  };
  f32x16 acc[NT], sum[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[t][r] = sum[t][r] = 0.f;
  double bias = 0.0;

  Index ahead = take_apart(min(slice, items - 1));
  Where w = where(ahead);
  if (slice < items) {
    request(w);
    request_units(w);
  }
  int chain = 0;
  for (int it = slice; it < items; it += q.split) {
    __syncthreads();                                     // the item before has been read
    // ---- dY to LDS, zeros where the item has no pixel
#pragma unroll
    for (int m = 0; m < M; ++m) {
      const bool inside = (pos[m] >> 16) < w.pairs && w.y0 + (pos[m] >> 8 & 255) < p.Ho && w.x0 + (pos[m] & 255) < p.Wo;
      if (lane + 64 * m < q.npx) {
        uint32_t at = (uint32_t)(wave * q.pxs + lane + 64 * m);
#pragma unroll
        for (int c = 0; c < kChans; ++c) {
          asm volatile("" : "+v"(at));                   // one address register, not one per channel kept across items
          dyl[at] = inside ? wd[c][m] : 0.f;
          at += kWaves * q.pxs;
        }
      }
    }
    // ---- aggregates of rows y0 S - 1 .., columns x0 S - 1 ..
    const int ix0 = w.x0 * S - 1;
    const int k_max = q.n_pairs == 1 ? group_frames(p, w.k) : p.K;
    if constexpr (DENSE) {
      // real-valued frames [T][B][Cin][H][W] (the continuous-valued first layer, Sec. 4.2)
      const size_t frame = (size_t)p.B * p.Cin * p.H * p.W;
      const float inv_cw = 1.0f / (float)q.cw;
      for (int e = tid; e < n_lines * q.cw; e += kThreads) {
        const int line = small_div(e, inv_cw), c = e - line * q.cw;
        const Line l = take_line(w, line);
        const int ix = ix0 + c;
        const float* const src = reinterpret_cast<const float*>(p.spikes) +
                                 (((size_t)l.k * p.K * p.B + l.b) * p.Cin + ci_first + l.ch) * p.H * p.W + (size_t)l.iy * p.W +
                                 min(max(ix, 0), p.W - 1);
        float a = 0.f;
        for (int j = 0; j < l.Kg; j += 4) {
          float f[4];
#pragma unroll
          for (int u = 0; u < 4; ++u) f[u] = src[(size_t)min(j + u, l.Kg - 1) * frame];
#pragma unroll
          for (int u = 0; u < 4; ++u)
            if (j + u < l.Kg) a = fmaf(l.wj[j + u], f[u], a);
        }
        agg[line * q.cw + c] = l.inside && ix >= 0 && ix < p.W ? a : 0.f;
      }
    } else {
      auto build = [&](const Unit& x, uint32_t (&f)[4], uint32_t (&f1)[4], bool loaded) {
        float a[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) a[i] = 0.f;
        for (int j = 0; j < k_max; j += 4) {
          if (!loaded || j > 0) load_frames(x, j, f, f1);
#pragma unroll
          for (int u = 0; u < 4; ++u) {
            if (j + u >= k_max) break;                   // (uniform; frames beyond a pair's own group weigh nothing)
            const float wt = x.l.wj[j + u];
            const uint32_t r0 = f[u] & x.mask, r1 = f1[u] & x.mask;
            if (p.pool2 == 1) {
              // mean of the four bits: counts of 0..4 in nibbles, pixel i of the word in nibble i / 2 of lo (even) or hi
              const uint32_t t = (r0 & 0x55555555u) + ((r0 >> 1) & 0x55555555u), b = (r1 & 0x55555555u) + ((r1 >> 1) & 0x55555555u);
              const uint32_t lo = (t & 0x33333333u) + (b & 0x33333333u), hi = ((t >> 2) & 0x33333333u) + ((b >> 2) & 0x33333333u);
#pragma unroll
              for (int i = 0; i < 16; ++i)
                a[i] += (0.25f * (float)__builtin_amdgcn_ubfe(i & 1 ? hi : lo, 4 * (i >> 1), 4)) * wt;
            } else {
              // pixel i at bit i, or with the max pool the OR of its block at bit 2 i
              uint32_t o = r0 | r1;
              o = p.pool2 ? pool_pairs(o) : o >> (16 * (x.unit & 1));
#pragma unroll
              for (int i = 0; i < 16; ++i) a[i] += (o >> i) & 1u ? wt : 0.f;
            }
            __builtin_amdgcn_sched_barrier(0);           // a frame after the other: the accumulators leave few registers
          }
        }
        float* const dst = agg + x.line * q.cw;
        const int c0 = x.unit * 16 - ix0;                // column of the unit's first pixel
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (c0 + i >= 0 && c0 + i < q.cw) dst[c0 + i] = a[i];
      };
      const int n_units = n_lines * units_of(w);
      int e = tid;
      if constexpr (AHEAD) {
#pragma unroll
        for (int a = 0; a < kAhead; ++a) {
          if (a > 0 && a * kThreads >= n_units) break;
          if (e < n_units) build(take_unit(w, e), pf[a], pf1[a], true);
          e += kThreads;
        }
      }
      for (; e < n_units; e += kThreads) {
        uint32_t f[4], f1[4];
        build(take_unit(w, e), f, f1, false);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    advance(ahead);
    const Where next = where(ahead);
    if (it + q.split < items) {
      request(next);
      request_units(next);
    }
    __syncthreads();
    // ---- MFMAs: a step is two quads, one per lane half.  Pixels that only fill a quad have dY = 0; where their aggregates
    //      may be infinite (real-valued frames) those are replaced as well.
    const float* const dy_lane = dyl + n * q.pxs;
    for (int i = wave; 2 * i < q.nq; i += kWaves) {
      const int quad = 2 * i + h;
      const f32x4 g = *reinterpret_cast<const f32x4*>(dy_lane + 4 * quad);
      const float* const a_quad = agg + qoff[quad];
      int real = 4;                                      // of the quad's pixels
      if constexpr (DENSE) {
        const int line = quad / quads_row, pr = line / q.rows;
        real = pr < w.pairs && w.y0 + line - pr * q.rows < p.Ho ? p.Wo - w.x0 - 4 * (quad - line * quads_row) : 0;
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
      if (col_first == 0) bias += (double)((g[0] + g[1]) + (g[2] + g[3]));
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        if (t + 1 < NT) fetch(t + 1);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(g[u], a[t & 1][u], acc[t], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (++chain == q.flush) {
      chain = 0;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          sum[t][r] += acc[t][r];
          acc[t][r] = 0.f;
        }
    }
    w = next;
  }
  // Register r of acc[t] on lane (n, h): output channel 8 (r / 4) + 4 h + r % 4, column n of tile t.  The waves' sums are
  // added through LDS first: one address takes an addition about every 0.1 us, and the chip some 200 a nanosecond.
  float* const red = reinterpret_cast<float*>(lds);      // [wave][register][lane]
#pragma unroll
  for (int t = 0; t < NT; ++t) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) red[(wave * 16 + r) * 64 + lane] = sum[t][r] + acc[t][r];
    __syncthreads();
    for (int r = wave; r < 16; r += kWaves) {
      float v = 0.f;
      for (int x = 0; x < kWaves; ++x) v += red[(x * 16 + r) * 64 + lane];
      const int co = co0 + 8 * (r >> 2) + 4 * h + (r & 3), col = col_first + n + 32 * t;
      if (co < p.Cout && col < n_cols) atomicAdd(p.grad_w + (size_t)co * n_cols + col, v);
    }
  }
  if (p.grad_bias && col_first == 0) {
    double* const red_b = reinterpret_cast<double*>(lds);
    __syncthreads();
    red_b[wave * 64 + lane] = bias;
    __syncthreads();
    if (tid < 32 && co0 + tid < p.Cout) {
      double v = 0.0;
      for (int x = 0; x < kWaves; ++x) v += red_b[x * 64 + tid] + red_b[x * 64 + 32 + tid];
      atomicAdd(p.grad_bias + co0 + tid, (float)v);
    }
  }
}

bool wgrad_f32_tile(const BackwardParams& p, int nt, WgradPlan& q) {
  const int S = p.stride, tiles = (9 * p.Cin + 31) / 32;
  q.co_tiles = (p.Cout + 31) / 32;
  q.col_groups = (tiles + nt - 1) / nt;
  q.n_ch = std::min(p.Cin, (nt * 32 + 8) / 9 + 1);
  const int npx_max = 64 * wgrad_m(nt, p.dense);
  const int limit = (wgrad_two_per_cu(nt, p.dense) ? 80 : 150) * 1024;
  const int all_pairs = p.G * p.B;
  auto fits = [&]() {
    q.pair_tiles = (all_pairs + q.n_pairs - 1) / q.n_pairs;
    q.npx = q.n_pairs * q.rows * q.xw;
    q.nq = q.npx / 4;
    q.pxs = q.npx + 4;
    if (q.pxs / 4 % 2 == 0) q.pxs += 4;                  // an odd number of 16-byte units: 16 channels cover the banks
    q.rows_in = (q.rows - 1) * S + 3;
    q.cp = q.n_pairs * q.rows_in * q.cw;
    q.off_a = 32 * q.pxs * 4;
    q.off_q = (q.off_a + q.n_ch * q.cp * 4 + 15) & ~15;
    q.off_w = q.off_q + (q.nq + 2) * 4;
    q.total = std::max(q.off_w + 2 * TAC_MAX_K * 4, kWaves * 16 * 64 * 4);
    return q.npx <= npx_max && q.total <= limit;
  };
  for (q.xw = std::min(64, (p.Wo + 3) / 4 * 4); q.xw >= 4; q.xw = (q.xw / 2 + 3) / 4 * 4) {
    q.n_segs = (p.Wo + q.xw - 1) / q.xw;
    q.cw = ((q.xw - 1) * S + 3) | 1;                     // odd: rows of a channel start in different LDS banks
    for (q.rows = std::max(1, std::min(p.Ho, npx_max / q.xw)); q.rows >= 1; --q.rows) {
      q.n_strips = (p.Ho + q.rows - 1) / q.rows;
      q.rows = (p.Ho + q.n_strips - 1) / q.n_strips;     // strips of the same height, as far as it goes
      q.n_pairs = 1;
      if (!fits()) continue;
      if (q.n_strips == 1 && q.n_segs == 1) {
        // several pairs, with 32-bit offsets between them, while every slice gets an item
        const int slices = std::max(1, wgrad_resident(nt, p.dense) / (q.co_tiles * q.col_groups));
        for (q.n_pairs = std::min((all_pairs + slices - 1) / slices, npx_max / q.npx); q.n_pairs > 1; --q.n_pairs)
          if ((long long)q.n_pairs * p.Cout * p.Ho * p.Wo < (1ll << 31) && fits()) break;
        fits();
      }
      return true;
    }
    if (q.xw == 4) break;
  }
  return false;
}

}  // namespace

// Which tile and how many slices: the estimated time, among those that keep a dW element's chain of additions in memory
// short (at most 48 slices, more only where dW has so few tiles that the chip would stand idle).
//   A workgroup's item takes about 2 us plus, per 512 pixels, 1 us and 2.25 us per tile; a round of workgroups 5 us more; a
//   slice's additions 1 us per 200 k elements, 0.1 us at least.  (128 -> 128 at 64 x 64: 5.4, 7.5 and 9.7 us an item of 512 pixels
//   for one, two and three tiles, 8.4 us one of 256 for five.)
// Backward calls without input gradient in us, and the error of dW against 64-bit sums for dY of both signs: the vector kernel;
// larger tiles in four waves with one chain per slice; this:
//   128 -> 128, 8 groups at 64 x 64, B = 64     41200 5.4e-7;  11700 11e-7;  9060 2.1e-7
//   32 -> 64, 7 groups at 14 x 14, B = 128       1290 1.6e-7;    161 4.1e-7;  169 1.4e-7
//   1 -> 32, 7 groups at 28 x 28, B = 128         192 5.4e-7;    118 3.8e-7;  101 3.0e-7
//   128 -> 128, 4 groups at 8 x 8, B = 16         375 1.0e-7;     55 1.5e-7;   40 1.0e-7
//   8 -> 32, 18 groups at 59 x 59, B = 17         460 2.0e-7;    184 4.0e-7;  198 2.5e-7
//   16 -> 16, 10 groups at 100 x 100, B = 16      512 2.0e-7;    343 4.2e-7;  400 2.4e-7
hipError_t backward_wgrad_f32_launch(const BackwardParams& p, hipStream_t s) {
  WgradPlan q{};
  int nt = 0;
  double least = 0.0;
  const double sum_us = std::max(0.1, 9.0 * p.Cin * p.Cout / 200e3);
  for (int t : {1, 2, 3, 5}) {
    if (p.dense && t != 1 && t != 3) continue;           // (real-valued frames: first layers have few columns)
    WgradPlan c{};
    if (!wgrad_f32_tile(p, t, c)) continue;
    const long long items = (long long)c.pair_tiles * c.n_strips * c.n_segs;
    const long long blocks = (long long)c.co_tiles * c.col_groups;
    const int resident = wgrad_resident(t, p.dense);
    const long long tiles = (long long)c.co_tiles * ((9 * p.Cin + 31) / 32);
    const long long most = std::min(items, std::max(48ll, 640 / tiles));
    const double item_us = 2.0 + c.npx / 512.0 * (1.0 + 2.25 * t);
    // whole rounds of resident workgroups, or halves and quarters of one
    for (int sixteenths : {1, 2, 4, 8, 16, 32, 48, 64}) {
      const long long split = std::max(1ll, std::min(sixteenths * resident / 16 / blocks, most));
      const double rounds = (double)((blocks * split + resident - 1) / resident);
      const double us = rounds * (5.0 + (double)((items + split - 1) / split) * item_us) + (double)split * sum_us;
      if (nt && us >= least) continue;
      nt = t;
      least = us;
      q = c;
      q.split = (int)split;
    }
  }
  if (!nt) return hipErrorInvalidValue;
  const long long items = (long long)q.pair_tiles * q.n_strips * q.n_segs;
  const long long grid = (long long)q.co_tiles * q.col_groups * q.split;
  if (grid >= (1ll << 31) || items >= (1ll << 31)) return hipErrorInvalidValue;
  // the chain of a wave's MFMAs (four per 16 quads of an item) about as long as the chain of their sums
  q.flush = std::max(2, (int)(std::sqrt((double)items / q.split * 4.0 / q.nq) + 0.5));
  auto launch = [&](auto kern) -> hipError_t {
    if (q.total > 64 * 1024) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 150 * 1024);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(kThreads), q.total, s, p, q);
    return hipGetLastError();
  };
  auto with_s = [&](auto s_) -> hipError_t {
    constexpr int S = decltype(s_)::value;
    if (p.dense) return nt == 3 ? launch(&wgrad_f32_kernel<S, 3, true>) : launch(&wgrad_f32_kernel<S, 1, true>);
    switch (nt) {
      case 5: return launch(&wgrad_f32_kernel<S, 5, false>);
      case 3: return launch(&wgrad_f32_kernel<S, 3, false>);
      case 2: return launch(&wgrad_f32_kernel<S, 2, false>);
      default: return launch(&wgrad_f32_kernel<S, 1, false>);
    }
  };
  return p.stride == 1 ? with_s(std::integral_constant<int, 1>{}) : with_s(std::integral_constant<int, 2>{});
}

}  // namespace tac
