// MFMA kernel for bf16 layers of up to 128 input channels (a multiple of 8) without a pool on either side and without recorded membranes, whose output rows
// have 17 to 64 pixels and whose groups have at most 16 frames.
//
// What bounds it: instructions.  A spike word has to become the bf16 aggregates of its pixels (per pixel and 8 channels some 25 vector instructions and four
// accesses to the LDS), and the fragments of a 32 x 32 x 16 product are two more.  The kernel of the shapes in between gave each of its four waves a row of 32
// pixels and 32 or 64 channels, so that a row of 45 took two blocks (30% of them empty), every tile of channels formed all aggregates again, and three LDS rows
// were formed for each output row.  Here
//  - rows are cut into segments of 16 pixels, and a block is any two of them: 45 columns are three segments, not four;
//  - a workgroup is up to 16 waves over rows and tiles of channels, so that aggregates are formed once for up to 128 channels and (rows + 2) LDS rows serve as
//    many rows as the LDS has room for; waves may also only load;
//  - each wave has its own jobs of whole spike words: words to fields across its registers, through a corner of the LDS of its own (no barrier) to one pixel per
//    lane, 16 bytes of aggregates per lane and store.  The next group's first job is on its way during the contraction;
//  - the weights stay in the LDS for the whole sequence.
// The plan (tac_row_plan.h) is the cheapest of some 150 by a fitted estimate.  Before and after: 48 -> 80 channels, 45x45, batch 24, 25 frames in groups of four:
// 103.7 -> 58.5 us; 128 -> 128, 28x28, groups of four with four LIF steps each, batch 16: 60 -> 39 us; 104 -> 103, 43x49, groups of two, batch 24: 557 -> 304 us.
// All sums are in the older kernel's order: the same bits.
#pragma once
#include "tac_row_plan.h"

namespace tac {

struct RowParams {
  MfmaParams m;
  RowPlan q;
  int K_last, n_lif_last;       // frames and LIF steps of a shorter last group (0: none)
  float decay_last;
};

namespace {

// KP: frames per table index (16: two indices of eight).  NNP: blocks of 32 pixels per wave.
template <int KP, int NNP>
__global__ __launch_bounds__(64 * row_max_waves(NNP), row_max_waves(NNP) / 4) void row_kernel(const RowParams dp) {
  constexpr int NCH = row_batch(KP);
  constexpr int kClasses = KP == 16 ? 8 : KP;
  constexpr uint32_t kOutside = 0x80000000u;
  const MfmaParams& p = dp.m;
  const RowPlan& q = dp.q;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int tid = threadIdx.x, lane = tid & 63, threads = blockDim.x, waves = threads >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int Cin = p.Cin, S = p.stride, C8 = Cin >> 3;
  const uint32_t row_tile = blockIdx.x / (uint32_t)q.co_tiles;
  const int co_tile = (int)(blockIdx.x - row_tile * (uint32_t)q.co_tiles);
  const int co_grp = wave / q.pw, px_wave = wave - co_grp * q.pw;
  const int co0 = (co_tile * q.nco + co_grp) * 32;
  // output rows are counted through all samples (fewer than 2^20), or the grid's z is the sample
  const SmallDiv by_ho(p.Ho);
  const int first_row = (int)row_tile * q.tr;
  const int b0 = q.flatten ? by_ho.quot(first_row) : (int)blockIdx.z;
  const int oy0 = q.flatten ? first_row - b0 * p.Ho : first_row;
  const int rows_valid = min(q.tr, (q.flatten ? p.B * p.Ho : p.Ho) - first_row);
  auto sample_of = [&](int rr) { return q.flatten ? by_ho.quot(oy0 + rr) : 0; };        // tile row -> sample - b0
  const size_t plane = (size_t)p.Ho * p.Wo;
  const int wws = (p.W + 31) >> 5;
  const uint32_t in_chan = (uint32_t)(p.H * wws);                      // words per channel
  const size_t t_stride = (size_t)p.B * Cin * in_chan;
  const int n_groups = p.G + (dp.K_last ? 1 : 0);
  uint32_t* const lut = reinterpret_cast<uint32_t*>(lds + q.off_lut);
  float* const bias_lds = reinterpret_cast<float*>(lds + q.off_bias);
  int32_t* const tab = reinterpret_cast<int32_t*>(lds + q.off_tab);
  uint32_t* const pairs = reinterpret_cast<uint32_t*>(lds + q.off_pair);
  u32x2* const pixels = reinterpret_cast<u32x2*>(lds + q.off_px);
  uint8_t* const stage = lds + q.off_stage + wave * q.stage_wave;
  auto col = [&](int xp) { return S == 1 ? xp : (xp & 1) * q.xh + (xp >> 1); };

  // ---- the tile's weights, [channel tile][k-step] fragments of 1 KiB, on their way while the tables are made
  for (int c = 0; c < q.nco; ++c) {
    const int blk = co_tile * q.nco + c, tile = blk / q.nmc_w;
    if (blk * 32 >= p.Cout) break;
    const uint8_t* const src = p.w + ((size_t)tile * q.nks * q.nmc_w + (blk - tile * q.nmc_w)) * 1024 + lane * 16;
    for (int ks = wave; ks < q.nks; ks += waves)
      lds_dma16<1, 0>(src + (size_t)ks * q.nmc_w * 1024, (uint32_t)(uintptr_t)(lds_void_ptr)(lds + q.off_w + (c * q.nks + ks) * 1024));
  }
  // ---- tables
  // words of the tile's rows: byte offset from (frame, first sample, channel), top bit: outside the image
  const int n_pairs = q.lr * wws, n_px = q.lr * p.W;
  const int n0 = min(p.Ho - oy0, q.tr) * S + (3 - S);                  // LDS rows of the tile's first sample
  const SmallDiv by_sample(p.Ho * S + (3 - S)), by_wws(wws), by_w(p.W);
  const int lr_used = (rows_valid - 1) * S + sample_of(rows_valid - 1) * (3 - S) + 3;
  for (int i = tid; i < n_pairs; i += threads) {
    const int row = by_wws.quot(i), word = i - row * wws;
    int bsel = 0, iy = oy0 * S - 1 + row;
    if (row >= n0) {
      const int over = by_sample.quot(row - n0);
      bsel = 1 + over;
      iy = row - n0 - over * by_sample.d - 1;
    }
    const bool inside = row < lr_used && iy >= 0 && iy < p.H;
    pairs[i] = inside ? ((uint32_t)(bsel * Cin) * in_chan + (uint32_t)(iy * wws + word)) * 4u : kOutside;
  }
  // pixels of the tile: byte offset of the class words among the staged ones of a job's first 8 channels, shift of the field (top byte); byte offset in a
  // plane of aggregates
  for (int i = tid; i < n_px; i += threads) {
    const int row = by_w.quot(i), x = i - row * p.W, c = x & (kClasses - 1);
    u32x2 e;
    e[0] = (uint32_t)(((row % q.lrp * wws + (x >> 5)) * q.stage_pair + c * 8) * 4) | (uint32_t)((x & 31) - c) << 24;
    e[1] = (uint32_t)(row * q.wpx + col(x + 1)) * 16;
    pixels[i] = e;
  }
  // the padding columns x = -1 and x = W stay zero
  for (int i = tid; i < C8 * q.lr * 2; i += threads) {
    const int side = i & 1, pl = (i >> 1) / q.lr, r = (i >> 1) - pl * q.lr;
    *reinterpret_cast<u32x4*>(lds + pl * q.plane + (r * q.wpx + col(side ? p.W + 1 : 0)) * 16) = u32x4{0, 0, 0, 0};
  }
  // where a k-step's lane half finds its channels and tap; entries behind the last step are only ever fetched ahead
  for (int i = tid; i < 2 * q.nks + kRowTabPad; i += threads) {
    const int kk = 8 * i, tap = SmallDiv(Cin).quot(kk), cin = kk - tap * Cin;
    const int ky = (tap * 11) >> 5, kx = tap - ky * 3;                 // tap / 3 for the nine taps
    tab[i] = tap < 9 ? (cin >> 3) * q.plane + (ky * q.wpx + col(kx)) * 16 : 0;
  }
  const float scale = 1.0f / (float)(1u << kFixShift);
  // (a shorter last group's weights are the last of a whole group's)
  if constexpr (KP >= 4) frame_tables<KP>(lut, q.lut_set / 4, dp.K_last ? 2 : 1, p.K - dp.K_last, p, tid, threads);
  if (tid < q.nco * 32) bias_lds[tid] = (p.bias && co_tile * q.nco * 32 + tid < p.Cout) ? p.bias[co_tile * q.nco * 32 + tid] : 0.f;
  lds_barrier();

  // ---- the loader.  A job is some blocks of 8 channels on some rows; a wave's jobs are wave, wave + waves, ..  Words to the wave's own corner of the LDS
  // as K-bit fields, [block][word][class][channel], then a pixel per lane.  Consecutive lanes load consecutive words of a channel.
  const int part_pairs = q.lrp * wws;
  const SmallDiv by_pairs(part_pairs);
  uint32_t wd[NCH][KP];
  auto job_units = [&](int job) { return 8 * min(q.cb, C8 - job / q.parts * q.cb) * part_pairs; };
  // Words are loaded through a buffer descriptor, which gives zeros for rows outside the image and frames that a group does not have.
  auto load_job = [&](int g, int job) {
    const int Kg = g == p.G ? dp.K_last : p.K, n_units = job_units(job), cg0 = job / q.parts * q.cb, part = job % q.parts;
    const size_t first = ((size_t)g * p.K * p.B + b0) * Cin * in_chan;
    const size_t bytes = ((size_t)(p.G * p.K + dp.K_last) * t_stride - first) * 4;
    const auto words = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(p.spikes + first), 0, (int)(bytes < 0x7fffffffu ? bytes : 0x7fffffffu), 0x00020000);
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      if (c > 0 && c * 64 >= n_units) break;             // (uniform)
      const int e = min(c * 64 + lane, n_units - 1), ch = by_pairs.quot(e);
      const uint32_t at = pairs[min(part * part_pairs + e - ch * part_pairs, n_pairs - 1)];
      const uint32_t off = at + (uint32_t)(cg0 * 8 + ch) * in_chan * 4u;
#pragma unroll
      for (int j = 0; j < KP; ++j)
        wd[c][j] = __builtin_amdgcn_raw_buffer_load_b32(words, (int)(j < Kg ? off : kOutside), (int)((uint32_t)(j < Kg ? j : 0) * (uint32_t)t_stride * 4u), 0);
    }
  };
  auto store_job = [&](int job) {
    const int n_units = job_units(job);
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      if (c > 0 && c * 64 >= n_units) break;
      const int e = c * 64 + lane, ch = by_pairs.quot(e);
      if constexpr (KP == 16) {
        frames_to_fields<8>(wd[c]);
        frames_to_fields<8>(wd[c] + 8);
      } else {
        frames_to_fields<KP>(wd[c]);
      }
      if (e < n_units) {
        uint32_t* const dst = reinterpret_cast<uint32_t*>(stage) + ((ch >> 3) * part_pairs + e - ch * part_pairs) * q.stage_pair + (ch & 7);
#pragma unroll
        for (int j = 0; j < KP; ++j) dst[j * 8] = wd[c][j];
      }
    }
  };
  const uint32_t two_lo = KP == 2 ? pack_bf16(0.f, (float)p.wq[0] * scale) : 0u;
  const uint32_t two_hi = KP == 2 ? pack_bf16((float)p.wq[1] * scale, (float)(p.wq[0] + p.wq[1]) * scale) : 0u;
  // (one frame left over: its weight is that of a whole group's second)
  const uint32_t two_lo_last = KP == 2 ? pack_bf16(0.f, (float)p.wq[1] * scale) : 0u;
  // a pixel's aggregates of 8 channels from its class words
  auto aggregates = [&](const u32x4 (&cw)[KP == 16 ? 4 : 2], uint32_t sh, uint32_t lo, const uint32_t* tb) {
    u32x4 v;
#pragma unroll
    for (int c2 = 0; c2 < 4; ++c2) {
      const uint32_t w0 = cw[c2 >> 1][2 * (c2 & 1)], w1 = cw[c2 >> 1][2 * (c2 & 1) + 1];
      const uint32_t t0 = __builtin_amdgcn_ubfe(w0, sh, kClasses), t1 = __builtin_amdgcn_ubfe(w1, sh, kClasses);
      if constexpr (KP == 1) {
        v[c2] = __umul24(t0 | t1 << 16, 0x3f80u);                      // one frame: its weight is 1, bf16 0x3f80
      } else if constexpr (KP == 2) {
        v[c2] = two_frame_pair(two_hi, lo, t0 | t1 << 16);
      } else if constexpr (KP == 4) {
        v[c2] = tb[t0 | t1 << 4];
      } else if constexpr (KP == 8) {
        v[c2] = tb[t0] | tb[t1] << 16;
      } else {
        const uint32_t h0 = cw[2 + (c2 >> 1)][2 * (c2 & 1)], h1 = cw[2 + (c2 >> 1)][2 * (c2 & 1) + 1];
        const uint32_t a0 = tb[t0] + tb[256 + __builtin_amdgcn_ubfe(h0, sh, 8)], a1 = tb[t1] + tb[256 + __builtin_amdgcn_ubfe(h1, sh, 8)];
        v[c2] = pack_bf16((float)a0 * scale, (float)a1 * scale);
      }
    }
    return v;
  };
  auto form_job = [&](int g, int job) {
    const bool last = g == p.G;
    const uint32_t* const tb = lut + (last ? q.lut_set / 4 : 0);
    const uint32_t lo = last ? two_lo_last : two_lo;
    const int cg0 = job / q.parts * q.cb, part = job % q.parts, n_c = min(q.cb, C8 - cg0);
    uint8_t* const planes = lds + cg0 * q.plane;
    const int stage_cg = part_pairs * q.stage_pair * 4;
    const int px_end = min((part + 1) * q.lrp, q.lr) * p.W;
    for (int e = part * q.lrp * p.W + lane; e < px_end; e += 64) {
      const u32x2 px = pixels[e];
      const uint8_t* src = stage + (px[0] & 0xffffffu);
      uint8_t* dst = planes + px[1];
      const uint32_t sh = px[0] >> 24;
      // some blocks of channels at a time, so that their trips to the LDS overlap
      auto some = [&]<int N>(std::integral_constant<int, N>) {
        u32x4 cw[N][KP == 16 ? 4 : 2], v[N];
#pragma unroll
        for (int i = 0; i < N; ++i) {
          cw[i][0] = *reinterpret_cast<const u32x4*>(src + i * stage_cg);
          cw[i][1] = *reinterpret_cast<const u32x4*>(src + i * stage_cg + 16);
          if constexpr (KP == 16) {
            cw[i][2] = *reinterpret_cast<const u32x4*>(src + i * stage_cg + 256);
            cw[i][3] = *reinterpret_cast<const u32x4*>(src + i * stage_cg + 272);
          }
        }
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = aggregates(cw[i], sh, lo, tb);
#pragma unroll
        for (int i = 0; i < N; ++i) *reinterpret_cast<u32x4*>(dst + i * q.plane) = v[i];
        src += N * stage_cg;
        dst += N * q.plane;
      };
      constexpr int kMany = KP >= 8 ? 2 : 4;
      int c = 0;
      for (; c + kMany <= n_c; c += kMany) some(std::integral_constant<int, kMany>{});
      for (; c < n_c; ++c) some(std::integral_constant<int, 1>{});
    }
  };
  const bool loader = wave < q.n_jobs;
  if (loader) load_job(0, wave);

  // ---- the lane's pixels: segment 2 block + n / 16 of the tile's rows; membranes are 32-bit byte offsets from the tile's (without a second sample
  // in the tile from its first row)
  const SmallDiv by_spr(q.spr);
  const int v_row = q.flatten ? 0 : oy0;
  LaneGeom lg;
  uint32_t pix[NNP];
#pragma unroll
  for (int np = 0; np < 2; ++np) { lg.ok[np] = false; lg.theta[np] = __builtin_inff(); lg.v_off[np] = 0; }
#pragma unroll
  for (int np = 0; np < NNP; ++np) {
    const int sg = 2 * (px_wave * NNP + np) + (n >> 4), rr0 = by_spr.quot(sg), ox = (sg - rr0 * q.spr) * 16 + (n & 15);
    const bool ok = rr0 < rows_valid && ox < p.Wo;
    const int rr = ok ? rr0 : 0, xx = ok ? ox : 0;
    const int bsel = sample_of(rr), oy = oy0 + rr - bsel * p.Ho;
    lg.ok[np] = ok;
    lg.theta[np] = ok ? p.theta : __builtin_inff();
    lg.v_off[np] = (uint32_t)((((size_t)bsel * p.Cout + 4 * h) * plane + (size_t)(oy - v_row) * p.Wo + xx) * 4);
    pix[np] = (uint32_t)(((rr * S + bsel * (3 - S)) * q.wpx + xx) * 16);
  }
  lg.co_lim = p.Cout - co0 - 4 * h;
  const size_t v_wave = ((size_t)b0 * p.Cout + co0) * plane + (size_t)v_row * p.Wo;
  const bool active = co_grp < q.nco && co0 < p.Cout && by_spr.quot(2 * px_wave * NNP) < rows_valid;      // wave-uniform
  float V[1][NNP][16];
#pragma unroll
  for (int np = 0; np < NNP; ++np)
#pragma unroll
    for (int r = 0; r < 16; ++r) V[0][np][r] = 0.f;
  if (p.v_inout) {
#pragma unroll
    for (int np = 0; np < NNP; ++np)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int c = 8 * (r >> 2) + (r & 3);
        if (lg.ok[np] && c < lg.co_lim)
          V[0][np][r] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(p.v_inout + v_wave) + (size_t)c * plane * 4 + lg.v_off[np]);
      }
  }
  // ---- output words: lane (r << 2) | (hi << 1) | np holds channel 8 (r / 4) + 4 hi + r % 4, pixel block np.  With an even number of segments a row a
  // block is a word, else its halves are halves of words, or a row's last word.
  const int st_np = lane & 1, st_co = co0 + 8 * (lane >> 4) + 4 * ((lane >> 1) & 1) + ((lane >> 2) & 3);
  const int out_words = (p.Wo + 31) >> 5;
  const size_t out_step = (size_t)p.B * p.Cout * p.Ho * out_words;
  const bool even = !(q.spr & 1);
  uint32_t st_at[2];                           // half-words from the step's first
  bool st_ok[2], st_last[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int sg = 2 * (px_wave * NNP + st_np) + s, rr = by_spr.quot(sg), x = sg - rr * q.spr;
    st_ok[s] = st_np < NNP && rr < rows_valid && st_co < p.Cout && (!even || s == 0);
    st_last[s] = x == q.spr - 1;
    const int bsel = sample_of(st_ok[s] ? rr : 0), oy = oy0 + rr - bsel * p.Ho;
    st_at[s] = (uint32_t)((((size_t)(b0 + bsel) * p.Cout + st_co) * p.Ho + oy) * out_words) * 2u + (uint32_t)x;
  }

  const uint8_t* const w_lane = lds + q.off_w + co_grp * q.nks * 1024 + lane * 16;
  const float* const bias_own = bias_lds + co_grp * 32;
  size_t step = 0;
  for (int g = 0; g < n_groups; ++g) {
    const bool last = g == p.G;
    const int n_lif = last ? dp.n_lif_last : p.n_lif;
    const float decay = last ? dp.decay_last : p.decay;
    // ---- 1. aggregates
    for (int job = wave; job < q.n_jobs; job += waves) {
      store_job(job);
      if (job + waves < q.n_jobs) load_job(g, job + waves);
      asm volatile("" ::: "memory");           // the wave's own LDS accesses execute in order; keep the compiler to it too
      form_job(g, job);
      asm volatile("" ::: "memory");
    }
    if (g == 0) lds_dma_wait();                // the weights
    lds_barrier();
    if (loader && g + 1 < n_groups) load_job(g + 1, wave);
    if (active) {
      // ---- 2. contraction: fragments are requested F - 1 steps ahead, table offsets F steps before that
      f32x16 acc[1][NNP];
#pragma unroll
      for (int np = 0; np < NNP; ++np)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][np][r] = bias_own[8 * (r >> 2) + 4 * h + (r & 3)];
      constexpr int F = kRowDepth;
      const int32_t* const tabh = tab + h;
      bf16x8 af[F][NNP], wf[F];
      int32_t off[F];
      auto fetch = [&](int ks, int set) {
        wf[set] = *reinterpret_cast<const bf16x8*>(w_lane + ks * 1024);
#pragma unroll
        for (int np = 0; np < NNP; ++np) af[set][np] = *reinterpret_cast<const bf16x8*>(lds + pix[np] + (uint32_t)off[set]);
        off[set] = tabh[2 * (ks + F)];
      };
#pragma unroll
      for (int d = 0; d < F; ++d) off[d] = tabh[2 * d];
#pragma unroll
      for (int d = 0; d < F - 1; ++d) fetch(d, d);
      auto multiply = [&](int set) {
#pragma unroll
        for (int np = 0; np < NNP; ++np) acc[0][np] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[set], af[set][np], acc[0][np], 0, 0, 0);
      };
      int ks = 0;
      for (; ks + F <= q.nks; ks += F) {
#pragma unroll
        for (int d = 0; d < F; ++d) {
          fetch(ks + d + F - 1, (d + F - 1) % F);
          multiply(d);
        }
      }
#pragma unroll
      for (int d = 0; d < F - 1; ++d)
        if (ks + d < q.nks) multiply(d);
      // ---- 3. LIF steps on Y_k = acc (bias included)
      for (int j = 0; j < n_lif; ++j) {
        uint32_t word[1][2] = {{0u, 0u}};
        lif_step<1, 64, false, NNP>(V, acc, decay, p.theta, lg, word, nullptr, plane);
        uint16_t* const out = reinterpret_cast<uint16_t*>(p.out + (step + j) * out_step);
        const uint32_t w = word[0][0];
        if (even) {
          if (st_ok[0]) *reinterpret_cast<uint32_t*>(out + st_at[0]) = w;
        } else {
#pragma unroll
          for (int s = 0; s < 2; ++s) {
            const uint32_t half = s ? w >> 16 : w & 0xffffu;
            if (st_ok[s]) {
              if (st_last[s]) *reinterpret_cast<uint32_t*>(out + st_at[s]) = half;       // the row's last word: its upper half is zero
              else out[st_at[s]] = (uint16_t)half;
            }
          }
        }
      }
    }
    step += n_lif;
    lds_barrier();                             // the group's fragments have been read
  }
  if (p.v_inout) {
#pragma unroll
    for (int np = 0; np < NNP; ++np)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int c = 8 * (r >> 2) + (r & 3);
        if (active && lg.ok[np] && c < lg.co_lim)
          *reinterpret_cast<float*>(reinterpret_cast<char*>(p.v_inout + v_wave) + (size_t)c * plane * 4 + lg.v_off[np]) = V[0][np][r];
      }
  }
}

template <int KP, int NNP>
hipError_t row_launch_t(const RowParams& p, hipStream_t s) {
  const auto kern = &row_kernel<KP, NNP>;
  if (p.q.total > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kRowLds);
    if (e != hipSuccess) return e;
  }
  const dim3 grid((unsigned)p.q.row_tiles * (unsigned)p.q.co_tiles, 1, p.q.flatten ? 1 : p.m.B);
  hipLaunchKernelGGL(kern, grid, dim3(64 * p.q.waves), p.q.total, s, p);
  return hipGetLastError();
}

template <int NNP>
hipError_t row_launch_kp(const RowParams& p, hipStream_t s) {
  switch (p.q.kp) {
    case 1: return row_launch_t<1, NNP>(p, s);
    case 2: return row_launch_t<2, NNP>(p, s);
    case 4: return row_launch_t<4, NNP>(p, s);
    case 8: return row_launch_t<8, NNP>(p, s);
    default: return row_launch_t<16, NNP>(p, s);
  }
}

}  // namespace

}  // namespace tac
