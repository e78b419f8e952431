// MFMA kernel for bf16 layers of 16 to 256 input channels (a multiple of 8), without a pool on load, whose output rows have at most 64 pixels and whose
// groups have at most 16 frames, where the other matrix-core kernels do not reach: more than 128 input channels at widths other than 32 and 64, or
// rows of aggregates too wide to share the LDS with a tile's weights (the last layers of the strided stack on frames of 64 x 64 .. 100 x 100, or of 48
// channels on 128 x 128).  They were the vector kernel's, at 1 TFLOP/s.  It reads that kernel's prepared weights.
//
// Such layers have few pixels, and what bounds them is the chain of steps that follow each other for every group of frames: load words, form
// aggregates, multiply, add up, step the neurons, store.  The membrane is the only thing that one group hands to the next, so a
// workgroup takes up to four groups at a time through all of it but the LIF steps (GB groups x PB pixel blocks = four sets of sums):
//   1. aggregates (Eq. 2) of GB groups into LDS, [group][8 channels][row][column][8].  A thread loads the K frame words of some channels of a
//      stretch of one row, turns them into K-bit fields (frames_to_fields) and goes along the pixels: one bit field per channel is the
//      index of its aggregate in a table (K = 2: of a byte permutation); nothing is staged.  The words of two turns of the threads are in hand,
//      through the end of a round into the next one.
//   2. the eight waves share the contraction of every block: a wave has an eighth of the k-steps, whose weights it keeps in
//      registers for the whole call (KS of them), the partial sums meet in LDS (over the aggregates) and are added in a fixed tree, whatever the
//      batch; every wave gets two of the 16 result registers of each block
//   3. bias, the LIF steps of the groups in their order, packed stores of up to four steps at a time
// Workgroup = 32 output channels x PB blocks of 32 pixels (a word of an output row, or several rows of 16, 8, 4 or 2 lanes, counted through the
// rows of all samples).  Forming the aggregates takes half the time (vector operations, and once per 32 output channels), the LIF steps and stores a quarter.
// us a call, vector kernel and this one: 192 -> 192 stride 2 at 12 x 12, B = 2, 24 frames, TAC K = 2 5990 / 73; at 10 x 10, B = 6, TAC-TP K = 4
// 2670 / 44; 256 -> 256 stride 2 at 13 x 13, B = 24, 8 single frames 5370 / 65; 192 -> 192 stride 2 at 32 x 32, B = 13, K = 8 2860 / 92; 96 -> 96 stride 2 at
// 64 x 64, B = 13, K = 8 2130 / 96.  (The words staged as K-bit fields by whole waves, as the kernel in between has them: 100 / 57 / 109 / 127 / 98.)
#pragma once
#include "tac_deep_plan.h"

namespace tac {

struct DeepParams {
  MfmaParams m;
  DeepPlan q;
  int K_last, n_lif_last;       // frames and LIF steps of a shorter last group (0: none)
  float decay_last;
};

hipError_t deep_launch_plain(const DeepParams& p, hipStream_t s);
hipError_t deep_launch_trace(const DeepParams& p, hipStream_t s);

namespace {

// KP: frames per table index (16: two indices of eight).  KS: k-steps of a wave at most.  GB groups x PB pixel blocks.
template <int KP, bool TRACE, int KS, int GB, int PB>
__global__ __launch_bounds__(kDeepThreads, 2) void deep_kernel(const DeepParams dp) {
  static_assert(GB * PB == kDeepSets);
  constexpr int UC = deep_unit_channels(KP, KS);           // channels of a unit
  constexpr uint32_t kOutside = 0x80000000u;
  const MfmaParams& p = dp.m;
  const DeepPlan& q = dp.q;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int Cin = p.Cin, S = p.stride;
  const uint32_t row_tile = blockIdx.x / (uint32_t)q.co_tiles;
  const int co_tile = (int)(blockIdx.x - row_tile * (uint32_t)q.co_tiles);
  const int co0 = co_tile * 32;
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
  u32x2* const pairs = reinterpret_cast<u32x2*>(lds + q.off_pair);
  auto col = [&](int xp) { return S == 1 ? xp : (xp & 1) * q.xh + (xp >> 1); };

  // ---- weights of the wave's eighth of the k-steps (a step behind its last is loaded and not multiplied)
  const int k0 = (q.nks * wave) >> 3, n_k = ((q.nks * (wave + 1)) >> 3) - k0;
  bf16x8 w_own[KS];
  {
    // the vector kernel's layout: [cin][tap][cout padded to 32] fp32, rounded to bf16; slots beyond 9 Cin are zero
    const SmallDiv by_cin(Cin);
    const int cp = q.co_tiles * 32;
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      const int kk = 16 * min(k0 + k, q.nks - 1) + 8 * h, tap = by_cin.quot(kk), cin = kk - tap * Cin;
      const float* const src = reinterpret_cast<const float*>(p.w) + (uint32_t)(tap < 9 ? cin * 9 + tap : 0) * (uint32_t)cp + co0 + n;
      float f[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) f[i] = src[(uint32_t)(i * 9 * cp)];
      u32x4 v;
#pragma unroll
      for (int i = 0; i < 4; ++i) v[i] = tap < 9 ? pack_bf16(f[2 * i], f[2 * i + 1]) : 0u;
      w_own[k] = __builtin_bit_cast(bf16x8, v);
    }
  }

  // ---- tables
  // rows and segments of the tile: byte offset of the words from (frame, first sample, channel), top bit: outside the image; byte offset
  // of the row in a plane of aggregates, first pixel (from bit 24 on), top bit: not there
  const int n_pairs = q.lr * q.nseg;
  for (int i = tid; i < n_pairs; i += kDeepThreads) {
    const int n0 = min(p.Ho - oy0, q.tr) * S + (3 - S);                // LDS rows of the tile's first sample
    const int per_sample = p.Ho * S + (3 - S);
    const int lr_used = (rows_valid - 1) * S + sample_of(rows_valid - 1) * (3 - S) + 3;
    const int row = SmallDiv(q.nseg).quot(i), seg = i - row * q.nseg;
    int bsel = 0, iy = oy0 * S - 1 + row;
    if (row >= n0) {
      const int over = SmallDiv(per_sample).quot(row - n0);
      bsel = 1 + over;
      iy = row - n0 - over * per_sample - 1;
    }
    const bool used = row < lr_used, inside = used && iy >= 0 && iy < p.H;
    u32x2 e;
    e[0] = inside ? ((uint32_t)(bsel * Cin) * in_chan + (uint32_t)(iy * wws + ((seg * q.xs) >> 5))) * 4u : kOutside;
    e[1] = (uint32_t)(row * q.wpx * 16) | (uint32_t)(seg * q.xs) << 24 | (used ? 0u : kOutside);
    pairs[i] = e;
  }
  // where a k-step's lane half finds its channels and tap
  if (tid < 2 * q.nks) {
    const int kk = 8 * tid, tap = SmallDiv(Cin).quot(kk), cin = kk - tap * Cin;
    const int ky = (tap * 11) >> 5, kx = tap - ky * 3;                 // tap / 3 for the nine taps
    tab[tid] = tap < 9 ? (cin >> 3) * q.plane + (ky * q.wpx + col(kx)) * 16 : 0;
  }
  const float scale = 1.0f / (float)(1u << kFixShift);
  // (a shorter last group's weights are the last of a whole group's)
  if constexpr (KP >= 4) frame_tables<KP>(lut, q.lut_set / 4, dp.K_last ? 2 : 1, p.K - dp.K_last, p, tid, kDeepThreads);
  if (tid < 32) bias_lds[tid] = (p.bias && co0 + tid < p.Cout) ? p.bias[co0 + tid] : 0.f;
  lds_barrier();

  // ---- the units of a round: (row and segment, channels, group), the first fastest; a thread has one of them a turn
  const int CC = Cin / UC, units = n_pairs * CC;
  const SmallDiv by_pairs(n_pairs), by_cc(CC);
  const int turns = (q.gb * units + kDeepThreads - 1) / kDeepThreads;
  struct Unit {
    int gb, cc;
    u32x2 e;
  };
  auto unit_of = [&](int u) {
    Unit x;
    const int v = by_pairs.quot(u);
    x.gb = by_cc.quot(v);
    x.cc = v - x.gb * CC;
    x.e = pairs[u - v * n_pairs];
    return x;
  };
  // Words are loaded through a buffer descriptor, which gives zeros for rows outside the image and frames that a group does not have.
  auto load_unit = [&](int g0, int turn, uint32_t (&wd)[UC][KP]) {
    const int gn = min(q.gb, n_groups - g0);
    const Unit x = unit_of(min(turn * kDeepThreads + tid, gn * units - 1));
    const size_t first = ((size_t)g0 * p.K * p.B + b0) * Cin * in_chan;
    const size_t bytes = ((size_t)(p.G * p.K + dp.K_last) * t_stride - first) * 4;
    const auto words = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t*>(p.spikes + first), 0, (int)(bytes < 0x7fffffffu ? bytes : 0x7fffffffu), 0x00020000);
    const int Kg = g0 + x.gb == p.G ? dp.K_last : p.K, frames = deep_round_frames(g0, p.G, p.K, dp.K_last);
    const uint32_t off = x.e[0] + ((uint32_t)x.gb * (uint32_t)p.K * (uint32_t)t_stride + (uint32_t)(x.cc * UC) * in_chan) * 4u;
#pragma unroll
    for (int j = 0; j < KP; ++j) {
      const uint32_t voff = j < Kg ? off : kOutside;
#pragma unroll
      for (int c = 0; c < UC; ++c)
        wd[c][j] = __builtin_amdgcn_raw_buffer_load_b32(words, (int)voff, (int)deep_scalar_offset(j, frames, (uint32_t)t_stride, c, in_chan), 0);
    }
  };
  const uint32_t two_lo = KP == 2 ? pack_bf16(0.f, (float)p.wq[0] * scale) : 0u;
  const uint32_t two_hi = KP == 2 ? pack_bf16((float)p.wq[1] * scale, (float)(p.wq[0] + p.wq[1]) * scale) : 0u;
  // (one frame left over: its weight is that of a whole group's second)
  const uint32_t two_lo_last = KP == 2 ? pack_bf16(0.f, (float)p.wq[1] * scale) : 0u;
  const uint32_t one = KP == 1 ? pack_bf16((float)p.wq[0] * scale, (float)p.wq[0] * scale) : 0u;
  auto form_unit = [&](int g0, int turn, uint32_t (&wd)[UC][KP]) {
    const int gn = min(q.gb, n_groups - g0), u = turn * kDeepThreads + tid;
    const Unit x = unit_of(min(u, gn * units - 1));
    const bool last = g0 + x.gb == p.G;
#pragma unroll
    for (int c = 0; c < UC; ++c) {
      if constexpr (KP == 16) {
        frames_to_fields<8>(wd[c]);
        frames_to_fields<8>(wd[c] + 8);
      } else {
        frames_to_fields<KP>(wd[c]);
      }
    }
    if (u >= gn * units || x.e[1] >> 31) return;
    const uint32_t* const tb = lut + (last ? q.lut_set / 4 : 0);
    const uint32_t lo = last ? two_lo_last : two_lo;
    uint8_t* const dst = lds + x.gb * q.group + x.cc / (8 / UC) * q.plane + (x.e[1] & 0xffffffu) + x.cc % (8 / UC) * (UC * 2);
    auto put = [](uint8_t* at, const uint32_t (&v)[UC / 2]) {
      if constexpr (UC == 8) *reinterpret_cast<u32x4*>(at) = u32x4{v[0], v[1], v[2], v[3]};
      else if constexpr (UC == 4) *reinterpret_cast<u32x2*>(at) = u32x2{v[0], v[1]};
      else *reinterpret_cast<uint32_t*>(at) = v[0];
    };
    // the aggregates of one pixel: sh, the field's bit; cl, its class
    auto pixel = [&](uint32_t (&v)[UC / 2], uint32_t sh, auto cl_) {
      constexpr int cl = decltype(cl_)::value;
      if constexpr (KP == 16) {
        uint32_t a[UC];
#pragma unroll
        for (int c = 0; c < UC; ++c) a[c] = tb[__builtin_amdgcn_ubfe(wd[c][cl], sh, 8)] + tb[256 + __builtin_amdgcn_ubfe(wd[c][8 + cl], sh, 8)];
#pragma unroll
        for (int c2 = 0; c2 < UC / 2; ++c2) v[c2] = pack_bf16((float)a[2 * c2] * scale, (float)a[2 * c2 + 1] * scale);
      } else {
#pragma unroll
        for (int c2 = 0; c2 < UC / 2; ++c2) {
          const uint32_t t0 = __builtin_amdgcn_ubfe(wd[2 * c2][cl], sh, KP), t1 = __builtin_amdgcn_ubfe(wd[2 * c2 + 1][cl], sh, KP);
          if constexpr (KP == 1) v[c2] = one & __umul24(t0 | t1 << 16, 0xffffu);
          else if constexpr (KP == 2) v[c2] = two_frame_pair(two_hi, lo, t0 | t1 << 16);
          else if constexpr (KP == 4) v[c2] = tb[t0 | t1 << 4];
          else v[c2] = tb[t0] | tb[t1] << 16;
        }
      }
    };
    constexpr int P = KP >= 8 ? 8 : 4;         // pixels a turn
    const int x0 = (int)(x.e[1] >> 24), x1 = min(x0 + q.xs, p.W);
#pragma clang loop unroll(disable)
    for (int xx = x0; xx < x1; xx += P) {
      uint32_t v[P][UC / 2];
      static_for<0, P>([&](auto c_) {
        constexpr int c = decltype(c_)::value, cl = c % (KP == 16 ? 8 : KP);
        pixel(v[c], (uint32_t)((xx & 31) + c - cl), std::integral_constant<int, cl>{});
      });
#pragma unroll
      for (int c = 0; c < P; ++c)
        if (c == 0 || xx + c < x1) put(dst + col(xx + c + 1) * 16, v[c]);
    }
    // the padding columns x = -1 and x = W (the partial sums have been over them)
    const uint32_t none[UC / 2] = {};
    if (x0 == 0) put(dst, none);
    if (x1 == p.W) put(dst + col(p.W + 1) * 16, none);
  };
  // two turns' words in hand; behind a round's the next round's (behind the last round the last one is asked for again)
  uint32_t wd[2][UC][KP];
  load_unit(0, 0, wd[0]);
  if (turns > 1) load_unit(0, 1, wd[1]);

  // ---- the lane's pixels; their membranes are 32-bit byte offsets from the tile's (without a second sample in the tile from its first row)
  const int r0 = wave * 2;                     // the wave steps registers r0 and r0 + 1 of every block
  const int v_row = q.flatten ? 0 : oy0;
  const size_t v_tile = ((size_t)b0 * p.Cout + co0) * plane + (size_t)v_row * p.Wo;
  const int co_lim = p.Cout - co0 - 4 * h;
  bool ok[PB];
  uint32_t v_off[PB], pix[PB];
#pragma unroll
  for (int np = 0; np < PB; ++np) {
    const int rr0 = (q.wb == 1 ? np : 0) * q.rpb + (n >> q.pw_shift), ox = (q.wb == 1 ? 0 : np * 32) + (n & ((1 << q.pw_shift) - 1));
    ok[np] = rr0 < rows_valid && ox < p.Wo;
    const int rr = ok[np] ? rr0 : 0, xx = ok[np] ? ox : 0;
    const int bsel = sample_of(rr), oy = oy0 + rr - bsel * p.Ho;
    v_off[np] = (uint32_t)((((size_t)bsel * p.Cout + 4 * h) * plane + (size_t)(oy - v_row) * p.Wo + xx) * 4);
    pix[np] = (uint32_t)(((rr * S + bsel * (3 - S)) * q.wpx + xx) * 16);
  }
  auto chan = [&](int r) { return 8 * ((r0 + r) >> 2) + ((r0 + r) & 3); };
  float V[PB][2];
#pragma unroll
  for (int np = 0; np < PB; ++np)
#pragma unroll
    for (int r = 0; r < 2; ++r) V[np][r] = 0.f;
  if (p.v_inout) {
#pragma unroll
    for (int np = 0; np < PB; ++np)
#pragma unroll
      for (int r = 0; r < 2; ++r)
        if (ok[np] && chan(r) < co_lim)
          V[np][r] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(p.v_inout + v_tile) + (size_t)chan(r) * plane * 4 + v_off[np]);
  }

  // ---- output words: lane 4 s + 2 i + hi holds register r0 + i, lane half hi, of the s-th step in hand
  const int st_r = r0 + ((lane >> 1) & 1), st_co = co0 + 8 * (st_r >> 2) + 4 * (lane & 1) + (st_r & 3);
  const int out_words = (p.Wo + 31) >> 5;
  const size_t out_step = (size_t)p.B * p.Cout * p.Ho * out_words;
  const uint32_t next_sample = (uint32_t)((p.Cout - 1) * p.Ho * out_words);              // what the row behind a sample's last one adds
  const uint32_t field = q.rpb > 1 ? (1u << (32 / q.rpb)) - 1u : 0xffffffffu;
  uint32_t* st_at[PB];                         // of the lane's step, channel and the block's first row
  int st_row[PB], st_rows[PB];                 // (wave-uniform)
#pragma unroll
  for (int np = 0; np < PB; ++np) {
    const int rr = (q.wb == 1 ? np : 0) * q.rpb;                       // the block's first tile row
    const int bsel = sample_of(min(rr, rows_valid - 1)), oy = oy0 + rr - bsel * p.Ho;
    st_row[np] = __builtin_amdgcn_readfirstlane(oy);
    st_rows[np] = min(q.rpb, rows_valid - rr);
    st_at[np] = p.out + (size_t)(lane >> 2) * out_step + (((size_t)(b0 + bsel) * p.Cout + st_co) * p.Ho + st_row[np]) * out_words + (q.wb > 1 ? np : 0);
  }
  auto store_words = [&](size_t step, const uint32_t (&word)[PB]) {
#pragma unroll
    for (int np = 0; np < PB; ++np) {
      uint32_t* at = st_at[np] + step * out_step;
      const uint32_t w = word[np];
      if (q.rpb == 1) {
        if (st_rows[np] > 0) *at = w;
        continue;
      }
#pragma clang loop unroll(disable)
      for (int s = 0, row = st_row[np]; s < st_rows[np]; ++s, ++at) {
        *at = (w >> (s << q.pw_shift)) & field;
        if (++row == p.Ho) { row = 0; at += next_sample; }
      }
    }
  };

  size_t step = 0;
  for (int g0 = 0; g0 < n_groups; g0 += q.gb) {
    const int gn = min(q.gb, n_groups - g0), g_next = g0 + q.gb < n_groups ? g0 + q.gb : g0;
    // ---- 1. aggregates
#pragma clang loop unroll(disable)
    for (int t = 0; t < turns; t += 2)
      static_for<0, 2>([&](auto s_) {
        constexpr int s = decltype(s_)::value;
        if (s > 0 && t + s >= turns) return;
        form_unit(g0, t + s, wd[s]);
        load_unit(t + s + 2 < turns ? g0 : g_next, t + s + 2 < turns ? t + s + 2 : s, wd[s]);
      });
    lds_barrier();
    // ---- 2. the wave's k-steps, nine blocks' fragments at a time
    f32x16 acc[kDeepSets];
#pragma unroll
    for (int i = 0; i < kDeepSets; ++i) {
      if (i / PB >= gn) continue;
      const uint32_t a = (uint32_t)(i / PB * q.group) + pix[i % PB];
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
#pragma unroll
      for (int kb = 0; kb < KS; kb += 9) {
        bf16x8 af[9];
#pragma unroll
        for (int k = 0; k < 9; ++k) af[k] = *reinterpret_cast<const bf16x8*>(lds + a + (uint32_t)tab[2 * min(k0 + kb + k, q.nks - 1) + h]);
#pragma unroll
        for (int k = 0; k < 9; ++k)
          if (kb + k < 1 || kb + k < n_k) acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w_own[kb + k], af[k], acc[i], 0, 0, 0);
      }
    }
    lds_barrier();                            // the aggregates have been read
    {
      f32x2* const part = reinterpret_cast<f32x2*>(lds) + lane;        // [set][wave][register pair][lane]
#pragma unroll
      for (int i = 0; i < kDeepSets; ++i)
        if (i / PB < gn)
#pragma unroll
          for (int r2 = 0; r2 < 8; ++r2) part[((i * 8 + wave) * 8 + r2) * 64] = f32x2{acc[i][2 * r2], acc[i][2 * r2 + 1]};
    }
    lds_barrier();
    float y[kDeepSets][2];
#pragma unroll
    for (int i = 0; i < kDeepSets; ++i) {
      if (i / PB >= gn) continue;
      const f32x2* const part = reinterpret_cast<const f32x2*>(lds) + lane + (i * 64 + wave) * 64;
      f32x2 in[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) in[k] = part[k * 512];
#pragma unroll
      for (int d = 1; d < 8; d *= 2)
#pragma unroll
        for (int k = 0; k + d < 8; k += 2 * d) {
          in[k][0] += in[k + d][0];
          in[k][1] += in[k + d][1];
        }
#pragma unroll
      for (int r = 0; r < 2; ++r) y[i][r] = in[0][r] + bias_lds[chan(r) + 4 * h];
    }
    lds_barrier();                            // the next aggregates may take the place of the partial sums
    // ---- 3. LIF steps
#pragma clang loop unroll(disable)
    for (int i = 0; i < gn; ++i) {
      const bool last = g0 + i == p.G;
      const int n_lif = last ? dp.n_lif_last : p.n_lif;
      const float decay = last ? dp.decay_last : p.decay;
      float yi[PB][2];
#pragma unroll
      for (int np = 0; np < PB; ++np)
#pragma unroll
        for (int r = 0; r < 2; ++r) {
          yi[np][r] = y[np][r];
#pragma unroll
          for (int k = 1; k < GB; ++k) yi[np][r] = i == k ? y[k * PB + np][r] : yi[np][r];
        }
#pragma clang loop unroll(disable)
      for (int j0 = 0; j0 < n_lif; j0 += 4) {
        uint32_t word[PB];
#pragma unroll
        for (int np = 0; np < PB; ++np) word[np] = 0;
        static_for<0, 4>([&](auto j_) {
          constexpr int j = decltype(j_)::value;
          if (j > 0 && j0 + j >= n_lif) return;                        // (uniform)
          [[maybe_unused]] char* const tl = reinterpret_cast<char*>(p.v_trace + (step + j) * ((size_t)p.B * p.Cout * plane) + v_tile);
#pragma unroll
          for (int np = 0; np < PB; ++np) {
            float v[2];
            uint64_t m[2];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
              v[r] = fmaf(decay, V[np][r], yi[np][r]);
              m[r] = __builtin_amdgcn_ballot_w64(ok[np] && v[r] >= p.theta);
            }
            const uint32_t x[2][2] = {{(uint32_t)m[0], (uint32_t)(m[0] >> 32)}, {(uint32_t)m[1], (uint32_t)(m[1] >> 32)}};
            word[np] = write_lanes<j * 4, 2, 1>(word[np], x);
#pragma unroll
            for (int r = 0; r < 2; ++r) {
              V[np][r] = __builtin_amdgcn_inverse_ballot_w64(m[r]) ? v[r] - p.theta : v[r];
              if (TRACE && ok[np] && chan(r) < co_lim) *reinterpret_cast<float*>(tl + (size_t)chan(r) * plane * 4 + v_off[np]) = v[r];
            }
          }
        });
        const int nj = min(4, n_lif - j0);
        if (lane < 4 * nj && st_co < p.Cout) store_words(step, word);
        step += nj;
      }
    }
  }
  if (p.v_inout) {
#pragma unroll
    for (int np = 0; np < PB; ++np)
#pragma unroll
      for (int r = 0; r < 2; ++r)
        if (ok[np] && chan(r) < co_lim)
          *reinterpret_cast<float*>(reinterpret_cast<char*>(p.v_inout + v_tile) + (size_t)chan(r) * plane * 4 + v_off[np]) = V[np][r];
  }
}

template <int KP, bool TRACE, int KS, int PB>
hipError_t deep_launch_t(const DeepParams& p, hipStream_t s) {
  const auto kern = &deep_kernel<KP, TRACE, KS, kDeepSets / PB, PB>;
  if (p.q.total > 64 * 1024) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kDeepLds);
    if (e != hipSuccess) return e;
  }
  const dim3 grid((unsigned)p.q.row_tiles * (unsigned)p.q.co_tiles, 1, p.q.flatten ? 1 : p.m.B);
  hipLaunchKernelGGL(kern, grid, dim3(kDeepThreads), p.q.total, s, p);
  return hipGetLastError();
}

template <bool TRACE, int KS, int PB>
hipError_t deep_launch_kp(const DeepParams& p, hipStream_t s) {
  switch (p.q.kp) {
    case 1: return deep_launch_t<1, TRACE, KS, PB>(p, s);
    case 2: return deep_launch_t<2, TRACE, KS, PB>(p, s);
    case 4: return deep_launch_t<4, TRACE, KS, PB>(p, s);
    case 8: return deep_launch_t<8, TRACE, KS, PB>(p, s);
    default: return deep_launch_t<16, TRACE, KS, PB>(p, s);
  }
}

// k-steps of a wave: nine up to 128 input channels, 18 up to 256
template <bool TRACE>
hipError_t deep_launch_any(const DeepParams& p, hipStream_t s) {
  if (deep_wave_steps(p.q.nks) == 9) return p.q.pb == 1 ? deep_launch_kp<TRACE, 9, 1>(p, s) : deep_launch_kp<TRACE, 9, 2>(p, s);
  return p.q.pb == 1 ? deep_launch_kp<TRACE, 18, 1>(p, s) : deep_launch_kp<TRACE, 18, 2>(p, s);
}

}  // namespace

}  // namespace tac
