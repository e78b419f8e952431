// First layers on the matrix cores: Cin * 9 <= 32, i.e. 1 input channel (rate-coded images) or 2 polarity channels (event
// cameras), packed spikes or real-valued frames, bf16 operands or fp32 ones.
//
// The whole contraction (tap, cin) fits one or two MFMA k-steps of 16 (fp32: 5 or 9 of 2), so im2col is done for real: a lane
// gathers the aggregated values under its output pixel's filter window from a small aggregate tile in LDS.  Weights and
// membrane stay in registers for the whole call.
//
// A pixel block is one packed word of an output row.  A wave owns two of them (consecutive words, or the two rows of a 2 x 2
// pool window) x 32 output channels; a workgroup is up to 8 waves, `pairs` block pairs x `blocks` channel blocks, that share
// the aggregate tile.  Per group of K frames:
//   1. every thread asks for the words (or values) of its pixels of the NEXT group, and forms their aggregates (Eq. 2) of this one in
//      the 24-bit fixed point of the large kernel (fp32 layers: in fp32; real-valued frames: in double), rounded once
//   2. one barrier (there are two tiles, so that nobody waits for the gathers of the group before)
//   3. gather, MFMAs, LIF steps (1, or K for TAC-TP), packed stores
// What bounds it is the vector ALU of the LIF steps, so the MFMA operands are swapped (pixels are the rows of the result: a lane holds
// 16 pixels of one channel, see lif_step_cols), four waves share a SIMD (128 registers), and the tile is aggregated while others run
// LIF steps.  With recorded membranes the pixels run along the lanes instead, as the stores want it, and the membranes' way to
// memory is the bound (537 MB of 2 -> 128 at 64 x 64, B = 16, 16 steps: 97 us, 5.5 TB/s; one wave per SIMD 158).
// Kernel times in us, and those of workgroups of four rows x 64 channels, one wave a row, three barriers a group and 16-bit gathers
// (fp32: of the vector kernel): 2 -> 64 at 128 x 128 stride 2, B = 32, TAC-TP K = 2, 16 frames 28 / 48 (B = 16: 19 / 39); real-valued
// 2 -> 128 at 64 x 64, B = 16, TAC-TP K = 4 24 / 45; 1 -> 32 at 28 x 28, B = 128, two groups of 4 7.5 / 18; fp32, 25 frames in groups
// of 8 18 / 50, with membranes in groups of 4 39 / 78.
#include "tac_first_plan.h"

namespace tac {

namespace {

// x / d by multiplication: the product is the quotient or one less
struct Div {
  uint32_t d, m;                               // m = 2^32 / d, at most 2^32 - 1
  Div() = default;
  explicit Div(uint32_t divisor) : d(divisor), m(divisor == 1 ? 0xffffffffu : (uint32_t)((1ull << 32) / divisor)) {}
  __device__ __forceinline__ uint32_t quot(uint32_t x) const {
    const uint32_t e = __umulhi(x, m);
    return x - e * d >= d ? e + 1 : e;
  }
};

struct FirstParams {
  const uint32_t* spikes;
  const void* w;
  const float* bias;
  float* v_inout;
  uint32_t* out;
  float* v_trace;
  int B, H, W, Ho, Wo, Cout, S, K, G, n_lif, K_last, n_lif_last, out_pool;
  int WW, Wwo;                                 // words per input and output row
  int n_pairs, pair_tiles, co_tiles, n_tiles;  // block pairs per sample; tiles over them, over the channels, in all
  int pairs, blocks, tile_words;               // per workgroup; 32-bit words of one aggregate tile
  Div by_wwo, by_blocks, by_pair_tiles, by_tiles;      // by_tiles: pair_tiles co_tiles
  uint32_t by_ww, by_w;                        // i / WW and i / W by multiplication (2^16 / WW + 1, 2^20 / W + 1)
  float decay, decay_last, theta;
  uint32_t wq[TAC_MAX_K + 8];                  // round(beta^(K-1-j) * 2^23), zeros behind the last
  float wj[TAC_MAX_K + 8];                     // beta^(K-1-j)
  double wjd[TAC_MAX_K + 8];
};

// KB: frames a thread asks for together, K's next power of two, at most 8 / CIN (frames beyond the group repeat its last and have
// the weight zero).  A larger group's further frames are waited for.
// NQ: quads of result registers with channels in them (4: all 32 channels of a block).  fp32 layers of up to 8 or 16 channels that record their
// membranes step and store 1 or 2, and fit 128 registers, four waves on a SIMD in the place of two: what bounds calls of few steps is a
// workgroup's chain from its parameters to its stores, about 8 us whatever it stores.  2 -> 8 at 60 x 40, B = 128, one group of two 31.3 -> 17.2 us,
// 2 -> 16 32.3 -> 20.4, 2 -> 8 at 83 x 12 23.6 -> 13.1.
template <int CIN, int KB, bool F32, bool DENSE, bool TRACE, int NQ = 4>
__global__ __launch_bounds__(kFirstWaves * 64, TRACE && NQ == 4 ? 2 : 4) void first_kernel(const FirstParams p) {
  static_assert(NQ == 4 || TRACE, "channels along the lanes: the registers are pixels");
  constexpr int NR = 4 * NQ;                                           // registers that are stepped
  constexpr int NS = F32 ? (9 * CIN + 1) / 2 : CIN;                    // k-steps
  constexpr int PX = DENSE ? 1 : 4;                                    // pixels a thread forms at a time
  extern __shared__ __attribute__((aligned(16))) uint32_t tiles[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int n_threads = p.pairs * p.blocks * 64;
  // the cache lines of the parameters are asked for together (one by one, where they are first needed, a workgroup that runs alone
  // waits for each)
  asm volatile("" :: "s"(p.B), "s"(p.n_pairs), "s"(p.theta), "s"(p.w));
  const int S = p.S, WP = first_row_words(p.W);

  // workgroups go to the 8 XCDs in turn: each takes consecutive tiles, which share input rows and output cache lines
  const uint32_t eighth = p.n_tiles >> 3;
  const uint32_t tile_id = blockIdx.x < eighth * 8 ? (blockIdx.x & 7) * eighth + (blockIdx.x >> 3) : blockIdx.x;
  const int b = p.by_tiles.quot(tile_id);
  const int in_sample = tile_id - b * p.by_tiles.d;
  const int co_tile = p.by_pair_tiles.quot(in_sample), pair0 = (in_sample - co_tile * p.pair_tiles) * p.pairs;
  const int wave_pair = p.by_blocks.quot(wave), pair = pair0 + wave_pair;
  const int co0 = (co_tile * p.blocks + wave - wave_pair * p.blocks) * 32;
  const bool active = pair < p.n_pairs && co0 < p.Cout;                // wave-uniform
  // output rows of the tile: first, and input rows behind them
  const int last_pair = min(pair0 + p.pairs, p.n_pairs) - 1;
  const int row0 = p.out_pool ? 2 * p.by_wwo.quot(pair0) : p.by_wwo.quot(2 * pair0);
  const int row1 = p.out_pool ? 2 * p.by_wwo.quot(last_pair) + 1 : min((int)p.by_wwo.quot(2 * last_pair + 1), p.Ho - 1);
  const int rows_in = (row1 - row0) * S + 3, iy0 = row0 * S - 1;

  // ---- the words (values) a thread turns into aggregates: item i is 4 pixels of a word, or one value, of every channel
  const int row_len = DENSE ? p.W : p.WW;
  const int n_items = DENSE ? rows_in * p.W : rows_in * p.WW * 8;
  const size_t in_chan = (size_t)p.H * row_len, frame = (size_t)p.B * CIN * in_chan;
  const int n_groups = p.G + (p.K_last ? 1 : 0);
  auto frames_of = [&](int g) { return g == p.G ? p.K_last : p.K; };
  struct Item {
    uint32_t off;                              // byte offset of the word from (frame, sample, first channel, first input row of the tile)
    int dst;                                   // word of the first pixel in the aggregate tile
    uint32_t keep;                             // pixels inside the image, a bit each
  };
  auto item = [&](int i) {
    const int t = DENSE ? i : i >> 3;
    const int row = DENSE ? (int)(((uint32_t)t * p.by_w) >> 20) : (int)(((uint32_t)t * p.by_ww) >> 16);
    const int col = t - row * row_len, x = DENSE ? col : col * 32 + (i & 7) * 4;
    const int iy = iy0 + row;
    Item it;
    it.off = (uint32_t)((min(max(iy, 0), p.H - 1) - max(iy0, 0)) * row_len + col) * 4;
    it.dst = row * WP + x + 1;
    it.keep = i < n_items && iy >= 0 && iy < p.H && x < p.W ? (p.W - x >= 4 ? 15u : (1u << (p.W - x)) - 1u) : 0u;
    if (i >= n_items) it.off = 0;
    return it;
  };
  const Item mine = item(tid);
  using Weight = std::conditional_t<DENSE, double, std::conditional_t<F32, float, uint32_t>>;
  const Weight* const weights = [&] {
    if constexpr (DENSE) return p.wjd;
    else if constexpr (F32) return p.wj;
    else return p.wq;
  }();
  Weight w_first[KB];                          // of a whole group's first frames
#pragma unroll
  for (int u = 0; u < KB; ++u) w_first[u] = weights[u];
  uint32_t next[CIN][KB];
  auto request = [&](const uint32_t* src, int left, uint32_t off) {
#pragma unroll
    for (int u = 0; u < KB; ++u) {
#pragma unroll
      for (int c = 0; c < CIN; ++c)
        next[c][u] = *reinterpret_cast<const uint32_t*>(reinterpret_cast<const char*>(src + c * in_chan) + off);
      size_t further = u + 1 < left ? frame : 0;
      asm volatile("" : "+s"(further));        // (the compiler is not to make a copy, and a wait, of a load that may repeat)
      src += further;
    }
  };
  const uint32_t* group_src = p.spikes + (size_t)b * CIN * in_chan + (size_t)max(iy0, 0) * row_len;
  request(group_src, frames_of(0), mine.off);

  // ---- weights: fragments of the channel block, kept in registers
  bf16x8 wf[CIN];
  float wf32[NS];
  if constexpr (F32) {
    const int cout_pad = (p.Cout + 31) & ~31;
#pragma unroll
    for (int s = 0; s < NS; ++s)
      wf32[s] = active && 2 * s + h < 9 * CIN ? static_cast<const float*>(p.w)[(size_t)(2 * s + h) * cout_pad + co0 + n] : 0.f;
  } else if constexpr (CIN == 2) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
      wf[ks] = *reinterpret_cast<const bf16x8*>(static_cast<const uint8_t*>(p.w) + (((active ? co0 : 0) / 32 * 2 + ks) * 64 + lane) * 16);
  } else {
    // one channel: the lane's slots are pairs of columns of a window row, (kx 0, kx 1) and (kx 2, nothing); prepared is tap 8 hh + i
    // at [lane half hh][i] of the first k-step
    const uint16_t* const w16 = static_cast<const uint16_t*>(p.w) + (size_t)((active ? co0 : 0) / 32) * 2 * 64 * 8;
    uint32_t pk[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int pair_no = 4 * h + i, tap = pair_no < 6 ? (pair_no >> 1) * 3 + (pair_no & 1) * 2 : 0;
      const uint32_t lo = w16[((tap >> 3) * 32 + n) * 8 + (tap & 7)], hi = w16[(((tap + 1) >> 3) * 32 + n) * 8 + ((tap + 1) & 7)];
      pk[i] = pair_no < 6 ? (pair_no & 1 ? lo : lo | (hi << 16)) : 0u;
    }
    wf[0] = __builtin_bit_cast(bf16x8, u32x4{pk[0], pk[1], pk[2], pk[3]});
  }
  // the bias is what the products are added to (pixels along the lanes: a register's own channel, kept in LDS)
  float* const bias_lds = reinterpret_cast<float*>(tiles + 2 * p.tile_words) + wave * 32;
  float bias = p.bias && co0 + n < p.Cout ? p.bias[co0 + n] : 0.f;
  if (TRACE && h == 0) bias_lds[n] = bias;

  // ---- the wave's two blocks
  int oy[2], word_of[2];
  bool ok[2];                                  // the block exists
#pragma unroll
  for (int np = 0; np < 2; ++np) {
    const int q = p.out_pool ? pair : 2 * pair + np, row = p.by_wwo.quot(q);
    oy[np] = p.out_pool ? 2 * row + np : row;
    word_of[np] = q - row * p.Wwo;
    ok[np] = active && oy[np] < p.Ho;
  }
  const size_t plane = (size_t)p.Ho * p.Wo;
  // LDS words of the window's first value and of the lane's contraction slots behind it (two channels in bf16: a word holds both;
  // one: a value and its right-hand neighbour)
  LaneGeom lg;
  int base[2], slot[F32 ? NS : 4];
#pragma unroll
  for (int np = 0; np < 2; ++np) {
    const int ox = 32 * word_of[np] + n;
    const bool in = ok[np] && ox < p.Wo;
    base[np] = in ? (oy[np] - row0) * S * WP + ox * S : 0;
    lg.ok[np] = in;
    lg.theta[np] = in ? p.theta : __builtin_inff();
    lg.v_off[np] = (uint32_t)((4 * h * plane + (size_t)(in ? (oy[np] - row0) * p.Wo + ox : 0)) * 4);
  }
  lg.co_lim = p.Cout - co0 - 4 * h;
  if constexpr (F32) {
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      const int kk = min(2 * s + h, 9 * CIN - 1), cin = kk / 9, tap = kk - cin * 9;
      slot[s] = cin * (p.tile_words / CIN) + (tap / 3) * WP + tap % 3;
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int tap = 4 * h + i, pair_no = min(4 * h + i, 5);
      slot[i] = CIN == 2 ? (tap / 3) * WP + tap % 3 : (pair_no >> 1) * WP + (pair_no & 1) * 2;
    }
  }

  // ---- membranes
  float V[1][2][16];
  float* const v_wave = p.v_inout + ((size_t)b * p.Cout + co0) * plane + (size_t)row0 * p.Wo;     // of the tile's first row
  float* const turn = reinterpret_cast<float*>(tiles + 2 * p.tile_words) + wave * kTurnFloats;   // only there where it is used
#pragma unroll
  for (int np = 0; np < 2; ++np)
#pragma unroll
    for (int r = 0; r < 16; ++r) V[0][np][r] = 0.f;
  if (p.v_inout && active) {
#pragma unroll
    for (int np = 0; np < 2; ++np)
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        // (lanes outside the image or the channels load a membrane that is inside; nobody stores theirs)
        const int c = min(8 * (r >> 2) + (r & 3), lg.co_lim - 1);
        V[0][np][r] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(v_wave) + (c >= 0 ? (size_t)c * plane * 4 + lg.v_off[np] : 0));
      }
    if constexpr (!TRACE) {
#pragma unroll
      for (int np = 0; np < 2; ++np) turn_block(V[0][np], turn, n, h);
    }
  }

  // ---- packed stores.  Channel per lane: lane (n, h) stores channel n of block h; pixels along the lanes: lane
  // (r << 2) | (hi << 1) | np channel 8 (r / 4) + 4 hi + r % 4 of block np
  const int st_np = TRACE ? lane & 1 : h;
  const int st_co = co0 + (TRACE ? 8 * (lane >> 4) + 4 * ((lane >> 1) & 1) + ((lane >> 2) & 3) : n);
  const int st_px = p.Wo - 32 * word_of[st_np];                        // pixels from the word's first to the row's end
  const uint32_t st_mask = st_px >= 32 ? 0xffffffffu : (1u << st_px) - 1u;
  const int Wwp = ((p.Wo >> 1) + 31) >> 5;
  const size_t out_plane = p.out_pool ? (size_t)(p.Ho >> 1) * Wwp : (size_t)p.Ho * p.Wwo;
  const size_t out_step = (size_t)p.B * p.Cout * out_plane;
  uint32_t* st_out = p.out + ((size_t)b * p.Cout + st_co) * out_plane +
                     (p.out_pool ? (size_t)(oy[0] >> 1) * Wwp + (word_of[0] >> 1) : (size_t)oy[st_np] * p.Wwo + word_of[st_np]);
  const bool st_ok = st_co < p.Cout && (p.out_pool ? active && st_np == 0 : ok[st_np]);
  auto store = [&](uint32_t word) {            // pooled: 16 pixels, half a word (the last one of an odd count closes its word)
    if (!st_ok) return;
    if (!p.out_pool) *st_out = word & st_mask;
    else if (word_of[0] & 1) reinterpret_cast<uint16_t*>(st_out)[1] = (uint16_t)word;
    else if (word_of[0] == p.Wwo - 1) *st_out = word;
    else reinterpret_cast<uint16_t*>(st_out)[0] = (uint16_t)word;
  };
  const uint32_t pool_mask = st_px >= 32 ? 0xffffu : (1u << (st_px >> 1)) - 1u;

  for (int i = tid; i < 2 * p.tile_words; i += n_threads) tiles[i] = 0;       // the padding columns stay zero
  __syncthreads();

  // ---- 1. aggregates of group g -> its tile; the first frames of the next group are requested
  auto aggregate = [&](int g) {
    uint32_t* const tile = tiles + (g & 1) * p.tile_words;
    const int Kg = frames_of(g), first = p.K - Kg;                     // a shorter last group's weights are the last ones
    for (int i0 = 0; i0 + wave * 64 < n_items; i0 += n_threads) {
      Item it = mine;
      if (i0) it = item(i0 + tid);
      Weight a[CIN][PX];
#pragma unroll
      for (int c = 0; c < CIN; ++c)
#pragma unroll
        for (int k = 0; k < PX; ++k) a[c][k] = 0;
      const uint32_t* src = group_src;
      for (int j0 = 0; j0 < Kg; j0 += KB, src += KB * frame) {
        if (i0 | j0) request(src, Kg - j0, it.off);
        Weight w[KB];
#pragma unroll
        for (int u = 0; u < KB; ++u) w[u] = w_first[u];
        if (first + j0) {
#pragma unroll
          for (int u = 0; u < KB; ++u) w[u] = weights[first + j0 + u];
        }
#pragma unroll
        for (int u = 0; u < KB; ++u) {
          if constexpr (DENSE) {
            // real-valued frames: products and sums in double, rounded one by one (a frame beyond the group is not multiplied by
            // zero: it may hold an infinity)
            if (u == 0 || j0 + u < Kg) {
#pragma unroll
              for (int c = 0; c < CIN; ++c)
                a[c][0] = __dadd_rn(a[c][0], __dmul_rn(w[u], (double)__uint_as_float(next[c][u])));
            }
          } else {
#pragma unroll
            for (int c = 0; c < CIN; ++c) {
              const uint32_t bits = (next[c][u] >> ((tid & 7) * 4)) & it.keep;
#pragma unroll
              for (int k = 0; k < PX; ++k) {
                if constexpr (F32) a[c][k] += __uint_as_float((0u - ((bits >> k) & 1u)) & __float_as_uint(w[u]));
                else a[c][k] = __umul24(__builtin_amdgcn_ubfe(bits, k, 1), w[u]) + a[c][k];
              }
            }
          }
        }
      }
      if (!it.keep) continue;                  // outside the image, where the tile was cleared
      uint32_t* const dst = tile + it.dst;
      float f[CIN][PX];
#pragma unroll
      for (int c = 0; c < CIN; ++c)
#pragma unroll
        for (int k = 0; k < PX; ++k) {
          if constexpr (DENSE) f[c][k] = (float)a[c][k];
          else if constexpr (F32) f[c][k] = a[c][k];
          else f[c][k] = (float)a[c][k] * (1.0f / (float)(1u << kFixShift));
        }
#pragma unroll
      for (int k = 0; k < PX; ++k) {           // (zeros behind the row's end)
        if constexpr (F32) {
#pragma unroll
          for (int c = 0; c < CIN; ++c) reinterpret_cast<float*>(dst)[c * (p.tile_words / CIN) + k] = f[c][k];
        } else if constexpr (CIN == 2) {
          dst[k] = pack_bf16(f[0][k], f[CIN - 1][k]);
        } else if (k + 1 < PX) {
          dst[k] = pack_bf16(f[0][k], f[0][(k + 1) % PX]);
        } else {
          reinterpret_cast<uint16_t*>(dst + k)[0] = (uint16_t)pack_bf16(f[0][k], 0.f);
        }
      }
      if constexpr (!F32 && CIN == 1) reinterpret_cast<uint16_t*>(dst)[-1] = (uint16_t)pack_bf16(f[0][0], 0.f);   // right-hand neighbour of x - 1
    }
    group_src += (size_t)p.K * frame;
    if (g + 1 < n_groups) request(group_src, frames_of(g + 1), mine.off);
  };
  // what was loaded so far arrives here: a wait for it inside the loop would be a wait for the next group's words as well
  __builtin_amdgcn_s_waitcnt(0x0f70);
  asm volatile("" : "+v"(bias));
  size_t step = 0;
  for (int g = -1; g < n_groups; ++g) {        // (turn -1 forms the first group's aggregates)
    const bool last = g == p.G;
    const int n_lif = last ? p.n_lif_last : p.n_lif;
    const float decay = last ? p.decay_last : p.decay;
    const uint32_t* const tile = tiles + (g & 1) * p.tile_words;
    if (g + 1 < n_groups) aggregate(g + 1);    // (in front of the products: there are no accumulators yet)
    // ---- 2. gather the filter windows, multiply
    f32x16 acc[1][2];
    const bool busy = active && g >= 0;
    if (busy) {
#pragma unroll
      for (int np = 0; np < 2; ++np) asm volatile("" : "+v"(base[np]));          // (no registers for sums with the slots,
      asm volatile("" : "+v"(bias));                                             // nor for copies of the bias)
      auto first_products = [&](auto multiply) {                       // a product without a bias needs no registers of zeros
        if (p.bias) {
          f32x16 c;
#pragma unroll
          for (int r = 0; r < 16; ++r) c[r] = r >= NR ? 0.f : TRACE ? bias_lds[8 * (r >> 2) + 4 * h + (r & 3)] : bias;
          multiply(c);
        } else {
          f32x16 c = {};
          multiply(c);
        }
      };
      if constexpr (F32) {
        first_products([&](const f32x16& c) { acc[0][0] = c; acc[0][1] = c; });
#pragma unroll
        for (int np = 0; np < 2; ++np) {
          float af[NS];
#pragma unroll
          for (int s = 0; s < NS; ++s) {
            af[s] = __uint_as_float(tile[base[np] + slot[s]]);
            if (2 * s + 1 >= 9 * CIN) af[s] = h ? 0.f : af[s];         // the slot beyond the window
          }
#pragma unroll
          for (int s = 0; s < NS; ++s)
            acc[0][np] = TRACE ? __builtin_amdgcn_mfma_f32_32x32x2f32(wf32[s], af[s], acc[0][np], 0, 0, 0)
                               : __builtin_amdgcn_mfma_f32_32x32x2f32(af[s], wf32[s], acc[0][np], 0, 0, 0);
        }
      } else {
        bf16x8 af[2][CIN];
#pragma unroll
        for (int np = 0; np < 2; ++np) {
          uint32_t pk[4];
#pragma unroll
          for (int i = 0; i < 4; ++i) pk[i] = tile[base[np] + slot[i]];
          if constexpr (CIN == 1) {            // the window has no fourth column, and the upper lanes but one row
            pk[1] &= 0xffffu;
            pk[3] = h ? 0u : pk[3] & 0xffffu;
            pk[2] = h ? 0u : pk[2];
          }
          af[np][0] = __builtin_bit_cast(bf16x8, u32x4{pk[0], pk[1], pk[2], pk[3]});
          if constexpr (CIN == 2) {
            const uint32_t t8 = tile[base[np] + 2 * WP + 2];
            af[np][1] = __builtin_bit_cast(bf16x8, u32x4{h ? 0u : t8, 0u, 0u, 0u});
          }
        }
        auto product = [&](int ks, int np, const f32x16& c) {
          acc[0][np] = TRACE ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[ks], af[np][ks], c, 0, 0, 0)
                             : __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[np][ks], wf[ks], c, 0, 0, 0);
        };
        first_products([&](const f32x16& c) { product(0, 0, c); product(0, 1, c); });
        if constexpr (CIN == 2) { product(1, 0, acc[0][0]); product(1, 1, acc[0][1]); }
      }
    }
    // ---- 3. LIF steps on Y_k = acc (bias included)
    if (busy) {
      for (int j = 0; j < n_lif; ++j, ++step, st_out += out_step) {
        if constexpr (TRACE) {
          uint32_t word[1][2] = {{0u, 0u}};
          float* const tl = p.v_trace + step * ((size_t)p.B * p.Cout * plane) + ((size_t)b * p.Cout + co0) * plane + (size_t)row0 * p.Wo;
          lif_step<1, 64, true, 2, NQ>(V, acc, decay, p.theta, lg, word, tl, plane);
          // pooled: the two rows of a window stand in neighbouring lanes
          store(p.out_pool ? pool_pairs(word[0][0] | (uint32_t)__shfl_xor((int)word[0][0], 1, 64)) : word[0][0]);
        } else {
          uint32_t bits[2];
          lif_step_cols<2>(V[0], acc[0], decay, p.theta, bits);
          store(p.out_pool ? pooled_of_cols(bits) & pool_mask : words_of_cols(bits));
        }
      }
    }
    if (g + 1 < n_groups) __syncthreads();
  }

  if (p.v_inout && active) {
#pragma unroll
    for (int np = 0; np < 2; ++np) {
      if constexpr (!TRACE) turn_block(V[0][np], turn, n, h);
#pragma unroll
      for (int r = 0; r < NR; ++r) {
        const int c = 8 * (r >> 2) + (r & 3);
        if (lg.ok[np] && c < lg.co_lim)
          *reinterpret_cast<float*>(reinterpret_cast<char*>(v_wave) + (size_t)c * plane * 4 + lg.v_off[np]) = V[0][np][r];
      }
    }
  }
}

// OIHW fp32 -> [32-cout block][k-step][lane][8] bf16: lane l of block mc holds cout 32 mc + l % 32 and the
// contraction slots kk = 16 ks + 8 (l / 32) + i, slot kk = (tap kk / Cin, cin kk % Cin); slots
// beyond 9 Cin and channels beyond Cout are zero.
__global__ void small_prepare_kernel(const float* __restrict__ w, uint32_t* __restrict__ out, int Cin, int Cout, int nmc) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;                // one thread per bf16 pair
  if (i >= nmc * 2 * 64 * 4) return;
  const int e2 = i & 3, l = (i >> 2) & 63, ks = (i >> 8) & 1, mc = i >> 9;
  const int co = mc * 32 + (l & 31);
  float v[2];
  for (int u = 0; u < 2; ++u) {
    const int kk = 16 * ks + 8 * (l >> 5) + 2 * e2 + u;
    const int tap = kk / Cin, cin = kk - tap * Cin;
    v[u] = (tap < 9 && co < Cout) ? w[((size_t)co * Cin + cin) * 9 + tap] : 0.f;
  }
  out[i] = pack_bf16(v[0], v[1]);
}

template <int CIN, int KB, bool F32, bool DENSE>
hipError_t first_launch_t(const FirstParams& p, size_t lds, hipStream_t s) {
  const dim3 grid((unsigned)p.n_tiles), block((unsigned)(p.pairs * p.blocks * 64));
  auto kern = p.v_trace ? &first_kernel<CIN, KB, F32, DENSE, true> : &first_kernel<CIN, KB, F32, DENSE, false>;
  if constexpr (F32) {
    if (p.v_trace && p.Cout <= 16) kern = p.Cout <= 8 ? &first_kernel<CIN, KB, F32, DENSE, true, 1> : &first_kernel<CIN, KB, F32, DENSE, true, 2>;
  }
  if (lds > 64 * 1024) {                       // (fp32, two channels, stride 2 on wide rows, with a membrane to turn)
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 80 * 1024);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, grid, block, lds, s, p);
  return hipGetLastError();
}

template <int CIN, bool F32, bool DENSE>
hipError_t first_launch_k(const FirstParams& p, size_t lds, hipStream_t s) {
  if (p.K == 1) return first_launch_t<CIN, 1, F32, DENSE>(p, lds, s);
  if (p.K == 2) return first_launch_t<CIN, 2, F32, DENSE>(p, lds, s);
  if (p.K <= 4 || CIN == 2) return first_launch_t<CIN, 4, F32, DENSE>(p, lds, s);
  return first_launch_t<CIN, 8 / CIN, F32, DENSE>(p, lds, s);
}

template <int CIN, bool F32>
hipError_t first_launch_c(const LayerParams& l, const FirstParams& p, size_t lds, hipStream_t s) {
  return l.dense ? first_launch_k<CIN, F32, true>(p, lds, s) : first_launch_k<CIN, F32, false>(p, lds, s);
}

hipError_t first_launch(const LayerParams& l, hipStream_t s) {
  FirstParams p{};
  p.spikes = l.spikes; p.w = l.w; p.bias = l.bias; p.v_inout = l.v_inout; p.out = l.out; p.v_trace = l.v_trace;
  p.B = l.B; p.H = l.H; p.W = l.W; p.Ho = l.Ho; p.Wo = l.Wo; p.Cout = l.Cout; p.S = l.stride;
  p.K = l.K; p.G = l.G; p.n_lif = l.n_lif; p.K_last = l.K_last; p.n_lif_last = l.n_lif_last; p.out_pool = l.out_pool;
  p.WW = l.Wwi; p.Wwo = l.Wwo;
  p.by_ww = (1u << 16) / p.WW + 1;             // exact for fewer than 2^14 words, 2^13 pixels of a tile
  p.by_w = (1u << 20) / p.W + 1;
  p.decay = l.decay; p.decay_last = l.decay_last; p.theta = l.theta;
  for (int j = 0; j < l.K; ++j) {
    p.wq[j] = (uint32_t)((double)l.wj[j] * (double)(1u << kFixShift) + 0.5);
    p.wj[j] = l.wj[j];
    p.wjd[j] = l.wjd[j];
  }
  const FirstPlan plan = first_plan(l);
  p.n_pairs = plan.n_pairs; p.pair_tiles = plan.pair_tiles; p.co_tiles = plan.co_tiles; p.n_tiles = (int)plan.workgroups;
  p.pairs = plan.pairs; p.blocks = plan.blocks; p.tile_words = plan.tile_words;
  p.by_wwo = Div(p.Wwo); p.by_blocks = Div(p.blocks); p.by_pair_tiles = Div(p.pair_tiles); p.by_tiles = Div(p.pair_tiles * p.co_tiles);
  if (l.bf16) return l.Cin == 1 ? first_launch_c<1, false>(l, p, plan.lds, s) : first_launch_c<2, false>(l, p, plan.lds, s);
  return l.Cin == 1 ? first_launch_c<1, true>(l, p, plan.lds, s) : first_launch_c<2, true>(l, p, plan.lds, s);
}

}  // namespace

bool mfma_small_supported(const tac_layer_desc_t& d) {
  if (d.precision != TAC_BF16 || (d.in_format != TAC_IN_BITS && d.in_format != TAC_IN_F32)) return false;
  if (d.Cin < 1 || d.Cin > 2) return false;
  return d.W <= kFirstMaxW;
}

size_t mfma_small_weight_bytes(const tac_layer_desc_t& d) {
  const int nmc = d.Cout <= 32 ? 1 : 2;                        // blocks are stored in pairs
  return (size_t)((d.Cout + nmc * 32 - 1) / (nmc * 32)) * nmc * 2 * 64 * 16;
}

hipError_t mfma_small_prepare(const tac_layer_desc_t& d, const float* w_oihw, void* w_prepared, hipStream_t s) {
  const int per = d.Cout <= 32 ? 1 : 2;
  const int nmc = (d.Cout + per * 32 - 1) / (per * 32) * per;
  const int total = nmc * 2 * 64 * 4;
  hipLaunchKernelGGL(small_prepare_kernel, dim3((total + 255) / 256), dim3(256), 0, s, w_oihw,
                     static_cast<uint32_t*>(w_prepared), d.Cin, d.Cout, nmc);
  return hipGetLastError();
}

hipError_t mfma_small_launch(const LayerParams& p, hipStream_t s) { return first_launch(p, s); }

hipError_t first_f32_launch(const LayerParams& p, hipStream_t s) { return first_launch(p, s); }

}  // namespace tac
