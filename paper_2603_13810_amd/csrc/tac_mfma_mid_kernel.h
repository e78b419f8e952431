// MFMA kernel for the layers in between: input channels a multiple of 8 up to 128, any width up to 128 with at most 64
// output pixels per row, any input format made of bits (as they are, or through the 2 x 2 mean or max pool on load),
// any number of output channels.  It takes the shapes the large kernel does not (widths other than 32 / 64, fewer than
// 128 output channels, the mean pool), e.g. the second convolution of the rate-coded network (32 -> 64 at 14 x 14 after
// Pool(2), Sec. 5.1) and the deep 16 x 16 .. 2 x 2 blocks of the event-data network.
//
// Same GEMM orientation and LIF epilogue as the other MFMA kernels.  A pixel block is 32 lanes: a word of an output row,
// or, where rows have at most 16 pixels, several rows of 16, 8, 4 or 2 lanes each, counted over the rows of all samples,
// so that small images fill the lanes (a block per row of 14, 8 or 4 pixels would leave 56, 75 or 88 % of the matrix
// cores' columns empty).  Workgroup = 4 waves = up to 4 NNP pixel blocks x NMC blocks of 32 output channels, membrane in
// registers and the tile's weights (all taps, all input channels) in LDS for the whole call.  Per group of K frames:
//   1. aggregate tile A_k (Eq. 2) in LDS as [8 channels][row][column][8], so that neighbouring pixels are neighbouring
//      16-byte reads.  A wave forms its share of the tile (some 8-channel groups, some rows) without meeting the others:
//      it loads the packed words, each word once (consecutive lanes take consecutive words of a channel), turns the K
//      frame words of 32 pixels into per-pixel K-bit fields in registers (frames_to_fields), stages them in its own
//      corner of the LDS, and then, a pixel per lane, looks the aggregates of 8 channels up in a table.  The next words
//      are requested before that, through the end of a group into the next one.  On the small layers this kernel serves
//      a wave has a SIMD nearly to itself and what counts is the number of instructions and of LDS round trips, so a
//      wave does its share in one piece where the LDS allows (`job`), with what it needs to know about its words and
//      pixels in tables made once.
//   2. contraction over slots kk = tap * Cin + cin in steps of 16 (two 8-channel groups, one per lane half)
//   3. bias, LIF steps (1, or K for TAC-TP), ballot, packed stores
// F32: the fp32 layers of these shapes on the same structure with v_mfma_f32_32x32x2_f32: aggregate tile and weights in
// LDS as float32, two contraction slots per MFMA, products and sums in fp32.
//
// DIRECT: groups of one or two frames where a thread has at most kMidDirect pixels of 8 channels; no staging, no tables.
//
// A shorter last group (T mod K frames) is one more turn of the loop with tables of its own, the membrane still in
// registers.
//
// Measured against one row per wave, every thread gathering the bits of its own 8 values from global memory and the
// shorter last group a launch of its own, calls in us: 48 -> 80 at 45 x 45, B = 24, 25 frames in groups of 4: 531 -> 107; blocks
// of 128 -> 128 at 16 x 16 / 8 x 8 / 4 x 4, B = 16, TAC-TP K = 4, 16 frames: 136 / 85 / 62 -> 34 / 32 / 33; fp32 32 -> 64 at
// 14 x 14 behind the mean pool, B = 128, 25 frames in groups of 8: 423 -> 84.  The small ones have 64 to 256 workgroups and are
// bound by one wave's instruction stream and LDS trips (a step reads 2 KiB of fragments for one MFMA; the LDS delivers 128
// bytes a cycle): tables, aggregates, MFMAs and LIF steps of a group follow each other.
#pragma once
#include "tac_mfma_common.h"

namespace tac {

constexpr int kMidThreads = 256;
constexpr int kMidRanges = 8;   // partial sums of an output where waves share a pixel block, whatever their number
constexpr int kMidRangeSteps = 9;        // k-steps of one at most (128 input channels)
constexpr int kMidTabPad = 24;  // entries of the slot table behind the last k-step (fetched ahead)
// Sets of operand fragments in flight: with few MFMAs per step (32 cycles each) a step is shorter than an LDS read
__host__ __device__ constexpr int mid_depth(int nmc, int nnp) { return nmc * nnp == 1 ? 4 : nmc * nnp == 2 ? 3 : 2; }

// Geometry of one launch, resolved on the host (mid_plan).  Byte offsets are from the start of the LDS.
struct MidPlan {
  int pw_shift, rpb, wb;        // lanes of a row within a block = 1 << pw_shift, rows per block, blocks per row
  int trg, tr;                  // row groups (of rpb rows) and output rows per tile
  int lr;                       // LDS rows of the largest tile
  int flatten;                  // output rows are counted through all samples (a tile may straddle two)
  int row_tiles, co_tiles;      // tiles over the rows (per sample, or over all of them), over the output channels
  int cg, parts_shift, parts, lrp;      // a job = cg groups of 8 channels x lrp LDS rows; parts: jobs over the rows, a power of two
  int loaders;                  // waves, of every four, that form aggregates: all four unless their staging areas do not fit the LDS
  int direct;                   // no jobs: every thread forms up to kMidDirect pixels of 8 channels from words of its own
  int srows, wws, hs;           // stored rows per LDS row (2: pool on load), words per stored row, stored rows per channel
  int rw, rws;                  // (stored row, word) pairs per job and channel; staged dwords per pair and 8 channels
  int n_jobs, chunks, batches;  // jobs per tile; (chunk of frames, 64 U units) pairs per job, the same in batches of kMidBatch
  int nb;                       // table chunks of 8 frames
  int wpx, xh, plane;           // columns of the aggregate tile, of its even half (stride 2), bytes per channel group
  int nks, nmc_w;               // k-steps; 32-channel blocks per tile of the prepared weights
  int off_w, off_tab, off_bias, off_wq, off_unit, off_px, off_lut, off_stage, stage_wave, total;
  int nco;                      // tiles of output channels per workgroup, four waves each, over one aggregate tile
  int split, off_part;          // eight waves, `split` of which share a pixel block (0: four waves with blocks of their own); their partial sums
};

struct MidParams {
  MfmaParams m;
  MidPlan q;
  int K_last, n_lif_last;       // frames and LIF steps of a shorter last group (0: none)
  float decay_last;
};

hipError_t mid_launch_bf16(const MidParams& p, int kp, int nmc, int nnp, hipStream_t s);
hipError_t mid_launch_bf16_trace(const MidParams& p, int kp, int nmc, int nnp, hipStream_t s);
hipError_t mid_launch_f32(const MidParams& p, int kp, int nnp, hipStream_t s);
hipError_t mid_launch_f32_trace(const MidParams& p, int kp, int nnp, hipStream_t s);

namespace {

constexpr int kMidBatch = 4;    // chunks of words a wave loads at a time
constexpr int kMidDirect = 2;   // pixels of 8 channels per thread that go without staging
// units a lane takes per chunk
__host__ __device__ constexpr int mid_units(int kp) { return kp <= 2 ? 2 : 1; }

// KP: frames per table index (1, 2, 4 or 8; missing frames are zero words).  NMC x NNP: blocks of 32 channels x 32 pixels
// per wave.  DIRECT: the plan's direct.  SPLIT: the plan's split, see below.
//
// SPLIT.  Images of at most 16 x 16 pixels on many channels have few pixel blocks: a workgroup's waves stood idle while one or two of
// them multiplied 72 k-steps and made the LIF steps.  There eight waves share 8 / SPLIT pixel blocks of 32 channels, SPLIT waves
// each: a wave multiplies its part of the k-steps, whose weights it keeps in registers for the whole call, the partial sums
// meet in LDS, and each wave adds up and steps 16 / SPLIT registers of the block.  The sum is that of eight ranges of k-steps in
// a fixed tree whatever SPLIT is.  A wave that has one job in every group keeps its entries of the tables in registers, and up to
// four steps leave in one store.  128 -> 128, B = 16, TAC-TP K = 4, 16 frames, pooled, us a call before and now: 16 x 16 33.3 / 23.5, 8 x 8
// 29.8 / 19.5, 4 x 4 31.0 / 18.4 (with membranes 48 / 28, 43 / 22, 44 / 20).  Of the 18.4 the products are less than one: what
// remains is forming the aggregates (two thirds) and the chain of barriers and LDS trips.
//
// NCO (fp32).  Four waves per tile of output channels, NCO tiles over one aggregate tile, which is formed once for them instead of
// once per 32 channels: 32 -> 64 at 14 x 14 behind the mean pool, B = 128, 25 frames, groups of 8 81 -> 69 us, groups of 4 with membranes
// 124 -> 115.  (bf16 layers have their 64-channel tiles; two or three tiles of 32 over one aggregate tile were not faster: 48 -> 80 at
// 45 x 45 99 us so or so, 32 -> 128 at 40 x 40 72 -> 80 and 100, one large workgroup in step with itself against two that fill each
// other's gaps.)
template <int KP, int NMC, int NNP, bool TRACE, bool F32, bool DIRECT, int SPLIT = 0, int NCO = 1>
__global__ __launch_bounds__(SPLIT ? 512 : kMidThreads * NCO,
                             NCO == 1 && ((TRACE && NMC * NNP == 4) || (F32 && NNP == 2)) ? 1 : 2) void mid_kernel(const MidParams mp) {
  static_assert(!F32 || NMC == 1, "fp32: 32-channel tiles (the partial sums take the registers of a second block)");
  static_assert(NCO == 1 || F32, "tiles of several channel blocks: fp32");
  static_assert(!SPLIT || (NMC * NNP == 1 && !F32 && NCO == 1), "waves that share a pixel block: one block of bf16 operands");
  constexpr int NT = SPLIT ? 512 : kMidThreads * NCO;
  constexpr uint32_t kNone = 0xffffffffu;
  const MfmaParams& p = mp.m;
  const MidPlan& q = mp.q;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int n = lane & 31, h = lane >> 5;
  const int Cin = p.Cin, S = p.stride, C8 = Cin >> 3;

  const uint32_t row_tile = blockIdx.x / (uint32_t)q.co_tiles;
  const int co_tile = (int)(blockIdx.x - row_tile * (uint32_t)q.co_tiles);
  // output rows are counted through all samples (fewer than 2^20), or the grid's z is the sample
  const SmallDiv by_ho(p.Ho);
  const int first_row = (int)row_tile * q.tr;
  const int b0 = q.flatten ? by_ho.quot(first_row) : (int)blockIdx.z;
  const int oy0 = q.flatten ? first_row - b0 * p.Ho : first_row;
  const int rows_valid = min(q.tr, (q.flatten ? p.B * p.Ho : p.Ho) - first_row);
  auto sample_of = [&](int rr) { return q.flatten ? by_ho.quot(oy0 + rr) : 0; };     // tile row -> sample - b0
  const int px4 = NCO == 1 || SPLIT ? wave : wave & 3, co_grp = NCO == 1 ? 0 : wave >> 2;      // the wave among the four of its channels
  const int co_first = co_tile * (NCO * NMC * 32), co0 = co_first + co_grp * (NMC * 32);
  const size_t plane = (size_t)p.Ho * p.Wo;
  const size_t in_chan = (size_t)q.hs * q.wws;
  const size_t t_stride = (size_t)p.B * Cin * in_chan;

  uint8_t* const w_lds = lds + q.off_w + co_grp * q.nks * NMC * (F32 ? 256 : 1024);
  int32_t* const tab = reinterpret_cast<int32_t*>(lds + q.off_tab);
  float* const bias_all = reinterpret_cast<float*>(lds + q.off_bias);
  const float* const bias_lds = bias_all + co_grp * (NMC * 32);
  u32x2* const unit = reinterpret_cast<u32x2*>(lds + q.off_unit);
  u32x2* const pxt = reinterpret_cast<u32x2*>(lds + q.off_px);
  uint32_t* const lut = reinterpret_cast<uint32_t*>(lds + q.off_lut);
  uint8_t* const stage = lds + q.off_stage + wave * q.stage_wave;

  // ---- the tile's weights: [k-step][block] fragments of 1 KiB (fp32: 256 bytes), on their way while the tables are made
  constexpr int kShare = SPLIT ? SPLIT : 1, kOwn = SPLIT ? kMidRanges / kShare : 1;                 // SPLIT: ranges of k-steps per wave
  [[maybe_unused]] const int k_part = SPLIT ? wave % kShare : 0, px_wave = SPLIT ? wave / kShare : 0;
  auto range_start = [&](int i) { return (q.nks * (k_part * kOwn + i)) >> 3; };
  bf16x8 w_own[kOwn][SPLIT ? kMidRangeSteps : 1];
  if constexpr (SPLIT) {
    const int tile = co_tile / q.nmc_w;
    const uint8_t* const src = p.w + ((size_t)tile * q.nks * q.nmc_w + (co_tile - tile * q.nmc_w)) * 1024 + lane * 16;
#pragma unroll
    for (int i = 0; i < kOwn; ++i)
#pragma unroll
      for (int k = 0; k < kMidRangeSteps; ++k)                         // (a step behind the range's last is loaded and not multiplied)
        w_own[i][k] = *reinterpret_cast<const bf16x8*>(src + (size_t)min(range_start(i) + k, q.nks - 1) * q.nmc_w * 1024);
  } else {
    if constexpr (F32) {
      const uint8_t* const src = p.w + (co0 < p.Cout ? (size_t)(co_tile * NCO + co_grp) * q.nks * 256 : (size_t)0) + lane * 16;
      for (int f = px4; f < q.nks / 4; f += 4) lds_dma16<1, 0>(src + (size_t)f * 1024, (uint32_t)(uintptr_t)(lds_void_ptr)(w_lds + f * 1024));
    } else {
#pragma unroll
      for (int mc = 0; mc < NMC; ++mc) {
        const int blk = (co_tile * NCO + co_grp) * NMC + mc, tile = blk / q.nmc_w;
        // (a block beyond the channels is multiplied but never stored)
        const uint8_t* const src =
            p.w + (blk * 32 < p.Cout ? ((size_t)tile * q.nks * q.nmc_w + (blk - tile * q.nmc_w)) * 1024 : (size_t)0) + lane * 16;
        for (int ks = px4; ks < q.nks; ks += 4)
          lds_dma16<1, 0>(src + (size_t)ks * q.nmc_w * 1024, (uint32_t)(uintptr_t)(lds_void_ptr)(w_lds + (ks * NMC + mc) * 1024));
      }
    }
  }
  // ---- tables
  const int n0 = min(p.Ho - oy0, q.tr) * S + (3 - S);                  // LDS rows of the tile's first sample
  const int per_sample = p.Ho * S + (3 - S);
  const int lr_used = (rows_valid - 1) * S + sample_of(rows_valid - 1) * (3 - S) + 3;
  auto input_row = [&](int row, int& bsel, int& iy) {                  // LDS row -> sample - b0, row of its image
    bsel = 0;
    iy = oy0 * S - 1 + row;
    if (row >= n0) {
      const int over = SmallDiv(per_sample).quot(row - n0);
      bsel = 1 + over;
      iy = row - n0 - over * per_sample - 1;
    }
  };
  const int n_units = 8 * q.cg * q.rw;                                 // per job
  const int stage_cg = q.rw * q.rws * 4;
  // which words a job loads: unit (channel, stored row, word) -> dword offset from (frame, first sample, first channel
  // of the job), top bit: outside the image; byte offset in the staging area
  const SmallDiv by_rw(q.rw), by_wws(q.wws), by_ch(8 * q.cg);
#pragma clang loop unroll(disable)
  for (int i = tid; i < (DIRECT ? 0 : q.parts * n_units); i += NT) {
    const int pc = by_rw.quot(i), rw = i - pc * q.rw;
    const int part = by_ch.quot(pc), ch = pc - part * 8 * q.cg;
    const int srow = by_wws.quot(rw), word = rw - srow * q.wws;
    const int row = part * q.lrp + (srow >> (q.srows - 1));
    int bsel, iy;
    input_row(row, bsel, iy);
    const bool inside = row < lr_used && iy >= 0 && iy < p.H;
    const int sy = p.pool ? 2 * iy + (srow & (q.srows - 1)) : iy;
    u32x2 u;
    u[0] = inside ? (uint32_t)((size_t)(bsel * Cin + ch) * in_chan + (size_t)sy * q.wws + word) : 0x80000000u;
    u[1] = row < lr_used ? (uint32_t)((ch >> 3) * stage_cg + (rw * q.rws + (ch & 7)) * 4) : kNone;
    unit[i] = u;
  }
  __syncthreads();

  // ---- the loader: a wave's jobs are wave, wave + loaders, ..  A job's words come in batches of kMidBatch chunks, a
  // chunk being 64 U units of up to KP frames; the registers of a batch are requested again as soon as it has been staged.
  // Every load of a chunk is issued, from an address inside the tensor, whatever the lane's word is for (a load under a
  // lane's condition makes the compiler wait for it at once); words outside the image and frames beyond the group become zero when they
  // are staged.
  constexpr int U = mid_units(KP);
  const int n_groups = p.G + (mp.K_last ? 1 : 0);
  auto frames_of = [&](int g) { return g == p.G ? mp.K_last : p.K; };
  const int n_uc = q.nb == 1 ? q.chunks : q.chunks / q.nb;
  uint32_t wd[kMidBatch][U][KP];
  // SPLIT: a wave that has one job of one batch in every group keeps what the tables say about it in registers
  const bool own_job = SPLIT && q.n_jobs <= 2 * q.loaders && q.batches == 1;
  u32x2 own_un[SPLIT ? kMidBatch : 1][U];
  if constexpr (SPLIT && !DIRECT) {
    if (own_job) {
#pragma unroll
      for (int c = 0; c < kMidBatch; ++c)
#pragma unroll
        for (int u = 0; u < U; ++u) {
          const int e = ((c < n_uc ? c : c % n_uc) * U + u) * 64 + lane;
          own_un[c][u] = unit[(wave & (q.parts - 1)) * n_units + min(e, n_units - 1)];
          if (e >= n_units) own_un[c][u][1] = kNone;
        }
    }
  }
  auto chunk_of = [&](int c, int& nb, int& uc) {
    nb = 0;
    uc = c;
    while (uc >= n_uc) { uc -= n_uc; ++nb; }
  };
  auto load_batch = [&](int g, int job, int batch) {
    const int Kg = frames_of(g), part = job & (q.parts - 1);
    const u32x2* const units = unit + part * n_units;
    const uint32_t* const base =
        p.spikes + (((size_t)g * p.K) * p.B + b0) * Cin * in_chan + (size_t)(job >> q.parts_shift) * q.cg * 8 * in_chan;
    uint32_t off[kMidBatch][U];
    int f0[kMidBatch];
#pragma unroll
    for (int c = 0; c < kMidBatch; ++c) {
      if (c > 0 && batch * kMidBatch + c >= q.chunks) break;           // (wave-uniform: small jobs have one or two chunks)
      int nb, uc;
      chunk_of(batch * kMidBatch + c, nb, uc);
      f0[c] = nb * KP;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (SPLIT && own_job) off[c][u] = own_un[c][u][0] & 0x7fffffffu;
        else off[c][u] = units[min((uc * U + u) * 64 + lane, n_units - 1)][0] & 0x7fffffffu;
      }
    }
#pragma unroll
    for (int c = 0; c < kMidBatch; ++c) {
      if (c > 0 && batch * kMidBatch + c >= q.chunks) break;
#pragma unroll
      for (int j = 0; j < KP; ++j) {
        const uint32_t* const frame = base + (size_t)min(f0[c] + j, Kg - 1) * t_stride;
#pragma unroll
        for (int u = 0; u < U; ++u) wd[c][u][j] = frame[off[c][u]];
      }
    }
  };
  auto store_batch = [&](int Kg, int job, int batch) {
    const u32x2* const units = unit + (job & (q.parts - 1)) * n_units;
    u32x2 un[kMidBatch][U];
    int f0[kMidBatch];
#pragma unroll
    for (int c = 0; c < kMidBatch; ++c) {
      int nb, uc;
      const int chunk = batch * kMidBatch + c;
      if (c > 0 && chunk >= q.chunks) break;
      chunk_of(chunk, nb, uc);
      f0[c] = nb * KP;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (SPLIT && own_job) {
          un[c][u] = own_un[c][u];
          continue;
        }
        const int e = (uc * U + u) * 64 + lane;
        un[c][u] = units[min(e, n_units - 1)];
        if (e >= n_units) un[c][u][1] = kNone;
      }
    }
#pragma unroll
    for (int c = 0; c < kMidBatch; ++c) {
      if (c > 0 && batch * kMidBatch + c >= q.chunks) break;
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const uint32_t keep = un[c][u][0] >> 31 ? 0u : 0xffffffffu;
#pragma unroll
        for (int j = 0; j < KP; ++j) wd[c][u][j] &= f0[c] + j < Kg ? keep : 0u;
        frames_to_fields<KP>(wd[c][u]);
        if (un[c][u][1] != kNone) {
          uint32_t* dst = reinterpret_cast<uint32_t*>(stage + un[c][u][1]) + f0[c] * 8;
#pragma unroll
          for (int j = 0; j < KP; ++j) dst[j * 8] = wd[c][u][j];
        }
      }
    }
  };
  const int job0 = min(wave, q.n_jobs - 1);

  // Groups of one or two frames on few channels: the words are few, and what the staging takes is its chain of LDS round trips
  // (8 -> 32 at 59 x 39, B = 17, 18 frames one by one: 52 us a call, of which staging 14, requests 8 and the passes over the
  // pixels 10; 33 us so.  16 -> 16 at 64 x 41, B = 37, TAC-TP K = 2, 12 frames: 57 -> 39 us).  A thread asks for the 8 words (times
  // two frames, or two rows with a pool on load) of each of its pixels one group ahead and keeps what it needs to know
  // about them in registers.
  static_assert(!DIRECT || KP <= 2, "groups of one or two frames");
  uint32_t dw[kMidDirect][2][8], d_off[kMidDirect], d_dst[kMidDirect];  // dw: two frames, or two rows of the pool
  auto load_direct = [&](int g) {
    if constexpr (DIRECT) {
      const uint32_t* const base = p.spikes + (((size_t)g * p.K) * p.B + b0) * Cin * in_chan;
      const size_t second = KP == 2 ? (frames_of(g) > 1 ? t_stride : 0) : p.pool ? (size_t)q.wws : 0;
#pragma unroll
      for (int i = 0; i < kMidDirect; ++i) {
        if (i > 0 && i * NT >= C8 * q.lr * p.W) break;        // (uniform)
        const uint32_t* const src = base + (d_off[i] & 0x7fffffffu);
#pragma unroll
        for (int c = 0; c < 8; ++c) dw[i][0][c] = src[c * in_chan];
        if (KP == 2 || p.pool) {
#pragma unroll
          for (int c = 0; c < 8; ++c) dw[i][1][c] = src[second + c * in_chan];
        }
      }
    }
  };
  if constexpr (DIRECT) {
    const SmallDiv by_w(p.W), by_lr(q.lr);
#pragma unroll
    for (int i = 0; i < kMidDirect; ++i) {
      const int e = tid + i * NT, line = by_w.quot(min(e, C8 * q.lr * p.W - 1));
      const int x = min(e, C8 * q.lr * p.W - 1) - line * p.W, cg = by_lr.quot(line), row = line - cg * q.lr;
      int bsel, iy;
      input_row(row, bsel, iy);
      const bool used = e < C8 * q.lr * p.W && row < lr_used, inside = used && iy >= 0 && iy < p.H;
      const int xs = p.pool ? 2 * x : x, xp = x + 1;
      d_off[i] = inside ? (uint32_t)((size_t)(bsel * Cin + cg * 8) * in_chan + (size_t)(p.pool ? 2 * iy : iy) * q.wws + (xs >> 5)) : 0x80000000u;
      d_dst[i] = used ? (uint32_t)(cg * (F32 ? 2 : 1) * q.plane + (row * q.wpx + (S == 1 ? xp : (xp & 1) * q.xh + (xp >> 1))) * 16) | (uint32_t)(xs & 31) << 24
                      : kNone;
    }
    load_direct(0);
  } else {
    load_batch(0, job0, 0);
  }

  // which pixels a job forms: byte offset of the pixel's class words, shift of its field (top byte); byte offset in LDS
  // from the job's first plane
  const SmallDiv by_w(p.W), by_lrp(q.lrp), by_cg(q.cg);
  const int n_px = q.cg * q.lrp * p.W;                                 // per job
#pragma clang loop unroll(disable)
  for (int i = tid; i < (DIRECT ? 0 : q.parts * n_px); i += NT) {
    const int line = by_w.quot(i), x = i - line * p.W;                 // (part, channel group, row)
    const int pcg = by_lrp.quot(line), rl = line - pcg * q.lrp;
    const int part = by_cg.quot(pcg), cg = pcg - part * q.cg, row = part * q.lrp + rl;
    const int xs = p.pool ? 2 * x : x;
    const int c = xs & (KP - 1), xp = x + 1;
    u32x2 u;
    u[0] = (uint32_t)(cg * stage_cg + ((rl * q.srows * q.wws + (xs >> 5)) * q.rws + c * 8) * 4) | ((uint32_t)((xs & 31) - c) << 24);
    u[1] = row < lr_used ? (uint32_t)(cg * (F32 ? 2 : 1) * q.plane + (row * q.wpx + (S == 1 ? xp : (xp & 1) * q.xh + (xp >> 1))) * 16) : kNone;
    pxt[i] = u;
  }
  // the padding columns x = -1 and x = W stay zero
  const SmallDiv by_lr(q.lr), by_cin(Cin);
#pragma clang loop unroll(disable)
  for (int i = tid; i < C8 * (F32 ? 2 : 1) * q.lr * 2; i += NT) {
    const int side = i & 1, pl = by_lr.quot(i >> 1), r = (i >> 1) - pl * q.lr;
    const int xp = side ? p.W + 1 : 0;
    *reinterpret_cast<u32x4*>(lds + pl * q.plane + (r * q.wpx + (S == 1 ? xp : (xp & 1) * q.xh + (xp >> 1))) * 16) = u32x4{0, 0, 0, 0};
  }
  // slot table: k-step ks, lane half hh -> byte offset of its channels (tap, cin) from the window's first pixel.  Slots
  // beyond 9 Cin meet zero weights; entries behind the last step are only ever fetched ahead.
#pragma clang loop unroll(disable)
  for (int i = tid; i < q.nks * 2 + kMidTabPad; i += NT) {
    const int kk0 = F32 ? i : 8 * i;                                   // fp32: k-step i / 2, lane half i % 2 -> slot i
    const int tap = by_cin.quot(kk0), cin = kk0 - tap * Cin;
    const int ky = (tap * 11) >> 5, kx = tap - ky * 3;                 // tap / 3 for the nine taps
    const int col = S == 1 ? kx : (kx & 1) * q.xh + (kx >> 1);
    const int ch = F32 ? (cin >> 2) * q.plane + (cin & 3) * 4 : (cin >> 3) * q.plane;
    tab[i] = tap < 9 ? ch + (ky * q.wpx + col) * 16 : 0;
  }
  uint32_t* const wq = reinterpret_cast<uint32_t*>(lds + q.off_wq);    // read with lane-dependent indices below
  if (tid < TAC_MAX_K) wq[tid] = p.wq[tid];
  if (tid < NCO * NMC * 32) bias_all[tid] = (p.bias && co_first + tid < p.Cout) ? p.bias[co_first + tid] : 0.f;
  // aggregates by frame bits: pairs of channels as two bf16 (groups of up to four frames), one bf16 (up to eight), or
  // 2^-23 fixed-point sums per chunk of eight frames (more frames, the mean pool's counts, fp32)
  const bool sums = F32 || q.nb > 1 || p.pool == 1;
  const float scale = p.pool == 1 ? 0.25f / (float)(1u << kFixShift) : 1.0f / (float)(1u << kFixShift);
  auto make_lut = [&](int first) {                                     // first: weight index of the group's first frame
    const int n_lut = sums ? q.nb << KP : KP == 8 ? 256 : 1 << (2 * KP);
#pragma clang loop unroll(disable)
    for (int i = tid; i < n_lut; i += NT) {
      // low KP bits: a channel's frames; the bits above: the pair's second channel, or the chunk of frames
      uint32_t a[2] = {0, 0};
      const int second = sums || KP == 8 ? 0 : i >> KP, j0 = first + (sums ? (i >> KP) * KP : 0);
#pragma unroll
      for (int j = 0; j < KP; ++j) {
        const uint32_t w = wq[min(j0 + j, TAC_MAX_K - 1)];
        a[0] += (i >> j) & 1 ? w : 0u;
        a[1] += (second >> j) & 1 ? w : 0u;
      }
      lut[i] = sums ? a[0] : pack_bf16((float)a[0] * scale, (float)a[1] * scale);
    }
  };

  // ---- the lane's pixels.  Their membranes are 32-bit byte offsets from the wave's; without a second sample in the tile they are
  // counted from the tile's first row, which keeps planes of up to 2^28 neurons in reach.
  const int v_row = q.flatten ? 0 : oy0;
  LaneGeom lg;
  uint32_t pix_base[NNP];
  const int word_w = SPLIT || q.wb == 1 ? 0 : px4 & 1;
  const int rg_w = SPLIT ? px_wave : (q.wb == 1 ? px4 : px4 >> 1) * NNP;      // the wave's first row group; block np: row group + np
#pragma unroll
  for (int np = 0; np < 2; ++np) { lg.ok[np] = false; lg.theta[np] = __builtin_inff(); lg.v_off[np] = 0; }
#pragma unroll
  for (int np = 0; np < NNP; ++np) {
    const int rr0 = (rg_w + np) * q.rpb + (n >> q.pw_shift), ox = word_w * 32 + (n & ((1 << q.pw_shift) - 1));
    const bool ok = rg_w + np < q.trg && rr0 < rows_valid && ox < p.Wo;
    const int rr = ok ? rr0 : 0;
    const int bsel = sample_of(rr), oy = oy0 + rr - bsel * p.Ho;
    lg.ok[np] = ok;
    lg.theta[np] = ok ? p.theta : __builtin_inff();
    lg.v_off[np] = (uint32_t)((((size_t)bsel * p.Cout + 4 * h) * plane + (size_t)(oy - v_row) * p.Wo + (ok ? ox : 0)) * 4);
    pix_base[np] = (uint32_t)(((rr * S + bsel * (3 - S)) * q.wpx + (ok ? ox : 0)) * 16);
  }
  lg.co_lim = p.Cout - co0 - 4 * h;
  const size_t v_wave = ((size_t)b0 * p.Cout + co0) * plane + (size_t)v_row * p.Wo;
  const bool wave_active = rg_w < q.trg && rg_w * q.rpb < rows_valid && (NCO == 1 || co0 < p.Cout);      // wave-uniform

  constexpr int kRegs = 16 / kShare;         // registers of a block that the wave steps, from r0 on
  const int r0 = SPLIT ? k_part * kRegs : 0;
  float V[NMC][NNP][kRegs];
#pragma unroll
  for (int mc = 0; mc < NMC; ++mc)
#pragma unroll
    for (int np = 0; np < NNP; ++np)
#pragma unroll
      for (int r = 0; r < kRegs; ++r) V[mc][np][r] = 0.f;
  if (p.v_inout) {
#pragma unroll
    for (int mc = 0; mc < NMC; ++mc)
#pragma unroll
      for (int np = 0; np < NNP; ++np)
#pragma unroll
        for (int r = 0; r < kRegs; ++r) {
          const int c = mc * 32 + 8 * ((r0 + r) >> 2) + ((r0 + r) & 3);
          if (lg.ok[np] && c < lg.co_lim)
            V[mc][np][r] = *reinterpret_cast<const float*>(reinterpret_cast<const char*>(p.v_inout + v_wave) +
                                                           (size_t)c * plane * 4 + lg.v_off[np]);
        }
  }

  // ---- output words: lane (r << 2) | (hi << 1) | np holds channel 8 (r / 4) + 4 hi + r % 4, pixel block np.  SPLIT: lane 2 kRegs j + 2 i + hi,
  // register r0 + i of the j-th step in hand
  const int st_r = SPLIT ? r0 + ((lane % (2 * kRegs)) >> 1) : lane >> 2, st_hi = SPLIT ? lane & 1 : (lane >> 1) & 1, st_np = SPLIT ? 0 : lane & 1;
  const int st_co = co0 + 8 * (st_r >> 2) + 4 * st_hi + (st_r & 3);
  const int Wwo = (p.Wo + 31) >> 5;
  const int st_rr = (rg_w + st_np) * q.rpb;                            // the block's first tile row
  const bool st_ok = st_np < NNP && rg_w + st_np < q.trg && (!SPLIT || lane < 8 * kRegs);
  const int st_bsel = sample_of(st_rr), st_b = b0 + st_bsel, st_oy = oy0 + st_rr - st_bsel * p.Ho;
  const int out_rows = p.out_pool ? p.Ho >> 1 : p.Ho;                  // stored rows and words per channel
  const int out_words = p.out_pool ? 1 : Wwo;
  const size_t out_step = (size_t)p.B * p.Cout * out_rows * out_words;
  const int st_row = p.out_pool ? st_oy >> 1 : st_oy;
  // word offset of the block's first row within a step, and what the row behind a sample's last one adds to the next row
  const uint32_t st_off = (uint32_t)((((size_t)st_b * p.Cout + st_co) * out_rows + st_row) * out_words);
  const uint32_t next_sample = (uint32_t)((p.Cout - 1) * out_rows * out_words);
  const int st_rows = st_ok ? min(q.rpb, rows_valid - st_rr) : 0;      // rows of the block
  const uint32_t field = q.rpb > 1 ? (1u << (32 / q.rpb)) - 1u : 0xffffffffu;
  auto store_words = [&](size_t step, const uint32_t (&word)[NMC][2]) {
    uint32_t* const out = p.out + step * out_step;
#pragma unroll
    for (int mc = 0; mc < NMC; ++mc) {
      const bool ok = st_co + mc * 32 < p.Cout;
      const uint32_t wd = word[mc][0];
      uint32_t at = st_off + (uint32_t)(mc * 32 * out_rows * out_words);
      if (!p.out_pool) {
        at += word_w;
        if (q.rpb == 1) {
          if (ok && st_rows > 0) out[at] = wd;
          continue;
        }
        for (int s = 0, row = st_row; s < q.rpb; ++s, ++at) {
          if (ok && s < st_rows) out[at] = (wd >> (s << q.pw_shift)) & field;
          if (++row == out_rows) { row = 0; at += next_sample; }
        }
      } else if (q.rpb > 1) {
        // 2 x 2 max pool: both rows of a window are in the lane's word (rows per sample are even)
        for (int s = 0, row = st_row; s < q.rpb; s += 2, ++at) {
          const uint32_t two = (wd >> (s << q.pw_shift)) | (wd >> ((s + 1) << q.pw_shift));
          if (ok && s < st_rows) out[at] = pool_pairs(two & field);
          if (++row == out_rows) { row = 0; at += next_sample; }
        }
      } else {
        // the wave's two blocks are the two rows of a pooled row (NNP = 2): neighbouring lanes; 16 pooled pixels per
        // word of the unpooled row
        const uint32_t pooled = pool_pairs(wd | (uint32_t)__shfl_xor((int)wd, 1, 64));
        if (ok && st_np == 0 && st_rows > 0) {
          if (q.wb == 1) out[at] = pooled;
          else reinterpret_cast<uint16_t*>(out + at)[word_w] = (uint16_t)pooled;
        }
      }
    }
  };

  // the right-hand neighbour's field stands at the same bit of the next class word (single frames: at the next bit)
  auto right = [](int corner) { return KP == 1 ? 0 : (corner & 1) * 8; };
  // max pool on load: the other three pixels of the block are OR-ed to the first one's class words
  auto or_corners = [&]<int PX>(const u32x2 (&px)[PX], int nb, u32x4 (&c0)[PX], u32x4 (&c1)[PX]) {
    for (int corner = 1; corner < 4; ++corner)
#pragma unroll
      for (int k = 0; k < PX; ++k) {
        const uint8_t* sk = stage + (px[k][0] & 0xffffffu) + ((corner >> 1) * q.wws * q.rws + nb * KP * 8 + right(corner)) * 4;
        c0[k] |= *reinterpret_cast<const u32x4*>(sk) >> (KP == 1 ? corner & 1 : 0);
        c1[k] |= *reinterpret_cast<const u32x4*>(sk + 16) >> (KP == 1 ? corner & 1 : 0);
      }
  };
  // the pixels of a job, PX per lane at a time: all reads of a stage before the next (table address, class words, table,
  // tile), so that PX chains of LDS latencies overlap
  // (Single frames have two aggregates, 0 and the weight: a mask and the weight take the place of the table: two layers at
  // 26 x 26 in fp32 160 -> 149 us.)
  const uint32_t one = KP != 1 ? 0u : sums ? p.wq[0] : pack_bf16((float)p.wq[0] * scale, (float)p.wq[0] * scale);
  u32x2 own_px[2];
  auto build_job = [&](int job) {
    uint8_t* const pl = lds + (job >> q.parts_shift) * q.cg * (F32 ? 2 : 1) * q.plane;
    const u32x2* const px_part = pxt + (job & (q.parts - 1)) * n_px;
    if (!sums) {
      auto pass = [&]<int PX>(std::integral_constant<int, PX>, int e0) {
        u32x2 px[PX];
        u32x4 c0[PX], c1[PX], v[PX];
#pragma unroll
        for (int k = 0; k < PX; ++k) {
          if (SPLIT && PX <= 2 && own_job && n_px <= 128) {
            px[k] = own_px[k];
            continue;
          }
          px[k] = px_part[min(e0 + 64 * k, n_px - 1)];
          if (e0 + 64 * k >= n_px) px[k][1] = kNone;
        }
#pragma unroll
        for (int k = 0; k < PX; ++k) {
          const uint8_t* src = stage + (px[k][0] & 0xffffffu);
          c0[k] = *reinterpret_cast<const u32x4*>(src);
          c1[k] = *reinterpret_cast<const u32x4*>(src + 16);
        }
        if (p.pool == 2) or_corners(px, 0, c0, c1);
#pragma unroll
        for (int k = 0; k < PX; ++k) {
          const uint32_t sh = px[k][0] >> 24;
#pragma unroll
          for (int c2 = 0; c2 < 4; ++c2) {
            if constexpr (KP == 1) {
              const uint32_t m0 = 0u - __builtin_amdgcn_ubfe(c2 < 2 ? c0[k][2 * c2] : c1[k][2 * c2 - 4], sh, 1);
              const uint32_t m1 = 0u - __builtin_amdgcn_ubfe(c2 < 2 ? c0[k][2 * c2 + 1] : c1[k][2 * c2 - 3], sh, 1);
              v[k][c2] = one & ((m0 & 0xffffu) | (m1 << 16));
              continue;
            }
            const uint32_t lo = __builtin_amdgcn_ubfe(c2 < 2 ? c0[k][2 * c2] : c1[k][2 * c2 - 4], sh, KP);
            const uint32_t hi = __builtin_amdgcn_ubfe(c2 < 2 ? c0[k][2 * c2 + 1] : c1[k][2 * c2 - 3], sh, KP);
            if constexpr (KP == 8) v[k][c2] = lut[lo] | (lut[hi] << 16);
            else v[k][c2] = lut[lo | (hi << KP)];
          }
        }
#pragma unroll
        for (int k = 0; k < PX; ++k)
          if (px[k][1] != kNone) *reinterpret_cast<u32x4*>(pl + px[k][1]) = v[k];
      };
      int e0 = lane;
      if constexpr (KP == 1) {
        for (; e0 - lane + 64 < n_px; e0 += 128) pass(std::integral_constant<int, 2>{}, e0);
      } else {
        // (128 pixels of a job are a pass of two)
        for (; e0 - lane + 128 < n_px; e0 += 256) pass(std::integral_constant<int, 4>{}, e0);
        if (e0 - lane + 64 < n_px) {
          pass(std::integral_constant<int, 2>{}, e0);
          e0 += 128;
        }
      }
      if (e0 - lane < n_px) pass(std::integral_constant<int, 1>{}, e0);                  // 64 or fewer are left
      return;
    }
    constexpr int PX = KP == 1 ? 1 : 2;        // (without lookups there is little to overlap)
    for (int e0 = lane; e0 < n_px; e0 += 64 * PX) {
      u32x2 px[PX];
      uint32_t a[PX][8];
#pragma unroll
      for (int k = 0; k < PX; ++k) {
        px[k] = px_part[min(e0 + 64 * k, n_px - 1)];
        if (e0 + 64 * k >= n_px) px[k][1] = kNone;
#pragma unroll
        for (int c = 0; c < 8; ++c) a[k][c] = 0;
      }
      const int corners = p.pool == 1 ? 4 : 1;                         // mean pool: the sum over the block's four pixels
      for (int nb = 0; nb < q.nb; ++nb)
        for (int corner = 0; corner < corners; ++corner) {
          [[maybe_unused]] const uint32_t* const tb = lut + (nb << KP);
          u32x4 c0[PX], c1[PX];
#pragma unroll
          for (int k = 0; k < PX; ++k) {
            const uint8_t* sk = stage + (px[k][0] & 0xffffffu) + ((corner >> 1) * q.wws * q.rws + nb * KP * 8 + right(corner)) * 4;
            c0[k] = *reinterpret_cast<const u32x4*>(sk);
            c1[k] = *reinterpret_cast<const u32x4*>(sk + 16);
          }
          if (p.pool == 2) or_corners(px, nb, c0, c1);
#pragma unroll
          for (int k = 0; k < PX; ++k)
#pragma unroll
            for (int c = 0; c < 8; ++c) {
              const uint32_t bits = __builtin_amdgcn_ubfe(c < 4 ? c0[k][c] : c1[k][c - 4], (px[k][0] >> 24) + (KP == 1 ? corner & 1 : 0), KP);
              if constexpr (KP == 1) a[k][c] += one & (0u - bits);
              else a[k][c] += tb[bits];
            }
        }
#pragma unroll
      for (int k = 0; k < PX; ++k) {
        if (px[k][1] == kNone) continue;
        uint8_t* const dst = pl + px[k][1];
        if constexpr (F32) {
          // the fixed-point sum is exact; one rounding to fp32
          *reinterpret_cast<f32x4v*>(dst) = f32x4v{(float)a[k][0] * scale, (float)a[k][1] * scale, (float)a[k][2] * scale, (float)a[k][3] * scale};
          *reinterpret_cast<f32x4v*>(dst + q.plane) = f32x4v{(float)a[k][4] * scale, (float)a[k][5] * scale, (float)a[k][6] * scale, (float)a[k][7] * scale};
        } else {
          u32x4 v;
#pragma unroll
          for (int c2 = 0; c2 < 4; ++c2) v[c2] = pack_bf16((float)a[k][2 * c2] * scale, (float)a[k][2 * c2 + 1] * scale);
          *reinterpret_cast<u32x4*>(dst) = v;
        }
      }
    }
  };

  auto build_direct = [&](int Kg) {
    if constexpr (DIRECT) {
      const uint32_t w0 = p.wq[p.K - Kg], w1 = KP == 2 && Kg == 2 ? p.wq[1] : 0u;
#pragma unroll
      for (int i = 0; i < kMidDirect; ++i) {
        if (i > 0 && i * NT >= C8 * q.lr * p.W) break;
        const uint32_t keep = d_off[i] >> 31 ? 0u : 0xffffffffu, sh = d_dst[i] >> 24 & 31;
        uint32_t a[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
          const uint32_t f0 = dw[i][0][c] & keep, f1 = dw[i][1][c] & keep;
          if (KP == 2) {
            a[c] = ((0u - __builtin_amdgcn_ubfe(f0, sh, 1)) & w0) + ((0u - __builtin_amdgcn_ubfe(f1, sh, 1)) & w1);
          } else if (!p.pool) {
            a[c] = (0u - __builtin_amdgcn_ubfe(f0, sh, 1)) & w0;
          } else {
            const uint32_t top = __builtin_amdgcn_ubfe(f0, sh, 2), bottom = __builtin_amdgcn_ubfe(f1, sh, 2);
            a[c] = p.pool == 1 ? __umul24(__popc(top | bottom << 2), w0) : (top | bottom) ? w0 : 0u;
          }
        }
        if (d_dst[i] == kNone) continue;
        uint8_t* const dst = lds + (d_dst[i] & 0xffffffu);
        if constexpr (F32) {
          *reinterpret_cast<f32x4v*>(dst) = f32x4v{(float)a[0] * scale, (float)a[1] * scale, (float)a[2] * scale, (float)a[3] * scale};
          *reinterpret_cast<f32x4v*>(dst + q.plane) = f32x4v{(float)a[4] * scale, (float)a[5] * scale, (float)a[6] * scale, (float)a[7] * scale};
        } else {
          u32x4 v;
#pragma unroll
          for (int c2 = 0; c2 < 4; ++c2) v[c2] = pack_bf16((float)a[2 * c2] * scale, (float)a[2 * c2 + 1] * scale);
          *reinterpret_cast<u32x4*>(dst) = v;
        }
      }
    }
  };

  // SPLIT: where the wave's k-steps find their channels and taps
  int32_t tab_own[kOwn][SPLIT ? kMidRangeSteps : 1];
  if constexpr (SPLIT) {
    __syncthreads();                           // the tables
    if (!DIRECT && own_job) {
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        own_px[k] = pxt[(wave & (q.parts - 1)) * n_px + min(lane + 64 * k, n_px - 1)];
        if (lane + 64 * k >= n_px) own_px[k][1] = kNone;
      }
    }
#pragma unroll
    for (int i = 0; i < kOwn; ++i)
#pragma unroll
      for (int k = 0; k < kMidRangeSteps; ++k) tab_own[i][k] = tab[2 * min(range_start(i) + k, q.nks - 1) + h];
  }
  size_t step = 0;
  for (int g = 0; g < n_groups; ++g) {
    const bool last = g == p.G;                // the shorter last group
    const int Kg = frames_of(g), n_lif = last ? mp.n_lif_last : p.n_lif;
    const float decay = last ? mp.decay_last : p.decay;
    if (!SPLIT) __syncthreads();               // the previous group's fragment reads are done (first group: the tables are made)
    if ((g == 0 || last) && !DIRECT) {
      make_lut(last ? p.K - mp.K_last : 0);    // a shorter last group's weights are the last of a whole group's
      __syncthreads();
    }
    // ---- 1. aggregate
    if constexpr (DIRECT) {
      build_direct(Kg);
      load_direct(min(g + 1, n_groups - 1));     // behind the last group it is asked for again
    }
    const int loaders = NT / 256 * q.loaders;
    for (int job = wave; !DIRECT && job < q.n_jobs && wave < loaders; job += loaders) {
      for (int batch = 0; batch < q.batches; ++batch) {
        store_batch(Kg, job, batch);
        const bool more = batch + 1 < q.batches, next_job = job + loaders < q.n_jobs;
        // what to request next; behind the last batch of the call any batch will do
        load_batch(more || next_job ? g : min(g + 1, n_groups - 1), more ? job : next_job ? job + loaders : job0, more ? batch + 1 : 0);
      }
      asm volatile("" ::: "memory");           // the wave's own LDS accesses execute in order; keep the compiler to it too
      build_job(job);
      asm volatile("" ::: "memory");
    }
    if (!SPLIT && g == 0) lds_dma_wait();      // the weights
    __syncthreads();
    if constexpr (SPLIT) {
      // ---- 2. this wave's k-steps
      if (wave_active) {
        f32x16 sum[kOwn];
#pragma unroll
        for (int i = 0; i < kOwn; ++i) {
          const int k0 = range_start(i), n_k = range_start(i + 1) - k0;
          bf16x8 af[kMidRangeSteps];
#pragma unroll
          for (int k = 0; k < kMidRangeSteps; ++k) af[k] = *reinterpret_cast<const bf16x8*>(lds + pix_base[0] + (uint32_t)tab_own[i][k]);
#pragma unroll
          for (int r = 0; r < 16; ++r) sum[i][r] = 0.f;
#pragma unroll
          for (int k = 0; k < kMidRangeSteps; ++k)
            if (k < n_k) sum[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w_own[i][k], af[k], sum[i], 0, 0, 0);
        }
#pragma unroll
        for (int d = 1; d < kOwn; d *= 2)
#pragma unroll
          for (int i = 0; i + d < kOwn; i += 2 * d)
#pragma unroll
            for (int r = 0; r < 16; ++r) sum[i][r] += sum[i + d][r];
        f32x2* const part = reinterpret_cast<f32x2*>(lds + q.off_part) + wave * 512 + lane;        // [wave][register pair][lane]
#pragma unroll
        for (int r2 = 0; r2 < 8; ++r2) part[r2 * 64] = f32x2{sum[0][2 * r2], sum[0][2 * r2 + 1]};
      }
      __syncthreads();
      if (!wave_active) { step += n_lif; continue; }
      // ---- 3. the block's partial sums of the wave's registers, LIF steps
      float y[kRegs];
      {
        f32x2 in[SPLIT][kRegs / 2];
        const f32x2* const part = reinterpret_cast<const f32x2*>(lds + q.off_part) + px_wave * SPLIT * 512 + (r0 / 2) * 64 + lane;
#pragma unroll
        for (int k = 0; k < SPLIT; ++k)
#pragma unroll
          for (int r2 = 0; r2 < kRegs / 2; ++r2) in[k][r2] = part[k * 512 + r2 * 64];
#pragma unroll
        for (int d = 1; d < SPLIT; d *= 2)
#pragma unroll
          for (int k = 0; k + d < SPLIT; k += 2 * d)
#pragma unroll
            for (int r2 = 0; r2 < kRegs / 2; ++r2) {
              in[k][r2][0] += in[k + d][r2][0];
              in[k][r2][1] += in[k + d][r2][1];
            }
#pragma unroll
        for (int r = 0; r < kRegs; ++r) y[r] = in[0][r >> 1][r & 1] + bias_lds[8 * ((r0 + r) >> 2) + 4 * h + ((r0 + r) & 3)];
      }
      // up to four steps' words are gathered, 2 kRegs lanes each, and stored together: a step of two or four registers is shorter than
      // what leads to its store
      for (int j0 = 0; j0 < n_lif; j0 += 4) {
        uint32_t word[1][2] = {{0u, 0u}};
        static_for<0, 4>([&](auto j_) {
          constexpr int j = decltype(j_)::value;
          if (j > 0 && j0 + j >= n_lif) return;                        // (uniform)
          [[maybe_unused]] char* const tl = reinterpret_cast<char*>(p.v_trace + (step + j) * ((size_t)p.B * p.Cout * plane) + v_wave);
          static_for<0, kRegs / 2>([&](auto r2_) {
            constexpr int r = decltype(r2_)::value * 2;
            float v[2];
            uint64_t m[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
              v[i] = fmaf(decay, V[0][0][r + i], y[r + i]);
              m[i] = __builtin_amdgcn_ballot_w64(v[i] >= lg.theta[0]);
            }
            const uint32_t x[2][2] = {{(uint32_t)m[0], (uint32_t)(m[0] >> 32)}, {(uint32_t)m[1], (uint32_t)(m[1] >> 32)}};
            word[0][0] = write_lanes<j * 2 * kRegs + 2 * r, 2, 1>(word[0][0], x);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
              V[0][0][r + i] = __builtin_amdgcn_inverse_ballot_w64(m[i]) ? v[i] - p.theta : v[i];
              const int c = 8 * ((r0 + r + i) >> 2) + ((r0 + r + i) & 3);
              if (TRACE && lg.ok[0] && c < lg.co_lim) *reinterpret_cast<float*>(tl + (size_t)c * plane * 4 + lg.v_off[0]) = v[i];
            }
          });
        });
        if (lane < 2 * kRegs * (n_lif - j0)) store_words(step + lane / (2 * kRegs), word);
        step += min(4, n_lif - j0);
      }
      continue;
    } else {
      if (!wave_active) { step += n_lif; continue; }
      // ---- 2. contraction
      f32x16 acc[NMC][NNP];
#pragma unroll
      for (int mc = 0; mc < NMC; ++mc)
#pragma unroll
        for (int np = 0; np < NNP; ++np)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[mc][np][r] = bias_lds[mc * 32 + 8 * (r >> 2) + 4 * h + (r & 3)];
      const int32_t* const tabh = tab + h;
      if constexpr (F32) {
        // Four partial sums per output (k-steps ks % 4), added at the end: the rounding error of a long fp32 sum grows
        // with its length, and a quarter of the length keeps the membrane within the fp32 bar where one chain of
        // 9 Cin terms does not.
        f32x16 part[3][NNP];
#pragma unroll
        for (int i = 0; i < 3; ++i)
#pragma unroll
          for (int np = 0; np < NNP; ++np)
#pragma unroll
            for (int r = 0; r < 16; ++r) part[i][np][r] = 0.f;
        // nks is a multiple of 4 (9 Cin / 2, Cin a multiple of 8); operands of four steps are fetched ahead
        float wf[2][4], af[2][4][NNP];
        int32_t off[4];
        auto fetch = [&](int ks, float (&w)[4], float (&a)[4][NNP]) {
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            w[i] = *reinterpret_cast<const float*>(w_lds + ((ks + i) * 64 + lane) * 4);
#pragma unroll
            for (int np = 0; np < NNP; ++np) a[i][np] = *reinterpret_cast<const float*>(lds + pix_base[np] + (uint32_t)off[i]);
          }
        };
        auto offsets = [&](int ks) {
#pragma unroll
          for (int i = 0; i < 4; ++i) off[i] = tabh[2 * (ks + i)];
        };
        auto multiply = [&](const float (&w)[4], const float (&a)[4][NNP]) {
#pragma unroll
          for (int np = 0; np < NNP; ++np) {
            acc[0][np] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[0], a[0][np], acc[0][np], 0, 0, 0);
            part[0][np] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[1], a[1][np], part[0][np], 0, 0, 0);
            part[1][np] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[2], a[2][np], part[1][np], 0, 0, 0);
            part[2][np] = __builtin_amdgcn_mfma_f32_32x32x2f32(w[3], a[3][np], part[2][np], 0, 0, 0);
          }
        };
        // eight steps a turn and no way out of its middle (the accumulators would change registers on every turn); behind the last
        // step the last four are fetched again
        offsets(0);
        fetch(0, wf[0], af[0]);
        offsets(min(4, q.nks - 4));
        int ks = 0;
        for (; ks + 8 <= q.nks; ks += 8) {
          fetch(ks + 4, wf[1], af[1]);
          offsets(min(ks + 8, q.nks - 4));
          __builtin_amdgcn_sched_barrier(0);               // in front of the MFMAs: else they wait for reads just issued
          multiply(wf[0], af[0]);
          __builtin_amdgcn_sched_barrier(0);
          fetch(min(ks + 8, q.nks - 4), wf[0], af[0]);
          offsets(min(ks + 12, q.nks - 4));
          __builtin_amdgcn_sched_barrier(0);
          multiply(wf[1], af[1]);
          __builtin_amdgcn_sched_barrier(0);
        }
        if (ks < q.nks) multiply(wf[0], af[0]);
#pragma unroll
        for (int np = 0; np < NNP; ++np)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[0][np][r] = (acc[0][np][r] + part[0][np][r]) + (part[1][np][r] + part[2][np][r]);
      } else {
        // fragments are requested F - 1 steps ahead, table offsets F steps before that; beyond the last step the fetches read
        // what lies behind the weights (inside the LDS) and nobody uses it
        constexpr int F = mid_depth(NMC, NNP);
        bf16x8 af[F][NNP], wf[F][NMC];
        int32_t off[F];
        const uint8_t* const w_lane = w_lds + lane * 16;
        auto fetch = [&](int ks, int set) {
#pragma unroll
          for (int mc = 0; mc < NMC; ++mc) wf[set][mc] = *reinterpret_cast<const bf16x8*>(w_lane + (ks * NMC + mc) * 1024);
#pragma unroll
          for (int np = 0; np < NNP; ++np) af[set][np] = *reinterpret_cast<const bf16x8*>(lds + pix_base[np] + (uint32_t)off[set]);
          off[set] = tabh[2 * (ks + F)];
        };
#pragma unroll
        for (int d = 0; d < F; ++d) off[d] = tabh[2 * d];
#pragma unroll
        for (int d = 0; d < F - 1; ++d) fetch(d, d);
        auto multiply = [&](int set) {
#pragma unroll
          for (int mc = 0; mc < NMC; ++mc)
#pragma unroll
            for (int np = 0; np < NNP; ++np)
              acc[mc][np] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[set][mc], af[set][np], acc[mc][np], 0, 0, 0);
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
      }
      // ---- 3. LIF steps on Y_k = acc (bias included)
      for (int j = 0; j < n_lif; ++j, ++step) {
        uint32_t word[NMC][2];
#pragma unroll
        for (int mc = 0; mc < NMC; ++mc) word[mc][0] = word[mc][1] = 0u;
        float* tl = TRACE ? p.v_trace + step * ((size_t)p.B * p.Cout * plane) + v_wave : nullptr;
        lif_step<NMC, 64, TRACE, NNP>(V, acc, decay, p.theta, lg, word, tl, plane);
        store_words(step, word);
      }
    }
  }

  if (p.v_inout) {
#pragma unroll
    for (int mc = 0; mc < NMC; ++mc)
#pragma unroll
      for (int np = 0; np < NNP; ++np)
#pragma unroll
        for (int r = 0; r < kRegs; ++r) {
          const int c = mc * 32 + 8 * ((r0 + r) >> 2) + ((r0 + r) & 3);
          if (lg.ok[np] && c < lg.co_lim)
            *reinterpret_cast<float*>(reinterpret_cast<char*>(p.v_inout + v_wave) + (size_t)c * plane * 4 + lg.v_off[np]) =
                V[mc][np][r];
        }
  }
}

template <int KP, int NMC, int NNP, bool TRACE, bool F32, int SPLIT = 0, int NCO = 1>
hipError_t mid_launch_t(const MidParams& p, hipStream_t s) {
  auto kern = &mid_kernel<KP, NMC, NNP, TRACE, F32, false, SPLIT, NCO>;
  if constexpr (KP <= 2 && NCO == 1) {
    if (p.q.direct) kern = &mid_kernel<KP, NMC, NNP, TRACE, F32, true, SPLIT>;
  }
  if (p.q.total > 64 * 1024) {
    hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
  }
  const dim3 grid((unsigned)p.q.row_tiles * (unsigned)p.q.co_tiles, 1, p.q.flatten ? 1 : p.m.B);
  hipLaunchKernelGGL(kern, grid, dim3(SPLIT ? 512 : kMidThreads * NCO), p.q.total, s, p);
  return hipGetLastError();
}

template <int KP, bool TRACE>
hipError_t mid_launch_bf16_kp(const MidParams& p, int nmc, int nnp, hipStream_t s) {
  if (p.q.split == 8) return mid_launch_t<KP, 1, 1, TRACE, false, 8>(p, s);
  if (p.q.split == 4) return mid_launch_t<KP, 1, 1, TRACE, false, 4>(p, s);
  if (nmc == 1) return nnp == 1 ? mid_launch_t<KP, 1, 1, TRACE, false>(p, s) : mid_launch_t<KP, 1, 2, TRACE, false>(p, s);
  return nnp == 1 ? mid_launch_t<KP, 2, 1, TRACE, false>(p, s) : mid_launch_t<KP, 2, 2, TRACE, false>(p, s);
}

template <int KP, bool TRACE>
hipError_t mid_launch_f32_kp(const MidParams& p, int nnp, hipStream_t s) {
  if constexpr (KP >= 2) {
    if (p.q.nco == 2) return mid_launch_t<KP, 1, 1, TRACE, true, 0, 2>(p, s);
  }
  return nnp == 1 ? mid_launch_t<KP, 1, 1, TRACE, true>(p, s) : mid_launch_t<KP, 1, 2, TRACE, true>(p, s);
}

}  // namespace

}  // namespace tac
