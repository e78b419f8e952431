// Weight and bias gradient of first layers (one or two input channels, bits or real-valued frames, no pool on load) in fp32 on the vector units:
//   dW[co][ci][ky][kx] = sum over groups k, samples b, output pixels of dY_k[co][pixel] * A_k[ci][pixel's input under the tap].
// dW has 9 or 18 columns, which fill a third or half of a matrix-core tile, and its operands would have to be turned around in LDS; every dY value
// is used 9 or 18 times only, so what bounds the layer is reading dY once.  Here a lane owns four neighbouring pixels: it reads its dY of a channel as 16
// consecutive bytes (a wave's load is 1 KiB of consecutive addresses), the 3 x 6 aggregates around them from LDS once for four channels, and adds
// the products to 36 Cin sums of its own.
//
// Workgroup = eight waves = `ncg` groups of four output channels x 8 / ncg shares of the pixels, over a slice of the items (some (group, sample) pairs of a small
// image, or a strip of rows of one).  The aggregates of an item are rebuilt from the frames into LDS.
//
// Error: a lane's chains of products end after 64 of them (kFirstWgradChain); the sums of the 64 lanes then meet in a tree and go on in 64 bits, in LDS, one set for
// each wave.  What is rounded to fp32 again is a workgroup's sum, of which the slices (64; 128 with real-valued frames) add one each in memory.  Without the end of the
// chains the error grew with the data: 1 -> 128, 2 steps of spikes everywhere at 64 x 64, B = 640, dY the same everywhere (chains of 640 equal products): 7.2e-7 of the norm, now
// 1.0e-7, that kernel 1.2e-7.  Ending them costs less than a call's times differ.
//
// Backward calls without input gradient in us, that kernel (tac_backward_wgrad_f32.hip) and this one, with their errors (norm against 64-bit sums, dY of both signs):
//   1 -> 32, 7 groups at 28 x 28, B = 128               102 2.9e-7    67 1.5e-7   (the kernel alone 63 / 30; dY is 90 MB)
//   2 -> 128, real values, 4 groups at 64 x 64, B = 16  135 2.3e-7   115 2.3e-7
//   2 -> 128, 4 groups at 64 x 64, B = 16               125 2.0e-7   101 1.8e-7
//   2 -> 64 stride 2, 8 groups at 128 x 128, B = 32     255 2.5e-7   240 2.0e-7
//   1 -> 16, one group at 100 x 100, B = 128            128 2.7e-7    64 1.6e-7
//   1 -> 64, 32 steps at 128 x 128, B = 48             5830 3.0e-7  4830 1.6e-7
// The kernel alone on 271 random first layers that it takes: 1.36 times as fast as that kernel at the median, eight slower (from 0.83: 10.5 us against 8.7).
#include "tac_wgrad_first_plan.h"

namespace tac {

namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int kThreads = kFirstWgradThreads;
constexpr int CPW = kFirstWgradChannels;

__device__ __forceinline__ int group_frames(const BackwardParams& p, int k) {
  return (k == p.G - 1 && p.K_last) ? p.K_last : p.K;
}

// Value of lane ^ (1 << STEP).
template <int STEP>
__device__ __forceinline__ float across(float v) {
  const int i = __builtin_bit_cast(int, v);
  if constexpr (STEP == 0) return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(i, 0xb1, 0xf, 0xf, true));       // lanes 1, 0, 3, 2 of four
  else if constexpr (STEP == 1) return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(i, 0x4e, 0xf, 0xf, true));  // lanes 2, 3, 0, 1
  else return __shfl_xor(v, 1 << STEP, 64);
}

// Sums of v[0 .. N) over the 64 lanes.  In each of six steps a lane gives half of its values to the other lane of a pair and gets that one's part of
// the other half: N exchanges in all in the place of 6 N.  The value that ends in v[j] of lane l is lane_sum_index<N>(j, l); one without a partner
// is in both lanes.
template <int N, int STEP, int M>
__device__ __forceinline__ void lane_sums(float (&v)[M], int lane) {
  if constexpr (STEP < 6) {
    const bool odd = (lane >> STEP) & 1;
    static_for<0, N / 2>([&](auto i_) {
      constexpr int i = decltype(i_)::value;
      const float keep = odd ? v[2 * i + 1] : v[2 * i], give = odd ? v[2 * i] : v[2 * i + 1];
      v[i] = keep + across<STEP>(give);
    });
    if constexpr (N & 1) v[N >> 1] = v[N - 1] + across<STEP>(v[N - 1]);
    lane_sums<(N + 1) / 2, STEP + 1>(v, lane);
  }
}
template <int N, int STEP = 0>
__device__ __forceinline__ int lane_sum_index(int j, int lane) {
  if constexpr (STEP == 6) return j;
  else return min(2 * lane_sum_index<(N + 1) / 2, STEP + 1>(j, lane) + ((lane >> STEP) & 1), N - 1);
}
constexpr int lane_sum_left(int n) {
  for (int i = 0; i < 6; ++i) n = (n + 1) / 2;
  return n;
}

// VEC: rows of dY are whole quads at 16-byte addresses.
template <int S, int CIN, bool DENSE, bool VEC>
__global__ __launch_bounds__(kThreads, 4) void wgrad_first_kernel(const BackwardParams p, const FirstWgradPlan q) {
  constexpr int NS = CPW * 9 * CIN;                      // sums of a lane
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  float* const agg = reinterpret_cast<float*>(lds);
  float* const wl = reinterpret_cast<float*>(lds + q.off_w);           // frame weights: a whole group's, the last group's
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  double* const red = reinterpret_cast<double*>(lds + q.off_sum);      // [wave][channel][ci][tap]
  double* const red_b = red + 8 * 72;                    // [wave][channel]
  const int slice = (int)(blockIdx.x % (uint32_t)q.split), co_group = (int)(blockIdx.x / (uint32_t)q.split);
  const int cg = wave % q.ncg, share = wave / q.ncg, shares = 8 / q.ncg;
  const int co0 = (co_group * q.ncg + cg) * CPW;
  const size_t plane = (size_t)p.Ho * p.Wo;
  if (tid < 2 * TAC_MAX_K) {
    const int j = tid & (TAC_MAX_K - 1);
    wl[tid] = tid < TAC_MAX_K ? (j < p.K ? p.wj[j] : 0.f) : (j < p.K_last ? p.wj_last[j] : 0.f);
  }

  float acc[NS];                                         // [channel][ci][tap], of the last items
  for (int i = lane; i < NS; i += 64) red[wave * NS + i] = 0.0;        // (the wave's own)
  double bias[CPW];
#pragma unroll
  for (int c = 0; c < CPW; ++c) {
    bias[c] = 0.0;
  }
#pragma unroll
  for (int i = 0; i < NS; ++i) acc[i] = 0.f;

  const int all_pairs = p.G * p.B, items = q.pair_tiles * q.n_strips;
  const float inv_quads = 1.0f / (float)q.quads, inv_b = 1.0f / (float)p.B;
  int chain = 0;
  const int units_row = q.cw >> 3;                       // units of eight aggregates
  const float inv_units = 1.0f / (float)units_row, inv_cw = 1.0f / (float)q.cw, inv_cin_rows = 1.0f / (float)(CIN * q.rows_in);
  for (int it = slice; it < items; it += q.split) {
    const int pt = it / q.n_strips, y0 = (it - pt * q.n_strips) * q.rows;
    const int pair0 = pt * q.n_pairs, pairs = min(q.n_pairs, all_pairs - pair0), rows = min(q.rows, p.Ho - y0);
    __syncthreads();                                     // the item before has been read
    // ---- aggregates [pair][channel][row][column], column 0 the padding left of the image; zeros outside it
    // (what row of which image a line of them is: (sample, group), channel, row)
    struct Line { int k, b, ci, iy; };
    auto take_line = [&](int line) {
      const int pr = small_div(line, inv_cin_rows), cr = line - pr * (CIN * q.rows_in);
      const int ci = CIN == 1 ? 0 : cr >= q.rows_in, k = small_div(pair0 + pr, inv_b);
      return Line{k, pair0 + pr - k * p.B, ci, y0 * S - 1 + cr - ci * q.rows_in};
    };
    const int n_lines = pairs * CIN * q.rows_in;
    if constexpr (DENSE) {
      // real-valued frames [T][B][Cin][H][W], a thread per value
      const size_t frame = (size_t)p.B * p.Cin * p.H * p.W;
      // four of them at a time, so that their trips to memory overlap
      constexpr int kMany = 4;
      for (int e0 = tid; e0 < n_lines * q.cw; e0 += kMany * kThreads) {
        const float* src[kMany];
        const float* wj[kMany];
        float a[kMany];
        int Kg[kMany], most = 0;
#pragma unroll
        for (int i = 0; i < kMany; ++i) {
          const int e = min(e0 + i * kThreads, n_lines * q.cw - 1), line = small_div(e, inv_cw), ix = e - line * q.cw - 1;
          const Line l = take_line(line);
          const bool inside = l.iy >= 0 && l.iy < p.H && ix >= 0 && ix < p.W;
          Kg[i] = inside ? group_frames(p, l.k) : 0;
          most = max(most, Kg[i]);
          wj[i] = wl + (group_frames(p, l.k) == p.K ? 0 : TAC_MAX_K);
          src[i] = reinterpret_cast<const float*>(p.spikes) + (inside ? ((((size_t)l.k * p.K * p.B + l.b) * p.Cin + l.ci) * p.H + l.iy) * p.W + ix : 0);
          a[i] = 0.f;
        }
        for (int j = 0; j < most; j += 4) {
          float f[kMany][4];
#pragma unroll
          for (int i = 0; i < kMany; ++i)
#pragma unroll
            for (int u = 0; u < 4; ++u) f[i][u] = src[i][(size_t)max(min(j + u, Kg[i] - 1), 0) * frame];
#pragma unroll
          for (int i = 0; i < kMany; ++i)
#pragma unroll
            for (int u = 0; u < 4; ++u)
              if (j + u < Kg[i]) a[i] = fmaf(wj[i][j + u], f[i][u], a[i]);
        }
#pragma unroll
        for (int i = 0; i < kMany; ++i)
          if (e0 + i * kThreads < n_lines * q.cw) agg[e0 + i * kThreads] = a[i];
      }
    } else {
      const size_t frame = (size_t)p.B * p.Cin * p.H * p.Wwi;
      for (int e = tid; e < n_lines * units_row; e += kThreads) {
        const int line = small_div(e, inv_units), x0 = (e - line * units_row) * 8 - 1;
        const Line l = take_line(line);
        float a[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) a[i] = 0.f;
        if (l.iy >= 0 && l.iy < p.H) {
          const int Kg = group_frames(p, l.k);
          const float* const wj = wl + (Kg == p.K ? 0 : TAC_MAX_K);
          // the eight bits from x0 on: of one word or two
          const uint32_t* const src = p.spikes + ((((size_t)l.k * p.K * p.B + l.b) * p.Cin + l.ci) * p.H + l.iy) * p.Wwi;
          const uint32_t inside = x0 + 8 <= p.W ? 0xffu : (1u << max(p.W - x0, 0)) - 1u;
          const int w0 = min(max(x0, 0) >> 5, p.Wwi - 1), w1 = min((x0 + 7) >> 5, p.Wwi - 1);
          for (int j = 0; j < Kg; j += 4) {
            uint32_t lo[4], hi[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              lo[u] = src[(size_t)min(j + u, Kg - 1) * frame + w0];
              hi[u] = src[(size_t)min(j + u, Kg - 1) * frame + w1];
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
              if (j + u >= Kg) break;
              const uint32_t bits = (x0 < 0 ? lo[u] << 1 : (uint32_t)((((uint64_t)hi[u] << 32) | lo[u]) >> (x0 & 31))) & inside;
              const float wt = wj[j + u];
#pragma unroll
              for (int i = 0; i < 8; ++i) a[i] += (bits >> i) & 1u ? wt : 0.f;
            }
          }
        }
        float* const dst = agg + line * q.cw + (x0 + 1);
        *reinterpret_cast<f32x4*>(dst) = f32x4{a[0], a[1], a[2], a[3]};
        *reinterpret_cast<f32x4*>(dst + 4) = f32x4{a[4], a[5], a[6], a[7]};
      }
    }
    __syncthreads();
    // ---- the wave's quads
    const int per_pair = rows * q.quads, nq = pairs * per_pair;
    const float inv_pair = 1.0f / (float)per_pair;
    for (int e = share * 64 + lane; e < nq; e += shares * 64) {
      const int pr = small_div(e, inv_pair), in_pair = e - pr * per_pair;
      const int y = small_div(in_pair, inv_quads), x = (in_pair - y * q.quads) * 4;
      const int pair = pair0 + pr;
      const float* const src = p.grad_y + (size_t)pair * p.Cout * plane + (size_t)(y0 + y) * p.Wo + x;
      f32x4 g[CPW];
#pragma unroll
      for (int c = 0; c < CPW; ++c) {
        const float* const at = src + (size_t)min(co0 + c, p.Cout - 1) * plane;         // (channels beyond Cout are not stored)
        if constexpr (VEC) g[c] = *reinterpret_cast<const f32x4*>(at);
        else {
#pragma unroll
          for (int u = 0; u < 4; ++u) g[c][u] = at[min(u, p.Wo - 1 - x)];
        }
      }
      const int real = VEC ? 4 : min(4, p.Wo - x);       // of the quad's pixels
      if constexpr (!VEC) {
#pragma unroll
        for (int c = 0; c < CPW; ++c)
#pragma unroll
          for (int u = 1; u < 4; ++u) g[c][u] = u < real ? g[c][u] : 0.f;
      }
#pragma unroll
      for (int c = 0; c < CPW; ++c) bias[c] += (double)((g[c][0] + g[c][1]) + (g[c][2] + g[c][3]));
      const float* const a_quad = agg + (pr * CIN * q.rows_in + y * S) * q.cw + x * S;
#pragma unroll
      for (int i = 0; i < CIN; ++i)
#pragma unroll
        for (int ky = 0; ky < 3; ++ky) {
          const float* const row = a_quad + (i * q.rows_in + ky) * q.cw;
          float a[12];
          *reinterpret_cast<f32x4*>(a) = *reinterpret_cast<const f32x4*>(row);
          if constexpr (S == 1) *reinterpret_cast<f32x2*>(a + 4) = *reinterpret_cast<const f32x2*>(row + 4);
          else {
            *reinterpret_cast<f32x4*>(a + 4) = *reinterpret_cast<const f32x4*>(row + 4);
            a[8] = row[8];
          }
#pragma unroll
          for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int kx = 0; kx < 3; ++kx) {
              // An infinite frame value is not multiplied by the zero of a pixel that is not there: only the first such pixel's left column is in the image.
              const float v = DENSE && !VEC && u > 0 && kx == 0 ? (u < real ? a[u * S] : 0.f) : a[u * S + kx];
#pragma unroll
              for (int c = 0; c < CPW; ++c) acc[(c * CIN + i) * 9 + ky * 3 + kx] = fmaf(g[c][u], v, acc[(c * CIN + i) * 9 + ky * 3 + kx]);
            }
        }
    }
    // ---- a chain of products ends: its 64 lanes' sums meet, and go on in 64 bits
    if (++chain == q.flush || it + q.split >= items) {   // (uniform)
      chain = 0;
      int l = lane;
      asm volatile("" : "+v"(l));                        // what depends on the lane is formed here: nothing of it is kept across items
      lane_sums<NS, 0>(acc, l);
      static_for<0, lane_sum_left(NS)>([&](auto j_) {
        constexpr int j = decltype(j_)::value;
        red[wave * NS + lane_sum_index<NS>(j, l)] += (double)acc[j];          // (lanes with the same value read, then write it, together)
      });
#pragma unroll
      for (int i = 0; i < NS; ++i) acc[i] = 0.f;
    }
  }
  // ---- the waves that share a group of channels, then the slices
#pragma unroll
  for (int c = 0; c < CPW; ++c) {
    double v = bias[c];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if (lane == 0) red_b[wave * CPW + c] = v;
  }
  __syncthreads();
  for (int e = tid; e < q.ncg * NS; e += kThreads) {
    const int g = e / NS, at = e - g * NS, co = (co_group * q.ncg + g) * CPW + at / (9 * CIN);
    double v = 0.0;
    for (int s = 0; s < shares; ++s) v += red[(s * q.ncg + g) * NS + at];
    if (co < p.Cout) atomicAdd(p.grad_w + (size_t)co * (9 * CIN) + at % (9 * CIN), (float)v);
  }
  if (p.grad_bias && tid < q.ncg * CPW) {
    const int g = tid / CPW, c = tid - g * CPW, co = (co_group * q.ncg + g) * CPW + c;
    double v = 0.0;
    for (int s = 0; s < shares; ++s) v += red_b[(s * q.ncg + g) * CPW + c];
    if (co < p.Cout) atomicAdd(p.grad_bias + co, (float)v);
  }
}

}  // namespace

bool backward_wgrad_first_launch(const BackwardParams& p, hipStream_t s, hipError_t& e) {
  FirstWgradPlan q{};
  if (!first_wgrad_plan(p, q)) return false;
  const bool vec = p.Wo % 4 == 0 && ((uintptr_t)p.grad_y & 15) == 0;
  auto launch = [&](auto s_, auto cin_, auto dense_) {
    constexpr int S = decltype(s_)::value, CIN = decltype(cin_)::value;
    constexpr bool DENSE = decltype(dense_)::value;
    const auto kern = vec ? &wgrad_first_kernel<S, CIN, DENSE, true> : &wgrad_first_kernel<S, CIN, DENSE, false>;
    if (q.total > 64 * 1024) {
      e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, kFirstWgradLds);
      if (e != hipSuccess) return;
    }
    hipLaunchKernelGGL(kern, dim3((unsigned)(q.co_groups * q.split)), dim3(kThreads), q.total, s, p, q);
    e = hipGetLastError();
  };
  auto with_cin = [&](auto s_, auto cin_) {
    if (p.dense) launch(s_, cin_, std::true_type{});
    else launch(s_, cin_, std::false_type{});
  };
  auto with_s = [&](auto s_) {
    if (p.Cin == 1) with_cin(s_, std::integral_constant<int, 1>{});
    else with_cin(s_, std::integral_constant<int, 2>{});
  };
  if (p.stride == 1) with_s(std::integral_constant<int, 1>{});
  else with_s(std::integral_constant<int, 2>{});
  return true;
}

}  // namespace tac
