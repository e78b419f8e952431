// Backward pass of the conv-LIF layer with a surrogate gradient (Sec. 5.1 "Training", App. C):
// the LIF recurrence backwards in time, then the two gradients of Y_k = bias + Conv2d(A_k, W); one
// convolution-gradient stage per group of K frames, like the forward pass (T/K stages for TAC and TAC-TP, T for the
// per-step layer).
//
//   lif_backward_kernel  dL/dY_k from dL/ds and the membranes the forward pass recorded
//   dgrad_kernel         dL/dS_{kK+j} = beta^(Kg-1-j) * (dY_k convolved back through W): fp32 vector arithmetic, any shape (stride 2, few input channels)
// and the choice among the matrix-core kernels of the other files.
#include "tac_dgrad_plan.h"

namespace tac {

namespace {

constexpr int kThreads = 256;
constexpr int kCiTile = 4;        // input channels per dgrad thread

// ds/dV in x = V - theta
__device__ __forceinline__ float surrogate(int kind, float alpha, float x) {
  if (kind == TAC_SG_FAST_SIGMOID) {
    const float t = 1.0f + alpha * fabsf(x);
    return 1.0f / (t * t);
  }
  const float t = 1.5707963267948966f * alpha * x;
  return 0.5f * alpha / (1.0f + t * t);
}

__device__ __forceinline__ int group_frames(const BackwardParams& p, int k) {
  return (k == p.G - 1 && p.K_last) ? p.K_last : p.K;
}

// dL/ds of output step n at neuron i: stored per step, or once per group of the next layer's frames
// (dL/dS_{kK+j} = beta^(Kg-1-j) dL/dA_k, Eq. 2) and multiplied by that layer's factor here
__device__ __forceinline__ float grad_out_at(const BackwardParams& p, size_t n, size_t n_out, size_t i) {
  size_t step = n;
  float f = 1.0f;
  if (p.go_K > 1) {
    const int kc = (int)n / p.go_K, j = (int)n - kc * p.go_K;
    f = (p.go_last && kc == p.go_G - 1) ? p.go_w_last[j] : p.go_w[j];
    step = (size_t)kc;
  }
  if (!p.out_pool) return p.go_K > 1 ? f * p.grad_out[step * n_out + i] : p.grad_out[step * n_out + i];
  // The layer stored the 2 x 2 max pool of its spikes (the OR of the four bits): the gradient of a pooled spike
  // goes to the first maximal spike of its window in row-major order (the first set bit, else the first neuron),
  // the spikes being what the forward pass decided on the recorded membranes of output step n, V >= theta.
  const int x = (int)(i % p.Wo), y = (int)((i / p.Wo) % p.Ho);
  const size_t bc = i / ((size_t)p.Wo * p.Ho);
  const float* v = p.v_trace + n * n_out + (bc * p.Ho + (y & ~1)) * p.Wo + (x & ~1);
  const uint32_t bits = (v[0] >= p.theta ? 1u : 0u) | (v[1] >= p.theta ? 2u : 0u) | (v[p.Wo] >= p.theta ? 4u : 0u) |
                        (v[p.Wo + 1] >= p.theta ? 8u : 0u);
  const int first = bits ? __ffs(bits) - 1 : 0;
  if (first != (y & 1) * 2 + (x & 1)) return 0.0f;
  const size_t ip = (bc * (p.Ho >> 1) + (y >> 1)) * (p.Wo >> 1) + (x >> 1);
  return f * p.grad_out[step * (n_out >> 2) + ip];
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// VEC consecutive neurons of one row as one load or store (VEC = 4: 16 bytes per lane, 2: 8 bytes)
template <int VEC>
struct Lanes {
  float v[VEC];
};
template <int VEC>
__device__ __forceinline__ Lanes<VEC> load_lanes(const float* src) {
  Lanes<VEC> r;
  if constexpr (VEC == 4) {
    const f32x4 t = *reinterpret_cast<const f32x4*>(src);
#pragma unroll
    for (int e = 0; e < 4; ++e) r.v[e] = t[e];
  } else if constexpr (VEC == 2) {
    const f32x2 t = *reinterpret_cast<const f32x2*>(src);
    r.v[0] = t[0];
    r.v[1] = t[1];
  } else {
    r.v[0] = *src;
  }
  return r;
}
// four floats that nobody reads again
__device__ __forceinline__ Lanes<4> load_once(const float* src) {
  const f32x4 t = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(src));
  return Lanes<4>{{t[0], t[1], t[2], t[3]}};
}
template <int VEC>
__device__ __forceinline__ void store_lanes(float* dst, const Lanes<VEC>& a) {
  if constexpr (VEC == 4)
    *reinterpret_cast<f32x4*>(dst) = f32x4{a.v[0], a.v[1], a.v[2], a.v[3]};
  else if constexpr (VEC == 2)
    *reinterpret_cast<f32x2*>(dst) = f32x2{a.v[0], a.v[1]};
  else
    *dst = a.v[0];
}

// dL/ds of output step n at the VEC neurons from i on (VEC = 4: unpooled output only)
template <int VEC>
__device__ __forceinline__ Lanes<VEC> grad_out_lanes(const BackwardParams& p, size_t n, size_t n_out, size_t i) {
  if constexpr (VEC == 1) {
    return Lanes<1>{{grad_out_at(p, n, n_out, i)}};
  } else {
    size_t step = n;
    float f = 1.0f;
    if (p.go_K > 1) {
      const int kc = (int)n / p.go_K, j = (int)n - kc * p.go_K;
      f = (p.go_last && kc == p.go_G - 1) ? p.go_w_last[j] : p.go_w[j];
      step = (size_t)kc;
    }
    Lanes<VEC> g = load_lanes<VEC>(p.grad_out + step * n_out + i);
    if (p.go_K > 1) {
#pragma unroll
      for (int e = 0; e < VEC; ++e) g.v[e] = f * g.v[e];
    }
    return g;
  }
}

// The sums dW and dbias start from: cleared by the LIF recurrence, which comes first, or by clear_kernel where that has too few
// threads for it (backward_launch) or dW has held something else in between.
__device__ __forceinline__ void clear_sums(const BackwardParams& p, size_t first, size_t threads) {
  const size_t n_w = (size_t)p.Cout * p.Cin * 9;
  for (size_t i = first; i < n_w; i += threads) p.grad_w[i] = 0.0f;
  if (p.grad_bias)
    for (size_t i = first; i < (size_t)p.Cout; i += threads) p.grad_bias[i] = 0.0f;
}

__global__ __launch_bounds__(kThreads) void clear_kernel(const BackwardParams p) {
  clear_sums(p, (size_t)blockIdx.x * kThreads + threadIdx.x, (size_t)gridDim.x * kThreads);
}

// Where a LIF step stands in its group, walking backwards.
struct StepCursor {
  int k, j;                                     // group, LIF step within it
  float decay;
  bool first;                                   // first step of the group (in this order)
  __device__ __forceinline__ void enter(const BackwardParams& p, int group) {
    k = group;
    first = true;
    if (k < 0) return;
    j = (p.mode == TAC_PRESERVE ? group_frames(p, k) : 1) - 1;
    decay = p.mode == TAC_COLLAPSE ? (group_frames(p, k) == p.K ? p.decay_full : p.decay_last) : p.beta;
  }
};

// One thread per VEC output neurons; the LIF steps backwards, c = dL/dV' carried.  The loads of U steps are issued
// together, only the chain through c is serial.  dL/dY_k is the sum of dL/dV over the LIF steps of group k (one step,
// or the group's frames with TAC-TP).
template <int VEC, int U>
__global__ __launch_bounds__(kThreads) void lif_backward_kernel(const BackwardParams p, int clear) {
  const size_t n_out = (size_t)p.B * p.Cout * p.Ho * p.Wo;
  const size_t thread = (size_t)blockIdx.x * kThreads + threadIdx.x;
  if (clear) clear_sums(p, thread, (size_t)gridDim.x * kThreads);
  const size_t i = thread * VEC;
  if (i >= n_out) return;
  float c[VEC], acc[VEC];
#pragma unroll
  for (int e = 0; e < VEC; ++e) c[e] = acc[e] = 0.0f;
  int n = p.n_steps;
  StepCursor at;
  at.enter(p, p.G - 1);
  while (n > 0) {
    const int m = min(U, n);
    Lanes<VEC> v[U], g[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u < m) {
        v[u] = load_lanes<VEC>(p.v_trace + (size_t)(n - 1 - u) * n_out + i);
        g[u] = grad_out_lanes<VEC>(p, (size_t)(n - 1 - u), n_out, i);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u < m) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
          const float sg = surrogate(p.surrogate, p.alpha, v[u].v[e] - p.theta);
          const float gv = g[u].v[e] * sg + c[e] * (p.detach_reset ? 1.0f : 1.0f - p.theta * sg);
          acc[e] = at.first ? gv : acc[e] + gv;
          c[e] = at.decay * gv;
        }
        at.first = false;
        if (at.j == 0) {
          Lanes<VEC> out;
#pragma unroll
          for (int e = 0; e < VEC; ++e) out.v[e] = acc[e];
          store_lanes<VEC>(p.grad_y + (size_t)at.k * n_out + i, out);
          at.enter(p, at.k - 1);
        } else {
          --at.j;
        }
      }
    }
    n -= m;
  }
}

// The same where the layer stored the 2 x 2 max pool of its spikes.  A thread owns the two rows and VEC columns of
// VEC / 2 windows, so that a membrane is read once (one neuron per thread reads its window's four membranes, five loads
// for one gradient), the window's route is decided in registers and the pooled gradient is read once.  Bound by HBM on
// large layers, by the chain of loads over the steps on small ones: 128 channels, B = 16, 16 steps at 64 x 64 / 32 x 32 /
// 16 x 16 take 140 / 37 / 18 us (one neuron per thread: 540 / 141 / 46 us).
// ONCE: the membranes are read past the caches (backward_launch).
template <int VEC, int U, bool ONCE = false>
__global__ __launch_bounds__(kThreads) void lif_backward_pooled_kernel(const BackwardParams p, int clear) {
  constexpr int WIN = VEC / 2;
  const size_t n_out = (size_t)p.B * p.Cout * p.Ho * p.Wo;
  const size_t thread = (size_t)blockIdx.x * kThreads + threadIdx.x;
  if (clear) clear_sums(p, thread, (size_t)gridDim.x * kThreads);
  if (thread >= n_out / (2 * VEC)) return;
  const uint32_t per_row = (uint32_t)p.Wo / VEC;
  const size_t row2 = thread / per_row;                                   // row pair over all channels and samples
  const size_t i = row2 * 2 * p.Wo + (thread - row2 * per_row) * VEC;     // upper left neuron
  const size_t ip = thread * WIN;                                         // its window in the pooled tensor
  float c[2][VEC], acc[2][VEC];
#pragma unroll
  for (int y = 0; y < 2; ++y)
#pragma unroll
    for (int e = 0; e < VEC; ++e) c[y][e] = acc[y][e] = 0.0f;
  int n = p.n_steps;
  StepCursor at;
  at.enter(p, p.G - 1);
  while (n > 0) {
    const int m = min(U, n);
    Lanes<VEC> v[U][2];
    Lanes<WIN> g[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u < m) {
        const size_t step = (size_t)(n - 1 - u);
        const float* const src = p.v_trace + step * n_out + i;
        if constexpr (ONCE) {
          v[u][0] = load_once(src);
          v[u][1] = load_once(src + p.Wo);
        } else {
          v[u][0] = load_lanes<VEC>(src);
          v[u][1] = load_lanes<VEC>(src + p.Wo);
        }
        size_t gstep = step;
        float f = 1.0f;
        if (p.go_K > 1) {
          const int kc = (int)step / p.go_K, j = (int)step - kc * p.go_K;
          f = (p.go_last && kc == p.go_G - 1) ? p.go_w_last[j] : p.go_w[j];
          gstep = (size_t)kc;
        }
        g[u] = load_lanes<WIN>(p.grad_out + gstep * (n_out >> 2) + ip);
#pragma unroll
        for (int w = 0; w < WIN; ++w) g[u].v[w] = f * g[u].v[w];
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (u < m) {
#pragma unroll
        for (int w = 0; w < WIN; ++w) {
          // the first maximal spike of the window in row-major order: the first set bit, else the first neuron
          const float v0 = v[u][0].v[2 * w], v1 = v[u][0].v[2 * w + 1], v2 = v[u][1].v[2 * w], v3 = v[u][1].v[2 * w + 1];
          const bool s0 = v0 >= p.theta, s1 = v1 >= p.theta, s2 = v2 >= p.theta, s3 = v3 >= p.theta;
          const bool to[4] = {s0 || !(s1 || s2 || s3), !s0 && s1, !s0 && !s1 && s2, !s0 && !s1 && !s2 && s3};
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int y = q >> 1, e = 2 * w + (q & 1);
            const float sg = surrogate(p.surrogate, p.alpha, v[u][y].v[e] - p.theta);
            const float gv = (to[q] ? g[u].v[w] : 0.0f) * sg + c[y][e] * (p.detach_reset ? 1.0f : 1.0f - p.theta * sg);
            acc[y][e] = at.first ? gv : acc[y][e] + gv;
            c[y][e] = at.decay * gv;
          }
        }
        at.first = false;
        if (at.j == 0) {
#pragma unroll
          for (int y = 0; y < 2; ++y) {
            Lanes<VEC> out;
#pragma unroll
            for (int e = 0; e < VEC; ++e) out.v[e] = acc[y][e];
            store_lanes<VEC>(p.grad_y + (size_t)at.k * n_out + i + (size_t)y * p.Wo, out);
          }
          at.enter(p, at.k - 1);
        } else {
          --at.j;
        }
      }
    }
    n -= m;
  }
}

// Thread = one input pixel (iy, ix) of (group k, sample b), kCiTile input channels: sums
// dY_k[co][y][x] W[co][ci][ky][kx] over the outputs (y, x) whose window covers the pixel, then
// writes the gradient of each of the group's frames, dA scaled by the frame's weight.
// OVER: more tiles of input channels than a grid has in y; the rest follows in x behind the pixels (dgrad_vector_tiles).  One after the other in a loop, the stores would keep the
// weights out of scalar loads: 2.4 times the time.
template <bool OVER>
__global__ __launch_bounds__(kThreads) void dgrad_kernel(const BackwardParams p) {
  const uint32_t blocks = OVER ? ((uint32_t)(p.H * p.W) + kThreads - 1) / kThreads : 0, over = OVER ? blockIdx.x / blocks : 0;
  const int ci0 = (int)((over * gridDim.y + blockIdx.y) * kCiTile);
  const int b = blockIdx.z % p.B, k = blockIdx.z / p.B;
  const int px = (int)((blockIdx.x - over * blocks) * kThreads + threadIdx.x);
  if (px >= p.H * p.W) return;
  const int iy = px / p.W, ix = px - iy * p.W;
  const size_t plane = (size_t)p.Ho * p.Wo;
  // the outputs that see this pixel through tap (ky, kx): y = (iy + 1 - ky) / stride when that divides
  int off[9];
#pragma unroll
  for (int t = 0; t < 9; ++t) {
    const int ny = iy + 1 - t / 3, nx = ix + 1 - t % 3;
    const bool ok = ny >= 0 && nx >= 0 && ny % p.stride == 0 && nx % p.stride == 0 && ny / p.stride < p.Ho && nx / p.stride < p.Wo;
    off[t] = ok ? (ny / p.stride) * p.Wo + nx / p.stride : -1;
  }
  float dA[kCiTile];
#pragma unroll
  for (int c = 0; c < kCiTile; ++c) dA[c] = 0.0f;
  const float* dy = p.grad_y + ((size_t)k * p.B + b) * p.Cout * plane;
  for (int co = 0; co < p.Cout; ++co) {
    float g[9];
#pragma unroll
    for (int t = 0; t < 9; ++t) g[t] = off[t] >= 0 ? dy[(size_t)co * plane + off[t]] : 0.0f;
#pragma unroll
    for (int c = 0; c < kCiTile; ++c) {
      if (ci0 + c < p.Cin) {
        const float* w = p.w + ((size_t)co * p.Cin + ci0 + c) * 9;     // uniform over the workgroup
#pragma unroll
        for (int t = 0; t < 9; ++t) dA[c] = fmaf(g[t], w[t], dA[c]);
      }
    }
  }
  const int Kg = group_frames(p, k);
  const float* wj = Kg == p.K ? p.wj : p.wj_last;
  const size_t in_plane = (size_t)p.H * p.W;
  if (p.pool2) {
    // gradient of the unpooled frames [2H][2W]: a quarter to each input of the mean pool; all of it to the first
    // maximal input of the max pool's window in row-major order (the first set bit, or the first input when none is set)
    const int W2 = 2 * p.W;
    const size_t fs = (size_t)p.B * p.Cin * 2 * p.H * p.Wwi;
    for (int j = 0; j < Kg; ++j)
#pragma unroll
      for (int c = 0; c < kCiTile; ++c)
        if (ci0 + c < p.Cin) {
          const size_t chan = ((size_t)(k * p.K + j) * p.B + b) * p.Cin + ci0 + c;
          float* dst = p.grad_in + chan * 4 * in_plane + (size_t)(2 * iy) * W2 + 2 * ix;
          const float g = wj[j] * dA[c];
          float q[4] = {0.25f * g, 0.25f * g, 0.25f * g, 0.25f * g};
          if (p.pool2 == 2) {
            const uint32_t* src = p.spikes + chan * 2 * p.H * p.Wwi + (size_t)(2 * iy) * p.Wwi + (ix >> 4);
            const uint32_t two = ((src[0] >> (2 * ix & 31)) & 3u) | (((src[p.Wwi] >> (2 * ix & 31)) & 3u) << 2);
            const int best = two ? __ffs(two) - 1 : 0;
#pragma unroll
            for (int e = 0; e < 4; ++e) q[e] = e == best ? g : 0.0f;
          }
          dst[0] = q[0]; dst[1] = q[1]; dst[W2] = q[2]; dst[W2 + 1] = q[3];
        }
    return;
  }
  if (p.grad_in_group) {
#pragma unroll
    for (int c = 0; c < kCiTile; ++c)
      if (ci0 + c < p.Cin) p.grad_in[(((size_t)k * p.B + b) * p.Cin + ci0 + c) * in_plane + px] = dA[c];
    return;
  }
  for (int j = 0; j < Kg; ++j)
#pragma unroll
    for (int c = 0; c < kCiTile; ++c)
      if (ci0 + c < p.Cin)
        p.grad_in[(((size_t)(k * p.K + j) * p.B + b) * p.Cin + ci0 + c) * in_plane + px] = wj[j] * dA[c];
}

}  // namespace

hipError_t backward_launch(const BackwardParams& p, hipStream_t s) {
  const size_t n_out = (size_t)p.B * p.Cout * p.Ho * p.Wo;
  // the wide-tile input gradient uses grad_w as scratch for its prepared weights: it runs before grad_w is cleared
  const bool dgrad_tile = p.grad_in && backward_dgrad_tile_supported(p);
  const uintptr_t bases = (uintptr_t)p.v_trace | (uintptr_t)p.grad_out | (uintptr_t)p.grad_y;
  auto blocks = [](size_t threads) { return dim3((unsigned)((threads + kThreads - 1) / kThreads)); };
  // Two windows per thread: 16-byte membrane accesses, enough threads to fill the chip from 2^20 neurons on.  Small layers wait
  // for memory, step after step: one window per thread, four steps asked for together.  Without a pool four neurons per thread
  // where rows allow 16-byte accesses; with 16 bytes per lane one step in flight per thread keeps the memory busy, the scalar
  // form asks for four steps at once.
  const bool windows2 = p.out_pool && p.Wo % 4 == 0 && (bases & 15) == 0 && n_out >= ((size_t)1 << 20);
  const bool windows1 = p.out_pool && !windows2 && (bases & 7) == 0;
  const bool neurons4 = !p.out_pool && n_out % 4 == 0 && (bases & 15) == 0;
  const size_t threads = windows2 ? n_out / 8 : windows1 || neurons4 ? n_out / 4 : n_out;
  const int clear = !dgrad_tile && backward_clear_in_recurrence(threads, (size_t)p.Cout * p.Cin * 9);
  // Membranes that do not fit the 256 MiB of the last cache are read past it, one step in flight per thread: a backward call without input
  // gradient of 2 -> 128 at 64 x 64, B = 16, 16 steps (512 MiB) 210 -> 187 us, B = 64 777 -> 738, 2 -> 64 at 128 x 128, B = 4 (256 MiB)
  // 121 -> 113; below they may still be there: B = 16 at 32 x 32 (128 MiB) 57 -> 61.  Without a pool there is no difference (2062 / 2056).
  const bool once = windows2 && n_out * (size_t)p.n_steps >= ((size_t)64 << 20);
  if (once) hipLaunchKernelGGL((lif_backward_pooled_kernel<4, 1, true>), blocks(threads), dim3(kThreads), 0, s, p, clear);
  else if (windows2) hipLaunchKernelGGL((lif_backward_pooled_kernel<4, 2>), blocks(threads), dim3(kThreads), 0, s, p, clear);
  else if (windows1) hipLaunchKernelGGL((lif_backward_pooled_kernel<2, 4>), blocks(threads), dim3(kThreads), 0, s, p, clear);
  else if (neurons4) hipLaunchKernelGGL((lif_backward_kernel<4, 1>), blocks(threads), dim3(kThreads), 0, s, p, clear);
  else hipLaunchKernelGGL((lif_backward_kernel<1, 4>), blocks(threads), dim3(kThreads), 0, s, p, clear);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;

  if (dgrad_tile) {
    e = backward_dgrad_tile_launch(p, s);
    if (e != hipSuccess) return e;
  }
  if (!clear) hipLaunchKernelGGL(clear_kernel, blocks((size_t)p.Cout * p.Cin * 9), dim3(kThreads), 0, s, p);
  if (p.bf16 && !p.dense && p.pool2 != 1 && backward_wgrad_mfma_supported(p)) {
    e = backward_wgrad_mfma_launch(p, s);
    if (e != hipSuccess) return e;
  } else {
    if (!backward_wgrad_first_launch(p, s, e)) e = backward_wgrad_f32_launch(p, s);
    if (e != hipSuccess) return e;
  }

  if (dgrad_tile) {
    // done above
  } else if (p.grad_in && p.bf16 && p.pool2 != 1 && backward_dgrad_mfma_supported(p)) {
    e = backward_dgrad_mfma_launch(p, s);
  } else if (p.grad_in && backward_dgrad_f32_supported(p)) {
    e = backward_dgrad_f32_launch(p, s);
  } else if (p.grad_in) {
    unsigned across, over;
    dgrad_vector_tiles(p.Cin, across, over);
    const dim3 grid((p.H * p.W + kThreads - 1) / kThreads * over, across, p.G * p.B);
    if (over == 1) hipLaunchKernelGGL(dgrad_kernel<false>, grid, dim3(kThreads), 0, s, p);
    else hipLaunchKernelGGL(dgrad_kernel<true>, grid, dim3(kThreads), 0, s, p);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace tac
