// Dense 0/1 bytes <-> bit-packed rows, rows padded to whole words with zero bits.
#include "tac_internal.h"

namespace tac {

// four bytes -> four bits, set where the byte is not zero
__device__ __forceinline__ uint32_t nonzero_bytes(uint32_t v) {
  const uint32_t t = ((((v & 0x7f7f7f7fu) + 0x7f7f7f7fu) | v) >> 7) & 0x01010101u;
  return (t * 0x10204080u) >> 28;               // bit 8 i -> bit 28 + i; nothing below carries that far
}

// A thread per packed word.  ALIGNED: rows are multiples of 16 bytes from a 16-byte aligned address, a word is one or two
// 16-byte loads; otherwise the tensor and its rows may start anywhere in a dword and the word's up to nine dwords are shifted
// into place.  (`dense` is then the dword that holds the tensor's first byte, `skip` that byte's place in it; n_bytes: from there to
// the tensor's end; a dword that reaches beyond the tensor is read byte by byte.)
// One wave per 64 pixels with a ballot reads 64 bytes a load instruction: 16.8 MB of 128-pixel rows 24.5 us, now 5.4 us; from an
// address that is one byte off a call takes 9.8 us (21.7 with the ballot, 29.4 byte by byte).
template <bool ALIGNED>
__global__ __launch_bounds__(256) void pack_kernel(const uint8_t* __restrict__ dense, uint32_t* __restrict__ packed, int64_t words,
                                                   int64_t n_bytes, int W, int Ww, int skip) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words; i += stride) {
    const int64_t row = i / Ww;
    const int word = (int)(i - row * Ww);
    const int64_t first = row * W + 32 * word + (ALIGNED ? 0 : skip);
    const int n = min(32, W - 32 * word);
    uint32_t bits = 0;
    if constexpr (ALIGNED) {
      const uint4 a = *reinterpret_cast<const uint4*>(dense + first);
      uint4 b = make_uint4(0, 0, 0, 0);
      if (n > 16) b = *reinterpret_cast<const uint4*>(dense + first + 16);
      bits = nonzero_bytes(a.x) | nonzero_bytes(a.y) << 4 | nonzero_bytes(a.z) << 8 | nonzero_bytes(a.w) << 12 |
             nonzero_bytes(b.x) << 16 | nonzero_bytes(b.y) << 20 | nonzero_bytes(b.z) << 24 | nonzero_bytes(b.w) << 28;
    } else {
      const int64_t base = first & ~(int64_t)3;
      const int lead = (int)(first - base);     // bytes of the first dword that belong to the pixel before
      uint64_t all = 0;
#pragma unroll
      for (int d = 0; d < 9; ++d) {
        if (4 * d >= lead + n) break;
        const int64_t at = base + 4 * d;
        uint32_t v = 0;
        if (at >= skip && at + 4 <= n_bytes) {
          v = *reinterpret_cast<const uint32_t*>(dense + at);
        } else {
          for (int k = 0; k < 4; ++k)
            if (at + k >= skip && at + k < n_bytes) v |= (uint32_t)dense[at + k] << (8 * k);
        }
        all |= (uint64_t)nonzero_bytes(v) << (4 * d);
      }
      bits = (uint32_t)(all >> lead);
      if (n < 32) bits &= (1u << n) - 1u;
    }
    packed[i] = bits;
  }
}

__global__ __launch_bounds__(256) void unpack_kernel(const uint32_t* __restrict__ packed,
                                                     uint8_t* __restrict__ dense,
                                                     int64_t rows, int W, int Ww) {
  const int64_t n = rows * W;
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const int64_t row = i / W;
    const int x = (int)(i - row * W);
    dense[i] = (uint8_t)((packed[row * Ww + (x >> 5)] >> (x & 31)) & 1u);
  }
}

static int grid_for(int64_t work_per_block_units) {
  int64_t g = work_per_block_units;
  if (g < 1) g = 1;
  if (g > 256 * 32) g = 256 * 32;
  return (int)g;
}

hipError_t pack_launch(const uint8_t* dense, uint32_t* packed, int64_t rows, int W, hipStream_t s) {
  const int Ww = (W + 31) / 32;
  const int64_t words = rows * Ww;
  const dim3 grid(grid_for((words + 255) / 256));
  const int skip = (int)((uintptr_t)dense & 3u);
  if (W % 16 == 0 && ((uintptr_t)dense & 15u) == 0)
    hipLaunchKernelGGL(pack_kernel<true>, grid, dim3(256), 0, s, dense, packed, words, rows * W, W, Ww, 0);
  else
    hipLaunchKernelGGL(pack_kernel<false>, grid, dim3(256), 0, s, dense - skip, packed, words, rows * W + skip, W, Ww, skip);
  return hipGetLastError();
}

hipError_t unpack_launch(const uint32_t* packed, uint8_t* dense, int64_t rows, int W, hipStream_t s) {
  const int Ww = (W + 31) / 32;
  hipLaunchKernelGGL(unpack_kernel, dim3(grid_for((rows * W + 255) / 256)), dim3(256), 0, s, packed, dense, rows, W, Ww);
  return hipGetLastError();
}

// Batch norm (inference statistics) folded into weights and bias: one workgroup per output
// channel; the scale is formed in double from the fp32 statistics and rounded once.
__global__ void fold_bn_kernel(const float* __restrict__ w, const float* __restrict__ bias, const float* __restrict__ gamma,
                               const float* __restrict__ beta_bn, const float* __restrict__ mean,
                               const float* __restrict__ var, float eps, int per, float* w_out, float* bias_out) {
  const int co = blockIdx.x;
  const double sc = (double)gamma[co] / sqrt((double)var[co] + (double)eps);
  for (int i = threadIdx.x; i < per; i += blockDim.x)
    w_out[(size_t)co * per + i] = (float)((double)w[(size_t)co * per + i] * sc);
  if (threadIdx.x == 0)
    bias_out[co] = (float)((((bias ? (double)bias[co] : 0.0) - (double)mean[co]) * sc) + (double)beta_bn[co]);
}

hipError_t fold_bn_launch(const float* w, const float* bias, const float* gamma, const float* beta_bn, const float* mean,
                          const float* var, float eps, int Cout, int per, float* w_out, float* bias_out, hipStream_t s) {
  hipLaunchKernelGGL(fold_bn_kernel, dim3(Cout), dim3(256), 0, s, w, bias, gamma, beta_bn, mean, var, eps, per, w_out,
                     bias_out);
  return hipGetLastError();
}

}  // namespace tac
