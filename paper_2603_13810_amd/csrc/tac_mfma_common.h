// Pieces shared by the MFMA kernels: vector types, kernel parameters, the lane-to-pixel
// geometry of the MFMA result and the LIF step on the accumulators.
#pragma once
#include <type_traits>

#include "tac_internal.h"

namespace tac {

namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4v;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((address_space(3))) void* lds_void_ptr;
typedef const __attribute__((address_space(1))) void* global_void_ptr;

constexpr int kFixShift = 23;                  // fixed-point scale of the aggregation weights

struct MfmaParams {
  const uint32_t* __restrict__ spikes;
  const uint8_t* __restrict__ w;       // prepared: [cout_tile][chunk][tap][mc][lane][8] bf16, scaled 2^-23
  const float* __restrict__ bias;
  float* __restrict__ v_inout;
  uint32_t* __restrict__ out;
  float* __restrict__ v_trace;
  int B, Cin, H, W, Ho, Wo, Cout, stride, K, G, n_lif, row_tiles, maxpool;
  float decay, theta;
  uint32_t wq[TAC_MAX_K];              // round(beta^(K-1-j) * 2^23)
  int out_pool;                        // 2 x 2 max pool of the output spikes before they are stored
  int pool;                            // mid kernel: 2 x 2 pool on load, 1 mean, 2 max
};

// The parameters of a layer; the tiles are the launcher's.
inline void fill_params(MfmaParams& mp, const LayerParams& p) {
  mp.spikes = p.spikes; mp.w = static_cast<const uint8_t*>(p.w); mp.bias = p.bias; mp.v_inout = p.v_inout;
  mp.out = p.out; mp.v_trace = p.v_trace;
  mp.B = p.B; mp.Cin = p.Cin; mp.H = p.H; mp.W = p.W; mp.Ho = p.Ho; mp.Wo = p.Wo; mp.Cout = p.Cout; mp.stride = p.stride;
  mp.K = p.K; mp.G = p.G; mp.n_lif = p.n_lif; mp.maxpool = p.pool2 == 2; mp.pool = p.pool2; mp.out_pool = p.out_pool;
  mp.row_tiles = 0;
  mp.decay = p.decay; mp.theta = p.theta;
  for (int j = 0; j < TAC_MAX_K; ++j) {
    // beta^(K-1-j) in 24-bit fixed point, from the fp32 table the host already rounded
    const double q = (double)p.wj[j] * (double)(1u << kFixShift);
    mp.wq[j] = j < p.K ? (uint32_t)(q + 0.5) : 0u;
  }
}

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  f32x2 f = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));   // v_cvt_pk_bf16_f32, nearest even
}

// i / d for a wave-uniform divisor of reciprocal r and i below 2^20: (i + 1/2) / d is at least 1 / (2 d) from every integer, more than
// the rounding of the reciprocal and the product moves it
__device__ __forceinline__ int small_div(int i, float r) { return (int)(((float)i + 0.5f) * r); }
struct SmallDiv {
  int d;
  float r;
  __device__ __forceinline__ explicit SmallDiv(int divisor) : d(divisor), r(1.0f / (float)divisor) {}
  __device__ __forceinline__ int quot(int i) const { return small_div(i, r); }
};

// Workgroup barrier that orders LDS traffic only: the compiler waits for this wave's LDS
// accesses and for its direct-to-LDS loads, but leaves ordinary global loads in flight.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// vdst[lane L0 + i * STEP + (j ? HALF : 0)] = x[i][j] for the wave-uniform values x[4][2]; other
// lanes keep `old`.  The s_nop covers the two wait states this chip needs between a vector
// instruction that wrote an SGPR (the compare, or a spill reload) and a vector instruction that
// reads it: the assembler text is opaque to the compiler's hazard pass.
template <int L0, int STEP, int HALF>
__device__ __forceinline__ uint32_t write_lanes(uint32_t old, const uint32_t (&x)[4][2]) {
  uint32_t r;
  asm volatile(
      "s_nop 1\n\t"
      "v_writelane_b32 %0, %1, %9\n\tv_writelane_b32 %0, %2, %10\n\t"
      "v_writelane_b32 %0, %3, %11\n\tv_writelane_b32 %0, %4, %12\n\t"
      "v_writelane_b32 %0, %5, %13\n\tv_writelane_b32 %0, %6, %14\n\t"
      "v_writelane_b32 %0, %7, %15\n\tv_writelane_b32 %0, %8, %16"
      : "=v"(r)
      : "s"(x[0][0]), "s"(x[0][1]), "s"(x[1][0]), "s"(x[1][1]), "s"(x[2][0]), "s"(x[2][1]), "s"(x[3][0]),
        "s"(x[3][1]), "n"(L0), "n"(L0 + HALF), "n"(L0 + STEP), "n"(L0 + STEP + HALF), "n"(L0 + 2 * STEP),
        "n"(L0 + 2 * STEP + HALF), "n"(L0 + 3 * STEP), "n"(L0 + 3 * STEP + HALF), "0"(old));
  return r;
}

// the same for two pairs
template <int L0, int STEP, int HALF>
__device__ __forceinline__ uint32_t write_lanes(uint32_t old, const uint32_t (&x)[2][2]) {
  uint32_t r;
  asm volatile(
      "s_nop 1\n\tv_writelane_b32 %0, %1, %5\n\tv_writelane_b32 %0, %2, %6\n\t"
      "v_writelane_b32 %0, %3, %7\n\tv_writelane_b32 %0, %4, %8"
      : "=v"(r)
      : "s"(x[0][0]), "s"(x[0][1]), "s"(x[1][0]), "s"(x[1][1]), "n"(L0), "n"(L0 + HALF), "n"(L0 + STEP), "n"(L0 + STEP + HALF), "0"(old));
  return r;
}

// (a & m) | (b & ~m): one v_bfi_b32
__device__ __forceinline__ uint32_t bfi(uint32_t m, uint32_t a, uint32_t b) { return (a & m) | (b & ~m); }

// K frame words -> K class words, in place (K a power of two up to 8): class word c holds the pixels p = c (mod K),
// pixel p as the K-bit field [bit j = frame j] at bit position p - c.  Recursion: the two
// halves of the frames give class words with K/2-bit fields; class c of the result takes the
// even fields of both (low half of the new field from the first half of the frames), class
// c + K/2 the odd ones.
template <int K>
__device__ __forceinline__ void frames_to_fields(uint32_t* w) {
  if constexpr (K >= 2) {
    frames_to_fields<K / 2>(w);
    frames_to_fields<K / 2>(w + K / 2);
    constexpr uint32_t m = K == 2 ? 0x55555555u : (K == 4 ? 0x33333333u : 0x0f0f0f0fu);
#pragma unroll
    for (int c = 0; c < K / 2; ++c) {
      const uint32_t lo = w[c], hi = w[c + K / 2];
      w[c] = bfi(m, lo, hi << (K / 2));
      w[c + K / 2] = bfi(m, lo >> (K / 2), hi);
    }
  }
}

// The aggregates (Eq. 2) of a group of two frames, two channels at once: t, their frame bits at bits 0 and 16; the four bf16 entries in the halves of lo and hi.
__device__ __forceinline__ uint32_t two_frame_pair(uint32_t hi, uint32_t lo, uint32_t t) {
  return __builtin_amdgcn_perm(hi, lo, __umul24(t, 0x0202u) + 0x01000100u);
}

// Aggregates by frame bits: KP = 4, pairs of channels as two bf16; KP = 8, one bf16; KP = 16, 2^-23 fixed-point sums of frames 0 .. 7 and 8 .. 15.  `sets` tables of `words`
// entries, the second one with the weights from first_last on.
template <int KP>
__device__ __forceinline__ void frame_tables(uint32_t* lut, int words, int sets, int first_last, const MfmaParams& p, int tid, int threads) {
  const float scale = 1.0f / (float)(1u << kFixShift);
#pragma clang loop unroll(disable)
  for (int i = tid; i < words * sets; i += threads) {
    const int set = i >= words, t = i - (set ? words : 0), f0 = set ? first_last : 0;
    uint32_t a[2] = {0, 0};
#pragma unroll
    for (int j = 0; j < (KP == 4 ? 4 : 8); ++j) {
      const int jj = f0 + j + (KP == 16 ? (t >> 8) * 8 : 0);
      const uint32_t w = p.wq[min(jj, TAC_MAX_K - 1)];
      a[0] += (t >> j) & 1 ? w : 0u;
      if constexpr (KP == 4) a[1] += (t >> (4 + j)) & 1 ? w : 0u;
    }
    lut[i] = KP == 16 ? a[0] : pack_bf16((float)a[0] * scale, (float)a[1] * scale);
  }
}

// 2 x 2 max pool of bits, horizontal part: OR of neighbouring bit pairs, even bits gathered into the low half;
// 32 pixels -> 16 pooled pixels.
__device__ __forceinline__ uint32_t pool_pairs(uint32_t v) {
  v = (v | (v >> 1)) & 0x55555555u;
  v = (v | (v >> 1)) & 0x33333333u;
  v = (v | (v >> 2)) & 0x0f0f0f0fu;
  v = (v | (v >> 4)) & 0x00ff00ffu;
  return (v | (v >> 8)) & 0x0000ffffu;
}

// N (1 or 2) direct-to-LDS loads of 16 bytes per lane from one global address to one LDS base address, the n-th
// with the immediate offset OFF0 + 1024 n added to both.  Written as an assembly statement on purpose: while a
// direct-to-LDS load that the compiler knows of is pending, it turns every wait on the LDS counter into a wait for
// zero, and in the chunk loops that use it one always is, so each tap would wait for the LDS reads and writes it has only just
// issued.  The compiler therefore does not know of these loads at all: the reader of what they write waits for
// vmcnt(0) (lds_dma_wait) in front of the workgroup barrier that separates writer and reader, and the kernel waits
// once more before it ends.  The waits the compiler places for its own loads count these loads too, which only
// makes them stricter.  M0 holds the LDS address; one wait state between its write and the load.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int N, int OFF0>
__device__ __forceinline__ void lds_dma16(const void* gsrc, uint32_t lds_base) {
  static_assert(N == 1 || N == 2, "one or two loads");
  if constexpr (N == 1)
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off offset:%2"
                 :: "v"(gsrc), "s"(lds_base), "n"(OFF0) : "m0", "memory");
  else
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off offset:%2\n\t"
                 "global_load_lds_dwordx4 %0, off offset:%3"
                 :: "v"(gsrc), "s"(lds_base), "n"(OFF0), "n"(OFF0 + 1024) : "m0", "memory");
}
// one dword per lane, from the wave-uniform address sbase plus the lane's byte offset voff: lane l's word goes to
// lds_base + 4 l
__device__ __forceinline__ void lds_dma4(uint32_t voff, const void* sbase, uint32_t lds_base) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dword %0, %1" :: "v"(voff), "s"(sbase), "s"(lds_base) : "m0", "memory");
}
#pragma clang diagnostic pop
__device__ __forceinline__ void lds_dma_wait() { __builtin_amdgcn_s_waitcnt(0x0f70); }   // vmcnt(0), other counters untouched

template <int I, int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// Per-lane constants of the epilogue: where the lane's two pixels (np = 0, 1) sit.
struct LaneGeom {
  uint32_t v_off[2];     // byte offset of (4 h channels, local row, column) in the wave's membrane block
  float theta[2];        // the threshold, or +inf where the pixel's output row is outside the image
  bool ok[2];            // the pixel is inside the image
  int co_lim;            // channels (counted from the wave's first) that exist for this lane's half
};

// One LIF step on a wave's NMC x NP MFMA tiles (NP = 2; 1: the lanes of pixel block 1 stay zero and are not stored): V <- decay V + Y, spike iff V >= theta,
// subtractive reset.  Register r of tile (mc, np) on lane (n, h) is channel
// 32 mc + 8 (r/4) + 4 h + r%4 at the wave's pixel 32 np + n.  The ballot of a register is two
// 32-bit halves (h = 0, 1), each the packed spikes of 32 consecutive output pixels of one
// channel; they are handed, one per lane, to the store registers word[mc][..]:
//   output width 64 or 32: lane (r << 2) | (h << 1) | np of word[mc][0] holds pixel block np;
//   output width 16:       a half is two rows of 16 pixels; lane
//                          ((r & 7) << 3) | (h << 2) | (np << 1) | sub of word[mc][r >> 3] holds
//                          row 2 np + sub.
// NQ: quads of registers that hold channels (fewer than four where a layer has at most 8 NQ of them; the others are left alone).
template <int NMC, int WO, bool TRACE, int NP = 2, int NQ = 4>
__device__ __forceinline__ void lif_step(float (&V)[NMC][NP][16], const f32x16 (&acc)[NMC][NP], float decay, float theta,
                                         const LaneGeom& lg, uint32_t (&word)[NMC][2], float* __restrict__ trace_wave,
                                         size_t plane) {
  static_for<0, NMC>([&](auto mc_) {
    constexpr int mc = decltype(mc_)::value;
    static_for<0, NP>([&](auto np_) {
      constexpr int np = decltype(np_)::value;
      // four registers at a time: all four membranes and compares first, then the four ballot
      // hand-overs, then the four resets, so that no instruction waits on the one before it
      static_for<0, NQ>([&](auto r4_) {
        constexpr int r0 = decltype(r4_)::value * 4;
        float v[4];
        uint64_t m[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = fmaf(decay, V[mc][np][r0 + i], acc[mc][np][r0 + i]);
#pragma unroll
        for (int i = 0; i < 4; ++i) m[i] = __builtin_amdgcn_ballot_w64(v[i] >= lg.theta[np]);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (WO >= 32) {
          // registers r0 .. r0+3: lanes (r << 2) | np (low half) and (r << 2) | 2 | np (high half)
          uint32_t x[4][2];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            x[i][0] = (uint32_t)m[i];
            x[i][1] = (uint32_t)(m[i] >> 32);
          }
          word[mc][0] = write_lanes<(r0 << 2) | np, 4, 2>(word[mc][0], x);
        } else {
          // a ballot half is two rows of 16 pixels: lanes base | sub (low half), base | 4 | sub (high)
          constexpr int base = ((r0 & 7) << 3) | (np << 1);
          uint32_t x[4][2];
#pragma unroll
          for (int sub = 0; sub < 2; ++sub) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const uint32_t lo = (uint32_t)m[i], hi = (uint32_t)(m[i] >> 32);
              x[i][0] = sub ? lo >> 16 : lo & 0xffffu;
              x[i][1] = sub ? hi >> 16 : hi & 0xffffu;
            }
            if (sub == 0)
              word[mc][r0 >> 3] = write_lanes<base, 8, 4>(word[mc][r0 >> 3], x);
            else
              word[mc][r0 >> 3] = write_lanes<base | 1, 8, 4>(word[mc][r0 >> 3], x);
          }
        }
        __builtin_amdgcn_sched_barrier(0);
        [[maybe_unused]] int co_lim = lg.co_lim;
        // (compared again in every step: the conditions of all registers together do not fit the scalar registers)
        if constexpr (TRACE) asm volatile("" : "+v"(co_lim));
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          V[mc][np][r0 + i] = __builtin_amdgcn_inverse_ballot_w64(m[i]) ? v[i] - theta : v[i];
          if constexpr (TRACE) {
            if (lg.ok[np] && mc * 32 + 8 * ((r0 + i) >> 2) + ((r0 + i) & 3) < co_lim)
              *reinterpret_cast<float*>(reinterpret_cast<char*>(trace_wave) +
                                        (size_t)(mc * 32 + 8 * ((r0 + i) >> 2) + ((r0 + i) & 3)) * plane * 4 +
                                        lg.v_off[np]) = v[i];
          }
        }
        // the new membranes count as used here: otherwise the compiler moves the resets behind
        // the whole step and keeps all 128 ballots alive until then (in spilled scalar registers)
#pragma unroll
        for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(V[mc][np][r0 + i]));
        __builtin_amdgcn_sched_barrier(0);   // keep only a few ballots alive
      });
    });
  });
}

// One LIF step with a channel per lane: the operands of the MFMAs swapped (pixels as rows, channels as columns), register r of a
// block on lane (n, h) is pixel 8 (r / 4) + 4 h + r % 4 of channel n.  A ballot costs two v_writelane per register on the way to a
// store, and select and subtraction two more instructions; here the lanes that spike are what EXEC holds while the threshold is
// subtracted and the pixel's bit set, four vector instructions per register instead of 6.25, and one scalar move that other
// waves' vector instructions run beside.  Measured, ns per register and step on a SIMD, against compare, subtract, select and
// a v_addc that shifts the mask into the bits (five): 6.8 / 8.9 with four waves on the SIMD, 8.2 / 9.3 with two, 12.5 / 10.9 with one.
// The membranes v are formed outside: they read MFMA results, whose wait states the compiler knows.
template <int R0>
__device__ __forceinline__ void spike_reset4(float (&v)[4], float theta, uint32_t& bits) {
  uint64_t m[4], all;
  asm("v_cmp_ge_f32_e64 %5, %1, %10\n\tv_cmp_ge_f32_e64 %6, %2, %10\n\tv_cmp_ge_f32_e64 %7, %3, %10\n\tv_cmp_ge_f32_e64 %8, %4, %10\n\t"
      "s_mov_b64 %9, exec\n\t"
      "s_mov_b64 exec, %5\n\tv_subrev_f32_e32 %1, %10, %1\n\tv_or_b32_e32 %0, %11, %0\n\t"
      "s_mov_b64 exec, %6\n\tv_subrev_f32_e32 %2, %10, %2\n\tv_or_b32_e32 %0, %12, %0\n\t"
      "s_mov_b64 exec, %7\n\tv_subrev_f32_e32 %3, %10, %3\n\tv_or_b32_e32 %0, %13, %0\n\t"
      "s_mov_b64 exec, %8\n\tv_subrev_f32_e32 %4, %10, %4\n\tv_or_b32_e32 %0, %14, %0\n\t"
      "s_mov_b64 exec, %9"
      : "+v"(bits), "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "=&s"(m[0]), "=&s"(m[1]), "=&s"(m[2]), "=&s"(m[3]), "=&s"(all)
      : "s"(theta), "n"(1 << (2 * R0)), "n"(2 << (2 * R0)), "n"(4 << (2 * R0)), "n"(8 << (2 * R0)));
}

// The same with compare, subtraction, select and a v_addc that shifts the mask into the bits (v[0] first): for kernels with one wave
// on a SIMD, where nothing runs beside the moves of EXEC.
__device__ __forceinline__ void spike_reset4_shift(float (&v)[4], float theta, uint32_t& bits) {
  uint64_t m[4];
  float t[4];
  asm("v_cmp_ge_f32_e64 %5, %1, %13\n\tv_cmp_ge_f32_e64 %6, %2, %13\n\tv_cmp_ge_f32_e64 %7, %3, %13\n\tv_cmp_ge_f32_e64 %8, %4, %13\n\t"
      "v_subrev_f32_e32 %9, %13, %1\n\tv_subrev_f32_e32 %10, %13, %2\n\tv_subrev_f32_e32 %11, %13, %3\n\tv_subrev_f32_e32 %12, %13, %4\n\t"
      "v_addc_co_u32_e64 %0, vcc, %0, %0, %5\n\tv_addc_co_u32_e64 %0, vcc, %0, %0, %6\n\t"
      "v_addc_co_u32_e64 %0, vcc, %0, %0, %7\n\tv_addc_co_u32_e64 %0, vcc, %0, %0, %8\n\t"
      "v_cndmask_b32_e64 %1, %1, %9, %5\n\tv_cndmask_b32_e64 %2, %2, %10, %6\n\t"
      "v_cndmask_b32_e64 %3, %3, %11, %7\n\tv_cndmask_b32_e64 %4, %4, %12, %8"
      : "+v"(bits), "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "=&s"(m[0]), "=&s"(m[1]), "=&s"(m[2]), "=&s"(m[3]),
        "=&v"(t[0]), "=&v"(t[1]), "=&v"(t[2]), "=&v"(t[3])
      : "s"(theta)
      : "vcc");
}

// bits[np]: the spikes of the lane's 16 pixels at their places in the packed word, the upper lane half's four bits too low.
// ALONE: one wave on the SIMD.
template <int NP, bool ALONE = false>
__device__ __forceinline__ void lif_step_cols(float (&V)[NP][16], const f32x16 (&y)[NP], float decay, float theta, uint32_t (&bits)[2]) {
  bits[0] = bits[1] = 0;
  [[maybe_unused]] uint32_t all = 0;             // ALONE: bit 16 np + r, the last register first
  static_for<0, NP * 4>([&](auto q_) {
    constexpr int q = ALONE ? NP * 4 - 1 - decltype(q_)::value : decltype(q_)::value, np = q >> 2, r0 = (q & 3) * 4;
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = fmaf(decay, V[np][r0 + (ALONE ? 3 - i : i)], y[np][r0 + (ALONE ? 3 - i : i)]);
    if constexpr (ALONE) spike_reset4_shift(v, theta, all);
    else spike_reset4<r0>(v, theta, bits[np]);
#pragma unroll
    for (int i = 0; i < 4; ++i) V[np][r0 + (ALONE ? 3 - i : i)] = v[i];
  });
  if constexpr (ALONE) {                       // nibble i of a block -> byte i
    const uint32_t even = all & 0x0f0f0f0fu, odd = (all >> 4) & 0x0f0f0f0fu;
    bits[0] = __builtin_amdgcn_perm(odd, even, 0x05010400u);
    if (NP == 2) bits[1] = __builtin_amdgcn_perm(odd, even, 0x07030602u);
  }
}

// A 32 x 32 block between its two layouts, through 33 floats per channel of LDS that belong to the wave: register r on lane (n, h)
// is channel 8 (r / 4) + 4 h + r % 4 of pixel n, or that pixel of channel n.
constexpr int kTurnFloats = 32 * 33;
__device__ __forceinline__ void turn_block(float (&v)[16], float* t, int n, int h) {
  // the wave's own LDS accesses execute in order; keep the compiler to it too
  asm volatile("" ::: "memory");
#pragma unroll
  for (int r = 0; r < 16; ++r) t[(8 * (r >> 2) + 4 * h + (r & 3)) * 33 + n] = v[r];
  asm volatile("" ::: "memory");
#pragma unroll
  for (int r = 0; r < 16; ++r) v[r] = t[n * 33 + 8 * (r >> 2) + 4 * h + (r & 3)];
  asm volatile("" ::: "memory");
}

// The packed words of two blocks: lane n gets block 0's word of channel n, lane 32 + n block 1's.
__device__ __forceinline__ uint32_t words_of_cols(const uint32_t (&bits)[2]) {
  const auto w = __builtin_amdgcn_permlane32_swap(bits[0], bits[1], false, false);
  return w[0] | (w[1] << 4);
}

// The same for two blocks that are the two rows of a 2 x 2 max pool: 16 pooled pixels of channel n in either half.
__device__ __forceinline__ uint32_t pooled_of_cols(const uint32_t (&bits)[2]) {
  const uint32_t rows = bits[0] | bits[1];
  const auto w = __builtin_amdgcn_permlane32_swap(rows, rows, false, false);
  return pool_pairs(w[0] | (w[1] << 4));
}

// MaxPool(2) of the output spikes in the layer that writes them (the Conv -> BN -> LIF -> MaxPool(2) blocks of
// Sec. 5.1): on 0/1 spikes the maximum of a 2 x 2 window is the OR of its four bits, so the packed words of one
// LIF step are pooled before they are stored and the tensor crosses HBM at a quarter of its bytes.
// `word` holds the step's packed output as lif_step leaves it for output rows of 32 pixels and more (lane
// (r << 2) | (hi << 1) | np: channel 8 (r / 4) + 4 hi + r % 4 of 32-channel block mc, 32-pixel block np of the
// wave).  A lane pools its 32 pixels horizontally to 16 bits and puts them into the exchange area in LDS
//     ex: uint32 [rows][ctile],  low half = pooled block 0, high half = pooled block 1,
// the workgroup meets at a barrier, and the threads then OR the two rows of every pooled row and store the words (rows have at most
// 64 pixels, one pooled word): pooled row pr of channel c = ex[2 pr][c] | ex[2 pr + 1][c].
//   two_rows   the wave's two blocks are two rows of 32 pixels (np = row) instead of two halves of one row
//   row0       first row of the wave within the tile
//   out_tile   address of (this step, sample, first channel of the tile, pooled row y0 / 2)
//   plane_p    words per channel of the pooled tensor
//   rows_p     pooled rows of the tile inside the image
// Called by all threads of the workgroup (it contains a barrier); consecutive steps alternate between two areas.
//   c_first    first channel of the wave within the tile
// COLS: the words as words_of_cols leaves them (lane 32 np + n: channel n).  MC: 32-channel blocks of the tile (NMC of them the wave's).  GH = 2:
// the wave's words are those of registers 0 .. 7, in lanes 0 .. 31.
template <int NMC, bool COLS, int MC = NMC, int GH = 1>
__device__ __forceinline__ void pooled_store(const uint32_t (&word)[NMC][2], uint32_t* ex, int tid, int nthreads, int rows,
                                             bool two_rows, int row0, int c_first, uint32_t* out_tile, size_t plane_p, int rows_p) {
  constexpr int ctile = MC * 32;
  const int lane = tid & 63;
  const int r = lane >> 2, hi = (lane >> 1) & 1, np = COLS ? lane >> 5 : lane & 1;
  const int c_lane = COLS ? lane & 31 : 8 * (r >> 2) + 4 * hi + (r & 3);
#pragma unroll
  for (int mc = 0; mc < NMC; ++mc) {
    const uint32_t hp = pool_pairs(word[mc][0]);
    const int c = c_first + mc * 32 + c_lane;
    if (GH == 2 && lane >= 32) continue;
    if (two_rows)
      ex[(row0 + np) * ctile + c] = hp;
    else
      reinterpret_cast<uint16_t*>(ex)[((row0 * ctile + c) << 1) + np] = (uint16_t)hp;
  }
  __syncthreads();
  const int items = (rows >> 1) * ctile;
  for (int i = tid; i < items; i += nthreads) {
    const int c = i % ctile, pr = i / ctile;
    const uint32_t v = ex[2 * pr * ctile + c] | ex[(2 * pr + 1) * ctile + c];
    if (pr < rows_p) out_tile[(size_t)c * plane_p + pr] = v;
  }
}

__host__ __device__ constexpr int pool_exchange_bytes(int rows, int ctile) { return 2 * rows * ctile * 4; }

}  // namespace

}  // namespace tac
