// Proposal network kernels: 1-D convolutions on BF16 MFMA with FP32
// accumulation, the weight-gradient reduction, softmax cross-entropy, the
// proposal (argmax + window mass) and Adam.
//
// Row layout. Series s owns rows [s SR + 2, s SR + 2 + K_s) of the row buffers
// (SR = roundup(max_K + 4, 16)); kernels mask rows outside the series, the zero
// padding of the kernel-5 convolutions.
//
// A layer y[t][o] = b[o] + sum_{k<5, i<CIN} W[o][i][k] x[t + k - 2][i] is an
// implicit GEMM with M = output channels (16 per MFMA tile), N = rows (16) and
// reduction index j = k * CIN + i (32 per v_mfma_f32_16x16x32_bf16). The
// input gradient of a layer is the same convolution of the output gradient
// with W'[i][o][k] = W[o][i][4 - k].
#pragma once

#include <type_traits>

#include "ks.h"
#include "ks_wave.hpp"

namespace ks {
namespace cnn {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int KW = 5;
constexpr int NTC = 256;

// float -> bfloat16 bits, round to nearest even (finite inputs)
__device__ __forceinline__ uint16_t f2bf(float f) {
  const uint32_t u = __float_as_uint(f);
  return (uint16_t)((u + 0x7fffu + ((u >> 16) & 1u)) >> 16);
}

__device__ __forceinline__ float relu(float v) { return v > 0.0f ? v : 0.0f; }

__device__ __forceinline__ f32x4 mfma16(const u32x4& a, const u32x4& b, const f32x4& c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                 0, 0);
}

// Position channels of row t of a K-row series (double, rounded to float).
__device__ __forceinline__ float pos_frac(uint32_t t, uint32_t K) {
  return (float)((double)t / (double)(K > 1 ? K - 1 : 1));
}
__device__ __forceinline__ float pos_centre(uint32_t t, uint32_t K) {
  return (float)(4.0 * (double)t * (double)(K - t) / ((double)K * (double)K));
}

// ------------------------------------------------------------ fused forward
// The whole network over tiles of at most FT rows of one series. A K-row series
// has ceil(K / FT) tiles of equal length (so that none is nearly empty), and a
// tile computes only the 16-row blocks that its own rows need.
//
// What bounds it: with one 16-channel tile per wave every activation operand was
// read from LDS by all four waves, 1 KB per 16-cycle MFMA and SIMD, twice what
// LDS delivers; one wave now owns 32 output channels (its weights of layers 1
// and 2 stay in registers, 160 of them, which leaves two waves per SIMD) and
// half of the row blocks, so each operand read feeds two MFMAs. Weights are the
// A operand and rows the B operand: a lane then holds four consecutive channels
// of one row, stored as one 8-byte LDS write after two v_cvt_pk_bf16_f32 (the
// other way round it held one channel of four rows: four 2-byte writes and the
// rounding in integer code). Each output accumulates the same products in the
// same MFMA steps, bias last, so logits are the same bits.
//
// Buffers hold bf16 rows: x row r is series row t0 - 8 + r, layer l's output
// row r (l = 0, 1, 2) is series row t0 - 6 + 2 l + r and reads input rows
// r .. r + 4; rows outside the series are zero (the convolutions' padding).
// FT + 12 = 128 rows of layer 0 make eight blocks.
constexpr int FT = 116;
constexpr int FROWS = 16 * 8 + 4;  // buffer rows: eight blocks and the taps past them
// A 64-channel buffer in LDS: two planes of rows, the 8-channel chunks 0, 2, 4, 6
// in one and 1, 3, 5, 7 in the other, 80 bytes a row. An operand read takes
// chunk kg (+ 4) of row m for lane (m, kg), and the hardware serves lanes m = 0..3
// of one kg together with m = 4..7 of the next: in one 144-byte row of all chunks
// those met on the same banks (45% of the fused forward's LDS cycles), here
// they are eight different rows at 80 bytes.
constexpr int FPS = 32 + 8;                             // row stride of a plane (bf16)
constexpr int FPL = (FROWS * FPS * 2 + 127) / 128 * 64;  // one plane, whole turns of the banks
__device__ __forceinline__ constexpr uint32_t act_at(uint32_t row, uint32_t chunk) {
  return (chunk & 1u) * FPL + row * FPS + (chunk >> 1) * 8u;
}
constexpr int FXS = 16 + 8;        // LDS row stride of the 16-channel input buffer
constexpr int FW3 = 320 + 8;       // LDS row stride of the last layer's weights
constexpr int FWGS = 2;            // workgroups per CU (registers)

struct FusedSmem {
  uint16_t act[2][2 * FPL];
  uint16_t x[FROWS * FXS];
  uint16_t w3[2 * FW3];  // row 0: W3[0][j]; row 1: zeros (output channels 1..15)
  float bias[3 * 64];
  uint32_t count;
};

// Two floats as bf16 bits, rounded to nearest even (v_cvt_pk_bf16_f32; the same
// bits as f2bf for every number).
__device__ __forceinline__ uint32_t pack_bf(float a, float b) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const f32x2 v{a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// Products of a CIN-channel kernel-5 layer for G row blocks 32 rows apart and
// this wave's 32 output channels: in points at this lane's row of the first
// block (tap 0; its chunk kg for 64 channels), Wt holds W[o][32 q + 8 kg .. + 7] of its two channel tiles.
template <int CIN, int NQ, int G>
__device__ __forceinline__ void conv_blocks(const uint16_t* __restrict__ in, const u32x4 (&Wt)[NQ][2], uint32_t kg,
                                            f32x4 (&acc)[G][2]) {
  constexpr int ST = CIN == 64 ? FPS : FXS;
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int n = 0; n < 2; ++n) acc[g][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  // row operands one step ahead of the MFMAs; the scheduling barrier keeps the
  // compiler from hoisting every step's loads (and their registers)
  auto load = [&](int q, u32x4 (&x)[G]) {
    const int j0 = q * 32 + (int)kg * 8;
    const int k = CIN == 64 ? q / 2 : j0 / CIN, i0 = CIN == 64 ? (q & 1) * 16 : j0 % CIN;
#pragma unroll
    for (int g = 0; g < G; ++g)
      x[g] = (NQ * 32 <= KW * CIN || j0 < KW * CIN) ? *reinterpret_cast<const u32x4*>(&in[(32 * g + k) * ST + i0])
                                                    : u32x4{0u, 0u, 0u, 0u};
  };
  u32x4 x0[G], x1[G];
  load(0, x0);
#pragma unroll
  for (int q = 0; q < NQ; ++q) {
    u32x4(&cur)[G] = (q & 1) ? x1 : x0;
    u32x4(&nxt)[G] = (q & 1) ? x0 : x1;
    if (q + 1 < NQ) load(q + 1, nxt);
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int n = 0; n < 2; ++n) acc[g][n] = mfma16(Wt[q][n], cur[g], acc[g][n]);
    __builtin_amdgcn_sched_barrier(0);
  }
}

// A copy of v that the compiler takes for a new value: what is computed from it
// (a layer's LDS addresses) is computed there again and not kept in registers
// over the tiles beside the weights.
__device__ __forceinline__ uint32_t renew(uint32_t v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Calls run(tag<G>, first block) over a wave's nb <= 4 row blocks, at most GM
// (4 or 2) at once.
template <int GM, class Run>
__device__ __forceinline__ void for_blocks(uint32_t nb, Run&& run) {
  if (GM == 4 && nb == 4) {
    run(std::integral_constant<int, GM>{}, 0u);
  } else {
#pragma unroll 1
    for (uint32_t b = 0; b + 2 <= nb; b += 2) run(std::integral_constant<int, 2>{}, b);
    if (nb & 1) run(std::integral_constant<int, 1>{}, nb - 1);
  }
}

// One layer with 64 output channels over nb row blocks for this wave's 32
// channels: out row r = bf16(relu(b + products)) where series row tb + r is in
// [0, K), else 0.
template <int CIN, int NQ>
__device__ __forceinline__ void fused_layer(const uint16_t* __restrict__ in, const u32x4 (&Wt)[NQ][2],
                                            const float* __restrict__ bias, uint16_t* __restrict__ out, int32_t tb,
                                            uint32_t K, uint32_t nb, uint32_t rh, uint32_t ch, uint32_t lane) {
  lane = renew(lane);
  const uint32_t m = lane & 15u, kg = lane >> 4;
  // layer 0's weights are not kept: two blocks at a time leave them room
  for_blocks<CIN == 64 ? 4 : 2>((nb + 1 - rh) / 2, [&](auto tag, uint32_t b0) {
    constexpr int G = decltype(tag)::value;
    const uint32_t r0 = 32 * b0 + 16 * rh + m;  // blocks rh, rh + 2, ...
    f32x4 acc[G][2];
    conv_blocks<CIN, NQ, G>(in + (CIN == 64 ? act_at(r0, kg) : r0 * FXS), Wt, kg, acc);
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const f32x4 bv = *reinterpret_cast<const f32x4*>(&bias[ch + 16 * n + 4 * kg]);
#pragma unroll
      for (int g = 0; g < G; ++g) {
        const uint32_t r = r0 + 32 * g;
        const bool v = (uint32_t)(tb + (int32_t)r) < K;
        const f32x4 y = acc[g][n] + bv;
        const uint32_t lo = pack_bf(relu(y[0]), relu(y[1])), hi = pack_bf(relu(y[2]), relu(y[3]));
        *reinterpret_cast<uint2*>(&out[act_at(r, ch / 8 + 2 * n + kg / 2) + (kg & 1u) * 4]) =
            v ? make_uint2(lo, hi) : make_uint2(0u, 0u);
      }
    }
  });
}

struct ForwardArgs {
  // input: slot rows x0 [rows][16] bf16 with each series' K in Ks, or (feat
  // given) the caller's features with K from the descriptors
  const uint16_t* x0;
  uint32_t* Ks;
  const float* feat;
  uint64_t feat_rows;
  const ks_desc* desc;
  uint32_t max_K, SR, num_series, tiles_per_series;
  const uint16_t* w[4];
  const float* b[4];
  float* logits;  // slot rows, or
  float* out;     // the caller's rows aux_offset + t (series that fit in out_rows)
  uint64_t out_rows;
  // training: the input rows and activations kept for the backward pass (slot
  // rows), each series' K written to Ks; the labels >= 1 counted into nsig and
  // the loss cleared (labels given) by the first workgroup
  uint16_t* keep[4];
  const int32_t* labels;
  uint32_t* nsig;
  float* loss;
};

// K of series s under the caller's descriptor, 0 where it is skipped.
__device__ __forceinline__ uint32_t feature_K(const ks_desc& d, uint32_t max_K, uint64_t feat_rows) {
  return d.K >= 2 && d.K <= max_K && d.aux_offset <= feat_rows && d.K <= feat_rows - d.aux_offset ? d.K : 0u;
}

template <bool FEAT, bool TRAIN>
__global__ __launch_bounds__(NTC) __attribute__((amdgpu_waves_per_eu(FWGS, FWGS))) void fused_forward_kernel(ForwardArgs A) {
  static_assert(FEAT || !TRAIN, "training starts from the caller's features");
  __shared__ __align__(16) FusedSmem sm;
  const uint32_t tid = threadIdx.x, lane = lane_id(), w = wave_id();
  const uint32_t m = lane & 15u, kg = lane >> 4;
  const uint32_t ch = 32 * (w & 1u), rh = w >> 1;  // this wave's channels and row blocks
  u32x4 W1[10][2], W2[10][2];
#pragma unroll
  for (int q = 0; q < 10; ++q)
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const uint32_t at = (ch + 16 * n + m) * 320 + q * 32 + kg * 8;
      W1[q][n] = *reinterpret_cast<const u32x4*>(A.w[1] + at);
      W2[q][n] = *reinterpret_cast<const u32x4*>(A.w[2] + at);
    }
  for (uint32_t q = tid; q < 2u * FW3; q += NTC) sm.w3[q] = q < 320u ? A.w[3][q] : (uint16_t)0;
  if (tid < 192u) sm.bias[tid] = A.b[tid / 64u][tid % 64u];
  const float bias3 = A.b[3][0];
  if (TRAIN && A.labels && blockIdx.x == 0) {
    if (tid == 0) sm.count = 0;
    __syncthreads();
    uint32_t local = 0;
    for (uint32_t s = tid; s < A.num_series; s += NTC) local += A.labels[s] >= 1 ? 1u : 0u;
    atomicAdd(&sm.count, local);
    __syncthreads();
    if (tid == 0) {
      *A.nsig = sm.count;
      *A.loss = 0.0f;
    }
  }
  const uint64_t ntiles = (uint64_t)A.num_series * A.tiles_per_series;
  for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const uint32_t ser = (uint32_t)(tile / A.tiles_per_series), f = (uint32_t)(tile - (uint64_t)ser * A.tiles_per_series);
    ks_desc d;
    uint32_t K;
    if constexpr (FEAT) {
      d = A.desc[ser];
      K = feature_K(d, A.max_K, A.feat_rows);
    } else {
      K = A.Ks[ser];
    }
    if (TRAIN && f == 0 && tid == 0) A.Ks[ser] = K;
    const uint32_t nt = (K + FT - 1) / FT;
    if (f >= nt) continue;  // block-uniform
    const uint32_t len = (K + nt - 1) / nt, t0 = f * len, T = min(len, K - t0);
    const uint64_t base = (uint64_t)ser * A.SR + 2;
    // the tile's own rows of a finished LDS buffer (from row `off`) to memory
    auto keep = [&](int l, uint32_t off) {
      if constexpr (TRAIN) {
        const uint16_t* in = l == 0 ? sm.x : sm.act[(l + 1) & 1];
        const uint32_t sh = l == 0 ? 1u : 3u, msk = (1u << sh) - 1u;
        for (uint32_t q = tid; q < T << sh; q += NTC) {
          const uint32_t r = off + (q >> sh), c = q & msk;
          *reinterpret_cast<u32x4*>(A.keep[l] + (((base + t0) << sh) + q) * 8) =
              *reinterpret_cast<const u32x4*>(&in[l == 0 ? r * FXS + c * 8 : act_at(r, c)]);
        }
      }
    };
    __syncthreads();
    if constexpr (FEAT) {  // one row per thread: nine features and the two position channels
      static_assert(FT + 16 <= NTC, "a thread per input row");
      if (tid < T + 16) {
        const int32_t t = (int32_t)(t0 + tid) - 8;
        u32x4 lo{0u, 0u, 0u, 0u}, hi{0u, 0u, 0u, 0u};
        if ((uint32_t)t < K) {
          const float* p = A.feat + (d.aux_offset + (uint32_t)t) * 9;
          lo = u32x4{pack_bf(p[0], p[1]), pack_bf(p[2], p[3]), pack_bf(p[4], p[5]), pack_bf(p[6], p[7])};
          hi = u32x4{pack_bf(p[8], pos_frac((uint32_t)t, K)), pack_bf(pos_centre((uint32_t)t, K), 0.0f), 0u, 0u};
        }
        *reinterpret_cast<u32x4*>(&sm.x[tid * FXS]) = lo;
        *reinterpret_cast<u32x4*>(&sm.x[tid * FXS + 8]) = hi;
      }
    } else {
      for (uint32_t q = tid; q < 2u * (T + 16); q += NTC) {
        const uint32_t r = q >> 1, h = q & 1u;
        const int32_t t = (int32_t)(t0 + r) - 8;
        u32x4 v{0u, 0u, 0u, 0u};
        if ((uint32_t)t < K) v = *reinterpret_cast<const u32x4*>(A.x0 + (base + (uint32_t)t) * 16 + h * 8);
        *reinterpret_cast<u32x4*>(&sm.x[r * FXS + h * 8]) = v;
      }
    }
    __syncthreads();
    keep(0, 8);
    const int32_t tb = (int32_t)t0 - 6;
    {
      u32x4 W0[3][2];
      const uint16_t* w0p = A.w[0];
      asm volatile("" : "+v"(w0p));  // read per tile: keeps the compiler from pinning W0 in registers
#pragma unroll
      for (int q = 0; q < 3; ++q)
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          const int j0 = q * 32 + (int)kg * 8;
          W0[q][n] = j0 < 80 ? *reinterpret_cast<const u32x4*>(w0p + (ch + 16 * n + m) * 80 + j0) : u32x4{0u, 0u, 0u, 0u};
        }
      fused_layer<16, 3>(sm.x, W0, sm.bias, sm.act[0], tb, K, (T + 12 + 15) / 16, rh, ch, lane);
    }
    __syncthreads();
    keep(1, 6);
    fused_layer<64, 10>(sm.act[0], W1, sm.bias + 64, sm.act[1], tb + 2, K, (T + 8 + 15) / 16, rh, ch, lane);
    __syncthreads();
    keep(2, 4);
    fused_layer<64, 10>(sm.act[1], W2, sm.bias + 128, sm.act[0], tb + 4, K, (T + 4 + 15) / 16, rh, ch, lane);
    __syncthreads();
    keep(3, 2);
    // last layer (one output channel, of 16): wave w takes row blocks w and w + 4
    const uint32_t nb = (T + 15) / 16;
    if (w < nb) {
      const uint32_t ln = renew(lane), m = ln & 15u, kg = ln >> 4;
      const uint16_t* w3row = &sm.w3[m == 0 ? 0 : FW3];
      const bool two = w + 4 < nb;
      const uint16_t* in = &sm.act[0][act_at(16 * w + m, kg)];
      f32x4 acc[2];
      acc[0] = acc[1] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int q = 0; q < 10; ++q) {
        const int at = (q / 2) * FPS + (q & 1) * 16;
        const u32x4 a = *reinterpret_cast<const u32x4*>(&w3row[q * 32 + kg * 8]);
        acc[0] = mfma16(a, *reinterpret_cast<const u32x4*>(&in[at]), acc[0]);
        if (two) acc[1] = mfma16(a, *reinterpret_cast<const u32x4*>(&in[at + 64 * FPS]), acc[1]);
      }
      if (kg == 0) {  // channel 0 of row m of each block
        float* dst = A.logits + base;
        if (FEAT && A.out)
          dst = d.aux_offset <= A.out_rows && K <= A.out_rows - d.aux_offset ? A.out + d.aux_offset : nullptr;
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          const uint32_t r = 16 * w + 64 * g + m;
          if (r < T && dst) dst[t0 + r] = acc[g][0] + bias3;
        }
      }
    }
  }
}

// ------------------------------------------------------------ fused backward
// The input gradients of layers 3, 2, 1 over tiles of at most BT rows of one
// series, on the forward's plan (32 channels and half of the row blocks per
// wave, both 64-channel layers' flipped weights in registers): dz -> dy2 -> dy1
// -> dy0, the gradients at the pre-activations, masked where the layer input
// (a3, a2, a1) is 0 and zero outside the series. The LDS buffers hold bf16 rows
// for the next layer; the fp32 values of the tile's own rows go to memory for
// the weight and bias gradients. (A launch per layer with element-wise 2-byte
// loads took 27 + 52 + 51 us on 69632 rows, this one 28.)
//
// dz row r is series row t0 - 6 + r; dy2, dy1, dy0 row r is t0 - 4 + r, t0 - 2 +
// r, t0 + r. BT + 8 = 128 rows of dy2 make eight blocks.
constexpr int BT = 120;

struct BackSmem {
  uint16_t dy[2][2 * FPL];
  uint16_t dz[FROWS + 4];
  uint16_t w3[64 * 8];    // flipped taps of layer 3: [input channel][tap]
};

struct BackwardArgs {
  const float* dz;  // slot rows
  const uint32_t* Ks;
  uint32_t SR, num_series, tiles_per_series;
  const uint16_t* a[3];   // a3, a2, a1, slot rows
  const uint16_t* wb[3];  // layers 3, 2, 1: [cin][5 cout_pad], taps flipped
  float* dy[3];           // dy2, dy1, dy0, slot rows
};

__global__ __launch_bounds__(NTC) __attribute__((amdgpu_waves_per_eu(FWGS, FWGS))) void fused_backward_kernel(BackwardArgs A) {
  __shared__ __align__(16) BackSmem sm;
  const uint32_t tid = threadIdx.x, lane = lane_id(), w = wave_id();
  const uint32_t m = lane & 15u, kg = lane >> 4;
  const uint32_t ch = 32 * (w & 1u), rh = w >> 1;
  u32x4 W2[10][2], W1[10][2];
#pragma unroll
  for (int q = 0; q < 10; ++q)
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const uint32_t at = (ch + 16 * n + m) * 320 + q * 32 + kg * 8;
      W2[q][n] = *reinterpret_cast<const u32x4*>(A.wb[1] + at);
      W1[q][n] = *reinterpret_cast<const u32x4*>(A.wb[2] + at);
    }
  for (uint32_t q = tid; q < 64u * 8u; q += NTC) sm.w3[q] = (q & 7u) < 5u ? A.wb[0][(q >> 3) * 80 + (q & 7u) * 16] : (uint16_t)0;
  const uint32_t ntiles = A.num_series * A.tiles_per_series;
  for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const uint32_t ser = tile / A.tiles_per_series, f = tile - ser * A.tiles_per_series;
    const uint32_t K = (uint32_t)__builtin_amdgcn_readfirstlane((int)A.Ks[ser]);
    const uint32_t nt = (K + BT - 1) / BT;
    if (f >= nt) continue;  // block-uniform
    const uint32_t len = (K + nt - 1) / nt, t0 = f * len, T = min(len, K - t0);
    const uint64_t base = (uint64_t)ser * A.SR + 2;
    // the layer inputs whose zeros mask a lane's products, fetched before the
    // products are made
    auto masks = [&](auto gtag, int l, uint2* mk, uint32_t r0, uint32_t kg, uint32_t off) {
      constexpr int G = decltype(gtag)::value;
#pragma unroll
      for (int g = 0; g < G; ++g)
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          const uint32_t t = t0 + r0 + 32 * g - off;  // wraps below row 0: not < K
          mk[g * 2 + n] = t < K ? *reinterpret_cast<const uint2*>(A.a[l] + (base + t) * 64 + ch + 16 * n + 4 * kg)
                                : make_uint2(0u, 0u);
        }
    };
    // masks one layer's products and stores them as out rows; the tile's own
    // rows (off .. off + T - 1) also in fp32
    auto finish = [&](auto gtag, int l, const f32x4* acc, const uint2* mks, uint32_t r0, uint32_t kg, uint32_t off,
                      uint16_t* out) {
      constexpr int G = decltype(gtag)::value;
#pragma unroll
      for (int n = 0; n < 2; ++n) {
        const uint32_t c = ch + 16 * n + 4 * kg;
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const uint32_t r = r0 + 32 * g;
          const uint32_t t = t0 + r - off;  // wraps below row 0: not < K
          const bool v = t < K;
          const uint2 mk = mks[g * 2 + n];
          f32x4 d = acc[g * 2 + n];
          d[0] = (mk.x & 0xffffu) ? d[0] : 0.0f;
          d[1] = (mk.x >> 16) ? d[1] : 0.0f;
          d[2] = (mk.y & 0xffffu) ? d[2] : 0.0f;
          d[3] = (mk.y >> 16) ? d[3] : 0.0f;
          if (l < 2)  // dy0 feeds no further layer
            *reinterpret_cast<uint2*>(&out[act_at(r, c / 8) + (c & 4u)]) =
                make_uint2(pack_bf(d[0], d[1]), pack_bf(d[2], d[3]));
          if (v && r >= off && r < off + T) *reinterpret_cast<f32x4*>(A.dy[l] + (base + t) * 64 + c) = d;
        }
      }
    };
    auto layer = [&](int l, const u32x4 (&Wt)[10][2], const uint16_t* in, uint32_t rows, uint32_t off, uint16_t* out) {
      for_blocks<4>(((rows + 15) / 16 + 1 - rh) / 2, [&](auto tag, uint32_t b0) {
        constexpr int G = decltype(tag)::value;
        const uint32_t ln = renew(lane), kg = ln >> 4, r0 = 32 * b0 + 16 * rh + (ln & 15u);
        f32x4 acc[G][2];
        uint2 mk[G * 2];
        masks(tag, l, mk, r0, kg, off);
        conv_blocks<64, 10, G>(in + act_at(r0, kg), Wt, kg, acc);
        finish(tag, l, &acc[0][0], mk, r0, kg, off, out);
      });
    };
    __syncthreads();
    for (uint32_t r = tid; r < (uint32_t)FROWS + 4; r += NTC) {
      const uint32_t t = t0 + r - 6;
      sm.dz[r] = t < K && r < T + 12 ? f2bf(A.dz[base + t]) : (uint16_t)0;
    }
    __syncthreads();
    // layer 3: one channel, so of each 32-deep step only the first element of
    // lane groups 0 and 2 (taps 2 q and 2 q + 1) is not 0
    for_blocks<4>(((T + 8 + 15) / 16 + 1 - rh) / 2, [&](auto tag, uint32_t b0) {
      constexpr int G = decltype(tag)::value;
      const uint32_t ln = renew(lane), m = ln & 15u, kg = ln >> 4, r0 = 32 * b0 + 16 * rh + m;
      f32x4 acc[G][2];
      uint2 mk[G * 2];
      masks(tag, 0, mk, r0, kg, 4);
#pragma unroll
      for (int q = 0; q < 3; ++q) {
        const uint32_t k = 2 * q + (kg >> 1);
        const bool on = (kg & 1u) == 0 && k < 5u;
        u32x4 a[2];
#pragma unroll
        for (int n = 0; n < 2; ++n) a[n] = u32x4{on ? (uint32_t)sm.w3[(ch + 16 * n + m) * 8 + k] : 0u, 0u, 0u, 0u};
#pragma unroll
        for (int g = 0; g < G; ++g) {
          const u32x4 x{on ? (uint32_t)sm.dz[r0 + 32 * g + k] : 0u, 0u, 0u, 0u};
#pragma unroll
          for (int n = 0; n < 2; ++n) acc[g][n] = mfma16(a[n], x, q == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[g][n]);
        }
      }
      finish(tag, 0, &acc[0][0], mk, r0, kg, 4, sm.dy[0]);
    });
    __syncthreads();
    layer(1, W2, sm.dy[0], T + 4, 2, sm.dy[1]);
    __syncthreads();
    layer(2, W1, sm.dy[1], T, 0, nullptr);
  }
}

// ------------------------------------------------------------ weight gradients
//   dW[o][k][i] = sum over rows t of bf16(dY[t][o]) X[t + k - 2][i],
//   db[o] = sum over rows t of dY[t][o]
// as GEMMs reduced over rows, one launch for the four layers (blockIdx.y).
// Workgroup g takes the 64-row tiles g, g + G, ... of the slot rows and keeps its
// sums in registers; the partials are added in the order of g by finish_kernel.
// The order of every sum is fixed, whatever tile shape would be faster (weights
// in 32-row matrix steps, biases row after row in fp32): the first Adam step of
// a parameter is the sign of its gradient, so one whose gradient is within
// rounding of 0 moves by 2 lr when any order changes, and b3's gradient is
// nothing but the rounding of all the others (a softmax gradient sums to 0).
// Both operands need eight consecutive rows of one channel per lane: the tiles
// lie in LDS as they do in memory (rows of channels, whole 16-byte copies) and
// ds_read_b64_tr_b16 reads them transposed, four rows by 16 channels per 16
// lanes, at any row, so a tap is a row offset. (Transposed copies in LDS cost a
// 2-byte write per element and eight 2-byte reads per operand and tap: 154 us
// for a 64 x 64 layer of 69632 rows.) A wave takes 16 input channels, all 64
// output channels and the five taps: 18 operand reads for 20 MFMAs. Rows 160
// bytes apart put the four rows of a read on different banks.
constexpr int DT = 64;         // rows per tile
constexpr int DST = 64 + 16;   // LDS row stride (bf16)
constexpr uint32_t kDwGrid = 256;  // workgroups (partials) per layer at most
constexpr uint32_t kBiasPart = 224;  // bias partials per workgroup (193, padded)
constexpr uint32_t kDwN0 = 5 * 64 * 16, kDwN1 = 5 * 64 * 64, kDwN3 = 5 * 64;
constexpr uint32_t kDwPart = kDwN0 + 2 * kDwN1 + kDwN3;  // partial sums of a workgroup, all layers
__host__ __device__ constexpr uint32_t dw_base(int l) { return l == 0 ? 0u : l == 1 ? kDwN0 : l == 2 ? kDwN0 + kDwN1 : kDwN0 + 2 * kDwN1; }
__host__ __device__ constexpr uint32_t dw_size(int l) { return l == 0 ? kDwN0 : l == 3 ? kDwN3 : kDwN1; }

struct DwArgs {
  const float* dz;
  const float* dy[3];     // of layers 0, 1, 2
  const uint16_t* x[4];   // inputs of layers 0 .. 3
  const uint32_t* Ks;
  uint32_t SR, num_series;
  float* part;            // layer l, workgroup g at G dw_base(l) + g dw_size(l): [k][o][i] ([k][i] for layer 3)
  float* bpart;           // [g][kBiasPart]: b0[64] b1[64] b2[64] b3
};

// Rows r .. r + 7 (r = 8 kg of a 32-row step) of 16 channels from c0, transposed:
// lane (m, kg) gets channel c0 + m of them. tile: LDS rows of DST, or of 16
// channels unpadded.
template <int ST>
__device__ __forceinline__ u32x4 read_rows(const uint16_t* tile, uint32_t r, uint32_t c0, uint32_t lane) {
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4* lds_p;
  const uint16_t* p = tile + (r + ((lane & 15u) >> 2)) * ST + c0 + (lane & 3u) * 4;
  const s16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(p));
  const s16x4 b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_p)(p + 4 * ST));
  const uint2 ua = __builtin_bit_cast(uint2, a), ub = __builtin_bit_cast(uint2, b);
  return u32x4{ua.x, ua.y, ub.x, ub.y};
}

struct DwSmem {
  uint16_t xs[(DT + 4) * DST];  // X rows r0 - 2 + r
  uint16_t ys[DT * DST];        // dY rows r0 + r (layer 3: dz) in bf16
  float yf[DT * 64];            // and in fp32
};

template <int L>
__device__ __forceinline__ void dw_layer(DwSmem& sm, const DwArgs& A) {
  constexpr int CX = L == 0 ? 16 : 64;       // input channels
  constexpr int XST = L == 0 ? 16 : DST;
  constexpr int NT = L == 1 || L == 2 ? 4 : 1;  // output-channel tiles per wave
  const uint32_t tid = threadIdx.x, lane = lane_id(), w = wave_id();
  const uint32_t m = lane & 15u, kg = lane >> 4;
  f32x4 acc[KW][NT];
#pragma unroll
  for (int k = 0; k < KW; ++k)
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[k][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  float db = 0.0f;  // bias gradient of channel tid
  const uint64_t rows = (uint64_t)A.num_series * A.SR;
  const uint64_t ntiles = (rows + DT - 1) / DT;
  for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const uint64_t r0 = tile * DT;
    const uint32_t s0 = (uint32_t)(r0 / A.SR), rem = (uint32_t)(r0 - (uint64_t)s0 * A.SR);
    // slot row r0 + r (r from -2 on) holds data; the last two rows of a slot never do
    auto valid = [&](int32_t r) {
      const int32_t p = (int32_t)rem + r;
      if (p < 2) return false;
      const uint32_t ds = (uint32_t)p / A.SR, t = (uint32_t)p - ds * A.SR;
      return s0 + ds < A.num_series && t >= 2u && t - 2u < A.Ks[s0 + ds];
    };
    __syncthreads();
    for (uint32_t q = tid; q < (DT + 4) * (CX / 8u); q += NTC) {
      const int32_t r = (int32_t)(q / (CX / 8u)) - 2;
      const uint32_t c = q % (CX / 8u) * 8;
      u32x4 v{0u, 0u, 0u, 0u};
      if (valid(r)) v = *reinterpret_cast<const u32x4*>(A.x[L] + (r0 + r) * CX + c);
      *reinterpret_cast<u32x4*>(&sm.xs[(r + 2) * XST + c]) = v;
    }
    if constexpr (L == 3) {
      if (tid < (uint32_t)DT) {
        const float z = valid((int32_t)tid) ? A.dz[r0 + tid] : 0.0f;
        sm.yf[tid] = z;
        sm.ys[tid] = f2bf(z);
      }
    } else {
      for (uint32_t q = tid; q < DT * 16u; q += NTC) {
        const uint32_t r = q >> 4, c = (q & 15u) * 4;
        f32x4 v{0.f, 0.f, 0.f, 0.f};
        if (valid((int32_t)r)) v = *reinterpret_cast<const f32x4*>(A.dy[L] + (r0 + r) * 64 + c);
        *reinterpret_cast<f32x4*>(&sm.yf[r * 64 + c]) = v;
        *reinterpret_cast<uint2*>(&sm.ys[r * DST + c]) = make_uint2(pack_bf(v[0], v[1]), pack_bf(v[2], v[3]));
      }
    }
    __syncthreads();
    if (tid < (L == 3 ? 1u : 64u)) {
#pragma unroll 16
      for (int r = 0; r < DT; ++r) db += sm.yf[L == 3 ? r : r * 64 + (int)tid];
    }
#pragma unroll
    for (uint32_t q = 0; q < DT / 32; ++q) {
      const uint32_t r = 32 * q + 8 * kg;
      u32x4 a[NT];
      if constexpr (L == 3) {  // one output channel of 16
        const u32x4 z = *reinterpret_cast<const u32x4*>(&sm.ys[r]);
        a[0] = m == 0 ? z : u32x4{0u, 0u, 0u, 0u};
      } else {
#pragma unroll
        for (int t = 0; t < NT; ++t) a[t] = read_rows<DST>(sm.ys, r, 16 * (NT == 4 ? t : (int)w), lane);
      }
#pragma unroll
      for (int k = 0; k < KW; ++k) {
        const u32x4 x = read_rows<XST>(sm.xs, r + k, L == 0 ? 0 : 16 * w, lane);
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[k][t] = mfma16(a[t], x, acc[k][t]);
      }
    }
  }
  float* out = A.part + (uint64_t)gridDim.x * dw_base(L) + (uint64_t)blockIdx.x * dw_size(L);
#pragma unroll
  for (int k = 0; k < KW; ++k) {
    if constexpr (L == 3) {
      if (kg == 0) out[k * 64 + 16 * w + m] = acc[k][0][0];
    } else {
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          out[(k * 64 + 16 * (NT == 4 ? t : (int)w) + 4 * kg + e) * CX + (L == 0 ? 0 : 16 * w) + m] = acc[k][t][e];
    }
  }
  if (tid < (L == 3 ? 1u : 64u)) A.bpart[blockIdx.x * kBiasPart + L * 64u + tid] = db;
}

__global__ __launch_bounds__(NTC) __attribute__((amdgpu_waves_per_eu(4))) void dw_kernel(DwArgs A) {
  __shared__ __align__(16) DwSmem sm;
  switch (blockIdx.y) {
    case 0: dw_layer<0>(sm, A); break;
    case 1: dw_layer<1>(sm, A); break;
    case 2: dw_layer<2>(sm, A); break;
    default: dw_layer<3>(sm, A);
  }
}

// ---------------------------------------------------------------- parameters
//
// Master vector (fp32, 44993): W0[64][11][5] b0[64] W1[64][64][5] b1[64]
// W2[64][64][5] b2[64] W3[1][64][5] b3[1]. Input channels of layer 0: the nine
// decile features, then t / (K-1) and 4 t (K - t) / K^2.
struct Layer {
  int cin, cout, cin_pad, cout_pad;
  uint32_t w_off, b_off;
};
__device__ __host__ inline Layer layer_info(int l) {
  switch (l) {
    case 0: return Layer{11, 64, 16, 64, 0u, 3520u};
    case 1: return Layer{64, 64, 64, 64, 3584u, 24064u};
    case 2: return Layer{64, 64, 64, 64, 24128u, 44608u};
    default: return Layer{64, 1, 64, 16, 44672u, 44992u};
  }
}
constexpr uint32_t kNumParams = 44993;

// Entries of all shadow copies (forward weights and biases of every layer).
constexpr uint32_t kShadowEntries = (64 * 5 * 16 + 64) + 2 * (64 * 5 * 64 + 64) + (16 * 5 * 64 + 16);

// Device copies used by the kernels.
struct Shadow {
  uint16_t* wf[4];  // forward: [cout_pad][5 cin_pad], j = k cin_pad + i
  uint16_t* wb[4];  // backward data (l >= 1): [cin_pad][5 cout_pad], j = k cout_pad + o, tap flipped
  float* b[4];      // [cout_pad]
};

// Rebuild every shadow copy from the master vector (one thread per entry).
__global__ __launch_bounds__(NTC) void shadow_kernel(const float* __restrict__ theta, Shadow sh) {
  const uint32_t t = blockIdx.x * NTC + threadIdx.x;
  uint32_t base = 0;
  for (int l = 0; l < 4; ++l) {
    const Layer L = layer_info(l);
    const uint32_t nf = (uint32_t)(L.cout_pad * KW * L.cin_pad);
    if (t >= base && t < base + nf) {
      const uint32_t q = t - base, o = q / (KW * L.cin_pad), j = q - o * (KW * L.cin_pad);
      const uint32_t k = j / L.cin_pad, i = j - k * L.cin_pad;
      const float v = ((int)o < L.cout && (int)i < L.cin) ? theta[L.w_off + (o * L.cin + i) * KW + k] : 0.0f;
      sh.wf[l][q] = f2bf(v);
      if (l >= 1) {
        // wb[i][k' cout_pad + o] = W[o][i][4 - k']
        const uint32_t kp = KW - 1 - k;
        sh.wb[l][i * (KW * L.cout_pad) + kp * L.cout_pad + o] = f2bf(v);
      }
    }
    base += nf;
    if (t >= base && t < base + (uint32_t)L.cout_pad) {
      const uint32_t o = t - base;
      sh.b[l][o] = (int)o < L.cout ? theta[L.b_off + o] : 0.0f;
    }
    base += L.cout_pad;
  }
}

// Adds the G <= kDwGrid partials of every parameter's gradient, in order, and, with `apply`, makes its Adam step (Kingma & Ba) and
// rewrites the device copies that the kernels read. A workgroup takes kFinP
// parameters (in the partials' order: weights of layers 0 .. 3, then the
// biases): all its threads fetch their partials to LDS at once, and one thread
// per parameter adds them there. (A thread walking its 256 partials in memory
// took 61 us per layer on the latency of its loads.) The padding of the copies
// stays as shadow_kernel left it (0).
constexpr uint32_t kFinP = 32;  // parameters of a workgroup
__global__ __launch_bounds__(NTC) void finish_kernel(const float* __restrict__ part, uint32_t G,
                                                     const float* __restrict__ bpart,
                                                     float* __restrict__ theta, float* __restrict__ mom1,
                                                     float* __restrict__ mom2, float* __restrict__ grad_out, Shadow sh,
                                                     float lr, float bc1, float bc2, int apply) {
  __shared__ float red[kDwGrid][kFinP];
  constexpr uint32_t GRP = NTC / kFinP;
  const uint32_t c = threadIdx.x % kFinP, grp = threadIdx.x / kFinP;
  const uint32_t q = blockIdx.x * kFinP + c;
  const bool bias = q >= kDwPart;
  int l = 3;
  const float* src = bpart + (q - kDwPart);  // the padding past 193 is read and dropped
  uint32_t stride = kBiasPart;
  if (!bias) {
    l = q < dw_base(1) ? 0 : q < dw_base(2) ? 1 : q < dw_base(3) ? 2 : 3;
    src = part + (uint64_t)G * dw_base(l) + (q - dw_base(l));
    stride = dw_size(l);
  }
#pragma unroll 8
  for (uint32_t g = grp; g < G; g += GRP) red[g][c] = src[(uint64_t)g * stride];
  __syncthreads();
  if (grp) return;
  float gv = 0.0f;
#pragma unroll 8
  for (uint32_t g = 0; g < G; ++g) gv += red[g][c];
  uint32_t p, o = 0, k = 0, i = 0;
  if (!bias) {
    const Layer L = layer_info(l);
    const uint32_t r = q - dw_base(l), oi = (uint32_t)(L.cout * L.cin_pad);
    k = r / oi;
    o = (r - k * oi) / (uint32_t)L.cin_pad;
    i = r - k * oi - o * (uint32_t)L.cin_pad;
    if (i >= (uint32_t)L.cin) return;
    p = L.w_off + (o * L.cin + i) * KW + k;
  } else {
    const uint32_t r = q - kDwPart;
    if (r > 192u) return;
    l = (int)(r / 64u);
    o = r % 64u;
    p = layer_info(l).b_off + o;
  }
  grad_out[p] = gv;
  if (!apply) return;
  const float m = 0.9f * mom1[p] + 0.1f * gv;
  const float v = 0.999f * mom2[p] + 0.001f * gv * gv;
  mom1[p] = m;
  mom2[p] = v;
  const float th = theta[p] - lr * (m / bc1) / (sqrtf(v / bc2) + 1e-8f);
  theta[p] = th;
  const Layer L = layer_info(l);
  if (bias) {
    sh.b[l][o] = th;
  } else {
    sh.wf[l][(o * KW + k) * L.cin_pad + i] = f2bf(th);
    if (l >= 1) sh.wb[l][(i * KW + KW - 1 - k) * L.cout_pad + o] = f2bf(th);
  }
}
constexpr uint32_t kFinishGrid = (kDwPart + kBiasPart) / kFinP;
static_assert(dw_base(1) % kFinP == 0 && dw_base(2) % kFinP == 0 && dw_base(3) % kFinP == 0 && kDwPart % kFinP == 0 &&
                  kBiasPart % kFinP == 0,
              "whole workgroups, each of one kind");

// p[i] = 0 for i < n (a plain fill kernel rather than a memset node, so that a
// captured graph replays it like any other kernel).
__global__ __launch_bounds__(NTC) void zero_kernel(float* __restrict__ p, uint32_t n) {
  const uint32_t i = blockIdx.x * NTC + threadIdx.x;
  if (i < n) p[i] = 0.0f;
}

// ---------------------------------------------------------------- series heads

// Softmax over rows t = 1..K-1 of each series (one wave per series).
// Training (labels != null): loss += -log p[label] / B_sig and dlogit rows (fp32)
// = (p - onehot) / B_sig on rows 1..K-1 of series with label >= 1, zero on the
// series' other rows. Inference: proposal =
// argmax (smallest row on ties), confidence = softmax mass of rows within
// +-w of it.
__global__ __launch_bounds__(NTC) void softmax_kernel(const float* __restrict__ logits, uint32_t num_series,
                                                      uint32_t SR, const uint32_t* __restrict__ Ks,
                                                      const int32_t* __restrict__ labels,
                                                      const uint32_t* __restrict__ nsig, float* __restrict__ loss,
                                                      float* __restrict__ dz, uint32_t w,
                                                      int32_t* __restrict__ proposal, float* __restrict__ conf) {
  const uint32_t lane = lane_id();
  const uint32_t s = blockIdx.x * (NTC / kWave) + wave_id();
  if (s >= num_series) return;
  const uint32_t K = Ks[s];
  const uint64_t base = (uint64_t)s * SR + 2;
  if (K < 2) {
    if (proposal && lane == 0) {
      proposal[s] = 0;
      conf[s] = 0.0f;
    }
    return;
  }
  // max and argmax over t = 1..K-1
  float mx = -3.402823466e38f;
  uint32_t am = 0xffffffffu;
  for (uint32_t t = 1 + lane; t < K; t += kWave) {
    const float z = logits[base + t];
    if (z > mx || (z == mx && t < am)) {
      mx = z;
      am = t;
    }
  }
  for (int o = 32; o >= 1; o >>= 1) {
    const float zm = __shfl_xor(mx, o);
    const uint32_t ta = (uint32_t)__shfl_xor((int)am, o);
    if (zm > mx || (zm == mx && ta < am)) {
      mx = zm;
      am = ta;
    }
  }
  float sum = 0.0f;
  for (uint32_t t = 1 + lane; t < K; t += kWave) sum += __expf(logits[base + t] - mx);
  for (int o = 32; o >= 1; o >>= 1) sum += __shfl_xor(sum, o);
  if (proposal) {
    const uint32_t lo = am > w ? am - w : 1u, hi = min(K - 1, am + w);
    float part = 0.0f;
    for (uint32_t t = lo + lane; t <= hi; t += kWave) part += __expf(logits[base + t] - mx);
    for (int o = 32; o >= 1; o >>= 1) part += __shfl_xor(part, o);
    if (lane == 0) {
      proposal[s] = (int32_t)am;
      conf[s] = part / sum;
    }
  }
  if (dz) {
    const int32_t lab = labels[s];
    const bool use = lab >= 1 && (uint32_t)lab < K;
    const float inv = 1.0f / (float)max(*nsig, 1u);
    for (uint32_t t = lane; t < K; t += kWave) {
      float d = 0.0f;
      if (use && t >= 1) d = (__expf(logits[base + t] - mx) / sum - (t == (uint32_t)lab ? 1.0f : 0.0f)) * inv;
      dz[base + t] = d;
    }
    if (use && lane == 0) atomicAdd(loss, (logf(sum) - (logits[base + lab] - mx)) * inv);
  }
}

// Proposal without the network: the row after the largest jump of the per-row
// median (feature 5, the fifth decile), |f_t - f_(t-1)| in FP64 (exact for
// floats), ties to the smaller row; confidence 1 (always refined). One wave per
// series, features from the feature pass's slot rows.
__global__ __launch_bounds__(NTC) void median_jump_kernel(const float* __restrict__ feat, uint32_t num_series,
                                                          uint32_t SR, const uint32_t* __restrict__ Ks,
                                                          int32_t* __restrict__ proposal,
                                                          float* __restrict__ conf) {
  const uint32_t lane = lane_id();
  const uint32_t s = blockIdx.x * (NTC / kWave) + wave_id();
  if (s >= num_series) return;
  const uint32_t K = Ks[s];
  const uint64_t base = (uint64_t)s * SR + 2;
  double best = -1.0;
  uint32_t arg = 0;
  for (uint32_t t = 1 + lane; t < K; t += kWave) {
    const double j = fabs((double)feat[(base + t) * 9 + 4] - (double)feat[(base + t - 1) * 9 + 4]);
    if (j > best) {  // t grows within a lane: the first maximum is kept
      best = j;
      arg = t;
    }
  }
  for (int o = 32; o >= 1; o >>= 1) {
    const double bo = __shfl_xor(best, o);
    const uint32_t ao = (uint32_t)__shfl_xor((int)arg, o);
    if (bo > best || (bo == best && ao < arg && ao != 0)) {
      best = bo;
      arg = ao;
    }
  }
  if (lane == 0) {
    proposal[s] = K >= 2 ? (int32_t)arg : 0;
    conf[s] = K >= 2 ? 1.0f : 0.0f;
  }
}

// Caller logit gradients (fp32 rows aux_offset + t) -> slot rows; zero for a
// series that does not fit.
__global__ __launch_bounds__(NTC) void pack_dlogits_kernel(const float* __restrict__ src, uint64_t src_rows,
                                                           const ks_desc* __restrict__ desc, uint32_t num_series,
                                                           uint32_t SR, const uint32_t* __restrict__ Ks,
                                                           float* __restrict__ dz) {
  const uint32_t s = blockIdx.x;
  if (s >= num_series) return;
  const ks_desc d = desc[s];
  const uint32_t K = Ks[s];
  const bool fits = d.aux_offset <= src_rows && K <= src_rows - d.aux_offset;
  for (uint32_t t = threadIdx.x; t < K; t += NTC) dz[(uint64_t)s * SR + 2 + t] = fits ? src[d.aux_offset + t] : 0.0f;
}

// Per-layer values of one forward (and backward) pass -> caller rows
// aux_offset + t, as floats: acts row = x0[11] a1[64] a2[64] a3[64] logit
// (KS_CNN_TRACE_ACTS), gin row = dlogit, then the gradients at y2, y1, y0
// [64 each] (KS_CNN_TRACE_GRADS). dyf0 == nullptr: no backward values.
__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

__global__ __launch_bounds__(NTC) void trace_copy_kernel(const ks_desc* __restrict__ desc, uint32_t num_series,
                                                         uint32_t SR, const uint32_t* __restrict__ Ks,
                                                         const uint16_t* __restrict__ x0,
                                                         const uint16_t* __restrict__ a1,
                                                         const uint16_t* __restrict__ a2,
                                                         const uint16_t* __restrict__ a3,
                                                         const float* __restrict__ logits,
                                                         const float* __restrict__ dz, const float* __restrict__ dyf0,
                                                         const float* __restrict__ dyf1, const float* __restrict__ dyf2,
                                                         float* __restrict__ acts, float* __restrict__ gin,
                                                         uint64_t out_rows) {
  constexpr uint32_t NA = 11 + 3 * 64 + 1, NG = 1 + 3 * 64;
  const uint32_t s = blockIdx.x;
  if (s >= num_series) return;
  const ks_desc d = desc[s];
  const uint32_t K = Ks[s];
  if (!(d.aux_offset <= out_rows && K <= out_rows - d.aux_offset)) return;
  for (uint32_t q = threadIdx.x; q < K * NA && acts; q += NTC) {
    const uint32_t t = q / NA, c = q - t * NA;
    const uint64_t row = (uint64_t)s * SR + 2 + t;
    float v;
    if (c < 11) v = bf2f(x0[row * 16 + c]);
    else if (c < 75) v = bf2f(a1[row * 64 + (c - 11)]);
    else if (c < 139) v = bf2f(a2[row * 64 + (c - 75)]);
    else if (c < 203) v = bf2f(a3[row * 64 + (c - 139)]);
    else v = logits[row];
    acts[(d.aux_offset + t) * NA + c] = v;
  }
  for (uint32_t q = threadIdx.x; q < K * NG && gin && dyf0; q += NTC) {
    const uint32_t t = q / NG, c = q - t * NG;
    const uint64_t row = (uint64_t)s * SR + 2 + t;
    float v;
    if (c == 0) v = dz[row];
    else if (c < 65) v = dyf0[row * 64 + (c - 1)];
    else if (c < 129) v = dyf1[row * 64 + (c - 65)];
    else v = dyf2[row * 64 + (c - 129)];
    gin[(d.aux_offset + t) * NG + c] = v;
  }
}

}  // namespace cnn
}  // namespace ks
