// What the measurement workflow does around one detection: the outlier check
// and interval widening of workflow step 3 (ks_check_batch), the L2 segment
// alignment (ks_align_batch) and the cache-line-size scoring (ks_line_batch).
// All three run on results already on the device (ks_result, ks_row_stats);
// the reading of each rule is stated in include/ks_sweep.h.
#include <hip/hip_runtime.h>

#include <cmath>

#include "ks.h"
#include "ks_ctx.hpp"
#include "ks_scan.hpp"
#include "ks_select.hpp"
#include "ks_sweep.h"

static_assert(sizeof(ks_check) == 32 && sizeof(ks_line) == 24 && sizeof(ks_row_stats) == 32, "ABI struct sizes");

using namespace ks_host;

namespace {

typedef unsigned __int128 u128;

constexpr uint32_t kLineMaxJ = 64, kLineMaxA = 256;

// Lower median x_(floor((n - 1) / 2)).
struct MedianRank {
  static constexpr uint32_t kCount = 1;
  __device__ static uint32_t rank(uint32_t, uint32_t N) { return (N - 1) / 2; }
};

// Lower median of the values v(e) (step lane + 64 e) whose bit e of `in` is
// set, n >= 1 of them over the wave; wave-uniform. V: steps per lane (K <= 64 V).
template <int V, class Value>
__device__ __forceinline__ uint32_t lower_median(ks::SelLds& L, Value&& v, uint32_t in, uint32_t n, uint32_t lane) {
  uint32_t mn = 0xffffffffu, mx = 0u;
#pragma unroll
  for (int e = 0; e < V; ++e)
    if ((in >> e) & 1u) {
      mn = min(mn, v(e));
      mx = max(mx, v(e));
    }
  mn = ks::wave_min_u32(mn);
  mx = ks::wave_max_u32(mx);
  if (mx == mn) return mn;
  const uint32_t b = 32u - __clz(mx - mn);
  uint32_t k[V];
#pragma unroll
  for (int e = 0; e < V; ++e) k[e] = ((in >> e) & 1u) ? v(e) - mn : 0xffffffffu;
  const uint32_t key = ks::wave_select<V, MedianRank>(L, k, b, n, lane);
  return (uint32_t)__builtin_amdgcn_readfirstlane((int)key) + mn;  // lane 0 holds the median's key
}

// Level (median), spread (MAD) and disturbed-step count of the steps [a, b). One
// loop makes both medians, |v - 0| and |v - med|, so that the select is in the
// code once and inlined (called four times, it took its values through scratch
// memory: 300 sweeps of 2048 steps 20 us, 13 so).
template <int V>
__device__ __forceinline__ void side_check(ks::SelLds& L, const uint32_t (&v)[V], uint32_t a, uint32_t b, uint32_t k,
                                           uint32_t lane, uint32_t& med, uint32_t& mad, uint32_t& disturbed) {
  uint32_t in = 0;
#pragma unroll
  for (int e = 0; e < V; ++e) {
    const uint32_t i = lane + ks::kWave * (uint32_t)e;
    in |= (i >= a && i < b) ? 1u << e : 0u;
  }
  const uint32_t n = b - a;
  uint32_t from = 0;
  auto dev = [&](int e) { return v[e] > from ? v[e] - from : from - v[e]; };
#pragma unroll 1
  for (int pass = 0; pass < 2; ++pass) {
    const uint32_t m = lower_median<V>(L, dev, in, n, lane);
    if (pass == 0) from = m;
    else mad = m;
  }
  med = from;
  const uint64_t thr = (uint64_t)k * max(mad, max(1u, med / 64u));
  uint32_t cnt = 0;
#pragma unroll
  for (int e = 0; e < V; ++e) cnt += (uint32_t)__popcll(ks::ballot(((in >> e) & 1u) && dev(e) > thr));
  disturbed = cnt;
}

// One wave per sweep, a workgroup each, with as many steps per lane as max_K
// asks for (with 32 for every K and four sweeps to a workgroup, eight sweeps of
// 256 steps took 17 us, on scratch memory).
template <int V>
__global__ __launch_bounds__(64) void check_kernel(const ks_desc* __restrict__ desc, uint32_t num_series,
                                                    uint32_t max_K, const ks_result* __restrict__ res,
                                                    const ks_row_stats* __restrict__ stats, uint64_t stats_rows,
                                                    uint32_t edge, uint32_t k, ks_check* __restrict__ out) {
  static_assert(V * ks::kWave <= (int)KS_MAX_K, "steps of a sweep");
  __shared__ ks::SelLds L;
  const uint32_t lane = ks::lane_id();
  const uint32_t s = blockIdx.x;
  if (s >= num_series) return;
  const ks_desc d = desc[s];
  const ks_result r = res[s];
  const uint32_t K = d.K;
  const bool bad = K < 2 || K > max_K || (r.flags & (KS_BAD_SHAPE | KS_OUT_OF_RANGE)) != 0 ||
                   d.aux_offset > stats_rows || (uint64_t)K > stats_rows - d.aux_offset ||
                   ((r.flags & KS_SIGNIFICANT) && (r.cp < 1 || r.cp >= K));
  if (bad) {
    if (lane == 0) out[s] = ks_check{KS_CHECK_INVALID, 0u, 0, 0, 0u, 0u, 0u, 0u};
    return;
  }
  uint32_t v[V];
#pragma unroll
  for (int e = 0; e < V; ++e) {
    const uint32_t i = lane + ks::kWave * (uint32_t)e;
    v[e] = i < K ? stats[d.aux_offset + i].p50 : 0u;
  }
  const bool sig = (r.flags & KS_SIGNIFICANT) != 0;
  uint32_t med_lo = 0, mad_lo = 0, med_hi = 0, mad_hi = 0, disturbed = 0;
#pragma unroll 1
  for (uint32_t side = 0; side < (sig ? 2u : 1u); ++side) {
    uint32_t med, mad, n;
    side_check<V>(L, v, side ? r.cp : 0u, sig && !side ? r.cp : K, k, lane, med, mad, n);
    if (side == 0) {
      med_lo = med;
      mad_lo = mad;
    }
    med_hi = med;  // without a change the one side's
    mad_hi = mad;
    disturbed += n;
  }
  uint32_t flags = 0;
  int32_t lo = 0, hi = (int32_t)K;
  if (!sig) {
    flags |= KS_CHECK_NO_CHANGE;
    lo = -(int32_t)K;
    hi = 2 * (int32_t)K;
  } else {
    if (r.cp < edge) {
      flags |= KS_CHECK_EDGE_LOW;
      lo = -(int32_t)K;
    }
    if (K - r.cp < edge) {
      flags |= KS_CHECK_EDGE_HIGH;
      hi = 2 * (int32_t)K;
    }
  }
  if (disturbed) {
    flags |= KS_CHECK_DISTURBED;
    lo = min(lo, -(int32_t)(K / 2));
    hi = max(hi, (int32_t)(K + K / 2));
  }
  if (lane == 0) out[s] = ks_check{flags, disturbed, lo, hi, med_lo, med_hi, mad_lo, mad_hi};
}

// One thread per item: the nearest of T / k, k = floor(T / S) - 1 .. + 2
// (k >= 1), distances |S - T / k| = |S k - T| / k compared exactly.
__global__ __launch_bounds__(256) void align_kernel(const uint64_t* __restrict__ measured,
                                                    const uint64_t* __restrict__ total, uint32_t n,
                                                    uint32_t* __restrict__ segments, double* __restrict__ aligned,
                                                    double* __restrict__ distance) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i >= n) return;
  const uint64_t S = measured[i], T = total[i];
  constexpr uint64_t kLim = 1ull << 50;
  if (S < 1 || T < 1 || S >= kLim || T >= kLim || T / S > 0xfffffff0ull) {
    segments[i] = 0;
    aligned[i] = NAN;
    distance[i] = NAN;
    return;
  }
  const uint64_t k0 = T / S;
  uint64_t bk = 0, bnum = 0;
  for (uint64_t kk = k0 > 1 ? k0 - 1 : 1; kk <= k0 + 2; ++kk) {
    const uint64_t a = S * kk;  // <= T + 2 S < 2^52
    const uint64_t num = a > T ? a - T : T - a;
    if (bk == 0 || (u128)num * bk < (u128)bnum * kk) {
      bk = kk;
      bnum = num;
    }
  }
  segments[i] = (uint32_t)bk;
  aligned[i] = (double)T / (double)bk;      // both exact in FP64
  distance[i] = (double)bnum / (double)T;   // bnum < 2^52: exact
}

// The scores of one experiment's strides w, w + step, ... by the calling wave,
// lanes over the array sizes (a = lane + 64 t).
__device__ __forceinline__ void line_scores(const ks_row_stats* __restrict__ x, uint32_t A, uint32_t J, uint32_t w,
                                            uint32_t step, uint32_t lane, uint64_t* score) {
  constexpr int T = kLineMaxA / ks::kWave;
  uint32_t P[T], M[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const uint32_t a = lane + ks::kWave * (uint32_t)t;
    P[t] = a < A ? x[a].p50 : 0u;
    M[t] = a < A ? x[(uint64_t)(J - 1) * A + a].p50 : 0u;
  }
  for (uint32_t j = w; j < J; j += step) {
    uint64_t acc = 0;
#pragma unroll
    for (int t = 0; t < T; ++t) {
      const uint32_t a = lane + ks::kWave * (uint32_t)t;
      if (a < A) {
        const uint32_t v = x[(uint64_t)j * A + a].p50;
        const uint64_t dp = v > P[t] ? v - P[t] : P[t] - v;
        const uint64_t dm = v > M[t] ? v - M[t] : M[t] - v;
        const uint64_t q = dp + dm ? (dp << 32) / (dp + dm) : 0ull;
        acc += (uint64_t)(a + 1) * q;  // < 2^8 * 2^32 per term, < 2^48 summed
      }
    }
    uint32_t unused = 0;
    ks::wave_total_32_64(unused, acc);
    if (lane == 0) score[j] = acc;
  }
}

// The record of one experiment from its scores (one thread).
__device__ __forceinline__ ks_line line_record(const uint64_t* score, uint32_t A, uint32_t J,
                                               const uint32_t* __restrict__ strides) {
  const uint64_t W = (uint64_t)A * (A + 1) / 2;
  const uint64_t half = W << 31;
  uint32_t jstar = J;
  for (uint32_t j = 1; j < J; ++j)
    if (score[j] > half) {
      jstar = j;
      break;
    }
  // adapted score: the running maximum from jstar on; increases between
  // consecutive power-of-two strides
  uint64_t run = 0, prev = 0;
  int64_t best = 0;
  uint32_t best_line = 0, ncand = 0, prev_stride = 0;
  for (uint32_t j = 0; j < J; ++j) {
    uint64_t sc = score[j];
    if (j >= jstar) {
      run = max(run, sc);
      sc = run;
    }
    const uint32_t st = strides[j];
    if (st == 0 || (st & (st - 1)) != 0) continue;
    if (ncand > 0) {
      const int64_t inc = (int64_t)sc - (int64_t)prev;
      if (ncand == 1 || inc > best) {
        best = inc;
        best_line = prev_stride;
      }
    }
    prev = sc;
    prev_stride = st;
    ++ncand;
  }
  uint32_t flags = jstar < J ? 0u : KS_LINE_NO_MAX_LIKE;
  if (ncand < 2) return ks_line{0u, jstar, flags | KS_LINE_INCONCLUSIVE, 0u, 0.0};
  if (best <= 0) flags |= KS_LINE_NO_INCREASE;
  return ks_line{best_line, jstar, flags, 0u, (double)best / (double)(W << 32)};
}

// E experiments to a workgroup of four waves. E = 1: the waves share the strides
// (a wave taking 16 strides in turn, a 64-bit division each, took 16 us on 256
// experiments). E = 4, for thousands of experiments: a wave each, with nothing
// read or started four times (60000 of 2 x 64 43 us, 69 with E = 1).
template <uint32_t E>
__global__ __launch_bounds__(256) void line_kernel(const ks_desc* __restrict__ desc, uint32_t num_exp,
                                                   const ks_row_stats* __restrict__ stats, uint64_t stats_rows,
                                                   uint32_t J, const uint32_t* __restrict__ strides,
                                                   ks_line* __restrict__ out) {
  __shared__ uint64_t scores[E][kLineMaxJ];
  const uint32_t lane = ks::lane_id(), w = ks::wave_id();
  const uint32_t e = E == 1 ? blockIdx.x : blockIdx.x * E + w;
  const bool first = E == 1 ? threadIdx.x == 0 : lane == 0;
  uint64_t* score = scores[E == 1 ? 0 : w];
  if (e >= num_exp) return;
  const ks_desc d = desc[e];
  const uint32_t K = d.K, A = K / J;
  const bool bad = A < 1 || A > kLineMaxA || A * J != K || d.aux_offset > stats_rows ||
                   (uint64_t)K > stats_rows - d.aux_offset;
  if (bad) {
    if (first) out[e] = ks_line{0u, 0u, KS_LINE_INVALID, 0u, 0.0};
    return;
  }
  line_scores(stats + d.aux_offset, A, J, E == 1 ? w : 0u, E == 1 ? 4u : 1u, lane, score);
  if constexpr (E == 1) ks::block_publish();
  else ks::wave_lds_sync();
  if (first) out[e] = line_record(score, A, J, strides);
}

}  // namespace

extern "C" int ks_check_batch(ks_ctx* ctx, const ks_desc* desc, uint32_t num_series, uint32_t max_K,
                              const ks_result* res, const ks_row_stats* stats, uint64_t stats_rows, uint32_t edge,
                              uint32_t k, ks_check* out, void* stream) {
  if (!ctx) return KS_E_INVALID;
  if (max_K == 0) max_K = KS_MAX_K;
  if (max_K < 2 || max_K > KS_MAX_K) return KS_E_RANGE;
  if (edge < 1 || k < 1) return KS_E_INVALID;
  if (num_series == 0) return KS_OK;
  if (!desc || !res || !stats || !out) return KS_E_INVALID;
  DeviceGuard g(ctx->device);
  if (g.err != hipSuccess) return hip_fail(g.err, "hipSetDevice");
  auto run = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(num_series), dim3(64), 0, (hipStream_t)stream, desc, num_series, max_K, res, stats,
                       stats_rows, edge, k, out);
  };
  if (max_K <= 256) run(check_kernel<4>);
  else if (max_K <= 512) run(check_kernel<8>);
  else if (max_K <= 1024) run(check_kernel<16>);
  else run(check_kernel<32>);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? KS_OK : hip_fail(e, "check launch");
}

extern "C" int ks_align_batch(const uint64_t* measured, const uint64_t* total, uint32_t n, uint32_t* segments,
                              double* aligned, double* distance, void* stream) {
  if (n == 0) return KS_OK;
  if (!measured || !total || !segments || !aligned || !distance) return KS_E_INVALID;
  hipLaunchKernelGGL(align_kernel, dim3((n + 255) / 256), dim3(256), 0, (hipStream_t)stream, measured, total, n,
                     segments, aligned, distance);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? KS_OK : hip_fail(e, "align launch");
}

extern "C" int ks_line_batch(ks_ctx* ctx, const ks_desc* desc, uint32_t num_exp, const ks_row_stats* stats,
                             uint64_t stats_rows, uint32_t J, const uint32_t* strides, ks_line* out, void* stream) {
  if (!ctx) return KS_E_INVALID;
  if (J < 2 || J > kLineMaxJ) return KS_E_RANGE;
  if (num_exp == 0) return KS_OK;
  if (!desc || !stats || !strides || !out) return KS_E_INVALID;
  DeviceGuard g(ctx->device);
  if (g.err != hipSuccess) return hip_fail(g.err, "hipSetDevice");
  // a wave per experiment: of two or three strides from 1024 experiments on (2000 of
  // 2 x 256 9 us against 13, 20000 of 2 x 64 18 against 26; 6000 of 8 x 32 17.4 against
  // 16.5), of up to 16 from 32768 (60000 of 8 x 32 117 against 136, of 16 x 32 220
  // against 238; of 64 x 16 829 against 804), and where a grid of 2^32 - 1 threads
  // does not hold a workgroup each
  const bool many = num_exp > (J < 4 ? 1024u : J <= 16 ? 32768u : (1u << 24) - 1u);
  auto run = [&](auto kernel, uint32_t grid) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(256), 0, (hipStream_t)stream, desc, num_exp, stats, stats_rows, J,
                       strides, out);
  };
  if (many) run(line_kernel<4>, (num_exp + 3) / 4);
  else run(line_kernel<1>, num_exp);
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? KS_OK : hip_fail(e, "line launch");
}
