// Per-row latency statistics (ks_stats_batch): the average as the main result,
// with p50, p95, standard deviation, minimum and maximum beside it, for every
// row of every series in one read of the samples: the row pass of the learned
// path's deciles with two other ranks.
#include <hip/hip_runtime.h>

#include <cmath>

#include "ks.h"
#include "ks_ctx.hpp"
#include "ks_plan.hpp"
#include "ks_scan.hpp"
#include "ks_select.hpp"

static_assert(sizeof(ks_desc) == 24 && sizeof(ks_result) == 48 && sizeof(ks_params) == 32 &&
                  sizeof(ks_row_stats) == 32,
              "ABI struct sizes");

using namespace ks_host;

namespace {

// p50 and p95: x_(floor(q (N - 1))) for q = 0.5, 0.95.
struct StatRanks {
  static constexpr uint32_t kCount = 2;
  __device__ static uint32_t rank(uint32_t j, uint32_t N) {
    return j == 0 ? (N - 1) / 2u : (uint32_t)((95ull * (N - 1)) / 100u);
  }
};

typedef unsigned __int128 u128;

// u128 -> double, rounded to nearest even once: the top 64 significant bits
// with a sticky bit for everything below, converted, then scaled exactly.
__device__ double u128_to_double(u128 v) {
  const uint64_t hi = (uint64_t)(v >> 64);
  if (hi == 0) return (double)(uint64_t)v;
  const int sh = 64 - __clzll(hi);  // bits above the low 64
  const uint64_t top = (uint64_t)(v >> sh);
  const bool sticky = (v & (((u128)1 << sh) - 1)) != 0;
  return ldexp((double)(top | (uint64_t)sticky), sh);
}

// a row's exact results, staged until S rows are done; the records (mean, std
// in FP64) are then made by S lanes at once. 64 rows for rows of two or more
// load batches (fewer, longer write bursts among the reads), 16 otherwise.
template <uint32_t S>
struct RowStage {
  uint64_t s1[S], s2[S];
  uint32_t s2h[S], rmin[S], rmax[S], p50[S], p95[S];
};
constexpr uint32_t stats_stage_rows(int NB) { return NB == 1 || NB == (int)ks::kGrouped ? 16u : 64u; }

// The calling wave's rows `sp` of one series of row class NB; every kStage
// rows' records are written as contiguous 16-byte stores (records written one
// at a time, by waves interleaved row by row, left partly written cache lines
// behind).
template <int NB, int W>
__device__ __forceinline__ void stats_rows(ks::RowLds* sel, ks::CoopLds<W>& co, void* stage,
                                           const uint32_t* __restrict__ samples, const ks_desc& d, uint32_t c,
                                           uint32_t C, uint32_t num_series, uint32_t w, uint32_t lane,
                                           ks_row_stats* __restrict__ o) {
  constexpr uint32_t kStage = stats_stage_rows(NB);
  static_assert(kStage <= (uint32_t)ks::kWave, "a flush makes one record per lane");
  const uint32_t N = d.N;
  const ks::RowSpan sp = ks::row_span<NB, W>(d.K, d.N, c, C, num_series, w);
  RowStage<kStage>& st = reinterpret_cast<RowStage<kStage>*>(stage)[w];
  // row i's results; its p50 and p95 on lanes first and first + 1
  ks::select_rows<NB, StatRanks, W>(sel, co, samples, d.offset, N, sp, w, lane,
                                    [&](uint32_t i, const ks::RowOut& r, uint32_t first) {
    const uint32_t p50 = (uint32_t)__builtin_amdgcn_readlane((int)r.sel, (int)first);
    const uint32_t p95 = (uint32_t)__builtin_amdgcn_readlane((int)r.sel, (int)first + 1);
    const uint32_t j = (i - sp.begin) % kStage;
    if (lane == 0) {
      st.s1[j] = r.s1;
      st.s2[j] = r.s2;
      st.s2h[j] = r.s2h;
      st.rmin[j] = r.rmin;
      st.rmax[j] = r.rmax;
      st.p50[j] = p50;
      st.p95[j] = p95;
    }
    if (j + 1 == kStage || i + 1 == sp.end) {  // rows i - j .. i: lane q makes row i - j + q's record
      ks::wave_lds_sync();
      if (lane <= j) {
        const uint64_t a1 = st.s1[lane];
        const u128 S2 = ((u128)st.s2h[lane] << 64) | st.s2[lane];
        const u128 num = (u128)N * S2 - (u128)a1 * a1;  // >= 0 (Cauchy-Schwarz), < 2^113
        const double nn = (double)N * (double)N;
        const ks_row_stats rec{(double)a1 / (double)N, sqrt(u128_to_double(num) / nn), st.rmin[lane], st.p50[lane],
                               st.p95[lane], st.rmax[lane]};
        static_assert(sizeof(ks_row_stats) == 32, "a record is two 16-byte stores");
        ks::u32x4 v0, v1;
        __builtin_memcpy(&v0, &rec, 16);
        __builtin_memcpy(&v1, reinterpret_cast<const char*>(&rec) + 16, 16);
        ks::u32x4* dst = reinterpret_cast<ks::u32x4*>(o + (i - j) + lane);
        ks::row_out_store<NB>(v0, dst);
        ks::row_out_store<NB>(v1, dst + 1);
      }
      ks::wave_lds_sync();
    }
  });
}

// One launch over the row classes of MASK, one workgroup per (series, chunk of
// its rows). With a plan the series come in its order (each class largest
// first), without one in descriptor order. Malformed series are class 1's.
template <uint32_t MASK>
__global__ __launch_bounds__(ks::row_pass_threads(MASK)) __attribute__((amdgpu_waves_per_eu(ks::row_pass_waves(MASK)))) void row_stats_kernel(
    const uint32_t* __restrict__ samples, uint64_t num_samples, const ks_desc* __restrict__ desc, uint32_t num_series,
    uint32_t max_K, ks_row_stats* __restrict__ out, uint64_t out_rows, const uint32_t* __restrict__ plan, uint32_t C) {
  constexpr int NT = ks::row_pass_threads(MASK), W = NT / ks::kWave;
  constexpr uint32_t kStageMax = MASK == ks::kRowsOne ? 16u : 64u;
  __shared__ ks::RowLds sel[W];
  __shared__ RowStage<kStageMax> stage[W];
  __shared__ ks::CoopLds<W> co;
  const uint32_t t = blockIdx.x / C, c = blockIdx.x - t * C;
  const uint32_t s = ks::row_pass_series<MASK>(plan, num_series, t);
  if (s >= num_series) return;
  const ks_desc d = desc[s];
  const uint32_t lane = ks::lane_id(), w = ks::wave_id();
  const bool bad = ks::check_desc(d, num_samples, max_K) || d.N > KS_FEATURE_MAX_N;
  const uint32_t nb = bad ? 1u : ks::feat_batches(d.N);
  if (!((MASK >> ks::feat_class_index(nb)) & 1u)) return;
  const bool fits = d.aux_offset <= out_rows && (uint64_t)d.K <= out_rows - d.aux_offset;
  if (!fits) return;
  ks_row_stats* o = out + d.aux_offset;
  if (bad) {
    for (uint64_t i = (uint64_t)c * NT + threadIdx.x; i < d.K; i += (uint64_t)C * NT)
      o[i] = ks_row_stats{NAN, NAN, 0u, 0u, 0u, 0u};
    return;
  }
  auto rows = [&](auto tag) {
    constexpr int NB = decltype(tag)::value;
    if constexpr ((MASK >> ks::feat_class_index(NB)) & 1u)
      if (nb == (uint32_t)NB) stats_rows<NB, W>(sel, co, stage, samples, d, c, C, num_series, w, lane, o);
  };
  rows(std::integral_constant<int, 1>{});
  rows(std::integral_constant<int, 2>{});
  rows(std::integral_constant<int, (int)ks::kStreamed>{});
  rows(std::integral_constant<int, (int)ks::kGrouped>{});
}

}  // namespace

extern "C" int ks_stats_batch(ks_ctx* ctx, const uint32_t* samples, uint64_t num_samples, const ks_desc* desc,
                              uint32_t num_series, uint32_t max_K, ks_row_stats* out, uint64_t out_rows, void* stream) {
  if (!ctx) return KS_E_INVALID;
  if (max_K == 0) max_K = KS_MAX_K;
  if (max_K < 2 || max_K > KS_MAX_K) return KS_E_RANGE;
  if (num_series == 0) return KS_OK;
  if (!samples || !desc || !out) return KS_E_INVALID;
  DeviceGuard g(ctx->device);
  if (g.err != hipSuccess) return hip_fail(g.err, "hipSetDevice");
  hipStream_t st = (hipStream_t)stream;
  auto launch = [&](auto kernel, uint32_t mask, const uint32_t* plan) {
    const uint32_t C = ks::row_pass_chunks((uint32_t)ctx->num_cus, num_series, max_K, num_samples, mask);
    hipLaunchKernelGGL(kernel, dim3(num_series * C), dim3(ks::row_pass_threads(mask)), 0, st, samples, num_samples, desc,
                       num_series, max_K, out, out_rows, plan, C);
  };
  if (num_series <= ks::kRowPassOneLaunch) {
    launch(row_stats_kernel<ks::kRowsAll>, ks::kRowsAll, nullptr);
  } else {
    // the series order per row class (the feature pass's plan), kept in the
    // context's scan workspace (its queue items: 512 bytes per series)
    if (int rc = ensure_workspace(ctx, num_series, 0)) return rc;
    uint32_t* plan = reinterpret_cast<uint32_t*>(ctx->items);
    hipLaunchKernelGGL(ks::feature_plan_kernel, dim3(1), dim3(ks::kFeatPlanNT), 0, st, desc, num_series, num_samples,
                       max_K, plan);
    launch(row_stats_kernel<ks::kRowsOne>, ks::kRowsOne, plan);
    launch(row_stats_kernel<ks::kRowsMid>, ks::kRowsMid, plan);
  }
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? KS_OK : hip_fail(e, "row stats launch");
}
