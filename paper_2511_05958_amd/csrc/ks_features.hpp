// Learned-proposal stage 1: one read of every sample gives, per row,
//   - the moments (sum r, sum r^2) that the exact refine turns into eq. 2 keys,
//   - the nine deciles x_(floor(k (N-1) / 10)), k = 1..9, by the wave-level
//     select of ks_select.hpp (a 1024-bin window of the keys above the row's
//     minimum or a base just below it, radix levels only past the window),
// and per series the minimum m, then features f = (double)(x - m) / max(m, 1)
// rounded to float (project-defined inputs of the network).
#pragma once

#include "ks_cnn.hpp"
#include "ks_scan.hpp"
#include "ks_plan.hpp"
#include "ks_select.hpp"

namespace ks {

// Per-row moments of the learned path (the refine's input), per-series min.
struct LearnWs {
  uint64_t* s1;     // [num_series * SR] (row slot of series s: s * SR + 2 + i)
  uint64_t* s2lo;
  uint32_t* s2hi;
  uint32_t* smin;   // [num_series]: written by the pack step
  uint32_t* cmin;   // [num_series * Cs]: minima of the feature pass's row chunks
  uint32_t* K;      // [num_series]: K when the series was valid, 0 otherwise
};

// Per-wave staging of a wave's per-row outputs: a wave takes a contiguous
// block of rows and writes every kFeatStage rows' deciles and moments as
// contiguous stores (rows written one at a time, by waves interleaved row by
// row, left partly written cache lines behind; they cost 5 - 15% of the
// pass and made its time depend on where the buffers lay in memory). Rows of
// two or more load batches stage 64 rows (fewer, longer write bursts among
// the reads: the learned step on 8192 x 1024 x 2048 ran 1 - 4% faster than
// with 16), one-batch and short rows 16; a kernel's LDS is for the largest of
// its classes.
// (at most 64: a flush writes one row's moments per lane)
__host__ __device__ constexpr uint32_t feat_stage_rows(int NB) { return NB == 1 || NB == (int)kGrouped ? 16u : 64u; }

template <uint32_t S>
struct FeatStage {
  uint32_t dec[S * 9];
  uint64_t s1[S], s2lo[S];
  uint32_t s2hi[S];
};

// The calling wave's rows `sp` of one series of row class NB. Writes per row
// the deciles (as raw samples, at row slot s * SR + 2 + i of feat_ws) and the
// refine workspace's moments; returns the least of its rows' minima.
template <int NB, int W>
__device__ __forceinline__ uint32_t feature_rows(RowLds* sel, CoopLds<W>& co, void* stage,
                                                 const uint32_t* __restrict__ samples, const ks_desc& d, uint32_t c,
                                                 uint32_t C, uint32_t num_series, uint32_t w, uint32_t lane, uint64_t slot,
                                                 LearnWs lw,
                                                 float* __restrict__ feat_ws) {
  constexpr uint32_t kFeatStage = feat_stage_rows(NB);
  static_assert(kFeatStage <= (uint32_t)kWave, "a flush writes one row's moments per lane");
  const RowSpan sp = row_span<NB, W>(d.K, d.N, c, C, num_series, w);
  FeatStage<kFeatStage>& st = reinterpret_cast<FeatStage<kFeatStage>*>(stage)[w];
  uint32_t gmin = 0xffffffffu;
  // row i's results; its deciles on lanes first .. first + 8
  select_rows<NB, DecileRanks, W>(sel, co, samples, d.offset, d.N, sp, w, lane,
                                  [&](uint32_t i, const RowOut& o, uint32_t first) {
    const uint32_t j = (i - sp.begin) % kFeatStage;
    if (lane == 0) {
      st.s1[j] = o.s1;
      st.s2lo[j] = o.s2;
      st.s2hi[j] = o.s2h;
    }
    gmin = min(gmin, o.rmin);
    // feature numerators x - m need the series minimum: keep x itself
    if (lane - first < 9u) st.dec[j * 9 + lane - first] = o.sel;
    if (j + 1 == kFeatStage || i + 1 == sp.end) {  // flush rows i - j .. i
      wave_lds_sync();
      const uint64_t r0 = slot + i - j;
      for (uint32_t q = lane; q < (j + 1) * 9; q += kWave)
        row_out_store<NB>(__uint_as_float(st.dec[q]), &feat_ws[r0 * 9 + q]);
      if (lane <= j) {
        row_out_store<NB>(st.s1[lane], &lw.s1[r0 + lane]);
        row_out_store<NB>(st.s2lo[lane], &lw.s2lo[r0 + lane]);
        row_out_store<NB>(st.s2hi[lane], &lw.s2hi[r0 + lane]);
      }
      wave_lds_sync();
    }
  });
  return gmin;
}

// First step: one launch over the row classes of MASK, one workgroup per
// (series, chunk of its rows; row_pass_chunks, at most Cs), the series in the
// plan's order (descriptor order without one). Malformed series (class 1's) are marked with
// K = 0. Each chunk leaves its minimum in cmin; chunk 0 writes the series' K.
template <uint32_t MASK>
__global__ __launch_bounds__(row_pass_threads(MASK)) __attribute__((amdgpu_waves_per_eu(row_pass_waves(MASK)))) void features_kernel(
    const uint32_t* __restrict__ samples, uint64_t num_samples, const ks_desc* __restrict__ desc, uint32_t num_series,
    uint32_t max_K, uint32_t SR, LearnWs lw, float* __restrict__ feat_ws, const uint32_t* __restrict__ plan,
    uint32_t C, uint32_t Cs) {
  constexpr int W = row_pass_threads(MASK) / kWave;
  constexpr uint32_t kStageMax = MASK == kRowsOne ? 16u : 64u;
  __shared__ RowLds sel[W];
  __shared__ FeatStage<kStageMax> stage[W];
  __shared__ CoopLds<W> co;
  __shared__ uint32_t red[W];
  const uint32_t t = blockIdx.x / C, c = blockIdx.x - t * C;
  const uint32_t s = row_pass_series<MASK>(plan, num_series, t);
  if (s >= num_series) return;
  const ks_desc d = desc[s];
  const uint32_t tid = threadIdx.x, lane = lane_id(), w = wave_id();
  const bool bad = check_desc(d, num_samples, max_K) || d.N > KS_FEATURE_MAX_N;
  const uint32_t nb = bad ? 1u : feat_batches(d.N);
  if (!((MASK >> feat_class_index(nb)) & 1u)) return;
  if (bad) {  // no rows to pack
    if (tid == 0 && c == 0) lw.K[s] = 0;
    return;
  }
  uint32_t gmin = 0xffffffffu;
  auto rows = [&](auto tag) {
    constexpr int NB = decltype(tag)::value;
    if constexpr ((MASK >> feat_class_index(NB)) & 1u)
      if (nb == (uint32_t)NB)
        gmin = feature_rows<NB, W>(sel, co, stage, samples, d, c, C, num_series, w, lane, (uint64_t)s * SR + 2, lw,
                                   feat_ws);
  };
  rows(std::integral_constant<int, 1>{});
  rows(std::integral_constant<int, 2>{});
  rows(std::integral_constant<int, (int)kStreamed>{});
  rows(std::integral_constant<int, (int)kGrouped>{});
  if (lane == 0) red[w] = gmin;
  __syncthreads();
  if (tid == 0) {
#pragma unroll
    for (int u = 0; u < W; ++u) gmin = min(gmin, red[u]);
    lw.cmin[(uint64_t)s * Cs + c] = gmin;  // 0xffffffff for a chunk past the series' rows
    if (c == 0) {
      for (uint32_t q = C; q < Cs; ++q) lw.cmin[(uint64_t)s * Cs + q] = 0xffffffffu;
      lw.K[s] = d.K;
    }
  }
}

// Second step, one workgroup per (series, chunk of NT slot rows): the deciles
// x of the series' rows become the features f = (double)(x - m) / max(m, 1)
// rounded to float (m the series minimum), in place and into the caller's
// buffer, element by element (consecutive threads, consecutive elements);
// then the chunk's network input rows (bf16 of the nine features and the two
// position channels, channels 11..15 zero), staged in LDS, are written as
// 16-byte stores. Only the series' own rows: the network masks what lies outside.
template <int NT>
__global__ __launch_bounds__(NT) void feature_pack_kernel(const ks_desc* __restrict__ desc, uint32_t num_series,
                                                          float* __restrict__ feat_out, uint64_t feat_rows,
                                                          uint16_t* __restrict__ x0, uint32_t SR, LearnWs lw,
                                                          float* __restrict__ feat_ws, uint32_t Cs) {
  static_assert(kRowPassChunks <= (uint32_t)NT, "one thread per chunk minimum");
  __shared__ __align__(16) uint16_t bf[NT * 16];
  __shared__ uint32_t red[NT / kWave];
  const uint32_t s = blockIdx.x;
  if (s >= num_series) return;
  const uint32_t tid = threadIdx.x;
  const uint32_t r0 = blockIdx.y * NT;
  if (r0 >= SR) return;
  const uint32_t nr = SR - r0 < (uint32_t)NT ? SR - r0 : (uint32_t)NT;
  const uint32_t K = lw.K[s];
  const uint64_t row0 = (uint64_t)s * SR + r0;
  // rows [lo, hi) of the chunk hold data
  const uint32_t lo = r0 < 2u ? 2u - r0 : 0u;
  const uint32_t hi = K + 2u > r0 ? (K + 2u - r0 < nr ? K + 2u - r0 : nr) : 0u;
  if (lo >= hi) return;
  const uint32_t gmin = block_min_u32<NT>(tid < Cs ? lw.cmin[(uint64_t)s * Cs + tid] : 0xffffffffu, red);
  if (blockIdx.y == 0 && tid == 0) lw.smin[s] = gmin;
  const double denom = (double)(gmin > 1 ? gmin : 1u);
  const ks_desc d = desc[s];
  const bool to_user = feat_out && d.aux_offset <= feat_rows && K <= feat_rows - d.aux_offset;
  for (uint32_t q = lo * 9u + tid; q < hi * 9u; q += NT) {
    const uint32_t rr = q / 9u, k = q - rr * 9u;
    const uint64_t e = row0 * 9u + q;
    const uint32_t x = __float_as_uint(feat_ws[e]);
    const float f = (float)((double)(x - gmin) / denom);
    feat_ws[e] = f;
    if (to_user) feat_out[(d.aux_offset + r0 + rr - 2) * 9 + k] = f;
    bf[rr * 16 + k] = cnn::f2bf(f);
  }
  __syncthreads();
  for (uint32_t q = lo * 2u + tid; q < hi * 2u; q += NT) {
    const uint32_t rr = q >> 1, h = q & 1u, t = r0 + rr - 2;
    u32x4 v;
    if (h == 0) {
      v = *reinterpret_cast<const u32x4*>(&bf[rr * 16]);
    } else {
      const uint32_t b8 = bf[rr * 16 + 8];
      const uint32_t p9 = cnn::f2bf(cnn::pos_frac(t, K)), p10 = cnn::f2bf(cnn::pos_centre(t, K));
      v = u32x4{b8 | (p9 << 16), p10, 0u, 0u};
    }
    *reinterpret_cast<u32x4*>(x0 + (row0 + rr) * 16 + h * 8) = v;
  }
}

}  // namespace ks
