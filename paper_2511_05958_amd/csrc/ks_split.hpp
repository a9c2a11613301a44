// Exact scan of batches too small to fill the device with one workgroup per
// series (KS_LAUNCH_ORDERED with few series). One workgroup streams a series
// with a few waves, sorts its keys in a chain of radix passes and walks all
// candidates alone: 6 series of 1024 rows of 2048 samples took 547 us on six of
// 256 CUs (33 us spread as below, 50 MB at 1.5 TB/s; launch gaps and the two
// short kernels bound it). Here a series is spread over the device:
//
//   split_moments_kernel  a workgroup per chunk of rows: the moments and the
//                         minimum of every row, to the workspace;
//   split_rank_kernel     a workgroup per 64 rows: every workgroup makes all K
//                         keys, each of its rows' ranks is a count of smaller
//                         keys (K^2 compares, spread over K / 64 workgroups, in
//                         place of a chain of radix passes in one), and the
//                         keys are written in order;
//   split_walk_kernel     a workgroup per 64 candidates, its waves sharing the
//                         sorted positions; the last one of a series to finish
//                         makes the choice.
//
// tiny_scan_kernel does all of it in one launch, with one workgroup of 16 waves
// per series, for series that such a workgroup reads in a few microseconds (one
// sweep of 64 x 256: 8 us a call; the plan and the four-wave scan took 27).
//
// Keys: Q (at most 96 bits) and the row index make one 107-bit number, kept as
// lo = (Q << 11) | row and hi = Q >> 53; all are distinct, so ranks are a
// permutation and equal Q come in row order, as in the stable radix sort. hi is
// 0 for every row of most series (Q < 2^53), and then only lo is compared.
#pragma once

#include "ks_scan.hpp"

namespace ks {

constexpr uint32_t kSplitWGs = 8;  // workgroups per CU stream the rows
constexpr uint32_t kSplitNT = 256;
constexpr uint32_t kSplitWalkNT = 512;
constexpr uint32_t kSplitSlots = KS_MAX_K / kWave;  // 64-candidate slots of a series
constexpr int kTinyNT = 1024;
static_assert(KS_MAX_K == 1u << 11, "a row index takes 11 bits of a key");

struct SortKey {
  uint64_t lo, hi;
};

struct SplitWs {
  RowMom* mom;       // series s, row i at s * max_K + i
  SortKey* sorted;   // the same layout, in key order
  uint32_t* best;    // series s, slot j: U and c at (s * kSplitSlots + j) * 2
  uint32_t* ticket;  // per series: finished slots (nullptr: no walk follows the moments)
};

// Series and slot (or chunk) of the calling workgroup. Workgroups go to the eight
// XCDs in turn, and there to the four shader engines: series after series, with 32
// slots each, every series' first slots met on one engine of one XCD, and where K
// is far below max_K only those have work (under max_K 0 256 series of 64 x 64 took
// 44 us a call, of 512 x 4 167; 20 and 100 now). So where C, the slots of a series,
// has a power of two g in common with these 32 places, the slots of each g are
// exchanged by the series. With more than 32 series per XCD, whose sizes even out,
// the rank and the walk go slot after slot instead, all slots of a series on one
// XCD, whose L2 keeps its keys (384 series of 1024 x 64: 302 us exchanged, 249 so;
// 160 uneven ones up to 2048 x 4096: 283 exchanged, 352 so).
constexpr uint32_t kXcds = 8, kPlacesLog = 5, kTurnedSeries = 32 * kXcds;
struct SplitAt {
  uint32_t s, slot;
};
__device__ __forceinline__ SplitAt turned_at(uint32_t C) {
  const uint32_t l = min((uint32_t)__builtin_ctz(C), kPlacesLog);  // g = 1 << l
  return SplitAt{blockIdx.y, blockIdx.x ^ ((blockIdx.y >> (kPlacesLog - l)) & ((1u << l) - 1u))};
}
__device__ __forceinline__ SplitAt split_at(uint32_t num_series, uint32_t rows) {
  return num_series > kTurnedSeries ? SplitAt{blockIdx.x, blockIdx.y} : turned_at((rows + kWave - 1) / kWave);
}
inline dim3 split_grid(uint32_t num_series, uint32_t rows) {
  const uint32_t slots = (rows + kWave - 1) / kWave;
  return num_series > kTurnedSeries ? dim3((num_series + kXcds - 1) / kXcds * kXcds, slots) : dim3(slots, num_series);
}

__device__ __forceinline__ SortKey sort_key(uint64_t s1, uint64_t s2lo, uint32_t s2hi, uint32_t i, uint32_t N,
                                            uint32_t gmin) {
  const u128 s2 = ((u128)s2hi << 64) | s2lo;
  const u128 q = s2 + (u128)((uint64_t)gmin * gmin) * N - (u128)s1 * (2ull * gmin);
  return SortKey{((uint64_t)q << 11) | i, (uint64_t)(q >> 53)};
}

// Number of keys [j0, j1) below (lo, hi); `wide`: some key's hi is not 0.
__device__ __forceinline__ uint32_t count_below(const uint64_t* __restrict__ lo, const uint64_t* __restrict__ hi,
                                                uint32_t j0, uint32_t j1, uint64_t mylo, uint64_t myhi, bool wide) {
  uint32_t n = 0;
  if (!wide) {
#pragma unroll 8
    for (uint32_t j = j0; j < j1; ++j) n += lo[j] < mylo ? 1u : 0u;
  } else {
    for (uint32_t j = j0; j < j1; ++j) n += (hi[j] < myhi || (hi[j] == myhi && lo[j] < mylo)) ? 1u : 0u;
  }
  return n;
}

// Any thread's v nonzero (all threads get the answer).
template <int NT>
__device__ __forceinline__ bool block_any(bool v, uint32_t* red) {
  const uint64_t b = ballot(v);
  if (lane_id() == 0) red[wave_id()] = b != 0 ? 1u : 0u;
  __syncthreads();
  uint32_t any = 0;
#pragma unroll
  for (int k = 0; k < NT / kWave; ++k) any |= red[k];
  __syncthreads();
  return any != 0;
}

namespace {  // kernels are compiled into each translation unit that launches them

__global__ __launch_bounds__(kSplitNT) void split_moments_kernel(const uint32_t* __restrict__ samples,
                                                                 uint64_t num_samples, const ks_desc* __restrict__ desc,
                                                                 uint32_t max_K, ks_result* __restrict__ out,
                                                                 SplitWs ws) {
  constexpr uint32_t W = kSplitNT / kWave;
  __shared__ uint64_t p1[W], p2[W];
  __shared__ uint32_t p2h[W], pm[W];
  const uint32_t C = gridDim.x;
  const SplitAt at = turned_at(C);
  const uint32_t s = at.s, c = at.slot;
  const ks_desc d = desc[s];
  const uint32_t bad = check_desc(d, num_samples, max_K);
  if (bad) {
    if (out && c == 0 && threadIdx.x == 0) write_result(out + s, 0, 0, 0, 0, 0.0, 0.0, 1.0, bad);
    return;
  }
  if (ws.ticket && c == 0 && threadIdx.x == 0) ws.ticket[s] = 0;
  const uint32_t K = d.K, N = d.N, lane = lane_id(), w = wave_id();
  uint32_t R = (K + C - 1) / C;
  // fewer rows than waves and more than a batch of samples per wave: all waves on each row
  const bool coop = R < W && N > W * 16u * kWave;
  if (!coop) {  // whole steps of the waves (short rows go 4 or 2 to a wave)
    const uint32_t step = W * (N <= 256u ? 4u : (N <= 512u ? 2u : 1u));
    R = (R + step - 1) / step * step;
  }
  if ((uint64_t)c * R >= K) return;
  const uint32_t r0 = c * R, r1 = min(K, r0 + R);
  RowMom* mom = ws.mom + (uint64_t)s * max_K;
  if (!coop) {
    stream_rows<true>(samples, d.offset, N, r0 + w, r1, W, lane,
                      [&](uint32_t i, uint64_t s1, uint64_t s2, uint32_t s2h, uint32_t rmin) {
                        if (lane == 0) mom[i] = RowMom{s1, s2, s2h, rmin};
                      });
    return;
  }
  for (uint32_t i = r0; i < r1; ++i) {
    const RowGeo g = row_geo(samples, d.offset + (uint64_t)i * N, N);
    uint64_t s1 = 0, s2 = 0;
    uint32_t s2h = 0, mn = 0xffffffffu;
    Batch A, B;
    uint32_t u = w;  // batches w, w + W, ...
    if (u < g.nb) load_batch(A, samples, g, u, lane);
    while (u < g.nb) {
      if (u + W < g.nb) load_batch(B, samples, g, u + W, lane);
      acc_batch(A, mn, s1, s2, s2h);
      u += W;
      if (u >= g.nb) break;
      if (u + W < g.nb) load_batch(A, samples, g, u + W, lane);
      acc_batch(B, mn, s1, s2, s2h);
      u += W;
    }
    wave_total_64_96(s1, s2, s2h);
    mn = wave_min_u32(mn);
    __syncthreads();  // the previous row's parts have been read
    if (lane == 0) {
      p1[w] = s1;
      p2[w] = s2;
      p2h[w] = s2h;
      pm[w] = mn;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
      uint64_t t1 = 0;
      u128 t2 = 0;
      uint32_t tm = 0xffffffffu;
      for (uint32_t v = 0; v < W; ++v) {
        t1 += p1[v];
        t2 += ((u128)p2h[v] << 64) | p2[v];
        tm = min(tm, pm[v]);
      }
      mom[i] = RowMom{t1, (uint64_t)t2, (uint32_t)(t2 >> 64), tm};
    }
  }
}

// out: where series of a bad shape or range are flagged (nullable).
inline void launch_split_moments(uint32_t num_cus, const uint32_t* samples, uint64_t num_samples, const ks_desc* desc,
                                 uint32_t num_series, uint32_t max_K, ks_result* out, const SplitWs& ws,
                                 hipStream_t st) {
  const uint32_t chunks = (kSplitWGs * num_cus + num_series - 1) / num_series;
  hipLaunchKernelGGL(split_moments_kernel, dim3(chunks < max_K ? chunks : max_K, num_series), dim3(kSplitNT), 0, st,
                     samples, num_samples, desc, max_K, out, ws);
}

__global__ __launch_bounds__(kSplitNT) void split_rank_kernel(uint64_t num_samples, const ks_desc* __restrict__ desc,
                                                              uint32_t num_series, uint32_t max_K, SplitWs ws) {
  constexpr uint32_t W = kSplitNT / kWave;
  __shared__ uint64_t lo[KS_MAX_K], hi[KS_MAX_K];
  __shared__ uint32_t part[W * kWave], red[W];
  const SplitAt at = split_at(num_series, max_K);
  const uint32_t s = at.s, r0 = at.slot * kWave;
  if (s >= num_series) return;
  const ks_desc d = desc[s];
  if (check_desc(d, num_samples, max_K) || r0 >= d.K) return;
  const uint32_t K = d.K, N = d.N, tid = threadIdx.x, lane = lane_id(), w = wave_id();
  const RowMom* mom = ws.mom + (uint64_t)s * max_K;
  uint32_t mn = 0xffffffffu;
  for (uint32_t i = tid; i < K; i += kSplitNT) mn = min(mn, mom[i].pad);
  const uint32_t gmin = block_min_u32<kSplitNT>(mn, red);
  bool w53 = false;
  for (uint32_t i = tid; i < K; i += kSplitNT) {
    const RowMom r = mom[i];
    const SortKey k = sort_key(r.s1, r.s2lo, r.s2hi, i, N, gmin);
    lo[i] = k.lo;
    hi[i] = k.hi;
    w53 |= k.hi != 0;
  }
  const bool wide = block_any<kSplitNT>(w53, red);  // its barriers publish the keys
  const uint32_t row = r0 + lane;
  const uint32_t own = min(row, K - 1);
  const uint32_t len = (K + W - 1) / W;
  const uint32_t j0 = min(K, w * len), j1 = min(K, j0 + len);
  part[w * kWave + lane] = count_below(lo, hi, j0, j1, lo[own], hi[own], wide);
  __syncthreads();
  if (w == 0 && row < K) {
    uint32_t rank = 0;
#pragma unroll
    for (uint32_t v = 0; v < W; ++v) rank += part[v * kWave + lane];
    ws.sorted[(uint64_t)s * max_K + rank] = SortKey{lo[row], hi[row]};
  }
}

// Sorted position p ends a group of equal Q: the next key's Q differs.
__device__ __forceinline__ bool group_end(const SortKey& a, const SortKey& b) {
  return (a.lo >> 11) != (b.lo >> 11) || a.hi != b.hi;
}

__global__ __launch_bounds__(kSplitWalkNT) void split_walk_kernel(uint64_t num_samples, const ks_desc* __restrict__ desc,
                                                                  uint32_t num_series, uint32_t max_K, ks_params prm,
                                                                  ks_result* __restrict__ out,
                                                                  uint32_t* __restrict__ allU, uint64_t allU_len,
                                                                  SplitWs ws) {
  constexpr uint32_t W = kSplitWalkNT / kWave;
  __shared__ __align__(16) uint16_t is[KS_MAX_K];
  __shared__ uint16_t pos[KS_MAX_K];
  __shared__ uint64_t tie[kSplitSlots];
  __shared__ uint32_t partU[W * kWave], red[W];
  const SplitAt at = split_at(num_series, max_K - 1);
  const uint32_t s = at.s, slot = at.slot;
  if (s >= num_series) return;
  const ks_desc d = desc[s];
  const uint32_t K = d.K, tid = threadIdx.x, lane = lane_id(), w = wave_id();
  if (check_desc(d, num_samples, max_K) || 1u + slot * kWave > K - 1u) return;
  const SortKey* sorted = ws.sorted + (uint64_t)s * max_K;
  bool tied = false;
  for (uint32_t p0 = w * kWave; p0 < K; p0 += kSplitWalkNT) {
    const uint32_t p = p0 + lane;
    bool end = false;
    if (p < K) {
      const SortKey a = sorted[p];
      const uint32_t i = (uint32_t)a.lo & (KS_MAX_K - 1u);
      is[p] = (uint16_t)i;
      pos[i] = (uint16_t)p;
      end = p + 1 == K || group_end(a, sorted[p + 1]);
    }
    const uint64_t m = ballot(end);
    if (lane == 0) tie[p0 / kWave] = m;
    tied |= m != ballot(p < K);
  }
  const bool ties = block_any<kSplitWalkNT>(tied, red);  // its barriers publish the order
  const uint32_t len = ((K + W - 1) / W + 7u) & ~7u;  // positions per wave
  const uint32_t pa = min(K, w * len), pb = min(K, pa + len);
  uint32_t c[1] = {1u + slot * kWave + lane}, U[1] = {0};
  if (pa < pb) walk_pass<KS_MAX_K, 1>(is, pos, tie, ties, K, pa, pb, c, U);
  partU[w * kWave + lane] = U[0];
  __syncthreads();
  if (w != 0) return;
#pragma unroll
  for (uint32_t v = 1; v < W; ++v) U[0] = max(U[0], partU[v * kWave + lane]);
  const bool valid = c[0] <= K - 1u;
  if (allU && d.aux_offset <= allU_len && K <= allU_len - d.aux_offset) {
    if (valid) allU[d.aux_offset + c[0]] = U[0];
    if (slot == 0 && lane == 0) allU[d.aux_offset] = 0;
  }
  uint32_t bU = valid ? U[0] : 0u, bC = valid ? c[0] : 0u;
  wave_best(bU, bC, K);
  const uint32_t ns = (K - 1u + kWave - 1u) / kWave;
  if (ns > 1) {
    // the slots' winners meet in the workspace; the last workgroup to arrive reads them all
    uint32_t* best = ws.best + (uint64_t)s * kSplitSlots * 2;
    uint32_t done = 0;
    if (lane == 0) {
      __hip_atomic_store(best + slot * 2, bU, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(best + slot * 2 + 1, bC, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      done = __hip_atomic_fetch_add(ws.ticket + s, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
    }
    if ((uint32_t)__builtin_amdgcn_readfirstlane((int)done) != ns - 1u) return;
    bU = 0;
    bC = 0;
    if (lane < ns) {
      bU = __hip_atomic_load(best + lane * 2, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      bC = __hip_atomic_load(best + lane * 2 + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    wave_best(bU, bC, K);
  }
  if (lane == 0) write_choice(out + s, bU, bC, K, prm, 0u);
}

// ---------------------------------------------------------------- one workgroup
// Keys, order and the most significant split of one series or window whose row
// moments are at hand, by one workgroup: every row's rank counted (a few threads
// to a row where there are fewer rows than threads), the walk shared by all
// waves. That is a handful of barriers, where the radix sort of finish_series makes
// four for each of some ten digits.
template <int KMAX, int NT>
struct RankSmem {
  static constexpr uint32_t W = NT / kWave;
  uint64_t lo[KMAX], hi[KMAX];
  uint32_t rank[KMAX];
  __align__(16) uint16_t is[KMAX];
  uint16_t pos[KMAX];
  uint64_t tie[(KMAX + kWave - 1) / kWave];
  uint32_t partU[NT], bestU[W], bestC[W], red[W];
};

constexpr uint32_t kRankBlock = 256;

// Ends of the groups of equal Q to sm.tie, where sorted position p's key is at
// at(p); whether some two are equal.
template <int KMAX, int NT, class At>
__device__ __forceinline__ bool group_ends(RankSmem<KMAX, NT>& sm, uint32_t K, uint32_t w, At&& at) {
  const uint32_t lane = lane_id();
  bool tied = false;
  for (uint32_t p0 = w * kWave; p0 < K; p0 += NT) {
    const uint32_t p = p0 + lane;
    bool end = false;
    if (p < K) {
      const uint32_t i = at(p), j = at(min(p + 1, K - 1));
      end = p + 1 == K || group_end(SortKey{sm.lo[i], sm.hi[i]}, SortKey{sm.lo[j], sm.hi[j]});
    }
    const uint64_t m = ballot(end);
    if (lane == 0) sm.tie[p0 / kWave] = m;
    tied |= m != ballot(p < K);
  }
  return block_any<NT>(tied, sm.red);
}

// Order of K > kRankBlock keys: ranks are counted within blocks of kRankBlock keys,
// which are then in order in LDS, and searched for in every other block (2048
// keys: 256 compares and 63 reads a key in place of 2048 compares; with the masked
// walk a segmentation's window of 2048 rows takes 220 us alone on its CU, 603
// before). Leaves keys, is and pos in order; whether some two Q are equal.
template <int KMAX, int NT, class Key>
__device__ __forceinline__ bool order_blocks(RankSmem<KMAX, NT>& sm, Key&& key, uint32_t K, uint32_t w) {
  constexpr int E = (KMAX + NT - 1) / NT;
  const uint32_t tid = threadIdx.x, w0 = w * kWave;
  bool w53 = false;
  SortKey mine[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint32_t i = tid + e * NT;
    mine[e] = SortKey{0, 0};
    if (i < K) {
      mine[e] = key(i);
      sm.lo[i] = mine[e].lo;
      sm.hi[i] = mine[e].hi;
      w53 |= mine[e].hi != 0;
    }
  }
  const bool wide = block_any<NT>(w53, sm.red);
  uint32_t rank[E];
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint32_t b0 = (w0 + e * NT) & ~(kRankBlock - 1), b1 = min(K, b0 + kRankBlock);  // the wave's block
    rank[e] = b0 < K ? b0 + count_below(sm.lo, sm.hi, b0, b1, mine[e].lo, mine[e].hi, wide) : 0u;
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < E; ++e)
    if (tid + e * NT < K) {
      sm.lo[rank[e]] = mine[e].lo;
      sm.hi[rank[e]] = mine[e].hi;
    }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint32_t own = (w0 + e * NT) & ~(kRankBlock - 1);
    if (own >= K) continue;
    rank[e] -= own;
    for (uint32_t b0 = 0; b0 < K; b0 += kRankBlock) {
      if (b0 == own) continue;
      const uint32_t n = min(K - b0, kRankBlock);
      auto below = [&](uint32_t j) {  // key j of the block (j < n) is below this one
        const uint64_t lo = sm.lo[b0 + j];
        if (!wide) return lo < mine[e].lo;
        const uint64_t hi = sm.hi[b0 + j];
        return hi < mine[e].hi || (hi == mine[e].hi && lo < mine[e].lo);
      };
      uint32_t at = 0;
#pragma unroll
      for (uint32_t s = kRankBlock / 2; s; s >>= 1)
        if (at + s <= n && below(at + s - 1)) at += s;
      rank[e] += at + (at < n && below(at) ? 1u : 0u);
    }
  }
  __syncthreads();
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const uint32_t i = tid + e * NT;
    if (i < K) {
      sm.lo[rank[e]] = mine[e].lo;
      sm.hi[rank[e]] = mine[e].hi;
      sm.is[rank[e]] = (uint16_t)i;
      sm.pos[i] = (uint16_t)rank[e];
    }
  }
  __syncthreads();
  return group_ends(sm, K, w, [](uint32_t p) { return p; });
}

// The same for fewer keys, every rank one count over all of them; the keys stay in
// row order.
template <int KMAX, int NT, class Key>
__device__ __forceinline__ bool order_counts(RankSmem<KMAX, NT>& sm, Key&& key, uint32_t K, uint32_t w) {
  const uint32_t tid = threadIdx.x;
  bool w53 = false;
  for (uint32_t i = tid; i < K; i += NT) {
    const SortKey k = key(i);
    sm.lo[i] = k.lo;
    sm.hi[i] = k.hi;
    sm.rank[i] = 0;
    w53 |= k.hi != 0;
  }
  const bool wide = block_any<NT>(w53, sm.red);
  {  // several threads count for one row where there are fewer rows than threads
    const uint32_t KR = min((K + kWave - 1u) & ~(uint32_t)(kWave - 1), (uint32_t)NT), P = NT / KR;
    const uint32_t i0 = tid % KR, q = tid / KR, len = (K + P - 1) / P;
    const uint32_t j0 = min(K, q * len), j1 = min(K, j0 + len);
    if (q < P)
      for (uint32_t i = i0; i < K; i += KR)
        atomicAdd(&sm.rank[i], count_below(sm.lo, sm.hi, j0, j1, sm.lo[i], sm.hi[i], wide));
  }
  __syncthreads();
  for (uint32_t i = tid; i < K; i += NT) {
    const uint32_t p = sm.rank[i];
    sm.is[p] = (uint16_t)i;
    sm.pos[i] = (uint16_t)p;
  }
  __syncthreads();
  return group_ends(sm, K, w, [&](uint32_t p) { return (uint32_t)sm.is[p]; });
}

// key(i): row i's key (i < K). Candidates c_lo .. c_hi; their statistics to
// allU (nullable). Wave 0 returns the winner (c = 0: no candidate).
template <int KMAX, int NT, class Key>
__device__ __forceinline__ void rank_walk(RankSmem<KMAX, NT>& sm, Key&& key, uint32_t K, uint32_t c_lo, uint32_t c_hi,
                                          uint32_t* __restrict__ allU, uint32_t& bU, uint32_t& bC) {
  constexpr uint32_t W = NT / kWave;
  const uint32_t tid = threadIdx.x, lane = lane_id(), w = wave_id();
  bool ties;
  if (KMAX > (int)kRankBlock && K > kRankBlock) ties = order_blocks<KMAX, NT>(sm, key, K, w);
  else ties = order_counts<KMAX, NT>(sm, key, K, w);
  // 64-candidate slots: the waves of a slot share the positions (shares of a
  // multiple of 8), or a wave walks its slots one after the other
  const uint32_t ns = (c_hi - c_lo + kWave) / kWave;
  bU = 0;
  bC = 0;
  auto consider = [&](uint32_t c, uint32_t U) {
    if (c > c_hi) return;
    if (allU) allU[c] = U;
    if (bC == 0 || more_significant(U, c, bU, bC, K)) {
      bU = U;
      bC = c;
    }
  };
  if (ns < W) {
    const uint32_t Q = W / ns, slot = w / Q, share = w % Q;
    const uint32_t len = ((K + Q - 1) / Q + 7u) & ~7u;
    uint32_t c[1] = {c_lo + slot * kWave + lane}, U[1] = {0};
    if (slot < ns) {
      const uint32_t pa = min(K, share * len), pb = min(K, pa + len);
      if (pa < pb) walk_pass<KMAX, 1, (KMAX > (int)kRankBlock)>(sm.is, sm.pos, sm.tie, ties, K, pa, pb, c, U);
    }
    sm.partU[tid] = U[0];
    __syncthreads();
    if (slot < ns && share == 0) {
      for (uint32_t q = 1; q < Q; ++q) U[0] = max(U[0], sm.partU[tid + q * kWave]);
      consider(c[0], U[0]);
    }
  } else {
    for (uint32_t slot = w; slot < ns; slot += W) {
      uint32_t c[1] = {c_lo + slot * kWave + lane}, U[1];
      walk_pass<KMAX, 1, (KMAX > (int)kRankBlock)>(sm.is, sm.pos, sm.tie, ties, K, 0, K, c, U);
      consider(c[0], U[0]);
    }
  }
  wave_best(bU, bC, K);
  if (lane == 0) {
    sm.bestU[w] = bU;
    sm.bestC[w] = bC;
  }
  __syncthreads();
  if (w == 0) {
    bU = lane < W ? sm.bestU[lane] : 0u;
    bC = lane < W ? sm.bestC[lane] : 0u;
    wave_best(bU, bC, K);
  }
}

template <int KMAX>
__global__ __launch_bounds__(kTinyNT) void tiny_scan_kernel(const uint32_t* __restrict__ samples, uint64_t num_samples,
                                                            const ks_desc* __restrict__ desc, ks_params prm,
                                                            uint32_t max_K, ks_result* __restrict__ out,
                                                            uint32_t* __restrict__ allU, uint64_t allU_len) {
  constexpr uint32_t W = kTinyNT / kWave;
  __shared__ uint64_t s1[KMAX], s2lo[KMAX];
  __shared__ uint32_t s2hi[KMAX];
  __shared__ RankSmem<KMAX, kTinyNT> sm;
  const uint32_t s = blockIdx.x;
  const ks_desc d = desc[s];
  const uint32_t tid = threadIdx.x, lane = lane_id(), w = wave_id();
  const uint32_t bad = check_desc(d, num_samples, max_K);
  if (bad) {
    if (tid == 0) write_result(out + s, 0, 0, 0, 0, 0.0, 0.0, 1.0, bad);
    return;
  }
  const uint32_t K = d.K, N = d.N;
  const uint32_t mn = stream_rows(samples, d.offset, N, w, K, W, lane,
                                  [&](uint32_t i, uint64_t a, uint64_t b, uint32_t h, uint32_t) {
                                    if (lane == 0) {
                                      s1[i] = a;
                                      s2lo[i] = b;
                                      s2hi[i] = h;
                                    }
                                  });
  const uint32_t gmin = block_min_u32<kTinyNT>(mn, sm.red);  // its barriers publish the moments
  const bool fits = allU && d.aux_offset <= allU_len && K <= allU_len - d.aux_offset;
  uint32_t* au = fits ? allU + d.aux_offset : nullptr;
  uint32_t U, c;
  rank_walk(sm, [&](uint32_t i) { return sort_key(s1[i], s2lo[i], s2hi[i], i, N, gmin); }, K, 1u, K - 1u, au, U, c);
  if (tid != 0) return;
  if (fits) au[0] = 0;
  write_choice(out + s, U, c, K, prm, 0u);
}

}  // namespace
}  // namespace ks
