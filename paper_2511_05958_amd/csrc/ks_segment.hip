// Binary segmentation over a batch: every level boundary of each series, in one
// launch with one workgroup per series (more than 2^21 in several).
//
// The row moments (sum r, sum r^2) and minima of a series are kept in LDS. A
// window [a, b) of rows is a series of its own, but its eq. 2 keys need only its
// rows' moments and the window's minimum (the least row minimum), so the samples
// are read once. The workgroup takes windows from a stack: keys, ranks by
// counting smaller keys, the walk shared by all waves, the choice; a significant
// split is recorded and opens both sides. At the end one thread per boundary
// finds its place and its p-value.
//
// (One launch per depth for all open windows, with a split kernel after each, a
// read-back of the window counts every few depths and a sort at the end took 14
// depths x 10 - 25 us after a root pass of 107 us on 512 series of 256 rows of
// 1024 samples, 333 us a call, most depths with a handful of windows; the call
// takes 145 us now, of which the rows' stream is about 95.)
//
// A workgroup streams its own series' rows when there are enough series to keep
// HBM busy that way; with fewer, split_moments_kernel has spread the rows over
// the device and left the moments in the workspace.
#include <hip/hip_runtime.h>

#include <new>

#include "ks.h"
#include "ks_ctx.hpp"
#include "ks_scan.hpp"
#include "ks_select.hpp"
#include "ks_split.hpp"
#include "ks_wave.hpp"

using namespace ks_host;

namespace ks_host {

void free_seg(SegBuffers& b) {
  (void)hipFree(b.rows);
  b = SegBuffers{};
}

}  // namespace ks_host

namespace {

// Threads of a series' workgroup: barriers of eight waves are cheaper, and for
// K classes of up to 256 rows eight waves are enough for a window (4096 series
// of 256 x 1024 741 us, 769 with sixteen; 512 of up to 512 x 4096 354 and 269).
constexpr int tree_nt(int kmax) { return kmax <= 256 ? 512 : 1024; }

constexpr uint32_t kTreeSeries = 1u << 21;  // series of a launch

constexpr uint32_t kSmall = ks::kWave;  // windows of up to this many rows are a wave's work

template <int KMAX>
struct TreeSmem {
  static constexpr int NT = tree_nt(KMAX);
  static constexpr uint32_t W = NT / ks::kWave;
  uint64_t s1[KMAX], s2lo[KMAX];  // the series' rows
  uint32_t s2hi[KMAX], rmin[KMAX];
  union {
    ks::RankSmem<KMAX, NT> rw;  // a window that the workgroup shares
    struct {  // a wave's window
      uint64_t lo[kSmall], hi[kSmall];
      uint64_t stack[kSmall / 2];
      uint32_t order[kSmall];
    } wave[W];
  };
  // open windows, a | b << 16 | depth << 32, disjoint: those of more than
  // kSmall rows (the workgroup's stack), and the others (the waves' list)
  uint64_t stack[KMAX / kSmall + 1], small[KMAX / 2];
  uint32_t fU[KMAX];              // boundaries found: statistic, window, split, depth
  uint16_t fa[KMAX], fb[KMAX], fc[KMAX], fd[KMAX];
  uint32_t split;                 // the window's split if significant, else 0
  uint32_t found, next;           // the waves' counters
};

__device__ __forceinline__ uint64_t pack_window(uint32_t a, uint32_t b, uint32_t depth) {
  return (uint64_t)depth << 32 | (uint64_t)b << 16 | a;
}

// A window of at most kSmall rows and every window that opens inside it, by the
// calling wave: a row per lane, keys and order in the wave's own LDS, no
// workgroup barrier.
template <int KMAX>
__device__ __forceinline__ void tree_small(TreeSmem<KMAX>& sm, uint64_t window, uint32_t N, double c_alpha,
                                           uint32_t max_levels, uint32_t w, uint32_t lane) {
  auto& S = sm.wave[w];
  uint32_t top = 0;
  for (;;) {
    const uint32_t a = (uint32_t)window & 0xffffu, b = (uint32_t)(window >> 16) & 0xffffu;
    const uint32_t depth = (uint32_t)(window >> 32), K = b - a;
    const bool row = lane < K;
    const uint32_t at = a + (row ? lane : 0u);
    const uint32_t gmin = ks::wave_min_u32(sm.rmin[at]);
    const ks::SortKey k = ks::sort_key(sm.s1[at], sm.s2lo[at], sm.s2hi[at], lane, N, gmin);
    const bool wide = ks::ballot(row && k.hi != 0) != 0;
    S.lo[lane] = k.lo;
    S.hi[lane] = k.hi;
    ks::wave_lds_sync();
    const uint32_t rank = ks::count_below(S.lo, S.hi, 0, K, k.lo, k.hi, wide);
    if (row) S.order[rank] = lane;
    ks::wave_lds_sync();
    // lane p: the row at sorted position p
    const uint32_t mine = S.order[row ? lane : 0u], after = S.order[lane + 1 < K ? lane + 1 : 0u];
    const bool end = row && (lane + 1 == K || ks::group_end(ks::SortKey{S.lo[mine], S.hi[mine]},
                                                            ks::SortKey{S.lo[after], S.hi[after]}));
    const uint64_t tie = ks::ballot(end);
    const int32_t c = (int32_t)lane + 1, up = (int32_t)K - c;
    int32_t D = 0, mx = 0, mn = 0;
    for (uint32_t p = 0; p < K; ++p) {
      const int32_t r = __builtin_amdgcn_readlane((int)mine, (int)p);
      D += r < c ? up : -c;
      if ((tie >> p) & 1u) {
        mx = max(mx, D);
        mn = min(mn, D);
      }
    }
    uint32_t bU = (uint32_t)c < K ? (uint32_t)max(mx, -mn) : 0u, bC = (uint32_t)c < K ? (uint32_t)c : 0u;
    ks::wave_best(bU, bC, K);
    if (ks::significant(bU, bC, K, c_alpha)) {
      if (lane == 0) {
        const uint32_t n = atomicAdd(&sm.found, 1u);
        sm.fU[n] = bU;
        sm.fa[n] = (uint16_t)a;
        sm.fb[n] = (uint16_t)b;
        sm.fc[n] = (uint16_t)(a + bC);
        sm.fd[n] = (uint16_t)depth;
      }
      if (max_levels == 0 || depth + 1 < max_levels) {
        if (K - bC >= 2) S.stack[top++] = pack_window(a + bC, b, depth + 1);  // every lane the same value
        if (bC >= 2) S.stack[top++] = pack_window(a, a + bC, depth + 1);
      }
    }
    ks::wave_lds_sync();
    if (top == 0) return;
    window = S.stack[--top];
    window = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(window >> 32)) << 32 |
             (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)window);
    ks::wave_lds_sync();
  }
}

// The most significant split of the window of rows a .. a + K - 1; sm.split gets
// it if it is significant, and record n of the boundaries is written then.
template <int KMAX>
__device__ __forceinline__ void tree_window(TreeSmem<KMAX>& sm, uint32_t a, uint32_t K, uint32_t depth, uint32_t N,
                                            double c_alpha, uint32_t n) {
  constexpr uint32_t kTreeNT = TreeSmem<KMAX>::NT;
  const uint32_t tid = threadIdx.x;
  uint32_t mn = 0xffffffffu;
  for (uint32_t i = tid; i < K; i += kTreeNT) mn = min(mn, sm.rmin[a + i]);
  const uint32_t gmin = ks::block_min_u32<kTreeNT>(mn, sm.rw.red);
  uint32_t bU, bC;
  ks::rank_walk(
      sm.rw, [&](uint32_t i) { return ks::sort_key(sm.s1[a + i], sm.s2lo[a + i], sm.s2hi[a + i], i, N, gmin); }, K, 1u,
      K - 1u, nullptr, bU, bC);
  if (tid == 0) {
    const bool sig = ks::significant(bU, bC, K, c_alpha);
    sm.split = sig ? bC : 0u;
    if (sig) {
      sm.fU[n] = bU;
      sm.fa[n] = (uint16_t)a;
      sm.fb[n] = (uint16_t)(a + K);
      sm.fc[n] = (uint16_t)(a + bC);
      sm.fd[n] = (uint16_t)depth;
    }
  }
  ks::block_publish();
}

// rows: the moments of series s at s * max_K (nullptr: streamed here).
template <int KMAX>
__global__ __launch_bounds__(tree_nt(KMAX)) void seg_tree_kernel(const uint32_t* __restrict__ samples, uint64_t num_samples,
                                                           const ks_desc* __restrict__ desc, ks_params prm,
                                                           uint32_t max_K, const ks::RowMom* __restrict__ rows,
                                                           uint32_t max_levels, uint32_t max_cp,
                                                           ks_result* __restrict__ cps, uint32_t* __restrict__ counts) {
  constexpr uint32_t kTreeNT = TreeSmem<KMAX>::NT, kTreeW = TreeSmem<KMAX>::W;
  __shared__ TreeSmem<KMAX> sm;
  const uint32_t s = blockIdx.x, tid = threadIdx.x, lane = ks::lane_id();
  const ks_desc d = desc[s];
  if (ks::check_desc(d, num_samples, max_K)) {
    if (tid == 0) counts[s] = KS_SEGMENT_BAD;
    return;
  }
  const uint32_t K = d.K, N = d.N;
  if (rows) {
    const ks::RowMom* rm = rows + (uint64_t)s * max_K;
    for (uint32_t i = tid; i < K; i += kTreeNT) {
      const ks::RowMom r = rm[i];
      sm.s1[i] = r.s1;
      sm.s2lo[i] = r.s2lo;
      sm.s2hi[i] = r.s2hi;
      sm.rmin[i] = r.pad;
    }
  } else {
    ks::stream_rows<true>(samples, d.offset, N, ks::wave_id(), K, kTreeW, lane,
                          [&](uint32_t i, uint64_t s1, uint64_t s2, uint32_t s2h, uint32_t rmin) {
                            if (lane == 0) {
                              sm.s1[i] = s1;
                              sm.s2lo[i] = s2;
                              sm.s2hi[i] = s2h;
                              sm.rmin[i] = rmin;
                            }
                          });
  }
  uint32_t top = 0, small = 0, found = 0;  // every thread keeps the same
  auto open = [&](uint32_t a, uint32_t b, uint32_t depth) {
    const bool big = b - a > kSmall;
    if (tid == 0) (big ? sm.stack[top] : sm.small[small]) = pack_window(a, b, depth);
    big ? ++top : ++small;
  };
  open(0, K, 0);
  ks::block_publish();
  while (top > 0) {  // what is read from LDS here is the same for every thread: scalars, so that the loop is the scalar unit's
    const uint64_t e = sm.stack[--top];
    const uint32_t ab = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)e);
    const uint32_t depth = (uint32_t)__builtin_amdgcn_readfirstlane((int)(e >> 32));
    const uint32_t a = ab & 0xffffu, b = ab >> 16;
    tree_window<KMAX>(sm, a, b - a, depth, N, prm.c_alpha, found);
    const uint32_t c = (uint32_t)__builtin_amdgcn_readfirstlane((int)sm.split);
    if (c != 0) {
      ++found;
      if (max_levels == 0 || depth + 1 < max_levels) {
        if (b - a - c >= 2) open(a + c, b, depth + 1);
        if (c >= 2) open(a, a + c, depth + 1);
      }
    }
    ks::block_publish();
  }
  if (tid == 0) {
    sm.found = found;
    sm.next = 0;
  }
  ks::block_publish();
  for (;;) {  // the small windows, a wave each
    uint32_t j = 0;
    if (lane == 0) j = atomicAdd(&sm.next, 1u);
    j = (uint32_t)__builtin_amdgcn_readfirstlane((int)j);
    if (j >= small) break;
    tree_small<KMAX>(sm, sm.small[j], N, prm.c_alpha, max_levels, ks::wave_id(), lane);
  }
  __syncthreads();
  found = sm.found;
  if (tid == 0) counts[s] = found;
  ks_result* out = cps + (uint64_t)s * max_cp;
  for (uint32_t j = tid; j < found; j += kTreeNT) {
    const uint32_t cp = sm.fc[j];
    uint32_t at = 0;
    for (uint32_t q = 0; q < found; ++q) at += sm.fc[q] < cp ? 1u : 0u;
    if (at >= max_cp) continue;
    ks_result r;
    const uint32_t a = sm.fa[j];
    ks::write_choice(&r, sm.fU[j], cp - a, sm.fb[j] - a, prm, 0u);
    r.cp = cp;
    r.pad = sm.fd[j];
    out[at] = r;
  }
}

template <int KMAX>
void launch_tree(uint32_t num_series, hipStream_t st, const uint32_t* samples, uint64_t num_samples, const ks_desc* desc,
                 const ks_params& prm, uint32_t max_K, const ks::RowMom* rows, uint32_t max_levels, uint32_t max_cp,
                 ks_result* cps, uint32_t* counts) {
  hipLaunchKernelGGL(seg_tree_kernel<KMAX>, dim3(num_series), dim3(tree_nt(KMAX)), 0, st, samples, num_samples, desc, prm,
                     max_K, rows, max_levels, max_cp, cps, counts);
}

int ensure_seg(ks_ctx* c, uint64_t rows) {
  SegBuffers& b = c->seg;
  if (rows <= b.cap_rows) return KS_OK;
  hipError_t e = hipDeviceSynchronize();
  if (e != hipSuccess) return hip_fail(e, "hipDeviceSynchronize");
  free_seg(b);
  if (hipMalloc(&b.rows, sizeof(ks::RowMom) * rows) != hipSuccess) {
    free_seg(b);
    (void)hipGetLastError();
    return KS_E_NOMEM;
  }
  b.cap_rows = rows;
  return KS_OK;
}

}  // namespace

extern "C" int ks_segment_batch(ks_ctx* ctx, const uint32_t* samples, uint64_t num_samples, const ks_desc* desc,
                                uint32_t num_series, const ks_params* params, uint32_t max_levels, uint32_t max_cp,
                                ks_result* cps, uint32_t* counts, void* stream) {
  if (!ctx || !params) return KS_E_INVALID;
  if (int rc = check_params(params)) return rc;
  if (num_series == 0) return KS_OK;
  if (!samples || !desc || !cps || !counts || max_cp == 0) return KS_E_INVALID;
  const uint32_t max_K = params->max_K ? params->max_K : KS_MAX_K;
  if (max_K < 2 || max_K > KS_MAX_K) return KS_E_RANGE;
  DeviceGuard g(ctx->device);
  if (g.err != hipSuccess) return hip_fail(g.err, "hipSetDevice");
  hipStream_t st = (hipStream_t)stream;
  const ks::RowMom* rows = nullptr;
  // fewer than two workgroups per CU: the rows are spread over the device first
  if (num_series < 2u * (uint32_t)ctx->num_cus) {
    if (int rc = ensure_seg(ctx, (uint64_t)num_series * max_K)) return rc;
    const ks::SplitWs ws{ctx->seg.rows, nullptr, nullptr, nullptr};
    ks::launch_split_moments((uint32_t)ctx->num_cus, samples, num_samples, desc, num_series, max_K, nullptr, ws, st);
    rows = ctx->seg.rows;
  }
  auto run = [&](auto f) {
    // a grid holds up to 2^32 - 1 threads
    for (uint32_t s = 0, n; s < num_series; s += n) {
      n = num_series - s < kTreeSeries ? num_series - s : kTreeSeries;
      f(n, st, samples, num_samples, desc + s, *params, max_K, rows, max_levels, max_cp, cps + (uint64_t)s * max_cp,
        counts + s);
    }
  };
  switch (k_class(max_K)) {
    case 0: run(launch_tree<64>); break;
    case 1: run(launch_tree<128>); break;
    case 2: run(launch_tree<256>); break;
    case 3: run(launch_tree<512>); break;
    case 4: run(launch_tree<1024>); break;
    default: run(launch_tree<2048>);
  }
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? KS_OK : hip_fail(e, "segmentation launch");
}
