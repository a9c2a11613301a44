// C ABI of the K-S change-point library: contexts, workspace, validation,
// launch plans (direct grid or planned persistent launch captured in a
// hipGraph) and the tuning table.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <new>
#include <tuple>

#include "ks.h"
#include "ks_ctx.hpp"
#include "ks_persist.hpp"
#include "ks_split.hpp"

using namespace ks_host;

namespace ks_host {

thread_local char g_hip_msg[256] = "HIP error";

int hip_fail(hipError_t e, const char* what) {
  snprintf(g_hip_msg, sizeof(g_hip_msg), "HIP error in %s: %s", what, hipGetErrorString(e));
  return KS_E_HIP;
}

// the variant tables, one per object built from ks_scan_variants.hip
extern const ScanKernels scan_table_0[kNumKClasses], scan_table_1[kNumKClasses], scan_table_2[kNumKClasses],
    scan_table_3[kNumKClasses], scan_table_4[kNumKClasses], scan_table_5[kNumKClasses];
static_assert(kNumVariants == 6, "one table per variant");

const ScanKernels& scan_kernels(int kclass, int variant) {
  static const ScanKernels* const tables[kNumVariants] = {scan_table_0, scan_table_1, scan_table_2,
                                                          scan_table_3, scan_table_4, scan_table_5};
  return tables[variant][kclass];
}

}  // namespace ks_host

// Scratch of ks_scan_batch_noalloc: the ordered plan's header (256 B), then
// items, per-series moment bases, completion counts and minima laid out for
// KS_NOALLOC_MAX_SERIES series. Each device holds its own copy for the life
// of the process; host code reaches it only through the address that
// hipGetSymbolAddress returns for the current device.
namespace {
constexpr uint64_t kScratchItems = 256;
constexpr uint64_t kScratchBase = kScratchItems + 8ull * KS_NOALLOC_MAX_SERIES;
constexpr uint64_t kScratchDone = kScratchBase + 8ull * KS_NOALLOC_MAX_SERIES;
constexpr uint64_t kScratchMin = kScratchDone + 4ull * KS_NOALLOC_MAX_SERIES;
constexpr uint64_t kScratchBytes = kScratchMin + 4ull * KS_NOALLOC_MAX_SERIES;
static_assert(sizeof(ks::Item) == 8, "item layout");
}  // namespace

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
unsigned char* g_scratch[kMaxDevices] = {};  // device address of `scratch` per device

// Resolve the scratch array's address on `device` (made current by the caller), once per device.
int resolve_scratch(int device) {
  if (device < 0 || device >= kMaxDevices) return KS_E_RANGE;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  if (g_scratch[device]) return KS_OK;
  void* p = nullptr;
  const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
  if (e != hipSuccess || !p) return hip_fail(e != hipSuccess ? e : hipErrorInvalidSymbol, "hipGetSymbolAddress");
  g_scratch[device] = static_cast<unsigned char*>(p);
  return KS_OK;
}

unsigned char* scratch_of(int device) {
  if (device < 0 || device >= kMaxDevices) return nullptr;
  std::lock_guard<std::mutex> lk(g_scratch_mu);
  return g_scratch[device];
}

// Batches of few series under the default plan (ks_split.hpp). The spread scan
// serves up to 384 series (one and a half per CU) of any K: there it is ahead of a
// workgroup per series of variant 0 throughout (384 of 1024 x 64: 249 us against
// 272, of 1024 x 1024 468 against 530, of 64 x 4 under max_K 0 18 against 23) and
// ahead of variant 2's by far where series are uneven (384 up to 2048 x 4096: 734
// against 1332), behind it by up to a third for equal ones of 1024 rows and more
// (256 of 2048 x 64: 565 against 440); past 384 equal ones are behind by more. The
// one-launch scan serves up to 1024 series of at most 256 rows and (on average)
// 256 KB: 1024 of 64 x 256 take 27 us against 29, 512 of 256 x 64 34 against 57; a
// series of more than 256 KB keeps its one workgroup busy for longer than the
// spread scan's two more launches take.
uint32_t split_max_series(const ks_ctx* c) { return 3u * (uint32_t)c->num_cus / 2u; }
uint32_t tiny_max_series(const ks_ctx* c) { return 4u * (uint32_t)c->num_cus; }
constexpr int kTinyMaxClass = 2;                 // K <= 256
constexpr uint64_t kTinyMaxSamples = 1u << 16;   // 256 KB a series

void free_workspace(ks_ctx* c) {
  (void)hipFree(c->hdr);
  (void)hipFree(c->items);
  (void)hipFree(c->mom_base);
  (void)hipFree(c->done);
  (void)hipFree(c->smin);
  (void)hipFree(c->mom);
  c->hdr = nullptr;
  c->items = nullptr;
  c->mom_base = nullptr;
  c->done = nullptr;
  c->smin = nullptr;
  c->mom = nullptr;
  c->cap_series = c->cap_rows = 0;
}

void free_split(ks_ctx* c) {
  (void)hipFree(c->split_mom);
  (void)hipFree(c->split_sorted);
  (void)hipFree(c->split_best);
  (void)hipFree(c->split_ticket);
  c->split_mom = nullptr;
  c->split_sorted = nullptr;
  c->split_best = nullptr;
  c->split_ticket = nullptr;
}

// The spread scan's workspace, for all that it serves (31 MB) at once: it never
// moves, and calls that were captured keep theirs. KS_E_NOMEM also where there is
// none yet and `st` is being captured: the caller runs the ordered grid then.
int ensure_split(ks_ctx* c, hipStream_t st) {
  if (c->split_ticket) return KS_OK;
  const uint64_t ns = split_max_series(c), rows = ns * KS_MAX_K;
  hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(st, &capture) != hipSuccess || capture != hipStreamCaptureStatusNone) {
    (void)hipGetLastError();
    return KS_E_NOMEM;
  }
  if (hipMalloc(&c->split_mom, sizeof(ks::RowMom) * rows) != hipSuccess ||
      hipMalloc(&c->split_sorted, sizeof(ks::SortKey) * rows) != hipSuccess ||
      hipMalloc(&c->split_best, sizeof(uint32_t) * 2 * ns * ks::kSplitSlots) != hipSuccess ||
      hipMalloc(&c->split_ticket, sizeof(uint32_t) * ns) != hipSuccess) {
    free_split(c);
    (void)hipGetLastError();
    return KS_E_NOMEM;
  }
  return KS_OK;
}

}  // namespace

// Grow the workspace to hold num_series series and rows split-series rows.
int ks_host::ensure_workspace(ks_ctx* c, uint64_t num_series, uint64_t rows) {
  if (num_series <= c->cap_series && rows <= c->cap_rows && c->hdr) return KS_OK;
  const uint64_t ns = num_series > c->cap_series ? num_series : c->cap_series;
  const uint64_t nr = rows > c->cap_rows ? rows : c->cap_rows;
  hipError_t e = hipDeviceSynchronize();
  if (e != hipSuccess) return hip_fail(e, "hipDeviceSynchronize");
  free_workspace(c);
  if (hipMalloc(&c->hdr, 256) != hipSuccess || hipMalloc(&c->items, sizeof(ks::Item) * ks::kMaxChunks * ns) != hipSuccess ||
      hipMalloc(&c->mom_base, sizeof(uint64_t) * ns) != hipSuccess || hipMalloc(&c->done, sizeof(uint32_t) * ns) != hipSuccess ||
      hipMalloc(&c->smin, sizeof(uint32_t) * ns) != hipSuccess ||
      hipMalloc(&c->mom, sizeof(ks::RowMom) * (nr ? nr : 1)) != hipSuccess) {
    free_workspace(c);
    (void)hipGetLastError();
    return KS_E_NOMEM;
  }
  c->cap_series = ns;
  c->cap_rows = nr;
  return KS_OK;
}

namespace {

ks::Workspace workspace_of(const ks_ctx* c) {
  return ks::Workspace{c->hdr, c->items, c->mom_base, c->done, c->smin, c->mom};
}

struct ScanArgs {
  const uint32_t* samples;
  uint64_t num_samples;
  const ks_desc* desc;
  uint32_t num_series;
  ks_params prm;
  uint32_t max_K;
  ks_result* out;
  uint32_t* allU;
  uint64_t allU_len;
  uint32_t chunk;
  ks::Workspace ws;
};

// Launch the grid scan of variant v (one workgroup per series, descriptor order).
hipError_t launch_grid(int kc, int v, const ScanArgs& a, hipStream_t st) {
  ScanArgs x = a;
  const uint32_t* order = nullptr;
  void* args[] = {&x.samples, &x.num_samples, &x.desc, &x.num_series, &x.prm, &x.max_K,
                  &x.out, &x.allU, &x.allU_len, &order};
  return hipLaunchKernel(scan_kernels(kc, v).grid, dim3(x.num_series), dim3(kVariants[v].nt), args, 0, st);
}

int persistent_grid(ks_ctx* c, int kc, int v, uint32_t& grid) {
  if (!c->occupancy[kc][v]) {
    int nb = 0;
    hipError_t e =
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, scan_kernels(kc, v).persistent, kVariants[v].nt, 0);
    if (e != hipSuccess) return hip_fail(e, "hipOccupancyMaxActiveBlocksPerMultiprocessor");
    c->occupancy[kc][v] = nb > 0 ? nb : 1;
  }
  grid = (uint32_t)(c->num_cus * c->occupancy[kc][v]);
  return KS_OK;
}

// Launch the plan's kernels (directly, or from a cached hipGraph whose kernel
// arguments are updated for this call).
int launch_plan(ks_ctx* c, int kc, int v, int mode, const ScanArgs& a, bool use_graph, hipStream_t st) {
  const uint32_t nt = (uint32_t)kVariants[v].nt;
  const ScanKernels& K = scan_kernels(kc, v);
  ScanArgs x = a;
  const uint32_t* order = reinterpret_cast<const uint32_t*>(x.ws.items);
  void* plan_args[] = {&x.desc, &x.num_series, &x.num_samples, &x.max_K, &x.chunk, &x.ws};
  void* grid_args[] = {&x.samples, &x.num_samples, &x.desc, &x.num_series, &x.prm, &x.max_K,
                       &x.out, &x.allU, &x.allU_len, &order};
  void* pers_args[] = {&x.samples, &x.num_samples, &x.desc, &x.num_series, &x.prm, &x.max_K,
                       &x.out, &x.allU, &x.allU_len, &x.chunk, &x.ws};
  void* fin_args[] = {&x.num_samples, &x.desc, &x.num_series, &x.prm, &x.max_K, &x.out,
                      &x.allU, &x.allU_len, &x.chunk, &x.ws};
  hipKernelNodeParams np[3] = {};
  int n = 0;
  np[n].blockDim = dim3(ks::kPlanNT);
  np[n].gridDim = dim3(1);
  np[n].func = reinterpret_cast<void*>(&ks::plan_kernel);
  np[n++].kernelParams = plan_args;
  uint32_t grid = x.num_series;
  if (mode == KS_LAUNCH_PERSISTENT) {
    if (int rc = persistent_grid(c, kc, v, grid)) return rc;
    np[n].blockDim = dim3(nt);
    np[n].gridDim = dim3(grid);
    np[n].func = const_cast<void*>(K.persistent);
    np[n++].kernelParams = pers_args;
    np[n].blockDim = dim3(nt);
    np[n].gridDim = dim3(x.num_series);
    np[n].func = const_cast<void*>(K.finish);
    np[n++].kernelParams = fin_args;
  } else {
    np[n].blockDim = dim3(nt);
    np[n].gridDim = dim3(x.num_series);
    np[n].func = const_cast<void*>(K.grid);
    np[n++].kernelParams = grid_args;
  }
  hipError_t e;
  if (!use_graph) {
    for (int i = 0; i < n; ++i) {
      e = hipLaunchKernel(np[i].func, np[i].gridDim, np[i].blockDim, np[i].kernelParams, 0, st);
      if (e != hipSuccess) return hip_fail(e, "plan launch");
    }
    return KS_OK;
  }
  // the graph topology depends on the grid sizes only through the nodes'
  // parameters, so one graph per (mode, K class, variant, persistent grid) is reused
  auto key = std::make_tuple(mode, kc, v, mode == KS_LAUNCH_PERSISTENT ? grid : 0u);
  auto it = c->graphs.find(key);
  if (it == c->graphs.end()) {
    GraphEntry g;
    if ((e = hipGraphCreate(&g.graph, 0)) != hipSuccess) return hip_fail(e, "hipGraphCreate");
    for (int i = 0; i < n && e == hipSuccess; ++i)
      e = hipGraphAddKernelNode(&g.node[i], g.graph, i ? &g.node[i - 1] : nullptr, i ? 1 : 0, &np[i]);
    if (e == hipSuccess) e = hipGraphInstantiate(&g.exec, g.graph, nullptr, nullptr, 0);
    if (e != hipSuccess) {
      (void)hipGraphDestroy(g.graph);
      return hip_fail(e, "graph build");
    }
    g.nodes = n;
    it = c->graphs.emplace(key, g).first;
  } else {
    for (int i = 0; i < n; ++i)
      if ((e = hipGraphExecKernelNodeSetParams(it->second.exec, it->second.node[i], &np[i])) != hipSuccess)
        return hip_fail(e, "graph update");
  }
  if ((e = hipGraphLaunch(it->second.exec, st)) != hipSuccess) return hip_fail(e, "hipGraphLaunch");
  return KS_OK;
}

// Whether a batch takes the one-launch scan (by the mean size of its series, if
// the sample buffer holds no more than the batch; any series is scanned right).
bool tiny_batch(const ks_ctx* c, int kc, const ScanArgs& a) {
  return kc <= kTinyMaxClass && a.num_series <= tiny_max_series(c) && a.num_samples / a.num_series <= kTinyMaxSamples;
}

// The scan of a batch of few series (KS_E_NOMEM, nothing launched, where its
// workspace cannot be had). Launched directly: replaying one or three
// kernels from a graph costs more on the host (27 us a call for one sweep,
// against 8).
int launch_split(ks_ctx* c, int kc, const ScanArgs& a, hipStream_t st) {
  if (tiny_batch(c, kc, a)) {
    auto run = [&](auto kernel) {
      hipLaunchKernelGGL(kernel, dim3(a.num_series), dim3(ks::kTinyNT), 0, st, a.samples, a.num_samples, a.desc, a.prm,
                         a.max_K, a.out, a.allU, a.allU_len);
    };
    switch (kc) {
      case 0: run(ks::tiny_scan_kernel<64>); break;
      case 1: run(ks::tiny_scan_kernel<128>); break;
      default: run(ks::tiny_scan_kernel<256>);
    }
  } else {
    if (int rc = ensure_split(c, st)) return rc;
    const ks::SplitWs ws{c->split_mom, c->split_sorted, c->split_best, c->split_ticket};
    ks::launch_split_moments((uint32_t)c->num_cus, a.samples, a.num_samples, a.desc, a.num_series, a.max_K, a.out, ws, st);
    hipLaunchKernelGGL(ks::split_rank_kernel, ks::split_grid(a.num_series, a.max_K), dim3(ks::kSplitNT), 0, st,
                       a.num_samples, a.desc, a.num_series, a.max_K, ws);
    hipLaunchKernelGGL(ks::split_walk_kernel, ks::split_grid(a.num_series, a.max_K - 1), dim3(ks::kSplitWalkNT), 0, st,
                       a.num_samples, a.desc, a.num_series, a.max_K, a.prm, a.out, a.allU, a.allU_len, ws);
  }
  const hipError_t e = hipGetLastError();
  return e == hipSuccess ? KS_OK : hip_fail(e, "split scan launch");
}

// {KS_LAUNCH_ORDERED, 1 MiB, 1, 0}, recorded or not, is the default plan: the
// library chooses (default_cfg). Every other record is run as it says.
bool is_default(const LaunchCfg& c) {
  return c.mode == KS_LAUNCH_ORDERED && c.chunk_bytes == 1u << 20 && c.graph == 1 && c.variant == 0;
}

LaunchCfg recorded(const ks_ctx* c, int kc, uint32_t num_series) {
  const auto it = c->tuned.find(std::make_tuple(kc, num_series));
  return it != c->tuned.end() ? it->second : LaunchCfg{};
}

// What a batch runs under the default plan: the scan of few series, or the ordered
// grid with the kernel variant by size and a direct launch (a graph's update costs
// more on the host than the second kernel's launch: 1100 series of 64 x 64 30
// us a call from a graph, 24 direct). Variant 2, eight waves per series instead of
// four, for K classes of 1024 and 2048 rows, whose LDS allows as many workgroups
// either way (1024 series of 2048 x 64 1702 us with four, 1137 with eight; 4096 of
// 1024 x 256 1722 and 1507), and in the 512-row class for series of more than 640 KB
// on average up to 40 of them per CU, where a wait for the largest ones' stream is
// left at the end: 4096 uneven ones up to 512 x 4096 755 us with four waves, 530
// with eight, 8192 of them 1010 and 951; 16384 1807 and 1876, as there is always
// another series to hide it. Of smaller equal series the barriers cost more: 8192
// of 512 x 256 972 and 1033, of 512 x 384 1257 and 1259, of 512 x 512 1512 and 1459
// (variant 5, two walk slots, is within 1% of variant 0 in all of these).
// Smaller classes have waves enough: 4096 of 256 x 1024 take 668 and 671. From 2^23
// series on a grid of 2^32 - 1 threads does not hold them with eight waves each.
LaunchCfg default_cfg(const ks_ctx* c, int kc, const ScanArgs& a) {
  LaunchCfg cfg;
  cfg.graph = 0;
  cfg.spread = a.num_series <= split_max_series(c) || tiny_batch(c, kc, a);
  const bool few = a.num_series <= 40u * (uint32_t)c->num_cus;
  const bool long_series =
      kKClass[kc] >= 1024 || (kKClass[kc] >= 512 && few && a.num_samples / a.num_series > (160u << 10));
  if (long_series && a.num_series < (1u << 23)) cfg.variant = 2;
  return cfg;
}

// The plan of a call: the record of its shape, with the modes and the graph that
// its options override.
LaunchCfg config_for(const ks_ctx* c, int kc, const ScanArgs& a, uint32_t opts) {
  LaunchCfg cfg = recorded(c, kc, a.num_series);
  if (opts & KS_OPT_GRID) cfg.mode = KS_LAUNCH_GRID;
  if (opts & KS_OPT_PERSISTENT) cfg.mode = KS_LAUNCH_PERSISTENT;
  if (is_default(cfg)) cfg = default_cfg(c, kc, a);
  if (opts & KS_OPT_NO_GRAPH) cfg.graph = 0;
  return cfg;
}

int scan_with(ks_ctx* ctx, const ScanArgs& a, int kc, const LaunchCfg& cfg, hipStream_t st) {
  if (cfg.mode == KS_LAUNCH_GRID) {
    hipError_t e = launch_grid(kc, cfg.variant, a, st);
    return e == hipSuccess ? KS_OK : hip_fail(e, "scan launch");
  }
  if (cfg.spread) {
    const int rc = launch_split(ctx, kc, a, st);
    if (rc != KS_E_NOMEM) return rc;
  }
  const bool split = cfg.mode == KS_LAUNCH_PERSISTENT;
  if (int rc = ensure_workspace(ctx, a.num_series, split ? (uint64_t)a.num_series * a.max_K : 0)) return rc;
  ScanArgs b = a;
  b.chunk = split ? cfg.chunk_bytes : ks::kNoSplit;  // the ordered grid never splits
  b.ws = workspace_of(ctx);
  return launch_plan(ctx, kc, cfg.variant, cfg.mode, b, cfg.graph != 0, st);
}

bool valid_launch(const ks_launch* c) {
  return c && c->mode <= KS_LAUNCH_ORDERED && c->graph <= 1 && c->chunk_bytes >= 4096u &&
         c->chunk_bytes <= (1u << 30) && c->variant < (uint32_t)kNumVariants;
}

LaunchCfg from_launch(const ks_launch* c) {
  LaunchCfg l;
  l.mode = (int)c->mode;
  l.chunk_bytes = c->chunk_bytes;
  l.graph = (int)c->graph;
  l.variant = (int)c->variant;
  return l;
}

ks_launch to_launch(const LaunchCfg& l) {
  return ks_launch{(uint32_t)l.mode, l.chunk_bytes, (uint32_t)l.graph, (uint32_t)l.variant};
}

// Tune-cache lines: "<arch> <cus> <kclass> <num_series> <mode> <chunk_bytes> <graph> <variant>".
void load_tune_cache(ks_ctx* c) {
  const char* path = std::getenv("KS_TUNE_CACHE");
  if (!path || !*path) return;
  FILE* f = std::fopen(path, "r");
  if (!f) return;
  char arch[128];
  int cus, kc, pers, graph, var;
  unsigned ns, chunk;
  while (std::fscanf(f, "%127s %d %d %u %d %u %d %d", arch, &cus, &kc, &ns, &pers, &chunk, &graph, &var) == 8) {
    ks_launch l{(uint32_t)pers, chunk, (uint32_t)graph, (uint32_t)var};
    if (c->arch == arch && cus == c->num_cus && kc >= 0 && kc < kNumKClasses && var >= 0 && valid_launch(&l))
      c->tuned[std::make_tuple(kc, (uint32_t)ns)] = from_launch(&l);
  }
  std::fclose(f);
}

void append_tune_cache(const ks_ctx* c, int kc, uint32_t ns, const LaunchCfg& l) {
  const char* path = std::getenv("KS_TUNE_CACHE");
  if (!path || !*path) return;
  FILE* f = std::fopen(path, "a");
  if (!f) return;
  std::fprintf(f, "%s %d %d %u %d %u %d %d\n", c->arch.c_str(), c->num_cus, kc, ns, l.mode, l.chunk_bytes, l.graph,
               l.variant);
  std::fclose(f);
}

}  // namespace

extern "C" {

int ks_version(void) { return KS_VERSION; }

const char* ks_status_string(int status) {
  switch (status) {
    case KS_OK: return "ok";
    case KS_E_INVALID: return "invalid argument (null pointer or bad parameter)";
    case KS_E_RANGE: return "size outside the documented limits";
    case KS_E_STATE: return "call order or workspace state mismatch";
    case KS_E_HIP: return g_hip_msg;
    case KS_E_MODEL: return "bad model handle, file or weights";
    case KS_E_NOMEM: return "device allocation failed";
    default: return "unknown status";
  }
}

int ks_params_init(ks_params* p, double alpha) {
  if (!p || !(alpha > 0.0 && alpha < 1.0)) return KS_E_INVALID;
  p->alpha = alpha;
  p->c_alpha = -0.5 * std::log(alpha / 2.0);
  p->max_K = 0;
  p->w = 8;
  p->tau = 0.5f;
  p->opts = 0;
  return KS_OK;
}

int ks_ctx_create(int device, ks_ctx** out) {
  if (!out) return KS_E_INVALID;
  *out = nullptr;
  int n = 0;
  hipError_t e = hipGetDeviceCount(&n);
  if (e != hipSuccess) return hip_fail(e, "hipGetDeviceCount");
  if (device < 0 || device >= n) return KS_E_RANGE;
  hipDeviceProp_t prop;
  e = hipGetDeviceProperties(&prop, device);
  if (e != hipSuccess) return hip_fail(e, "hipGetDeviceProperties");
  {
    DeviceGuard g(device);
    if (g.err != hipSuccess) return hip_fail(g.err, "hipSetDevice");
    if (int rc = resolve_scratch(device)) return rc;
  }
  ks_ctx* c = new (std::nothrow) ks_ctx();
  if (!c) return KS_E_NOMEM;
  c->device = device;
  c->num_cus = prop.multiProcessorCount;
  c->arch = prop.gcnArchName;
  const size_t colon = c->arch.find(':');
  if (colon != std::string::npos) c->arch.resize(colon);
  load_tune_cache(c);
  *out = c;
  return KS_OK;
}

int ks_ctx_destroy(ks_ctx* ctx) {
  if (!ctx) return KS_E_INVALID;
  {
    DeviceGuard g(ctx->device);
    (void)hipDeviceSynchronize();
    for (auto& kv : ctx->graphs) {
      (void)hipGraphExecDestroy(kv.second.exec);
      (void)hipGraphDestroy(kv.second.graph);
    }
    free_workspace(ctx);
    free_split(ctx);
    free_learn(ctx->learn);
    free_seg(ctx->seg);
  }
  delete ctx;
  return KS_OK;
}

int ks_reserve(ks_ctx* ctx, uint32_t max_series, uint64_t max_total_steps) {
  if (!ctx) return KS_E_INVALID;
  DeviceGuard g(ctx->device);
  if (g.err != hipSuccess) return hip_fail(g.err, "hipSetDevice");
  if (int rc = ensure_workspace(ctx, max_series, max_total_steps)) return rc;
  // and the scan of few series, which does without where the device is full
  const int rc = max_series ? ensure_split(ctx, nullptr) : KS_OK;
  return rc == KS_E_NOMEM ? KS_OK : rc;
}

int ks_scan_batch(ks_ctx* ctx, const uint32_t* samples, uint64_t num_samples, const ks_desc* desc,
                  uint32_t num_series, const ks_params* params, ks_result* out, uint32_t* all_U,
                  uint64_t all_U_len, void* stream) {
  if (!ctx || !params || !out) return KS_E_INVALID;
  if (int rc = check_params(params)) return rc;
  if (num_series == 0) return KS_OK;
  if (!samples || !desc) return KS_E_INVALID;
  if (num_series > (1u << 30)) return KS_E_RANGE;
  DeviceGuard g(ctx->device);
  if (g.err != hipSuccess) return hip_fail(g.err, "hipSetDevice");
  const uint32_t max_K = params->max_K ? params->max_K : KS_MAX_K;
  const int kc = k_class(max_K);
  ScanArgs a{samples, num_samples, desc, num_series, *params, max_K, out, all_U, all_U_len, 0, {}};
  return scan_with(ctx, a, kc, config_for(ctx, kc, a, params->opts), (hipStream_t)stream);
}

int ks_launch_set(ks_ctx* ctx, uint32_t max_K, uint32_t num_series, const ks_launch* cfg) {
  if (!ctx || !cfg) return KS_E_INVALID;
  if (!valid_launch(cfg)) return KS_E_RANGE;
  ctx->tuned[std::make_tuple(k_class(max_K ? max_K : KS_MAX_K), num_series)] = from_launch(cfg);
  return KS_OK;
}

int ks_launch_get(ks_ctx* ctx, uint32_t max_K, uint32_t num_series, ks_launch* cfg) {
  if (!ctx || !cfg) return KS_E_INVALID;
  *cfg = to_launch(recorded(ctx, k_class(max_K ? max_K : KS_MAX_K), num_series));
  return KS_OK;
}

int ks_autotune(ks_ctx* ctx, const uint32_t* samples, uint64_t num_samples, const ks_desc* desc,
                uint32_t num_series, const ks_params* params, ks_result* out, void* stream, ks_launch* best,
                float* best_ms) {
  if (!ctx || !params || !out) return KS_E_INVALID;
  if (int rc = check_params(params)) return rc;
  if (num_series == 0) return KS_OK;
  if (!samples || !desc) return KS_E_INVALID;
  if (num_series > (1u << 30)) return KS_E_RANGE;
  DeviceGuard g(ctx->device);
  if (g.err != hipSuccess) return hip_fail(g.err, "hipSetDevice");
  const uint32_t max_K = params->max_K ? params->max_K : KS_MAX_K;
  const int kc = k_class(max_K);
  hipStream_t st = (hipStream_t)stream;
  ScanArgs a{samples, num_samples, desc, num_series, *params, max_K, out, nullptr, 0, 0, {}};
  hipEvent_t e0, e1;
  hipError_t e;
  if ((e = hipEventCreate(&e0)) != hipSuccess) return hip_fail(e, "hipEventCreate");
  if ((e = hipEventCreate(&e1)) != hipSuccess) {
    (void)hipEventDestroy(e0);
    return hip_fail(e, "hipEventCreate");
  }
  // one warm-up (builds graphs, grows the workspace), then the best of three
  auto time_cfg = [&](const LaunchCfg& cfg, float& tmin) -> int {
    int rc = scan_with(ctx, a, kc, cfg, st);
    for (int r = 0; r < 3 && rc == KS_OK; ++r) {
      if ((e = hipEventRecord(e0, st)) != hipSuccess) return hip_fail(e, "hipEventRecord");
      if ((rc = scan_with(ctx, a, kc, cfg, st)) != KS_OK) return rc;
      if ((e = hipEventRecord(e1, st)) != hipSuccess || (e = hipEventSynchronize(e1)) != hipSuccess)
        return hip_fail(e, "hipEventSynchronize");
      float ms = 0.f;
      (void)hipEventElapsedTime(&ms, e0, e1);
      if (r == 0 || ms < tmin) tmin = ms;
    }
    return rc;
  };
  // every scan-kernel variant (tile, sort radix, walk window) under every
  // launch plan: the plain grid, the ordered grid from a hipGraph (variant 0: the
  // default plan) and direct, the persistent queue with 1 / 4 / 16 MiB splits from a hipGraph and direct
  // (the variants rank differently under different plans)
  int rc = KS_OK;
  LaunchCfg bcfg;
  float bms = 0.f;
  bool have = false;
  for (int v = 0; v < kNumVariants && rc == KS_OK; ++v) {
    LaunchCfg plans[9];
    int np = 0;
    plans[np++] = LaunchCfg{KS_LAUNCH_GRID, 1u << 20, 0, v};
    plans[np++] = LaunchCfg{KS_LAUNCH_ORDERED, 1u << 20, 1, v};
    plans[np++] = LaunchCfg{KS_LAUNCH_ORDERED, 1u << 20, 0, v};
    for (uint32_t chunk : {1u << 20, 4u << 20, 16u << 20}) {
      plans[np++] = LaunchCfg{KS_LAUNCH_PERSISTENT, chunk, 1, v};
      plans[np++] = LaunchCfg{KS_LAUNCH_PERSISTENT, chunk, 0, v};
    }
    for (int i = 0; i < np && rc == KS_OK; ++i) {
      float t = 0.f;
      const LaunchCfg run = is_default(plans[i]) ? default_cfg(ctx, kc, a) : plans[i];
      rc = time_cfg(run, t);
      if (rc == KS_OK && (!have || t < bms)) {
        bcfg = run.spread ? plans[i] : run;  // the scan of few series has no record but the default
        bms = t;
        have = true;
      }
    }
  }
  (void)hipEventDestroy(e0);
  (void)hipEventDestroy(e1);
  if (rc) return rc;
  ctx->tuned[std::make_tuple(kc, num_series)] = bcfg;
  append_tune_cache(ctx, kc, num_series, bcfg);
  if (best) *best = to_launch(bcfg);
  if (best_ms) *best_ms = bms;
  return KS_OK;
}

int ks_scan_batch_noalloc(ks_ctx* ctx, const uint32_t* samples, uint64_t num_samples, const ks_desc* desc,
                          uint32_t num_series, const ks_params* params, ks_result* out, uint32_t* all_U,
                          uint64_t all_U_len, void* stream) {
  if (!ctx || !params || !out) return KS_E_INVALID;
  if (int rc = check_params(params)) return rc;
  if (num_series == 0) return KS_OK;
  if (!samples || !desc) return KS_E_INVALID;
  if (num_series > KS_NOALLOC_MAX_SERIES) return KS_E_RANGE;
  unsigned char* base = scratch_of(ctx->device);
  if (!base) return KS_E_STATE;  // ks_ctx_create resolves it; not reached for a valid context
  DeviceGuard g(ctx->device);
  if (g.err != hipSuccess) return hip_fail(g.err, "hipSetDevice");
  const uint32_t max_K = params->max_K ? params->max_K : KS_MAX_K;
  const int kc = k_class(max_K);
  // the plan kernel rewrites the header, every item and every per-series word
  // it reads later, so nothing is cleared here
  ks::Workspace ws{reinterpret_cast<uint32_t*>(base), reinterpret_cast<ks::Item*>(base + kScratchItems),
                   reinterpret_cast<uint64_t*>(base + kScratchBase), reinterpret_cast<uint32_t*>(base + kScratchDone),
                   reinterpret_cast<uint32_t*>(base + kScratchMin), nullptr};
  ScanArgs a{samples, num_samples, desc, num_series, *params, max_K, out, all_U, all_U_len, ks::kNoSplit, ws};
  return launch_plan(ctx, kc, config_for(ctx, kc, a, 0).variant, KS_LAUNCH_ORDERED, a, false, (hipStream_t)stream);
}

}  // extern "C"
