// C ABI of the learned proposal: model lifecycle and checkpoints, the feature
// pass, network forward, proposal, exact refine and one training step.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <vector>

#include "ks.h"
#include "ks_cnn.hpp"
#include "ks_ctx.hpp"
#include "ks_features.hpp"
#include "ks_refine.hpp"

using namespace ks_host;
namespace C = ks::cnn;

namespace ks_host {

void free_learn(LearnBuffers& b) {
  void* ptrs[] = {b.s1, b.s2lo, b.s2hi, b.smin, b.cmin, b.K, b.feat, b.x0, b.act[0], b.act[1], b.act[2], b.logits,
                  b.dz, b.dy[0], b.dy[1], b.dy[2], b.part, b.bpart,
                  b.nsig};
  for (void* p : ptrs) (void)hipFree(p);
  b = LearnBuffers{};
}

}  // namespace ks_host

namespace {

uint32_t slot_rows(uint32_t max_K) { return (max_K + 4 + 15) / 16 * 16; }

template <typename T>
bool alloc(T*& p, uint64_t n) {
  return hipMalloc(&p, sizeof(T) * (n ? n : 1)) == hipSuccess;
}

// Grow the learned-path buffers for `rows` slot rows and `series` series
// (training buffers too when `train`).
int ensure_learn(ks_ctx* c, uint64_t rows, uint64_t series, bool train) {
  LearnBuffers& b = c->learn;
  const bool have_train = b.dz != nullptr;
  if (rows <= b.cap_rows && series <= b.cap_series && (!train || have_train)) return KS_OK;
  const uint64_t R = rows > b.cap_rows ? rows : b.cap_rows;
  const uint64_t S = series > b.cap_series ? series : b.cap_series;
  const bool T = train || have_train;
  hipError_t e = hipDeviceSynchronize();
  if (e != hipSuccess) return hip_fail(e, "hipDeviceSynchronize");
  free_learn(b);
  bool ok = alloc(b.s1, R) && alloc(b.s2lo, R) && alloc(b.s2hi, R) && alloc(b.smin, S) && alloc(b.cmin, S + ks::kChunkWGs) &&
            alloc(b.K, S) &&
            alloc(b.feat, R * 9) && alloc(b.x0, R * 16) && alloc(b.act[0], R * 64) && alloc(b.act[1], R * 64) &&
            alloc(b.act[2], R * 64) && alloc(b.logits, R);
  if (ok && T) {
    ok = alloc(b.dz, R) && alloc(b.dy[0], R * 64) && alloc(b.dy[1], R * 64) && alloc(b.dy[2], R * 64) &&
         alloc(b.part, (uint64_t)C::kDwGrid * C::kDwPart) &&
         alloc(b.bpart, (uint64_t)C::kDwGrid * C::kBiasPart) && alloc(b.nsig, 4);
  }
  if (!ok) {
    free_learn(b);
    (void)hipGetLastError();
    return KS_E_NOMEM;
  }
  b.cap_rows = R;
  b.cap_series = S;
  return KS_OK;
}

ks::LearnWs learn_ws(ks_ctx* c) {
  return ks::LearnWs{c->learn.s1, c->learn.s2lo, c->learn.s2hi, c->learn.smin, c->learn.cmin, c->learn.K};
}

C::Shadow shadow_of(const ks_model* m) {
  C::Shadow sh;
  for (int l = 0; l < 4; ++l) {
    sh.wf[l] = m->wf[l];
    sh.wb[l] = m->wb[l];
    sh.b[l] = m->b[l];
  }
  return sh;
}

C::ForwardArgs forward_args(ks_ctx* c, const ks_model* m, uint32_t num_series, uint32_t SR, uint32_t max_K) {
  LearnBuffers& b = c->learn;
  C::ForwardArgs A{};
  A.x0 = b.x0;
  A.Ks = b.K;
  A.max_K = max_K;
  A.SR = SR;
  A.num_series = num_series;
  A.tiles_per_series = (max_K + C::FT - 1) / C::FT;
  for (int l = 0; l < 4; ++l) {
    A.w[l] = m->wf[l];
    A.b[l] = m->b[l];
  }
  A.logits = b.logits;
  return A;
}

// Resident workgroups of the fused network kernels, at most one per tile.
uint32_t fused_grid(const ks_ctx* c, uint32_t num_series, uint32_t tiles_per_series) {
  const uint64_t tiles = (uint64_t)num_series * tiles_per_series, cap = (uint64_t)c->num_cus * C::FWGS;
  return (uint32_t)(tiles < cap ? tiles : cap);
}

// The whole network in one launch, activations kept in LDS.
template <bool FEAT, bool TRAIN = false>
hipError_t launch_forward(ks_ctx* c, const C::ForwardArgs& A, hipStream_t st) {
  auto kernel = C::fused_forward_kernel<FEAT, TRAIN>;
  hipLaunchKernelGGL(kernel, dim3(fused_grid(c, A.num_series, A.tiles_per_series)), dim3(C::NTC), 0, st, A);
  return hipGetLastError();
}

// The training forward from the caller's features: activations a1..a3, input
// rows, logits and each series' K kept for the backward pass; with labels their
// count in nsig and *loss cleared.
hipError_t forward_train(ks_ctx* c, const ks_model* m, const float* features, uint64_t feature_rows,
                         const ks_desc* desc, uint32_t num_series, uint32_t max_K, const int32_t* labels, float* loss,
                         hipStream_t st) {
  LearnBuffers& b = c->learn;
  C::ForwardArgs A = forward_args(c, m, num_series, slot_rows(max_K), max_K);
  A.feat = features;
  A.feat_rows = feature_rows;
  A.desc = desc;
  A.keep[0] = b.x0;
  for (int l = 0; l < 3; ++l) A.keep[l + 1] = b.act[l];
  A.labels = labels;
  A.nsig = b.nsig;
  A.loss = loss;
  return launch_forward<true, true>(c, A, st);
}

// Backward pass from the logit gradient in dz, with the activations of the last
// forward_train: the gradients at y2, y1, y0 in dy[0..2] and, into `grads`
// (nullable), the parameters' gradient; with `step` also the Adam step.
hipError_t backward(ks_ctx* c, const ks_model* model, uint32_t num_series, uint32_t max_K, float* grads,
                    const float* step, hipStream_t st) {
  LearnBuffers& b = c->learn;
  const uint32_t SR = slot_rows(max_K);
  C::BackwardArgs A{};
  A.dz = b.dz;
  A.Ks = b.K;
  A.SR = SR;
  A.num_series = num_series;
  A.tiles_per_series = (max_K + C::BT - 1) / C::BT;
  for (int l = 0; l < 3; ++l) {
    A.a[l] = b.act[2 - l];
    A.wb[l] = model->wb[3 - l];
    A.dy[l] = b.dy[l];
  }
  hipLaunchKernelGGL(C::fused_backward_kernel, dim3(fused_grid(c, num_series, A.tiles_per_series)), dim3(C::NTC), 0, st,
                     A);
  if (!grads) return hipGetLastError();
  C::DwArgs D{};
  D.dz = b.dz;
  D.x[0] = b.x0;
  for (int l = 0; l < 3; ++l) {
    D.dy[l] = b.dy[2 - l];
    D.x[l + 1] = b.act[l];
  }
  D.Ks = b.K;
  D.SR = SR;
  D.num_series = num_series;
  D.part = b.part;
  D.bpart = b.bpart;
  const uint64_t tiles = ((uint64_t)num_series * SR + C::DT - 1) / C::DT;
  const uint32_t G = (uint32_t)(tiles < C::kDwGrid ? tiles : C::kDwGrid);
  hipLaunchKernelGGL(C::dw_kernel, dim3(G, 4), dim3(C::NTC), 0, st, D);
  hipLaunchKernelGGL(C::finish_kernel, dim3(C::kFinishGrid), dim3(C::NTC), 0, st, b.part, G, b.bpart, model->theta,
                     model->m1, model->m2, grads, shadow_of(model), step ? step[0] : 0.0f, step ? step[1] : 1.0f,
                     step ? step[2] : 1.0f, step ? 1 : 0);
  return hipGetLastError();
}

template <int KMAX>
void launch_refine(const ks_desc* desc, uint32_t n, uint64_t num_samples, uint32_t max_K, const ks_params& prm,
                   const int32_t* prop, const float* conf, ks::LearnWs lw, uint32_t SR, ks_result* out,
                   hipStream_t st) {
  // K classes of 1024 and 2048 rows in 512-thread workgroups: their LDS, not
  // registers, limits the workgroups per CU, so twice the threads per
  // workgroup doubles the waves walking the fallback series (the learned
  // step on 8192 x 1024 x 2048 0.5% faster)
  constexpr int RNT = KMAX >= 1024 ? 512 : kNT;
  hipLaunchKernelGGL((ks::refine_kernel<KMAX, RNT, kRB>), dim3(n), dim3(RNT), 0, st, desc, n, num_samples, max_K, prm,
                     prop, conf, lw, SR, out);
}

hipError_t shadow(ks_model* m, hipStream_t st) {
  hipLaunchKernelGGL(C::shadow_kernel, dim3((C::kShadowEntries + C::NTC - 1) / C::NTC), dim3(C::NTC), 0, st, m->theta,
                     shadow_of(m));
  return hipGetLastError();
}

void free_model(ks_model* m) {
  void* ptrs[] = {m->theta, m->m1, m->m2, m->grad, m->wf[0], m->wf[1], m->wf[2], m->wf[3],
                  m->wb[1], m->wb[2], m->wb[3], m->b[0], m->b[1], m->b[2], m->b[3]};
  for (void* p : ptrs) (void)hipFree(p);
}

// splitmix64 (Steele, Lea, Flood 2014) for the initial weights
uint64_t splitmix64(uint64_t& s) {
  uint64_t z = (s += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

uint64_t fnv1a(const void* p, size_t n, uint64_t h = 0xcbf29ce484222325ull) {
  const unsigned char* c = static_cast<const unsigned char*>(p);
  for (size_t i = 0; i < n; ++i) h = (h ^ c[i]) * 0x100000001b3ull;
  return h;
}

const char kMagic[8] = {'K', 'S', 'C', 'N', 'N', '0', '0', '1'};

int check_learn_args(const ks_desc* desc, uint32_t num_series, uint32_t max_K) {
  if (!desc && num_series) return KS_E_INVALID;
  if (num_series > (1u << 26)) return KS_E_RANGE;
  if (max_K < 2 || max_K > KS_MAX_K) return KS_E_RANGE;
  return KS_OK;
}

}  // namespace

extern "C" {

int ks_model_create(ks_ctx* ctx, uint64_t seed, ks_model** out) {
  if (!ctx || !out) return KS_E_INVALID;
  *out = nullptr;
  DeviceGuard g(ctx->device);
  if (g.err != hipSuccess) return hip_fail(g.err, "hipSetDevice");
  ks_model* m = new (std::nothrow) ks_model();
  if (!m) return KS_E_NOMEM;
  m->device = ctx->device;
  bool ok = alloc(m->theta, C::kNumParams) && alloc(m->m1, C::kNumParams) && alloc(m->m2, C::kNumParams) &&
            alloc(m->grad, C::kNumParams);
  for (int l = 0; l < 4 && ok; ++l) {
    const C::Layer L = C::layer_info(l);
    ok = alloc(m->wf[l], (uint64_t)L.cout_pad * 5 * L.cin_pad) && alloc(m->b[l], L.cout_pad);
    if (ok && l >= 1) ok = alloc(m->wb[l], (uint64_t)L.cin_pad * 5 * L.cout_pad);
  }
  if (!ok) {
    free_model(m);
    delete m;
    (void)hipGetLastError();
    return KS_E_NOMEM;
  }
  // He-uniform weights U(-a, a), a = sqrt(6 / fan_in), zero biases
  std::vector<float> h(C::kNumParams, 0.0f);
  uint64_t st = seed;
  for (int l = 0; l < 4; ++l) {
    const C::Layer L = C::layer_info(l);
    const double a = std::sqrt(6.0 / (L.cin * 5.0));
    for (uint32_t p = L.w_off; p < L.b_off; ++p) {
      const double u = (double)(splitmix64(st) >> 11) * 0x1p-53;
      h[p] = (float)((2.0 * u - 1.0) * a);
    }
  }
  int rc = ks_model_set_params(m, h.data());
  if (rc) {
    free_model(m);
    delete m;
    return rc;
  }
  *out = m;
  return KS_OK;
}

int ks_model_destroy(ks_model* m) {
  if (!m) return KS_E_INVALID;
  DeviceGuard g(m->device);
  (void)hipDeviceSynchronize();
  free_model(m);
  delete m;
  return KS_OK;
}

int ks_model_set_params(ks_model* m, const float* host) {
  if (!m || !host) return KS_E_INVALID;
  DeviceGuard g(m->device);
  if (g.err != hipSuccess) return hip_fail(g.err, "hipSetDevice");
  for (uint32_t p = 0; p < C::kNumParams; ++p)
    if (!std::isfinite(host[p])) return KS_E_MODEL;
  hipError_t e;
  if ((e = hipMemcpy(m->theta, host, sizeof(float) * C::kNumParams, hipMemcpyHostToDevice)) != hipSuccess ||
      (e = hipMemset(m->m1, 0, sizeof(float) * C::kNumParams)) != hipSuccess ||
      (e = hipMemset(m->m2, 0, sizeof(float) * C::kNumParams)) != hipSuccess ||
      (e = hipMemset(m->grad, 0, sizeof(float) * C::kNumParams)) != hipSuccess)
    return hip_fail(e, "ks_model_set_params");
  if ((e = shadow(m, nullptr)) != hipSuccess || (e = hipDeviceSynchronize()) != hipSuccess)
    return hip_fail(e, "shadow weights");
  m->step = 0;
  return KS_OK;
}

int ks_model_get_params(ks_model* m, float* host) {
  if (!m || !host) return KS_E_INVALID;
  DeviceGuard g(m->device);
  hipError_t e = hipMemcpy(host, m->theta, sizeof(float) * C::kNumParams, hipMemcpyDeviceToHost);
  return e == hipSuccess ? KS_OK : hip_fail(e, "ks_model_get_params");
}

int ks_model_grads(ks_model* m, float* host) {
  if (!m || !host) return KS_E_INVALID;
  DeviceGuard g(m->device);
  hipError_t e = hipMemcpy(host, m->grad, sizeof(float) * C::kNumParams, hipMemcpyDeviceToHost);
  return e == hipSuccess ? KS_OK : hip_fail(e, "ks_model_grads");
}

// File: magic "KSCNN001", u32 parameter count, u64 step, then theta, m1, m2
// (fp32), then the FNV-1a 64 hash of everything before it.
int ks_model_save(ks_model* m, const char* path) {
  if (!m || !path) return KS_E_INVALID;
  DeviceGuard g(m->device);
  std::vector<float> buf(3 * (size_t)C::kNumParams);
  hipError_t e;
  if ((e = hipMemcpy(buf.data(), m->theta, sizeof(float) * C::kNumParams, hipMemcpyDeviceToHost)) != hipSuccess ||
      (e = hipMemcpy(buf.data() + C::kNumParams, m->m1, sizeof(float) * C::kNumParams, hipMemcpyDeviceToHost)) !=
          hipSuccess ||
      (e = hipMemcpy(buf.data() + 2 * C::kNumParams, m->m2, sizeof(float) * C::kNumParams,
                     hipMemcpyDeviceToHost)) != hipSuccess)
    return hip_fail(e, "ks_model_save");
  const uint32_t n = C::kNumParams;
  uint64_t h = fnv1a(kMagic, 8);
  h = fnv1a(&n, 4, h);
  h = fnv1a(&m->step, 8, h);
  h = fnv1a(buf.data(), buf.size() * 4, h);
  FILE* f = std::fopen(path, "wb");
  if (!f) return KS_E_INVALID;
  const bool ok = std::fwrite(kMagic, 1, 8, f) == 8 && std::fwrite(&n, 4, 1, f) == 1 &&
                  std::fwrite(&m->step, 8, 1, f) == 1 && std::fwrite(buf.data(), 4, buf.size(), f) == buf.size() &&
                  std::fwrite(&h, 8, 1, f) == 1;
  return (std::fclose(f) == 0 && ok) ? KS_OK : KS_E_INVALID;
}

int ks_model_load(ks_model* m, const char* path) {
  if (!m || !path) return KS_E_INVALID;
  FILE* f = std::fopen(path, "rb");
  if (!f) return KS_E_INVALID;
  char magic[8];
  uint32_t n = 0;
  uint64_t step = 0, h = 0;
  std::vector<float> buf(3 * (size_t)C::kNumParams);
  const bool ok = std::fread(magic, 1, 8, f) == 8 && std::fread(&n, 4, 1, f) == 1 && n == C::kNumParams &&
                  std::fread(&step, 8, 1, f) == 1 && std::fread(buf.data(), 4, buf.size(), f) == buf.size() &&
                  std::fread(&h, 8, 1, f) == 1;
  std::fclose(f);
  if (!ok || std::memcmp(magic, kMagic, 8) != 0) return KS_E_MODEL;
  uint64_t hh = fnv1a(kMagic, 8);
  hh = fnv1a(&n, 4, hh);
  hh = fnv1a(&step, 8, hh);
  hh = fnv1a(buf.data(), buf.size() * 4, hh);
  if (hh != h) return KS_E_MODEL;
  if (int rc = ks_model_set_params(m, buf.data())) return rc;
  DeviceGuard g(m->device);
  hipError_t e;
  if ((e = hipMemcpy(m->m1, buf.data() + C::kNumParams, sizeof(float) * C::kNumParams, hipMemcpyHostToDevice)) !=
          hipSuccess ||
      (e = hipMemcpy(m->m2, buf.data() + 2 * C::kNumParams, sizeof(float) * C::kNumParams,
                     hipMemcpyHostToDevice)) != hipSuccess)
    return hip_fail(e, "ks_model_load");
  m->step = step;
  return KS_OK;
}

int ks_learn_reserve(ks_ctx* ctx, uint32_t max_series, uint32_t max_K, int train) {
  if (!ctx) return KS_E_INVALID;
  if (max_K == 0) max_K = KS_MAX_K;
  if (int rc = check_learn_args(nullptr, 0, max_K)) return rc;
  if (max_series > (1u << 26)) return KS_E_RANGE;
  if (max_series == 0) return KS_OK;
  DeviceGuard g(ctx->device);
  if (g.err != hipSuccess) return hip_fail(g.err, "hipSetDevice");
  return ensure_learn(ctx, (uint64_t)max_series * slot_rows(max_K), max_series, train != 0);
}

int ks_features(ks_ctx* ctx, const uint32_t* samples, uint64_t num_samples, const ks_desc* desc,
                uint32_t num_series, uint32_t max_K, float* features, uint64_t feature_rows, void* stream) {
  if (!ctx) return KS_E_INVALID;
  if (max_K == 0) max_K = KS_MAX_K;
  if (int rc = check_learn_args(desc, num_series, max_K)) return rc;
  if (num_series == 0) return KS_OK;
  if (!samples) return KS_E_INVALID;
  DeviceGuard g(ctx->device);
  if (g.err != hipSuccess) return hip_fail(g.err, "hipSetDevice");
  const uint32_t SR = slot_rows(max_K);
  if (int rc = ensure_learn(ctx, (uint64_t)num_series * SR, num_series, false)) return rc;
  hipStream_t st = (hipStream_t)stream;
  LearnBuffers& b = ctx->learn;
  const bool one = num_series <= ks::kRowPassOneLaunch;
  uint32_t Cs = 1;  // most chunks that a launch below makes of a series
  for (uint32_t mask : {ks::kRowsOne, ks::kRowsMid, ks::kRowsAll})
    if ((mask == ks::kRowsAll) == one) Cs = std::max(Cs, ks::row_pass_chunks((uint32_t)ctx->num_cus, num_series, max_K, num_samples, mask));
  auto launch = [&](auto kernel, uint32_t mask, const uint32_t* plan) {
    const uint32_t C = ks::row_pass_chunks((uint32_t)ctx->num_cus, num_series, max_K, num_samples, mask);
    hipLaunchKernelGGL(kernel, dim3(num_series * C), dim3(ks::row_pass_threads(mask)), 0, st, samples, num_samples, desc,
                       num_series, max_K, SR, learn_ws(ctx), b.feat, plan, C, Cs);
  };
  if (one) {
    launch(ks::features_kernel<ks::kRowsAll>, ks::kRowsAll, nullptr);
  } else {
    // the series order per row class, kept in the logits buffer (num_series +
    // 10 words <= its rows; nothing reads the logits before the forward
    // rewrites them)
    uint32_t* plan = reinterpret_cast<uint32_t*>(b.logits);
    hipLaunchKernelGGL(ks::feature_plan_kernel, dim3(1), dim3(ks::kFeatPlanNT), 0, st, desc, num_series, num_samples,
                       max_K, plan);
    launch(ks::features_kernel<ks::kRowsOne>, ks::kRowsOne, plan);
    launch(ks::features_kernel<ks::kRowsMid>, ks::kRowsMid, plan);
  }
  hipLaunchKernelGGL((ks::feature_pack_kernel<kNT>), dim3(num_series, (SR + kNT - 1) / kNT), dim3(kNT), 0, st, desc,
                     num_series, features, feature_rows, b.x0, SR, learn_ws(ctx), b.feat, Cs);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "features launch");
  b.stamp_desc = desc;
  b.stamp_series = num_series;
  b.stamp_SR = SR;
  b.stamp_maxK = max_K;
  b.stamp_valid = true;
  return KS_OK;
}

int ks_cnn_forward(ks_ctx* ctx, const ks_model* model, const float* features, uint64_t feature_rows,
                   const ks_desc* desc, uint32_t num_series, uint32_t max_K, float* logits, uint64_t logit_rows,
                   void* stream) {
  if (!ctx || !model) return KS_E_INVALID;
  if (max_K == 0) max_K = KS_MAX_K;
  if (int rc = check_learn_args(desc, num_series, max_K)) return rc;
  if (num_series == 0) return KS_OK;
  if (!features || !logits) return KS_E_INVALID;
  DeviceGuard g(ctx->device);
  if (g.err != hipSuccess) return hip_fail(g.err, "hipSetDevice");
  ctx->learn.stamp_valid = false;  // a refine after this call needs its own proposal pass
  C::ForwardArgs A = forward_args(ctx, model, num_series, slot_rows(max_K), max_K);
  A.feat = features;
  A.feat_rows = feature_rows;
  A.desc = desc;
  A.out = logits;
  A.out_rows = logit_rows;
  const hipError_t e = launch_forward<true>(ctx, A, (hipStream_t)stream);
  return e == hipSuccess ? KS_OK : hip_fail(e, "cnn forward");
}

int ks_propose(ks_ctx* ctx, const ks_model* model, const uint32_t* samples, uint64_t num_samples,
               const ks_desc* desc, uint32_t num_series, const ks_params* params, int32_t* proposal,
               float* confidence, float* features, uint64_t feature_rows, void* stream) {
  if (!ctx || !params) return KS_E_INVALID;
  if (int rc = check_params(params)) return rc;
  if (num_series == 0) return KS_OK;
  if (!proposal || !confidence) return KS_E_INVALID;
  const uint32_t max_K = params->max_K ? params->max_K : KS_MAX_K;
  if (int rc = ks_features(ctx, samples, num_samples, desc, num_series, max_K, features, feature_rows, stream))
    return rc;
  DeviceGuard g(ctx->device);
  hipStream_t st = (hipStream_t)stream;
  LearnBuffers& b = ctx->learn;
  const uint32_t SR = b.stamp_SR;
  const uint32_t per = C::NTC / 64;
  if (!model) {  // the method without the network: the largest jump of the per-row median
    hipLaunchKernelGGL(C::median_jump_kernel, dim3((num_series + per - 1) / per), dim3(C::NTC), 0, st, b.feat,
                       num_series, SR, b.K, proposal, confidence);
    hipError_t e = hipGetLastError();
    return e == hipSuccess ? KS_OK : hip_fail(e, "propose");
  }
  hipError_t e = launch_forward<false>(ctx, forward_args(ctx, model, num_series, SR, max_K), st);
  if (e == hipSuccess) {
    hipLaunchKernelGGL(C::softmax_kernel, dim3((num_series + per - 1) / per), dim3(C::NTC), 0, st, b.logits,
                       num_series, SR, b.K, (const int32_t*)nullptr, (const uint32_t*)nullptr, (float*)nullptr,
                       (float*)nullptr, params->w, proposal, confidence);
    e = hipGetLastError();
  }
  return e == hipSuccess ? KS_OK : hip_fail(e, "propose");
}

int ks_refine(ks_ctx* ctx, const ks_desc* desc, uint32_t num_series, uint64_t num_samples, const int32_t* proposal,
              const float* confidence, const ks_params* params, ks_result* out, void* stream) {
  if (!ctx || !params || !out) return KS_E_INVALID;
  if (int rc = check_params(params)) return rc;
  if (num_series == 0) return KS_OK;
  if (!desc || !proposal || !confidence) return KS_E_INVALID;
  const uint32_t max_K = params->max_K ? params->max_K : KS_MAX_K;
  LearnBuffers& b = ctx->learn;
  if (!b.stamp_valid || b.stamp_desc != desc || b.stamp_series != num_series || b.stamp_maxK != max_K)
    return KS_E_STATE;
  DeviceGuard g(ctx->device);
  if (g.err != hipSuccess) return hip_fail(g.err, "hipSetDevice");
  hipStream_t st = (hipStream_t)stream;
  const ks::LearnWs lw = learn_ws(ctx);
  switch (k_class(max_K)) {
    case 0: launch_refine<64>(desc, num_series, num_samples, max_K, *params, proposal, confidence, lw, b.stamp_SR, out, st); break;
    case 1: launch_refine<128>(desc, num_series, num_samples, max_K, *params, proposal, confidence, lw, b.stamp_SR, out, st); break;
    case 2: launch_refine<256>(desc, num_series, num_samples, max_K, *params, proposal, confidence, lw, b.stamp_SR, out, st); break;
    case 3: launch_refine<512>(desc, num_series, num_samples, max_K, *params, proposal, confidence, lw, b.stamp_SR, out, st); break;
    case 4: launch_refine<1024>(desc, num_series, num_samples, max_K, *params, proposal, confidence, lw, b.stamp_SR, out, st); break;
    default: launch_refine<2048>(desc, num_series, num_samples, max_K, *params, proposal, confidence, lw, b.stamp_SR, out, st);
  }
  hipError_t e = hipGetLastError();
  return e == hipSuccess ? KS_OK : hip_fail(e, "refine launch");
}

int ks_train_step(ks_ctx* ctx, ks_model* model, const float* features, uint64_t feature_rows, const ks_desc* desc,
                  const int32_t* labels, uint32_t num_series, uint32_t max_K, float lr, float* loss, void* stream) {
  if (!ctx || !model) return KS_E_INVALID;
  if (max_K == 0) max_K = KS_MAX_K;
  if (int rc = check_learn_args(desc, num_series, max_K)) return rc;
  if (num_series == 0) return KS_OK;
  if (!features || !labels || !(lr >= 0.0f) || !std::isfinite(lr)) return KS_E_INVALID;
  DeviceGuard g(ctx->device);
  if (g.err != hipSuccess) return hip_fail(g.err, "hipSetDevice");
  const uint32_t SR = slot_rows(max_K);
  const uint64_t rows = (uint64_t)num_series * SR;
  if (int rc = ensure_learn(ctx, rows, num_series, true)) return rc;
  hipStream_t st = (hipStream_t)stream;
  LearnBuffers& b = ctx->learn;
  b.stamp_valid = false;
  float* loss_acc = loss ? loss : reinterpret_cast<float*>(b.nsig + 1);  // discarded when the caller wants no loss
  hipError_t e = forward_train(ctx, model, features, feature_rows, desc, num_series, max_K, labels, loss_acc, st);
  if (e != hipSuccess) return hip_fail(e, "train forward");
  // loss and logit gradient
  const uint32_t per = C::NTC / 64;
  hipLaunchKernelGGL(C::softmax_kernel, dim3((num_series + per - 1) / per), dim3(C::NTC), 0, st, b.logits, num_series,
                     SR, b.K, labels, b.nsig, loss_acc, b.dz, 0u, (int32_t*)nullptr, (float*)nullptr);
  // gradients and Adam
  model->step += 1;
  const float step[3] = {lr, (float)(1.0 - std::pow(0.9, (double)model->step)),
                         (float)(1.0 - std::pow(0.999, (double)model->step))};
  e = backward(ctx, model, num_series, max_K, model->grad, step, st);
  return e == hipSuccess ? KS_OK : hip_fail(e, "train step");
}

int ks_cnn_backward(ks_ctx* ctx, const ks_model* model, const float* features, uint64_t feature_rows,
                    const ks_desc* desc, uint32_t num_series, uint32_t max_K, const float* dlogits,
                    uint64_t dlogit_rows, float* grads, void* stream) {
  if (!ctx || !model) return KS_E_INVALID;
  if (max_K == 0) max_K = KS_MAX_K;
  if (int rc = check_learn_args(desc, num_series, max_K)) return rc;
  if (!grads) return KS_E_INVALID;
  if (num_series && (!features || !dlogits)) return KS_E_INVALID;
  DeviceGuard g(ctx->device);
  if (g.err != hipSuccess) return hip_fail(g.err, "hipSetDevice");
  hipStream_t st = (hipStream_t)stream;
  const uint32_t SR = slot_rows(max_K);
  const uint64_t rows = (uint64_t)(num_series ? num_series : 1) * SR;
  if (int rc = ensure_learn(ctx, rows, num_series ? num_series : 1, true)) return rc;
  LearnBuffers& b = ctx->learn;
  b.stamp_valid = false;
  hipError_t e;
  if (num_series == 0) {  // an empty batch has a zero gradient
    hipLaunchKernelGGL(C::zero_kernel, dim3((C::kNumParams + C::NTC - 1) / C::NTC), dim3(C::NTC), 0, st, grads,
                       C::kNumParams);
    e = hipGetLastError();
    return e == hipSuccess ? KS_OK : hip_fail(e, "gradient reset");
  }
  if ((e = forward_train(ctx, model, features, feature_rows, desc, num_series, max_K, nullptr, nullptr, st)) != hipSuccess)
    return hip_fail(e, "backward: forward");
  hipLaunchKernelGGL(C::pack_dlogits_kernel, dim3(num_series), dim3(C::NTC), 0, st, dlogits, dlogit_rows, desc,
                     num_series, SR, b.K, b.dz);
  e = backward(ctx, model, num_series, max_K, grads, nullptr, st);
  return e == hipSuccess ? KS_OK : hip_fail(e, "backward");
}

int ks_cnn_trace(ks_ctx* ctx, const ks_model* model, const float* features, uint64_t feature_rows,
                 const ks_desc* desc, uint32_t num_series, uint32_t max_K, const int32_t* labels,
                 const float* dlogits, uint64_t dlogit_rows, float* acts, float* grads_in, uint64_t trace_rows,
                 float* grads, void* stream) {
  if (!ctx || !model) return KS_E_INVALID;
  if (max_K == 0) max_K = KS_MAX_K;
  if (int rc = check_learn_args(desc, num_series, max_K)) return rc;
  if (num_series == 0) return KS_OK;
  if (!features) return KS_E_INVALID;
  const bool bwd = labels || dlogits;
  if ((grads_in || grads) && !bwd) return KS_E_INVALID;
  DeviceGuard g(ctx->device);
  if (g.err != hipSuccess) return hip_fail(g.err, "hipSetDevice");
  hipStream_t st = (hipStream_t)stream;
  const uint32_t SR = slot_rows(max_K);
  const uint64_t rows = (uint64_t)num_series * SR;
  if (int rc = ensure_learn(ctx, rows, num_series, true)) return rc;
  LearnBuffers& b = ctx->learn;
  b.stamp_valid = false;
  float* loss_acc = reinterpret_cast<float*>(b.nsig + 1);  // the training step's loss goes to a scratch word
  hipError_t e = forward_train(ctx, model, features, feature_rows, desc, num_series, max_K, labels, loss_acc, st);
  if (e != hipSuccess) return hip_fail(e, "trace forward");
  if (labels) {  // the training step's logit gradient
    const uint32_t per = C::NTC / 64;
    hipLaunchKernelGGL(C::softmax_kernel, dim3((num_series + per - 1) / per), dim3(C::NTC), 0, st, b.logits,
                       num_series, SR, b.K, labels, b.nsig, loss_acc, b.dz, 0u, (int32_t*)nullptr, (float*)nullptr);
  } else if (dlogits) {
    hipLaunchKernelGGL(C::pack_dlogits_kernel, dim3(num_series), dim3(C::NTC), 0, st, dlogits, dlogit_rows, desc,
                       num_series, SR, b.K, b.dz);
  }
  if (bwd && (e = backward(ctx, model, num_series, max_K, grads, nullptr, st)) != hipSuccess)
    return hip_fail(e, "trace backward");
  if (acts || grads_in)
    hipLaunchKernelGGL(C::trace_copy_kernel, dim3(num_series), dim3(C::NTC), 0, st, desc, num_series, SR, b.K, b.x0,
                       b.act[0], b.act[1], b.act[2], b.logits, b.dz, bwd ? b.dy[0] : nullptr, b.dy[1], b.dy[2],
                       acts, grads_in, trace_rows);
  e = hipGetLastError();
  return e == hipSuccess ? KS_OK : hip_fail(e, "trace");
}

}  // extern "C"
