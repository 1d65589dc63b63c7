// mkf_capi.hip -- host runtime behind the C ABI declared in include/mkf.h:
// argument validation, device buffers owned by the context, stream
// ordering, and the drivers of the two find forms.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <exception>
#include <mutex>
#include <new>
#include <string>
#include <thread>
#include <vector>

#include "../../include/mkf.h"
#include "mkf_kernels.hpp"

using namespace mkf;

namespace {

// grow-only device buffer
struct DevBuf {
  void *ptr = nullptr;
  size_t bytes = 0;
  hipError_t ensure(size_t n) {
    if (n <= bytes && ptr) return hipSuccess;
    if (ptr) {
      hipError_t e = hipFree(ptr);
      if (e != hipSuccess) return e;
      ptr = nullptr;
      bytes = 0;
    }
    size_t alloc = n ? n : 256;
    hipError_t e = hipMalloc(&ptr, alloc);
    if (e == hipSuccess) bytes = alloc;
    return e;
  }
  void release() {
    if (ptr) (void)hipFree(ptr);
    ptr = nullptr;
    bytes = 0;
  }
  template <class T> T *as() const { return static_cast<T *>(ptr); }
};

// mkf_get_tracks: records per pinned slot (4.8 MB), and the slots, each
// emptied by a host thread of its own.  A copy into fresh pages of the caller's
// array runs at 10 GB/s on one thread, the device writes the records at 46
// GB/s, so about five threads keep up with it; eight leave room.  500,000
// records (146 MB): 67 ms when the host assembled them from the result rows,
// 3.6 ms now, 2.6 ms of it the link's copy rate (57 GB/s).
constexpr int64_t kCopyRecords = 16384;
constexpr int kCopyThreads = 8;
constexpr int kCopyParts = 4;  // of a call that needs one slot (at most kCopyThreads)
// A slot is pinned when it is first used and kept; the first one has a smaller
// size for small events, since pinning and first touching 4.8 MB takes 100 us.
// (With an allocation of exactly what a call needs, 64 calls of 250 to 16,000
// records pinned 64 times, 85 ms in all instead of 8.)
constexpr int64_t kFewRecords = 1024;

// The calling thread's device while a context's own is needed; the caller's
// again afterwards.
struct DeviceScope {
  int before = -1;
  hipError_t enter(int device) {
    int d = -1;
    hipError_t e = hipGetDevice(&d);
    if (e != hipSuccess || d == device) return e;
    e = hipSetDevice(device);
    if (e == hipSuccess) before = d;
    return e;
  }
  ~DeviceScope() {
    if (before >= 0) (void)hipSetDevice(before);
  }
};

enum Stage { kCreated = 0, kGeometry = 1, kHits = 2, kSeeds = 3, kFound = 4 };

}  // namespace

// Scratch of mkf_surrogate_grad_noalloc, for callers that cannot allocate:
// the per-wave partial gradient rows of up to kNoAllocMaxSamples samples,
// their first-level sums and the per-sample weights.  Each GPU holds one
// copy (5.5 MB) for the life of the process; host code reaches it only
// through the address hipGetSymbolAddress gives on that device.
constexpr int kNoAllocMaxSamples = MKF_NOALLOC_MAX_SAMPLES;
constexpr int kNoAllocMaxWaves = kNoAllocMaxSamples / 64;
constexpr size_t kNoAllocPartial = (size_t)kNoAllocMaxWaves * (kNParam + 1);
constexpr size_t kNoAllocPartial2 = (size_t)(kNoAllocMaxWaves / kReduceGroup + 1) * (kNParam + 1);
constexpr size_t kNoAllocFloats = kNoAllocPartial + kNoAllocPartial2 + kNoAllocMaxSamples;
static __device__ __align__(256) float scratch[kNoAllocFloats];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
float *g_scratch[kMaxDevices] = {};  // device address of scratch, per device

// Resolves scratch's device address on the current device, once per device.
hipError_t resolve_scratch(int dev) {
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch[dev]) return hipSuccess;
  void *ptr = nullptr;
  hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
  if (e != hipSuccess) return e;
  g_scratch[dev] = static_cast<float *>(ptr);
  return hipSuccess;
}

float *scratch_on(int dev) {
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  return dev >= 0 && dev < kMaxDevices ? g_scratch[dev] : nullptr;
}

}  // namespace

struct mkf_ctx {
  mkf_config cfg{};
  hipStream_t stream = nullptr;
  std::string err;
  int stage = kCreated;

  int n_layers = 0;
  mkf_layer user_layers[kMaxLayers]{};  // as loaded (bin counts before the tuning's shifts)
  DevLayer layers[kMaxLayers]{};
  int bins_per_event = 0;
  DevBuf d_layers;
  int n_regions = 0;  // region steering (0: plans from each seed's helix)
  DevBuf d_regions;
  DevMat mat{};       // material map (mat.tab == nullptr: constant angle)
  DevBuf d_mat;
  DevField field{};   // parameterised field (field.on == 0: uniform bz)

  // hits
  int n_events = 0;
  int64_t n_hits = 0;
  std::vector<int64_t> ev_off;
  DevBuf d_ev_off, d_x, d_y, d_z, d_vu, d_vv, d_layer;  // (the arrays: host inputs on their way)
  DevBuf d_bin_rank, d_counts, d_bin_start, d_scan_tmp, d_sorted, d_byorig, d_raw;

  // seeds
  int64_t n_seeds = 0;
  DevBuf d_seed_event, d_seed_hits, d_seed_state, d_seed_ok, d_plan_len, d_plan;
  DevBuf d_seed_chi2, d_seed_fit;
  DevBuf d_cell_counts, d_cell_start, d_cell_rank;  // the processing order's counting sort
  DevBuf d_order, d_pos, d_pstate, d_pinfo, d_pevent, d_pplan;
  DevBuf d_bf_tmp;  // backward fit: state between its FP64 and FP32 parts
  DevBuf d_sm_wk, d_sm_n;  // smoothing: forward-pass states per surface, surface counts
  // triplet seeding: counts (with cursors), offsets, scan scratch, kept triplets
  DevBuf d_tr_cnt, d_tr_off, d_tr_tmp, d_tr_kept, d_tr_at;
  DevBuf d_dup_h, d_dup_n, d_dup_cnt, d_dup_off, d_dup_fill, d_dup_list, d_dup_tmp, d_dup_total;
  DevBuf d_clean_key;  // seed cleaning: what a pair of seeds is compared by
  std::vector<int64_t> active_at_step;  // seeds (in processing order) with plan_len > step
  int max_plan_len = 0;
  int64_t n_seeds_ok = 0;

  // find
  DevBuf d_cand, d_fin_key, d_fin_rec, d_fin_meta, d_bp;
  DevBuf d_out;  // result rows (kOut*), n_seeds words each
  hipEvent_t ev_a = nullptr, ev_b = nullptr, ev_m0 = nullptr, ev_m1 = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t graph_exec = nullptr;
  int graph_launches = 0;
  mkf_stats stats{};
  // pinned host words the find's step count and counters are read back
  // into: [0] steps, then kCounters x kCounterSlots
  unsigned long long *h_cnt = nullptr;
  int *h_len = nullptr;  // pinned: the seeds' counts by plan length; other counts read back
  int *h_bad = nullptr;  // pinned: set by the device where an input is out of range
  // pinned slots that the track records pass through on their way to the
  // caller (mkf_get_tracks), and an event for each
  mkf_track *h_slot[kCopyThreads] = {};
  int64_t h_slot0_n = 0;  // records of the first; the others hold kCopyRecords
  hipEvent_t ev_copy[kCopyThreads] = {};
  int n_cu = 0;
  int device = 0;  // the device current at mkf_create
  std::string arch;
  mkf_tuning tuning{2, 8, 0, 0, 0};
  bool tuned = false;  // a launch shape was set: it is used as it is

  // learned surrogate: master weights, Adam moments, BF16 images, counters
  DevBuf d_mlp_param, d_mlp_m, d_mlp_v, d_W1p, d_W2p, d_W3p, d_W2T, d_W3T, d_mb1, d_mb2, d_mb3;
  DevBuf d_cnt, d_radii, d_tx, d_tt, d_tvalid, d_partial, d_partial2, d_loss, d_grad;
  int mlp_step = 0;  // Adam steps taken

  // fit scratch (host-side inputs are staged here)
  ~mkf_ctx() {
    DevBuf *all[] = {&d_layers, &d_regions, &d_mat, &d_ev_off, &d_x, &d_y, &d_z, &d_vu, &d_vv,
                     &d_layer, &d_bin_rank, &d_counts, &d_bin_start, &d_scan_tmp, &d_sorted,
                     &d_byorig, &d_raw, &d_seed_event, &d_seed_hits, &d_seed_state, &d_seed_ok,
                     &d_plan_len, &d_plan, &d_cell_counts, &d_cell_start, &d_cell_rank,
                     &d_order, &d_pos, &d_pstate, &d_pinfo, &d_pevent, &d_pplan, &d_cand, &d_fin_key, &d_fin_rec, &d_fin_meta,
                     &d_bp, &d_out, &d_mlp_param, &d_mlp_m, &d_mlp_v, &d_W1p,
                     &d_W2p, &d_W3p, &d_W2T, &d_W3T, &d_mb1, &d_mb2, &d_mb3, &d_cnt, &d_radii,
                     &d_tx, &d_tt, &d_tvalid, &d_partial, &d_partial2, &d_loss, &d_grad,
                     &d_bf_tmp, &d_sm_wk, &d_sm_n, &d_tr_cnt, &d_tr_off, &d_tr_tmp, &d_tr_kept,
                     &d_tr_at, &d_dup_h, &d_dup_n, &d_dup_cnt, &d_dup_off, &d_dup_fill,
                     &d_dup_list, &d_dup_tmp, &d_dup_total, &d_clean_key, &d_seed_chi2,
                     &d_seed_fit};
    for (DevBuf *b : all) b->release();
    if (graph_exec) (void)hipGraphExecDestroy(graph_exec);
    if (graph) (void)hipGraphDestroy(graph);
    if (ev_a) (void)hipEventDestroy(ev_a);
    if (ev_b) (void)hipEventDestroy(ev_b);
    if (ev_m0) (void)hipEventDestroy(ev_m0);
    if (ev_m1) (void)hipEventDestroy(ev_m1);
    if (h_cnt) (void)hipHostFree(h_cnt);  // (h_len and h_bad lie behind it)
    for (mkf_track *slot : h_slot)
      if (slot) (void)hipHostFree(slot);
    for (hipEvent_t e : ev_copy)
      if (e) (void)hipEventDestroy(e);
  }
};

namespace {

std::string g_create_error = "no error";

mkf_status fail(mkf_ctx *c, mkf_status st, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  if (c) c->err = buf;
  else g_create_error = buf;
  return st;
}

#define HIP_TRY(c, expr)                                                                 \
  do {                                                                                   \
    hipError_t e_ = (expr);                                                              \
    if (e_ != hipSuccess)                                                                \
      return fail((c), MKF_E_HIP, "%s failed: %s", #expr, hipGetErrorString(e_));         \
  } while (0)

DevCfg dev_cfg(const mkf_config &c) {
  DevCfg d{};
  d.mkb = -c.kappa * c.bz;
  d.chi2_cut = c.chi2_cut;
  d.ms_var = c.ms_sigma * c.ms_sigma;
  d.edge_margin = c.edge_margin;
  d.l_min = c.l_min;
  d.n_cand = c.n_cand;
  d.max_holes = c.max_holes;
  for (int i = 0; i < 6; ++i) d.init_var[i] = c.init_var[i];
  return d;
}

bool has_stereo(const mkf_ctx *c) {
  for (int i = 0; i < c->n_layers; ++i)
    if (c->user_layers[i].stereo != 0.f) return true;
  return false;
}

FindParams params(mkf_ctx *c) {
  FindParams P{};
  P.layers = c->d_layers.as<DevLayer>();
  P.n_layers = c->n_layers;
  P.cfg = dev_cfg(c->cfg);
  P.cfg.mat = c->mat;
  P.cfg.field = c->field;
  P.n_events = c->n_events;
  P.ev_off = c->d_ev_off.as<int64_t>();
  P.raw = has_stereo(c) ? c->d_raw.as<float2>() : nullptr;
  P.sorted = c->d_sorted.as<HitRec>();
  P.byorig = c->d_byorig.as<HitRec>();
  P.bin_start = c->d_bin_start.as<int>();
  P.bins_per_event = c->bins_per_event;
  P.n_seeds = c->n_seeds;
  P.seed_event = c->d_seed_event.as<int>();
  P.seed_state = c->d_seed_state.as<float>();
  P.seed_ok = c->d_seed_ok.as<int>();
  P.plan_len = c->d_plan_len.as<int>();
  P.plan = c->d_plan.as<int8_t>();
  P.order = c->d_order.as<int>();
  P.pstate = c->d_pstate.as<float>();
  P.pinfo = c->d_pinfo.as<int>();
  P.pevent = c->d_pevent.as<int>();
  P.pplan = c->d_pplan.as<int8_t>();
  P.out = c->d_out.as<float>();
  // the layer-synchronous form's lane groups: 6 lanes hold budgets up to 6
  P.slots = c->cfg.n_cand <= 6 ? 6 : 8;
  P.cand = c->d_cand.as<float>();
  P.fin_key = c->d_fin_key.as<unsigned long long>();
  P.fin_rec = c->d_fin_rec.as<float>();
  P.fin_meta = c->d_fin_meta.as<int>();
  P.bp = c->d_bp.as<int>();
  // one allocation, cleared by one fill: step count, counters, tile counters
  unsigned long long *clear = c->d_cnt.as<unsigned long long>();
  P.tile_counter = reinterpret_cast<int *>(clear + kTileWord0);
  P.max_plan = c->max_plan_len;
  P.n_steps = clear;
  P.mlp = MlpWeights{c->d_W1p.as<__bf16>(), c->d_W2p.as<__bf16>(), c->d_W3p.as<__bf16>(),
                     c->d_W2T.as<__bf16>(), c->d_W3T.as<__bf16>(), c->d_mb1.as<float>(),
                     c->d_mb2.as<float>(), c->d_mb3.as<float>()};
  P.counters = clear + 1;
  return P;
}

bool finite_f(float v) { return std::isfinite(v); }

MlpBuffers mlp_buffers(mkf_ctx *c) {
  MlpBuffers B{};
  B.param = c->d_mlp_param.as<float>();
  B.m = c->d_mlp_m.as<float>();
  B.v = c->d_mlp_v.as<float>();
  B.W1p = c->d_W1p.as<__bf16>();
  B.W2p = c->d_W2p.as<__bf16>();
  B.W3p = c->d_W3p.as<__bf16>();
  B.W2T = c->d_W2T.as<__bf16>();
  B.W3T = c->d_W3T.as<__bf16>();
  B.b1 = c->d_mb1.as<float>();
  B.b2 = c->d_mb2.as<float>();
  B.b3 = c->d_mb3.as<float>();
  return B;
}

// Surrogate buffers and the initial weights: Glorot-uniform from a fixed
// seed (reproducible), zero biases and Adam moments, zero image padding.
hipError_t mlp_setup(mkf_ctx *c) {
  const size_t bf = sizeof(__bf16);
  hipError_t e = hipSuccess;
  DevBuf *f32[] = {&c->d_mlp_param, &c->d_mlp_m, &c->d_mlp_v};
  for (DevBuf *b : f32)
    if (e == hipSuccess) e = b->ensure(sizeof(float) * kNParam);
  if (e == hipSuccess) e = c->d_W1p.ensure(bf * 64 * kLdW1);
  if (e == hipSuccess) e = c->d_W2p.ensure(bf * 64 * kLdW2);
  if (e == hipSuccess) e = c->d_W3p.ensure(bf * 32 * kLdW3);
  if (e == hipSuccess) e = c->d_W2T.ensure(bf * 64 * kLdW2);
  if (e == hipSuccess) e = c->d_W3T.ensure(bf * 64 * kLdW3T);
  if (e == hipSuccess) e = c->d_mb1.ensure(sizeof(float) * 64);
  if (e == hipSuccess) e = c->d_mb2.ensure(sizeof(float) * 64);
  if (e == hipSuccess) e = c->d_mb3.ensure(sizeof(float) * 32);
  if (e == hipSuccess) e = c->d_cnt.ensure(sizeof(unsigned long long) * kClearWords);
  if (e != hipSuccess) return e;
  DevBuf *zero[] = {&c->d_mlp_m, &c->d_mlp_v, &c->d_W1p, &c->d_W2p, &c->d_W3p, &c->d_W2T,
                    &c->d_W3T, &c->d_mb1, &c->d_mb2, &c->d_mb3, &c->d_cnt};
  for (DevBuf *b : zero)
    if (e == hipSuccess) e = hipMemsetAsync(b->ptr, 0, b->bytes, c->stream);
  std::vector<float> p(kNParam, 0.f);
  uint64_t st = 0x5EEDF00Dull;
  auto uni = [&]() {  // SplitMix64 stream
    st += 0x9E3779B97F4A7C15ull;
    uint64_t z = st;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    return (double)(z >> 11) * (1.0 / 9007199254740992.0);
  };
  auto fill = [&](int off, int fan_out, int fan_in) {
    const double a = std::sqrt(6.0 / (fan_in + fan_out));
    for (int i = 0; i < fan_out * fan_in; ++i) p[off + i] = (float)((2.0 * uni() - 1.0) * a);
  };
  fill(kOffW1, kNH, kNI);
  fill(kOffW2, kNH, kNH);
  fill(kOffW3, kNO, kNH);
  if (e == hipSuccess)
    e = hipMemcpyAsync(c->d_mlp_param.ptr, p.data(), sizeof(float) * kNParam,
                       hipMemcpyHostToDevice, c->stream);
  if (e == hipSuccess) {
    launch_mlp_images(c->stream, mlp_buffers(c));
    e = hipGetLastError();
  }
  if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
  c->mlp_step = 0;
  return e;
}

void drop_graph(mkf_ctx *c) {
  if (c->graph_exec) (void)hipGraphExecDestroy(c->graph_exec);
  if (c->graph) (void)hipGraphDestroy(c->graph);
  c->graph_exec = nullptr;
  c->graph = nullptr;
}

// copy a caller array (host or device) into a context buffer
mkf_status stage_in(mkf_ctx *c, DevBuf &dst, const void *src, size_t bytes, int mem) {
  HIP_TRY(c, dst.ensure(bytes));
  if (bytes == 0) return MKF_OK;
  HIP_TRY(c, hipMemcpyAsync(dst.ptr, src, bytes,
                            mem == MKF_MEM_DEVICE ? hipMemcpyDeviceToDevice
                                                  : hipMemcpyHostToDevice,
                            c->stream));
  return MKF_OK;
}

}  // namespace

extern "C" {

mkf_status mkf_create(const mkf_config *cfg, void *stream, mkf_ctx **out) {
  if (!out) return fail(nullptr, MKF_E_ARG, "out is NULL");
  *out = nullptr;
  if (!cfg) return fail(nullptr, MKF_E_ARG, "cfg is NULL");
  if (!(cfg->n_cand >= 1 && cfg->n_cand <= MKF_MAX_CAND))
    return fail(nullptr, MKF_E_ARG, "n_cand must be in 1..%d", MKF_MAX_CAND);
  if (cfg->max_holes < 0 || cfg->max_holes > 32)
    return fail(nullptr, MKF_E_ARG, "max_holes must be in 0..32");
  const float fv[] = {cfg->bz, cfg->kappa, cfg->chi2_cut, cfg->ms_sigma, cfg->edge_margin,
                      cfg->l_min};
  for (float v : fv)
    if (!finite_f(v)) return fail(nullptr, MKF_E_ARG, "non-finite setting");
  if (!(cfg->chi2_cut > 0.f) || cfg->ms_sigma < 0.f || cfg->edge_margin < 0.f ||
      !(cfg->l_min > 0.f) || !(cfg->kappa > 0.f))
    return fail(nullptr, MKF_E_ARG, "chi2_cut, kappa, l_min must be > 0; ms_sigma, edge_margin >= 0");
  for (int i = 0; i < 6; ++i)
    if (!(cfg->init_var[i] > 0.f) || !finite_f(cfg->init_var[i]))
      return fail(nullptr, MKF_E_ARG, "init_var must be finite and > 0");
  if (cfg->flags & ~(MKF_F_BATCHED | MKF_F_GRAPH | MKF_F_SURROGATE | MKF_F_CHECKED))
    return fail(nullptr, MKF_E_ARG, "unknown flag bits 0x%x", (unsigned)cfg->flags);
  mkf_ctx *c = new (std::nothrow) mkf_ctx();
  if (!c) return fail(nullptr, MKF_E_CAPACITY, "out of host memory");
  c->cfg = *cfg;
  c->stream = static_cast<hipStream_t>(stream);
  hipError_t e = hipEventCreate(&c->ev_a);
  if (e == hipSuccess) e = hipEventCreate(&c->ev_b);
  if (e == hipSuccess) e = hipEventCreate(&c->ev_m0);
  if (e == hipSuccess) e = hipEventCreate(&c->ev_m1);
  for (int k = 0; k < kCopyThreads && e == hipSuccess; ++k)
    e = hipEventCreateWithFlags(&c->ev_copy[k], hipEventDisableTiming);
  if (e == hipSuccess)
    e = hipHostMalloc(reinterpret_cast<void **>(&c->h_cnt),
                      sizeof(unsigned long long) * kFindWords +
                          sizeof(int) * (kLenSlots * kLenWords + 1),
                      hipHostMallocDefault);
  if (e != hipSuccess) {
    delete c;
    return fail(nullptr, MKF_E_HIP, "HIP setup failed: %s", hipGetErrorString(e));
  }
  c->h_len = reinterpret_cast<int *>(c->h_cnt + kFindWords);
  c->h_bad = c->h_len + kLenSlots * kLenWords;
  int dev = 0, n_cu = 0;
  (void)hipGetDevice(&dev);
  (void)hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev);
  c->n_cu = std::max(1, n_cu);
  c->device = dev;
  if (hipError_t es = resolve_scratch(dev)) {
    delete c;
    return fail(nullptr, MKF_E_HIP, "scratch address on device %d: %s", dev,
                hipGetErrorString(es));
  }
  if (hipError_t em = mlp_setup(c)) {
    delete c;
    return fail(nullptr, MKF_E_HIP, "surrogate setup failed: %s", hipGetErrorString(em));
  }
  hipDeviceProp_t prop;
  if (hipGetDeviceProperties(&prop, dev) == hipSuccess) c->arch = prop.gcnArchName;
  for (char &ch : c->arch)
    if (ch == ' ' || ch == ':') ch = '_';
  c->err = "no error";
  *out = c;
  return MKF_OK;
}

void mkf_destroy(mkf_ctx *ctx) {
  if (!ctx) return;
  if (ctx->stream) (void)hipStreamSynchronize(ctx->stream);
  else (void)hipDeviceSynchronize();
  delete ctx;
}

const char *mkf_last_error(const mkf_ctx *ctx) {
  return ctx ? ctx->err.c_str() : g_create_error.c_str();
}

}  // extern "C"

namespace {

int shifted_bins(int n, int shift, int max) {
  const int64_t v = shift >= 0 ? (int64_t)n << shift : (int64_t)n >> -shift;
  return (int)std::min<int64_t>(std::max<int64_t>(v, 1), max);
}

// Device layer records from the loaded layers and the tuning's bin shifts.
mkf_status upload_layers(mkf_ctx *c) {
  int base = 0;
  DevLayer dl[kMaxLayers]{};
  for (int i = 0; i < c->n_layers; ++i) {
    const mkf_layer &L = c->user_layers[i];
    const int nphi = shifted_bins(L.n_phi_bins, c->tuning.phi_bin_shift, 4096);
    const int nq = shifted_bins(L.n_q_bins, c->tuning.q_bin_shift, 1024);
    DevLayer &d = dl[i];
    d.kind = L.kind;
    d.pos = L.pos;
    d.lo = L.ext_lo;
    d.hi = L.ext_hi;
    d.vu_max = L.var_u_max;
    d.vv_max = L.var_v_max;
    d.nphi = nphi;
    d.nq = nq;
    d.bin_base = base;
    d.q_lo = L.ext_lo;
    d.q_scale = (float)nq / (L.ext_hi - L.ext_lo);
    d.phi_scale = (float)nphi / kTwoPi;
    d.cs = L.stereo == 0.f ? 1.f : std::cos(L.stereo);
    d.sn = L.stereo == 0.f ? 0.f : std::sin(L.stereo);
    d.hole_lo = L.hole_lo < L.hole_hi ? L.hole_lo : 0.f;
    d.hole_hi = L.hole_lo < L.hole_hi ? L.hole_hi : 0.f;
    base += nphi * nq;
  }
  HIP_TRY(c, c->d_layers.ensure(sizeof(DevLayer) * kMaxLayers));
  HIP_TRY(c, hipMemcpyAsync(c->d_layers.ptr, dl, sizeof(dl), hipMemcpyHostToDevice, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  std::memcpy(c->layers, dl, sizeof(dl));
  c->bins_per_event = base;
  return MKF_OK;
}

// The binned hit index (records and counts, scan, scatter) for the current
// layer records: of the given hits, or (in.x null) again of the loaded ones.
mkf_status build_index(mkf_ctx *c, const HitArrays &in) {
  const int64_t n_hits = c->n_hits;
  const int64_t total_bins = (int64_t)c->n_events * c->bins_per_event;
  if (total_bins >= ((int64_t)1 << 31) - 1)
    return fail(c, MKF_E_CAPACITY, "events x bins exceed the index size");
  const size_t H = (size_t)std::max<int64_t>(n_hits, 1);
  HIP_TRY(c, c->d_bin_rank.ensure(sizeof(int2) * H));
  HIP_TRY(c, c->d_counts.ensure(sizeof(int) * (size_t)std::max<int64_t>(total_bins, 1)));
  HIP_TRY(c, c->d_bin_start.ensure(sizeof(int) * (size_t)(total_bins + 1)));
  HIP_TRY(c, c->d_scan_tmp.ensure(sizeof(int) * (size_t)scan_tmp_words(total_bins)));
  HIP_TRY(c, c->d_sorted.ensure(sizeof(HitRec) * (H + kHitPad)));
  HIP_TRY(c, c->d_byorig.ensure(sizeof(HitRec) * H));
  if (has_stereo(c)) HIP_TRY(c, c->d_raw.ensure(sizeof(float2) * H));
  const FindParams P = params(c);
  *c->h_bad = 0;
  HIP_TRY(c, hipEventRecord(c->ev_a, c->stream));
  launch_fill_i32(c->stream, c->d_counts.as<int>(), total_bins, 0);
  launch_hits_in(c->stream, P, n_hits, in, c->d_byorig.as<HitRec>(),
                 has_stereo(c) ? c->d_raw.as<float2>() : nullptr, c->d_bin_rank.as<int2>(),
                 c->d_counts.as<int>(), c->h_bad);
  launch_scan(c->stream, c->d_counts.as<int>(), c->d_bin_start.as<int>(), total_bins,
              c->d_scan_tmp.as<int>());
  launch_scatter(c->stream, P, n_hits, c->d_bin_rank.as<int2>(), c->d_sorted.as<HitRec>());
  HIP_TRY(c, hipGetLastError());
  HIP_TRY(c, hipEventRecord(c->ev_b, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  if (*c->h_bad) return fail(c, MKF_E_ARG, "hits: non-finite value, variance <= 0 or bad layer");
  float ms = 0.f;
  HIP_TRY(c, hipEventElapsedTime(&ms, c->ev_a, c->ev_b));
  c->stats.index_ms = ms;
  return MKF_OK;
}

}  // namespace

extern "C" {

mkf_status mkf_load_geometry(mkf_ctx *c, const mkf_layer *layers, int32_t n_layers) {
  if (!c) return MKF_E_ARG;
  if (!layers || n_layers <= 0 || n_layers > MKF_MAX_LAYERS)
    return fail(c, MKF_E_ARG, "need 1..%d layers", MKF_MAX_LAYERS);
  for (int i = 0; i < n_layers; ++i) {
    const mkf_layer &L = layers[i];
    if (L.kind != MKF_BARREL && L.kind != MKF_DISK)
      return fail(c, MKF_E_GEOMETRY, "layer %d: bad kind %d", i, L.kind);
    if (!finite_f(L.pos) || !finite_f(L.ext_lo) || !finite_f(L.ext_hi) ||
        !(L.ext_lo < L.ext_hi))
      return fail(c, MKF_E_GEOMETRY, "layer %d: bad position or extent", i);
    if (L.kind == MKF_BARREL && !(L.pos > 0.f))
      return fail(c, MKF_E_GEOMETRY, "layer %d: barrel radius must be > 0", i);
    if (L.kind == MKF_DISK && !(L.ext_lo >= 0.f))
      return fail(c, MKF_E_GEOMETRY, "layer %d: disk inner radius must be >= 0", i);
    if (!(L.var_u_max > 0.f) || !(L.var_v_max > 0.f) || !finite_f(L.var_u_max) ||
        !finite_f(L.var_v_max))
      return fail(c, MKF_E_GEOMETRY, "layer %d: variance bounds must be > 0", i);
    if (L.n_phi_bins < 1 || L.n_phi_bins > 4096 || L.n_q_bins < 1 || L.n_q_bins > 1024)
      return fail(c, MKF_E_GEOMETRY, "layer %d: bin counts out of range", i);
    if (!finite_f(L.stereo) || !(std::fabs(L.stereo) < 1.5707f))
      return fail(c, MKF_E_GEOMETRY, "layer %d: stereo angle must lie in (-pi/2, pi/2)", i);
    if (!finite_f(L.hole_lo) || !finite_f(L.hole_hi))
      return fail(c, MKF_E_GEOMETRY, "layer %d: bad hole", i);
  }
  std::memcpy(c->user_layers, layers, sizeof(mkf_layer) * n_layers);
  c->n_layers = n_layers;
  mkf_status st = upload_layers(c);
  if (st != MKF_OK) return st;
  c->n_regions = 0;
  c->stage = kGeometry;
  return MKF_OK;
}

mkf_status mkf_load_material(mkf_ctx *c, const mkf_material_info *info, const float *x_x0,
                             const float *xi) {
  if (!c) return MKF_E_ARG;
  if (!info) {
    c->mat = DevMat{};
    drop_graph(c);
    return MKF_OK;
  }
  if (info->n_r < 1 || info->n_z < 1 || info->n_r > 4096 || info->n_z > 4096 ||
      (int64_t)info->n_r * info->n_z > (1 << 22))
    return fail(c, MKF_E_ARG, "material map: need 1..4096 bins per axis, at most 2^22 in all");
  if (!finite_f(info->r_max) || !(info->r_max > 0.f) || !finite_f(info->z_max) ||
      !(info->z_max > 0.f))
    return fail(c, MKF_E_ARG, "material map: r_max and z_max must be finite and > 0");
  if (!finite_f(info->mass) || !(info->mass > 0.f) || !finite_f(info->k_max) ||
      !(info->k_max >= 1.f))
    return fail(c, MKF_E_ARG, "material map: need mass > 0 and k_max >= 1");
  if (!x_x0 || !xi) return fail(c, MKF_E_ARG, "material map: NULL table");
  const size_t n = (size_t)info->n_r * (size_t)info->n_z;
  std::vector<float2> tab(n);
  for (size_t i = 0; i < n; ++i) {
    if (!finite_f(x_x0[i]) || !(x_x0[i] >= 0.f) || !(x_x0[i] <= 1.f) || !finite_f(xi[i]) ||
        !(xi[i] >= 0.f) || !(xi[i] <= 100.f))
      return fail(c, MKF_E_ARG, "material map: bin %zu out of range (0 <= x/X0 <= 1, 0 <= xi <= 100)",
                  i);
    tab[i] = make_float2(x_x0[i], xi[i]);
  }
  HIP_TRY(c, c->d_mat.ensure(sizeof(float2) * n));
  HIP_TRY(c, hipMemcpyAsync(c->d_mat.ptr, tab.data(), sizeof(float2) * n, hipMemcpyHostToDevice,
                            c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  DevMat m{};
  m.tab = c->d_mat.as<float2>();
  m.nr = info->n_r;
  m.nz = info->n_z;
  m.r_scale = (float)info->n_r / info->r_max;
  m.z_max = info->z_max;
  m.z_scale = (float)info->n_z / (2.f * info->z_max);
  m.mass = info->mass;
  m.k_max = info->k_max;
  c->mat = m;
  drop_graph(c);
  return MKF_OK;
}

mkf_status mkf_load_field(mkf_ctx *c, const mkf_field *f) {
  if (!c) return MKF_E_ARG;
  if (!f) {
    c->field = DevField{};
    drop_graph(c);
    return MKF_OK;
  }
  if (!finite_f(f->b0) || f->b0 == 0.f || !finite_f(f->c_r2) || !finite_f(f->c_z2) ||
      !finite_f(f->c_z4))
    return fail(c, MKF_E_ARG, "field: coefficients must be finite and b0 != 0");
  if (!finite_f(f->h_max) || !(f->h_max >= 0.01f) || !(f->h_max <= 100.f))
    return fail(c, MKF_E_ARG, "field: h_max must lie in [0.01, 100] cm");
  DevField d{};
  d.on = 1;
  d.kb0 = -c->cfg.kappa * f->b0;
  d.c_r2 = f->c_r2;
  d.c_z2 = f->c_z2;
  d.c_z4 = f->c_z4;
  d.h_max = f->h_max;
  c->field = d;
  drop_graph(c);
  return MKF_OK;
}

mkf_status mkf_load_steering(mkf_ctx *c, const mkf_region *regions, int32_t n_regions) {
  if (!c) return MKF_E_ARG;
  if (c->stage < kGeometry) return fail(c, MKF_E_ORDER, "load_geometry first");
  if (n_regions < 0 || n_regions > MKF_MAX_REGIONS || (n_regions > 0 && !regions))
    return fail(c, MKF_E_ARG, "need 0..%d regions", MKF_MAX_REGIONS);
  DevRegion dr[kMaxRegions]{};
  for (int r = 0; r < n_regions; ++r) {
    const mkf_region &g = regions[r];
    if (std::isnan(g.eta_lo) || std::isnan(g.eta_hi) || !(g.eta_lo < g.eta_hi))
      return fail(c, MKF_E_ARG, "region %d: need eta_lo < eta_hi", r);
    if (g.n_layers < 0 || g.n_layers > MKF_MAX_PLAN)
      return fail(c, MKF_E_ARG, "region %d: need 0..%d layers", r, MKF_MAX_PLAN);
    bool seen[kMaxLayers] = {};
    for (int k = 0; k < g.n_layers; ++k) {
      const int L = g.layers[k];
      if (L < 0 || L >= c->n_layers)
        return fail(c, MKF_E_ARG, "region %d: layer id %d not in the geometry", r, L);
      if (seen[L]) return fail(c, MKF_E_ARG, "region %d: layer %d listed twice", r, L);
      seen[L] = true;
      dr[r].layers[k] = (int8_t)L;
    }
    dr[r].eta_lo = g.eta_lo;
    dr[r].eta_hi = g.eta_hi;
    dr[r].n = g.n_layers;
  }
  HIP_TRY(c, c->d_regions.ensure(sizeof(dr)));
  HIP_TRY(c, hipMemcpyAsync(c->d_regions.ptr, dr, sizeof(dr), hipMemcpyHostToDevice, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  c->n_regions = n_regions;
  return MKF_OK;
}

mkf_status mkf_load_hits(mkf_ctx *c, int32_t n_events, const int64_t *ev_off, const float *x,
                         const float *y, const float *z, const float *var_u,
                         const float *var_v, const int32_t *layer, int32_t mem) {
  if (!c) return MKF_E_ARG;
  if (c->stage < kGeometry) return fail(c, MKF_E_ORDER, "load_geometry first");
  if (n_events < 0 || !ev_off) return fail(c, MKF_E_ARG, "bad event offsets");
  if (mem != MKF_MEM_HOST && mem != MKF_MEM_DEVICE) return fail(c, MKF_E_ARG, "bad mem");
  if (ev_off[0] != 0) return fail(c, MKF_E_ARG, "ev_off[0] must be 0");
  for (int e = 0; e < n_events; ++e) {
    const int64_t n = ev_off[e + 1] - ev_off[e];
    if (n < 0) return fail(c, MKF_E_ARG, "event offsets must not decrease");
    if (n >= (int64_t)0x7FFFFF) return fail(c, MKF_E_CAPACITY, "event %d has too many hits", e);
  }
  const int64_t n_hits = ev_off[n_events];
  if (n_hits > 0 && (!x || !y || !z || !var_u || !var_v || !layer))
    return fail(c, MKF_E_ARG, "hit array is NULL");
  if (n_hits >= ((int64_t)1 << 31)) return fail(c, MKF_E_CAPACITY, "too many hits");
  const int64_t total_bins = (int64_t)n_events * c->bins_per_event;
  if (total_bins >= ((int64_t)1 << 31) - 1)
    return fail(c, MKF_E_CAPACITY, "events x bins exceed the index size");
  if (mem == MKF_MEM_HOST) {
    for (int64_t i = 0; i < n_hits; ++i) {
      if (!finite_f(x[i]) || !finite_f(y[i]) || !finite_f(z[i]) || !finite_f(var_u[i]) ||
          !finite_f(var_v[i]) || !(var_u[i] > 0.f) || !(var_v[i] > 0.f))
        return fail(c, MKF_E_ARG, "hit %lld: non-finite value or variance <= 0", (long long)i);
      if (layer[i] < 0 || layer[i] >= c->n_layers)
        return fail(c, MKF_E_ARG, "hit %lld: layer %d out of range", (long long)i, layer[i]);
    }
  }
  c->stage = kGeometry;
  drop_graph(c);
  const size_t fb = sizeof(float) * (size_t)n_hits;
  mkf_status st;
  if ((st = stage_in(c, c->d_ev_off, ev_off, sizeof(int64_t) * (n_events + 1), MKF_MEM_HOST))) return st;
  HitArrays in{x, y, z, var_u, var_v, layer};
  if (mem == MKF_MEM_HOST && n_hits > 0) {
    if ((st = stage_in(c, c->d_x, x, fb, mem))) return st;
    if ((st = stage_in(c, c->d_y, y, fb, mem))) return st;
    if ((st = stage_in(c, c->d_z, z, fb, mem))) return st;
    if ((st = stage_in(c, c->d_vu, var_u, fb, mem))) return st;
    if ((st = stage_in(c, c->d_vv, var_v, fb, mem))) return st;
    if ((st = stage_in(c, c->d_layer, layer, sizeof(int) * (size_t)n_hits, mem))) return st;
    in = HitArrays{c->d_x.as<float>(),  c->d_y.as<float>(),  c->d_z.as<float>(),
                   c->d_vu.as<float>(), c->d_vv.as<float>(), c->d_layer.as<int>()};
  }
  c->n_events = n_events;
  c->n_hits = n_hits;
  c->ev_off.assign(ev_off, ev_off + n_events + 1);
  if ((st = build_index(c, in))) return st;
  c->stage = kHits;
  c->n_seeds = 0;
  return MKF_OK;
}

mkf_status mkf_seed(mkf_ctx *c, int64_t n_seeds, const int32_t *seed_event,
                    const int32_t *seed_hits, int32_t mem) {
  if (!c) return MKF_E_ARG;
  if (c->stage < kHits) return fail(c, MKF_E_ORDER, "load_hits first");
  if (n_seeds < 0 || n_seeds >= ((int64_t)1 << 28)) return fail(c, MKF_E_ARG, "bad seed count");
  if (n_seeds > 0 && (!seed_event || !seed_hits)) return fail(c, MKF_E_ARG, "seed array is NULL");
  if (mem != MKF_MEM_HOST && mem != MKF_MEM_DEVICE) return fail(c, MKF_E_ARG, "bad mem");
  const size_t N = (size_t)std::max<int64_t>(n_seeds, 1);
  if (mem == MKF_MEM_DEVICE && n_seeds > 0) {
    FindParams V = params(c);
    V.n_seeds = n_seeds;
    *c->h_bad = 0;
    launch_validate_seeds(c->stream, V, seed_event, seed_hits, c->h_bad);
    HIP_TRY(c, hipGetLastError());
    HIP_TRY(c, hipStreamSynchronize(c->stream));
  }
  if (mem == MKF_MEM_HOST || (n_seeds > 0 && *c->h_bad)) {
    // host arrays, or device arrays with an index out of range: the first one
    std::vector<int32_t> h_ev, h_hits;
    const int32_t *sev = seed_event, *sh = seed_hits;
    if (mem == MKF_MEM_DEVICE) {
      h_ev.resize(n_seeds);
      h_hits.resize(3 * n_seeds);
      HIP_TRY(c, hipMemcpyAsync(h_ev.data(), seed_event, 4 * n_seeds, hipMemcpyDeviceToHost,
                                c->stream));
      HIP_TRY(c, hipMemcpyAsync(h_hits.data(), seed_hits, 12 * n_seeds, hipMemcpyDeviceToHost,
                                c->stream));
      HIP_TRY(c, hipStreamSynchronize(c->stream));
      sev = h_ev.data();
      sh = h_hits.data();
    }
    for (int64_t i = 0; i < n_seeds; ++i) {
      if (sev[i] < 0 || sev[i] >= c->n_events)
        return fail(c, MKF_E_ARG, "seed %lld: event %d out of range", (long long)i, sev[i]);
      const int64_t nh = c->ev_off[sev[i] + 1] - c->ev_off[sev[i]];
      for (int k = 0; k < 3; ++k)
        if (sh[3 * i + k] < 0 || sh[3 * i + k] >= nh)
          return fail(c, MKF_E_ARG, "seed %lld: hit index out of range", (long long)i);
    }
  }
  c->stage = kHits;
  drop_graph(c);
  const bool batched = (c->cfg.flags & MKF_F_BATCHED) != 0;
  // cells of the processing order: no more than a few per seed
  SeedCells cells{0, std::max(1, c->n_events), batched ? 0 : 1};
  while (cells.n_groups > 1 && cells.cells() > std::max<int64_t>(1 << 16, 4 * n_seeds)) {
    ++cells.event_shift;
    cells.n_groups = (int)(((int64_t)c->n_events + ((int64_t)1 << cells.event_shift) - 1) >>
                           cells.event_shift);
  }
  const int64_t n_cells = cells.cells(), n_len = kLenSlots * kLenWords;
  HIP_TRY(c, c->d_seed_event.ensure(4 * N));
  HIP_TRY(c, c->d_seed_hits.ensure(12 * N));
  HIP_TRY(c, c->d_seed_state.ensure(sizeof(float) * kSeedWords * N));
  HIP_TRY(c, c->d_seed_ok.ensure(4 * N));
  HIP_TRY(c, c->d_plan_len.ensure(4 * N));
  HIP_TRY(c, c->d_plan.ensure(kMaxPlan * N));
  HIP_TRY(c, c->d_seed_chi2.ensure(4 * N));
  HIP_TRY(c, c->d_seed_fit.ensure(sizeof(double) * kSeedFit * N));
  HIP_TRY(c, c->d_cell_counts.ensure(sizeof(int) * (size_t)(n_cells + n_len)));
  HIP_TRY(c, c->d_cell_start.ensure(sizeof(int) * (size_t)(n_cells + 1)));
  HIP_TRY(c, c->d_cell_rank.ensure(sizeof(int2) * N));
  HIP_TRY(c, c->d_scan_tmp.ensure(sizeof(int) * (size_t)scan_tmp_words(n_cells)));
  HIP_TRY(c, c->d_order.ensure(4 * N));
  HIP_TRY(c, c->d_pos.ensure(4 * N));
  HIP_TRY(c, c->d_pstate.ensure(sizeof(float) * kSeedWords * N));
  HIP_TRY(c, c->d_pinfo.ensure(4 * N));
  HIP_TRY(c, c->d_pevent.ensure(4 * N));
  HIP_TRY(c, c->d_pplan.ensure(kMaxPlan * N));
  HIP_TRY(c, c->d_out.ensure(sizeof(float) * kOutWords * N));
  if (!batched) {  // the layer-synchronous form's state between steps
    HIP_TRY(c, c->d_cand.ensure(sizeof(float) * kCandFields * kGroup * N));
    HIP_TRY(c, c->d_fin_key.ensure(8 * N));
    HIP_TRY(c, c->d_fin_rec.ensure(sizeof(float) * 28 * N));
    HIP_TRY(c, c->d_fin_meta.ensure(4 * N));
    HIP_TRY(c, c->d_bp.ensure(4 * (size_t)kMaxPlan * kGroup * N));
  }
  // (device arrays are read, and copied, by the seed kernel)
  const int *src_event = mem == MKF_MEM_DEVICE ? seed_event : c->d_seed_event.as<int>();
  const int *src_hits = mem == MKF_MEM_DEVICE ? seed_hits : c->d_seed_hits.as<int>();
  mkf_status st;
  if (mem == MKF_MEM_HOST) {
    if ((st = stage_in(c, c->d_seed_event, seed_event, 4 * (size_t)n_seeds, mem))) return st;
    if ((st = stage_in(c, c->d_seed_hits, seed_hits, 12 * (size_t)n_seeds, mem))) return st;
  }
  c->n_seeds = n_seeds;
  const FindParams P = params(c);
  int *len_counts = c->d_cell_counts.as<int>() + n_cells;
  launch_fill_i32(c->stream, c->d_cell_counts.as<int>(), n_cells + n_len, 0);
  HIP_TRY(c, hipEventRecord(c->ev_a, c->stream));
  launch_seed(c->stream, P, src_event, src_hits, c->d_seed_event.as<int>(),
              c->d_seed_hits.as<int>(), c->d_seed_state.as<float>(), c->d_seed_ok.as<int>(),
              c->d_plan_len.as<int>(), c->d_plan.as<int8_t>(), c->d_seed_chi2.as<float>(),
              c->d_seed_fit.as<double>(),
              c->n_regions > 0 ? c->d_regions.as<DevRegion>() : nullptr, c->n_regions, cells,
              c->d_cell_counts.as<int>(), c->d_cell_rank.as<int2>(), len_counts);
  HIP_TRY(c, hipGetLastError());
  HIP_TRY(c, hipEventRecord(c->ev_b, c->stream));
  launch_scan(c->stream, c->d_cell_counts.as<int>(), c->d_cell_start.as<int>(), n_cells,
              c->d_scan_tmp.as<int>());
  launch_place_seeds(c->stream, P, c->d_cell_rank.as<int2>(), c->d_cell_start.as<int>(),
                     c->d_order.as<int>(), c->d_pos.as<int>(), c->d_pstate.as<float>(),
                     c->d_pinfo.as<int>(), c->d_pevent.as<int>(), c->d_pplan.as<int8_t>());
  HIP_TRY(c, hipGetLastError());
  HIP_TRY(c, hipMemcpyAsync(c->h_len, len_counts, sizeof(int) * n_len, hipMemcpyDeviceToHost,
                            c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  float ms = 0.f;
  HIP_TRY(c, hipEventElapsedTime(&ms, c->ev_a, c->ev_b));
  c->stats.seed_ms = ms;
  int64_t len[kLenWords] = {};
  for (int k = 0; k < n_len; ++k) len[k % kLenWords] += c->h_len[k];
  c->n_seeds_ok = len[kPlanLens];
  c->max_plan_len = 0;
  c->active_at_step.assign(kMaxPlan, 0);
  int64_t longer = 0;
  for (int k = kMaxPlan; k > 0; --k) {
    longer += len[k];
    if (longer > 0) c->max_plan_len = std::max(c->max_plan_len, k);
    // the layer-synchronous form keeps the longest plans first: the seeds
    // still active at step k - 1 form a prefix of the positions
    c->active_at_step[k - 1] = batched ? n_seeds : longer;
  }
  c->stats.n_seeds = n_seeds;
  c->stats.n_seeds_ok = c->n_seeds_ok;
  c->stats.max_plan_len = c->max_plan_len;
  c->stage = kSeeds;
  return MKF_OK;
}

mkf_status mkf_get_seed_states(mkf_ctx *c, float *par, float *cov, int32_t *ok,
                               int32_t *plan_len, int8_t *plan, float *chi2) {
  if (!c) return MKF_E_ARG;
  if (c->stage < kSeeds) return fail(c, MKF_E_ORDER, "seed first");
  const size_t n = (size_t)c->n_seeds;
  if (n == 0) return MKF_OK;
  std::vector<float> st(kSeedWords * n);
  HIP_TRY(c, hipMemcpyAsync(st.data(), c->d_seed_state.ptr, sizeof(float) * kSeedWords * n,
                            hipMemcpyDeviceToHost, c->stream));
  if (ok) HIP_TRY(c, hipMemcpyAsync(ok, c->d_seed_ok.ptr, 4 * n, hipMemcpyDeviceToHost, c->stream));
  if (plan_len)
    HIP_TRY(c, hipMemcpyAsync(plan_len, c->d_plan_len.ptr, 4 * n, hipMemcpyDeviceToHost, c->stream));
  if (plan)
    HIP_TRY(c, hipMemcpyAsync(plan, c->d_plan.ptr, kMaxPlan * n, hipMemcpyDeviceToHost, c->stream));
  if (chi2)
    HIP_TRY(c, hipMemcpyAsync(chi2, c->d_seed_chi2.ptr, 4 * n, hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  for (size_t i = 0; i < n; ++i) {
    if (par)
      for (int k = 0; k < 6; ++k) par[6 * i + k] = st[kSeedWords * i + k];
    if (cov)
      for (int k = 0; k < 21; ++k) cov[21 * i + k] = st[kSeedWords * i + 6 + k];
  }
  return MKF_OK;
}

// Launch shape of the persistent find where none was set: as many waves per SIMD
// as its tiles fill, from two up to three, the most that run without spilling
// much; four where that takes all tiles at once, though not with the surrogate,
// which spills far more there.  Measured at 18 numbers of tiles, events of 5,000
// seeds, at two, three and four waves (us; on 1,024 SIMDs the lines are 2,048, 3,072
// and 4,096 tiles):
//   2,000 tiles 116, 118, 141    2,100  183, 124, 148   3,000  198, 128, 150
//   3,100       202, 195, 166    4,090  203, 212, 172   4,150  252, 223, 240
//   24,000      868, 684, 787
//   with material and field  2,000  195, 207, 235   3,000 304, 218, 249
//                            4,000  341, 341, 294   4,150 353, 349, 376
//   with the surrogate       3,000  221, 147, 189   3,600 238, 233, 291
// No more blocks than are resident: the starting value of eight per CU left the
// blocks beyond them to a second turn (1.85 ms for 1.79 at two waves, 100 events).
static void launch_shape(const mkf_ctx *c, int &waves, int &blocks_per_cu) {
  waves = c->tuning.waves_per_simd;
  blocks_per_cu = c->tuning.blocks_per_cu;
  if (c->tuned) return;
  const int seeds = c->cfg.n_cand > 6 || c->tuning.lane_group == 8 ? 8 : 10;
  const int64_t tiles = (c->n_seeds + seeds - 1) / seeds, simds = 4 * (int64_t)c->n_cu;
  const bool all_in_four = tiles > 3 * simds && tiles <= 4 * simds;
  waves = tiles <= 2 * simds ? 2
          : all_in_four && !(c->cfg.flags & MKF_F_SURROGATE) ? 4 : 3;
  blocks_per_cu = waves;
}

// Queue the whole find on the context stream.  main_a/main_b (may be
// null) bracket the layer-step kernels.
static int enqueue_find(mkf_ctx *c, const FindParams &P, hipEvent_t main_a, hipEvent_t main_b) {
  int launches = 0;
  launch_fill_u64(c->stream, c->d_cnt.as<unsigned long long>(), kClearWords, 0ull);
  ++launches;
  if (c->cfg.flags & MKF_F_BATCHED) {
    if (main_a) (void)hipEventRecord(main_a, c->stream);
    int waves, blocks_per_cu;
    launch_shape(c, waves, blocks_per_cu);
    launch_find_persistent(c->stream, P, blocks_per_cu * c->n_cu, waves,
                           (c->cfg.flags & MKF_F_SURROGATE) != 0, c->tuning.lane_group);
    ++launches;
    c->stats.main_launches = 1;
  } else {
    launch_find_init(c->stream, P);
    ++launches;
    if (main_a) (void)hipEventRecord(main_a, c->stream);
    int n = 0;
    for (int s = 0; s < c->max_plan_len; ++s) {
      launch_find_step(c->stream, P, s, c->active_at_step[s]);
      ++n;
    }
    launches += n;
    c->stats.main_launches = n;
  }
  if (main_b) (void)hipEventRecord(main_b, c->stream);
  if (!(c->cfg.flags & MKF_F_BATCHED)) {
    launch_finalize(c->stream, P);
    ++launches;
  }
  return launches;
}

mkf_status mkf_find(mkf_ctx *c) {
  if (!c) return MKF_E_ARG;
  if (c->stage < kSeeds) return fail(c, MKF_E_ORDER, "seed first");
  FindParams P = params(c);
  int launches = 0;
  const bool graph = (c->cfg.flags & MKF_F_GRAPH) != 0;
  if (graph && !c->graph_exec) {
    if (!c->stream)
      return fail(c, MKF_E_ARG, "graph replay needs a non-default stream at mkf_create");
    HIP_TRY(c, hipStreamBeginCapture(c->stream, hipStreamCaptureModeThreadLocal));
    c->graph_launches = enqueue_find(c, P, nullptr, nullptr);
    hipError_t e = hipStreamEndCapture(c->stream, &c->graph);
    if (e == hipSuccess) e = hipGetLastError();
    if (e == hipSuccess) e = hipGraphInstantiate(&c->graph_exec, c->graph, nullptr, nullptr, 0);
    if (e != hipSuccess) {
      drop_graph(c);
      return fail(c, MKF_E_HIP, "graph capture failed: %s", hipGetErrorString(e));
    }
  }
  HIP_TRY(c, hipEventRecord(c->ev_a, c->stream));
  if (graph) {
    HIP_TRY(c, hipGraphLaunch(c->graph_exec, c->stream));
    launches = c->graph_launches;
  } else {
    launches = enqueue_find(c, P, c->ev_m0, c->ev_m1);
  }
  HIP_TRY(c, hipGetLastError());
  HIP_TRY(c, hipEventRecord(c->ev_b, c->stream));
  // (after the timed region: the checked find's record invariants)
  if (c->cfg.flags & MKF_F_CHECKED) {
    launch_check_results(c->stream, P);
    HIP_TRY(c, hipGetLastError());
  }
  // the step count and counters: one copy into pinned memory behind the
  // find on its stream, then one wait, which also completes the events
  const unsigned long long *cnt = c->h_cnt + 1;
  HIP_TRY(c, hipMemcpyAsync(c->h_cnt, c->d_cnt.ptr, sizeof(unsigned long long) * kFindWords,
                            hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  float ms = 0.f, mms = -1.f;
  HIP_TRY(c, hipEventElapsedTime(&ms, c->ev_a, c->ev_b));
  if (!graph) HIP_TRY(c, hipEventElapsedTime(&mms, c->ev_m0, c->ev_m1));
  const unsigned long long steps = c->h_cnt[0];
  int64_t tot[kCounters] = {};
  for (int k = 0; k < kCounters; ++k)
    for (int j = 0; j < kCounterSlots; ++j) tot[k] += (int64_t)cnt[k * kCounterSlots + j];
  c->stats.sur_kept = tot[kCntSurKept];
  c->stats.sur_rejected = tot[kCntSurRejected];
  c->stats.n_near_cut = tot[kCntNearCut];
  c->stats.n_rk_steps = tot[kCntRk];
  c->stats.n_newton = tot[kCntNewton];
  c->stats.n_check_failed = tot[kCntCheckFailed];
  c->stats.find_ms = ms;
  c->stats.main_ms = mms;
  c->stats.n_steps = (int64_t)steps;
  c->stats.n_launches = launches;
  c->stage = kFound;
  if (c->stats.n_check_failed > 0)
    return fail(c, MKF_E_NUMERIC, "checked find: %lld result records violate the find's invariants",
                (long long)c->stats.n_check_failed);
  return MKF_OK;
}

static hipError_t pin_records(mkf_track **slot, int64_t n) {
  return hipHostMalloc(reinterpret_cast<void **>(slot), sizeof(mkf_track) * (size_t)n,
                       hipHostMallocDefault);
}

mkf_status mkf_get_tracks(mkf_ctx *c, mkf_track *out, int64_t capacity, int64_t *n_total) {
  if (!c) return MKF_E_ARG;
  if (c->stage < kFound) return fail(c, MKF_E_ORDER, "find first");
  if (n_total) *n_total = c->n_seeds;
  if (capacity < 0 || (capacity > 0 && !out)) return fail(c, MKF_E_ARG, "bad output buffer");
  auto too_few = [&]() {
    return fail(c, MKF_E_CAPACITY, "capacity %lld < %lld tracks", (long long)capacity,
                (long long)c->n_seeds);
  };
  const int64_t n = std::min(capacity, c->n_seeds);
  if (n > 0) {
    // (kernels and events want the context's device to be current)
    DeviceScope scope;
    HIP_TRY(c, scope.enter(c->device));
    const int slots = (int)std::min<int64_t>(kCopyThreads, (n + kCopyRecords - 1) / kCopyRecords);
    const int64_t want = n <= kFewRecords ? kFewRecords : kCopyRecords;
    if (c->h_slot0_n < want) {
      if (c->h_slot[0]) (void)hipHostFree(c->h_slot[0]);
      c->h_slot[0] = nullptr;
      c->h_slot0_n = 0;
      HIP_TRY(c, pin_records(&c->h_slot[0], want));
      c->h_slot0_n = want;
    }
    const FindParams P = params(c);
    if (slots == 1) {
      // few records: in up to kCopyParts parts, so that the first are copied out
      // while the device writes the next
      const int64_t part = std::max<int64_t>(1024, (n + kCopyParts - 1) / kCopyParts);
      int parts = 0;
      for (int64_t first = 0; first < n; first += part, ++parts) {
        launch_tracks(c->stream, P, c->d_pos.as<int>(), first, std::min(part, n - first),
                      reinterpret_cast<int *>(c->h_slot[0] + first));
        HIP_TRY(c, hipGetLastError());
        HIP_TRY(c, hipEventRecord(c->ev_copy[parts], c->stream));
      }
      for (int k = 0; k < parts; ++k) {
        HIP_TRY(c, hipEventSynchronize(c->ev_copy[k]));
        const int64_t first = k * part;
        std::memcpy(out + first, c->h_slot[0] + first,
                    sizeof(mkf_track) * (size_t)std::min(part, n - first));
      }
      return capacity < c->n_seeds ? too_few() : MKF_OK;
    }
    std::atomic<int64_t> next{0};
    std::atomic<int> status{(int)hipSuccess};
    // takes chunks of seeds until none are left: the device writes a chunk's
    // records into slot k, which are then copied out
    auto work = [&](int k) {
      hipError_t e = k == 0 ? hipSuccess : hipSetDevice(c->device);
      if (e == hipSuccess && !c->h_slot[k] &&
          pin_records(&c->h_slot[k], kCopyRecords) != hipSuccess)
        return;  // no slot for this thread: the others take all chunks (the first has one)
      mkf_track *slot = c->h_slot[k];
      while (e == hipSuccess) {
        const int64_t first = next.fetch_add(kCopyRecords);
        if (first >= n) break;
        const int64_t m = std::min(kCopyRecords, n - first);
        launch_tracks(c->stream, P, c->d_pos.as<int>(), first, m, reinterpret_cast<int *>(slot));
        e = hipGetLastError();
        if (e == hipSuccess) e = hipEventRecord(c->ev_copy[k], c->stream);
        if (e == hipSuccess) e = hipEventSynchronize(c->ev_copy[k]);
        if (e == hipSuccess) std::memcpy(out + first, slot, sizeof(mkf_track) * (size_t)m);
      }
      if (e != hipSuccess) status = (int)e;
    };
    std::thread helper[kCopyThreads];
    int started = 1;
    try {
      for (; started < slots; ++started) helper[started] = std::thread(work, started);
    } catch (const std::exception &) {
      // no further thread to be had: those that started take all chunks
    }
    work(0);
    for (int k = 1; k < started; ++k) helper[k].join();
    if (status != (int)hipSuccess)
      return fail(c, MKF_E_HIP, "copying the tracks failed: %s",
                  hipGetErrorString((hipError_t)status.load()));
  }
  return capacity < c->n_seeds ? too_few() : MKF_OK;
}

mkf_status mkf_propagate(mkf_ctx *c, int64_t n, const float *par, const float *cov,
                         const int32_t *layer, float *out_par, float *out_cov, float *out_l,
                         int32_t *out_status) {
  if (!c) return MKF_E_ARG;
  if (c->stage < kGeometry) return fail(c, MKF_E_ORDER, "load_geometry first");
  if (n < 0) return fail(c, MKF_E_ARG, "n < 0");
  if (n > 0 && (!par || !cov || !layer || !out_par || !out_cov || !out_l || !out_status))
    return fail(c, MKF_E_ARG, "NULL array");
  FindParams P = params(c);
  launch_propagate(c->stream, P, n, par, cov, layer, out_par, out_cov, out_l, out_status);
  HIP_TRY(c, hipGetLastError());
  return MKF_OK;
}

mkf_status mkf_fit(mkf_ctx *c, int64_t n_tracks, int32_t n_steps, const int8_t *kind,
                   const float *pos, const float *x, const float *y, const float *z,
                   const float *var_u, const float *var_v, const int32_t *len,
                   const float *init_par, const float *init_cov, float *out_par, float *out_cov,
                   float *out_chi2, int32_t *out_status) {
  if (!c) return MKF_E_ARG;
  if (n_tracks < 0 || n_steps < 0) return fail(c, MKF_E_ARG, "negative size");
  if (n_tracks > 0 && (!len || !init_par || !init_cov || !out_par || !out_cov || !out_chi2 ||
                       !out_status))
    return fail(c, MKF_E_ARG, "NULL array");
  if (n_tracks > 0 && n_steps > 0 && (!kind || !pos || !x || !y || !z || !var_u || !var_v))
    return fail(c, MKF_E_ARG, "NULL hit array");
  HIP_TRY(c, hipEventRecord(c->ev_a, c->stream));
  DevCfg fcfg = dev_cfg(c->cfg);
  fcfg.mat = c->mat;
  fcfg.field = c->field;
  launch_fit(c->stream, fcfg, n_tracks, n_steps, kind, pos, x, y, z, var_u, var_v, len,
             init_par, init_cov, out_par, out_cov, out_chi2, out_status);
  HIP_TRY(c, hipGetLastError());
  HIP_TRY(c, hipEventRecord(c->ev_b, c->stream));
  return MKF_OK;
}

mkf_status mkf_backward_fit(mkf_ctx *c, float *out_par, float *out_cov, float *out_chi2,
                            int32_t *out_status) {
  if (!c) return MKF_E_ARG;
  if (c->stage < kFound) return fail(c, MKF_E_ORDER, "find first");
  if (c->n_seeds > 0 && (!out_par || !out_cov || !out_chi2 || !out_status))
    return fail(c, MKF_E_ARG, "NULL output array");
  HIP_TRY(c, c->d_bf_tmp.ensure(sizeof(float) * 32 * (size_t)std::max<int64_t>(c->n_seeds, 1)));
  FindParams P = params(c);
  launch_backfit(c->stream, P, c->d_seed_hits.as<int>(), c->d_bf_tmp.as<float>(), out_par,
                 out_cov, out_chi2, out_status);
  HIP_TRY(c, hipGetLastError());
  return MKF_OK;
}

mkf_status mkf_smooth(mkf_ctx *c, float *out_par, float *out_cov, int32_t *out_n) {
  if (!c) return MKF_E_ARG;
  if (c->stage < kFound) return fail(c, MKF_E_ORDER, "find first");
  if (c->n_seeds > 0 && (!out_par || !out_cov || !out_n))
    return fail(c, MKF_E_ARG, "NULL output array");
  const size_t N = (size_t)std::max<int64_t>(c->n_seeds, 1);
  HIP_TRY(c, c->d_sm_wk.ensure(sizeof(float) * 91 * (size_t)(c->max_plan_len + 1) * N));
  HIP_TRY(c, c->d_sm_n.ensure(sizeof(int) * N));
  FindParams P = params(c);
  launch_smooth(c->stream, P, c->d_seed_hits.as<int>(), c->d_sm_wk.as<float>(),
                c->d_sm_n.as<int>(), out_par, out_cov, out_n);
  HIP_TRY(c, hipGetLastError());
  return MKF_OK;
}

mkf_status mkf_make_seeds(mkf_ctx *c, const mkf_seeding *sc, int64_t capacity,
                          int32_t *out_event, int32_t *out_hits, int64_t *n_total) {
  if (!c) return MKF_E_ARG;
  if (c->stage < kHits) return fail(c, MKF_E_ORDER, "load_hits first");
  if (!sc || !n_total || capacity < 0) return fail(c, MKF_E_ARG, "NULL argument");
  if (capacity > 0 && (!out_event || !out_hits)) return fail(c, MKF_E_ARG, "NULL output array");
  for (int k = 0; k < 3; ++k) {
    const int L = sc->layers[k];
    if (L < 0 || L >= c->n_layers || c->layers[L].kind != MKF_BARREL)
      return fail(c, MKF_E_ARG, "seeding layer %d is not a barrel layer", L);
    if (k > 0 && !(c->layers[L].pos > c->layers[sc->layers[k - 1]].pos))
      return fail(c, MKF_E_ARG, "seeding layers must have increasing radii");
  }
  if (!(sc->pt_min > 0.f) || !(sc->d0_max > 0.f) || !(sc->z0_max > 0.f) || !(sc->dz_max > 0.f))
    return fail(c, MKF_E_ARG, "seeding cuts must be positive");
  if (c->cfg.bz == 0.f) return fail(c, MKF_E_ARG, "triplet seeding needs a field");
  if (c->n_events > 65535) return fail(c, MKF_E_CAPACITY, "triplet seeding takes <= 65535 events");
  *n_total = 0;
  const int64_t n = c->n_hits;
  if (n == 0) return MKF_OK;
  DevSeeding ds{};
  for (int k = 0; k < 3; ++k) ds.layer[k] = sc->layers[k];
  ds.pt_min = sc->pt_min;
  ds.d0_max = sc->d0_max;
  ds.z0_max = sc->z0_max;
  ds.dz_max = sc->dz_max;
  // triplets that may pass are kept in as many places as there are hits (16 B
  // each); where a hit's do not fit, they are found again when they are written
  const int64_t room = n / kTripletSegs;
  const int64_t n_cursor = kTripletSegs * kTilePad + 1;
  HIP_TRY(c, c->d_tr_cnt.ensure(sizeof(int) * (size_t)(n + n_cursor)));
  HIP_TRY(c, c->d_tr_off.ensure(sizeof(int) * (size_t)(n + 1)));
  HIP_TRY(c, c->d_tr_tmp.ensure(sizeof(int) * (size_t)scan_tmp_words(n)));
  HIP_TRY(c, c->d_tr_kept.ensure(sizeof(int4) * (size_t)(room * kTripletSegs)));
  HIP_TRY(c, c->d_tr_at.ensure(sizeof(int2) * (size_t)n));
  int *cnt = c->d_tr_cnt.as<int>();
  const TripletStore st{c->d_tr_kept.as<int4>(), (int)room, cnt + n, cnt + n + n_cursor - 1,
                        c->d_tr_at.as<int2>()};
  FindParams P = params(c);
  int64_t max_ev = 0;
  for (int e = 0; e < c->n_events; ++e) max_ev = std::max(max_ev, c->ev_off[e + 1] - c->ev_off[e]);
  launch_fill_i32(c->stream, cnt, n + n_cursor, 0);
  launch_triplets(c->stream, P, ds, n, max_ev, cnt, st);
  HIP_TRY(c, hipGetLastError());
  launch_scan(c->stream, cnt, c->d_tr_off.as<int>(), n, c->d_tr_tmp.as<int>());
  HIP_TRY(c, hipGetLastError());
  HIP_TRY(c, hipMemcpyAsync(c->h_len, c->d_tr_off.as<int>() + n, sizeof(int),
                            hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(c, hipMemcpyAsync(c->h_len + 1, st.n_again, sizeof(int), hipMemcpyDeviceToHost,
                            c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  const int total = c->h_len[0];
  if (total < 0) return fail(c, MKF_E_CAPACITY, "more than 2^31 triplets");
  *n_total = total;
  if (total > capacity)
    return fail(c, MKF_E_CAPACITY, "%d triplets, capacity %lld", total, (long long)capacity);
  launch_triplets_write(c->stream, P, ds, n, max_ev, cnt, c->d_tr_off.as<int>(), st,
                        c->h_len[1] > 0, out_event, out_hits);
  HIP_TRY(c, hipGetLastError());
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  return MKF_OK;
}

mkf_status mkf_find_duplicates(mkf_ctx *c, float frac, int32_t *out_dup, int64_t *n_dup) {
  if (!c) return MKF_E_ARG;
  if (c->stage < kFound) return fail(c, MKF_E_ORDER, "find first");
  if (!n_dup || (c->n_seeds > 0 && !out_dup)) return fail(c, MKF_E_ARG, "NULL argument");
  if (!(frac > 0.f && frac <= 1.f)) return fail(c, MKF_E_ARG, "frac must lie in (0, 1]");
  *n_dup = 0;
  if (c->n_seeds == 0) return MKF_OK;
  const size_t N = (size_t)c->n_seeds, H = (size_t)std::max<int64_t>(c->n_hits, 1);
  HIP_TRY(c, c->d_dup_h.ensure(sizeof(int) * kDupStride * N));
  HIP_TRY(c, c->d_dup_n.ensure(sizeof(int) * N));
  HIP_TRY(c, c->d_dup_cnt.ensure(sizeof(int) * H));
  HIP_TRY(c, c->d_dup_off.ensure(sizeof(int) * (H + 1)));
  HIP_TRY(c, c->d_dup_fill.ensure(sizeof(int) * H));
  HIP_TRY(c, c->d_dup_list.ensure(sizeof(int) * (kDupStride - 1) * N));
  HIP_TRY(c, c->d_dup_tmp.ensure(sizeof(int) * (size_t)scan_tmp_words((int64_t)H)));
  HIP_TRY(c, c->d_dup_total.ensure(sizeof(int)));
  FindParams P = params(c);
  launch_fill_i32(c->stream, c->d_dup_cnt.as<int>(), (int64_t)H, 0);
  launch_fill_i32(c->stream, c->d_dup_fill.as<int>(), (int64_t)H, 0);
  launch_fill_i32(c->stream, c->d_dup_total.as<int>(), 1, 0);
  launch_dup_prep(c->stream, P, c->d_seed_hits.as<int>(), c->d_dup_h.as<int>(),
                  c->d_dup_n.as<int>(), c->d_dup_cnt.as<int>());
  launch_scan(c->stream, c->d_dup_cnt.as<int>(), c->d_dup_off.as<int>(), (int64_t)H,
              c->d_dup_tmp.as<int>());
  launch_dup_fill(c->stream, P, c->d_dup_h.as<int>(), c->d_dup_n.as<int>(),
                  c->d_dup_off.as<int>(), c->d_dup_fill.as<int>(), c->d_dup_list.as<int>());
  launch_dup_decide(c->stream, P, c->d_seed_hits.as<int>(), c->d_dup_h.as<int>(),
                    c->d_dup_n.as<int>(), c->d_dup_off.as<int>(), c->d_dup_list.as<int>(), frac,
                    out_dup, c->d_dup_total.as<int>());
  HIP_TRY(c, hipGetLastError());
  int total = 0;
  HIP_TRY(c, hipMemcpyAsync(&total, c->d_dup_total.ptr, sizeof(int), hipMemcpyDeviceToHost,
                            c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  *n_dup = total;
  return MKF_OK;
}

mkf_status mkf_clean_seeds(mkf_ctx *c, const mkf_cleaning *cc, int32_t *out_keep,
                           int64_t *n_keep) {
  if (!c) return MKF_E_ARG;
  if (c->stage < kSeeds) return fail(c, MKF_E_ORDER, "seed first");
  if (!cc || !n_keep || (c->n_seeds > 0 && !out_keep)) return fail(c, MKF_E_ARG, "NULL argument");
  if (!(cc->tol_ipt >= 0.f) || !(cc->tol_eta >= 0.f) || !(cc->tol_phi >= 0.f))
    return fail(c, MKF_E_ARG, "tolerances must not be negative");
  *n_keep = 0;
  if (c->n_seeds == 0) return MKF_OK;
  const size_t N = (size_t)c->n_seeds, H = (size_t)std::max<int64_t>(c->n_hits, 1);
  // the duplicate-removal scratch serves here too (3 hits per seed)
  HIP_TRY(c, c->d_dup_h.ensure(sizeof(int) * 3 * N));
  HIP_TRY(c, c->d_clean_key.ensure(sizeof(float) * 3 * N));
  HIP_TRY(c, c->d_dup_cnt.ensure(sizeof(int) * H));
  HIP_TRY(c, c->d_dup_off.ensure(sizeof(int) * (H + 1)));
  HIP_TRY(c, c->d_dup_fill.ensure(sizeof(int) * H));
  HIP_TRY(c, c->d_dup_list.ensure(sizeof(int) * 3 * N));
  HIP_TRY(c, c->d_dup_tmp.ensure(sizeof(int) * (size_t)scan_tmp_words((int64_t)H)));
  HIP_TRY(c, c->d_dup_total.ensure(sizeof(int)));
  FindParams P = params(c);
  DevCleaning dc{cc->tol_ipt, cc->tol_eta, cc->tol_phi};
  launch_fill_i32(c->stream, c->d_dup_cnt.as<int>(), (int64_t)H, 0);
  launch_fill_i32(c->stream, c->d_dup_fill.as<int>(), (int64_t)H, 0);
  launch_fill_i32(c->stream, c->d_dup_total.as<int>(), 1, 0);
  launch_clean_prep(c->stream, P, c->d_seed_hits.as<int>(), c->d_dup_h.as<int>(),
                    c->d_clean_key.as<float>(), c->d_dup_cnt.as<int>());
  launch_scan(c->stream, c->d_dup_cnt.as<int>(), c->d_dup_off.as<int>(), (int64_t)H,
              c->d_dup_tmp.as<int>());
  launch_clean_fill(c->stream, P, c->d_dup_h.as<int>(), c->d_dup_off.as<int>(),
                    c->d_dup_fill.as<int>(), c->d_dup_list.as<int>());
  launch_clean_decide(c->stream, P, c->d_seed_hits.as<int>(), c->d_seed_chi2.as<float>(),
                      c->d_dup_h.as<int>(), c->d_clean_key.as<float>(), c->d_dup_off.as<int>(),
                      c->d_dup_list.as<int>(), dc, out_keep, c->d_dup_total.as<int>());
  HIP_TRY(c, hipGetLastError());
  int total = 0;
  HIP_TRY(c, hipMemcpyAsync(&total, c->d_dup_total.ptr, sizeof(int), hipMemcpyDeviceToHost,
                            c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  *n_keep = total;
  return MKF_OK;
}

mkf_status mkf_get_stats(mkf_ctx *c, mkf_stats *out) {
  if (!c || !out) return MKF_E_ARG;
  *out = c->stats;
  return MKF_OK;
}

}  // extern "C"

namespace {

bool tuning_ok(const mkf_ctx *c, const mkf_tuning &t) {
  return t.waves_per_simd >= 1 && t.waves_per_simd <= 4 && t.blocks_per_cu >= 1 &&
         t.blocks_per_cu <= 32 &&
         (t.lane_group == 0 || t.lane_group == 8 || (t.lane_group == 6 && c->cfg.n_cand <= 6)) &&
         t.phi_bin_shift >= -2 && t.phi_bin_shift <= 2 && t.q_bin_shift >= -2 &&
         t.q_bin_shift <= 2;
}

// Apply a tuning; a change of the binning rebuilds the layer records and
// the index of loaded hits.
mkf_status apply_tuning(mkf_ctx *c, const mkf_tuning &t) {
  const bool rebin =
      t.phi_bin_shift != c->tuning.phi_bin_shift || t.q_bin_shift != c->tuning.q_bin_shift;
  c->tuning = t;
  drop_graph(c);
  if (!rebin || c->n_layers == 0) return MKF_OK;
  mkf_status st = upload_layers(c);
  if (st == MKF_OK && c->stage >= kHits) st = build_index(c, HitArrays{});
  return st;
}

}  // namespace

extern "C" {

mkf_status mkf_set_tuning(mkf_ctx *c, const mkf_tuning *t) {
  if (!c) return MKF_E_ARG;
  if (!t || !tuning_ok(c, *t)) return fail(c, MKF_E_ARG, "tuning out of range");
  // the starting values set back, say with other bins, set no shape
  if (t->waves_per_simd != c->tuning.waves_per_simd || t->blocks_per_cu != c->tuning.blocks_per_cu)
    c->tuned = true;
  return apply_tuning(c, *t);
}

mkf_status mkf_get_tuning(mkf_ctx *c, mkf_tuning *t) {
  if (!c || !t) return MKF_E_ARG;
  *t = c->tuning;
  return MKF_OK;
}

mkf_status mkf_autotune(mkf_ctx *c, int32_t repeats, const char *cache_path, mkf_tuning *best) {
  if (!c) return MKF_E_ARG;
  if (c->stage < kSeeds) return fail(c, MKF_E_ORDER, "seed first");
  if (!(c->cfg.flags & MKF_F_BATCHED)) return fail(c, MKF_E_ARG, "autotune needs MKF_F_BATCHED");
  if (repeats < 1) return fail(c, MKF_E_ARG, "repeats must be >= 1");
  // workload key: architecture, compute units, kernel form, candidate
  // budget, sizes
  int lg = 0;
  while (((int64_t)1 << (lg + 1)) <= c->n_seeds) ++lg;
  const bool ext = c->mat.tab || c->field.on, sur = (c->cfg.flags & MKF_F_SURROGATE) != 0;
  const char *form = ext ? (sur ? "extended-surrogate" : "extended")
                         : (sur ? "surrogate" : "plain");
  char key[256];
  snprintf(key, sizeof key, "%s cu%d %s cand%d seeds2^%d events%d layers%d",
           c->arch.empty() ? "unknown" : c->arch.c_str(), c->n_cu, form, c->cfg.n_cand, lg,
           c->n_events, c->n_layers);
  if (cache_path) {
    if (FILE *f = fopen(cache_path, "r")) {
      char line[512];
      mkf_tuning hit{0, 0, 0, 0, 0};
      bool found = false;
      while (fgets(line, sizeof line, f)) {
        const size_t kl = strlen(key);
        mkf_tuning t{};
        if (strncmp(line, key, kl) == 0 && line[kl] == '\t' &&
            sscanf(line + kl + 1, "%d %d %d %d %d", &t.waves_per_simd, &t.blocks_per_cu,
                   &t.lane_group, &t.phi_bin_shift, &t.q_bin_shift) == 5 &&
            tuning_ok(c, t)) {
          hit = t;
          found = true;
        }
      }
      fclose(f);
      if (found) {
        c->tuned = true;
        mkf_status st = apply_tuning(c, hit);
        if (st == MKF_OK && best) *best = hit;
        return st;
      }
    }
  }
  const uint32_t flags = c->cfg.flags;
  c->cfg.flags &= ~MKF_F_GRAPH;  // time eager launches
  const mkf_tuning keep = c->tuning;
  const bool keep_tuned = c->tuned;
  c->tuned = true;
  mkf_tuning win = c->tuning;
  float win_ms = 1e30f;
  mkf_status st = MKF_OK;
  auto time_shape = [&](const mkf_tuning &t) -> mkf_status {
    mkf_status s2 = apply_tuning(c, t);
    if (s2 != MKF_OK) return s2;
    float ms = 1e30f;
    for (int r = 0; r < repeats; ++r) {
      s2 = mkf_find(c);
      if (s2 != MKF_OK) return s2;
      ms = std::min(ms, c->stats.main_ms);
    }
    if (ms < win_ms) {
      win_ms = ms;
      win = c->tuning;
    }
    return MKF_OK;
  };
  // launch shape at the current binning
  const int groups[2] = {6, 8};
  for (int gi = c->cfg.n_cand <= 6 ? 0 : 1; gi < 2 && st == MKF_OK; ++gi)
    for (int w = 1; w <= 4 && st == MKF_OK; ++w)
      for (int mult = 1; mult <= 2 && st == MKF_OK; ++mult)
        st = time_shape(mkf_tuning{w, w * mult, groups[gi], keep.phi_bin_shift, keep.q_bin_shift});
  // binning at that shape: phi and q bin counts x 2^s, s in -1..2 each
  const mkf_tuning shape = win;
  for (int sp = -1; sp <= 2 && st == MKF_OK; ++sp)
    for (int sq = -1; sq <= 2 && st == MKF_OK; ++sq) {
      if (sp == shape.phi_bin_shift && sq == shape.q_bin_shift) continue;
      mkf_tuning t = shape;
      t.phi_bin_shift = sp;
      t.q_bin_shift = sq;
      st = time_shape(t);
    }
  c->cfg.flags = flags;
  if (st != MKF_OK) {
    std::string e = c->err;
    (void)apply_tuning(c, keep);
    c->tuned = keep_tuned;
    c->err = e;
    return st;
  }
  st = apply_tuning(c, win);
  if (st != MKF_OK) return st;
  if (best) *best = win;
  if (cache_path) {
    if (FILE *f = fopen(cache_path, "a")) {
      fprintf(f, "%s\t%d %d %d %d %d %.4f\n", key, win.waves_per_simd, win.blocks_per_cu,
              win.lane_group, win.phi_bin_shift, win.q_bin_shift, win_ms);
      fclose(f);
    }
  }
  return MKF_OK;
}

}  // extern "C"

// ---- learned propagation surrogate

namespace {

// ascending distinct barrel radii of the loaded geometry
std::vector<float> barrel_radii(const mkf_ctx *c) {
  std::vector<float> r;
  for (int i = 0; i < c->n_layers; ++i)
    if (c->layers[i].kind == MKF_BARREL) r.push_back(c->layers[i].pos);
  std::sort(r.begin(), r.end());
  r.erase(std::unique(r.begin(), r.end()), r.end());
  return r;
}

mkf_status gen_samples(mkf_ctx *c, int64_t n, uint64_t seed, float *x, float *t, float *valid) {
  const std::vector<float> radii = barrel_radii(c);
  if (radii.size() < 2) return fail(c, MKF_E_GEOMETRY, "the sampler needs >= 2 barrel layers");
  HIP_TRY(c, c->d_radii.ensure(sizeof(float) * radii.size()));
  HIP_TRY(c, hipMemcpyAsync(c->d_radii.ptr, radii.data(), sizeof(float) * radii.size(),
                            hipMemcpyHostToDevice, c->stream));
  launch_mlp_datagen(c->stream, params(c), n, seed, c->d_radii.as<float>(), (int)radii.size(),
                     x, t, valid);
  HIP_TRY(c, hipGetLastError());
  return MKF_OK;
}

constexpr int64_t kMaxBatch = 1 << 20;

}  // namespace

extern "C" {

mkf_status mkf_surrogate_samples(mkf_ctx *c, int64_t n, uint64_t seed, float *x, float *t,
                                 float *valid) {
  if (!c) return MKF_E_ARG;
  if (c->stage < kGeometry) return fail(c, MKF_E_ORDER, "load_geometry first");
  if (n < 0 || (n > 0 && (!x || !t || !valid))) return fail(c, MKF_E_ARG, "bad sample buffers");
  if (n == 0) return MKF_OK;
  mkf_status st = gen_samples(c, n, seed, x, t, valid);
  if (st != MKF_OK) return st;
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  return MKF_OK;
}

mkf_status mkf_surrogate_train(mkf_ctx *c, const mkf_train_cfg *cfg, mkf_train_report *rep) {
  if (!c) return MKF_E_ARG;
  if (c->stage < kGeometry) return fail(c, MKF_E_ORDER, "load_geometry first");
  if (!cfg) return fail(c, MKF_E_ARG, "null training settings");
  if (cfg->batch < 64 || cfg->batch % 64 != 0 || cfg->batch > kMaxBatch)
    return fail(c, MKF_E_ARG, "batch must be a multiple of 64 in 64..%lld",
                (long long)kMaxBatch);
  if (cfg->n_samples < cfg->batch) return fail(c, MKF_E_ARG, "n_samples must be >= batch");
  if (cfg->epochs < 1) return fail(c, MKF_E_ARG, "epochs must be >= 1");
  if (!(cfg->lr > 0.f) || !finite_f(cfg->lr)) return fail(c, MKF_E_ARG, "lr must be > 0");
  for (int j = 0; j < kNO; ++j)
    if (!(cfg->loss_w[j] >= 0.f) || !finite_f(cfg->loss_w[j]))
      return fail(c, MKF_E_ARG, "loss weights must be finite and >= 0");
  const int64_t n = cfg->n_samples;
  const int64_t per_epoch = n / cfg->batch;
  const int64_t steps64 = per_epoch * cfg->epochs;
  if (steps64 > (1 << 24)) return fail(c, MKF_E_ARG, "too many training steps");
  const int steps = (int)steps64;
  if (cfg->first_step < 0 || cfg->first_step >= steps)
    return fail(c, MKF_E_ARG, "first_step %d outside the schedule's %d steps", cfg->first_step,
                steps);
  if (cfg->n_steps < 0 || cfg->n_steps > steps - cfg->first_step)
    return fail(c, MKF_E_ARG, "n_steps %d beyond the schedule's end", cfg->n_steps);
  if (cfg->first_step > 0 && c->mlp_step != cfg->first_step)
    return fail(c, MKF_E_ORDER, "the optimizer state is at step %d, not %d", c->mlp_step,
                cfg->first_step);
  const int s0 = cfg->first_step;
  const int s1 = cfg->n_steps ? s0 + cfg->n_steps : steps;
  const int run = s1 - s0;
  const int waves = cfg->batch / 64;
  HIP_TRY(c, c->d_tx.ensure(sizeof(float) * 8 * n));
  HIP_TRY(c, c->d_tt.ensure(sizeof(float) * 7 * n));
  HIP_TRY(c, c->d_tvalid.ensure(sizeof(float) * n));
  HIP_TRY(c, c->d_partial.ensure(sizeof(float) * (size_t)waves * (kNParam + 1)));
  HIP_TRY(c, c->d_partial2.ensure(sizeof(float) * (size_t)(waves / kReduceGroup + 1) *
                                  (kNParam + 1)));
  HIP_TRY(c, c->d_loss.ensure(sizeof(float) * run));
  HIP_TRY(c, hipEventRecord(c->ev_a, c->stream));
  mkf_status st = gen_samples(c, n, cfg->seed, c->d_tx.as<float>(), c->d_tt.as<float>(),
                              c->d_tvalid.as<float>());
  if (st != MKF_OK) return st;
  HIP_TRY(c, hipEventRecord(c->ev_b, c->stream));
  if (s0 == 0) {  // a run from its start has fresh moments
    HIP_TRY(c, hipMemsetAsync(c->d_mlp_m.ptr, 0, sizeof(float) * kNParam, c->stream));
    HIP_TRY(c, hipMemsetAsync(c->d_mlp_v.ptr, 0, sizeof(float) * kNParam, c->stream));
  }
  HIP_TRY(c, hipEventRecord(c->ev_m0, c->stream));
  const MlpBuffers B = mlp_buffers(c);
  const float lr_min = cfg->lr * 0.01f;
  for (int s = s0; s < s1; ++s) {
    const double u = steps > 1 ? (double)s / (steps - 1) : 0.0;
    const float lr = lr_min + 0.5f * (cfg->lr - lr_min) * (float)(1.0 + std::cos(M_PI * u));
    const int64_t begin = (s % per_epoch) * cfg->batch;
    launch_mlp_grad(c->stream, B.weights(), c->d_tx.as<float>(), c->d_tt.as<float>(),
                    c->d_tvalid.as<float>(), n, begin, cfg->batch, cfg->loss_w,
                    c->d_partial.as<float>());
    launch_mlp_reduce(c->stream, B, c->d_partial.as<float>(), waves, s + 1, lr, 1, nullptr,
                      c->d_loss.as<float>() + (s - s0), c->d_partial2.as<float>());
  }
  HIP_TRY(c, hipGetLastError());
  HIP_TRY(c, hipEventRecord(c->ev_m1, c->stream));
  std::vector<float> loss(run), valid(n);
  HIP_TRY(c, hipMemcpyAsync(loss.data(), c->d_loss.ptr, sizeof(float) * run,
                            hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(c, hipMemcpyAsync(valid.data(), c->d_tvalid.ptr, sizeof(float) * n,
                            hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  c->mlp_step = s1;
  if (rep) {
    float gen_ms = 0.f, train_ms = 0.f;
    HIP_TRY(c, hipEventElapsedTime(&gen_ms, c->ev_a, c->ev_b));
    HIP_TRY(c, hipEventElapsedTime(&train_ms, c->ev_m0, c->ev_m1));
    const int k = std::max(1, run / 100);
    double first = 0.0, last = 0.0;
    for (int i = 0; i < k; ++i) {
      first += loss[i];
      last += loss[run - k + i];
    }
    int64_t nv = 0;
    for (float v : valid) nv += v != 0.f;
    rep->steps = run;
    rep->loss_first = (float)(first / k);
    rep->loss_last = (float)(last / k);
    rep->datagen_ms = gen_ms;
    rep->train_ms = train_ms;
    rep->n_valid = nv;
  }
  return MKF_OK;
}

mkf_status mkf_surrogate_get(mkf_ctx *c, float *params) {
  if (!c) return MKF_E_ARG;
  if (!params) return fail(c, MKF_E_ARG, "null parameter buffer");
  HIP_TRY(c, hipMemcpyAsync(params, c->d_mlp_param.ptr, sizeof(float) * kNParam,
                            hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  return MKF_OK;
}

mkf_status mkf_surrogate_set(mkf_ctx *c, const float *params) {
  if (!c) return MKF_E_ARG;
  if (!params) return fail(c, MKF_E_ARG, "null parameter buffer");
  for (int i = 0; i < kNParam; ++i)
    if (!finite_f(params[i])) return fail(c, MKF_E_ARG, "parameter %d is not finite", i);
  HIP_TRY(c, hipMemcpyAsync(c->d_mlp_param.ptr, params, sizeof(float) * kNParam,
                            hipMemcpyHostToDevice, c->stream));
  HIP_TRY(c, hipMemsetAsync(c->d_mlp_m.ptr, 0, sizeof(float) * kNParam, c->stream));
  HIP_TRY(c, hipMemsetAsync(c->d_mlp_v.ptr, 0, sizeof(float) * kNParam, c->stream));
  launch_mlp_images(c->stream, mlp_buffers(c));
  HIP_TRY(c, hipGetLastError());
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  c->mlp_step = 0;
  return MKF_OK;
}

mkf_status mkf_surrogate_get_state(mkf_ctx *c, float *params, float *m, float *v,
                                   int32_t *step) {
  if (!c) return MKF_E_ARG;
  if (!params || !m || !v || !step) return fail(c, MKF_E_ARG, "null state buffer");
  HIP_TRY(c, hipMemcpyAsync(params, c->d_mlp_param.ptr, sizeof(float) * kNParam,
                            hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(c, hipMemcpyAsync(m, c->d_mlp_m.ptr, sizeof(float) * kNParam, hipMemcpyDeviceToHost,
                            c->stream));
  HIP_TRY(c, hipMemcpyAsync(v, c->d_mlp_v.ptr, sizeof(float) * kNParam, hipMemcpyDeviceToHost,
                            c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  *step = c->mlp_step;
  return MKF_OK;
}

mkf_status mkf_surrogate_set_state(mkf_ctx *c, const float *params, const float *m,
                                   const float *v, int32_t step) {
  if (!c) return MKF_E_ARG;
  if (!params || !m || !v) return fail(c, MKF_E_ARG, "null state buffer");
  if (step < 0) return fail(c, MKF_E_ARG, "step must be >= 0");
  for (int i = 0; i < kNParam; ++i) {
    if (!finite_f(params[i]) || !finite_f(m[i]) || !finite_f(v[i]))
      return fail(c, MKF_E_ARG, "state entry %d is not finite", i);
    if (v[i] < 0.f) return fail(c, MKF_E_ARG, "second moment %d is negative", i);
  }
  HIP_TRY(c, hipMemcpyAsync(c->d_mlp_param.ptr, params, sizeof(float) * kNParam,
                            hipMemcpyHostToDevice, c->stream));
  HIP_TRY(c, hipMemcpyAsync(c->d_mlp_m.ptr, m, sizeof(float) * kNParam, hipMemcpyHostToDevice,
                            c->stream));
  HIP_TRY(c, hipMemcpyAsync(c->d_mlp_v.ptr, v, sizeof(float) * kNParam, hipMemcpyHostToDevice,
                            c->stream));
  launch_mlp_images(c->stream, mlp_buffers(c));
  HIP_TRY(c, hipGetLastError());
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  c->mlp_step = step;
  return MKF_OK;
}

// Blob layout: the 4 bytes "MKFS", then uint32 version, uint32 parameter
// count, int32 Adam step, then the parameters, the first and the second
// moments (FP32, little-endian as in memory).
namespace {
constexpr uint32_t kBlobVersion = 1;
constexpr size_t kBlobHeader = 16;
constexpr size_t kBlobBytes = kBlobHeader + 3 * sizeof(float) * kNParam;
}  // namespace

mkf_status mkf_surrogate_save(mkf_ctx *c, void *buf, size_t cap, size_t *n) {
  if (!c) return MKF_E_ARG;
  if (!n) return fail(c, MKF_E_ARG, "n is NULL");
  *n = kBlobBytes;
  if (!buf || cap < kBlobBytes)
    return fail(c, MKF_E_CAPACITY, "the blob takes %zu bytes", kBlobBytes);
  std::vector<float> st(3 * (size_t)kNParam);
  int32_t step = 0;
  const mkf_status r = mkf_surrogate_get_state(c, st.data(), st.data() + kNParam,
                                               st.data() + 2 * kNParam, &step);
  if (r != MKF_OK) return r;
  unsigned char *b = static_cast<unsigned char *>(buf);
  const uint32_t ver = kBlobVersion, np = kNParam;
  memcpy(b, "MKFS", 4);
  memcpy(b + 4, &ver, 4);
  memcpy(b + 8, &np, 4);
  memcpy(b + 12, &step, 4);
  memcpy(b + kBlobHeader, st.data(), 3 * sizeof(float) * kNParam);
  return MKF_OK;
}

mkf_status mkf_surrogate_load(mkf_ctx *c, const void *buf, size_t n) {
  if (!c) return MKF_E_ARG;
  if (!buf) return fail(c, MKF_E_ARG, "buf is NULL");
  if (n != kBlobBytes) return fail(c, MKF_E_ARG, "a blob has %zu bytes, not %zu", kBlobBytes, n);
  const unsigned char *b = static_cast<const unsigned char *>(buf);
  uint32_t ver = 0, np = 0;
  int32_t step = 0;
  memcpy(&ver, b + 4, 4);
  memcpy(&np, b + 8, 4);
  memcpy(&step, b + 12, 4);
  if (memcmp(b, "MKFS", 4) != 0 || ver != kBlobVersion || np != (uint32_t)kNParam)
    return fail(c, MKF_E_ARG, "not a surrogate blob of this version and size");
  std::vector<float> st(3 * (size_t)kNParam);
  memcpy(st.data(), b + kBlobHeader, 3 * sizeof(float) * kNParam);
  return mkf_surrogate_set_state(c, st.data(), st.data() + kNParam, st.data() + 2 * kNParam,
                                 step);
}

mkf_status mkf_surrogate_grad(mkf_ctx *c, int32_t n, const float *x, const float *t,
                              const float *loss_w, float *grad, float *loss) {
  if (!c) return MKF_E_ARG;
  if (n < 64 || n % 64 != 0 || n > kMaxBatch)
    return fail(c, MKF_E_ARG, "n must be a multiple of 64 in 64..%lld", (long long)kMaxBatch);
  if (!x || !t || !loss_w || !grad || !loss) return fail(c, MKF_E_ARG, "null argument");
  for (int j = 0; j < kNO; ++j)
    if (!finite_f(loss_w[j])) return fail(c, MKF_E_ARG, "loss weights must be finite");
  const int waves = n / 64;
  HIP_TRY(c, c->d_partial.ensure(sizeof(float) * (size_t)waves * (kNParam + 1)));
  HIP_TRY(c, c->d_partial2.ensure(sizeof(float) * (size_t)(waves / kReduceGroup + 1) *
                                  (kNParam + 1)));
  HIP_TRY(c, c->d_grad.ensure(sizeof(float) * (kNParam + 1)));
  HIP_TRY(c, c->d_tvalid.ensure(sizeof(float) * n));
  launch_fill_i32(c->stream, c->d_tvalid.as<int>(), n, 0x3F800000);  // 1.0f
  launch_mlp_grad(c->stream, mlp_buffers(c).weights(), x, t, c->d_tvalid.as<float>(), n, 0, n,
                  loss_w, c->d_partial.as<float>());
  launch_mlp_reduce(c->stream, mlp_buffers(c), c->d_partial.as<float>(), waves, 1, 0.f, 0,
                    c->d_grad.as<float>(), c->d_grad.as<float>() + kNParam,
                    c->d_partial2.as<float>());
  HIP_TRY(c, hipGetLastError());
  HIP_TRY(c, hipMemcpyAsync(grad, c->d_grad.ptr, sizeof(float) * kNParam, hipMemcpyDeviceToHost,
                            c->stream));
  HIP_TRY(c, hipMemcpyAsync(loss, c->d_grad.as<float>() + kNParam, sizeof(float),
                            hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  return MKF_OK;
}

mkf_status mkf_surrogate_grad_noalloc(mkf_ctx *c, int32_t n, const float *x, const float *t,
                                      const float *loss_w, float *grad, float *loss) {
  if (!c) return MKF_E_ARG;
  if (n < 64 || n % 64 != 0)
    return fail(c, MKF_E_ARG, "n must be a positive multiple of 64");
  if (n > kNoAllocMaxSamples)
    return fail(c, MKF_E_CAPACITY, "n = %d exceeds the %d samples the fixed scratch holds", n,
                kNoAllocMaxSamples);
  if (!x || !t || !loss_w || !grad || !loss) return fail(c, MKF_E_ARG, "null argument");
  for (int j = 0; j < kNO; ++j)
    if (!finite_f(loss_w[j])) return fail(c, MKF_E_ARG, "loss weights must be finite");
  float *base = scratch_on(c->device);
  if (!base) return fail(c, MKF_E_HIP, "no scratch on device %d", c->device);
  float *partial = base, *partial2 = base + kNoAllocPartial;
  float *weight = partial2 + kNoAllocPartial2;
  const int waves = n / 64;
  launch_fill_i32(c->stream, reinterpret_cast<int *>(weight), n, 0x3F800000);  // 1.0f
  launch_mlp_grad(c->stream, mlp_buffers(c).weights(), x, t, weight, n, 0, n, loss_w, partial);
  launch_mlp_reduce(c->stream, mlp_buffers(c), partial, waves, 1, 0.f, 0, grad, loss, partial2);
  HIP_TRY(c, hipGetLastError());
  return MKF_OK;
}

mkf_status mkf_surrogate_infer(mkf_ctx *c, int64_t n, const float *x, float *y) {
  if (!c) return MKF_E_ARG;
  if (n < 0 || (n > 0 && (!x || !y))) return fail(c, MKF_E_ARG, "bad buffers");
  launch_mlp_infer(c->stream, mlp_buffers(c).weights(), n, x, y);
  HIP_TRY(c, hipGetLastError());
  HIP_TRY(c, hipStreamSynchronize(c->stream));
  return MKF_OK;
}

}  // extern "C"
