// mkf_kernels.hip -- gfx950 kernels of the Kalman-filter track finding and
// fitting hot path (arXiv:1811.04141).
//
//  hit index   : per (event, layer) phi x q bins, CSR over 32-byte records
//  seeding     : triplet helix, 3-hit Kalman fit, per-seed layer plan
//  find        : the clone engine (Introduction): every candidate of a seed
//                is propagated to the next plan layer, all its window hits
//                are scored by chi2, the seed's best extensions are chosen
//                across its lane group, and only the kept ones are updated.
//                One lane per candidate slot, a group of 6 lanes per seed
//                (10 seeds per wavefront) for budgets up to 6, else 8.
//                Two forms share the step code: one launch per layer step
//                with the state in HBM, or one persistent launch that keeps
//                the state in VGPRs across all steps of a seed tile.
//  finalize    : best candidate per seed, hit history from back-pointers
//  propagate / fit : unit propagation and search-free Kalman fitting.
#include <hip/hip_runtime.h>
#include <stddef.h>

#include <algorithm>
#include <cmath>

#include "mkf_kernels.hpp"
#include "mkf_quotient.hpp"

namespace mkf {

typedef unsigned long long u64;
constexpr u64 kKeyMax = ~0ull;
constexpr unsigned kOrderNone = 0x7FFFFFu;  // misses and skips sort after every hit

// Ranking key of an extension: more hits first, then smaller accumulated
// chi2, then parent rank, then hit index (miss/skip last).  A total order:
// ties cannot occur between different extensions.
//   bits 58..63: 63 - n_hits   bits 26..57: chi2 (non-negative float bits)
//   bits 23..25: parent slot   bits 0..22 : hit index or kOrderNone
__device__ __forceinline__ u64 ext_key(int nh, float chi2, int parent, unsigned order) {
  return ((u64)(63 - nh) << 58) | ((u64)__float_as_uint(chi2) << 26) | ((u64)parent << 23) |
         (u64)order;
}
// Key of a finished candidate when the seed's result is chosen: final
// candidates (by slot) come before retired ones (by step, then slot) on
// equal hits and chi2.
__device__ __forceinline__ u64 final_key(int nh, float chi2, int retired, int step, int slot) {
  return ((u64)(63 - nh) << 58) | ((u64)__float_as_uint(chi2) << 26) | ((u64)retired << 25) |
         ((u64)step << 19) | ((u64)slot << 16);
}
__device__ __forceinline__ int fkey_step(u64 k) { return (int)((k >> 19) & 63); }
__device__ __forceinline__ int fkey_slot(u64 k) { return (int)((k >> 16) & 7); }

__device__ __forceinline__ u64 shfl_xor_u64(u64 v, int m) {
  unsigned lo = (unsigned)v, hi = (unsigned)(v >> 32);
  lo = __shfl_xor(lo, m);
  hi = __shfl_xor(hi, m);
  return ((u64)hi << 32) | lo;
}
// lane i <- lane i ^ 1 and i ^ 2 within quads, by DPP (no trip through the
// LDS crossbar)
template <int kCtrl>
__device__ __forceinline__ u64 dpp_u64(u64 v) {
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)v, kCtrl, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(v >> 32), kCtrl, 0xF, 0xF, true);
  return ((u64)(unsigned)hi << 32) | (u64)(unsigned)lo;
}
constexpr int kDppXor1 = 0xB1;  // quad_perm(1, 0, 3, 2)
constexpr int kDppXor2 = 0x4E;  // quad_perm(2, 3, 0, 1)

__device__ __forceinline__ u64 shfl_u64(u64 v, int src) {
  unsigned lo = (unsigned)v, hi = (unsigned)(v >> 32);
  lo = __shfl(lo, src);
  hi = __shfl(hi, src);
  return ((u64)hi << 32) | lo;
}

// Lane groups of a seed: G consecutive lanes of a wavefront, one per
// candidate slot.  G = 8 (8 seeds per wave, any candidate budget) reduces
// with xor butterflies; G = 6 (10 seeds per wave, lanes 60-63 idle, for
// budgets up to 6) reduces over the three lane pairs by rotation.
template <int G> struct Grp;
template <> struct Grp<8> {
  static constexpr int kSeeds = 8;
  __device__ static int slot(int lane) { return lane & 7; }
  __device__ static int base(int lane) { return lane & ~7; }
  __device__ static u64 min(u64 v, int lane) {
    u64 o = dpp_u64<kDppXor1>(v);
    v = o < v ? o : v;
    o = dpp_u64<kDppXor2>(v);
    v = o < v ? o : v;
    o = shfl_xor_u64(v, 4);
    return o < v ? o : v;
  }
};
template <> struct Grp<6> {
  static constexpr int kSeeds = 10;
  __device__ static int slot(int lane) { return lane % 6; }
  __device__ static int base(int lane) { return lane - lane % 6; }
  // pairs (0,1) (2,3) (4,5); then the next pair's minimum, then the one
  // after (whose value already includes the first pair)
  __device__ static u64 min(u64 v, int lane) {
    const int sl = lane % 6, b = lane - sl;
    u64 o = dpp_u64<kDppXor1>(v);
    v = o < v ? o : v;
    o = shfl_u64(v, b + (sl < 4 ? sl + 2 : sl - 4));
    v = o < v ? o : v;
    o = shfl_u64(v, b + (sl < 2 ? sl + 4 : sl - 2));
    return o < v ? o : v;
  }
};

// Sorted insertion into a register list (compile-time indices only; keys
// are distinct, empty entries hold kKeyMax).  All comparisons with k come
// first; then entry i keeps its key if that is smaller than k, else takes k
// (where entry i - 1 is smaller) or entry i - 1's key (shifted up).  One
// compare per entry, none of them next to the selects that read it.
template <int N>
__device__ __forceinline__ void insert_sorted(u64 (&lst)[N], u64 k) {
  // the comparisons read a copy of k that the compiler cannot see through
  // (an empty statement, no instruction), so that it keeps one compare per
  // entry for both selects instead of forming a minimum and a maximum
  u64 kc = k;
  asm("" : "+v"(kc));
  bool below[N];
#pragma unroll
  for (int i = 0; i < N; ++i) below[i] = lst[i] < kc;
#pragma unroll
  for (int i = N - 1; i > 0; --i) lst[i] = below[i] ? lst[i] : (below[i - 1] ? k : lst[i - 1]);
  lst[0] = below[0] ? lst[0] : k;
}
// k into position n of a sorted list whose first n entries are all smaller
// than k and whose others are empty (nothing when n >= N): the insertion of
// a key that ranks after every key in the list, without comparisons
template <int N>
__device__ __forceinline__ void put_at(u64 (&lst)[N], int n, u64 k) {
#pragma unroll
  for (int i = 0; i < N; ++i) lst[i] = i == n ? k : lst[i];
}
template <int N>
__device__ __forceinline__ void pop_front(u64 (&lst)[N]) {
#pragma unroll
  for (int i = 0; i < N - 1; ++i) lst[i] = lst[i + 1];
  lst[N - 1] = kKeyMax;
}

__device__ __forceinline__ void stage_layers(const FindParams &P, DevLayer *sl) {
  for (int i = threadIdx.x; i < P.n_layers; i += blockDim.x) sl[i] = P.layers[i];
}

// Adds a wavefront's value of find counter k (every lane of the wave must
// call this; lanes with nothing to count pass 0).  Skipped when the whole
// wave has nothing.
__device__ __forceinline__ void add_counter(const FindParams &P, int k, int v) {
  if (__ballot(v != 0) == 0ull) return;
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) v += __shfl_xor(v, m);
  if ((threadIdx.x & 63) == 0)
    atomicAdd(&P.counters[k * kCounterSlots + blockIdx.x % kCounterSlots],
              (unsigned long long)v);
}

struct Cand {
  float p[6];
  float c[21];
  float chi2;
  int nh, nm;
  bool active;
};

// The kernels outside the find that fit (seeds, tracks, backwards, smoothing)
// come in two forms, as the find does: kExt with the material map and the
// parameterised field, and without, where the crossing is the helix's and the
// scattering angle constant.  The uniform form keeps the stepped crossing's and
// the map's registers out of the kernel (fit 163 -> 112, backward tail 134 -> 110,
// smoothing 204 -> 157, seeds 396 -> 310) and takes the angle's sine and cosine
// once: 1 million fits of 26 hits 557 -> 511 us, backward fit of 500,000 tracks 436
// -> 387 us (its FP64 part at two waves per SIMD, ten registers spilled; 414 at
// one), 500,000 seeds 418 -> 378 us.
template <bool kExt>
__device__ __forceinline__ const DevField *field_of(const DevCfg &cfg) {
  return kExt ? &cfg.field : nullptr;
}
inline bool extended(const DevCfg &cfg) { return cfg.mat.tab || cfg.field.on; }
// a crossed layer's material on the way out; sth, cth: sine and cosine of p's
// theta, at hand from the propagation, which leaves theta as it was
template <bool kExt, typename T>
__device__ __forceinline__ void layer_material(const DevCfg &cfg, int kind, T *p, T *c, T sth,
                                               T cth, T *j33 = nullptr, T *j35 = nullptr) {
  if constexpr (kExt) {
    material<T>(cfg, kind, p, c, T(1), j33, j35);
  } else {
    add_ms(p, T(cfg.ms_var), c, sth, cth);
    if (j33) *j33 = T(1);
    if (j35) *j35 = T(0);
  }
}

__device__ __forceinline__ int clampi(int v, int lo, int hi) { return v < lo ? lo : (v > hi ? hi : v); }

// ------------------------------------------------------------ records
//
// Per-seed records a find keeps besides the candidates: the back-pointers
// of every step and the best retired candidate.  The layer-synchronous form
// keeps them in HBM by position; the persistent form keeps them in the
// wavefront's LDS for the seed tile it is working on.
struct GlobalRec {
  const FindParams *P;
  int64_t pos;
  __device__ void put_bp(int step, int slot, int v) const {
    P->bp[((size_t)step * (size_t)P->n_seeds + pos) * P->slots + slot] = v;
  }
  __device__ void put_fin(const Cand &cd) const {
    const size_t N = (size_t)P->n_seeds;
#pragma unroll
    for (int i = 0; i < 6; ++i) P->fin_rec[i * N + pos] = cd.p[i];
#pragma unroll
    for (int i = 0; i < 21; ++i) P->fin_rec[(6 + i) * N + pos] = cd.c[i];
    P->fin_rec[27 * N + pos] = cd.chi2;
    P->fin_meta[pos] = cd.nh | (cd.nm << 8);
  }
  __device__ void get_fin(float *p, float *c, float &chi2, int &meta) const {
    const size_t N = (size_t)P->n_seeds;
    for (int i = 0; i < 6; ++i) p[i] = P->fin_rec[i * N + pos];
    for (int i = 0; i < 21; ++i) c[i] = P->fin_rec[(6 + i) * N + pos];
    chi2 = P->fin_rec[27 * N + pos];
    meta = P->fin_meta[pos];
  }
};

struct LdsRec {
  int *bp;       // this seed's back-pointers: step s, slot j at bp[s * stride + j]
  int stride;
  float *fin;    // this seed's best retired candidate [kFinWords]
  __device__ void put_bp(int step, int slot, int v) const { bp[step * stride + slot] = v; }
  __device__ int get_bp(int step, int slot) const { return bp[step * stride + slot]; }
  __device__ void put_fin(const Cand &cd) const {
#pragma unroll
    for (int i = 0; i < 6; ++i) fin[i] = cd.p[i];
#pragma unroll
    for (int i = 0; i < 21; ++i) fin[6 + i] = cd.c[i];
    fin[27] = cd.chi2;
    fin[28] = __int_as_float(cd.nh | (cd.nm << 8));
  }
  __device__ void get_fin(float *p, float *c, float &chi2, int &meta) const {
    for (int i = 0; i < 6; ++i) p[i] = fin[i];
    for (int i = 0; i < 21; ++i) c[i] = fin[6 + i];
    chi2 = fin[27];
    meta = __float_as_int(fin[28]);
  }
};

// ---------------------------------------------------------------- window
//
// Bounding box of the chi2 < cut ellipse of every hit on the layer: with
// S_hit <= H C H^T + diag(var_max), |u| <= sqrt(cut S_uu) and |v| <= sqrt(cut
// S_vv).  Barrel: u = R_h sin(dphi) (hits in the same half), v = dz, so
// |dphi| <= asin(s) <= s / sqrt(1 - s^2) with s = du / R.  Disk: the hit is at
// (r' + v) rh + u t, so its radius lies in [r' - dv, sqrt((r' + dv)^2 +
// du^2)] and its azimuth within atan(du / (r' - dv)) <= du / (r' - dv).  The
// box only has to contain the ellipse (the chi2 test decides), so these
// cheaper upper bounds replace asin and atan; a small margin absorbs FP32
// rounding of the bin assignment.  Hits are read four at a time from one
// base address (the sorted array is padded past its end) so that their
// loads overlap.
// Azimuth of (x, y) for the window centre only, within 1e-6 rad (the
// window adds that to its margin): octant reduction, then atan(a) = a P(a^2)
// on [0, 1] with a degree-7 polynomial fitted to atan (largest error 1.3e-7
// rad including FP32 evaluation), the ratio taken with the hardware
// reciprocal.
__device__ __forceinline__ float window_azimuth(float y, float x) {
  const float ax = fabsf(x), ay = fabsf(y);
  const float mx = fmaxf(ax, ay), mn = fminf(ax, ay);
  const float a = mx > 0.f ? mn * __builtin_amdgcn_rcpf(mx) : 0.f;
  const float s = a * a;
  float r = -0.004054667f;
  r = fmaf(r, s, 0.021863315f);
  r = fmaf(r, s, -0.055912834f);
  r = fmaf(r, s, 0.096422337f);
  r = fmaf(r, s, -0.139086440f);
  r = fmaf(r, s, 0.199465677f);
  r = fmaf(r, s, -0.333298624f);
  r = fmaf(r, s, 0.999999344f);
  r *= a;
  if (ay > ax) r = 0.5f * kPi - r;
  if (x < 0.f) r = kPi - r;
  return copysignf(r, y);
}

// chi2 of a window hit, with the hardware reciprocal (1 ulp) in place of a
// correctly rounded division; both forms of the find score hits with it
__device__ __forceinline__ float chi2_hit(const Frame &f, float vu, float vv, float vuv, float u,
                                          float v) {
  const float suu = f.suu + vu, svv = f.svv + vv, suv = f.suv + vuv;
  const float det = fmaf(suu, svv, -suv * suv);
  return (svv * u * u - 2.f * suv * u * v + suu * v * v) * __builtin_amdgcn_rcpf(det);
}

// The window's bins: q rows qlo..qhi of the event's layer (base: the index
// of its first bin) and up to two azimuth segments per row, [seg[0],
// seg[1]] and [seg[2], seg[3]] (the second empty unless the window wraps).
__device__ __forceinline__ void window_bins(const FindParams &P, const DevLayer &L, int ev,
                                            const Prop &pr, const Frame &f, int &base, int &qlo,
                                            int &qhi, int (&seg)[4]) {
  const float cut = P.cfg.chi2_cut;
  // (hardware square roots, 1 ulp: the 0.1% widening covers them)
  const float du = __builtin_amdgcn_sqrtf(cut * (f.suu + L.vu_max)) * 1.001f + 1e-5f;
  const float dv = __builtin_amdgcn_sqrtf(cut * (f.svv + L.vv_max)) * 1.001f + 1e-5f;
  const float phic = window_azimuth(pr.p[1], pr.p[0]);
  float dphi, qmin, qmax;
  if (L.kind == 0) {
    // (hardware reciprocals below: the 1e-5 and 1e-4 widenings cover their ulp)
    const float s = du * __builtin_amdgcn_rcpf(L.pos * 0.99999f);
    dphi = s >= 0.99f ? kPi : s * rsqrtf(fmaf(-s, s, 1.f)) * 1.0001f;
    qmin = pr.p[2] - dv;
    qmax = pr.p[2] + dv;
  } else {
    const float r = __builtin_amdgcn_sqrtf(fmaf(pr.p[0], pr.p[0], pr.p[1] * pr.p[1]));
    const float rl = r - dv;
    qmin = rl;
    qmax = __builtin_amdgcn_sqrtf(fmaf(r + dv, r + dv, du * du));
    dphi = rl > 0.f ? fminf(du * __builtin_amdgcn_rcpf(rl) * 1.0001f, kPi) : kPi;
  }
  dphi += 6e-6f;
  qmin -= 1e-4f;
  qmax += 1e-4f;
  const int nphi = L.nphi;
  qlo = clampi((int)floorf((qmin - L.q_lo) * L.q_scale), 0, L.nq - 1);
  qhi = clampi((int)floorf((qmax - L.q_lo) * L.q_scale), 0, L.nq - 1);
  seg[0] = 0;
  seg[1] = nphi - 1;
  seg[2] = 1;
  seg[3] = 0;
  if (dphi < kPi) {
    const int blo = (int)floorf((phic - dphi + kPi) * L.phi_scale);
    const int bhi = (int)floorf((phic + dphi + kPi) * L.phi_scale);
    if (bhi - blo + 1 < nphi) {
      if (blo < 0) {
        seg[0] = blo + nphi; seg[1] = nphi - 1; seg[2] = 0; seg[3] = bhi;
      } else if (bhi >= nphi) {
        seg[0] = blo; seg[1] = nphi - 1; seg[2] = 0; seg[3] = bhi - nphi;
      } else {
        seg[0] = blo; seg[1] = bhi;
      }
    }
  }
  base = ev * P.bins_per_event + L.bin_base;
}

// One window hit against a candidate's prediction (point p, frame f): its
// chi2 (>= 0), or a negative value for a hit on the other half of a barrel.
__device__ __forceinline__ float hit_chi2(const float *p, const Frame &f, int kind,
                                          const float4 &a, const float4 &b) {
  float u, v;
  if (!residual(p, f, kind, a.x, a.y, a.z, u, v)) return -1.f;
  return fmaxf(chi2_hit(f, a.w, b.x, b.z, u, v), 0.f);
}

// A hit's chi2 within this band of the cut is a decision that rounding may
// take either way (the band of the parity checks: 1e-3 relative + 1e-2).
__device__ __forceinline__ float near_cut_band(float cut) { return fmaf(1e-3f, cut, 1e-2f); }

__device__ __forceinline__ float lane_value(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}

// A window of more than kWideBins bins or kWideRows rows (a candidate whose
// state is poorly measured: its window may span the whole layer) is scanned by
// the lanes that are here together; alone its lane would hold up the others for
// hundreds of hits.  Below the line a lane is done in one or two passes of four
// hits, about what the hand-over costs; lines at 24 bins and 3 rows and at 128
// and 8 measured within 1.5% of this one.
//
// Lanes that scan by themselves do so at the same time, windows scanned together
// come one after the other, and only the lanes with a live candidate that crosses
// the layer are here: one of 6 or 8 at a seed's first step, fewer in a small
// call.  So at most one lane in kWideShare hands its window over; where more are
// above the line, it rises by factors of four until only the widest are.  At 30 and
// 10 times the usual scattering and cuts of 30 and 200, layer form: 64 seeds 749 to
// 439 us (no hand-over 422), 5,000 seeds 2.30 to 1.26 ms (3.48), 64 and 5,000 seeds
// of the persistent form 522 to 285 and 986 to 446 us, against handing over all of
// them.  Shares of 4 and 16: 465 and 399 us, 1.40 and 2.09 ms, 284 and 232 us, 437
// and 677 us; the usual windows are the same up to 12 and 5% slower at 16.
constexpr int kWideBins = 48, kWideRows = 5, kWideShare = 8;

// The scan of lane o's window by every lane that is here: the lanes look up
// one run of bins each, then score the runs' hits one per lane; compatible hits
// go to lane o's list.  Lane o's values are read into scalar registers, so
// that this costs the kernels no more than two vector registers.  Bound, like
// the lane's own scan, by the latency of the run bounds and of the hits, here
// paid once per as many of them as lanes are here.  Find kernel without and with
// it: 2 events x 5,000 seeds 0.250 and 0.104 ms, 4 events x 28,000 triplet seeds
// 0.565 and 0.456 ms, 100 events x 5,000 seeds 1.56 and 1.40 ms (3 waves per SIMD);
// without it single tiles of 10 seeds took up to 500 us and the launch ended on
// them.
template <int N>
__device__ __forceinline__ void scan_wide(const FindParams &P, const DevLayer &L, int o,
                                          const Prop &pr, const Frame &f, float chi2_base, int nh,
                                          int slot, int base, int qlo, int qhi,
                                          const int (&seg)[4], u64 (&lst)[N], int &n_ext,
                                          int &n_near) {
  const float cut = P.cfg.chi2_cut;
  const float band = near_cut_band(cut);
  const float4 *hits = reinterpret_cast<const float4 *>(P.sorted);
  const unsigned long long here = __ballot(true);
  const int lane = threadIdx.x & 63, n_here = __popcll(here);
  const int rank = __builtin_amdgcn_mbcnt_hi((unsigned)(here >> 32),
                                             __builtin_amdgcn_mbcnt_lo((unsigned)here, 0u));
  const float op[3] = {lane_value(pr.p[0], o), lane_value(pr.p[1], o), lane_value(pr.p[2], o)};
  const Frame of{lane_value(f.tx, o),  lane_value(f.ty, o),  lane_value(f.rx, o),
                 lane_value(f.ry, o),  lane_value(f.suu, o), lane_value(f.suv, o),
                 lane_value(f.svv, o)};
  const int okind = __builtin_amdgcn_readlane(L.kind, o);
  const int onh = __builtin_amdgcn_readlane(nh, o);
  const int oslot = __builtin_amdgcn_readlane(slot, o);
  const float ochi2 = lane_value(chi2_base, o);
  const int onphi = __builtin_amdgcn_readlane(L.nphi, o);
  const int oqlo = __builtin_amdgcn_readlane(qlo, o);
  const int orow = __builtin_amdgcn_readlane(base, o) + oqlo * onphi;
  const int rows = __builtin_amdgcn_readlane(qhi, o) - oqlo + 1;
  const int s0 = __builtin_amdgcn_readlane(seg[0], o), s1 = __builtin_amdgcn_readlane(seg[1], o);
  const int s2 = __builtin_amdgcn_readlane(seg[2], o), s3 = __builtin_amdgcn_readlane(seg[3], o);
  const int runs = s2 <= s3 ? 2 * rows : rows;  // the second azimuth segments after the first
  for (int r0 = 0; r0 < runs; r0 += n_here) {
    int h0 = 0, h1 = 0;
    if (r0 + rank < runs) {
      const bool second = r0 + rank >= rows;
      const int row = orow + (second ? r0 + rank - rows : r0 + rank) * onphi;
      h0 = P.bin_start[row + (second ? s2 : s0)];
      h1 = P.bin_start[row + (second ? s3 : s1) + 1];
    }
    for (unsigned long long m = __ballot(h1 > h0); m != 0ull; m &= m - 1) {
      const int src = __ffsll(m) - 1;
      const int k1 = __builtin_amdgcn_readlane(h1, src);
      for (int k0 = __builtin_amdgcn_readlane(h0, src); k0 < k1; k0 += n_here) {
        const int k = k0 + rank;
        float c2 = -1.f;
        unsigned order = 0;
        if (k < k1) {
          const float4 a = hits[2 * (size_t)k], b = hits[2 * (size_t)k + 1];
          c2 = hit_chi2(op, of, okind, a, b);
          order = (unsigned)__float_as_int(b.y);
          n_near += fabsf(c2 - cut) <= band ? 1 : 0;
        }
        for (unsigned long long pm = __ballot(c2 >= 0.f && c2 < cut); pm != 0ull; pm &= pm - 1) {
          const int from = __ffsll(pm) - 1;
          const float pc2 = lane_value(c2, from);
          const unsigned po = (unsigned)__builtin_amdgcn_readlane((int)order, from);
          if (lane == o) {
            insert_sorted(lst, ext_key(onh + 1, ochi2 + pc2, oslot, po));
            ++n_ext;
          }
        }
      }
    }
  }
}

// The window scan of the lanes that are here: every hit of a lane's window, by
// the lane itself, four at a time, or by all of them (scan_wide).  n_near counts
// the hits whose chi2 lies within near_cut_band of the cut, in the lane that
// scored them.
template <int N>
__device__ __forceinline__ void scan_window(const FindParams &P, const DevLayer &L, int ev,
                                            const Prop &pr, const Frame &f, float chi2_base,
                                            int nh, int slot, u64 (&lst)[N], int &n_ext,
                                            int &n_near) {
  const float cut = P.cfg.chi2_cut;
  const float band = near_cut_band(cut);
  int base, qlo, qhi, seg[4];
  window_bins(P, L, ev, pr, f, base, qlo, qhi, seg);
  const int rows = qhi - qlo + 1;
  const int width = seg[1] - seg[0] + 1 + max(seg[3] - seg[2] + 1, 0);
  const int bins = rows * width;
  bool wide = rows > kWideRows || bins > kWideBins;
  unsigned long long wides = __ballot(wide);
  if (__builtin_expect(wides != 0ull, 0)) {
    const int n_here = __popcll(__ballot(true));
    for (int line = 4 * kWideBins; kWideShare * __popcll(wides) > n_here; line *= 4) {
      wide = bins > line;
      wides = __ballot(wide);
    }
    for (; wides != 0ull; wides &= wides - 1)
      scan_wide(P, L, __ffsll(wides) - 1, pr, f, chi2_base, nh, slot, base, qlo, qhi, seg, lst,
                n_ext, n_near);
    if (wide) qhi = qlo - 1;
  }
  for (int qb = qlo; qb <= qhi; ++qb) {
    const int row = base + qb * L.nphi;
#pragma unroll
    for (int sg = 0; sg < 2; ++sg) {
      const int lo = seg[2 * sg], hi = seg[2 * sg + 1];
      if (lo > hi) continue;
      const int h0 = P.bin_start[row + lo];
      const int h1 = P.bin_start[row + hi + 1];
      const float4 *hits = reinterpret_cast<const float4 *>(P.sorted);
      for (int k = h0; k < h1; k += 4) {
        // records k .. k + 3 from one base address: past the bin's last
        // hit they are the next bin's hits or the array's padding records
        // (kHitPad), read and not used
        const float4 *hk = hits + 2 * (size_t)k;
        float4 a[4];
        float4 b[4];  // (var_v, index, covariance uv, -)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          a[j] = hk[2 * j];
          b[j] = hk[2 * j + 1];
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          if (k + j >= h1) break;
          const float c2 = hit_chi2(pr.p, f, L.kind, a[j], b[j]);
          n_near += fabsf(c2 - cut) <= band ? 1 : 0;
          if (c2 >= 0.f && c2 < cut) {
            insert_sorted(lst, ext_key(nh + 1, chi2_base + c2, slot,
                                       (unsigned)__float_as_int(b[j].y)));
            ++n_ext;
          }
        }
      }
    }
  }
}

// ------------------------------------------------------------ one step
//
// One layer step of one seed, executed by its G-lane group.  On entry each
// lane holds one candidate (or none); on exit it holds the candidate of its
// rank among the kept extensions.  pos indexes the seed's find buffers.
// cnt: the lane's counters, cnt[0] near-cut chi2 decisions, and with kMat
// cnt[1] Runge-Kutta steps and cnt[2] Newton iterations of field crossings.
template <int G, bool kMat, class Rec>
__device__ __forceinline__ void group_step(const FindParams &P, const DevLayer *sl, Cand &cd,
                                           int lane, int slot, const Rec &rec, int ev,
                                           int64_t ev_base, int step, int lid, u64 &fin_key,
                                           int *cnt, float l_hint = 0.f,
                                           int *sur = nullptr, const float2 *mtab = nullptr,
                                           const float *trig = nullptr) {
  const DevLayer &L = sl[lid];
  Prop pr;
  int st = kNoCrossing;
  if (cd.active)
    st = propagate<true, float>(cd.p, cd.c, L, P.cfg.mkb, P.cfg.l_min, true, P.cfg.edge_margin, pr,
                                l_hint, sur, nullptr, kMat ? &P.cfg.field : nullptr, trig,
                                kMat ? cnt + 1 : nullptr);
  const bool ok = cd.active && st == kOk;
  // kMat: the material map's effects and the parameterised field (a separate
  // instantiation, so that the constant-angle uniform-field form keeps its
  // register allocation)
  if (ok) {
    if constexpr (kMat) material<float>(P.cfg, L.kind, pr.p, pr.c, 1.f, nullptr, nullptr, mtab);
    else add_ms(pr.p, P.cfg.ms_var, pr.c, pr.sth, pr.cth);
  }

  u64 lst[G];  // this lane's best extensions (G >= n_cand)
#pragma unroll
  for (int i = 0; i < G; ++i) lst[i] = kKeyMax;
  int n_ext = 0;
  if (cd.active) {
    if (!ok) {
      lst[0] = ext_key(cd.nh, cd.chi2, slot, kOrderNone);  // skip (the list is empty)
      n_ext = 1;
    } else {
      Frame f;
      make_frame(pr.p, pr.c, L.kind, f);
      scan_window(P, L, ev, pr, f, cd.chi2, cd.nh, slot, lst, n_ext, cnt[0]);
      if (cd.nm < P.cfg.max_holes) {
        // a miss has one hit fewer than each of the n_ext hit extensions, so
        // it ranks after all of them
        put_at(lst, n_ext, ext_key(cd.nh, cd.chi2, slot, kOrderNone));
        ++n_ext;
      }
    }
  }

  // a candidate without any extension stops; keep the seed's best such one
  // (the group reductions below are skipped, wave-uniformly, once no lane
  // of the wavefront has anything left to contribute)
  const bool retire = cd.active && n_ext == 0;
  if (__ballot(retire) != 0ull) {
    const u64 rkey = retire ? final_key(cd.nh, cd.chi2, 1, step, slot) : kKeyMax;
    const u64 rmin = Grp<G>::min(rkey, lane);
    if (rmin < fin_key) {
      if (rkey == rmin) rec.put_fin(cd);
      fin_key = rmin;
    }
  }

  // the seed's best n_cand extensions, rank r goes to slot r (the last
  // round's winner stays on its list, which is not read again)
  u64 mine = kKeyMax;
  const int n_cand = P.cfg.n_cand;
  for (int r = 0; r < n_cand; ++r) {
    if (__ballot(lst[0] != kKeyMax) == 0ull) break;
    const u64 m = Grp<G>::min(lst[0], lane);
    if (slot == r) mine = m;
    if (r + 1 == n_cand) break;
    if (m != kKeyMax && lst[0] == m) pop_front(lst);
  }

  // the kept hit's record is requested first, so that its latency overlaps
  // the state exchange below
  const unsigned order = mine != kKeyMax ? (unsigned)(mine & 0x7FFFFFu) : kOrderNone;
  float4 ha = make_float4(0.f, 0.f, 0.f, 0.f), hb = ha;
  if (order != kOrderNone) {
    const float4 *hr = reinterpret_cast<const float4 *>(P.byorig + ev_base + order);
    ha = hr[0];
    hb = hr[1];  // (vv, index, vuv, -)
  }

  // children read their parent's propagated state (or, for a skip, its
  // unpropagated state) across the group
  // (a candidate whose propagation failed hands on its unpropagated state;
  // the selects are skipped, wave-uniformly, when no lane has one: lanes
  // without a candidate are never chosen as parents)
  float src[27];
#pragma unroll
  for (int i = 0; i < 6; ++i) src[i] = pr.p[i];
#pragma unroll
  for (int i = 0; i < 21; ++i) src[6 + i] = pr.c[i];
  if (__ballot(cd.active && !ok) != 0ull) {
#pragma unroll
    for (int i = 0; i < 6; ++i) src[i] = ok ? pr.p[i] : cd.p[i];
#pragma unroll
    for (int i = 0; i < 21; ++i) src[6 + i] = ok ? pr.c[i] : cd.c[i];
  }
  const int src_meta = cd.nh | (cd.nm << 8) | (ok ? (1 << 16) : 0);
  const int parent = mine == kKeyMax ? slot : (int)((mine >> 23) & 7);
  const int src_lane = Grp<G>::base(lane) + parent;
  float np[27];
#pragma unroll
  for (int i = 0; i < 27; ++i) np[i] = __shfl(src[i], src_lane);
  const int pmeta = __shfl(src_meta, src_lane);

  int bpv = -1;
  if (mine != kKeyMax) {
    int nh = pmeta & 0xFF, nm = (pmeta >> 8) & 0xFF;
    const bool pok = (pmeta >> 16) & 1;
    int hitcode;
    if (order != kOrderNone) {
      const float hx = ha.x, hy = ha.y, hz = ha.z, vu = ha.w, vv = hb.x, vuv = hb.z;
      Frame f;
      make_frame(np, np + 6, L.kind, f);
      float u, v;
      residual(np, f, L.kind, hx, hy, hz, u, v);
      kf_update(np, np + 6, f, L.kind, vu, vv, vuv, u, v);
      ++nh;
      hitcode = (int)order;
    } else if (pok) {
      ++nm;
      hitcode = -1;
    } else {
      hitcode = -2;
    }
#pragma unroll
    for (int i = 0; i < 6; ++i) cd.p[i] = np[i];
#pragma unroll
    for (int i = 0; i < 21; ++i) cd.c[i] = np[6 + i];
    cd.chi2 = __uint_as_float((unsigned)(mine >> 26));
    cd.nh = nh;
    cd.nm = nm;
    cd.active = true;
    bpv = ((hitcode + 2) << 3) | parent;
  } else {
    cd.active = false;
  }
  rec.put_bp(step, slot, bpv);
}

// A seed's state; its record's last word, the index of its event's first
// hit, is returned.
__device__ __forceinline__ int load_seed(const FindParams &P, int64_t pos, Cand &cd) {
  // one seed's 28 words are contiguous: seven 16-byte loads
  const float4 *src = reinterpret_cast<const float4 *>(P.pstate + (size_t)pos * kSeedWords);
  float w[28];
#pragma unroll
  for (int k = 0; k < 7; ++k) {
    const float4 v = src[k];
    w[4 * k] = v.x;
    w[4 * k + 1] = v.y;
    w[4 * k + 2] = v.z;
    w[4 * k + 3] = v.w;
  }
#pragma unroll
  for (int i = 0; i < 6; ++i) cd.p[i] = w[i];
#pragma unroll
  for (int i = 0; i < 21; ++i) cd.c[i] = w[6 + i];
  cd.chi2 = 0.f;
  cd.nh = 3;
  cd.nm = 0;
  return __float_as_int(w[27]);
}

// A candidate slot's state and its meta word (hits, misses, active) as
// stored by store_cand.  The state words are requested together with the
// meta word, not after it, so that their latencies overlap (an empty
// slot's words are read and not used); the meta word is returned raw and
// unpacked by set_meta where it is first needed.
__device__ __forceinline__ int load_cand_raw(const FindParams &P, size_t idx, Cand &cd) {
  const size_t NS = (size_t)P.n_seeds * P.slots;
  const int meta = __float_as_int(P.cand[28 * NS + idx]);
#pragma unroll
  for (int i = 0; i < 6; ++i) cd.p[i] = P.cand[i * NS + idx];
#pragma unroll
  for (int i = 0; i < 21; ++i) cd.c[i] = P.cand[(6 + i) * NS + idx];
  cd.chi2 = P.cand[27 * NS + idx];
  return meta;
}
__device__ __forceinline__ void set_meta(Cand &cd, int meta) {
  cd.active = (meta >> 16) & 1;
  cd.nh = meta & 0xFF;
  cd.nm = (meta >> 8) & 0xFF;
}
__device__ __forceinline__ void load_cand(const FindParams &P, size_t idx, Cand &cd) {
  set_meta(cd, load_cand_raw(P, idx, cd));
}

__device__ __forceinline__ void store_cand(const FindParams &P, size_t idx, const Cand &cd) {
  const size_t NS = (size_t)P.n_seeds * P.slots;
  const int meta = cd.nh | (cd.nm << 8) | (cd.active ? (1 << 16) : 0);
  P.cand[28 * NS + idx] = __int_as_float(meta);
  if (cd.active) {
#pragma unroll
    for (int i = 0; i < 6; ++i) P.cand[i * NS + idx] = cd.p[i];
#pragma unroll
    for (int i = 0; i < 21; ++i) P.cand[(6 + i) * NS + idx] = cd.c[i];
    P.cand[27 * NS + idx] = cd.chi2;
  }
}

// The chosen candidate of a seed: state and counts, and its hit history
// followed back through the per-step back-pointers from (best_step,
// best_slot).  Plan steps after the candidate stopped read MKF_HIT_NONE.
__device__ __forceinline__ int *write_state(const FindParams &P, int64_t pos, const float *p,
                                           const float *c, float chi2, int nh, int nm) {
  float *out = P.out + (size_t)pos * kOutWords;
  float w[kOutHit];
#pragma unroll
  for (int i = 0; i < 6; ++i) w[kOutPar + i] = p[i];
#pragma unroll
  for (int i = 0; i < 21; ++i) w[kOutCov + i] = c[i];
  w[kOutChi2] = chi2;
  w[kOutMeta] = __int_as_float(nh | (nm << 8));
#pragma unroll
  for (int i = kOutMeta + 1; i < kOutHit; ++i) w[i] = 0.f;
#pragma unroll
  for (int k = 0; k < kOutHit / 4; ++k)
    reinterpret_cast<float4 *>(out)[k] =
        make_float4(w[4 * k], w[4 * k + 1], w[4 * k + 2], w[4 * k + 3]);
  return reinterpret_cast<int *>(out + kOutHit);
}

template <class Rec>
__device__ __forceinline__ void write_result(const FindParams &P, int64_t pos, const Rec &rec,
                                             const float *p, const float *c, float chi2, int nh,
                                             int nm, int best_step, int best_slot, int plen) {
  int *hit = write_state(P, pos, p, c, chi2, nh, nm);
  for (int s = plen - 1; s > best_step; --s) hit[s] = MKF_HIT_NONE;
  int sl = best_slot;
  for (int s = best_step; s >= 0; --s) {
    const int v = rec.get_bp(s, sl);
    hit[s] = (v >> 3) - 2;
    sl = v & 7;
  }
}

template <class Rec>
__device__ __forceinline__ void write_retired(const FindParams &P, int64_t pos, const Rec &rec,
                                              u64 fin, int plen) {
  float p[6], c[21], chi2;
  int fm;
  rec.get_fin(p, c, chi2, fm);
  write_result(P, pos, rec, p, c, chi2, fm & 0xFF, (fm >> 8) & 0xFF, fkey_step(fin) - 1,
               fkey_slot(fin), plen);
}

template <class Rec>
__device__ __forceinline__ void write_empty(const FindParams &P, int64_t pos, const Rec &rec) {
  const float z[21] = {};
  write_result(P, pos, rec, z, z, 0.f, 0, 0, -1, 0, 0);
}

// --------------------------------------------------- layer-synchronous form

__global__ __launch_bounds__(256) void k_find_init(FindParams P) {
  const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t pos = gid / P.slots;
  const int slot = (int)(gid % P.slots);
  if (pos >= P.n_seeds) return;
  Cand cd;
  cd.active = slot == 0 && ((P.pinfo[pos] >> 8) & 1);
  cd.nh = 3;
  cd.nm = 0;
  cd.chi2 = 0.f;
  if (cd.active) load_seed(P, pos, cd);
  store_cand(P, (size_t)pos * P.slots + slot, cd);
  if (slot == 0) P.fin_key[pos] = kKeyMax;
}

// One layer step of the layer-synchronous form: G-lane seed groups,
// Grp<G>::kSeeds seeds per wavefront (lanes 60-63 idle for G = 6).
// (the uniform-field form is compiled for four waves per SIMD, which its
// load latency needs; the extended form would spill far more there)
template <bool kMat, int G>
__global__ __launch_bounds__(256, kMat ? 1 : 4) void k_find_step(FindParams P, int step,
                                                                 int64_t n_active) {
  __shared__ DevLayer sl[kMaxLayers];
  // XCD x (blocks x, x + 8, ...) takes the x-th contiguous share of the
  // positions, so that an XCD's L2 serves a few events' hits
  // (the grid is a multiple of kQueues blocks, so this is a permutation)
  const int64_t per = gridDim.x / kQueues;
  const int64_t b = (int64_t)(blockIdx.x % kQueues) * per + blockIdx.x / kQueues;
  const int lane = threadIdx.x & 63;
  const int grp = lane / G;
  const int64_t pos = (b * 4 + (threadIdx.x >> 6)) * Grp<G>::kSeeds + grp;
  const int slot = Grp<G>::slot(lane);
  // a seed group takes part while the step is in its plan (the whole group
  // leaves together); the wave stays to add its counters.  The positions
  // below n_active are the seeds whose plans are longer than step (the
  // host orders the seeds longest plan first), so every word the step
  // starts from is requested at once, without waiting for the plan length,
  // and before the block stages the layer table.
  const bool in_range = grp < Grp<G>::kSeeds && pos < n_active;
  // (the plan length is the low byte of the seed's info word, read as a
  // byte so that nothing waits on it before the barrier)
  int meta = 0, plen = 0, lid = 0, ev = 0;
  u64 fin_key = kKeyMax;
  Cand cd;
  if (in_range) {
    meta = load_cand_raw(P, (size_t)pos * G + slot, cd);
    fin_key = P.fin_key[pos];
    plen = reinterpret_cast<const unsigned char *>(P.pinfo)[4 * pos];
    lid = P.pplan[(size_t)pos * kMaxPlan + step];
    ev = P.pevent[pos];
  }
  stage_layers(P, sl);
  __syncthreads();
  if (__ballot(in_range) == 0ull) return;
  set_meta(cd, meta);
  const bool live = in_range && step < plen;
  int cnt[3] = {0, 0, 0};
  if (live) {
    const u64 fk0 = fin_key;
    group_step<G, kMat>(P, sl, cd, lane, slot, GlobalRec{&P, pos}, ev, P.ev_off[ev], step, lid,
                        fin_key, cnt);
    store_cand(P, (size_t)pos * G + slot, cd);
    if (slot == 0 && fin_key != fk0) P.fin_key[pos] = fin_key;
  }
  add_counter(P, kCntNearCut, cnt[0]);
  if constexpr (kMat) {
    add_counter(P, kCntRk, cnt[1]);
    add_counter(P, kCntNewton, cnt[2]);
  }
}

// Block of the kernels that take one lane per track through its surfaces: one
// wavefront.  Their calls are often smaller than the chip (20,000 tracks are 316
// wavefronts for 1,024 SIMDs), and blocks of four put them on a third of the
// CUs.  Against blocks of 256, 20,000 tracks: forward smoothing 59 to 54 us,
// backward 100 to 82, results 29 to 26; 500,000 tracks: the backward fit's
// head 148 to 140, its tail 235 to 234.
constexpr int kTrackBlock = 64;
constexpr int64_t kManyTracks = 1 << 18;  // tracks above which smoothing takes blocks of 256

// Best of the final and the retired candidates of each seed (more hits,
// then smaller chi2) and the count of candidate-layer steps (1 for the seed
// at step 0, then every kept extension carried into the next step).  One
// lane per seed.
//
// The back-pointer rows of eight steps are requested at once, counted, and
// followed in registers: read one by one, 78 words for the count and then a
// chain of a load per step were waited for in turn (20,000 seeds of 14 steps: 26
// us, now 17).
template <int G>
__global__ __launch_bounds__(kTrackBlock) void k_finalize(FindParams P) {
  constexpr int kRows = 8;
  __shared__ unsigned long long block_steps;
  if (threadIdx.x == 0) block_steps = 0;
  __syncthreads();
  const int64_t pos = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (pos < P.n_seeds) {
    const int info = P.pinfo[pos];
    const int plen = info & 0xFF;
    const bool ok = (info >> 8) & 1;
    const size_t N = (size_t)P.n_seeds;
    const size_t NS = N * G;
    int cnt = (ok && plen > 0) ? 1 : 0;
    u64 m = kKeyMax;
    int best = 0;
    if (ok)
#pragma unroll
      for (int j = 0; j < G; ++j) {
        const int meta = __float_as_int(P.cand[28 * NS + pos * G + j]);
        if (!((meta >> 16) & 1)) continue;
        const u64 fk = final_key(meta & 0xFF, P.cand[27 * NS + pos * G + j], 0, 0, j);
        if (fk < m) {
          m = fk;
          best = j;
        }
      }
    const u64 fin = ok ? P.fin_key[pos] : kKeyMax;
    const bool live = m != kKeyMax && m < fin;
    const bool retired = !live && fin != kKeyMax;
    int last = -1, sl = 0;  // the best candidate's last step and its slot there
    int *hit;
    if (live) {
      Cand cd;
      load_cand(P, (size_t)pos * G + best, cd);
      hit = write_state(P, pos, cd.p, cd.c, cd.chi2, cd.nh, cd.nm);
      last = plen - 1;
      sl = best;
    } else if (retired) {
      float p[6], c[21], chi2;
      int fm;
      GlobalRec{&P, pos}.get_fin(p, c, chi2, fm);
      hit = write_state(P, pos, p, c, chi2, fm & 0xFF, (fm >> 8) & 0xFF);
      last = fkey_step(fin) - 1;
      sl = fkey_slot(fin);
    } else {
      const float z[21] = {};
      hit = write_state(P, pos, z, z, 0.f, 0, 0);
    }
    for (int s0 = (plen - 1) & ~(kRows - 1); s0 >= 0 && plen > 0; s0 -= kRows) {
      int v[kRows][G], h[kRows];
#pragma unroll
      for (int i = 0; i < kRows; ++i) {
        const int2 *row =
            reinterpret_cast<const int2 *>(P.bp + ((size_t)min(s0 + i, plen - 1) * N + pos) * G);
#pragma unroll
        for (int j = 0; j < G / 2; ++j) {
          const int2 w = row[j];
          v[i][2 * j] = w.x;
          v[i][2 * j + 1] = w.y;
        }
      }
#pragma unroll
      for (int i = kRows - 1; i >= 0; --i) {
        const int s = s0 + i;
        int w = v[i][0];
#pragma unroll
        for (int j = 0; j < G; ++j) {
          cnt += s + 1 < plen && v[i][j] >= 0;
          if (j == sl) w = v[i][j];
        }
        h[i] = MKF_HIT_NONE;
        if (s <= last) {
          h[i] = (w >> 3) - 2;
          sl = w & 7;
        }
      }
      // (words past the plan's end are never read)
      if (live || retired) {
#pragma unroll
        for (int i = 0; i < kRows; i += 4)
          *reinterpret_cast<int4 *>(hit + s0 + i) = make_int4(h[i], h[i + 1], h[i + 2], h[i + 3]);
      }
    }
    if (cnt) atomicAdd(&block_steps, (unsigned long long)cnt);
  }
  __syncthreads();
  if (threadIdx.x == 0 && block_steps) atomicAdd(P.n_steps, block_steps);
}

// ----------------------------------------------------- persistent form
//
// Each wavefront claims tiles of 8 seeds from a counter and carries them
// through all their layer steps with the candidates in VGPRs; the seed's
// result is chosen in registers at the end.  Only the hit index, the
// back-pointers and the results touch memory.

// kWaves: the occupancy the register allocation targets (waves per SIMD);
// more waves hide more latency but spill part of the state to scratch.
// The autotuner picks the instantiation.
// kSurr: barrel propagations start from the learned surrogate's path length
// (one wave-wide matrix-core inference per layer step, then one exact Newton
// step per lane, falling back to the closed form when it does not converge).
// G: lanes per seed (8, or 6 for candidate budgets up to 6).
// kMat: with the material map and/or the parameterised field (constant
// scattering angle and uniform field otherwise).
template <int kWaves, bool kSurr, int G, bool kMat>
__device__ __forceinline__ void find_persistent(const FindParams &P) {
  __shared__ DevLayer sl[kMaxLayers];
  __shared__ unsigned long long block_steps;
  // surrogate: the network's BF16 weight images and biases, shared by the
  // block, and one activation tile per wave (the input tile overlays it)
  constexpr int kW1n = 64 * kLdW1, kW2n = 64 * kLdW2, kW3n = 32 * kLdW3;
  __shared__ __attribute__((aligned(16))) __bf16 sMW[kSurr ? kW1n + kW2n + kW3n : 8];
  __shared__ __attribute__((aligned(16))) float sMB[kSurr ? 64 + 64 + 32 : 4];
  // (one sample row per seed: at most 10 rows, one 16-sample tile per wave)
  __shared__ __attribute__((aligned(16))) __bf16 sMH[kSurr ? 4 * 16 * kLdH : 8];
  // material: a table of up to kMatLds bins is read from LDS
  constexpr int kMatLds = 1024;
  __shared__ float2 sMat[kMat ? kMatLds : 1];
  const float2 *mtab = nullptr;
  if constexpr (kMat) {
    const int nb = P.cfg.mat.nr * P.cfg.mat.nz;
    if (P.cfg.mat.tab && nb <= kMatLds) {
      for (int i = threadIdx.x; i < nb; i += blockDim.x) sMat[i] = P.cfg.mat.tab[i];
      mtab = sMat;
    }
  }
  stage_layers(P, sl);
  MlpWeights mw{};
  if constexpr (kSurr) {
    const int4 *g1 = reinterpret_cast<const int4 *>(P.mlp.W1p);
    const int4 *g2 = reinterpret_cast<const int4 *>(P.mlp.W2p);
    const int4 *g3 = reinterpret_cast<const int4 *>(P.mlp.W3p);
    int4 *d = reinterpret_cast<int4 *>(sMW);
    for (int i = threadIdx.x; i < kW1n / 8; i += blockDim.x) d[i] = g1[i];
    for (int i = threadIdx.x; i < kW2n / 8; i += blockDim.x) d[kW1n / 8 + i] = g2[i];
    for (int i = threadIdx.x; i < kW3n / 8; i += blockDim.x) d[(kW1n + kW2n) / 8 + i] = g3[i];
    for (int i = threadIdx.x; i < 64; i += blockDim.x) {
      sMB[i] = P.mlp.b1[i];
      sMB[64 + i] = P.mlp.b2[i];
      if (i < 32) sMB[128 + i] = P.mlp.b3[i];
    }
    mw = MlpWeights{sMW, sMW + kW1n, sMW + kW1n + kW2n, nullptr, nullptr, sMB, sMB + 64, sMB + 128};
  }
  if (threadIdx.x == 0) {
    block_steps = 0;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int slot = Grp<G>::slot(lane);
  const int grp = lane / G;  // G = 6: lanes 60-63 form no seed group
  const int wv = threadIdx.x >> 6;
  // this wave's records in dynamic LDS: back-pointers [max_plan][kSeeds][G],
  // then the retired records [kSeeds][kFinWords]
  extern __shared__ int s_rec[];
  constexpr int kS = Grp<G>::kSeeds;
  int *wrec = s_rec + wv * persistent_rec_words(P.max_plan, G, kS);
  const int gi = grp < kS ? grp : 0;
  const LdsRec rec{wrec + gi * G, kS * G,
                   reinterpret_cast<float *>(wrec + P.max_plan * kS * G) + gi * kFinWords};
  int my_steps = 0, my_acc = 0, my_fb = 0;
  int cnt[3] = {0, 0, 0};  // near-cut decisions, field Runge-Kutta steps, Newton iterations
  int q = blockIdx.x % kQueues;  // this block's XCD
  // Queue k: positions queue_at(k) .. queue_at(k + 1) - 1.  (Equal runs, against
  // every eighth tile: 4 events of 28,000 triplet seeds 0.46 and 0.48 ms, 8
  // events of 5,000 seeds 0.185 and 0.203 ms, 100 such events 1.39 and 1.41 ms.)
  auto queue_at = [&](int k) { return P.n_seeds * k / kQueues; };
  int64_t q_lo = queue_at(q), q_hi = queue_at(q + 1);
  // A queue's first n_static tiles belong to the waves of its XCD, one each,
  // and need no claim; the counter hands out the tiles after them (the grid
  // is a multiple of kQueues blocks).
  const int n_static = gridDim.x / kQueues * (blockDim.x >> 6);
  // the next tile of queue q is claimed one tile ahead, so that the atomic's
  // latency overlaps the current tile's work (lane 0 holds it; -1: none)
  int ahead = blockIdx.x / kQueues * (blockDim.x >> 6) + wv;
  for (;;) {
    // (ahead is wave-uniform: a tile claimed ahead needs no wait here, so
    // the previous tile's result stores drain while this one starts)
    int64_t start = ahead >= 0 ? q_lo + (int64_t)ahead * Grp<G>::kSeeds : q_hi;
    ahead = -1;
    if (start >= q_hi) {
      // Queue exhausted: take a tile of the next queue that has one left.
      // All counters are read in one load, and only a queue that has tiles
      // left is asked (trying every queue with an atomic cost 750 us per
      // find on events of 200 and of 5,000 seeds: 65,000 atomics to one cache
      // line; with this, static first tiles and a grid no larger than the
      // tiles, 86 and 169 us; 500,000 seeds 1.73 -> 1.51 ms).  A counter never
      // falls, so the loop ends when every queue reads as handed out.
      const int qi = lane % kQueues;
      const int64_t lo_i = queue_at(qi), hi_i = queue_at(qi + 1);
      for (;;) {
        const int c = __hip_atomic_load(&P.tile_counter[qi * kTilePad], __ATOMIC_RELAXED,
                                        __HIP_MEMORY_SCOPE_AGENT);
        const bool left = lane < kQueues && lo_i + ((int64_t)n_static + c) * Grp<G>::kSeeds < hi_i;
        const unsigned m = (unsigned)__ballot(left);
        if (m == 0u) break;
        // the first such queue after this wave's own
        const unsigned rot = ((m | m << kQueues) >> (q + 1)) & ((1u << kQueues) - 1u);
        q = (q + 1 + __builtin_ctz(rot)) % kQueues;
        q_lo = queue_at(q);
        q_hi = queue_at(q + 1);
        int t = 0;
        if (lane == 0) t = atomicAdd(&P.tile_counter[q * kTilePad], 1);
        t = __builtin_amdgcn_readfirstlane(t);
        start = q_lo + ((int64_t)n_static + t) * Grp<G>::kSeeds;
        if (start < q_hi) break;
      }
      if (start >= q_hi) break;
    }
    const int64_t end = q_hi;
    // (no claim ahead where the queue's tiles were all dealt out statically)
    if (lane == 0 && start + Grp<G>::kSeeds < end &&
        q_lo + (int64_t)n_static * Grp<G>::kSeeds < end)
      ahead = n_static + atomicAdd(&P.tile_counter[q * kTilePad], 1);
    const int64_t pos = start + grp;
    const bool valid = grp < Grp<G>::kSeeds && pos < end;
    // Every lane reads the words of an existing seed (lanes past the tile
    // read its last one and use none of it), without branches, so that the
    // seed's info word, event, state and first plan words are all requested
    // before the first wait; a seed without a fit has its state read and
    // not used.
    const int64_t pc = valid ? pos : end - 1;
    const int info_w = P.pinfo[pc];
    const int ev_w = P.pevent[pc];
    Cand cd;
    const int ev_base_w = load_seed(P, pc, cd);
    // the plan is read four layer ids at a time, one word ahead
    const int *plan_w = reinterpret_cast<const int *>(P.pplan) + (size_t)pc * (kMaxPlan / 4);
    int w_cur = plan_w[0];
    int w_next = plan_w[1];
    const int info = valid ? info_w : 0;
    const int ev = valid ? ev_w : 0;
    const int64_t ev_base = valid ? (int64_t)ev_base_w : 0;
    const int plen = info & 0xFF;
    cd.active = valid && slot == 0 && ((info >> 8) & 1);
    cd.nh = 3;
    cd.nm = 0;
    cd.chi2 = 0.f;
    u64 fin_key = kKeyMax;
    // the tile's longest plan (at most kMaxPlan = 32 steps), by a binary
    // search over ballots: no round trips through the LDS crossbar.  At
    // least one step is taken (a step beyond every plan does nothing), so
    // that the loads above are not deferred behind a test for an empty
    // tile.
    int maxlen = 1;
#pragma unroll
    for (int b = 32; b >= 1; b >>= 1)
      if (__ballot(plen >= maxlen + b) != 0ull) maxlen += b;
    // the tile claimed ahead is read now: its atomic was issued before this
    // tile's loads, so it has returned with the info word
    ahead = __builtin_amdgcn_readfirstlane(__shfl(ahead, 0));
    for (int step = 0; step < maxlen; ++step) {
      const bool in_plan = step < plen;
      if (step > 0 && (step & 3) == 0) {
        w_cur = w_next;
        w_next = step + 4 < plen ? plan_w[step / 4 + 1] : 0;
      }
      const int lid = in_plan ? (w_cur >> (8 * (step & 3))) & 0xFF : 0;
      float l_hint = 0.f;
      float trig[4];  // sin, cos of phi and theta, shared by the inputs and the propagation
      if constexpr (kSurr) {
        // The candidates of a seed all head to the same layer from nearby
        // states: the network predicts the path of the seed's leading
        // candidate (slot 0), one sample row per seed, and every candidate
        // applies that relative correction to its own straight-line path
        // and checks it with its own Newton step (falling back to the
        // closed form when the check fails).
        // (the sines and cosines are taken for every candidate that steps,
        // barrel or disk, and always handed to the propagation: a pointer
        // chosen per lane would keep the array in scratch memory)
        const bool want = in_plan && cd.active && sl[lid].kind == 0;
        const bool lead = want && slot == 0;
        float xin[kNI];
        if (in_plan && cd.active) {
          sincosf(cd.p[4], &trig[0], &trig[1]);
          sincosf(cd.p[5], &trig[2], &trig[3]);
        }
        if (lead) {
          mlp_inputs(cd.p, trig, sl[lid].pos, P.cfg.mkb, xin);
        } else {
#pragma unroll
          for (int k = 0; k < kNI; ++k) xin[k] = 0.f;
        }
        // the leading candidates write their inputs to consecutive sample
        // rows (at most 10 per wavefront: one 16-sample tile); no inference
        // at all when none heads to a barrel layer
        const unsigned long long m = __ballot(lead);
        if (m != 0ull) {
          const int base = Grp<G>::base(lane);
          const unsigned long long below = base ? (m & ((1ull << base) - 1ull)) : 0ull;
          const int row = __popcll(below);  // this seed's sample row
          __bf16 *H = sMH + wv * 16 * kLdH;
          __bf16 *X = H;  // the input tile overlays the activation tile
          if (lead) {
            bf16x8 xv;
#pragma unroll
            for (int k = 0; k < kNI; ++k) xv[k] = (__bf16)xin[k];
            *reinterpret_cast<bf16x8 *>(X + row * kLdX) = xv;
          }
          wave_sync();
          f32x4 y;
          mlp_forward16(mw, X, H, y);
          const float y0 = mlp_output16(y, row, 0);
          wave_sync();  // the tiles are rewritten at the next step
          if (want) l_hint = surrogate_path(cd.p, trig, sl[lid].pos, P.cfg.mkb, y0);
        }
      }
      if (in_plan) {
        my_steps += cd.active ? 1 : 0;
        int sur = 0;
        group_step<G, kMat>(P, sl, cd, lane, slot, rec, ev, ev_base, step, lid, fin_key, cnt,
                            l_hint, &sur, mtab, kSurr ? trig : nullptr);
        my_acc += sur == 1;
        my_fb += sur == 2;
      }
    }
    wave_sync();  // the group's records were written by its other lanes
    if (valid) {
      const u64 fk = cd.active ? final_key(cd.nh, cd.chi2, 0, 0, slot) : kKeyMax;
      const u64 m = Grp<G>::min(fk, lane);
      if (m != kKeyMax && m < fin_key) {
        if (fk == m)
          write_result(P, pos, rec, cd.p, cd.c, cd.chi2, cd.nh, cd.nm, plen - 1, slot, plen);
      } else if (slot == 0) {
        if (fin_key != kKeyMax) write_retired(P, pos, rec, fin_key, plen);
        else write_empty(P, pos, rec);
      }
    }
    wave_sync();  // read before the next tile overwrites them
  }
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) my_steps += __shfl_xor(my_steps, m);
  if (lane == 0 && my_steps) atomicAdd(&block_steps, (unsigned long long)my_steps);
  if constexpr (kSurr) {
    add_counter(P, kCntSurKept, my_acc);
    add_counter(P, kCntSurRejected, my_fb);
  }
  add_counter(P, kCntNearCut, cnt[0]);
  if constexpr (kMat) {
    add_counter(P, kCntRk, cnt[1]);
    add_counter(P, kCntNewton, cnt[2]);
  }
  __syncthreads();
  if (threadIdx.x == 0 && block_steps) atomicAdd(P.n_steps, block_steps);
}

template <int kWaves, bool kSurr, int G>
__global__ __launch_bounds__(256, kWaves) void k_find_persistent(FindParams P) {
  find_persistent<kWaves, kSurr, G, false>(P);
}

template <int kWaves, bool kSurr, int G>
__global__ __launch_bounds__(256, kWaves) void k_find_persistent_mat(FindParams P) {
  find_persistent<kWaves, kSurr, G, true>(P);
}

// The seeds' results into processing order, so that every read of the find is
// by position.  Nine lanes per seed, 16 bytes each: seven of the state row,
// two of the plan.  Bound by HBM: 2 x 164 B per seed, the writes in runs of 112
// and 32 B.  500,000 seeds: 56 us (2.9 TB/s); one lane per seed, gathering 27 words from
// 27 arrays, took 418 us.
__global__ __launch_bounds__(256) void k_place_seeds(FindParams P, const int2 *cell_rank,
                                                     const int *cell_start, int *order,
                                                     int *pos_of, float4 *pstate, int *pinfo,
                                                     int *pevent, int4 *pplan) {
  constexpr int kState = kSeedWords / 4, kPlan = kMaxPlan / 16;
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t i = id / (kState + kPlan);
  const int k = (int)(id - i * (kState + kPlan));
  if (i >= P.n_seeds) return;
  const int2 cr = cell_rank[i];
  const int64_t pos = cell_start[cr.x] + cr.y;
  if (k < kState) {
    pstate[pos * kState + k] = reinterpret_cast<const float4 *>(P.seed_state)[i * kState + k];
  } else {
    pplan[pos * kPlan + k - kState] =
        reinterpret_cast<const int4 *>(P.plan)[i * kPlan + k - kState];
  }
  if (k == 0) {
    order[pos] = (int)i;
    pos_of[i] = (int)pos;
    pinfo[pos] = P.plan_len[i] | (P.seed_ok[i] << 8);
    pevent[pos] = P.seed_event[i];
  }
}

// The caller's track records, in seed order, written by the device straight
// into pinned host memory: one lane per 32-bit word, so that a wavefront reads
// words of one result row and writes 256 contiguous bytes.  Bound by the link
// to the host: 46 GB/s with the host's copies behind it, of the 57 GB/s that a
// plain copy to pinned memory reaches.
__global__ __launch_bounds__(256) void k_tracks(FindParams P, const int *pos_of, int64_t first,
                                                int64_t n, int *out) {
  static_assert(offsetof(mkf_track, par) == 24 && offsetof(mkf_track, cov) == 48 &&
                offsetof(mkf_track, plan) == 132 && offsetof(mkf_track, hit) == 164 &&
                sizeof(mkf_track) == 292, "record layout");
  constexpr int kPar = 6, kPlan = 33, kHit = 41;  // words
  const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t i = id / kTrackWords;
  const int w = (int)(id - i * kTrackWords);
  if (i >= n) return;
  const int seed = (int)(first + i);
  const int64_t pos = pos_of[seed];
  const int *row = reinterpret_cast<const int *>(P.out + (size_t)pos * kOutWords);
  const int info = P.pinfo[pos];
  const int ok = (info >> 8) & 1, plen = ok ? info & 0xFF : 0;
  int v;
  if (w >= kHit) {
    v = w - kHit < plen ? row[kOutHit + w - kHit] : MKF_HIT_NONE;
  } else if (w >= kPlan) {
    const int k = 4 * (w - kPlan);  // four layer ids, those past the plan's end -1
    v = -1;
    if (k < plen) {
      v = reinterpret_cast<const int *>(P.pplan + (size_t)pos * kMaxPlan)[w - kPlan];
      if (plen - k < 4) v |= (int)(~0u << (8 * (plen - k)));
    }
  } else if (w >= kPar) {
    v = row[kOutPar + w - kPar];  // (cov follows par in both)
  } else if (w == 5) {
    v = row[kOutChi2];
  } else if (w == 4) {
    v = plen;
  } else if (w >= 2) {
    v = (row[kOutMeta] >> (w == 2 ? 0 : 8)) & 0xFF;
  } else {
    v = w == 1 ? ok : seed;
  }
  out[id] = v;
}

// --------------------------------------------------------------- seeding
//
// Seeds come from outside (Section 2.2).  The circle through the three
// transverse points gives the centre and radius, the turning sense the
// charge, the tangent at the first hit phi, and the z rise over the arc
// theta.  A wide diagonal prior at the first hit is filtered through the
// three hits.  The layer plan is the paper's per-region list of layers to
// traverse (Section 2.1): with region steering, the list of the region that
// holds the seed's pseudorapidity, less the seed layers; without, it is built
// per seed: every other layer the seed helix crosses inside its widened
// extent, by increasing path length.
//
// Two kernels.  k_seed fits, one lane per seed, one wavefront per block; its 21
// covariances in FP64 leave it one wave per SIMD, bound by the latency of the
// FP64 chain.  k_seed_plan takes the crossings, four or eight lanes per seed, each
// with its share of the layers: few registers, many waves, and a chain of a few
// crossings instead of 25.  The whole of the seeding kernels: 200 seeds 23 us, 5,000
// 34 us, against 27 and 46 in one kernel with one lane per seed; 500,000 seeds 129 us
// of fit and 201 us of plans against 378.
constexpr int kSeedBlock = 64;
constexpr int kFewPlans = 24576;  // seeds up to which a plan has eight lanes

__global__ __launch_bounds__(256) void k_validate_seeds(FindParams P, const int *seed_event,
                                                        const int *seed_hits, int *bad) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P.n_seeds) return;
  const int ev = seed_event[i];
  bool good = ev >= 0 && ev < P.n_events;
  if (good) {
    const int64_t nh = P.ev_off[ev + 1] - P.ev_off[ev];
    for (int k = 0; k < 3; ++k) {
      const int h = seed_hits[3 * i + k];
      good = good && h >= 0 && h < nh;
    }
  }
  if (!good) *bad = 1;
}

template <bool kExt>
__global__ __launch_bounds__(kSeedBlock) void k_seed(
    FindParams P, const int *src_event, const int *src_hits, int *seed_event, int *seed_hits,
    float *seed_state, int *seed_ok, float *seed_chi2, double *fit) {
  __shared__ DevLayer sl[kMaxLayers];
  stage_layers(P, sl);
  __syncthreads();
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P.n_seeds) return;
  const int ev = src_event[i];
  const int64_t e0 = P.ev_off[ev];
  int sh[3];
  for (int k = 0; k < 3; ++k) sh[k] = src_hits[3 * i + k];
  if (src_event != seed_event) {
    seed_event[i] = ev;
    for (int k = 0; k < 3; ++k) seed_hits[3 * i + k] = sh[k];
  }
  // FP64: three updates shrink the wide prior by ~5 decades, more than FP32
  // keeps in C - K S K^T; the result is rounded to FP32 for the find
  double hx[3], hy[3], hz[3], hvu[3], hvv[3];
  int hl[3];
  for (int k = 0; k < 3; ++k) {
    const int64_t g = e0 + sh[k];
    const HitRec h = P.byorig[g];
    const float2 var = P.raw ? P.raw[g] : make_float2(h.vu, h.vv);
    hx[k] = h.x;
    hy[k] = h.y;
    hz[k] = h.z;
    hvu[k] = var.x;
    hvv[k] = var.y;
    hl[k] = h.layer;
  }
  const double mkb = P.cfg.mkb, l_min = P.cfg.l_min;
  int ok = 0;
  double p[6], c[21], chi2 = 0.0;
  do {
    const double ax = hx[1] - hx[0], ay = hy[1] - hy[0];
    const double bx = hx[2] - hx[0], by = hy[2] - hy[0];
    const double d = 2.0 * (ax * by - ay * bx);
    if (d == 0.0 || mkb == 0.0) break;
    const double a2 = ax * ax + ay * ay, b2 = bx * bx + by * by;
    const double ux = (by * a2 - ay * b2) / d;
    const double uy = (ax * b2 - bx * a2) / d;
    const double cx = hx[0] + ux, cy = hy[0] + uy;
    const double rho = sqrt(ux * ux + uy * uy);
    const double turn = (hx[1] - hx[0]) * (hy[2] - hy[1]) - (hy[1] - hy[0]) * (hx[2] - hx[1]);
    const bool ccw = turn > 0.0;  // omega > 0
    // omega = mkb * ipt and |omega| = 1/rho; a parameterised field is taken
    // at the middle hit
    const double mkb_s = kExt && P.cfg.field.on ? field_mkb(P.cfg.field, hx[1], hy[1], hz[1]) : mkb;
    if (mkb_s == 0.0) break;
    const double ipt = (ccw ? 1.0 : -1.0) / (mkb_s * rho);
    const double r1x = hx[0] - cx, r1y = hy[0] - cy;
    const double dirx = ccw ? -r1y : r1y, diry = ccw ? r1x : -r1x;
    const double phi1 = atan2(diry, dirx);
    const double r3x = hx[2] - cx, r3y = hy[2] - cy;
    const double dpsi = atan2(r1x * r3y - r1y * r3x, r1x * r3x + r1y * r3y);
    const double theta = atan2(rho * fabs(dpsi), hz[2] - hz[0]);
    p[0] = hx[0]; p[1] = hy[0]; p[2] = hz[0]; p[3] = ipt; p[4] = phi1; p[5] = theta;
    surface_prior(P.cfg, p, sl[hl[0]].kind, c);
    chi2 = 0.0;
    bool good = true;
    for (int k = 0; k < 3 && good; ++k) {
      const DevLayer &L = sl[hl[k]];
      if (k > 0) {
        PropT<double> pr;
        if (propagate<true, double>(p, c, L, mkb, l_min, false, 0.0, pr, 0.0, nullptr, nullptr,
                                    field_of<kExt>(P.cfg)) != kOk) {
          good = false;
          break;
        }
        for (int q = 0; q < 6; ++q) p[q] = pr.p[q];
        for (int q = 0; q < 21; ++q) c[q] = pr.c[q];
      }
      if constexpr (kExt) material<double>(P.cfg, L.kind, p, c, 1.0);
      else add_ms(p, (double)P.cfg.ms_var, c);
      FrameT<double> f;
      make_frame(p, c, L.kind, f);
      double u, v;
      if (!residual(p, f, L.kind, hx[k], hy[k], hz[k], u, v)) {
        good = false;
        break;
      }
      double vuu, vvv, vuv;
      hit_cov((double)L.cs, (double)L.sn, hvu[k], hvv[k], vuu, vvv, vuv);
      chi2 += chi2_of(f, vuu, vvv, vuv, u, v);
      kf_update(p, c, f, L.kind, vuu, vvv, vuv, u, v);
    }
    if (!good) break;
    ok = 1;
  } while (false);
  seed_ok[i] = ok;
  seed_chi2[i] = ok ? (float)chi2 : 0.f;
  float w[kSeedWords];
#pragma unroll
  for (int k = 0; k < 6; ++k) w[k] = ok ? (float)p[k] : 0.f;
#pragma unroll
  for (int k = 0; k < 21; ++k) w[6 + k] = ok ? (float)c[k] : 0.f;
  // the row's last word: the index of the event's first hit (below 2^31),
  // read with the state so that the find need not look it up
  w[27] = __int_as_float((int)e0);
  float4 *row = reinterpret_cast<float4 *>(seed_state + (size_t)i * kSeedWords);
#pragma unroll
  for (int k = 0; k < kSeedWords / 4; ++k)
    row[k] = make_float4(w[4 * k], w[4 * k + 1], w[4 * k + 2], w[4 * k + 3]);
  if (ok) {  // for the plan: the state, its sines and cosines, the seed's layers
    double f[kSeedFit];
#pragma unroll
    for (int k = 0; k < 6; ++k) f[k] = p[k];
    sincos_t(p[4], &f[6], &f[7]);
    sincos_t(p[5], &f[8], &f[9]);
    f[10] = (double)(hl[0] | hl[1] << 8 | hl[2] << 16);
    f[11] = 0.0;
    double2 *dst = reinterpret_cast<double2 *>(fit + (size_t)i * kSeedFit);
#pragma unroll
    for (int k = 0; k < kSeedFit / 2; ++k) dst[k] = make_double2(f[2 * k], f[2 * k + 1]);
  }
}

// Layer plans and places in the processing order, kLanes lanes per seed.
template <bool kExt, int kLanes>
__global__ __launch_bounds__(256) void k_seed_plan(
    FindParams P, const double *fit, int *plan_len, int8_t *plan, const DevRegion *regions,
    int n_regions, SeedCells cells, int *cell_counts, int2 *cell_rank, int *len_counts) {
  constexpr int kPlanSeeds = 256 / kLanes;
  __shared__ DevLayer sl[kMaxLayers];
  __shared__ double s_path[kPlanSeeds][kMaxLayers + 1];  // path to every layer, < 0: none
  __shared__ double s_l[kPlanSeeds][kMaxPlan + 1];       // the plan's path lengths
  __shared__ __attribute__((aligned(4))) uint8_t s_plan[kPlanSeeds][kMaxPlan];
  __shared__ int s_len[kLenWords];
  stage_layers(P, sl);
  for (int k = threadIdx.x; k < kLenWords; k += blockDim.x) s_len[k] = 0;
  __syncthreads();
  const int g = threadIdx.x / kLanes, sub = threadIdx.x % kLanes;
  const int64_t i0 = (int64_t)blockIdx.x * kPlanSeeds + g;
  const bool valid = i0 < P.n_seeds;
  const int64_t i = valid ? i0 : P.n_seeds - 1;  // (idle lanes repeat the last seed, unwritten)
  const bool ok = P.seed_ok[i] != 0;
  double p[6], trig[4];
  int hl[3] = {};
  if (ok) {
    const double *f = fit + (size_t)i * kSeedFit;
#pragma unroll
    for (int k = 0; k < 6; ++k) p[k] = f[k];
#pragma unroll
    for (int k = 0; k < 4; ++k) trig[k] = f[6 + k];
    const int h = (int)f[10];
#pragma unroll
    for (int k = 0; k < 3; ++k) hl[k] = (h >> (8 * k)) & 0xFF;
    if (n_regions == 0) {
      const double mkb = P.cfg.mkb, l_min = P.cfg.l_min, edge = P.cfg.edge_margin;
      for (int L = sub; L < P.n_layers; L += kLanes) {
        double l = -1.0;
        if (L != hl[0] && L != hl[1] && L != hl[2]) {
          PropT<double> pr;
          if (propagate<false, double>(p, nullptr, sl[L], mkb, l_min, true, edge, pr, 0.0,
                                       nullptr, nullptr, field_of<kExt>(P.cfg), trig) == kOk)
            l = pr.l;
        }
        s_path[g][L] = l;
      }
    }
  }
  int *plan_w = reinterpret_cast<int *>(s_plan[g]);
  for (int k = sub; k < kMaxPlan / 4; k += kLanes) plan_w[k] = -1;
  wave_sync();
  if (sub == 0 && valid) {
    int n = 0;
    if (ok && n_regions > 0) {
      const double eta = -log(tan(0.5 * p[5]));
      int r = 0;
      while (r < n_regions && !(eta >= regions[r].eta_lo && eta < regions[r].eta_hi)) ++r;
      if (r < n_regions) {
        const DevRegion &rg = regions[r];
        for (int k = 0; k < rg.n && n < kMaxPlan; ++k) {
          const int L = rg.layers[k];
          if (L == hl[0] || L == hl[1] || L == hl[2]) continue;
          s_plan[g][n++] = (uint8_t)L;
        }
      }
    } else if (ok) {
      // insertion by path length (ties by layer id)
      for (int L = 0; L < P.n_layers && n < kMaxPlan; ++L) {
        const double lf = s_path[g][L];
        if (lf < 0.0) continue;
        int j = n;
        while (j > 0 && s_l[g][j - 1] > lf) {
          s_l[g][j] = s_l[g][j - 1];
          s_plan[g][j] = s_plan[g][j - 1];
          --j;
        }
        s_l[g][j] = lf;
        s_plan[g][j] = (uint8_t)L;
        ++n;
      }
    }
    plan_len[i] = n;
    // the processing order's cell (a state that is not a number: cell 0)
    const float theta = ok ? (float)p[5] : 0.f, phi = ok ? (float)p[4] : 0.f;
    const float tc = theta * 8.f, pc = (phi + kPi) * (kPhiCells / kTwoPi);
    const int ti = tc > 0.f ? min((int)fminf(tc, 1e6f), kThetaCells - 1) : 0;
    const int pi = pc > 0.f ? min((int)fminf(pc, 1e6f), kPhiCells - 1) : 0;
    const int dir = ti * kPhiCells + pi;
    const int64_t grp = P.seed_event[i] >> cells.event_shift, len = kMaxPlan - n;
    const int64_t cell = (cells.by_length ? len * cells.n_groups + grp
                                          : grp * kPlanLens + len) * kDirCells + dir;
    cell_rank[i] = make_int2((int)cell, atomicAdd(&cell_counts[cell], 1));
    atomicAdd(&s_len[n], 1);
    if (ok) atomicAdd(&s_len[kPlanLens], 1);
  }
  wave_sync();
  if (valid)
    for (int k = sub; k < kMaxPlan / 4; k += kLanes)
      reinterpret_cast<int *>(plan + (size_t)i * kMaxPlan)[k] = plan_w[k];
  __syncthreads();
  for (int k = threadIdx.x; k < kLenWords; k += blockDim.x)
    if (s_len[k]) atomicAdd(&len_counts[blockIdx.x % kLenSlots * kLenWords + k], s_len[k]);
}

// ------------------------------------------------------------- hit index

__device__ __forceinline__ int event_of(const int64_t *ev_off, int n_events, int64_t i) {
  int lo = 0, hi = n_events;  // ev_off[lo] <= i < ev_off[hi]
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (ev_off[mid] <= i) lo = mid; else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ int bin_of(const DevLayer &L, float x, float y, float z) {
  const float phi = atan2f(y, x);
  const int pb = clampi((int)floorf((phi + kPi) * L.phi_scale), 0, L.nphi - 1);
  const float q = L.kind == 0 ? z : sqrtf(fmaf(x, x, y * y));
  const int qb = clampi((int)floorf((q - L.q_lo) * L.q_scale), 0, L.nq - 1);
  return L.bin_base + qb * L.nphi + pb;
}

// ------------------------------------------------------ triplet seeding
//
// The paper takes seeds from outside (Section 2.2); this builds them from
// the hits.  A seed is a triplet of hits a, b, c on three barrel layers
// (innermost first) whose helix is a plausible track from the beam line:
// with the circle through the three transverse points (centre c0, radius
// rho), pT = kappa |B| rho >= pt_min; the circle passes within d0_max of the
// beam line; a, b, c follow each other in the turning sense within half a
// turn; b lies within dz_max of the s-z line through a and c; and that line
// has |z| <= z0_max at the point of closest approach to the beam line, which
// precedes a within half a turn.  The cuts are evaluated in FP64.
//
// One wavefront per hit a of the first layer.  Its lanes take the second
// layer's hits b of an azimuth window (every z bin), drop the pairs whose
// straight-line z at the beam line is far outside z0_max, and gather the others;
// then each lane takes one pair and walks the third layer's hits c in an azimuth
// and z window around its extrapolation.  The windows only bound the search
// (their margins cover curvature, d0 and dz); the cuts decide.  Nearly all c
// fail the d0 or the dz cut, so both are first bounded from above in FP32
// (triplet_may_pass), and the lanes evaluate the few triplets left together.
//
// Bound by instruction issue in the walk over c (some 9 million candidates per
// event of 5,000 tracks).  20 events x 5,000 tracks: 2.0 ms for the whole call, of
// which gathering 1.93, the cuts 0.042 and the placing 0.015, against 51 ms with one
// lane per hit a and the FP64 cuts on every c, in two passes.

// exact cuts of one triplet (FP64)
__device__ __forceinline__ bool triplet_passes(const DevCfg &cfg, const DevSeeding &sc, double ax,
                                               double ay, double az, double bx, double by,
                                               double bz, double cx, double cy, double cz) {
  const double ux0 = bx - ax, uy0 = by - ay, vx0 = cx - ax, vy0 = cy - ay;
  const double cr = ux0 * vy0 - uy0 * vx0;
  if (cr == 0.0) return false;
  const double u2 = ux0 * ux0 + uy0 * uy0, v2 = vx0 * vx0 + vy0 * vy0;
  const double ox = ax + (vy0 * u2 - uy0 * v2) / (2.0 * cr);
  const double oy = ay + (ux0 * v2 - vx0 * u2) / (2.0 * cr);
  const double rho = sqrt((ox - ax) * (ox - ax) + (oy - ay) * (oy - ay));
  // kappa |B| = |mkb|
  if (fabs((double)cfg.mkb) * rho < (double)sc.pt_min) return false;
  const double dist = sqrt(ox * ox + oy * oy);
  if (dist == 0.0 || fabs(dist - rho) > (double)sc.d0_max) return false;
  const double sg = cr > 0.0 ? 1.0 : -1.0;
  const double two_pi = 6.283185307179586;
  const double qa = atan2(ay - oy, ax - ox), qb = atan2(by - oy, bx - ox);
  const double qc = atan2(cy - oy, cx - ox), q0 = atan2(-oy, -ox);
  auto turn = [&](double from, double to) {
    double t = sg * (to - from);
    if (t < 0.0) t += two_pi;
    if (t < 0.0) t += two_pi;
    return t;
  };
  const double pab = turn(qa, qb), pac = turn(qa, qc), p0a = turn(q0, qa);
  const double pi = 3.141592653589793;
  if (!(pab > 0.0 && pac > pab && pac < pi && p0a < pi)) return false;
  const double slope = (cz - az) / (rho * pac);
  const double dz = bz - (az + slope * rho * pab);
  if (fabs(dz) > (double)sc.dz_max) return false;
  const double z0 = az - slope * rho * p0a;
  return fabs(z0) <= (double)sc.z0_max;
}

// False only where the triplet cannot pass: its d0 or its dz is beyond the cut by
// more than FP32 can be wrong about them.  With u = b - a, v = c - a, w = c - b,
// cr = u x v and W = (v_y u^2 - u_y v^2, u_x v^2 - v_x u^2), the circle's centre
// is a + W / (2 cr), its radius rho = |W| / (2 |cr|) with |W| = |u| |v| |w|, and
//   d0 = |centre| - rho = (a^2 cr + a . W) / (|cr| (|centre| + rho)),
// a form without cancellation for straight tracks.  Every term on the left is
// a sum of products of differences of the coordinates, each rounded a few times:
// the error of a^2 cr + a . W and of d0_max cr centre is below 12 roundings
// (7e-7) of (|a| + d0_max) (|a| |u| |v| + |u| |v| (|u| + |v|)), taken here as 4e-6
// of a bound on that.  A chord turns by 2 asin(|u| / 2 rho), so the arcs that dz
// takes are s_ab / s_ac = asin(|u| k) / asin(|v| k), k = 1 / (2 rho), with asin(x) / x
// summed to x^6 (within 2e-5 for x <= 0.4; beyond, the triplet is let through), as
// is one straight enough (|cr| < 1e-5 (u^2 + v^2)) for FP64 to round d0 visibly.
__device__ __forceinline__ bool triplet_may_pass(const DevSeeding &sc, float ax, float ay,
                                                 float az, float ra, float ux, float uy, float u2,
                                                 float bx, float by, float uz, float cx, float cy,
                                                 float cz) {
  const float vx = cx - ax, vy = cy - ay, wx = cx - bx, wy = cy - by;
  const float v2 = fmaf(vx, vx, vy * vy), w2 = fmaf(wx, wx, wy * wy);
  const float cr = fmaf(ux, vy, -uy * vx);
  const float Wx = fmaf(vy, u2, -uy * v2), Wy = fmaf(ux, v2, -vx * u2);
  const float m = u2 + v2;
  const float lhs = fmaf(ra * ra, cr, fmaf(ax, Wx, ay * Wy));
  const float ox = fmaf(cr, ax, 0.5f * Wx), oy = fmaf(cr, ay, 0.5f * Wy);
  const float W = __builtin_amdgcn_sqrtf(u2 * v2 * w2);
  const float rhs = sc.d0_max * (0.5f * W + __builtin_amdgcn_sqrtf(fmaf(ox, ox, oy * oy)));
  const float err = 4e-6f * m * (ra + sc.d0_max) *
                    fmaf(0.75f, __builtin_amdgcn_sqrtf(m), 0.5f * ra);
  if (fabsf(cr) < 1e-5f * m) return true;
  if (fabsf(lhs) > fmaf(rhs, 1.0001f, err)) return false;
  const float k = fabsf(cr) * __builtin_amdgcn_rcpf(W);
  const float x = u2 * k * k, y = v2 * k * k;  // (|u| k)^2, (|v| k)^2
  if (!(y < 0.16f)) return true;
  const float pu = fmaf(x, fmaf(x, fmaf(x, 15.f / 336.f, 3.f / 40.f), 1.f / 6.f), 1.f);
  const float pv = fmaf(y, fmaf(y, fmaf(y, 15.f / 336.f, 3.f / 40.f), 1.f / 6.f), 1.f);
  const float ratio = __builtin_amdgcn_sqrtf(u2 * __builtin_amdgcn_rcpf(v2)) * pu *
                      __builtin_amdgcn_rcpf(pv);
  const float vz = cz - az;
  // (a value that is not a number passes)
  return !(fabsf(fmaf(-vz, ratio, uz)) >
           fmaf(1e-4f, fabsf(vz) + fabsf(uz) + sc.dz_max, sc.dz_max + 1e-5f));
}

// The azimuth window [phi - dphi, phi + dphi] of a layer as up to two runs of
// bins per row, [lo[0], hi[0]] and, where it wraps, [lo[1], hi[1]] (else empty).
struct PhiRuns {
  int lo[2], hi[2];
};
__device__ __forceinline__ PhiRuns phi_runs(const DevLayer &L, float phi, float dphi) {
  PhiRuns r{{0, 1}, {L.nphi - 1, 0}};
  if (dphi < kPi) {
    const int blo = (int)floorf((phi - dphi + kPi) * L.phi_scale);
    const int bhi = (int)floorf((phi + dphi + kPi) * L.phi_scale);
    if (bhi - blo + 1 < L.nphi) {
      if (blo < 0) {
        r.lo[0] = blo + L.nphi; r.lo[1] = 0; r.hi[1] = bhi;
      } else if (bhi >= L.nphi) {
        r.lo[0] = blo; r.lo[1] = 0; r.hi[1] = bhi - L.nphi;
      } else {
        r.lo[0] = blo; r.hi[0] = bhi;
      }
    }
  }
  return r;
}

// fn(position in the sorted hits, the record's first half) for every hit of
// rows [qlo, qhi] x runs, the records requested four at a time (the sorted array
// is padded past its end)
template <class Fn>
__device__ __forceinline__ void walk_runs(const FindParams &P, int base, int nphi,
                                          const PhiRuns &r, int qlo, int qhi, Fn fn) {
  const float4 *hits = reinterpret_cast<const float4 *>(P.sorted);
  for (int qb = qlo; qb <= qhi; ++qb) {
    const int row = base + qb * nphi;
#pragma unroll
    for (int sg = 0; sg < 2; ++sg) {
      if (r.lo[sg] > r.hi[sg]) continue;
      const int h0 = P.bin_start[row + r.lo[sg]], h1 = P.bin_start[row + r.hi[sg] + 1];
      for (int k = h0; k < h1; k += 4) {
        float4 h[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) h[j] = hits[2 * (size_t)(k + j)];
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (k + j < h1) fn(k + j, h[j]);
      }
    }
  }
}

// azimuth change between radii r0 < r1 of a circle of radius >= rho_min
// passing within d0 of the beam line, with room for rounding
__device__ __forceinline__ float bend_window(float r0, float r1, float rho_min, float d0) {
  const float s0 = fminf(1.f, r0 / (2.f * rho_min)), s1 = fminf(1.f, r1 / (2.f * rho_min));
  return asinf(s1) - asinf(s0) + d0 / r0 + d0 / r1 + 2e-3f;
}

__device__ __forceinline__ int wave_inclusive(int v, int lane) {
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const int u = __shfl_up(v, o);
    if (lane >= o) v += u;
  }
  return v;
}

// One wavefront per first-layer hit of event blockIdx.y, in the hit index's
// order; counts, offsets and kept are indexed by that sorted position.  The
// triplets of a hit come in the order of b, then of c, in the index.
//   gather: the triplets that may pass go to the store, up to kTripletList per
//     hit and while its segment has room; k_triplets_cut takes the cuts, one
//     lane per triplet, and k_triplets_place puts those that pass in place.
//     (With the cuts taken here, by the few lanes that hold a triplet, their
//     FP64 arithmetic was half of the kernel's instructions and left it three
//     waves per SIMD: 2.80 ms on 20 events x 5,000 tracks; gathering at four waves
//     per SIMD took 2.30, at six it takes 1.93.)
//   count, write: the same with the cuts, for the hits that did not fit.
// A lane notes a few c per walk, and the walk is repeated where one has more: the
// usual cuts leave few.  Loose ones leave hundreds, so gathering hands a hit over
// after kTripletRounds walks or as soon as its list is known to be too short, and
// the other modes note 32 at a time.  (With four in all modes, and gathered triplets
// counted before they were put: 66 million triplets of 20 events x 500 tracks 1.10 s,
// now 0.13; d0_max 1 cm on an event of 5,000 tracks 42 ms, now 5.9.)
enum TripletMode { kGather = 0, kCount = 1, kWriteOut = 2 };
constexpr int kTripletRounds = 4;
constexpr int kTripletList = 256;
template <int kMode>
__global__ __launch_bounds__(256, kMode == kGather ? 6 : 1) void k_triplets(
    FindParams P, DevSeeding sc, int *counts, const int *offsets, TripletStore st, int *out_event,
    int *out_hits) {
  constexpr int kKeep = kMode == kGather ? 4 : 32;  // c that a lane notes per walk
  __shared__ DevLayer sl[kMaxLayers];
  __shared__ int s_shift[4][64], s_end[4][64];  // runs of b: sorted position - ordinal, end ordinal
  __shared__ int s_pair[4][128];                // sorted positions of the gathered b
  __shared__ int s_c[4][kKeep][64];
  __shared__ int2 s_list[4][kMode == kGather ? kTripletList : 1];  // the hit's (b, c) so far
  if (kMode != kGather && *st.n_again == 0) return;
  stage_layers(P, sl);
  __syncthreads();
  const int e = blockIdx.y;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const DevLayer &L0 = sl[sc.layer[0]], &L1 = sl[sc.layer[1]], &L2 = sl[sc.layer[2]];
  const int ev0 = e * P.bins_per_event;
  const int first = P.bin_start[ev0 + L0.bin_base];
  const int last = P.bin_start[ev0 + L0.bin_base + L0.nq * L0.nphi];
  const float rho_min = sc.pt_min / fabsf(P.cfg.mkb);
  const float R0 = L0.pos, R1 = L1.pos, R2 = L2.pos;
  const float dphi1 = bend_window(R0, R1, rho_min, sc.d0_max);
  const float dphi2 = bend_window(R1, R2, rho_min, sc.d0_max);
  for (int idx = first + blockIdx.x * 4 + wv; idx < last; idx += gridDim.x * 4) {
    if (kMode != kGather && st.kept[idx].x >= 0) continue;
    const HitRec ha = P.sorted[idx];
    const float ax = ha.x, ay = ha.y, az = ha.z;
    const float ra = sqrtf(fmaf(ax, ax, ay * ay));
    int total = 0, n_pair = 0;  // (the same in all lanes)
    // up to 64 gathered pairs, one per lane
    auto take_pairs = [&](int n) {
      if (kMode == kGather && total > kTripletList) return;  // handed over
      const bool on = lane < n;
      const int kb = s_pair[wv][on ? lane : 0];
      const HitRec hb = P.sorted[kb];
      const float rb = sqrtf(fmaf(hb.x, hb.x, hb.y * hb.y));
      const float Z = hb.z - az;
      const float ux = hb.x - ax, uy = hb.y - ay, u2 = fmaf(ux, ux, uy * uy);
      const float k = (R2 - ra) / (rb - ra);
      const float zp = az + Z * k;
      const float hw = (0.1f * fabsf(Z) + 2.f * sc.dz_max) * k + 0.5f;
      const int qlo = clampi((int)floorf((zp - hw - L2.q_lo) * L2.q_scale), 0, L2.nq - 1);
      const int qhi = clampi((int)floorf((zp + hw - L2.q_lo) * L2.q_scale), 0, L2.nq - 1);
      const PhiRuns runs = phi_runs(L2, atan2f(hb.y, hb.x), dphi2);
      const int base = ev0 + L2.bin_base;
      // Rounds of kKeep noted c per lane, the walk repeated where a lane has more;
      // when all are counted, the places are known and the triplets are put
      // there, from the notes if there was one round, else in the same rounds
      // again.  (Gathering counts all that are noted: known after one walk.)
      int noted = 0, most = 0, n_c = 0, incl = 0, skip = 0;
      int64_t pos = 0;
      bool putting = false;
      for (;;) {
        int ord = 0;
        walk_runs(P, base, L2.nphi, runs, qlo, on ? qhi : qlo - 1, [&](int c, const float4 &h) {
          if (triplet_may_pass(sc, ax, ay, az, ra, ux, uy, u2, hb.x, hb.y, Z, h.x, h.y, h.z)) {
            if (ord >= skip && ord < skip + kKeep) s_c[wv][ord - skip][lane] = c;
            ++ord;
          }
        });
        if (!putting && skip == 0) {
          noted = ord;
          while (__ballot(noted > most) != 0ull) most += kKeep;
          if (most == 0) return;
          if constexpr (kMode == kGather) {
            incl = wave_inclusive(noted, lane);
            const int all = total + __shfl(incl, 63);
            if (most > kTripletRounds * kKeep || all > kTripletList) {
              total = kTripletList + 1;
              return;
            }
            pos = total + incl - noted;
            putting = true;
          }
        }
        unsigned pass = 0;  // which of this round's c pass
        if constexpr (kMode == kGather) {
          pass = (1u << clampi(noted - skip, 0, kKeep)) - 1u;
        } else {
#pragma unroll 1
          for (int t = 0; t < kKeep; ++t) {
            if (skip + t >= noted) break;
            const HitRec hc = P.sorted[s_c[wv][t][lane]];
            if (triplet_passes(P.cfg, sc, ax, ay, az, hb.x, hb.y, hb.z, hc.x, hc.y, hc.z))
              pass |= 1u << t;
          }
        }
        skip += kKeep;
        if (!putting) {
          n_c += __popc(pass);
          if (skip < most) continue;
          incl = wave_inclusive(n_c, lane);
          pos = (kMode == kWriteOut ? (int64_t)offsets[idx] : 0) + total + incl - n_c;
          if (kMode == kCount) break;
          putting = true;
          if (most > kKeep) {
            skip = 0;
            continue;
          }
        }
#pragma unroll 1
        for (int t = 0; t < kKeep; ++t)
          if ((pass >> t) & 1) {
            const int kc = s_c[wv][t][lane];
            if constexpr (kMode == kWriteOut) {
              out_event[pos] = e;
              out_hits[3 * pos] = ha.orig;
              out_hits[3 * pos + 1] = hb.orig;
              out_hits[3 * pos + 2] = P.sorted[kc].orig;
            } else {
              s_list[wv][pos] = make_int2(kb, kc);
            }
            ++pos;
          }
        if (skip >= most) break;
      }
      total += __shfl(incl, 63);
    };
    const PhiRuns runs = phi_runs(L1, atan2f(ay, ax), dphi1);
    const int segs = runs.lo[1] <= runs.hi[1] ? 2 : 1, n_runs = L1.nq * segs;
    for (int r0 = 0; r0 < n_runs; r0 += 64) {
      const int r = r0 + lane;
      int h0 = 0, len = 0;
      if (r < n_runs) {
        const int sg = segs == 2 ? r & 1 : 0;
        const int row = ev0 + L1.bin_base + (segs == 2 ? r >> 1 : r) * L1.nphi;
        h0 = P.bin_start[row + (sg ? runs.lo[1] : runs.lo[0])];
        len = P.bin_start[row + (sg ? runs.hi[1] : runs.hi[0]) + 1] - h0;
      }
      const int end = wave_inclusive(len, lane);
      s_shift[wv][lane] = h0 - (end - len);
      s_end[wv][lane] = end;
      const int n_b = __shfl(end, 63);
      wave_sync();
      for (int t0 = 0; t0 < n_b; t0 += 64) {
        const int t = t0 + lane;
        bool keep = t < n_b;
        int kb = 0;
        if (keep) {
          int lo = 0;  // the first run that ends beyond ordinal t
#pragma unroll
          for (int step = 32; step > 0; step >>= 1)
            if (s_end[wv][lo + step - 1] <= t) lo += step;
          kb = t + s_shift[wv][lo];
          const float4 h = reinterpret_cast<const float4 *>(P.sorted)[2 * (size_t)kb];
          const float rb = sqrtf(fmaf(h.x, h.x, h.y * h.y));
          const float Z = h.z - az;
          const float lever = ra / (rb - ra);
          // straight-line z at the beam line, against z0_max with room for
          // the arc-versus-radius differences (d0, bending) and dz
          const float z0e = az - Z * lever;
          keep = !(fabsf(z0e) > sc.z0_max + 1.f + (0.1f * fabsf(Z) + sc.dz_max) * (lever + 1.f));
        }
        const unsigned long long m = __ballot(keep);
        if (keep) s_pair[wv][n_pair + __popcll(m & ((1ull << lane) - 1ull))] = kb;
        n_pair += __popcll(m);
        wave_sync();
        if (n_pair >= 64) {
          take_pairs(64);
          n_pair -= 64;
          const int rest = s_pair[wv][64 + lane];
          wave_sync();
          if (lane < n_pair) s_pair[wv][lane] = rest;
          wave_sync();
        }
      }
      wave_sync();
    }
    if (n_pair > 0) take_pairs(n_pair);
    wave_sync();
    if constexpr (kMode == kGather) {
      int at = -1;
      if (lane == 0) {
        const int seg = (blockIdx.x + blockIdx.y * gridDim.x) % kTripletSegs;
        int *cursor = &st.cursor[seg * kTilePad];
        // (a full segment's cursor is left alone, so that it cannot wrap)
        if (total <= kTripletList &&
            __hip_atomic_load(cursor, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < st.seg_size) {
          const int a = total > 0 ? atomicAdd(cursor, total) : 0;
          if (a + total <= st.seg_size) {
            at = seg * st.seg_size + a;
          } else {  // the segment's end holds no triplet
            for (int t = a; t < st.seg_size; ++t) st.triplet[seg * st.seg_size + t].x = -1;
          }
        } else if (total == 0) {
          at = 0;
        }
        if (at < 0) atomicAdd(st.n_again, 1);
        st.kept[idx] = make_int2(at, total);
      }
      at = __builtin_amdgcn_readfirstlane(at);
      if (at >= 0)
        for (int t = lane; t < total; t += 64) {
          const int2 bc = s_list[wv][t];
          st.triplet[at + t] = make_int4(idx, bc.x, bc.y, 0);
        }
      wave_sync();  // read before the next hit's triplets overwrite the list
    } else if constexpr (kMode == kCount) {
      if (lane == 0) counts[idx] = total;
    }
  }
}

// The cuts of the gathered triplets, one lane each: .w = 1 for those that pass,
// counted by first hit.  One segment per blockIdx.x.
__global__ __launch_bounds__(256) void k_triplets_cut(FindParams P, DevSeeding sc, TripletStore st,
                                                      int *counts) {
  const int n = min(st.cursor[blockIdx.x * kTilePad], st.seg_size);
  int4 *triplet = st.triplet + (size_t)blockIdx.x * st.seg_size;
  const float4 *hits = reinterpret_cast<const float4 *>(P.sorted);
  for (int i = blockIdx.y * 256 + threadIdx.x; i < n; i += gridDim.y * 256) {
    const int4 t = triplet[i];
    if (t.x < 0) continue;
    const float4 a = hits[2 * (size_t)t.x], b = hits[2 * (size_t)t.y], c = hits[2 * (size_t)t.z];
    if (triplet_passes(P.cfg, sc, a.x, a.y, a.z, b.x, b.y, b.z, c.x, c.y, c.z)) {
      triplet[i].w = 1;
      atomicAdd(&counts[t.x], 1);
    }
  }
}

// The triplets that passed to their places, eight lanes per first-layer hit.
__global__ __launch_bounds__(256) void k_triplets_place(FindParams P, DevSeeding sc,
                                                        const int *counts, const int *offsets,
                                                        TripletStore st, int *out_event,
                                                        int *out_hits) {
  const int e = blockIdx.y;
  const DevLayer &L0 = P.layers[sc.layer[0]];
  const int first = P.bin_start[e * P.bins_per_event + L0.bin_base];
  const int last = P.bin_start[e * P.bins_per_event + L0.bin_base + L0.nq * L0.nphi];
  const int sub = threadIdx.x & 7, group = threadIdx.x & 56;
  for (int idx = first + (blockIdx.x * 256 + threadIdx.x) / 8; idx < last;
       idx += gridDim.x * 32) {
    const int2 kept = st.kept[idx];
    if (kept.x < 0 || counts[idx] == 0) continue;
    const int a = P.sorted[idx].orig;
    int64_t pos = offsets[idx];
    for (int t0 = 0; t0 < kept.y; t0 += 8) {
      const int4 t = t0 + sub < kept.y ? st.triplet[kept.x + t0 + sub] : make_int4(0, 0, 0, 0);
      const unsigned m = (unsigned)(__ballot(t.w != 0) >> group) & 0xFFu;
      if (t.w) {
        const int64_t p = pos + __popc(m & ((1u << sub) - 1u));
        out_event[p] = e;
        out_hits[3 * p] = a;
        out_hits[3 * p + 1] = P.sorted[t.y].orig;
        out_hits[3 * p + 2] = P.sorted[t.z].orig;
      }
      pos += __popc(m);
    }
  }
}

// ---------------------------------------------------- duplicate removal
//
// Removal of duplicate tracks (the paper lists it as not yet done,
// Introduction and Section 3).  The hits of a track are its three seed hits
// and its found hits.  Track u ranks before t if it has more hits; with as
// many, a smaller chi2; with the same chi2, a lexicographically smaller seed
// triplet.  t is a duplicate if a track ranking before it shares at least
// frac of the hits of the shorter of the two.  Tracks that share a hit are
// found through a hit -> tracks table (CSR over all hits of all events).

// per track: its hits as global indices, sorted, and their use counts.  The
// list is sorted in LDS and written in one run (60 us for 108,000 tracks when it
// was sorted in global memory, 32 us now).
constexpr int kDupBlock = 64;
__global__ __launch_bounds__(kDupBlock) void k_dup_prep(FindParams P, const int *seed_hits,
                                                        int *hbuf, int *hn, int *cnt) {
  __shared__ int s_h[kDupStride][kDupBlock];
  const int64_t pos = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (pos >= P.n_seeds) return;
  const int me = threadIdx.x;
  const int info = P.pinfo[pos];
  int n = 0;
  if ((info >> 8) & 1) {
    const int plen = info & 0xFF;
    const int4 *hit = reinterpret_cast<const int4 *>(P.out + (size_t)pos * kOutWords + kOutHit);
    const int64_t base = P.ev_off[P.pevent[pos]];
    const int *sh = seed_hits + (size_t)P.order[pos] * 3;
    auto insert = [&](int v) {  // insertion into the sorted prefix
      int j = n;
      while (j > 0 && s_h[j - 1][me] > v) {
        s_h[j][me] = s_h[j - 1][me];
        --j;
      }
      s_h[j][me] = v;
      ++n;
    };
    for (int k = 0; k < 3; ++k) insert((int)(base + sh[k]));
    for (int s = 0; s < plen; s += 4) {
      const int4 v = hit[s / 4];
      const int w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (s + q < plen && w[q] >= 0) insert((int)(base + w[q]));
    }
    int *h = hbuf + (size_t)pos * kDupStride;
    for (int k = 0; k < n; ++k) {
      h[k] = s_h[k][me];
      atomicAdd(&cnt[s_h[k][me]], 1);
    }
  }
  hn[pos] = n;
}

__global__ __launch_bounds__(256) void k_dup_fill(FindParams P, const int *hbuf, const int *hn,
                                                  const int *off, int *fill, int *list) {
  const int64_t pos = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (pos >= P.n_seeds) return;
  const int *h = hbuf + (size_t)pos * kDupStride;
  for (int k = 0; k < hn[pos]; ++k) list[off[h[k]] + atomicAdd(&fill[h[k]], 1)] = (int)pos;
}

// The decision, kDupLanes lanes per track, each with its share of the track's
// hits.  Bound by the latency of the look-ups (table, partner's rank, partner's
// hits), one after the other: 108,000 tracks of triplet seeds 187 us, against
// 367 us with one lane per track and 586 us when the shared hits were counted
// before the ranks were compared.
constexpr int kDupLanes = 8;
constexpr unsigned long long kDupFirst = 0x0101010101010101ull;  // the groups' first lanes
__global__ __launch_bounds__(256) void k_dup_decide(FindParams P, const int *seed_hits,
                                                    const int *hbuf, const int *hn, const int *off,
                                                    const int *list, float frac, int *out_dup,
                                                    int *n_dup) {
  const int64_t t0 = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) / kDupLanes;
  const bool on = t0 < P.n_seeds;
  const int64_t t = on ? t0 : P.n_seeds - 1;  // (idle lanes repeat the last track, unwritten)
  const int sub = threadIdx.x % kDupLanes;
  const int nt = hn[t];
  const int seed_t = P.order[t];
  bool dup = false;
  if (nt > 0) {
    const int *ht = hbuf + (size_t)t * kDupStride;
    const float chi_t = P.out[(size_t)t * kOutWords + kOutChi2];
    const int *st = seed_hits + (size_t)seed_t * 3;
    for (int k = sub; k < nt && !dup; k += kDupLanes) {
      const int g = ht[k];
      for (int j = off[g]; j < off[g + 1] && !dup; ++j) {
        const int u = list[j];
        if (u == t) continue;
        // a partner that ranks after t decides nothing, so the rank comes first:
        // it takes a word or two of the partner, the shared hits its whole list
        const int nu = hn[u];
        if (nu < nt) continue;
        if (nu == nt) {
          const float chi_u = P.out[(size_t)u * kOutWords + kOutChi2];
          if (chi_u != chi_t) {
            if (!(chi_u < chi_t)) continue;
          } else {
            const int *su = seed_hits + (size_t)P.order[u] * 3;
            int q = 0;
            while (q < 3 && su[q] == st[q]) ++q;
            if (q == 3 || su[q] > st[q]) continue;
          }
        }
        // shared hits, and the first of them in t's list: each partner is
        // weighed once, at the first hit the two share
        const int *hu = hbuf + (size_t)u * kDupStride;
        int a = 0, b = 0, shared = 0, first = -1;
        while (a < nt && b < nu) {
          const int x = ht[a], y = hu[b];
          if (x == y) {
            if (first < 0) first = a;
            ++shared;
            ++a;
            ++b;
          } else if (x < y) {
            ++a;
          } else {
            ++b;
          }
        }
        if (first != k) continue;
        // (nt <= nu: the shorter of the two is t)
        dup = (double)shared >= (double)frac * (double)nt;
      }
    }
  }
  // the group's verdict, and the wavefront's count of its groups
  unsigned long long m = __ballot(on && dup);
#pragma unroll
  for (int o = 1; o < kDupLanes; o <<= 1) m |= m >> o;
  m &= kDupFirst;
  if (on && sub == 0) out_dup[seed_t] = (m >> (threadIdx.x & 63)) & 1;
  if ((threadIdx.x & 63) == 0 && m != 0ull) atomicAdd(n_dup, (int)__popcll(m));
}

// -------------------------------------------------------- seed cleaning
//
// Seed cleaning (Section 2.2: seeds built from hits of the same outgoing
// particle are reduced to one, using the identity of their hits and their
// fitted pT, eta and phi).  Seeds sharing a hit are instances of one
// particle if their fitted q/pT agree within tol_ipt (relative to the
// larger), eta within tol_eta and phi within tol_phi.  Seed u ranks before t
// if its fit chi2 is smaller; with the same chi2, if its hit triplet is
// lexicographically smaller.  t is kept if its fit succeeded and no seed
// ranking before it is an instance of the same particle.  Seeds sharing a
// hit are found through a hit -> seeds table, as for duplicate tracks.

__device__ __forceinline__ float eta_of(float theta) { return -logf(tanf(0.5f * theta)); }

// What a pair of seeds is compared by is gathered first, an array each for q/pT,
// phi and theta: most partners share a hit with their neighbours in the array and
// fail the first comparison, so that a line of 16 q/pT serves many.  The decision
// alone, 563,000 triplet seeds: 452 us from the state rows of 112 bytes, 439 from
// 16 bytes per seed, 415 with eta in place of theta (its loads no longer wait for
// the comparison before), 377 so.
__global__ __launch_bounds__(256) void k_clean_prep(FindParams P, const int *seed_hits, int *hbuf,
                                                    float *key, int *cnt) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P.n_seeds) return;
  int h[3] = {-1, -1, -1};
  if (P.seed_ok[i]) {
    const int64_t base = P.ev_off[P.seed_event[i]];
#pragma unroll
    for (int k = 0; k < 3; ++k) h[k] = (int)(base + seed_hits[3 * i + k]);
    // sort three
    if (h[0] > h[1]) { const int t = h[0]; h[0] = h[1]; h[1] = t; }
    if (h[1] > h[2]) { const int t = h[1]; h[1] = h[2]; h[2] = t; }
    if (h[0] > h[1]) { const int t = h[0]; h[0] = h[1]; h[1] = t; }
#pragma unroll
    for (int k = 0; k < 3; ++k) atomicAdd(&cnt[h[k]], 1);
    const float *row = P.seed_state + (size_t)i * kSeedWords;
    key[i] = row[3];
    key[P.n_seeds + i] = row[4];
    key[2 * P.n_seeds + i] = row[5];
  }
#pragma unroll
  for (int k = 0; k < 3; ++k) hbuf[3 * i + k] = h[k];
}

__global__ __launch_bounds__(256) void k_clean_fill(FindParams P, const int *hbuf, const int *off,
                                                    int *fill, int *list) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= P.n_seeds || hbuf[3 * i] < 0) return;
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    const int g = hbuf[3 * i + k];
    list[off[g] + atomicAdd(&fill[g], 1)] = (int)i;
  }
}

__global__ __launch_bounds__(256) void k_clean_decide(FindParams P, const int *seed_hits,
                                                      const float *seed_chi2, const int *hbuf,
                                                      const float *key, const int *off,
                                                      const int *list, DevCleaning cc,
                                                      int *out_keep, int *n_keep) {
  const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= P.n_seeds) return;
  bool keep = P.seed_ok[t] != 0;
  if (keep) {
    const float *phi = key + P.n_seeds, *theta = phi + P.n_seeds;
    const float ipt_t = key[t], phi_t = phi[t];
    const float eta_t = eta_of(theta[t]);
    const float chi_t = seed_chi2[t];
    const int *ht = hbuf + 3 * t;
    for (int k = 0; k < 3 && keep; ++k) {
      const int g = ht[k];
      for (int j = off[g]; j < off[g + 1] && keep; ++j) {
        const int u = list[j];
        if (u == t) continue;
        // weigh each partner once, at the first hit the two share
        const int *hu = hbuf + 3 * (size_t)u;
        int first = -1;
        for (int a = 0; a < 3 && first < 0; ++a)
          if (ht[a] == hu[0] || ht[a] == hu[1] || ht[a] == hu[2]) first = a;
        if (first != k) continue;
        const float ipt_u = key[u];
        if (fabsf(ipt_t - ipt_u) > cc.tol_ipt * fmaxf(fabsf(ipt_t), fabsf(ipt_u))) continue;
        if (fabsf(eta_t - eta_of(theta[u])) > cc.tol_eta) continue;
        if (fabsf(wrap_phi(phi_t - phi[u])) > cc.tol_phi) continue;
        const float chi_u = seed_chi2[u];
        bool before;
        if (chi_u != chi_t) {
          before = chi_u < chi_t;
        } else {
          const int *su = seed_hits + 3 * (size_t)u, *st = seed_hits + 3 * t;
          int q = 0;
          while (q < 3 && su[q] == st[q]) ++q;
          before = q < 3 && su[q] < st[q];
        }
        if (before) keep = false;
      }
    }
  }
  out_keep[t] = keep ? 1 : 0;
  if (keep) atomicAdd(n_keep, 1);
}

// Event of hit i, known to lie in events e_lo .. e_hi (a block's hits span few).
__device__ __forceinline__ int event_between(const int64_t *ev_off, int e_lo, int e_hi, int64_t i) {
  while (e_lo < e_hi) {  // ev_off[e_lo] <= i < ev_off[e_hi + 1]
    const int mid = (e_lo + e_hi + 1) >> 1;
    if (ev_off[mid] <= i) e_lo = mid; else e_hi = mid - 1;
  }
  return e_lo;
}

// One lane per hit: record, check, bin.  Counting gives each hit its rank in
// its bin, so that the scatter needs no second count.  Bound by HBM and the
// atomics' look-ups: 24 B read, 40 B written and one counter per hit.  7.6
// million hits of 100 events: 0.37 ms, the scatter 0.25; the whole call 0.69 ms,
// against 1.10 when the arrays were copied, checked, binned and scattered one
// after the other.  (An XCD for each event's blocks, so that its L2 gathers the
// scattered records: 0.35 and 0.27 ms, no gain.)
template <bool kIn>
__global__ __launch_bounds__(256) void k_hits(FindParams P, int64_t n_hits, HitArrays in,
                                              HitRec *byorig, float2 *raw, int2 *bin_rank,
                                              int *counts, int *bad) {
  __shared__ DevLayer sl[kMaxLayers];
  __shared__ int s_ev[2];
  const int64_t i0 = (int64_t)blockIdx.x * blockDim.x;
  stage_layers(P, sl);
  if (threadIdx.x < 2)
    s_ev[threadIdx.x] =
        event_of(P.ev_off, P.n_events, threadIdx.x == 0 ? i0 : min(i0 + 255, n_hits - 1));
  __syncthreads();
  const int64_t i = i0 + threadIdx.x;
  if (i >= n_hits) return;
  const int e = event_between(P.ev_off, s_ev[0], s_ev[1], i);
  HitRec h;
  bool good = true;
  if constexpr (kIn) {
    const float vu = in.vu[i], vv = in.vv[i];
    h.x = in.x[i];
    h.y = in.y[i];
    h.z = in.z[i];
    h.layer = in.layer[i];
    good = isfinite(h.x) && isfinite(h.y) && isfinite(h.z) && isfinite(vu) && isfinite(vv) &&
           vu > 0.f && vv > 0.f && h.layer >= 0 && h.layer < P.n_layers;
    if (good) {
      const DevLayer &L = sl[h.layer];
      hit_cov(L.cs, L.sn, vu, vv, h.vu, h.vv, h.vuv);
      h.orig = (int)(i - P.ev_off[e]);
      byorig[i] = h;
      if (raw) raw[i] = make_float2(vu, vv);
    } else {
      *bad = 1;
    }
  } else {
    h = byorig[i];
  }
  int b = -1, rank = 0;
  if (good) {
    b = e * P.bins_per_event + bin_of(sl[h.layer], h.x, h.y, h.z);
    rank = atomicAdd(&counts[b], 1);
  }
  bin_rank[i] = make_int2(b, rank);
}

__global__ __launch_bounds__(256) void k_hit_scatter(FindParams P, int64_t n_hits,
                                                     const int2 *bin_rank, HitRec *sorted) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n_hits) return;
  const int2 br = bin_rank[i];
  if (br.x >= 0) sorted[P.bin_start[br.x] + br.y] = P.byorig[i];
}

// Exclusive sums in two launches: a block adds up its chunk of tiles; then
// every block adds the sums of the chunks before its own and scans its chunk
// tile by tile.  Bound by HBM (the input read twice, the output written once);
// chunks are four tiles long up to 8 Mi items and 16 beyond, where a block
// would otherwise read thousands of chunk sums.
__device__ __forceinline__ int4 scan_load(const int *in, int64_t k, int64_t n) {
  if (k + 4 <= n) return *reinterpret_cast<const int4 *>(in + k);
  return make_int4(k < n ? in[k] : 0, k + 1 < n ? in[k + 1] : 0, k + 2 < n ? in[k + 2] : 0, 0);
}

__device__ __forceinline__ int block_sum(int v, int *wsum) {
#pragma unroll
  for (int m = 1; m < 64; m <<= 1) v += __shfl_xor(v, m);
  if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = v;
  __syncthreads();
  v = wsum[0] + wsum[1] + wsum[2] + wsum[3];
  __syncthreads();
  return v;
}

__global__ __launch_bounds__(256) void k_scan_sums(const int *in, int64_t n, int tiles,
                                                   int *sums) {
  __shared__ int wsum[4];
  int v = 0;
  for (int t = 0; t < tiles; ++t) {
    const int64_t k = ((int64_t)blockIdx.x * tiles + t) * kScanTile + 4 * threadIdx.x;
    const int4 a = scan_load(in, k, n);
    v += a.x + a.y + a.z + a.w;
  }
  v = block_sum(v, wsum);
  if (threadIdx.x == 0) sums[blockIdx.x] = v;
}

__global__ __launch_bounds__(256) void k_scan_apply(const int *in, int *out, int64_t n, int tiles,
                                                    const int *sums) {
  __shared__ int wsum[4];
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  int before = 0;
  for (int b = threadIdx.x; b < (int)blockIdx.x; b += 256) before += sums[b];
  int run = block_sum(before, wsum);
  for (int t = 0; t < tiles; ++t) {
    const int64_t k = ((int64_t)blockIdx.x * tiles + t) * kScanTile + 4 * threadIdx.x;
    const int4 a = scan_load(in, k, n);
    const int s = a.x + a.y + a.z + a.w;
    int incl = s;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int u = __shfl_up(incl, o);
      if (lane >= o) incl += u;
    }
    if (lane == 63) wsum[wid] = incl;
    __syncthreads();
    int e = run + incl - s;
    for (int w = 0; w < wid; ++w) e += wsum[w];
    run += wsum[0] + wsum[1] + wsum[2] + wsum[3];
    __syncthreads();
    const int4 o4 = make_int4(e, e + a.x, e + a.x + a.y, e + a.x + a.y + a.z);
    if (k + 4 <= n) {
      *reinterpret_cast<int4 *>(out + k) = o4;
    } else {
      if (k < n) out[k] = o4.x;
      if (k + 1 < n) out[k + 1] = o4.y;
      if (k + 2 < n) out[k + 2] = o4.z;
    }
  }
  if (blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) out[n] = run;
}

// --------------------------------------------------------- unit kernels

__global__ __launch_bounds__(256) void k_propagate(FindParams P, int64_t n, const float *par,
                                                   const float *cov, const int *layer,
                                                   float *out_par, float *out_cov, float *out_l,
                                                   int *out_status) {
  __shared__ DevLayer sl[kMaxLayers];
  stage_layers(P, sl);
  __syncthreads();
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float p[6], c[21];
  for (int k = 0; k < 6; ++k) p[k] = par[i * 6 + k];
  for (int k = 0; k < 21; ++k) c[k] = cov[i * 21 + k];
  const int lid = layer[i];
  Prop pr;
  const int st = (lid < 0 || lid >= P.n_layers)
                     ? 3
                     : propagate<true, float>(p, c, sl[lid], P.cfg.mkb, P.cfg.l_min, true,
                                       P.cfg.edge_margin, pr, 0.f, nullptr, nullptr,
                                       &P.cfg.field);
  out_status[i] = st;
  for (int k = 0; k < 6; ++k) out_par[i * 6 + k] = st == kOk ? pr.p[k] : 0.f;
  for (int k = 0; k < 21; ++k) out_cov[i * 21 + k] = st == kOk ? pr.c[k] : 0.f;
  out_l[i] = st == kOk ? pr.l : 0.f;
}

// Search-free Kalman fit: one lane per track, the hit loop in registers;
// the per-step inputs are step-major so each step is a coalesced read.
template <bool kExt>
__global__ __launch_bounds__(256) void k_fit(DevCfg cfg, int64_t n, int n_steps,
                                             const int8_t *kind, const float *pos,
                                             const float *x, const float *y, const float *z,
                                             const float *vu, const float *vv, const int *len,
                                             const float *init_par, const float *init_cov,
                                             float *out_par, float *out_cov, float *out_chi2,
                                             int *out_status) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  float p[6], c[21];
#pragma unroll
  for (int k = 0; k < 6; ++k) p[k] = init_par[i * 6 + k];
#pragma unroll
  for (int k = 0; k < 21; ++k) c[k] = init_cov[i * 21 + k];
  float chi2 = 0.f;
  int status = 0;
  const int m = min(len[i], n_steps);
  // a step's surface and hit are requested one step ahead, while the step
  // before computes (the last step's words are requested twice, so that
  // every step issues the same loads)
  int nk = 0;
  float npos = 0.f, nx = 0.f, ny = 0.f, nz = 0.f, nvu = 0.f, nvv = 0.f;
  auto fetch = [&](int s) {
    const size_t j = (size_t)s * (size_t)n + i;
    nk = kind[j];
    npos = pos[j];
    nx = x[j];
    ny = y[j];
    nz = z[j];
    nvu = vu[j];
    nvv = vv[j];
  };
  if (m > 0) fetch(0);
  for (int s = 0; s < m; ++s) {
    DevLayer L;
    L.kind = nk;
    L.pos = npos;
    L.lo = 0.f;
    L.hi = 0.f;
    const float hx = nx, hy = ny, hz = nz, hvu = nvu, hvv = nvv;
    fetch(min(s + 1, m - 1));
    Prop pr;
    if (propagate<true, float>(p, c, L, cfg.mkb, cfg.l_min, false, 0.f, pr, 0.f, nullptr, nullptr,
                               field_of<kExt>(cfg)) != kOk) {
      status = s + 1;
      break;
    }
    layer_material<kExt>(cfg, L.kind, pr.p, pr.c, pr.sth, pr.cth);
    Frame f;
    make_frame(pr.p, pr.c, L.kind, f);
    float u, v;
    if (!residual(pr.p, f, L.kind, hx, hy, hz, u, v)) {
      status = s + 1;
      break;
    }
    chi2 += fmaxf(chi2_of(f, hvu, hvv, 0.f, u, v), 0.f);
    kf_update(pr.p, pr.c, f, L.kind, hvu, hvv, 0.f, u, v);
#pragma unroll
    for (int k = 0; k < 6; ++k) p[k] = pr.p[k];
#pragma unroll
    for (int k = 0; k < 21; ++k) c[k] = pr.c[k];
  }
#pragma unroll
  for (int k = 0; k < 6; ++k) out_par[i * 6 + k] = p[k];
#pragma unroll
  for (int k = 0; k < 21; ++k) out_cov[i * 21 + k] = c[k];
  out_chi2[i] = chi2;
  out_status[i] = status;
}

// ---------------------------------------------------------- backward fit
//
// The layer plan's steering marks layers used only when a track is fitted
// backwards (Section 2.1).  A found track is fitted backwards by the same
// Kalman filter (Introduction) run over its hits in the reverse order: its
// crossed plan layers from the last to the first, then its three seed
// layers from the third to the first.  The filter starts at the first of
// these surfaces from the track's final state, with the seed prior less its
// extent along that surface's normal, and on every surface it propagates
// (from the second on), adds the layer's scattering and takes the hit if
// the surface has one.  Backward propagation is forward propagation of the
// reversed helix (opposite charge, opposite direction).

// q/pT -> -q/pT, phi -> phi + pi, theta -> pi - theta; the covariance
// becomes D C D with D = diag(1, 1, 1, -1, 1, -1)
template <typename T>
__device__ __forceinline__ void flip_state(T *p, T *c) {
  p[3] = -p[3];
  p[4] = p[4] > T(0) ? p[4] - Consts<T>::pi() : p[4] + Consts<T>::pi();
  p[5] = Consts<T>::pi() - p[5];
  c[tri(0, 3)] = -c[tri(0, 3)];
  c[tri(1, 3)] = -c[tri(1, 3)];
  c[tri(2, 3)] = -c[tri(2, 3)];
  c[tri(3, 4)] = -c[tri(3, 4)];
  c[tri(0, 5)] = -c[tri(0, 5)];
  c[tri(1, 5)] = -c[tri(1, 5)];
  c[tri(2, 5)] = -c[tri(2, 5)];
  c[tri(4, 5)] = -c[tri(4, 5)];
}

// One surface of the backward fit: propagate the reversed helix to it
// (except on the first), add its scattering, take its hit (code >= 0).
// Returns false if the surface is not reached or the hit lies in the
// other half of the layer.
template <bool kExt, typename T>
__device__ __forceinline__ bool backfit_surface(const FindParams &P, const DevLayer &L,
                                                bool first, int code, int64_t ev_base, T *p,
                                                T *c, float &chi2) {
  if (first) {
    surface_prior(P.cfg, p, L.kind, c);
  } else {
    flip_state(p, c);
    PropT<T> pr;
    if (propagate<true, T>(p, c, L, T(P.cfg.mkb), T(P.cfg.l_min), false, T(0), pr, T(0), nullptr,
                           nullptr, field_of<kExt>(P.cfg)) != kOk)
      return false;
#pragma unroll
    for (int m = 0; m < 6; ++m) p[m] = pr.p[m];
#pragma unroll
    for (int m = 0; m < 21; ++m) c[m] = pr.c[m];
    flip_state(p, c);
  }
  // on the way back the track regains the layer's loss
  if constexpr (kExt) material<T>(P.cfg, L.kind, p, c, T(-1));
  else add_ms(p, T(P.cfg.ms_var), c);
  if (code >= 0) {
    const HitRec h = P.byorig[ev_base + code];
    FrameT<T> f;
    make_frame(p, c, L.kind, f);
    T u, v;
    if (!residual(p, f, L.kind, T(h.x), T(h.y), T(h.z), u, v)) return false;
    chi2 += fmaxf((float)chi2_of(f, T(h.vu), T(h.vv), T(h.vuv), u, v), 0.f);
    kf_update(p, c, f, L.kind, T(h.vu), T(h.vv), T(h.vuv), u, v);
  }
  return true;
}

// Surface t of a track's backward sequence: plan step t - 3 for t >= 3,
// seed hit t below.  False for a plan step the track did not cross.
__device__ __forceinline__ bool backfit_seq(const FindParams &P, const int *hit,
                                            const int8_t *plan, const int *sh, int64_t ev_base,
                                            int t, int &lid, int &code) {
  if (t >= 3) {
    code = hit[t - 3];
    lid = plan[t - 3];
    return code >= MKF_HIT_MISS;  // not crossed, or after the track ended
  }
  code = sh[t];
  lid = P.byorig[ev_base + code].layer;
  return true;
}

// Carried from the FP64 head to the FP32 tail, per processing position:
// state and covariance (27 words), chi2, then status, surfaces done and the
// next sequence index as integers.
constexpr int kBfWords = 32;

// Head, one lane per seed: as in the seed fit, the wide prior is filtered
// through the track's first three hits in FP64 (they shrink it by ~5
// decades, more than FP32 keeps in the covariance update).
template <bool kExt>
__global__ __launch_bounds__(kTrackBlock, kExt ? 1 : 2) void k_backfit_head(
    FindParams P, const int *seed_hits, float *tmp) {
  __shared__ DevLayer sl[kMaxLayers];
  stage_layers(P, sl);
  __syncthreads();
  const int64_t pos = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (pos >= P.n_seeds) return;
  const int info = P.pinfo[pos];
  const int plen = info & 0xFF;
  double pd[6], cd[21];
#pragma unroll
  for (int k = 0; k < 6; ++k) pd[k] = 0.0;
#pragma unroll
  for (int k = 0; k < 21; ++k) cd[k] = 0.0;
  float chi2 = 0.f;
  int status = 0, k = 0, t = -1;
  if ((info >> 8) & 1) {
    const float *row = P.out + (size_t)pos * kOutWords;
    const int *hit = reinterpret_cast<const int *>(row + kOutHit);
    const int8_t *plan = P.pplan + (size_t)pos * kMaxPlan;
    const int64_t ev_base = P.ev_off[P.pevent[pos]];
    const int64_t ev_hits = P.ev_off[P.pevent[pos] + 1] - ev_base;
    const int *sh = seed_hits + (size_t)P.order[pos] * 3;
#pragma unroll
    for (int m = 0; m < 6; ++m) pd[m] = row[kOutPar + m];
    status = 1;
    int taken = 0;
    for (t = plen + 2; t >= 0 && taken < 3; --t) {
      int lid, code;
      if (!backfit_seq(P, hit, plan, sh, ev_base, t, lid, code)) continue;
      if (lid < 0 || lid >= P.n_layers || code >= ev_hits ||
          !backfit_surface<kExt, double>(P, sl[lid], k == 0, code, ev_base, pd, cd, chi2)) {
        status = -(k + 1);
        break;
      }
      taken += code >= 0;
      ++k;
    }
  }
  float w[kBfWords];
#pragma unroll
  for (int m = 0; m < 6; ++m) w[m] = (float)pd[m];
#pragma unroll
  for (int m = 0; m < 21; ++m) w[6 + m] = (float)cd[m];
  w[27] = chi2;
  w[28] = __int_as_float(status);
  w[29] = __int_as_float(k);
  w[30] = __int_as_float(t);
  w[31] = 0.f;
  float4 *dst = reinterpret_cast<float4 *>(tmp + (size_t)pos * kBfWords);
#pragma unroll
  for (int q = 0; q < kBfWords / 4; ++q)
    dst[q] = make_float4(w[4 * q], w[4 * q + 1], w[4 * q + 2], w[4 * q + 3]);
}

// Tail, one lane per seed: the rest of the sequence in FP32; results by
// seed id (a failed fit reports zeros).
template <bool kExt>
__global__ __launch_bounds__(kTrackBlock) void k_backfit_tail(FindParams P, const int *seed_hits,
                                                      const float *tmp, float *out_par,
                                                      float *out_cov, float *out_chi2,
                                                      int *out_status) {
  __shared__ DevLayer sl[kMaxLayers];
  stage_layers(P, sl);
  __syncthreads();
  const int64_t pos = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (pos >= P.n_seeds) return;
  const int seed = P.order[pos];
  float w[kBfWords];
  const float4 *src = reinterpret_cast<const float4 *>(tmp + (size_t)pos * kBfWords);
#pragma unroll
  for (int q = 0; q < kBfWords / 4; ++q) {
    const float4 v = src[q];
    w[4 * q] = v.x;
    w[4 * q + 1] = v.y;
    w[4 * q + 2] = v.z;
    w[4 * q + 3] = v.w;
  }
  float p[6], c[21];
#pragma unroll
  for (int m = 0; m < 6; ++m) p[m] = w[m];
#pragma unroll
  for (int m = 0; m < 21; ++m) c[m] = w[6 + m];
  float chi2 = w[27];
  int status = __float_as_int(w[28]);
  int k = __float_as_int(w[29]);
  int t = __float_as_int(w[30]);
  if (status == 1) {
    const float *row = P.out + (size_t)pos * kOutWords;
    const int *hit = reinterpret_cast<const int *>(row + kOutHit);
    const int8_t *plan = P.pplan + (size_t)pos * kMaxPlan;
    const int64_t ev_base = P.ev_off[P.pevent[pos]];
    const int64_t ev_hits = P.ev_off[P.pevent[pos] + 1] - ev_base;
    const int *sh = seed_hits + (size_t)seed * 3;
    for (; t >= 0; --t) {
      int lid, code;
      if (!backfit_seq(P, hit, plan, sh, ev_base, t, lid, code)) continue;
      if (lid < 0 || lid >= P.n_layers || code >= ev_hits ||
          !backfit_surface<kExt, float>(P, sl[lid], k == 0, code, ev_base, p, c, chi2)) {
        status = -(k + 1);
        break;
      }
      ++k;
    }
  }
  if (status != 1) {
#pragma unroll
    for (int m = 0; m < 6; ++m) p[m] = 0.f;
#pragma unroll
    for (int m = 0; m < 21; ++m) c[m] = 0.f;
    chi2 = 0.f;
  }
#pragma unroll
  for (int m = 0; m < 6; ++m) out_par[(size_t)seed * 6 + m] = p[m];
#pragma unroll
  for (int m = 0; m < 21; ++m) out_cov[(size_t)seed * 21 + m] = c[m];
  out_chi2[seed] = chi2;
  out_status[seed] = status;
}

// ------------------------------------------------------------- smoothing
//
// Rauch-Tung-Striebel smoothing of the found tracks (the backward pass the
// layer plan's steering provides for, Section 2.1, applied to the Kalman
// filter of the Introduction): on the seed's third layer and on every plan
// layer a track crossed, its state given all its hits.
// * Forward (k_smooth_fwd, FP32): the find's filter along the track from the
//   seed state (propagate, add the layer's scattering, update with the hit
//   if there is one), keeping per surface the filtered state x, C, the
//   predicted state xp, Cp after scattering and F C (F: the transport from
//   the previous surface, C: the filtered covariance there).
// * Backward (k_smooth_bwd, FP32): from the last surface, where the smoothed
//   state is the filtered one,
//     xs(k) = x(k) + A (xs(k+1) - xp(k+1)),
//     Cs(k) = C(k) + A (Cs(k+1) - Cp(k+1)) A^T,   A = C(k) F^T Cp(k+1)^-1.
//   Cp(k+1) has no extent along its surface's normal and every vector it
//   meets lies in the surface, so the inverse is taken in the surface's five
//   free coordinates J: A = (J F C)^T (J Cp J^T)^-1 J, with a Cholesky
//   factor of J Cp J^T.

// per surface, SoA over positions: filtered 27, predicted 27, F C 36, layer
constexpr int kSmFields = 91;
constexpr int kSmFilt = 0, kSmPred = 27, kSmFC = 54, kSmLayer = 90;

template <bool kExt>
__global__ __launch_bounds__(256) void k_smooth_fwd(FindParams P, const int *seed_hits,
                                                    float *wk, int *n_surf) {
  __shared__ DevLayer sl[kMaxLayers];
  stage_layers(P, sl);
  __syncthreads();
  const int64_t pos = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (pos >= P.n_seeds) return;
  const size_t N = (size_t)P.n_seeds;
  auto at = [&](int j, int f) -> float & { return wk[((size_t)j * kSmFields + f) * N + pos]; };
  const int info = P.pinfo[pos];
  const int plen = info & 0xFF;
  int n = 0;
  if ((info >> 8) & 1) {
    const float *row = P.out + (size_t)pos * kOutWords;
    const int *hit = reinterpret_cast<const int *>(row + kOutHit);
    const int8_t *plan = P.pplan + (size_t)pos * kMaxPlan;
    const int64_t ev_base = P.ev_off[P.pevent[pos]];
    const int64_t ev_hits = P.ev_off[P.pevent[pos] + 1] - ev_base;
    const int *sh = seed_hits + (size_t)P.order[pos] * 3;
    float p[6], c[21];
    const float *st = P.pstate + (size_t)pos * kSeedWords;
#pragma unroll
    for (int m = 0; m < 6; ++m) p[m] = st[m];
#pragma unroll
    for (int m = 0; m < 21; ++m) c[m] = st[6 + m];
#pragma unroll
    for (int m = 0; m < 6; ++m) at(0, kSmFilt + m) = p[m];
#pragma unroll
    for (int m = 0; m < 21; ++m) at(0, kSmFilt + 6 + m) = c[m];
    at(0, kSmLayer) = __int_as_float(P.byorig[ev_base + sh[2]].layer);
    n = 1;
    for (int s = 0; s < plen; ++s) {
      const int code = hit[s];
      if (code < MKF_HIT_MISS) continue;  // not crossed, or after the track ended
      const int lid = plan[s];
      if (lid < 0 || lid >= P.n_layers || code >= ev_hits) {
        n = -1;
        break;
      }
      const DevLayer &L = sl[lid];
      Prop pr;
      float fc[36];
      if (propagate<true, float, true>(p, c, L, P.cfg.mkb, P.cfg.l_min, false, 0.f, pr, 0.f,
                                       nullptr, fc, field_of<kExt>(P.cfg)) != kOk) {
        n = -1;
        break;
      }
      float j33, j35;
      layer_material<kExt>(P.cfg, L.kind, pr.p, pr.c, pr.sth, pr.cth, &j33, &j35);
      // the transport to the prediction includes the loss's Jacobian
#pragma unroll
      for (int m = 0; m < 6; ++m) fc[18 + m] = j33 * fc[18 + m] + j35 * fc[30 + m];
#pragma unroll
      for (int m = 0; m < 6; ++m) at(n, kSmPred + m) = pr.p[m];
#pragma unroll
      for (int m = 0; m < 21; ++m) at(n, kSmPred + 6 + m) = pr.c[m];
#pragma unroll
      for (int m = 0; m < 36; ++m) at(n, kSmFC + m) = fc[m];
      if (code >= 0) {
        const HitRec h = P.byorig[ev_base + code];
        Frame f;
        make_frame(pr.p, pr.c, L.kind, f);
        float u, v;
        if (!residual(pr.p, f, L.kind, h.x, h.y, h.z, u, v)) {
          n = -1;
          break;
        }
        kf_update(pr.p, pr.c, f, L.kind, h.vu, h.vv, h.vuv, u, v);
      }
#pragma unroll
      for (int m = 0; m < 6; ++m) p[m] = pr.p[m];
#pragma unroll
      for (int m = 0; m < 21; ++m) c[m] = pr.c[m];
#pragma unroll
      for (int m = 0; m < 6; ++m) at(n, kSmFilt + m) = p[m];
#pragma unroll
      for (int m = 0; m < 21; ++m) at(n, kSmFilt + 6 + m) = c[m];
      at(n, kSmLayer) = __int_as_float(lid);
      ++n;
    }
  }
  n_surf[pos] = n;
}

// the surface's five free coordinates: u0 = a0 v0 + a1 v1 (barrel: along
// the azimuth; disk: x), u1 = b0 v0 + b1 v1 + b2 v2 (barrel: z; disk: y),
// u2..u4 = q/pT, phi, theta
struct FreeCoords {
  float a0, a1, b0, b1, b2;
  __device__ void apply(const float *v, float *u) const {
    u[0] = fmaf(a0, v[0], a1 * v[1]);
    u[1] = fmaf(b0, v[0], fmaf(b1, v[1], b2 * v[2]));
    u[2] = v[3];
    u[3] = v[4];
    u[4] = v[5];
  }
  // row a of J as a 6-vector
  __device__ void row(int a, float *r) const {
#pragma unroll
    for (int i = 0; i < 6; ++i) r[i] = 0.f;
    if (a == 0) {
      r[0] = a0;
      r[1] = a1;
    } else if (a == 1) {
      r[0] = b0;
      r[1] = b1;
      r[2] = b2;
    } else {
      r[a + 1] = 1.f;
    }
  }
};

// J M J^T (5 x 5, lower triangle packed by rows) of a symmetric 6 x 6 M
// (upper triangle packed)
__device__ __forceinline__ void sandwich5(const FreeCoords &J, const float *M, float *out) {
#pragma unroll
  for (int b = 0; b < 5; ++b) {
    float r[6], v[6];
    J.row(b, r);
#pragma unroll
    for (int i = 0; i < 6; ++i) {
      float a = 0.f;
#pragma unroll
      for (int j = 0; j < 6; ++j) a = fmaf(M[i <= j ? tri(i, j) : tri(j, i)], r[j], a);
      v[i] = a;
    }
    float u[5];
    J.apply(v, u);
#pragma unroll
    for (int a = b; a < 5; ++a) out[a * (a + 1) / 2 + b] = u[a];
  }
}

// solve (L L^T) x = b in place, L lower-triangular 5x5 packed by rows, inv: the
// reciprocals of its diagonal
__device__ __forceinline__ void chol_solve5(const float *Lp, const float *inv, float *b) {
  float y[5];
#pragma unroll
  for (int i = 0; i < 5; ++i) {
    float a = b[i];
#pragma unroll
    for (int k = 0; k < i; ++k) a = fmaf(-Lp[i * (i + 1) / 2 + k], y[k], a);
    y[i] = over(a, Lp[i * (i + 1) / 2 + i], inv[i]);
  }
#pragma unroll
  for (int i = 4; i >= 0; --i) {
    float a = y[i];
#pragma unroll
    for (int k = i + 1; k < 5; ++k) a = fmaf(-Lp[k * (k + 1) / 2 + i], b[k], a);
    b[i] = over(a, Lp[i * (i + 1) / 2 + i], inv[i]);
  }
}

// Backward pass, FP32: the 5 x 5 systems are well conditioned once scaled
// by their diagonal (condition numbers of the correlation matrices up to
// ~500 on the benchmark's tracks), which a Cholesky solve respects.  One
// lane per track: 20,000 tracks are 316 wavefronts, each bound by the issue of its
// own chain, of which 80 divisions per surface were the largest part.  20,000
// tracks of 14 surfaces 100 us with general divisions and blocks of 256, 82 with
// blocks of 64, 67 with the quotients of over() as well.  Eight lanes per track
// with the matrices in LDS took 83, four 113: the factor is then taken by every
// lane, and each surface waits for LDS four times.  Two waves per SIMD: three
// (153 registers) gain nothing on small calls, and on 2.5 M tracks of uneven
// events their stores of single words to 64 rows meet in the L2 (4.08 against 4.01 ms).
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 2))) void k_smooth_bwd(
    FindParams P, const float *wk, const int *n_surf, float *out_par, float *out_cov, int *out_n) {
  const int64_t pos = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (pos >= P.n_seeds) return;
  const size_t N = (size_t)P.n_seeds;
  auto at = [&](int j, int f) { return wk[((size_t)j * kSmFields + f) * N + pos]; };
  const int seed = P.order[pos];
  int n = n_surf[pos];
  float *op = out_par + (size_t)seed * (kMaxPlan + 1) * 6;
  float *oc = out_cov + (size_t)seed * (kMaxPlan + 1) * 21;
  if (n > 0) {
    float xs[6], Cs[21];
#pragma unroll
    for (int m = 0; m < 6; ++m) xs[m] = at(n - 1, kSmFilt + m);
#pragma unroll
    for (int m = 0; m < 21; ++m) Cs[m] = at(n - 1, kSmFilt + 6 + m);
#pragma unroll
    for (int m = 0; m < 6; ++m) op[(n - 1) * 6 + m] = xs[m];
#pragma unroll
    for (int m = 0; m < 21; ++m) oc[(n - 1) * 21 + m] = Cs[m];
    for (int k = n - 2; k >= 0; --k) {
      // the step's 91 words in one group of loads
      float pred[27], fc[36], filt[27];
      const int lid = __float_as_int(at(k + 1, kSmLayer));
#pragma unroll
      for (int m = 0; m < 27; ++m) pred[m] = at(k + 1, kSmPred + m);
#pragma unroll
      for (int m = 0; m < 36; ++m) fc[m] = at(k + 1, kSmFC + m);
#pragma unroll
      for (int m = 0; m < 27; ++m) filt[m] = at(k, kSmFilt + m);
      // surface k+1: its free coordinates at the predicted point
      float xp[6];
#pragma unroll
      for (int m = 0; m < 6; ++m) xp[m] = pred[m];
      FreeCoords J;
      if (P.layers[lid].kind == 0) {
        const float ir = rsqrtf(fmaf(xp[0], xp[0], xp[1] * xp[1]));
        J = FreeCoords{-xp[1] * ir, xp[0] * ir, 0.f, 0.f, 1.f};
      } else {
        J = FreeCoords{1.f, 0.f, 0.f, 1.f, 0.f};
      }
      // Sr = J Cp J^T, then dPr = J (Cs - Cp) J^T
      float Sr[15], dPr[15], inv[5];
      {
        float Cp[21];
#pragma unroll
        for (int m = 0; m < 21; ++m) Cp[m] = pred[6 + m];
        sandwich5(J, Cp, Sr);
#pragma unroll
        for (int m = 0; m < 21; ++m) Cs[m] -= Cp[m];
        sandwich5(J, Cs, dPr);
      }
      // Cholesky factor of Sr in place
      bool pd = true;
#pragma unroll
      for (int i = 0; i < 5; ++i) {
#pragma unroll
        for (int j = 0; j <= i; ++j) {
          float a = Sr[i * (i + 1) / 2 + j];
#pragma unroll
          for (int q = 0; q < j; ++q) a = fmaf(-Sr[i * (i + 1) / 2 + q], Sr[j * (j + 1) / 2 + q], a);
          if (i == j) {
            pd = pd && a > 0.f;
            Sr[i * (i + 1) / 2 + i] = sqrtf(a > 0.f ? a : 1.f);
            inv[i] = 1.f / Sr[i * (i + 1) / 2 + i];
          } else {
            Sr[i * (i + 1) / 2 + j] = over(a, Sr[j * (j + 1) / 2 + j], inv[j]);
          }
        }
      }
      if (!pd) {
        n = -2;
        break;
      }
      // u = Sr^-1 J (xs - xp)
      float d[6], u[5];
#pragma unroll
      for (int m = 0; m < 6; ++m) d[m] = xs[m] - xp[m];
      d[4] = wrap_phi(d[4]);
      J.apply(d, u);
      chol_solve5(Sr, inv, u);
      // M = J F C (5 x 6), one column at a time: xs(k) = x(k) + M^T u and
      // W = Sr^-1 M
      float W[5][6];
#pragma unroll
      for (int j = 0; j < 6; ++j) {
        float col[6], w[5];
#pragma unroll
        for (int i = 0; i < 6; ++i) col[i] = fc[i * 6 + j];
        J.apply(col, w);
        float a = filt[j];
#pragma unroll
        for (int q = 0; q < 5; ++q) a = fmaf(w[q], u[q], a);
        xs[j] = a;
        chol_solve5(Sr, inv, w);
#pragma unroll
        for (int q = 0; q < 5; ++q) W[q][j] = w[q];
      }
      xs[4] = wrap_phi(xs[4]);
      // Cs(k) = C(k) + W^T dPr W
#pragma unroll
      for (int i = 0; i < 6; ++i) {
        float t[5];
#pragma unroll
        for (int a = 0; a < 5; ++a) {
          float v = 0.f;
#pragma unroll
          for (int b = 0; b < 5; ++b)
            v = fmaf(dPr[a >= b ? a * (a + 1) / 2 + b : b * (b + 1) / 2 + a], W[b][i], v);
          t[a] = v;
        }
#pragma unroll
        for (int j = i; j < 6; ++j) {
          float v = filt[6 + tri(i, j)];
#pragma unroll
          for (int a = 0; a < 5; ++a) v = fmaf(t[a], W[a][j], v);
          Cs[tri(i, j)] = v;
        }
      }
#pragma unroll
      for (int m = 0; m < 6; ++m) op[k * 6 + m] = xs[m];
#pragma unroll
      for (int m = 0; m < 21; ++m) oc[k * 21 + m] = Cs[m];
    }
  }
  out_n[seed] = n;
}

__global__ void k_fill_u64(unsigned long long *p, int64_t n, unsigned long long v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
// (p 16-byte aligned)
__global__ __launch_bounds__(256) void k_fill_i32(int *p, int64_t n, int v) {
  const int64_t i = 4 * ((int64_t)blockIdx.x * blockDim.x + threadIdx.x);
  if (i + 4 <= n) {
    *reinterpret_cast<int4 *>(p + i) = make_int4(v, v, v, v);
  } else {
    for (int64_t k = i; k < n; ++k) p[k] = v;
  }
}

// The checked find's invariants of one seed's result record: a seed whose
// fit failed has no hits; otherwise each plan step holds a hit of the
// seed's event on that step's layer, a miss, a skip, or (once the candidate
// stopped, and from then on) none; the hit count is the three seed hits
// plus the hits taken, the miss count the misses; chi2 and the parameters
// are finite; the variances of q/pT, phi and theta are positive, those of
// the position at least -1e-5 of their (positive) sum.
__global__ __launch_bounds__(256) void k_check_results(FindParams P) {
  const int64_t pos = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  int bad = 0;
  if (pos < P.n_seeds) {
    const float *rec = P.out + (size_t)pos * kOutWords;
    const int *hit = reinterpret_cast<const int *>(rec + kOutHit);
    const int meta = __float_as_int(rec[kOutMeta]);
    const int nh = meta & 0xFF, nm = (meta >> 8) & 0xFF;
    const int info = P.pinfo[pos];
    const int plen = info & 0xFF;
    if (!((info >> 8) & 1)) {
      bad = nh != 0 || nm != 0;
    } else {
      const int ev = P.pevent[pos];
      const int64_t base = P.ev_off[ev], nev = P.ev_off[ev + 1] - base;
      int found = 0, miss = 0;
      bool stopped = false;
      for (int s = 0; s < plen; ++s) {
        const int h = hit[s];
        const int lid = P.pplan[(size_t)pos * kMaxPlan + s];
        if (h >= 0) {
          if (stopped || h >= nev) bad = 1;
          else if (P.byorig[base + h].layer != lid) bad = 1;
          ++found;
        } else if (h == MKF_HIT_MISS) {
          bad |= stopped;
          ++miss;
        } else if (h == MKF_HIT_SKIP) {
          bad |= stopped;
        } else if (h == MKF_HIT_NONE) {
          stopped = true;
        } else {
          bad = 1;
        }
      }
      bad |= nh != 3 + found || nm != miss;
      const float c2 = rec[kOutChi2];
      bad |= !(c2 >= 0.f) || !isfinite(c2);
      // (the state lies on its last surface: the variance along the
      // surface's normal is zero up to rounding, so a position variance
      // may be a rounding below zero; their sum must be positive)
      const float tp = rec[kOutCov + tri(0, 0)] + rec[kOutCov + tri(1, 1)] +
                       rec[kOutCov + tri(2, 2)];
      bad |= !(tp > 0.f) || !isfinite(tp);
      for (int i = 0; i < 6; ++i) {
        bad |= !isfinite(rec[kOutPar + i]);
        const float d = rec[kOutCov + tri(i, i)];
        bad |= !isfinite(d) || (i < 3 ? d < -1e-5f * tp : !(d > 0.f));
      }
    }
  }
  add_counter(P, kCntCheckFailed, bad);
}

// ------------------------------------------------------------- launchers

static inline unsigned blocks_for(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

void launch_hits_in(hipStream_t s, const FindParams &P, int64_t n_hits, const HitArrays &in,
                    HitRec *byorig, float2 *raw, int2 *bin_rank, int *counts, int *bad) {
  if (n_hits == 0) return;
  const dim3 grid(blocks_for(n_hits, 256));
  if (in.x)
    hipLaunchKernelGGL(k_hits<true>, grid, dim3(256), 0, s, P, n_hits, in, byorig, raw, bin_rank,
                       counts, bad);
  else
    hipLaunchKernelGGL(k_hits<false>, grid, dim3(256), 0, s, P, n_hits, in, byorig, raw, bin_rank,
                       counts, bad);
}

void launch_scatter(hipStream_t s, const FindParams &P, int64_t n_hits, const int2 *bin_rank,
                    HitRec *sorted) {
  if (n_hits == 0) return;
  hipLaunchKernelGGL(k_hit_scatter, dim3(blocks_for(n_hits, 256)), dim3(256), 0, s, P, n_hits,
                     bin_rank, sorted);
}

void launch_scan(hipStream_t s, const int *in, int *out, int64_t n, int *tmp) {
  const int tiles = n > (8 << 20) ? 16 : 4;
  const unsigned nb = n > 0 ? blocks_for(n, tiles * kScanTile) : 1;
  if (nb > 1) hipLaunchKernelGGL(k_scan_sums, dim3(nb), dim3(256), 0, s, in, n, tiles, tmp);
  hipLaunchKernelGGL(k_scan_apply, dim3(nb), dim3(256), 0, s, in, out, n, tiles, tmp);
}

void launch_validate_seeds(hipStream_t s, const FindParams &P, const int *seed_event,
                           const int *seed_hits, int *bad) {
  if (P.n_seeds == 0) return;
  hipLaunchKernelGGL(k_validate_seeds, dim3(blocks_for(P.n_seeds, 256)), dim3(256), 0, s, P,
                     seed_event, seed_hits, bad);
}

void launch_seed(hipStream_t s, const FindParams &P, const int *src_event, const int *src_hits,
                 int *seed_event, int *seed_hits, float *seed_state, int *seed_ok, int *plan_len,
                 int8_t *plan, float *seed_chi2, double *fit, const DevRegion *regions,
                 int n_regions, const SeedCells &sc, int *cell_counts, int2 *cell_rank,
                 int *len_counts) {
  if (P.n_seeds == 0) return;
  const bool ext = extended(P.cfg);
  const auto seed = ext ? k_seed<true> : k_seed<false>;
  hipLaunchKernelGGL(seed, dim3(blocks_for(P.n_seeds, kSeedBlock)), dim3(kSeedBlock), 0, s, P,
                     src_event, src_hits, seed_event, seed_hits, seed_state, seed_ok, seed_chi2,
                     fit);
  // Eight lanes per seed shorten the chain, which counts while they leave part of the
  // chip idle; four do less twice over.  Fit and plans together with eight and with
  // four: 5,000 seeds 30 and 33 us, 16,000 40 and 41, 24,000 48 and 48, 32,000 61 and 48,
  // 300,000 243 and 197; with material and field 10,000 0.93 and 1.02 ms, 16,000 1.03 and
  // 1.02, 32,000 1.66 and 1.49.
  const bool few = P.n_seeds <= kFewPlans;
  const int lanes = few ? 8 : 4;
  const auto plans = few ? (ext ? k_seed_plan<true, 8> : k_seed_plan<false, 8>)
                         : (ext ? k_seed_plan<true, 4> : k_seed_plan<false, 4>);
  hipLaunchKernelGGL(plans, dim3(blocks_for(P.n_seeds, 256 / lanes)), dim3(256), 0, s, P, fit,
                     plan_len, plan, regions, n_regions, sc, cell_counts, cell_rank, len_counts);
}

void launch_place_seeds(hipStream_t s, const FindParams &P, const int2 *cell_rank,
                        const int *cell_start, int *order, int *pos_of, float *pstate, int *pinfo,
                        int *pevent, int8_t *pplan) {
  if (P.n_seeds == 0) return;
  const int64_t lanes = P.n_seeds * (kSeedWords / 4 + kMaxPlan / 16);
  hipLaunchKernelGGL(k_place_seeds, dim3(blocks_for(lanes, 256)), dim3(256), 0, s, P, cell_rank,
                     cell_start, order, pos_of, reinterpret_cast<float4 *>(pstate), pinfo, pevent,
                     reinterpret_cast<int4 *>(pplan));
}

void launch_find_init(hipStream_t s, const FindParams &P) {
  if (P.n_seeds == 0) return;
  hipLaunchKernelGGL(k_find_init, dim3(blocks_for(P.n_seeds * P.slots, 256)), dim3(256), 0, s, P);
}

template <int G>
static void launch_find_step_g(hipStream_t s, const FindParams &P, int step, int64_t n_active) {
  const unsigned nb = blocks_for(n_active, 4 * Grp<G>::kSeeds);
  const unsigned grid = (nb + kQueues - 1) / kQueues * kQueues;  // whole XCD shares
  if (P.cfg.mat.tab || P.cfg.field.on)
    hipLaunchKernelGGL((k_find_step<true, G>), dim3(grid), dim3(256), 0, s, P, step, n_active);
  else hipLaunchKernelGGL((k_find_step<false, G>), dim3(grid), dim3(256), 0, s, P, step, n_active);
}

void launch_find_step(hipStream_t s, const FindParams &P, int step, int64_t n_active) {
  if (n_active == 0) return;
  if (P.slots == 6) launch_find_step_g<6>(s, P, step, n_active);
  else launch_find_step_g<8>(s, P, step, n_active);
}

template <int G, bool kSurr, bool kMat>
static void launch_persistent_g(hipStream_t s, const FindParams &P, int grid, int waves) {
  const size_t lds = 4 * sizeof(int) * persistent_rec_words(P.max_plan, G, Grp<G>::kSeeds);
  if constexpr (kMat) {
    switch (waves) {
      case 1: hipLaunchKernelGGL((k_find_persistent_mat<1, kSurr, G>), dim3(grid), dim3(256), lds, s, P); break;
      case 3: hipLaunchKernelGGL((k_find_persistent_mat<3, kSurr, G>), dim3(grid), dim3(256), lds, s, P); break;
      case 4: hipLaunchKernelGGL((k_find_persistent_mat<4, kSurr, G>), dim3(grid), dim3(256), lds, s, P); break;
      default: hipLaunchKernelGGL((k_find_persistent_mat<2, kSurr, G>), dim3(grid), dim3(256), lds, s, P); break;
    }
  } else {
    switch (waves) {
      case 1: hipLaunchKernelGGL((k_find_persistent<1, kSurr, G>), dim3(grid), dim3(256), lds, s, P); break;
      case 3: hipLaunchKernelGGL((k_find_persistent<3, kSurr, G>), dim3(grid), dim3(256), lds, s, P); break;
      case 4: hipLaunchKernelGGL((k_find_persistent<4, kSurr, G>), dim3(grid), dim3(256), lds, s, P); break;
      default: hipLaunchKernelGGL((k_find_persistent<2, kSurr, G>), dim3(grid), dim3(256), lds, s, P); break;
    }
  }
}

template <bool kSurr, bool kMat>
static void launch_persistent_k(hipStream_t s, const FindParams &P, int grid, int waves,
                                int group) {
  // 6-lane groups only hold budgets up to 6 candidates
  if (group == 8 || P.cfg.n_cand > 6) launch_persistent_g<8, kSurr, kMat>(s, P, grid, waves);
  else launch_persistent_g<6, kSurr, kMat>(s, P, grid, waves);
}

void launch_find_persistent(hipStream_t s, const FindParams &P, int grid_blocks, int waves,
                            bool surrogate, int group) {
  if (P.n_seeds == 0) return;
  // no more waves than tiles (each queue may end in a part-filled tile), and
  // whole XCD shares
  const int seeds = group == 8 || P.cfg.n_cand > 6 ? Grp<8>::kSeeds : Grp<6>::kSeeds;
  const int64_t tiles = (P.n_seeds + seeds - 1) / seeds + kQueues;
  const int64_t need = (tiles + 3) / 4;
  if (grid_blocks > need) grid_blocks = (int)need;
  grid_blocks = (grid_blocks + kQueues - 1) / kQueues * kQueues;
  if (P.cfg.mat.tab || P.cfg.field.on) {
    if (surrogate) launch_persistent_k<true, true>(s, P, grid_blocks, waves, group);
    else launch_persistent_k<false, true>(s, P, grid_blocks, waves, group);
  } else if (surrogate) launch_persistent_k<true, false>(s, P, grid_blocks, waves, group);
  else launch_persistent_k<false, false>(s, P, grid_blocks, waves, group);
}

void launch_finalize(hipStream_t s, const FindParams &P) {
  if (P.n_seeds == 0) return;
  const auto finalize = P.slots == 6 ? k_finalize<6> : k_finalize<8>;
  hipLaunchKernelGGL(finalize, dim3(blocks_for(P.n_seeds, kTrackBlock)), dim3(kTrackBlock), 0, s,
                     P);
}
void launch_check_results(hipStream_t s, const FindParams &P) {
  if (P.n_seeds == 0) return;
  hipLaunchKernelGGL(k_check_results, dim3(blocks_for(P.n_seeds, 256)), dim3(256), 0, s, P);
}

void launch_tracks(hipStream_t s, const FindParams &P, const int *pos_of, int64_t first, int64_t n,
                   int *out) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_tracks, dim3(blocks_for(n * kTrackWords, 256)), dim3(256), 0, s, P, pos_of,
                     first, n, out);
}

void launch_propagate(hipStream_t s, const FindParams &P, int64_t n, const float *par,
                      const float *cov, const int *layer, float *out_par, float *out_cov,
                      float *out_l, int *out_status) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_propagate, dim3(blocks_for(n, 256)), dim3(256), 0, s, P, n, par, cov,
                     layer, out_par, out_cov, out_l, out_status);
}

void launch_fit(hipStream_t s, const DevCfg &cfg, int64_t n, int n_steps, const int8_t *kind,
                const float *pos, const float *x, const float *y, const float *z,
                const float *vu, const float *vv, const int *len, const float *init_par,
                const float *init_cov, float *out_par, float *out_cov, float *out_chi2,
                int *out_status) {
  if (n == 0) return;
  const auto fit = extended(cfg) ? k_fit<true> : k_fit<false>;
  hipLaunchKernelGGL(fit, dim3(blocks_for(n, 256)), dim3(256), 0, s, cfg, n, n_steps, kind, pos, x,
                     y, z, vu, vv, len, init_par, init_cov, out_par, out_cov, out_chi2,
                     out_status);
}

void launch_backfit(hipStream_t s, const FindParams &P, const int *seed_hits, float *tmp,
                    float *out_par, float *out_cov, float *out_chi2, int *out_status) {
  if (P.n_seeds == 0) return;
  const bool ext = extended(P.cfg);
  const auto head = ext ? k_backfit_head<true> : k_backfit_head<false>;
  const auto tail = ext ? k_backfit_tail<true> : k_backfit_tail<false>;
  const dim3 grid(blocks_for(P.n_seeds, kTrackBlock));
  hipLaunchKernelGGL(head, grid, dim3(kTrackBlock), 0, s, P, seed_hits, tmp);
  hipLaunchKernelGGL(tail, grid, dim3(kTrackBlock), 0, s, P, seed_hits, tmp, out_par, out_cov,
                     out_chi2, out_status);
}

void launch_smooth(hipStream_t s, const FindParams &P, const int *seed_hits, float *wk,
                   int *n_surf, float *out_par, float *out_cov, int *out_n) {
  if (P.n_seeds == 0) return;
  const auto fwd = extended(P.cfg) ? k_smooth_fwd<true> : k_smooth_fwd<false>;
  // Where the chip is full many times over the two kernels are bound by HBM, and
  // blocks of four wavefronts, which read and write a kilobyte of each field, are the
  // faster: 2.5 M tracks of uneven events 6.23 ms against 6.50, of equal events
  // 6.47 against 6.53.  At 131,000 tracks the two are equal (backward 273 and 270
  // us), at 20,000 blocks of one take 67 against 82.
  const int block = P.n_seeds <= kManyTracks ? kTrackBlock : 256;
  const dim3 grid(blocks_for(P.n_seeds, block));
  hipLaunchKernelGGL(fwd, grid, dim3(block), 0, s, P, seed_hits, wk, n_surf);
  hipLaunchKernelGGL(k_smooth_bwd, grid, dim3(block), 0, s, P, wk, n_surf, out_par, out_cov, out_n);
}

// Blocks per event: in events alike, enough to fill the device some times over,
// each a few hits long.  A larger event gets more, by its share of the hits, so that
// one among thousands of small ones is not left to a few wavefronts; but every
// event gets as many, and blocks that find nothing cost 1.2 ns each where a
// first-layer hit, one in eleven, takes its wavefront some 20 us: the sum of both
// is least near the square root below.  An event of 3,000 tracks among 15,000 of 5
// takes 1.2 ms, 23 with one block per event; among 200, 0.20 ms (0.40).  The number
// is odd: blocks go round the XCDs and the segments of the store in turn, and
// in small events only the first few have a hit, so that with eight per event two
// XCDs did the work (2,000 events of 5 tracks 208 us, 112 with nine).
constexpr int kTripletBlocks = 16384;
static dim3 triplet_grid(const FindParams &P, int64_t n_hits, int64_t max_event_hits,
                         int per_block) {
  const double max = (double)max_event_hits;
  const double share = kTripletBlocks * (max / (double)n_hits);
  const double most = std::max((double)kTripletBlocks, std::sqrt(400.0 * max * P.n_events)) /
                      P.n_events;
  const int64_t per_event = std::max<int64_t>(1, (int64_t)std::min(share, most));
  const int64_t x = std::min<int64_t>((max_event_hits + per_block - 1) / per_block, per_event);
  return dim3((unsigned)x | 1u, (unsigned)P.n_events);
}

void launch_triplets(hipStream_t s, const FindParams &P, const DevSeeding &sc, int64_t n_hits,
                     int64_t max_event_hits, int *counts, const TripletStore &st) {
  if (max_event_hits == 0 || P.n_events == 0) return;
  const dim3 grid = triplet_grid(P, n_hits, max_event_hits, 4);
  hipLaunchKernelGGL(k_triplets<kGather>, grid, dim3(256), 0, s, P, sc, counts, nullptr, st,
                     nullptr, nullptr);
  hipLaunchKernelGGL(k_triplets_cut, dim3(kTripletSegs, 16), dim3(256), 0, s, P, sc, st, counts);
  hipLaunchKernelGGL(k_triplets<kCount>, grid, dim3(256), 0, s, P, sc, counts, nullptr, st,
                     nullptr, nullptr);
}

void launch_triplets_write(hipStream_t s, const FindParams &P, const DevSeeding &sc,
                           int64_t n_hits, int64_t max_event_hits, int *counts, const int *offsets,
                           const TripletStore &st, bool again, int *out_event, int *out_hits) {
  if (max_event_hits == 0 || P.n_events == 0) return;
  hipLaunchKernelGGL(k_triplets_place, triplet_grid(P, n_hits, max_event_hits, 32), dim3(256), 0, s,
                     P, sc, counts, offsets, st, out_event, out_hits);
  if (again)
    hipLaunchKernelGGL(k_triplets<kWriteOut>, triplet_grid(P, n_hits, max_event_hits, 4),
                       dim3(256), 0, s, P, sc, counts, offsets, st, out_event, out_hits);
}

void launch_dup_prep(hipStream_t s, const FindParams &P, const int *seed_hits, int *hbuf, int *hn,
                     int *cnt) {
  if (P.n_seeds == 0) return;
  hipLaunchKernelGGL(k_dup_prep, dim3(blocks_for(P.n_seeds, kDupBlock)), dim3(kDupBlock), 0, s, P,
                     seed_hits, hbuf, hn, cnt);
}

void launch_dup_fill(hipStream_t s, const FindParams &P, const int *hbuf, const int *hn,
                     const int *off, int *fill, int *list) {
  if (P.n_seeds == 0) return;
  hipLaunchKernelGGL(k_dup_fill, dim3(blocks_for(P.n_seeds, 256)), dim3(256), 0, s, P, hbuf, hn,
                     off, fill, list);
}

void launch_dup_decide(hipStream_t s, const FindParams &P, const int *seed_hits, const int *hbuf,
                       const int *hn, const int *off, const int *list, float frac, int *out_dup,
                       int *n_dup) {
  if (P.n_seeds == 0) return;
  hipLaunchKernelGGL(k_dup_decide, dim3(blocks_for(P.n_seeds, 256 / kDupLanes)), dim3(256), 0, s, P,
                     seed_hits, hbuf, hn, off, list, frac, out_dup, n_dup);
}

void launch_clean_prep(hipStream_t s, const FindParams &P, const int *seed_hits, int *hbuf,
                       float *key, int *cnt) {
  if (P.n_seeds == 0) return;
  hipLaunchKernelGGL(k_clean_prep, dim3(blocks_for(P.n_seeds, 256)), dim3(256), 0, s, P,
                     seed_hits, hbuf, key, cnt);
}

void launch_clean_fill(hipStream_t s, const FindParams &P, const int *hbuf, const int *off,
                       int *fill, int *list) {
  if (P.n_seeds == 0) return;
  hipLaunchKernelGGL(k_clean_fill, dim3(blocks_for(P.n_seeds, 256)), dim3(256), 0, s, P, hbuf,
                     off, fill, list);
}

void launch_clean_decide(hipStream_t s, const FindParams &P, const int *seed_hits,
                         const float *seed_chi2, const int *hbuf, const float *key,
                         const int *off, const int *list, const DevCleaning &cc, int *out_keep,
                         int *n_keep) {
  if (P.n_seeds == 0) return;
  hipLaunchKernelGGL(k_clean_decide, dim3(blocks_for(P.n_seeds, 256)), dim3(256), 0, s, P,
                     seed_hits, seed_chi2, hbuf, key, off, list, cc, out_keep, n_keep);
}

void launch_fill_u64(hipStream_t s, unsigned long long *p, int64_t n, unsigned long long v) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_fill_u64, dim3(blocks_for(n, 256)), dim3(256), 0, s, p, n, v);
}
void launch_fill_i32(hipStream_t s, int *p, int64_t n, int v) {
  if (n == 0) return;
  hipLaunchKernelGGL(k_fill_i32, dim3(blocks_for(n, 1024)), dim3(256), 0, s, p, n, v);
}

}  // namespace mkf
