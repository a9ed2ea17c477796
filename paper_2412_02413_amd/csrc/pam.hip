// Host side of the AS-TAX library: plan (the paper's pre-run, Section II-E),
// validation, workspace layout and kernel launches behind the C-ABI of pam.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "../../include/pam.h"
#include "kernels.hpp"
#include "k3_fields.hpp"
#include "k3_fields16.hpp"
#include "k3_factored.hpp"
#include "k2_fft.hpp"
#include "k3_fft.hpp"
#include "k3_tea.hpp"

namespace {

constexpr double kPi = 3.14159265358979323846;
constexpr int kMinSamples = 32;
constexpr int kMaxSamples = 16384;
constexpr int kMaxNx = 512;

struct DeviceGuard {
  int prev = -1;
  bool ok = false;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) != hipSuccess) return;
    ok = (prev == dev) || (hipSetDevice(dev) == hipSuccess);
  }
  ~DeviceGuard() {
    int cur = -1;
    if (ok && hipGetDevice(&cur) == hipSuccess && cur != prev && prev >= 0) (void)hipSetDevice(prev);
  }
};

// One bin subset per record length n_samples / 2^j.
struct Level {
  int n_t = 0;
  int stride = 1;        // 2^j
  int n_sel = 0;
  int32_t* d_ksel = nullptr;  // bin k on the level's own grid
  double* d_kz = nullptr;     // [n_sel][kz_row(N)] signed kz / (2 pi) of the selected bins
  double* d_kzff = nullptr;   // [n_sel][N2][N1] the same values at q = N2 q1 + q2 (factored kernels)
  int32_t* d_ev = nullptr;    // [n_sel] 1 if any lateral wavenumber of the bin is evanescent
};

bool finite_pos(double v) { return std::isfinite(v) && v > 0.0; }
bool is_pow2(int v) { return v > 0 && (v & (v - 1)) == 0; }
int ilog2(int v) {
  int r = 0;
  while ((1 << r) < v) ++r;
  return r;
}
size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

// round-to-nearest-even FP32 -> BF16 / FP16 bit patterns, and back
uint16_t to_bf16(float f) {
  uint32_t u;
  std::memcpy(&u, &f, 4);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
float from_bf16(uint16_t h) {
  const uint32_t u = (uint32_t)h << 16;
  float f;
  std::memcpy(&f, &u, 4);
  return f;
}
uint16_t to_fp16(float f) {
  const _Float16 h = (_Float16)f;
  uint16_t u;
  std::memcpy(&u, &h, 2);
  return u;
}
float from_fp16(uint16_t u) {
  _Float16 h;
  std::memcpy(&h, &u, 2);
  return (float)h;
}
bool is_split(int prec) { return prec != PAM_PREC_FP32; }
bool is_fp16(int prec) { return prec == PAM_PREC_SPLIT_FP16 || prec == PAM_PREC_FP16; }

}  // namespace

struct pam_plan_s {
  int device = 0;
  int L = 0, n_t = 0, N = 0, n_z = 0, n_sub = 0, n_bins = 0;
  double eps = 1e-3;
  int precision = 0, zero_evanescent = 0;
  int coherence = 0;          // adjacent-pixel cross-spectra with the n_sub = 1 sums
  std::vector<int32_t> bins;  // k on the plan grid
  std::vector<Level> levels;
  // device tables
  double* d_z = nullptr;       // [n_z]
  float2* d_tw = nullptr;      // [n_t/2] time-FFT twiddles
  float2* d_twx = nullptr;     // [N] lateral DFT twiddles
  float* d_masks = nullptr;    // [n_sub][L]
  int32_t col0 = 0, col_step = 1;  // grid column of element l: col0 + col_step * l
  uint16_t* d_bhi = nullptr;   // [N/8][N][8] basis (slot groups, x, slots), 16-bit hi (split kernels)
  uint16_t* d_blo = nullptr;   // same layout, 16-bit lo
  bool ff = false;             // factored inverse lateral transform: FP32, and the 16-bit forms at N = 256, 512
  uint16_t* d_ff_w16 = nullptr;  // [64][2][16] the same in 16-bit operand order, hi then lo per k-step
  float2* d_ff_tw = nullptr;   // [64][8] twiddles / 16 in stage-1 output order
  float2* d_ff_tw2 = nullptr;  // [64][8] N = 512 combination twiddles in stage-3 output order
  float2* d_ff_tw_vec = nullptr;  // [16][16] stage twiddles of the vector FFT kernel
  float2* d_ff_tw2_vec = nullptr;  // [16][16] N = 512 combination twiddles of the vector FFT kernel
  // frequency-domain delay-and-sum (pam_fd_tea_tax)
  double fs = 0, c = 0;        // sampling rate, sound speed
  double dx = 0;               // lateral grid spacing
  int32_t* d_units = nullptr;  // [(L + 7) / 8] sub-aperture sets of eight elements (tea_unit_code)
  bool mixed_units = false;    // some of the eight belong to different sets
  int k3_slots = 512;          // K3 workgroups resident on the device at once
  int n_cus = 256;             // compute units of the plan's device
  std::vector<void*> allocs;
};

namespace {

// allocation-failure injection for tests (pam_debug_fail_allocation) and the count of
// device allocations the library's plans hold (pam_debug_live_allocations)
std::atomic<int> g_fail_alloc{-1};
std::atomic<long long> g_live_allocs{0};

void free_plan(pam_plan_s* p) {
  if (!p) return;
  for (void* q : p->allocs) {
    (void)hipFree(q);
    --g_live_allocs;
  }
  delete p;
}

template <typename T>
pam_status_t upload(pam_plan_s* p, T** dst, const T* src, size_t n) {
  void* ptr = nullptr;
  const size_t bytes = std::max<size_t>(n, 1) * sizeof(T);
  int armed = g_fail_alloc.load();
  while (armed >= 0 && !g_fail_alloc.compare_exchange_weak(armed, armed - 1)) {
  }
  if (armed == 0) return PAM_ERR_OOM;  // injected failure (the counter is now disarmed)
  if (hipMalloc(&ptr, bytes) != hipSuccess) return PAM_ERR_OOM;
  p->allocs.push_back(ptr);
  ++g_live_allocs;
  if (n && hipMemcpy(ptr, src, n * sizeof(T), hipMemcpyHostToDevice) != hipSuccess) return PAM_ERR_DEVICE;
  *dst = static_cast<T*>(ptr);
  return PAM_OK;
}

// The vector FFT kernel's table for N columns, K = N / 16 (N / 32 beyond 256) points in stage 3.  K = 16 and 8: per row
// x1 the constants idft16_tw / idft8_tw fold the twiddles with, float4 k of row x1 at [k][x1].  Other K, and plain: the twiddles
// e^{2 pi i q2 x1 / 16 K} at [x1][j], q2 = j % CW the stage-1 column of lane j (K of the CW lanes of a depth hold one, the
// others a zero).
std::vector<float2> ft_table(int N, bool plain) {
  const int K = N > 256 ? N / 32 : N / 16, CW = K <= 2 ? 2 : (K <= 4 ? 4 : (K <= 8 ? 8 : 16));
  if (plain || (K != 16 && K != 8)) {
    std::vector<float2> tw(256, make_float2(0.f, 0.f));
    for (int x1 = 0; x1 < 16; ++x1)
      for (int j = 0; j < 16; ++j) {
        const int q2 = j % CW;
        const double th = 2.0 * kPi * (double)(q2 * x1) / (double)(16 * K);
        if (q2 < K) tw[x1 * 16 + j] = make_float2((float)std::cos(th), (float)std::sin(th));
      }
    return tw;
  }
  const int n4 = K == 16 ? 10 : 4;
  std::vector<float2> tw(n4 * 32);
  float* out = &tw[0].x;
  for (int x1 = 0; x1 < 16; ++x1) {
    double c[16], t[16];
    for (int n = 0; n < K; ++n) {
      const int turn = n * x1 % (16 * K);                       // of 16 K
      const double th = 2.0 * kPi * (double)turn / (double)(16 * K);
      const bool quarter = turn == 4 * K || turn == 12 * K;     // exact zero of the cosine
      c[n] = quarter ? std::ldexp(1.0, -30) : std::cos(th);
      t[n] = (quarter ? (turn == 4 * K ? 1.0 : -1.0) : std::sin(th)) / c[n];
    }
    const double C1 = std::cos(kPi / 8), S1 = std::sin(kPi / 8), R2 = std::cos(kPi / 4);
    double v[40] = {};
    if (K == 16) {
      const double s1 = c[1], s2 = c[2], rho = c[3] / c[1];
      const double q[9] = {s1, s2, rho, C1 * s1, R2 * s2, S1 / C1 * rho, R2 * s1, S1 * s1, -C1 / S1 * rho};
      for (int n2 = 0; n2 < 4; ++n2) {
        for (int n1 = 0; n1 < 4; ++n1) v[8 * n2 + n1] = t[4 * n1 + n2];
        v[8 * n2 + 4] = c[8 + n2] / c[n2];
        v[8 * n2 + 5] = c[4 + n2] / c[n2];
        v[8 * n2 + 6] = c[12 + n2] / c[4 + n2];
        v[8 * n2 + 7] = q[n2];
      }
      std::copy(q + 4, q + 9, v + 32);
    } else {
      for (int n = 1; n < 8; ++n) v[n - 1] = t[n];
      for (int n2 = 0; n2 < 4; ++n2) v[7 + n2] = c[4 + n2] / c[n2];
      const double q[4] = {c[1], c[2], c[3] / c[1], R2 * c[1]};
      std::copy(q, q + 4, v + 11);
    }
    for (int k = 0; k < n4; ++k)
      for (int e = 0; e < 4; ++e) out[(k * 16 + x1) * 4 + e] = (float)v[4 * k + e];
  }
  return tw;
}

pam_status_t validate(const pam_geometry_t* g) {
  if (!g) return PAM_ERR_INVALID_ARG;
  if (g->n_elements < 1 || !finite_pos(g->pitch_m) || !finite_pos(g->fs_hz) || !finite_pos(g->c_mps))
    return PAM_ERR_INVALID_ARG;
  if (g->n_samples < 2) return PAM_ERR_INVALID_ARG;
  if (!is_pow2(g->n_samples) || g->n_samples < kMinSamples || g->n_samples > kMaxSamples)
    return PAM_ERR_UNSUPPORTED;
  if (g->n_bands < 1 || !g->band_lo_hz || !g->band_hi_hz) return PAM_ERR_INVALID_ARG;
  for (int b = 0; b < g->n_bands; ++b) {
    const double lo = g->band_lo_hz[b], hi = g->band_hi_hz[b];
    if (!std::isfinite(lo) || !std::isfinite(hi) || lo < 0.0 || hi < lo) return PAM_ERR_INVALID_ARG;
  }
  if (g->n_depths < 1 || !g->depths_m) return PAM_ERR_INVALID_ARG;
  for (int d = 0; d < g->n_depths; ++d)
    if (!std::isfinite(g->depths_m[d]) || g->depths_m[d] < 0.0) return PAM_ERR_INVALID_ARG;
  if (g->n_x < g->n_elements || g->n_x < 2) return PAM_ERR_INVALID_ARG;
  if (g->n_x % 32 != 0 || g->n_x > kMaxNx) return PAM_ERR_UNSUPPORTED;
  if (g->lateral != PAM_LATERAL_PAD && g->lateral != PAM_LATERAL_STUFF) return PAM_ERR_INVALID_ARG;
  if (g->lateral == PAM_LATERAL_STUFF && g->n_x % g->n_elements != 0) return PAM_ERR_INVALID_ARG;
  if (g->n_sub < 1 || g->n_sub > 3) return PAM_ERR_INVALID_ARG;
  if (g->apod) {
    for (int i = 0; i < g->n_sub * g->n_elements; ++i)
      if (g->apod[i] > 1) return PAM_ERR_INVALID_ARG;
  } else if (g->pattern_m < 0) {
    return PAM_ERR_INVALID_ARG;
  }
  if (!(g->eps >= 0.0 && g->eps < 1.0)) return PAM_ERR_INVALID_ARG;
  if (g->precision < PAM_PREC_FP32 || g->precision > PAM_PREC_FP16) return PAM_ERR_INVALID_ARG;
  if (g->evanescent != PAM_EVAN_DECAY && g->evanescent != PAM_EVAN_ZERO) return PAM_ERR_INVALID_ARG;
  if (g->coherence != 0 && g->coherence != 1) return PAM_ERR_INVALID_ARG;
  if (g->coherence && (g->n_sub != 1 || g->n_x != 256 || (g->n_depths & 1))) return PAM_ERR_UNSUPPORTED;
  return PAM_OK;
}

// bins 0 < k < n_t/2 whose frequency k*fs/n_t lies in a closed band
std::vector<int32_t> select_bins(const pam_geometry_t* g) {
  std::vector<int32_t> ks;
  for (int k = 1; k < (g->n_samples + 1) / 2; ++k) {
    const double f = ((double)k * g->fs_hz) / (double)g->n_samples;
    for (int b = 0; b < g->n_bands; ++b) {
      if (g->band_lo_hz[b] <= f && f <= g->band_hi_hz[b]) {
        ks.push_back(k);
        break;
      }
    }
  }
  return ks;
}

struct LaunchShape {
  int n_dt, nw, xt, n_xg, n_split, bins_per_split;
  int ct;   // > 0: 16-depth kernels with ct 16-column tiles per consumer wave
  int fw;   // < 0: a factored kernel (k3fft, k3ff), all columns in a workgroup
};

// Workgroup tiling of one frame: depth tiles x column groups, before any bin split.
LaunchShape k3_tiles(const pam_plan_s* p) {
  LaunchShape s;
  s.xt = 1;
  s.ct = 0;
  s.fw = 0;
  if (p->ff) {
    // all columns per workgroup
    s.fw = -1;
    s.nw = pam::kFfWaves;
    const int dpw = pam::ft_depths_of(p->N);     // k3ff's at N = 256 and 512 too
    s.n_dt = (p->n_z + dpw - 1) / dpw;
    s.n_xg = 1;
  } else if (p->N % 64 == 0) {
    // 16 depths x 64 ct columns per workgroup (4 consumer + 4 producer waves)
    s.ct = p->N % 128 == 0 ? 2 : 1;
    s.nw = 4;
    s.n_dt = (p->n_z + 15) / 16;
    s.n_xg = p->N / (64 * s.ct);
  } else {
    // 32 depths x 32 nw columns per workgroup (nw consumer + nw producer waves)
    s.n_dt = (p->n_z + 31) / 32;
    const int tiles = p->N / 32;
    s.nw = (tiles % 4 == 0) ? 4 : (tiles % 2 == 0 ? 2 : 1);
    s.n_xg = p->N / (32 * s.nw * s.xt);
  }
  s.n_split = 1;
  s.bins_per_split = 0;
  return s;
}

int n_acc(int n_sub, int coherence = 0) { return n_sub == 3 ? 6 : (n_sub == 2 ? 3 : (coherence ? 5 : 1)); }

// Partial-sum planes a group's workspace holds beyond one per frame: room for two rounds of
// extra workgroups.  A group of F frames splits its bins at most 1 + spare / F ways, so its
// accumulator region (F + spare planes) and with it the workspace size never shrink as F
// grows: a workspace sized for F frames serves every call of fewer frames.
//
// The FP32 plans at sizes other than 128, 256 and 512 have few, wide workgroups per frame and so reserve many
// planes.  Where a caller's workspace (or the allocation-free entry point's scratch) does not hold that, the call
// runs with a smaller reservation (full = false), sized as for workgroups of 16 x 64 pixels (16 x 128 at 384
// columns, 32 x 32 where 64 does not divide N) on a device that holds 256 to 1,024 of them: its bins then split
// fewer ways, and the results differ by the order of the FP32 sums.
int64_t k3_spare_planes(const pam_plan_s* p, bool full = true) {
  const LaunchShape t = k3_tiles(p);
  const int64_t tiles = (int64_t)t.n_dt * t.n_xg;
  const int64_t spare = (2 * (int64_t)std::max(1, p->k3_slots) + tiles - 1) / tiles;
  if (is_split(p->precision) || p->N == 128 || p->N == 256 || p->N == 512) return spare;
  int64_t small_tiles, slots;
  if (p->N % 64 == 0) {
    const int cols = p->N % 128 == 0 ? 128 : 64;
    small_tiles = (int64_t)((p->n_z + 15) / 16) * (p->N / cols);
    slots = (cols == 64 ? 1280 : 1024) - 256 * p->n_sub;          // 1,024, 768, 512 or 768, 512, 256
  } else {
    small_tiles = (int64_t)((p->n_z + 31) / 32) * (p->N / 32);
    slots = p->n_sub == 1 ? 1024 : 512;
  }
  const int64_t small = (2 * slots + small_tiles - 1) / small_tiles;
  return full ? std::max(spare, small) : small;
}

// Estimated time of a K3 launch under the bins-per-workgroup cap b, in bin-times of a workgroup that has its CU to
// itself (measured 1.8, 2.8 and 4.0 us with one, two and three sub-apertures at 256 columns in FP32).  A CU's second and
// third workgroup slow each other down: a bin then takes 1.3 and 1.7 times as long (16-bit operands 1.65 and more), so
// workgroups beyond one per CU give much less than those up to it.  Four bin-times go to a launch's start and its end,
// two and a half to each further round, and every split adds a partial-sum plane per frame that K3 writes and K4 reads
// (2.5 TB/s for both).  Several groups of unequal workgroups: the work over the slots plus 0.7 of a longest workgroup.
double k3_time(const pam_plan_s* p, const int64_t* F, const int* n_sel, int n, int b) {
  const LaunchShape t = k3_tiles(p);
  const double tiles = (double)t.n_dt * t.n_xg, cus = std::max(1, p->n_cus);
  const int occ = std::max(1, p->k3_slots / std::max(1, p->n_cus));
  const double crowd = is_split(p->precision) ? 0.65 : 0.35;
  const auto bin_time = [&](int m) { return m == 0 ? 0.0 : 1.0 + crowd * (m - 1); };
  const double us = p->n_sub == 3 ? 4.0 : (p->n_sub == 2 ? 2.8 : 1.8);
  const double plane = (double)n_acc(p->n_sub, p->coherence) * p->n_z * p->N * 4.0 / 2.5e12 * 1e6 / us;
  double wg = 0, work = 0, planes = 0;
  int job = 0, live = 0;
  for (int g = 0; g < n; ++g) {
    if (F[g] == 0 || n_sel[g] == 0) continue;
    const int split = (n_sel[g] + b - 1) / b, bins = (n_sel[g] + split - 1) / split;
    ++live;
    wg += F[g] * tiles * split;
    work += F[g] * tiles * split * bins;
    planes += (double)F[g] * split;
    job = std::max(job, bins);
  }
  double k3 = 4.0;
  if (live > 1) {
    k3 += (work + 2.5 * wg) * bin_time(occ) / (occ * cus) + 0.7 * job;
  } else {
    const double per_cu = std::ceil(wg / cus), rounds = std::ceil(per_cu / occ);
    const double full = std::floor(per_cu / occ);
    k3 += 2.5 * (rounds - 1) + job * (full * bin_time(occ) + bin_time((int)(per_cu - full * occ)));
  }
  return k3 + plane * planes;
}

// The bin split of a K3 launch over n groups of frames (F[g] frames of n_sel[g] bins).
// A frame is tiles = n_dt n_xg workgroups; splitting its bins s ways makes s workgroups of
// ceil(n_sel / s) bins each, whose partial sums K4 adds.  The device holds p->k3_slots
// workgroups at once, so near-equal workgroups run in rounds: n workgroups of at most b bins
// take about ceil(n / slots) (b + c) bin-times, c (two bins) standing for a workgroup's
// start and its partial-sum write, and every split beyond the first costs K4 one more
// partial-sum plane per frame (n_acc pix floats, read at about 4 TB/s against about 5 us
// per bin).  Returns the bins-per-workgroup cap b (every group splits into ceil(n_sel / b)
// parts) that minimises the estimate, the largest such b on ties, among the caps whose
// splits fit the spare planes: at least 8 bins in *cap8, with its cost, and at least 4 in
// *cap4 (or the widest band when narrower).
void k3_caps(const pam_plan_s* p, const int64_t* F, const int* n_sel, int n, bool full, int* cap8, double* cost8,
             int* cap4) {
  const LaunchShape t = k3_tiles(p);
  const int64_t tiles = (int64_t)t.n_dt * t.n_xg;
  const int64_t spare = k3_spare_planes(p, full);
  int max_n = 0;
  for (int g = 0; g < n; ++g) max_n = std::max(max_n, n_sel[g]);
  *cap8 = *cap4 = std::max(1, max_n);
  *cost8 = 0;
  if (max_n == 0) return;
  const double slots = std::max(1, p->k3_slots);
  const double plane_cost = (double)n_acc(p->n_sub, p->coherence) * p->n_z * p->N * 4.0 / 4e12 / 5e-6;
  // The estimate is constant between the caps where some group's split count changes, so it is evaluated at the
  // top of each such piece: for every group g and split count s, the largest cap that splits g s ways
  // (n_g for s = 1, ceil(n_g / (s - 1)) - 1 after), in decreasing order (a merge over the groups' sequences,
  // no storage).  This equals trying every cap.
  const int min8 = std::min(8, max_n), min4 = std::min(4, max_n);
  auto top = [&](int g, int s) { return s == 1 ? n_sel[g] : (n_sel[g] + s - 2) / (s - 1) - 1; };
  int next_s[pam::kMaxGroups];
  int live = 0;
  for (int g = 0; g < n; ++g) {
    next_s[g] = 1;
    live += F[g] > 0 && n_sel[g] > 0;
  }
  double best = 0;
  for (bool first = true;; first = false) {
    int b = -1;
    for (int g = 0; g < n; ++g)
      if (F[g] > 0 && n_sel[g] > 0) b = std::max(b, top(g, next_s[g]));
    if (first) b = max_n;
    if (b < min4) break;
    for (int g = 0; g < n; ++g)      // step every group past this cap
      if (F[g] > 0 && n_sel[g] > 0)
        while (top(g, next_s[g]) >= b) ++next_s[g];
    int64_t n_wg = 0;
    int job = 0;
    double k4 = 0, work = 0;
    bool fits = true;
    for (int g = 0; g < n; ++g) {
      if (F[g] == 0 || n_sel[g] == 0) continue;
      const int split = (n_sel[g] + b - 1) / b;
      const int bins = (n_sel[g] + split - 1) / split;
      fits = fits && (int64_t)(split - 1) * F[g] <= spare;
      n_wg += F[g] * tiles * split;
      work += (double)F[g] * tiles * split * (bins + 2.0);
      job = std::max(job, bins);
      k4 += plane_cost * (double)F[g] * (split - 1);
    }
    if (!fits) break;                      // smaller caps split further still
    // equal workgroups (one group) run in rounds; unequal ones (several groups, longest first) take about
    // their total work over the slots plus one longest workgroup
    const double cost = live > 1 ? work / slots + (job + 2.0) + k4 : std::ceil((double)n_wg / slots) * (job + 2.0) + k4;
    if (b == max_n || cost < best - 1e-9) {
      best = cost;
      *cap4 = b;
      if (b >= min8) {
        *cap8 = b;
        *cost8 = cost;
      }
    }
  }
}

// The cap of a launch: the estimate's with at least 8 bins a workgroup, or with at least 4 where k3_time finds that
// faster by 7 % (its spread).  Down to 4 gains where CUs stand empty (one frame of 151 x 128 pixels and 205 bins 53.1 ->
// 45.7 us, one of 93 x 384 82.1 -> 65.9; over 300 drawn calls 1.18 on average where the two differ) and loses where each CU
// has a workgroup already (19 frames of 166 x 128 and 13 bins with two sub-apertures: 39.0 us in two splits, 44.7 in
// four); 2 bins measure the same as 4 or worse.  Plans with coherence keep 8: their sums become BF16 features, where
// another order of the FP32 sums moves the network's output.  *cost_out: the estimate at 8.
int k3_bin_cap(const pam_plan_s* p, const int64_t* F, const int* n_sel, int n, double* cost_out = nullptr,
               bool full = true) {
  int b8, b4;
  double cost;
  k3_caps(p, F, n_sel, n, full, &b8, &cost, &b4);
  if (cost_out) *cost_out = cost;
  if (b4 >= b8 || p->coherence) return b8;
  return k3_time(p, F, n_sel, n, b4) < 0.93 * k3_time(p, F, n_sel, n, b8) ? b4 : b8;
}

// The launch shape of one group: its tiling, and its bins split under the cap b.
LaunchShape k3_shape(const pam_plan_s* p, int n_sel, int b) {
  LaunchShape s = k3_tiles(p);
  if (n_sel == 0) {
    s.n_split = 1;
    s.bins_per_split = 0;
    return s;
  }
  const int split = (n_sel + b - 1) / b;
  s.bins_per_split = (n_sel + split - 1) / split;
  s.n_split = (n_sel + s.bins_per_split - 1) / s.bins_per_split;
  return s;
}

const Level* level_for(const pam_plan_s* p, int n_t) {
  for (const Level& lv : p->levels)
    if (lv.n_t == n_t) return &lv;
  return nullptr;
}

// bin_cap: the bins-per-workgroup cap of the launch this group is part of (-1: the group alone)
pam_status_t layout(const pam_plan_s* p, int64_t F, int n_t, pam_workspace_layout_t* out, int bin_cap = -1,
                    bool full = true) {
  const Level* lv = level_for(p, n_t);
  if (!lv) return PAM_ERR_INVALID_ARG;
  if (bin_cap < 0) bin_cap = k3_bin_cap(p, &F, &lv->n_sel, 1, nullptr, full);
  const LaunchShape s = k3_shape(p, lv->n_sel, bin_cap);
  const size_t pix = (size_t)p->n_z * p->N;
  const size_t n_blk = (pix + 255) / 256;
  pam_workspace_layout_t L{};
  size_t o = 0;
  L.spectra = o;  o = align256(o + (size_t)F * lv->n_sel * p->L * sizeof(float2));
  L.coeffs = o;   o = align256(o + (size_t)F * lv->n_sel * p->n_sub * p->N * sizeof(float2));
  L.scales = o;   o = align256(o + (size_t)F * lv->n_sel * sizeof(float));
  const size_t planes = F > 0 ? (size_t)F + (size_t)k3_spare_planes(p, full) : 0;   // >= n_split F
  L.accum = o;    o = align256(o + planes * n_acc(p->n_sub, p->coherence) * pix * sizeof(float));
  L.energy = o;   o = align256(o + (size_t)F * pix * sizeof(float));
  L.weight = o;   o = align256(o + (size_t)F * pix * sizeof(float));
  L.blockmax = o; o = align256(o + (size_t)F * n_blk * sizeof(float));
  L.total = std::max<size_t>(o, 256);
  L.n_sel = lv->n_sel;
  L.n_split = s.n_split;
  L.n_acc = n_acc(p->n_sub, p->coherence);
  *out = L;
  return PAM_OK;
}

// The layout of a call in a workspace of ws_bytes bytes: the full reservation where it fits, else the smaller one
// (PAM_ERR_WORKSPACE, *out still set to it, where that does not fit either).
pam_status_t layout_in(const pam_plan_s* p, int64_t F, int n_t, size_t ws_bytes, pam_workspace_layout_t* out) {
  pam_status_t st = layout(p, F, n_t, out);
  if (st == PAM_OK && out->total > ws_bytes) st = layout(p, F, n_t, out, -1, false);
  return st == PAM_OK && out->total > ws_bytes ? PAM_ERR_WORKSPACE : st;
}

// Where a K3 dispatch goes: a launch on stream st, or, with occ set, no launch but the
// number of the kernel's workgroups one CU holds (written to *occ).  n_cus: compute units of the launch's device.
struct Target {
  hipStream_t st;
  int* occ;
  int n_cus = 0;
};

// K3 kernels: NC consumer + NC producer waves, NC*32 columns per workgroup.
// LDS above 64 KiB needs the per-kernel attribute.
// (Every kernel shares one signature, so the attribute is set per launch rather
// than cached in a per-instantiation static.)
template <typename K>
hipError_t launch_with_lds(K kernel, int nc, size_t lds, const pam::K3Args& a, int blocks, Target st) {
  const hipError_t attr =
      hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (attr != hipSuccess) return attr;
  if (st.occ)
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(st.occ, reinterpret_cast<const void*>(kernel), nc * 128, lds);
  hipLaunchKernelGGL(kernel, dim3(blocks), dim3(nc * 128), lds, st.st, a);
  return hipGetLastError();
}

template <int NSUB, int NC>
hipError_t launch_prec(int precision, const pam::K3Args& a, int blocks, Target st) {
  switch (precision) {
    case PAM_PREC_SPLIT_BF16:
      return launch_with_lds(pam::k3_fields_split<__bf16, 3, NSUB, NC>, NC, pam::k3_split_lds<3, NSUB, NC>(), a, blocks, st);
    case PAM_PREC_SPLIT_FP16:
      return launch_with_lds(pam::k3_fields_split<_Float16, 3, NSUB, NC>, NC, pam::k3_split_lds<3, NSUB, NC>(), a, blocks, st);
    case PAM_PREC_BF16:
      return launch_with_lds(pam::k3_fields_split<__bf16, 1, NSUB, NC>, NC, pam::k3_split_lds<1, NSUB, NC>(), a, blocks, st);
    case PAM_PREC_FP16:
      return launch_with_lds(pam::k3_fields_split<_Float16, 1, NSUB, NC>, NC, pam::k3_split_lds<1, NSUB, NC>(), a, blocks, st);
    default: return hipErrorInvalidValue;          // FP32 takes the factored kernel at every N
  }
}

template <int NSUB, int CT>
hipError_t launch_prec16(int precision, const pam::K3Args& a, int blocks, Target st) {
  switch (precision) {
    case PAM_PREC_SPLIT_BF16:
      return launch_with_lds(pam::k3f16_split<__bf16, 3, NSUB, CT>, 4, pam::k3f16_split_lds<3, NSUB, CT>(), a, blocks, st);
    case PAM_PREC_SPLIT_FP16:
      return launch_with_lds(pam::k3f16_split<_Float16, 3, NSUB, CT>, 4, pam::k3f16_split_lds<3, NSUB, CT>(), a, blocks, st);
    case PAM_PREC_BF16:
      return launch_with_lds(pam::k3f16_split<__bf16, 1, NSUB, CT>, 4, pam::k3f16_split_lds<1, NSUB, CT>(), a, blocks, st);
    case PAM_PREC_FP16:
      return launch_with_lds(pam::k3f16_split<_Float16, 1, NSUB, CT>, 4, pam::k3f16_split_lds<1, NSUB, CT>(), a, blocks, st);
    default: return hipErrorInvalidValue;
  }
}

// Kernels with more than 64 KB of dynamic LDS: the attribute is set before each launch.
template <typename K>
hipError_t launch_big_lds(K kernel, int nw, size_t lds, const pam::K3Args& a, const pam::K3Groups& grp, int blocks,
                          Target st) {
  const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                              hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (attr != hipSuccess) return attr;
  if (st.occ)
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(st.occ, reinterpret_cast<const void*>(kernel), nw * 64, lds);
  hipLaunchKernelGGL(kernel, dim3(blocks), dim3(nw * 64), lds, st.st, a, grp);
  return hipGetLastError();
}

template <int NSUB, int R>
hipError_t launch_ff_r(int precision, const pam::K3Args& a, const pam::K3Groups& grp, int blocks, Target st) {
  using namespace pam;
  const size_t lds = k3ff_lds<NSUB, R>();
  switch (precision) {
    case PAM_PREC_SPLIT_BF16: return launch_big_lds(k3ff<__bf16, 3, NSUB, false, R>, kFfWaves, lds, a, grp, blocks, st);
    case PAM_PREC_SPLIT_FP16: return launch_big_lds(k3ff<_Float16, 3, NSUB, false, R>, kFfWaves, lds, a, grp, blocks, st);
    case PAM_PREC_BF16: return launch_big_lds(k3ff<__bf16, 1, NSUB, false, R>, kFfWaves, lds, a, grp, blocks, st);
    case PAM_PREC_FP16: return launch_big_lds(k3ff<_Float16, 1, NSUB, false, R>, kFfWaves, lds, a, grp, blocks, st);
    default: return hipErrorInvalidValue;
  }
}

// FP32 operands: the vector FFT kernel of the plan's lateral size.
template <int NSUB, int NN = 32>
hipError_t launch_fft(const pam::K3Args& a, const pam::K3Groups& grp, int blocks, Target st) {
  if (a.N == NN)
    return launch_big_lds(pam::k3fft<NSUB, false, NN>, pam::kFtWaves, pam::k3fft_lds<NSUB, NN>(), a, grp, blocks, st);
  if constexpr (NN < kMaxNx) return launch_fft<NSUB, NN + 32>(a, grp, blocks, st);
  return hipErrorInvalidValue;
}

template <int NSUB>
hipError_t launch_ff(int precision, const pam::K3Args& a, const pam::K3Groups& grp, int blocks, Target st) {
  if (precision == PAM_PREC_FP32) return launch_fft<NSUB>(a, grp, blocks, st);
  return a.N == 512 ? launch_ff_r<NSUB, 2>(precision, a, grp, blocks, st)
                    : launch_ff_r<NSUB, 1>(precision, a, grp, blocks, st);
}

template <int NSUB>
hipError_t launch_shape(int precision, const LaunchShape& s, const pam::K3Args& a, const pam::K3Groups& grp,
                        int blocks, Target st) {
  if (s.fw < 0) return launch_ff<NSUB>(precision, a, grp, blocks, st);
  if (grp.n > 0) return hipErrorInvalidValue;      // grouped work lists run on the factored kernels only
  if (s.ct == 2) return launch_prec16<NSUB, 2>(precision, a, blocks, st);
  if (s.ct == 1) return launch_prec16<NSUB, 1>(precision, a, blocks, st);
  if (s.nw == 4) return launch_prec<NSUB, 4>(precision, a, blocks, st);
  if (s.nw == 2) return launch_prec<NSUB, 2>(precision, a, blocks, st);
  return launch_prec<NSUB, 1>(precision, a, blocks, st);
}

// K2 of the factored plans: the lateral FFT kernel of the plan's size.
template <int NSUB, int NN = 32>
bool launch_k2(int n, dim3 grid, hipStream_t stream, const pam::K2Args& a) {
  if (n == NN) {
    hipLaunchKernelGGL((pam::k2_fft<NSUB, NN / 16>), grid, dim3(256), 0, stream, a);
    return true;
  }
  if constexpr (NN < kMaxNx) return launch_k2<NSUB, NN + 32>(n, grid, stream, a);
  return false;
}

hipError_t launch_k3(int precision, int n_sub, const LaunchShape& s, const pam::K3Args& a, const pam::K3Groups& grp,
                     int blocks, Target st, int coherence) {
  if (coherence) {
    using namespace pam;
    const size_t lds = k3ff_lds<1>();
    switch (precision) {
      case PAM_PREC_SPLIT_BF16: return launch_big_lds(k3ff<__bf16, 3, 1, true>, kFfWaves, lds, a, grp, blocks, st);
      case PAM_PREC_SPLIT_FP16: return launch_big_lds(k3ff<_Float16, 3, 1, true>, kFfWaves, lds, a, grp, blocks, st);
      case PAM_PREC_BF16: return launch_big_lds(k3ff<__bf16, 1, 1, true>, kFfWaves, lds, a, grp, blocks, st);
      case PAM_PREC_FP16: return launch_big_lds(k3ff<_Float16, 1, 1, true>, kFfWaves, lds, a, grp, blocks, st);
      default:
        // the form of which three workgroups fit a CU where that saves a round: at three per CU and beyond four (at k3fft)
        if (const int per_cu = st.n_cus > 0 ? (blocks + st.n_cus - 1) / st.n_cus : 0; per_cu == 3 || per_cu > 4)
          return launch_big_lds(k3fft<1, true, 256, true>, kFtWaves, k3fft_lds<1, 256, true>(), a, grp, blocks, st);
        return launch_big_lds(k3fft<1, true>, kFtWaves, k3fft_lds<1, 256, true>(), a, grp, blocks, st);
    }
  }
  switch (n_sub) {
    case 3: return launch_shape<3>(precision, s, a, grp, blocks, st);
    case 2: return launch_shape<2>(precision, s, a, grp, blocks, st);
    default: return launch_shape<1>(precision, s, a, grp, blocks, st);
  }
}

}  // namespace

extern "C" {

const char* pam_status_string(pam_status_t s) {
  switch (s) {
    case PAM_OK: return "ok";
    case PAM_ERR_INVALID_ARG: return "invalid argument";
    case PAM_ERR_OOM: return "out of memory";
    case PAM_ERR_DEVICE: return "device error";
    case PAM_ERR_UNSUPPORTED: return "unsupported size or mode";
    case PAM_ERR_WORKSPACE: return "workspace missing or too small";
  }
  return "unknown status";
}

pam_status_t pam_plan(const pam_geometry_t* g, int device, pam_plan_t* out) {
  if (!out) return PAM_ERR_INVALID_ARG;
  *out = nullptr;
  pam_status_t st = validate(g);
  if (st != PAM_OK) return st;
  std::vector<int32_t> ks = select_bins(g);
  if (ks.empty()) return PAM_ERR_INVALID_ARG;
  int n_dev = 0;
  if (hipGetDeviceCount(&n_dev) != hipSuccess || device < 0 || device >= n_dev) return PAM_ERR_DEVICE;
  DeviceGuard guard(device);
  if (!guard.ok) return PAM_ERR_DEVICE;

  pam_plan_s* p = new (std::nothrow) pam_plan_s();
  if (!p) return PAM_ERR_OOM;
  p->device = device;
  p->L = g->n_elements;
  p->n_t = g->n_samples;
  p->N = g->n_x;
  p->n_z = g->n_depths;
  p->n_sub = g->n_sub;
  p->n_bins = (int)ks.size();
  p->eps = g->eps > 0.0 ? g->eps : 1e-3;
  p->precision = g->precision;
  p->zero_evanescent = g->evanescent == PAM_EVAN_ZERO;
  p->coherence = g->coherence;
  p->bins = ks;
  const int L = p->L, N = p->N, HQ = N / 2 + 1;

  // lateral placement: grid column of each element and grid spacing
  double dx;
  if (g->lateral == PAM_LATERAL_PAD) {
    p->col0 = (N - L) / 2;
    p->col_step = 1;
    dx = g->pitch_m;
  } else {
    p->col0 = 0;
    p->col_step = N / L;
    dx = g->pitch_m / p->col_step;
  }
  p->fs = g->fs_hz;
  p->c = g->c_mps;
  p->dx = dx;
  // apodization masks: explicit or Pattern-m (a_i[l] = 1 iff floor(l/m) mod n == i)
  std::vector<float> masks((size_t)p->n_sub * L, 0.f);
  const int m = g->pattern_m > 0 ? g->pattern_m : 16;
  for (int i = 0; i < p->n_sub; ++i)
    for (int l = 0; l < L; ++l)
      masks[(size_t)i * L + l] = g->apod ? (float)g->apod[(size_t)i * L + l] : (((l / m) % p->n_sub) == i ? 1.f : 0.f);
  // kz / (2 pi) in cycles per metre for the folded half grid q = 0..N/2:
  // k / (2 pi) = f / c and kx_q / (2 pi) = q / (N dx); negative values mark
  // evanescent components (decay rate / (2 pi)).
  std::vector<double> kz((size_t)p->n_bins * HQ);
  for (int b = 0; b < p->n_bins; ++b) {
    const double f = ((double)ks[b] * g->fs_hz) / (double)g->n_samples;
    const double kc = f / g->c_mps;
    for (int q = 0; q < HQ; ++q) {
      const double kxc = (double)q / ((double)N * dx);
      const double d = kc * kc - kxc * kxc;
      kz[(size_t)b * HQ + q] = d >= 0.0 ? std::sqrt(d) : -std::sqrt(-d);
    }
  }
  std::vector<double> z(g->depths_m, g->depths_m + p->n_z);
  // transform tables from exact integer angles
  std::vector<float2> tw(p->n_t / 2), twx(N);
  for (int i = 0; i < p->n_t / 2; ++i) {
    const double a = 2.0 * kPi * (double)i / (double)p->n_t;
    tw[i] = make_float2((float)std::cos(a), (float)-std::sin(a));
  }
  for (int i = 0; i < N; ++i) {
    const double a = 2.0 * kPi * (double)i / (double)N;
    twx[i] = make_float2((float)std::cos(a), (float)-std::sin(a));
  }
  // Factored transform: FP32 at every N (vector FFT, k3_fft.hpp) and the 16-bit forms at N = 256 and 512
  // (k3_factored.hpp); the 16-bit forms' other sizes take the folded DFT basis (k3_fields*.hpp), built only for them.
  p->ff = !is_split(p->precision) || N == 256 || N == 512;
  std::vector<float> basis(p->ff ? 0 : (size_t)N * N);
  for (int s = 0; s < (p->ff ? 0 : N); ++s) {
    const int q = s >> 1;
    for (int x = 0; x < N; ++x) {
      double v;
      if ((s & 1) == 0) {
        v = std::cos(2.0 * kPi * (double)(((long long)q * x) % N) / (double)N);
      } else if (q == 0) {
        v = (x & 1) ? -1.0 : 1.0;  // cos(pi x)
      } else {
        v = std::sin(2.0 * kPi * (double)(((long long)q * x) % N) / (double)N);
      }
      basis[(size_t)s * N + x] = (float)v;
    }
  }

  std::vector<uint16_t> bhi, blo;
  if (is_split(p->precision) && !p->ff) {
    bhi.resize((size_t)N * N);
    blo.resize((size_t)N * N);
    const bool h16 = is_fp16(p->precision);
    for (int s = 0; s < N; ++s)
      for (int x = 0; x < N; ++x) {
        const float v = basis[(size_t)s * N + x];
        const uint16_t hi = h16 ? to_fp16(v) : to_bf16(v);
        const float r = v - (h16 ? from_fp16(hi) : from_bf16(hi));
        // groups of 8 slots, then x, then the 8 slots: one 16-byte piece per (group, x)
        const size_t o = ((size_t)(s / 8) * N + x) * 8 + s % 8;
        bhi[o] = hi;
        blo[o] = h16 ? to_fp16(r) : to_bf16(r);
      }
  }

  // Factored transform (N = 256 = 16 x 16; N = 512 as two such transforms over even and
  // odd q): the 16-point DFT matrix W(x, m) = e^{2 pi i m x / 16} in real form, rows
  // (x, re/im) = x + 16 ro, the stage twiddles and (N = 512) the combination twiddles, all
  // in lane order of the matrix-core operands.  Lane l: column c = l % 32, half h = l / 32.
  std::vector<uint16_t> ff_w16;
  std::vector<float2> ff_tw, ff_tw2, ff_tw_vec, ff_tw2_vec;
  if (p->ff && is_split(p->precision)) {
    auto wval = [](int row, int m, int ri) {
      const int x = row % 16, ro = row / 16;
      const double th = 2.0 * kPi * (double)((m * x) % 16) / 16.0;
      const double c = std::cos(th), sn = std::sin(th);
      return ro == 0 ? (ri == 0 ? c : -sn) : (ri == 0 ? sn : c);
    };
    ff_w16.resize(64 * 32);
    ff_tw.resize(64 * 8);
    const bool h16 = is_fp16(p->precision);
    for (int l = 0; l < 64; ++l) {
      const int c = l % 32, h = l / 32;
      // 16-bit k-step s, element j: k = 16s + 8h + j <-> m = 8h + 4s + j/2, re/im j%2
      for (int s2 = 0; s2 < 2; ++s2)
        for (int j = 0; j < 8; ++j) {
          const float v = (float)wval(c, 8 * h + 4 * s2 + j / 2, j % 2);
          const uint16_t hi = h16 ? to_fp16(v) : to_bf16(v);
          const float r = v - (h16 ? from_fp16(hi) : from_bf16(hi));
          ff_w16[l * 32 + s2 * 16 + j] = hi;
          ff_w16[l * 32 + s2 * 16 + 8 + j] = h16 ? to_fp16(r) : to_bf16(r);
        }
      // stage-1 output v (0..7) of lane l is x1 = 8(v/4) + 4h + v%4 of column q2 = c % 16
      for (int v = 0; v < 8; ++v) {
        const int x1 = 8 * (v / 4) + 4 * h + v % 4, q2 = c % 16;
        const double th = 2.0 * kPi * (double)((q2 * x1) % 256) / 256.0;
        const double sc = h16 ? 1.0 / 16.0 : 1.0;   // FP16 operands keep stage-1 results in range
        ff_tw[l * 8 + v] = make_float2((float)(std::cos(th) * sc), (float)(std::sin(th) * sc));
      }
    }
    // stage-3 output v of lane l is x' = c % 16 + 16 (8(v/4) + 4h + v%4) of half c / 16
    ff_tw2.assign(64 * 8, make_float2(0.f, 0.f));
    if (N == 512)
      for (int l = 0; l < 64; ++l)
        for (int v = 0; v < 8; ++v) {
          const int c = l % 32, h = l / 32, xp = c % 16 + 16 * (8 * (v / 4) + 4 * h + v % 4);
          const double th = 2.0 * kPi * (double)xp / 512.0;
          ff_tw2[l * 8 + v] = make_float2((float)std::cos(th), (float)std::sin(th));
        }
  } else if (p->ff) {
    // vector FFT kernel: stage-3 constants or twiddles and, beyond N = 256, [x2][j] = e^{2 pi i (j + 16 x2) / N}
    ff_tw_vec = ft_table(N, p->coherence != 0);
    ff_tw2_vec.assign(256, make_float2(0.f, 0.f));
    for (int x2 = 0; x2 < 16; ++x2)
      for (int j = 0; j < 16; ++j) {
        const double th = 2.0 * kPi * (double)(j + 16 * x2) / (double)N;
        if (N > 256) ff_tw2_vec[x2 * 16 + j] = make_float2((float)std::cos(th), (float)std::sin(th));
      }
  }

  do {
    if (is_split(p->precision) && !p->ff) {
      if ((st = upload(p, &p->d_bhi, bhi.data(), bhi.size())) != PAM_OK) break;
      if ((st = upload(p, &p->d_blo, blo.data(), blo.size())) != PAM_OK) break;
    }
    if (p->ff && is_split(p->precision)) {
      if ((st = upload(p, &p->d_ff_w16, ff_w16.data(), ff_w16.size())) != PAM_OK) break;
      if ((st = upload(p, &p->d_ff_tw, ff_tw.data(), ff_tw.size())) != PAM_OK) break;
      if ((st = upload(p, &p->d_ff_tw2, ff_tw2.data(), ff_tw2.size())) != PAM_OK) break;
    } else if (p->ff) {
      if ((st = upload(p, &p->d_ff_tw_vec, ff_tw_vec.data(), ff_tw_vec.size())) != PAM_OK) break;
      if ((st = upload(p, &p->d_ff_tw2_vec, ff_tw2_vec.data(), ff_tw2_vec.size())) != PAM_OK) break;
    }
    if ((st = upload(p, &p->d_z, z.data(), z.size())) != PAM_OK) break;
    if ((st = upload(p, &p->d_tw, tw.data(), tw.size())) != PAM_OK) break;
    if ((st = upload(p, &p->d_twx, twx.data(), twx.size())) != PAM_OK) break;
    if ((st = upload(p, &p->d_masks, masks.data(), masks.size())) != PAM_OK) break;
    {
      std::vector<int32_t> subs(L, 0);
      for (int i = 0; i < p->n_sub; ++i)
        for (int l = 0; l < L; ++l)
          if (masks[(size_t)i * L + l] != 0.f) subs[l] |= 1 << i;
      std::vector<int32_t> units;
      for (int l = 0; l < L; l += 8) units.push_back(pam::tea_unit_code(subs.data() + l, std::min(8, L - l)));
      for (int32_t c : units) p->mixed_units |= (c >> 24) == pam::kTeaMixed;
      if ((st = upload(p, &p->d_units, units.data(), units.size())) != PAM_OK) break;
    }
    // bin subsets for records of n_t / 2^j samples
    for (int stride = 1; p->n_t / stride >= kMinSamples; stride <<= 1) {
      Level lv;
      lv.n_t = p->n_t / stride;
      lv.stride = stride;
      std::vector<int32_t> ksel;
      std::vector<double> kz_lv;
      for (int b = 0; b < p->n_bins; ++b)
        if (ks[b] % stride == 0) {
          ksel.push_back(ks[b] / stride);
          kz_lv.insert(kz_lv.end(), kz.begin() + (size_t)b * HQ, kz.begin() + (size_t)(b + 1) * HQ);
          kz_lv.resize(kz_lv.size() + (pam::kz_row(N) - HQ), 0.0);
        }
      lv.n_sel = (int)ksel.size();
      if ((st = upload(p, &lv.d_ksel, ksel.data(), ksel.size())) != PAM_OK) break;
      if ((st = upload(p, &lv.d_kz, kz_lv.data(), kz_lv.size())) != PAM_OK) break;
      if (p->ff) {
        // [n_sel][r][q1] at q = (N / 16) q1 + r; kz depends on q through min(q, N - q)
        std::vector<double> kzff((size_t)lv.n_sel * N);
        const int n2 = N / 16;
        for (int b = 0; b < lv.n_sel; ++b)
          for (int r = 0; r < n2; ++r)
            for (int q1 = 0; q1 < 16; ++q1) {
              const int q = n2 * q1 + r, qf = std::min(q, N - q);
              kzff[(size_t)b * N + r * 16 + q1] = kz_lv[(size_t)b * pam::kz_row(N) + qf];
            }
        if ((st = upload(p, &lv.d_kzff, kzff.data(), kzff.size())) != PAM_OK) break;
        std::vector<int32_t> ev(lv.n_sel, 0);
        for (int b = 0; b < lv.n_sel; ++b)
          for (int q = 0; q < N; ++q) ev[b] |= kzff[(size_t)b * N + q] < 0.0 ? 1 : 0;
        if ((st = upload(p, &lv.d_ev, ev.data(), ev.size())) != PAM_OK) break;
      }
      p->levels.push_back(lv);
    }
  } while (false);
  if (st != PAM_OK) {
    free_plan(p);
    return st;
  }
  // the K3 workgroups the device holds at once: the bin split plans its launches in rounds of these
  {
    pam::K3Args a{};
    a.N = p->N;
    const pam::K3Groups none{};
    int occ = 0, cus = 0;
    if (launch_k3(p->precision, p->n_sub, k3_tiles(p), a, none, 0, Target{nullptr, &occ}, p->coherence) !=
            hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device) != hipSuccess || occ < 1 ||
        cus < 1) {
      free_plan(p);
      return PAM_ERR_DEVICE;
    }
    // (with coherence two per CU whatever fits: the split orders the FP32 sums, and these become BF16 features)
    p->k3_slots = (p->coherence && p->precision == PAM_PREC_FP32 ? std::min(occ, 2) : occ) * cus;
    p->n_cus = cus;
  }
  *out = p;
  return PAM_OK;
}

pam_status_t pam_plan_get_info(pam_plan_t p, pam_plan_info_t* info) {
  if (!p || !info) return PAM_ERR_INVALID_ARG;
  info->n_bins = p->n_bins;
  info->n_z = p->n_z;
  info->n_x = p->N;
  info->n_sub = p->n_sub;
  info->n_elements = p->L;
  info->n_samples = p->n_t;
  info->n_pairs = p->n_sub == 3 ? 3 : (p->n_sub == 2 ? 1 : 0);
  info->device = p->device;
  return PAM_OK;
}

pam_status_t pam_plan_get_bins(pam_plan_t p, int32_t* bins, int32_t capacity) {
  if (!p || !bins || capacity < p->n_bins) return PAM_ERR_INVALID_ARG;
  std::memcpy(bins, p->bins.data(), sizeof(int32_t) * p->n_bins);
  return PAM_OK;
}

pam_status_t pam_workspace_layout(pam_plan_t p, int64_t n_frames, int32_t n_t, pam_workspace_layout_t* out) {
  if (!p || !out || n_frames < 0) return PAM_ERR_INVALID_ARG;
  return layout(p, n_frames, n_t, out);
}

pam_status_t pam_workspace_layout_in(pam_plan_t p, int64_t n_frames, int32_t n_t, size_t ws_bytes,
                                     pam_workspace_layout_t* out) {
  if (!p || !out || n_frames < 0) return PAM_ERR_INVALID_ARG;
  return layout_in(p, n_frames, n_t, ws_bytes, out);
}

pam_status_t pam_workspace_size(pam_plan_t p, int64_t n_frames, int32_t n_t, size_t* bytes) {
  if (!bytes) return PAM_ERR_INVALID_ARG;
  pam_workspace_layout_t L;
  pam_status_t st = pam_workspace_layout(p, n_frames, n_t, &L);
  if (st == PAM_OK) *bytes = L.total;
  return st;
}

}  // extern "C"

namespace {

// method 0: angular spectrum (K1, K2, K3 fields, K4); method 1: frequency-domain
// delay-and-sum (K1, K3 TEA fields, K4; no lateral transform)
// Workspace of a grouped call: the groups' layouts back to back (each 256-byte aligned).
// *one_launch: the fields stage runs as one grouped launch over all groups (factored kernels, more than one
// group with frames, and the cost estimate of that launch below the sum of the groups' own launches); cap[g]:
// group g's bins-per-workgroup cap, the shared one for a grouped launch, else the group's own.
pam_status_t grouped_layout(const pam_plan_s* p, const pam_group_t* groups, int n_groups,
                            pam_workspace_layout_t* W, size_t* base, size_t* total,
                            int* cap, bool* one_launch, bool full = true) {
  if (n_groups < 1 || n_groups > pam::kMaxGroups || !groups) return PAM_ERR_INVALID_ARG;
  int64_t F_total = 0;
  int64_t F[pam::kMaxGroups];
  int n_sel[pam::kMaxGroups];
  int live = 0;
  for (int g = 0; g < n_groups; ++g) {
    if (groups[g].n_frames < 0) return PAM_ERR_INVALID_ARG;
    const Level* lv = level_for(p, groups[g].n_t);
    if (!lv) return PAM_ERR_INVALID_ARG;
    F[g] = groups[g].n_frames;
    n_sel[g] = lv->n_sel;
    F_total += groups[g].n_frames;
    live += groups[g].n_frames > 0;
  }
  if (F_total > 65535) return PAM_ERR_UNSUPPORTED;
  double separate = 0;
  for (int g = 0; g < n_groups; ++g) {
    double c = 0;
    cap[g] = k3_bin_cap(p, &F[g], &n_sel[g], 1, &c, full);
    separate += c;
  }
  // each further launch: about three bin-times (15 us) between its start and its drain (157 drawn group lists: with one,
  // the choice is 3.5 % from the faster of the two schedules on average, with three 2.7 %)
  separate += 3 * std::max(0, live - 1);
  *one_launch = false;
  if (p->ff && live > 1) {
    double together = 0;
    const int shared = k3_bin_cap(p, F, n_sel, n_groups, &together, full);
    if (together < separate) {
      *one_launch = true;
      for (int g = 0; g < n_groups; ++g) cap[g] = shared;
    }
  }
  size_t o = 0;
  for (int g = 0; g < n_groups; ++g) {
    const pam_status_t st = layout(p, groups[g].n_frames, groups[g].n_t, &W[g], cap[g], full);
    if (st != PAM_OK) return st;
    base[g] = o;
    o = align256(o + W[g].total);
  }
  *total = std::max<size_t>(o, 256);
  return PAM_OK;
}

// One call over groups of frames, each group one record length, frames packed group after
// group in rf and in the outputs.  K1, K2 and K4 run per group; K3 runs as one grouped
// work list on the factored kernels (else per group).  events: stage marks (one group only).
pam_status_t run_groups(pam_plan_t p, const float* rf, const pam_group_t* groups, int n_groups, float* image,
                        float* nncc, float* rho_pairs, void* workspace, size_t ws_bytes, void* hip_stream,
                        void* const* events, int method) {
  if (!p) return PAM_ERR_INVALID_ARG;
  // per group, fixed arrays of at most kMaxGroups entries: the call allocates no host memory either
  pam_workspace_layout_t W[pam::kMaxGroups];
  size_t wbase[pam::kMaxGroups];
  size_t total = 0;
  int cap[pam::kMaxGroups];
  bool one_launch = false;
  pam_status_t st = grouped_layout(p, groups, n_groups, W, wbase, &total, cap, &one_launch);
  if (st == PAM_OK && workspace && ws_bytes < total)        // the smaller reservation (one group: as layout_in)
    st = grouped_layout(p, groups, n_groups, W, wbase, &total, cap, &one_launch, false);
  if (st != PAM_OK) return st;
  if (events && n_groups != 1) return PAM_ERR_INVALID_ARG;
  int64_t F_total = 0;
  for (int g = 0; g < n_groups; ++g) F_total += groups[g].n_frames;
  if (F_total == 0) return PAM_OK;
  if (!rf || !image) return PAM_ERR_INVALID_ARG;
  if (!workspace || ws_bytes < total || (reinterpret_cast<uintptr_t>(workspace) & 255u)) return PAM_ERR_WORKSPACE;
  if (rho_pairs && p->n_sub == 1) return PAM_ERR_INVALID_ARG;
  DeviceGuard guard(p->device);
  if (!guard.ok) return PAM_ERR_DEVICE;
  hipStream_t stream = static_cast<hipStream_t>(hip_stream);
  auto mark = [&](int i) -> bool {
    return !events || hipEventRecord(static_cast<hipEvent_t>(events[i]), stream) == hipSuccess;
  };
  if (!mark(0)) return PAM_ERR_DEVICE;
  const int pix = p->n_z * p->N;
  const int n_pairs = p->n_sub == 3 ? 3 : (p->n_sub == 2 ? 1 : 0);

  // per group: its record length level, frames, workspace and output pointers
  struct G {
    const Level* lv;
    int F, n_t;
    const float* rf;
    float *image, *nncc, *rho;
    float2 *spectra, *coeffs;
    float *scales, *accum, *energy, *weight, *blockmax;
    LaunchShape s;
  };
  G gs[pam::kMaxGroups] = {};
  {
    size_t rf_off = 0, out_off = 0;
    for (int g = 0; g < n_groups; ++g) {
      G& q = gs[g];
      q.lv = level_for(p, groups[g].n_t);
      q.F = (int)groups[g].n_frames;
      q.n_t = groups[g].n_t;
      q.rf = rf + rf_off;
      q.image = image + out_off * pix;
      q.nncc = nncc ? nncc + out_off * pix : nullptr;
      q.rho = rho_pairs ? rho_pairs + out_off * n_pairs * pix : nullptr;
      char* ws = static_cast<char*>(workspace) + wbase[g];
      q.spectra = reinterpret_cast<float2*>(ws + W[g].spectra);
      q.coeffs = reinterpret_cast<float2*>(ws + W[g].coeffs);
      q.scales = reinterpret_cast<float*>(ws + W[g].scales);
      q.accum = reinterpret_cast<float*>(ws + W[g].accum);
      q.energy = reinterpret_cast<float*>(ws + W[g].energy);
      q.weight = reinterpret_cast<float*>(ws + W[g].weight);
      q.blockmax = reinterpret_cast<float*>(ws + W[g].blockmax);
      q.s = k3_shape(p, q.lv->n_sel, cap[g]);
      rf_off += (size_t)q.F * p->L * q.n_t;
      out_off += (size_t)q.F;
    }
  }

  // The stages of one group.
  // K1: time FFT, one workgroup per (channel, frame)
  auto stage_k1 = [&](const G& q) -> pam_status_t {
    if (q.F == 0) return PAM_OK;
    pam::K1Args a{q.rf, q.spectra, p->d_tw, q.lv->d_ksel, p->L, q.n_t, ilog2(q.n_t / 2), q.lv->stride, q.lv->n_sel,
                  q.F};
    // two channels per workgroup where they divide L (up to 4096 samples), else one
    const int ch = (p->L % 2 == 0 && q.n_t <= 4096) ? 2 : 1;
    const size_t lds = (size_t)ch * (q.n_t / 2 + q.n_t / 16) * sizeof(float2);   // ch k1_lds_points
    const long long items = (long long)p->L / ch * q.F;
    auto k1 = [&](auto kernel) -> bool {
      // n_t = 16384 takes more than 64 KiB of LDS: the kernel needs the attribute
      if (lds > 65536 && hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess)
        return false;
      // From 2048 samples one workgroup per channel group (the groups of a frame are resident together, so
      // their partial bin lines meet in L2: 0.047 vs 0.050 ms for 64 x 128 channels of 4096 samples); shorter
      // records persistent, as many workgroups as the device holds, each walking its groups with the next
      // group's samples prefetched (0.011 vs 0.012 ms for 64 x 64 channels of 1024 samples).
      int occ = 0;
      if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, reinterpret_cast<const void*>(kernel), 256 * ch, lds) !=
              hipSuccess ||
          occ < 1)
        return false;
      const unsigned blocks =
          (unsigned)(q.n_t >= 2048 ? items : std::min<long long>(items, (long long)occ * p->n_cus));
      hipLaunchKernelGGL(kernel, dim3(blocks), dim3(256 * ch), lds, stream, a);
      return true;
    };
    bool ok = false;
    switch (ilog2(q.n_t / 2) * 8 + ch) {   // n_t = 32 .. 16384
      case 4 * 8 + 1: ok = k1(pam::k1_time_fft<4>); break;
      case 5 * 8 + 1: ok = k1(pam::k1_time_fft<5>); break;
      case 6 * 8 + 1: ok = k1(pam::k1_time_fft<6>); break;
      case 7 * 8 + 1: ok = k1(pam::k1_time_fft<7>); break;
      case 8 * 8 + 1: ok = k1(pam::k1_time_fft<8>); break;
      case 9 * 8 + 1: ok = k1(pam::k1_time_fft<9>); break;
      case 10 * 8 + 1: ok = k1(pam::k1_time_fft<10>); break;
      case 11 * 8 + 1: ok = k1(pam::k1_time_fft<11>); break;
      case 12 * 8 + 1: ok = k1(pam::k1_time_fft<12>); break;
      case 13 * 8 + 1: ok = k1(pam::k1_time_fft<13>); break;
      case 4 * 8 + 2: ok = k1(pam::k1_time_fft<4, 2>); break;
      case 5 * 8 + 2: ok = k1(pam::k1_time_fft<5, 2>); break;
      case 6 * 8 + 2: ok = k1(pam::k1_time_fft<6, 2>); break;
      case 7 * 8 + 2: ok = k1(pam::k1_time_fft<7, 2>); break;
      case 8 * 8 + 2: ok = k1(pam::k1_time_fft<8, 2>); break;
      case 9 * 8 + 2: ok = k1(pam::k1_time_fft<9, 2>); break;
      case 10 * 8 + 2: ok = k1(pam::k1_time_fft<10, 2>); break;
      case 11 * 8 + 2: ok = k1(pam::k1_time_fft<11, 2>); break;
      default: return PAM_ERR_UNSUPPORTED;
    }
    if (!ok) return PAM_ERR_DEVICE;
    if (hipGetLastError() != hipSuccess) return PAM_ERR_DEVICE;
    return PAM_OK;
  };
  // K2: apodization + lateral transform, per (frame, bin)
  auto stage_k2 = [&](const G& q) -> pam_status_t {
    if (method != 0 || q.F == 0) return PAM_OK;
    const long long items = (long long)q.F * q.lv->n_sel;
    if (items > 0x7fffffffLL) return PAM_ERR_UNSUPPORTED;
    pam::K2Args a{q.spectra, q.coeffs, q.scales, p->d_twx, p->d_masks, p->L, p->N, p->n_sub, q.lv->n_sel,
                  p->col0, p->col_step, p->ff ? pam::kFfN1 : 0, is_fp16(p->precision) ? 1 : 0, (int32_t)items};
    if (p->ff) {
      // factored order: the lateral FFT, one wave per (frame, bin)
      const dim3 grid((unsigned)((items + 3) / 4));
      const bool known = p->n_sub == 3 ? launch_k2<3>(p->N, grid, stream, a)
                                       : (p->n_sub == 2 ? launch_k2<2>(p->N, grid, stream, a) : launch_k2<1>(p->N, grid, stream, a));
      if (!known) return PAM_ERR_UNSUPPORTED;
    } else {
      const size_t lds = (size_t)(p->N + 3 * p->L + 2 * p->n_sub * p->N) * sizeof(float2);
      if (p->n_sub == 3)
        hipLaunchKernelGGL(pam::k2_lateral<3>, dim3(q.lv->n_sel, q.F), dim3(256), lds, stream, a);
      else if (p->n_sub == 2)
        hipLaunchKernelGGL(pam::k2_lateral<2>, dim3(q.lv->n_sel, q.F), dim3(256), lds, stream, a);
      else
        hipLaunchKernelGGL(pam::k2_lateral<1>, dim3(q.lv->n_sel, q.F), dim3(256), lds, stream, a);
    }
    if (hipGetLastError() != hipSuccess) return PAM_ERR_DEVICE;
    return PAM_OK;
  };
  auto args_for = [&](const G& q) {
    return pam::K3Args{q.coeffs, q.scales, q.lv->d_kz, p->d_z, p->d_bhi, p->d_blo, q.accum,
                       p->N, p->n_z, q.lv->n_sel, q.F, q.s.n_dt, q.s.n_xg, q.s.n_split, q.s.bins_per_split,
                       p->zero_evanescent, q.lv->d_kzff, p->d_ff_w16, p->d_ff_tw, q.lv->d_ev,
                       p->d_ff_tw2, p->d_ff_tw_vec, p->d_ff_tw2_vec};
  };
  // K3: the fields and cross-spectra sums of one group (frequency-domain delay-and-sum for method 1,
  // else propagate / inverse lateral transform / cross-spectra)
  auto stage_k3 = [&](const G& q) -> pam_status_t {
    if (q.F == 0) return PAM_OK;
    if (method == 1) {
      pam::TeaArgs a{};
      a.spectra = q.spectra;
      a.ksel = q.lv->d_ksel;
      a.units = p->d_units;
      a.z = p->d_z;
      a.accum = q.accum;
      a.dx = p->dx;
      a.cyc = p->fs / ((double)q.n_t * p->c);
      a.L = p->L;
      a.N = p->N;
      a.n_z = p->n_z;
      a.n_sel = q.lv->n_sel;
      a.F = q.F;
      a.n_split = q.s.n_split;
      a.bins_per_split = q.s.bins_per_split;
      a.n_acc = n_acc(p->n_sub, p->coherence);
      a.col0 = p->col0;
      a.step = p->col_step;
      pam::tea_shape(a);
      const bool few = pam::tea_few(a);
      if (few) a.n_wg = (pix + 64 * pam::TEA_WAVES - 1) / (64 * pam::TEA_WAVES);
      const long long blocks = (long long)q.F * a.n_wg * q.s.n_split;
      if (blocks > 0x7fffffffLL) return PAM_ERR_UNSUPPORTED;
      const size_t lds = few ? 0 : pam::tea_lds(a);
      const dim3 grid((unsigned)blocks), block(64 * pam::TEA_WAVES);
      auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, lds, stream, a); };
      switch (few ? -p->n_sub : 2 * p->n_sub + p->mixed_units) {
        case -3: launch(pam::k3_tea_few<3>); break;
        case -2: launch(pam::k3_tea_few<2>); break;
        case -1: launch(pam::k3_tea_few<1>); break;
        case 7: launch(pam::k3_tea<3, true>); break;
        case 6: launch(pam::k3_tea<3, false>); break;
        case 5: launch(pam::k3_tea<2, true>); break;
        case 4: launch(pam::k3_tea<2, false>); break;
        case 3: launch(pam::k3_tea<1, true>); break;
        default: launch(pam::k3_tea<1, false>); break;
      }
      if (hipGetLastError() != hipSuccess) return PAM_ERR_DEVICE;
      return PAM_OK;
    }
    const pam::K3Groups none{};
    const long long blocks = (long long)q.F * q.s.n_dt * q.s.n_xg * q.s.n_split;
    if (blocks > 0x7fffffffLL) return PAM_ERR_UNSUPPORTED;
    if (launch_k3(p->precision, p->n_sub, q.s, args_for(q), none, (int)blocks, Target{stream, nullptr, p->n_cus}, p->coherence) !=
        hipSuccess)
      return PAM_ERR_DEVICE;
    return PAM_OK;
  };
  // K4: NCC / weight / energy, then NNCC and image
  auto stage_k4 = [&](int g) -> pam_status_t {
    const G& q = gs[g];
    if (q.F == 0) return PAM_OK;
    const int n_blk = (pix + 255) / 256;
    pam::K4Args a{q.accum, q.energy, q.weight, q.blockmax, q.rho, q.image, q.nncc, pix, q.F, W[g].n_split,
                  p->n_sub, n_blk, W[g].n_acc, p->eps};
    auto weight = [&](auto sg) {
      constexpr int SG = decltype(sg)::value;
      const dim3 grid(n_blk, q.F), block(256 * SG);
      if (p->n_sub == 3) hipLaunchKernelGGL((pam::k4_weight<3, SG>), grid, block, 0, stream, a);
      else if (p->n_sub == 2) hipLaunchKernelGGL((pam::k4_weight<2, SG>), grid, block, 0, stream, a);
      else hipLaunchKernelGGL((pam::k4_weight<1, SG>), grid, block, 0, stream, a);
    };
    // Four threads a pixel where a pixel has many splits to add and the pixels alone leave CUs with little to do: up to 256
    // workgroups of 256 pixels (512 with one sub-aperture) and from 16 splits.  This stage, with three sub-apertures: 76
    // workgroups of 52 splits 14.0 us with one thread a pixel and 12.0 with four, 152 of 32 12.2 / 11.7, 256 of 16 11.0 /
    // 11.2, 512 of 16 14.2 / 14.6, 1,216 of 4 12.2 / 14.4; with one sub-aperture 512 of 23 10.2 / 9.8, 2,432 of 4 11.2 / 16.7.
    if (W[g].n_split >= 16 && (long long)n_blk * q.F <= (p->n_sub == 1 ? 512 : 256)) weight(std::integral_constant<int, 4>());
    else weight(std::integral_constant<int, 1>());
    if (hipGetLastError() != hipSuccess) return PAM_ERR_DEVICE;
    hipLaunchKernelGGL(pam::k4_image, dim3(n_blk, q.F), dim3(256), 0, stream, a);
    if (hipGetLastError() != hipSuccess) return PAM_ERR_DEVICE;
    return PAM_OK;
  };

  if (!one_launch && n_groups > 1) {
    // group after group, each through all four stages: a group's fields launch reads the coefficients its
    // K2 has just written while they are still in the last-level cache (one group's worth; the stage-major
    // order made the fields launches of 4 + 4 + 4 frames of 256 elements 7-24 % slower)
    for (int g = 0; g < n_groups; ++g) {
      if ((st = stage_k1(gs[g])) != PAM_OK || (st = stage_k2(gs[g])) != PAM_OK ||
          (st = stage_k3(gs[g])) != PAM_OK || (st = stage_k4(g)) != PAM_OK)
        return st;
    }
    return PAM_OK;
  }
  // stage after stage (one group, with the stage marks, or one grouped fields launch)
  for (int g = 0; g < n_groups; ++g)
    if ((st = stage_k1(gs[g])) != PAM_OK) return st;
  if (!mark(1)) return PAM_ERR_DEVICE;
  for (int g = 0; g < n_groups; ++g)
    if ((st = stage_k2(gs[g])) != PAM_OK) return st;
  if (!mark(2)) return PAM_ERR_DEVICE;
  if (method == 0 && one_launch) {
    // one launch over every group: a grouped work list on the factored kernels
    pam::K3Groups grp{};
    long long blocks = 0;
    const G* first = nullptr;
    // the work list runs the groups with the longest workgroups first (a short tail)
    const G* order[pam::kMaxGroups];
    int n_order = 0;
    for (int g = 0; g < n_groups; ++g)
      if (gs[g].F > 0) order[n_order++] = &gs[g];
    for (int k = 1; k < n_order; ++k)      // stable insertion sort, longest workgroups first (no buffer)
      for (int m = k; m > 0 && order[m - 1]->s.bins_per_split < order[m]->s.bins_per_split; --m)
        std::swap(order[m - 1], order[m]);
    for (int k = 0; k < n_order; ++k) {
      const G* qp = order[k];
      const G& q = *qp;
      if (!first) first = &q;
      pam::K3Group& e = grp.g[grp.n++];
      e = pam::K3Group{q.coeffs, q.scales, q.lv->d_kzff, q.lv->d_ev, q.accum, (int32_t)blocks, q.F, q.lv->n_sel,
                       q.s.n_split, q.s.bins_per_split};
      blocks += (long long)q.F * q.s.n_dt * q.s.n_xg * q.s.n_split;
    }
    if (blocks > 0x7fffffffLL) return PAM_ERR_UNSUPPORTED;
    if (launch_k3(p->precision, p->n_sub, first->s, args_for(*first), grp, (int)blocks, Target{stream, nullptr, p->n_cus}, p->coherence) !=
        hipSuccess)
      return PAM_ERR_DEVICE;
  } else {
    for (int g = 0; g < n_groups; ++g)
      if ((st = stage_k3(gs[g])) != PAM_OK) return st;
  }
  if (!mark(3)) return PAM_ERR_DEVICE;
  for (int g = 0; g < n_groups; ++g)
    if ((st = stage_k4(g)) != PAM_OK) return st;
  if (!mark(4)) return PAM_ERR_DEVICE;
  return PAM_OK;
}

pam_status_t run_as_tax(pam_plan_t p, const float* rf, int64_t n_frames, int32_t n_t, float* image,
                        float* nncc, float* rho_pairs, void* workspace, size_t ws_bytes, void* hip_stream,
                        void* const* events, int method = 0) {
  if (!p || n_frames < 0) return PAM_ERR_INVALID_ARG;
  if (n_frames > 65535) return PAM_ERR_UNSUPPORTED;
  const pam_group_t one{n_t, n_frames};
  return run_groups(p, rf, &one, 1, image, nncc, rho_pairs, workspace, ws_bytes, hip_stream, events, method);
}

}  // namespace

extern "C" {

pam_status_t pam_as_tax(pam_plan_t p, const float* rf, int64_t n_frames, int32_t n_t, float* image,
                        float* nncc, float* rho_pairs, void* workspace, size_t ws_bytes, void* hip_stream) {
  return run_as_tax(p, rf, n_frames, n_t, image, nncc, rho_pairs, workspace, ws_bytes, hip_stream, nullptr);
}

pam_status_t pam_as_tax_events(pam_plan_t p, const float* rf, int64_t n_frames, int32_t n_t, float* image,
                               float* nncc, float* rho_pairs, void* workspace, size_t ws_bytes,
                               void* hip_stream, void* const* events) {
  if (!events) return PAM_ERR_INVALID_ARG;
  for (int i = 0; i < PAM_N_STAGE_EVENTS; ++i)
    if (!events[i]) return PAM_ERR_INVALID_ARG;
  return run_as_tax(p, rf, n_frames, n_t, image, nncc, rho_pairs, workspace, ws_bytes, hip_stream, events);
}

pam_status_t pam_fd_tea_tax(pam_plan_t p, const float* rf, int64_t n_frames, int32_t n_t, float* image,
                            float* nncc, float* rho_pairs, void* workspace, size_t ws_bytes, void* hip_stream) {
  return run_as_tax(p, rf, n_frames, n_t, image, nncc, rho_pairs, workspace, ws_bytes, hip_stream, nullptr, 1);
}

void pam_destroy(pam_plan_t p) { free_plan(p); }

pam_status_t pam_workspace_size_grouped(pam_plan_t p, const pam_group_t* groups, int32_t n_groups, size_t* bytes) {
  if (!p || !bytes) return PAM_ERR_INVALID_ARG;
  pam_workspace_layout_t W[pam::kMaxGroups];
  size_t base[pam::kMaxGroups];
  int cap[pam::kMaxGroups];
  bool one_launch = false;
  return grouped_layout(p, groups, n_groups, W, base, bytes, cap, &one_launch);
}

pam_status_t pam_as_tax_grouped(pam_plan_t p, const float* rf, const pam_group_t* groups, int32_t n_groups,
                                float* image, float* nncc, float* rho_pairs, void* workspace, size_t ws_bytes,
                                void* hip_stream) {
  return run_groups(p, rf, groups, n_groups, image, nncc, rho_pairs, workspace, ws_bytes, hip_stream, nullptr, 0);
}

void pam_debug_fail_allocation(int32_t n) { g_fail_alloc.store(n < 0 ? -1 : n); }

int64_t pam_debug_live_allocations(void) { return g_live_allocs.load(); }

int32_t pam_debug_grouped_one_launch(pam_plan_t p, const pam_group_t* groups, int32_t n_groups) {
  if (!p) return PAM_ERR_INVALID_ARG;
  pam_workspace_layout_t W[pam::kMaxGroups];
  size_t base[pam::kMaxGroups];
  size_t total = 0;
  int cap[pam::kMaxGroups];
  bool one_launch = false;
  const pam_status_t st = grouped_layout(p, groups, n_groups, W, base, &total, cap, &one_launch);
  return st != PAM_OK ? (int32_t)st : (one_launch ? 1 : 0);
}

}  // extern "C"

// ---------------------------------------------------------------------------
// Entry point that allocates nothing: the workspace is a file-scope device array.
// In host code `scratch` names a host-side stand-in, not device memory; its device
// address on each GPU comes from hipGetSymbolAddress (taken once per device, with
// that device current) and only that address is ever handed to kernels.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[PAM_NOALLOC_SCRATCH_BYTES];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on `device` (the caller has made it current).
pam_status_t scratch_address(int device, void** out) {
  if (device < 0 || device >= kMaxDevices) return PAM_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[device]) {
    void* ptr = nullptr;
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return PAM_ERR_DEVICE;
    g_scratch_ptr[device] = ptr;
  }
  *out = g_scratch_ptr[device];
  return PAM_OK;
}

}  // namespace

extern "C" {

pam_status_t pam_as_tax_noalloc(pam_plan_t p, const float* rf, int64_t n_frames, int32_t n_t, float* image,
                                float* nncc, float* rho_pairs, void* hip_stream) {
  if (!p || n_frames < 0) return PAM_ERR_INVALID_ARG;
  pam_workspace_layout_t W;
  pam_status_t st = layout_in(p, n_frames, n_t, (size_t)PAM_NOALLOC_SCRATCH_BYTES, &W);
  if (st != PAM_OK) return st;
  if (n_frames == 0) return PAM_OK;
  void* ws = nullptr;
  {
    DeviceGuard guard(p->device);
    if (!guard.ok) return PAM_ERR_DEVICE;
    if ((st = scratch_address(p->device, &ws)) != PAM_OK) return st;
  }
  return run_as_tax(p, rf, n_frames, n_t, image, nncc, rho_pairs, ws, (size_t)PAM_NOALLOC_SCRATCH_BYTES,
                    hip_stream, nullptr);
}

}  // extern "C"
