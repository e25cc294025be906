// Internal to libscf: the plan object, error reporting, workspace layouts
// and the launch helpers shared by the translation units of the C ABI
// (scf_api.cpp: plans, the step, batched and adjoint paths; scf_cadence.cpp:
// the refresh cadence, the density and the frame).
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdint>
#include <cstring>
#include <string>
#include <vector>

#include "../../include/scf.h"
#include "host_field.h"
#include "scf_internal.h"


using namespace scf;

namespace scf {
namespace api_detail {
// message of the last failed call on this thread (scf_last_error)
inline thread_local std::string g_last_error;
}  // namespace api_detail
}  // namespace scf

namespace {


scf_status fail(scf_status st, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  scf::api_detail::g_last_error = buf;
  return st;
}

#define HIP_TRY(expr)                                                                     \
  do {                                                                                    \
    hipError_t e_ = (expr);                                                               \
    if (e_ != hipSuccess)                                                                 \
      return fail(SCF_ERR_HIP, "%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_),     \
                  __FILE__, __LINE__);                                                    \
  } while (0)

size_t align256(size_t v) { return (v + 255) & ~size_t(255); }

// ---------------------------------------------------------------------------
// basis tables (double precision, host)
// ---------------------------------------------------------------------------
// Monic Gegenbauer recurrence p_n = xi p_{n-1} - beta_n p_{n-2}:
// from n C_n = 2(n+lambda-1) xi C_{n-1} - (n+2 lambda-2) C_{n-2} and the
// leading coefficient k_n = 2^n (lambda)_n / n!.
double gegen_beta(int n, double lam) {
  if (n < 2) return 0.0;
  return (n + 2.0 * lam - 2.0) * (n - 1.0) / (4.0 * (n + lam - 1.0) * (n + lam - 2.0));
}
double gegen_lead(int n, double lam) {
  return std::exp(n * std::log(2.0) + std::lgamma(lam + n) - std::lgamma(lam) - std::lgamma(n + 1.0));
}
// Monic-scaled associated Legendre recurrence Qt_l = c Qt_{l-1} - gamma Qt_{l-2}
double legendre_gamma(int l, int m) {
  if (l < m + 2) return 0.0;
  return (l + m - 1.0) * (l - m - 1.0) / ((2.0 * l - 1.0) * (2.0 * l - 3.0));
}
// rho_lm = d^m P_l / dx^m  /  Qt_l^m
double legendre_rho(int l, int m) {
  double r = 1.0;
  for (int k = 2 * m - 1; k > 1; k -= 2) r *= k;  // (2m-1)!!
  for (int ll = m + 1; ll <= l; ++ll) r *= (2.0 * ll - 1.0) / (ll - m);
  return r;
}
double ylm_norm(int l, int m) {
  double lg = std::lgamma(l - m + 1.0) - std::lgamma(l + m + 1.0);
  return std::sqrt((2.0 * l + 1.0) / (4.0 * M_PI) * std::exp(lg));
}

// f_nl(s) = -s^l q^(-alpha(2l+1)) C_n^(lambda)(xi) and its s-derivative,
// evaluated with the monic recurrence and its derivative.
void radial_f(double alpha, int l, int n, double s, double& f, double& df) {
  const double lam = (2.0 * l + 1.0) * alpha + 0.5;
  const double t = std::pow(s, 1.0 / alpha);
  const double q = 1.0 + t;
  const double xi = 1.0 - 2.0 / q;
  const double dt = (1.0 / alpha) * std::pow(s, 1.0 / alpha - 1.0);  // dt/ds
  const double dxi = 2.0 * dt / (q * q);
  double p0 = 1.0, p1 = xi, d0 = 0.0, d1 = 1.0, p = 1.0, dp = 0.0;
  if (n == 0) {
    p = 1.0;
    dp = 0.0;
  } else if (n == 1) {
    p = xi;
    dp = 1.0;
  } else {
    for (int k = 2; k <= n; ++k) {
      double b = gegen_beta(k, lam);
      double p2 = xi * p1 - b * p0;
      double d2 = p1 + xi * d1 - b * d0;
      p0 = p1;
      p1 = p2;
      d0 = d1;
      d1 = d2;
    }
    p = p1;
    dp = d1;
  }
  const double kn = gegen_lead(n, lam);
  const double pre = std::pow(s, double(l)) * std::pow(q, -alpha * (2.0 * l + 1.0));
  // d pre / ds = pre * (l/s - alpha(2l+1) dt / q)
  const double dpre = (l > 0 ? l * std::pow(s, l - 1.0) * std::pow(q, -alpha * (2.0 * l + 1.0)) : 0.0) -
                      pre * alpha * (2.0 * l + 1.0) * dt / q;
  f = -kn * pre * p;
  df = -kn * (dpre * p + pre * dp * dxi);
}

// Energy-norm normalisation N_nl = (b / 4 pi G) int_0^inf [s^2 f'^2 + l(l+1) f^2] ds.
// alpha = 1: closed form (Hernquist & Ostriker 1992).  Otherwise composite
// 16-point Gauss-Legendre quadrature in v = ln s over [-60, 60].
double norm_nl(double alpha, double b, double G, int n, int l) {
  if (alpha == 1.0) {
    const double K = 0.5 * n * (n + 4.0 * l + 3.0) + (l + 1.0) * (2.0 * l + 1.0);
    const double lg = std::lgamma(n + 4.0 * l + 3.0) - std::lgamma(n + 1.0) - 2.0 * std::lgamma(2.0 * l + 1.5);
    return b / G * K * std::exp(lg - (8.0 * l + 6.0) * std::log(2.0)) / (n + 2.0 * l + 1.5);
  }
  static double xs[16], ws[16];
  static bool init = false;
  if (!init) {
    for (int i = 0; i < 16; ++i) {  // Newton iteration on P_16
      double x = std::cos(M_PI * (i + 0.75) / 16.5);
      for (int it = 0; it < 100; ++it) {
        double p0 = 1.0, p1 = x;
        for (int k = 2; k <= 16; ++k) {
          double p2 = ((2.0 * k - 1.0) * x * p1 - (k - 1.0) * p0) / k;
          p0 = p1;
          p1 = p2;
        }
        double dp = 16.0 * (x * p1 - p0) / (x * x - 1.0);
        double dx = p1 / dp;
        x -= dx;
        if (std::fabs(dx) < 1e-16) break;
      }
      double p0 = 1.0, p1 = x;
      for (int k = 2; k <= 16; ++k) {
        double p2 = ((2.0 * k - 1.0) * x * p1 - (k - 1.0) * p0) / k;
        p0 = p1;
        p1 = p2;
      }
      double dp = 16.0 * (x * p1 - p0) / (x * x - 1.0);
      xs[i] = x;
      ws[i] = 2.0 / ((1.0 - x * x) * dp * dp);
    }
    init = true;
  }
  const int panels = 960;
  const double v0 = -60.0, v1 = 60.0, hw = (v1 - v0) / panels;
  double acc = 0.0;
  for (int pnl = 0; pnl < panels; ++pnl) {
    const double c = v0 + (pnl + 0.5) * hw;
    for (int i = 0; i < 16; ++i) {
      const double v = c + 0.5 * hw * xs[i];
      const double s = std::exp(v);
      double f, df;
      radial_f(alpha, l, n, s, f, df);
      double val = (s * s * df * df + l * (l + 1.0) * f * f) * s;
      if (std::isfinite(val)) acc += 0.5 * hw * ws[i] * val;
    }
  }
  return b / (4.0 * M_PI * G) * acc;
}

}  // namespace

struct scf_plan {
  scf_basis basis;
  int dtype;
  int device;
  int nmax, lmax, nmaxc;
  int64_t T;
  int amode;
  Engine* eng;
  int coef_variant = 0;
  int coef_div = 1;  // wave-units of the coefficient pass: one resident round / coef_div
  int field_variant = 0;
  int num_cu = 256;
  int resident[8] = {1, 1, 1, 1, 1, 1, 1, 1};  // resident wave-units per CU per variant
  int gamma_resident = 1;                        // same for the adjoint's gamma pass
  size_t rs;  // sizeof real
  void* d_beta_rad = nullptr;
  void* d_beta_ang = nullptr;
  double* d_cs = nullptr;
  double* d_fw = nullptr;
  double* d_kden = nullptr;  // density constants -K_nl / (4 pi G b^2), [l][n]
  double* d_dtab = nullptr;  // radial derivative table of the matrix-core field pass, [l][2][n]
  void* d_beta_img = nullptr;  // recurrence of the operand-image pass, [l][nmaxc + 2]
  double* d_rtab = nullptr;    // radial-weight factors (WeightTables)
  std::vector<double> h_cs, h_fw;
  // kernel timing
  bool prof = false;
  std::vector<hipEvent_t> ev_pool;
  size_t ev_next = 0;
  struct Rec {
    int kind;
    hipEvent_t a, b;
  };
  std::vector<Rec> recs;
  // batched mode: the captured per-step graph, the stream it is captured on,
  // and pinned host staging for the work list and the centre table
  hipStream_t cap_stream = nullptr;
  hipGraph_t graph = nullptr;
  hipGraphExec_t gexec = nullptr;
  hipGraph_t graph_g = nullptr;    // kGraphSteps middle steps in one graph
  hipGraphExec_t gexec_g = nullptr;
  std::vector<char> gkey;
  int graph_captures = 0;
  char* h_stage = nullptr;
  size_t h_stage_cap = 0;
  hipEvent_t ev_staging = nullptr;
  bool staging_pending = false;
  // the stream of the last batched call, and its end (batch_wait)
  hipStream_t batch_stream = nullptr;
  hipEvent_t ev_batch = nullptr;
  bool batch_pending = false;
};

namespace {

enum Kind { K_COEF = 0, K_REDUCE, K_FINALIZE, K_FIELD, K_STEP_FIELD, K_KICK, K_MAKE_W, K_FILL,
            K_BATCH_COEF, K_BATCH_FIELD, K_ADJ, K_SELECT, K_OTHER };
const char* kKindNames[SCF_KERNEL_KINDS] = {"coef", "reduce", "finalize", "field", "field_step",
                                            "kick_drift", "make_w", "fill", "batched_coef",
                                            "batched_step", "adjoint", "select", "other"};

// brackets one launch with events when the plan's timing is on
struct Timed {
  scf_plan* p;
  hipStream_t s;
  int kind;
  hipEvent_t b = nullptr;
  Timed(scf_plan* p_, hipStream_t s_, int k) : p(p_), s(s_), kind(k) {
    if (p && p->prof && p->ev_next + 2 <= p->ev_pool.size() &&
        !(p->cap_stream && s == p->cap_stream)) {
      hipEvent_t a = p->ev_pool[p->ev_next++];
      b = p->ev_pool[p->ev_next++];
      (void)hipEventRecord(a, s);
      p->recs.push_back({kind, a, b});
    }
  }
  ~Timed() {
    if (b) (void)hipEventRecord(b, s);
  }
};

// Coefficient launch geometry: one resident round of wave-units (the
// occupancy of the variant times the CU count), each taking an even share of
// the P-particle stages; returns the unit count and sets *stages.
int coef_units_v(const scf_plan* p, int64_t n, int v, int64_t* stages, int div = 1) {
  if (n <= 0) {
    *stages = 0;
    return 0;
  }
  const int P = p->eng->stage_particles(v);
  *stages = (n + P - 1) / P;
  const int64_t cap = (int64_t)p->resident[v] * p->num_cu / std::max(div, 1);
  return (int)std::min<int64_t>(*stages, std::max<int64_t>(cap, 1));
}

// the plan's variant, and its unit count (fewer, longer units suit small n:
// the per-unit set-up and partial row are amortised over more stages)
int coef_units(const scf_plan* p, int64_t n, int64_t* stages) {
  return coef_units_v(p, n, p->coef_variant, stages, p->coef_div);
}

// rows per unit of variant v when no unit sums more than max_stages stages:
// one when each folds once (its compensation row would stay zero)
int unit_rows(const scf_plan* p, int v, int64_t max_stages) {
  const int f = p->eng->fold_stages(v);
  return (f > 0 && max_stages <= f) ? 1 : p->eng->rows_per_unit(v);
}

// largest partial-row count over the coefficient variants (workspace sizing)
int coef_blocks_max(const scf_plan* p, int64_t n) {
  int nb = 0;
  for (int v = 0; v < p->eng->coef_variants(); ++v) {
    int64_t st;
    nb = std::max(nb, coef_units_v(p, n, v, &st) * p->eng->rows_per_unit(v));
  }
  return nb;
}

constexpr int kReduceChunks = 32;

// elements of one coefficient vector's field weights
size_t fw_elems(const scf_plan* p) {
  return (size_t)FwLayout::elems(p->nmaxc, p->lmax, p->rs == 4);
}
// Whether the matrix-core variants read the operand image in a run of one
// cluster of n particles, or of several of n on average.  The line is one of
// reproducibility, not of speed or accuracy: the image kernel is the faster one
// and no less exact at every n (us per step-mode launch at 10, 40 and 160 T
// points, image / the best of the others: nmax 6, lmax 4 3.8/4.9, 3.9/4.9,
// 4.1/5.1; nmax 10, lmax 6 5.6/6.5, 5.7/6.7, 7.9/9.5; nmax 16, lmax 10
// 11.6/12.3, 16.4/20.2, 40.6/48.7; force error against 64 bits 0.83e-7 and
// 0.91e-7 rms at 10 T of the first, 0.80e-7 and 1.00e-7 at 160 T of the last).
// But it sums in another order, and a run carries that into its coefficients:
// after ten steps of 0.01 they differ by about 1e-8 sqrt(T / n) (measured 4 to
// 14e-10 at n = 130 T over five basis sizes, Plummer and Hernquist).  From 160 T
// on that stays below 1e-9; runs of fewer particles keep their former kernels.
// A batch goes by its mean size, since a launch runs one kernel: with both in
// one, chosen per cluster, ten clusters of 1.2e6 particles, 18% of them in
// clusters below the line, took 589 us instead of 541 (585 with the vector kernel
// for all).  So a small cluster beside large ones is evaluated from the image.
// Single evaluations (scf_forces, the density) carry nothing on and use the
// image at every n.
constexpr int64_t kImageRatio = 160;
bool use_image(const scf_plan* p, int64_t n) { return n >= kImageRatio * p->T; }
// ... and the plan's field variant is one that reads it (the Hessian-vector pass
// goes by use_image alone)
bool image_variant(const scf_plan* p) {
  return p->rs == 4 && (p->field_variant == 2 || p->field_variant == 3);
}
bool field_image(const scf_plan* p, int64_t n) { return image_variant(p) && use_image(p, n); }
WeightTables weight_tables(const scf_plan* p, bool image) {
  return WeightTables{p->nmax, p->lmax, p->nmaxc, image && p->rs == 4, p->d_cs, p->d_fw,
                      p->d_rtab};
}

struct WsLayout {
  size_t partials, red1, coef, W, total;
};

WsLayout ws_layout(const scf_plan* p, int64_t n, int nclusters, int nblocks) {
  nblocks = std::max(nblocks, coef_blocks_max(p, n));  // layout independent of the variant
  WsLayout L;
  size_t off = 0;
  L.partials = off;
  off += align256((size_t)std::max(nblocks, 1) * p->T * p->rs);
  L.red1 = off;
  off += align256((size_t)kReduceChunks * p->T * sizeof(double) * std::max(nclusters, 1));
  L.coef = off;
  off += align256((size_t)p->T * sizeof(double) * std::max(nclusters, 1));
  L.W = off;
  off += align256(fw_elems(p) * p->rs * std::max(nclusters, 1));
  L.total = off;
  (void)n;
  return L;
}

size_t plain_need(const scf_plan* p, int64_t n) { return ws_layout(p, n, 1, 0).total; }

// Batched workspace: the common layout for nclusters, then the current centre
// rows and the region one copy fills at the start of a call: the step counter,
// the work lists and the first chunk of the centre table (BatchUpload).
constexpr int kCentreRows = 256;  // centre-table rows uploaded per chunk
constexpr int kGraphSteps = 8;    // middle steps replayed per graph launch

// Offsets of a call's upload: the step counter (zero), particle ranges and
// slots of U wave-units, partial-row ranges of the clusters, cluster and
// particle range of nblk field blocks, and `crows` centre-table rows.
struct BatchUpload {
  size_t ctr, seg_begin, seg_end, seg_slot, rows, blk_cluster, blk_begin, blk_end, tab, total;
  BatchUpload(int64_t U, int ncl, int64_t nblk, int64_t crows) {
    size_t off = 0;
    auto take = [&](size_t bytes) {
      const size_t at = off;
      off += align256(bytes);
      return at;
    };
    ctr = take(sizeof(int));
    seg_begin = take((size_t)U * 8);
    seg_end = take((size_t)U * 8);
    seg_slot = take((size_t)U * 4);
    rows = take((size_t)(ncl + 1) * 4);
    blk_cluster = take((size_t)nblk * 4);
    blk_begin = take((size_t)nblk * 8);
    blk_end = take((size_t)nblk * 8);
    tab = take((size_t)crows * ncl * 9 * sizeof(double));
    total = off;
  }
};

// Waits on the host until the last batched call's kernels are done.  Its staging
// is free earlier (ev_staging); this is for what must not happen beside it: a
// call on another stream (the workspace is usually the same one), and the end of
// a graph that it may still be replaying.
scf_status batch_wait(scf_plan* p) {
  if (!p->batch_pending) return SCF_OK;
  HIP_TRY(hipEventSynchronize(p->ev_batch));
  p->batch_pending = false;
  return SCF_OK;
}

// Bytes of pinned staging to allocate for a call that needs `need` (its upload
// and its whole centre table): a re-allocation costs 0.4 ms, so the first one
// takes what any call on as many particles and clusters needs for up to
// kCentreRows centre rows (`bound`, where that is at most 1 MiB more), and a
// longer run's leaves room for half as much again.
size_t staging_capacity(size_t need, size_t bound) {
  return need <= bound ? std::min(bound, need + (size_t(1) << 20)) : need + need / 2;
}

struct BatchLayout {
  WsLayout L;
  size_t cur, up, up_bytes, total;
  int max_units;
  int64_t max_blocks;
};

BatchLayout batch_layout(const scf_plan* p, int64_t n, int ncl) {
  BatchLayout B;
  int max_units = 0, max_rows = 0;
  for (int v = 0; v < p->eng->coef_variants(); ++v) {
    const int u = p->resident[v] * p->num_cu + ncl;
    max_units = std::max(max_units, u);
    max_rows = std::max(max_rows, u * p->eng->rows_per_unit(v));
  }
  B.max_units = max_units;
  B.max_blocks = (n + 255) / 256 + ncl;
  B.L = ws_layout(p, n, ncl, max_rows);
  size_t off = B.L.total;
  B.cur = off;
  off += align256((size_t)ncl * 9 * sizeof(double));
  B.up = off;
  B.up_bytes = BatchUpload(max_units, ncl, B.max_blocks, kCentreRows).total;
  off += B.up_bytes;
  B.total = off;
  return B;
}

template <typename R>
void fill_host_params(HostParams<R>& hp, const scf_host* h) {
  std::memset(&hp, 0, sizeof(hp));
  if (!h) return;
  hp.ncomp = h->ncomp;
  hp.G = R(h->G);
  for (int c = 0; c < h->ncomp; ++c) {
    hp.kind[c] = h->comp[c].kind;
    for (int k = 0; k < 3; ++k) hp.p[c][k] = R(h->comp[c].p[k]);
  }
}

scf_status check_host(const scf_host* h) {
  if (!h) return SCF_OK;
  if (h->ncomp < 0 || h->ncomp > SCF_MAX_HOST_COMP)
    return fail(SCF_ERR_INVALID_ARG, "host->ncomp = %d outside [0, %d]", h->ncomp, SCF_MAX_HOST_COMP);
  if (h->ncomp > 0 && !(h->G > 0.0)) return fail(SCF_ERR_INVALID_ARG, "host->G must be > 0");
  for (int c = 0; c < h->ncomp; ++c) {
    const int k = h->comp[c].kind;
    if (k < SCF_HOST_LOG || k > SCF_HOST_PLUMMER)
      return fail(SCF_ERR_INVALID_ARG, "host component %d has unknown kind %d", c, k);
    for (int q = 0; q < 3; ++q)
      if (!std::isfinite(h->comp[c].p[q]))
        return fail(SCF_ERR_INVALID_ARG, "host component %d parameter %d is not finite", c, q);
    if (k != SCF_HOST_MN && !(h->comp[c].p[1] > 0.0))
      return fail(SCF_ERR_INVALID_ARG, "host component %d: scale parameter must be > 0", c);
  }
  return SCF_OK;
}

// centre acceleration -grad psi_host(R) in double precision
void centre_accel(const HostParams<double>& H, const double* R, double* g) {
  double gx = 0, gy = 0, gz = 0;
  if (H.ncomp > 0) host_grad<double>(H, R[0], R[1], R[2], gx, gy, gz);
  g[0] = -gx;
  g[1] = -gy;
  g[2] = -gz;
}

template <typename R>
void fill_force_common(ForceArgs<R>& fa, const scf_plan* p) {
  std::memset(&fa, 0, sizeof(fa));
  fa.beta_rad = (const R*)p->d_beta_rad;
  fa.beta_ang = (const R*)p->d_beta_ang;
  fa.binv = R(1.0 / p->basis.b);
  fa.alpha = R(p->basis.alpha);
  fa.inv_alpha = R(1.0 / p->basis.alpha);
  fa.amode = p->amode;
  fa.dtab = p->d_dtab;
  fa.beta_img = (const R*)p->d_beta_img;
}

template <typename R>
void fill_coef_common(CoefArgs<R>& ca, const scf_plan* p) {
  using S = scalar_t<R>;
  std::memset(&ca, 0, sizeof(ca));
  ca.beta_rad = (const S*)p->d_beta_rad;
  ca.beta_ang = (const S*)p->d_beta_ang;
  ca.T = (int)p->T;
  ca.nmax = p->nmax;
  ca.binv = S(1.0 / p->basis.b);
  ca.alpha = S(p->basis.alpha);
  ca.inv_alpha = S(1.0 / p->basis.alpha);
  ca.amode = p->amode;
}

// Sum of `rows` partial rows (FP32 or FP64) in double precision, then the
// coefficients (coef, nullable), the force weights of a history row (W,
// nullable) and the field weights FW (nullable; with the operand image: image).  Up to
// kSmallRows rows: one pass (a block per (l, j)); otherwise chunk sums first
// (two launches, fixed order either way).
constexpr int kSmallRows = 2048;

scf_status reduce_and_finalize(scf_plan* p, const void* partials, int rows, double* coef, void* W,
                               void* FW, bool image, char* ws, const WsLayout& L, hipStream_t s) {
  const WeightTables wt = weight_tables(p, image);
  if (rows <= kSmallRows) {
    Timed t(p, s, K_REDUCE);
    HIP_TRY(launch_reduce_final(p->dtype, false, partials, rows, wt, coef, W, FW, s));
    return SCF_OK;
  }
  double* red1 = (double*)(ws + L.red1);
  const int nch = std::min(kReduceChunks, rows);
  {
    Timed t(p, s, K_REDUCE);
    HIP_TRY(launch_reduce(p->dtype, partials, rows, (int)p->T, nch, red1, s));
  }
  {
    Timed t(p, s, K_FINALIZE);
    HIP_TRY(launch_reduce_final(p->dtype, true, red1, nch, wt, coef, W, FW, s));
  }
  return SCF_OK;
}

// coefficients of n particles into coef (device, nullable) and, where the caller
// reads them, field weights FW (device, nullable; with the operand image: image);
// with W non-null also the force weights of a history row
template <typename R>
scf_status run_coeffs(scf_plan* p, int64_t n, const void* x, const void* y, const void* z,
                      const void* m, double* coef, void* FW, bool image, char* ws,
                      const WsLayout& L, hipStream_t s, void* W = nullptr) {
  int64_t stages;
  const int units = coef_units(p, n, &stages);
  const int rpu = units > 0 ? unit_rows(p, p->coef_variant, (stages + units - 1) / units) : 1;
  const int nb = units * rpu;
  if (n == 0) {
    // empty particle set: all coefficients vanish
    // (every caller with n = 0 passes coef and no history row)
    if (coef) {
      Timed t(p, s, K_FILL);
      HIP_TRY(launch_fill(coef, p->T, 0.0, s));
    }
    if (FW) {
      Timed t(p, s, K_MAKE_W);
      HIP_TRY(launch_make_w(p->dtype, coef ? coef : (double*)(ws + L.coef),
                            weight_tables(p, image), nullptr, FW, s));
    }
    return SCF_OK;
  }
  CoefArgs<R> ca;
  fill_coef_common(ca, p);
  ca.x = (const R*)x;
  ca.y = (const R*)y;
  ca.z = (const R*)z;
  ca.m = (const R*)m;
  ca.begin = 0;
  ca.stages = stages;
  ca.n = n;
  ca.partials = (R*)(ws + L.partials);
  ca.nunits = units;
  ca.one_row = rpu == 1;
  {
    Timed t(p, s, K_COEF);
    HIP_TRY(p->eng->launch_coef(&ca, units, p->coef_variant, s));
  }
  return reduce_and_finalize(p, ca.partials, nb, coef, W, FW, image, ws, L, s);
}

// Field pass over n particles.  mode 0: a (and psi) into ax, ay, az (pot);
// mode 1: kick by `kick`, drift by `drift` with the drifted positions written
// to xo (default: in place); mode 2: adjoint accumulation (see field_kernel).
// single: an evaluation that no run continues from (use_image).
template <typename R>
scf_status run_field(scf_plan* p, int64_t n, void* x, void* y, void* z, void* vx, void* vy,
                     void* vz, void* ax, void* ay, void* az, void* pot, const void* W,
                     const HostParams<R>& hp, const double* cen, int mode, double kick,
                     double drift, hipStream_t s, void* xo = nullptr, void* yo = nullptr,
                     void* zo = nullptr, const void* mass = nullptr, bool single = false) {
  if (n == 0) return SCF_OK;
  ForceArgs<R> fa;
  fill_force_common(fa, p);
  fa.x = (R*)x;
  fa.y = (R*)y;
  fa.z = (R*)z;
  fa.xo = (R*)(xo ? xo : x);
  fa.yo = (R*)(yo ? yo : y);
  fa.zo = (R*)(zo ? zo : z);
  fa.mass = (const R*)mass;
  fa.vx = (R*)vx;
  fa.vy = (R*)vy;
  fa.vz = (R*)vz;
  fa.ax = (R*)ax;
  fa.ay = (R*)ay;
  fa.az = (R*)az;
  fa.pot = (R*)pot;
  fa.W = (const R*)W;
  fa.n = n;
  fa.image = single || use_image(p, n);
  fa.kick = R(kick);
  fa.drift = R(drift);
  fa.host = hp;
  fa.cx = R(cen ? cen[0] : 0.0);
  fa.cy = R(cen ? cen[1] : 0.0);
  fa.cz = R(cen ? cen[2] : 0.0);
  fa.gcx = R(cen ? cen[3] : 0.0);
  fa.gcy = R(cen ? cen[4] : 0.0);
  fa.gcz = R(cen ? cen[5] : 0.0);
  Timed t(p, s, mode == 0 ? K_FIELD : (mode == 1 ? K_STEP_FIELD : K_ADJ));
  HIP_TRY(p->eng->launch_force(&fa, (n + 255) / 256, mode, p->field_variant, s));
  return SCF_OK;
}

// Basis tables of a plan for (alpha, b) (and its nmax, lmax, G): recurrence
// constants, per-coefficient sign and scale, density constants; uploaded to
// the plan's device buffers (allocated on the first call).
hipError_t fill_tables(scf_plan* p, const scf_basis* basis) {
  p->basis = *basis;
  p->amode = basis->alpha == 1.0 ? 0 : (basis->alpha == 0.5 ? 1 : 2);
  const int L1 = p->lmax + 1, NW = p->nmaxc + 1;
  // Legendre table: b_{l,m} at [m L1 + l] (b_{m,m} = -1 starts the order
  // recurrence of the field pass), then the integers 0..lmax at [L1 L1 + k]
  std::vector<double> brad((size_t)L1 * NW, 0.0), bang((size_t)L1 * L1 + L1, 0.0);
  for (int l = 0; l <= p->lmax; ++l) {
    const double lam = (2.0 * l + 1.0) * basis->alpha + 0.5;
    for (int n = 0; n <= p->nmaxc; ++n) brad[(size_t)l * NW + n] = gegen_beta(n, lam);
  }
  for (int m = 0; m <= p->lmax; ++m)
    for (int l = 0; l <= p->lmax; ++l) bang[(size_t)m * L1 + l] = l == m ? -1.0 : legendre_gamma(l, m);
  for (int k = 0; k <= p->lmax; ++k) bang[(size_t)L1 * L1 + k] = k;
  const int L2 = L1 * L1;
  p->h_cs.assign(p->T, 0.0);
  p->h_fw.assign(p->T, 0.0);
  for (int n = 0; n <= p->nmax; ++n) {
    for (int l = 0; l <= p->lmax; ++l) {
      const double lam = (2.0 * l + 1.0) * basis->alpha + 0.5;
      const double Nnl = norm_nl(basis->alpha, basis->b, basis->G, n, l);
      const double kn = gegen_lead(n, lam);
      for (int j = 0; j <= 2 * l; ++j) {
        const int m = (j + 1) / 2;
        const double kappa = -(kn / std::sqrt(Nnl)) * ylm_norm(l, m) * ((m & 1) ? -1.0 : 1.0) *
                             legendre_rho(l, m);
        const bool sin_part = j > 0 && (j % 2 == 0);
        const double sigma = sin_part ? 1.0 : -1.0;
        const double w = j == 0 ? 1.0 : (sin_part ? -2.0 : 2.0);
        const int64_t t = (int64_t)n * L2 + l * l + j;
        p->h_cs[t] = sigma * kappa;
        p->h_fw[t] = w * kappa;
      }
    }
  }
  // device copies: allocated on the first call, overwritten afterwards
  auto upload_real = [&](const std::vector<double>& v, void** dst) -> hipError_t {
    if (!*dst) {
      hipError_t e = hipMalloc(dst, v.size() * p->rs + 16);
      if (e != hipSuccess) return e;
    }
    if (p->rs == 4) {
      std::vector<float> f(v.begin(), v.end());
      return hipMemcpy(*dst, f.data(), f.size() * 4, hipMemcpyHostToDevice);
    }
    return hipMemcpy(*dst, v.data(), v.size() * 8, hipMemcpyHostToDevice);
  };
  hipError_t e = upload_real(brad, &p->d_beta_rad);
  if (e == hipSuccess) e = upload_real(bang, &p->d_beta_ang);
  if (e == hipSuccess && !p->d_cs) e = hipMalloc((void**)&p->d_cs, p->T * 8);
  if (e == hipSuccess) e = hipMemcpy(p->d_cs, p->h_cs.data(), p->T * 8, hipMemcpyHostToDevice);
  if (e == hipSuccess && !p->d_fw) e = hipMalloc((void**)&p->d_fw, p->T * 8);
  if (e == hipSuccess) e = hipMemcpy(p->d_fw, p->h_fw.data(), p->T * 8, hipMemcpyHostToDevice);
  {
    // density basis: the radial Laplacian of s^l (1 + s^(1/alpha))^(-p) C_n^lambda(xi)
    // is -K_nl s^(1/alpha - 2) (1 + s^(1/alpha))^(-2) times the same function,
    // K_nl = [n(n + 2 lambda) + p(p + 1)] / alpha^2, p = alpha (2l + 1)
    std::vector<double> kd((size_t)L1 * NW, 0.0);
    const double a = basis->alpha;
    for (int l = 0; l <= p->lmax; ++l)
      for (int n = 0; n <= p->nmax; ++n) {
        const double pp = a * (2.0 * l + 1.0), lam = pp + 0.5;
        const double K = (n * (n + 2.0 * lam) + pp * (pp + 1.0)) / (a * a);
        kd[(size_t)l * NW + n] = -K / (4.0 * M_PI * basis->G * basis->b * basis->b);
      }
    if (e == hipSuccess && !p->d_kden) e = hipMalloc((void**)&p->d_kden, kd.size() * 8);
    if (e == hipSuccess) e = hipMemcpy(p->d_kden, kd.data(), kd.size() * 8, hipMemcpyHostToDevice);
  }
  {
    // the xi-derivative of the monic Gegenbauer basis in the same basis:
    // d C_n^lam / d xi = 2 lam C_{n-1}^(lam+1) = 2 sum_{k = n-1, n-3, ..} (k + lam) C_k^lam,
    // so for p_n = C_n^lam / kappa_n (kappa_n = 2^n (lam)_n / n!, the leading
    // coefficient) d p_n / d xi = sum_k D_nk p_k with D_nk = 2 (k + lam) kappa_k / kappa_n
    // for odd n - k > 0.  The matrix-core field pass needs the coefficients
    // W'_k = sum_n D_nk W_n = 2 (k + lam) kappa_k S_k, S_k = sum_{n = k+1, k+3, ..} W_n / kappa_n,
    // a suffix sum it forms per row; stored per degree: [l][0][n] = 1 / kappa_n,
    // [l][1][k] = 2 (k + lam) kappa_k.
    std::vector<double> dt((size_t)L1 * 2 * NW, 0.0);
    for (int l = 0; l <= p->lmax; ++l) {
      const double lam = (2.0 * l + 1.0) * basis->alpha + 0.5;
      double kap = 1.0;
      for (int n = 0; n <= p->nmaxc; ++n) {
        dt[((size_t)l * 2 + 0) * NW + n] = 1.0 / kap;
        dt[((size_t)l * 2 + 1) * NW + n] = 2.0 * (n + lam) * kap;
        kap *= 2.0 * (lam + n) / (n + 1.0);
      }
    }
    if (e == hipSuccess && !p->d_dtab) e = hipMalloc((void**)&p->d_dtab, dt.size() * 8);
    if (e == hipSuccess) e = hipMemcpy(p->d_dtab, dt.data(), dt.size() * 8, hipMemcpyHostToDevice);
  }
  {
    // Radial weights of the operand image (FwLayout).  l >= 1: the factors of
    // W_{k-1} and W_{k+1} in W^r_k; l = 0: 1 / kappa_k and 2 (k + lam) kappa_k.
    const int NP = NW + 1;
    std::vector<double> rt((size_t)L1 * 2 * NP, 0.0), bi((size_t)L1 * NP, 0.0);
    const double ia = 1.0 / basis->alpha;
    for (int l = 0; l <= p->lmax; ++l) {
      const double lam = (2.0 * l + 1.0) * basis->alpha + 0.5;
      double* r0 = &rt[(size_t)l * 2 * NP];
      double* r1 = r0 + NP;
      double kap = 1.0;
      for (int k = 0; k < NP; ++k) {
        bi[(size_t)l * NP + k] = gegen_beta(k, lam);
        if (l == 0) {
          r0[k] = 1.0 / kap;
          r1[k] = 2.0 * (k + lam) * kap;
          kap *= 2.0 * (lam + k) / (k + 1.0);
        } else {
          r0[k] = -0.5 * ((2.0 * l + 1.0) + (k - 1.0) * ia);
          r1[k] = 0.5 * gegen_beta(k + 2, lam) * ((2.0 * l + 1.0) + (k + 2.0) * ia);
        }
      }
    }
    if (e == hipSuccess) e = upload_real(bi, &p->d_beta_img);
    if (e == hipSuccess && !p->d_rtab) e = hipMalloc((void**)&p->d_rtab, rt.size() * 8);
    if (e == hipSuccess) e = hipMemcpy(p->d_rtab, rt.data(), rt.size() * 8, hipMemcpyHostToDevice);
  }
  return e;
}

// ---------------------------------------------------------------------------
// adjoint
// ---------------------------------------------------------------------------
// gamma-pass launch geometry (one resident round, like the coefficient pass)
int gamma_units(const scf_plan* p, int64_t n, int64_t* stages) {
  if (n <= 0) {
    *stages = 0;
    return 0;
  }
  const int P = p->eng->gamma_stage_particles();
  *stages = (n + P - 1) / P;
  const int64_t cap = (int64_t)p->gamma_resident * p->num_cu;
  return (int)std::min<int64_t>(*stages, std::max<int64_t>(cap, 1));
}

// Adjoint workspace: the common layout (partials sized for both passes), the
// segment's positions X_k and field weights W_k (k = 0..nsteps), the gamma
// weights W', velocity and acceleration scratch, the Hessian-vector kernel's
// block sums of every kick and the per-kick host sums S_k.
struct AdjLayout {
  WsLayout L;
  size_t X, Wsv, Wp, V, A, hp, S, total;
  int64_t nblk;
  size_t wsz;
};

AdjLayout adj_layout(const scf_plan* p, int64_t n, int nsteps) {
  AdjLayout A;
  int64_t st;
  const int grows = gamma_units(p, n, &st) * p->eng->gamma_rows_per_unit();
  A.L = ws_layout(p, n, 1, grows);
  A.wsz = fw_elems(p);
  A.nblk = (n + 255) / 256;
  const size_t rs = p->rs;
  size_t off = A.L.total;
  A.X = off;
  off += align256((size_t)(nsteps + 1) * 3 * n * rs);
  A.Wsv = off;
  off += align256((size_t)(nsteps + 1) * A.wsz * rs);
  A.Wp = off;
  off += align256(A.wsz * rs);
  A.V = off;
  off += align256((size_t)3 * n * rs);
  A.A = off;
  off += align256((size_t)3 * n * rs);
  A.hp = off;
  off += align256((size_t)(nsteps + 1) * std::max<int64_t>(A.nblk, 1) * 32 * rs);
  A.S = off;
  off += align256((size_t)(nsteps + 1) * 32 * sizeof(double));
  A.total = off;
  return A;
}

// gamma_t = sum_i mu_i . grad b_t(x_i), mu = c (ex, ey, ez), turned into the
// field weights W' of Eq. (total_potential) (the same scales as the forward
// coefficients)
template <typename R>
scf_status run_gamma(scf_plan* p, int64_t n, const void* x, const void* y, const void* z,
                     const void* ex, const void* ey, const void* ez, double c, void* Wout, char* ws,
                     const WsLayout& L, hipStream_t s) {
  int64_t stages;
  const int units = gamma_units(p, n, &stages);
  CoefArgs<Dual<R>> ca;
  fill_coef_common(ca, p);
  ca.x = (const R*)x;
  ca.y = (const R*)y;
  ca.z = (const R*)z;
  ca.ex = (const R*)ex;
  ca.ey = (const R*)ey;
  ca.ez = (const R*)ez;
  ca.escale = R(c);
  ca.begin = 0;
  ca.n = n;
  ca.stages = stages;
  ca.nunits = units;
  ca.partials = (acc_t<Dual<R>>*)(ws + L.partials);
  const int fold = p->eng->gamma_fold_stages();
  ca.one_row = fold > 0 && (stages + units - 1) / units <= fold;
  {
    Timed t(p, s, K_ADJ);
    HIP_TRY(p->eng->launch_gamma(&ca, units, s));
  }
  const int rows = units * (ca.one_row ? 1 : p->eng->gamma_rows_per_unit());
  return reduce_and_finalize(p, ws + L.partials, rows, nullptr, nullptr, Wout, field_image(p, n),
                             ws, L, s);
}

bool ptr_ok(const void* q) { return q != nullptr; }

// workspace regions are laid out at 256-byte offsets from its start
bool ws_aligned(const void* ws) { return ((uintptr_t)ws & 255) == 0; }

}  // namespace
