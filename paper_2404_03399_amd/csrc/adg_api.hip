// C ABI of the ADG library: validation, reference operators, AT table,
// workspace layout, launch sequencing and hipGraph replay.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <tuple>
#include <vector>

#include "adg.h"
#include "adg_device.hpp"
#include "adg_launch.hpp"

using namespace adg;

namespace {

thread_local std::string g_err;

int fail(int code, const std::string& msg) {
  g_err = msg;
  return code;
}

// State vectors are read and written as 16-byte pairs of nodal values.
bool state_aligned(const void* p) { return ((uintptr_t)p & 15u) == 0; }

#define ADG_HIP(expr)                                                                         \
  do {                                                                                        \
    hipError_t e_ = (expr);                                                                   \
    if (e_ != hipSuccess) return fail(ADG_E_HIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
  } while (0)

constexpr int64_t kAlign = 256;
constexpr int kGraphSteps = 16;  // steps of a batch: an even number of launches, which ends in the caller's buffer
int64_t align_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }

// ------------------------------------------------ reference element (host) --
// Legendre P_p and P_p' at x by the three-term recurrence.
void legendre(int p, long double x, long double* P, long double* dP) {
  long double p0 = 1.0L, p1 = x;
  if (p == 0) { *P = 1.0L; *dP = 0.0L; return; }
  for (int k = 1; k < p; ++k) {
    const long double p2 = ((2 * k + 1) * x * p1 - k * p0) / (k + 1);
    p0 = p1;
    p1 = p2;
  }
  *P = p1;
  *dP = p * (x * p1 - p0) / (x * x - 1.0L);  // valid for |x| < 1
}

// Gauss-Lobatto-Legendre nodes: -1, roots of P_p' (Newton from the
// Chebyshev-Lobatto points), +1.
void gll(int p, long double* x) {
  x[0] = -1.0L;
  x[p] = 1.0L;
  for (int i = 1; i < p; ++i) {
    long double z = -std::cos(3.14159265358979323846264338327950288L * i / p);
    for (int it = 0; it < 100; ++it) {
      long double P, dP;
      legendre(p, z, &P, &dP);
      // (1 - z^2) P'' = 2 z P' - p (p + 1) P
      const long double d2P = (2.0L * z * dP - p * (p + 1) * P) / (1.0L - z * z);
      const long double step = dP / d2P;
      z -= step;
      if (std::fabs(step) < 1e-30L) break;
    }
    x[i] = z;
  }
  std::sort(x, x + p + 1);
}

// Monomial coefficients c[j][m] of the Lagrange cardinal polynomials.
void lagrange_monomials(int p, const long double* x, long double c[kMaxNp][kMaxNp]) {
  for (int j = 0; j <= p; ++j) {
    long double poly[kMaxNp] = {1.0L};
    int deg = 0;
    for (int m = 0; m <= p; ++m) {
      if (m == j) continue;
      const long double inv = 1.0L / (x[j] - x[m]);
      long double nxt[kMaxNp] = {0};
      for (int d = 0; d <= deg; ++d) {
        nxt[d + 1] += poly[d] * inv;
        nxt[d] -= poly[d] * x[m] * inv;
      }
      ++deg;
      std::memcpy(poly, nxt, sizeof(poly));
    }
    for (int m = 0; m <= p; ++m) c[j][m] = poly[m];
  }
}

long double mono_int(int k) { return (k % 2) ? 0.0L : 2.0L / (k + 1); }  // int_{-1}^{1} xi^k

// Solve A X = B (n x n, m right-hand sides) by Gaussian elimination with
// partial pivoting, in place (B becomes X).
void solve(int n, int m, long double A[kMaxNp][kMaxNp], long double B[kMaxNp][kMaxNp + 2]) {
  for (int c = 0; c < n; ++c) {
    int piv = c;
    for (int r = c + 1; r < n; ++r)
      if (std::fabs(A[r][c]) > std::fabs(A[piv][c])) piv = r;
    for (int k = 0; k < n; ++k) std::swap(A[c][k], A[piv][k]);
    for (int k = 0; k < m; ++k) std::swap(B[c][k], B[piv][k]);
    for (int r = 0; r < n; ++r) {
      if (r == c) continue;
      const long double f = A[r][c] / A[c][c];
      for (int k = 0; k < n; ++k) A[r][k] -= f * A[c][k];
      for (int k = 0; k < m; ++k) B[r][k] -= f * B[c][k];
    }
  }
  for (int r = 0; r < n; ++r)
    for (int k = 0; k < m; ++k) B[r][k] /= A[r][r];
}

// D = M^-1 S, lift_l = M^-1 e_0, lift_r = M^-1 e_p, w = M 1; M and S integrated
// exactly on monomials: M_ij = int phi_i phi_j, S_ij = int phi_j phi_i'.
void element_operators(int p, DevProblem* dp) {
  const int np = p + 1;
  long double x[kMaxNp], c[kMaxNp][kMaxNp];
  gll(p, x);
  lagrange_monomials(p, x, c);
  long double M[kMaxNp][kMaxNp] = {}, RHS[kMaxNp][kMaxNp + 2] = {};
  for (int i = 0; i < np; ++i)
    for (int j = 0; j < np; ++j) {
      long double m = 0.0L, s = 0.0L;
      for (int a = 0; a < np; ++a)
        for (int b = 0; b < np; ++b) {
          m += c[i][a] * c[j][b] * mono_int(a + b);
          if (b >= 1) s += c[j][a] * (b * c[i][b]) * mono_int(a + b - 1);
        }
      M[i][j] = m;
      RHS[i][j] = s;
    }
  long double w[kMaxNp] = {};
  for (int i = 0; i < np; ++i)
    for (int j = 0; j < np; ++j) w[i] += M[i][j];
  RHS[0][np] = 1.0L;       // e_0
  RHS[p][np + 1] = 1.0L;   // e_p
  solve(np, np + 2, M, RHS);
  for (int i = 0; i < kMaxNp * kMaxNp; ++i) dp->D[i] = 0.0;
  for (int i = 0; i < np; ++i) {
    for (int j = 0; j < np; ++j) dp->D[i * kMaxNp + j] = (double)RHS[i][j];
    dp->lift_l[i] = (double)RHS[i][np];
    dp->lift_r[i] = (double)RHS[i][np + 1];
    dp->wq[i] = (double)w[i];
  }
}

// AT coefficients in closed form: the moment conditions of the AT flux make
// c_j(k) the Lagrange weights extrapolating levels -(k+j) to 0:
// c_j(k) = prod_{m != j} (k + m) / (m - j)  (integers).
double at_coefficient(int q, int k, int j) {
  long long num = 1, den = 1;
  for (int m = 0; m < q; ++m) {
    if (m == j) continue;
    num *= (long long)(k + m);
    den *= (long long)(m - j);
  }
  return (double)(num / den);
}

int phys_of(const adg_problem& p) {
  if (p.equation == ADG_EQ_BURGERS) return PHYS_BURGERS_LLF;
  if (p.equation == ADG_EQ_VISCOUS_BURGERS) return PHYS_BURGERS_LDG;
  return p.flux == ADG_FLUX_CENTRAL ? PHYS_ADV_CENTRAL : PHYS_ADV_UPWIND;
}

int q_of(const adg_problem& p) {
  if (p.scheme != ADG_SCHEME_ADG_AT) return 1;
  return p.at_levels ? (int)p.at_levels : (int)p.degree + 1;
}

int64_t ld_of(const adg_problem& p) { return align_up(p.n_elem, 64); }

bool async_of(const adg_problem& p) { return p.scheme != ADG_SCHEME_DG && p.n_elem / p.pe_size > 1; }

int validate_one(const adg_problem& p, int idx) {
  const std::string at = "problem " + std::to_string(idx) + ": ";
  if (p.abi_version != ADG_ABI_VERSION) return fail(ADG_E_ABI, at + "abi_version mismatch");
  if (p.equation > ADG_EQ_VISCOUS_BURGERS) return fail(ADG_E_INVALID, at + "unknown equation");
  if (p.equation == ADG_EQ_VISCOUS_BURGERS && (p.flux != ADG_FLUX_LLF || !(p.viscosity >= 0.0) ||
                                               !std::isfinite(p.viscosity)))
    return fail(ADG_E_INVALID, at + "viscous Burgers needs the llf flux and a finite viscosity >= 0");
  if (p.equation != ADG_EQ_VISCOUS_BURGERS && p.viscosity != 0.0)
    return fail(ADG_E_INVALID, at + "viscosity is only for viscous Burgers");
  if (p.scheme > ADG_SCHEME_ADG_AT) return fail(ADG_E_INVALID, at + "unknown scheme");
  if (p.flux > ADG_FLUX_LLF) return fail(ADG_E_INVALID, at + "unknown flux");
  if (p.rk > ADG_LSRK4) return fail(ADG_E_INVALID, at + "unknown rk");
  if (p.degree < 1 || p.degree > 4) return fail(ADG_E_INVALID, at + "degree must be in 1..4");
  if (p.equation == ADG_EQ_ADVECTION && p.flux == ADG_FLUX_LLF)
    return fail(ADG_E_INVALID, at + "llf flux is for Burgers");
  if (p.equation == ADG_EQ_BURGERS && p.flux != ADG_FLUX_LLF)
    return fail(ADG_E_INVALID, at + "Burgers needs the llf flux");
  if (p.at_levels != 0 && p.scheme != ADG_SCHEME_ADG_AT)
    return fail(ADG_E_INVALID, at + "at_levels is only for ADG-AT");
  if (p.at_levels > (uint32_t)kMaxQ) return fail(ADG_E_INVALID, at + "at_levels must be <= 5");
  if (p.scheme == ADG_SCHEME_ADG_AT && p.at_levels == 0 && p.degree + 1 > (uint32_t)kMaxQ)
    return fail(ADG_E_INVALID, at + "q = degree + 1 exceeds 5");
  if (p.n_delays < 1 || p.n_delays > (uint32_t)kMaxL) return fail(ADG_E_INVALID, at + "n_delays must be in 1..8");
  if (p.delay_granularity > ADG_DELAY_CAA) return fail(ADG_E_INVALID, at + "bad delay_granularity");
  if (p.delay_granularity == ADG_DELAY_CAA && p.n_delays != 3)
    return fail(ADG_E_INVALID, at + "the communication-avoiding cycle needs n_delays = 3");
  if (p.reserved != 0) return fail(ADG_E_INVALID, at + "reserved must be 0");
  if (p.n_elem < 2 || p.n_elem > (int64_t)1 << 30) return fail(ADG_E_INVALID, at + "n_elem must be in 2..2^30");
  if (p.pe_size < 1 || p.n_elem % p.pe_size != 0) return fail(ADG_E_INVALID, at + "pe_size must divide n_elem");
  for (uint32_t i = 0; i + 1 < p.n_delays; ++i) {
    if (p.delay_threshold[i] > (1ull << 53)) return fail(ADG_E_INVALID, at + "threshold > 2^53");
    if (i > 0 && p.delay_threshold[i] < p.delay_threshold[i - 1])
      return fail(ADG_E_INVALID, at + "thresholds must be non-decreasing");
  }
  if (!(p.length > 0.0) || !std::isfinite(p.length)) return fail(ADG_E_INVALID, at + "length must be > 0");
  if (!(p.dt > 0.0) || !std::isfinite(p.dt)) return fail(ADG_E_INVALID, at + "dt must be > 0");
  if (!std::isfinite(p.x_left)) return fail(ADG_E_INVALID, at + "x_left must be finite");
  if (p.equation == ADG_EQ_ADVECTION && (!(p.speed != 0.0) || !std::isfinite(p.speed)))
    return fail(ADG_E_INVALID, at + "speed must be finite and non-zero");
  return ADG_OK;
}

int validate(const adg_problem* probs, int32_t n) {
  if (!probs || n < 1) return fail(ADG_E_INVALID, "need at least one problem");
  for (int32_t i = 0; i < n; ++i) {
    const int rc = validate_one(probs[i], i);
    if (rc) return rc;
  }
  for (int32_t i = 1; i < n; ++i) {
    const adg_problem &a = probs[0], &b = probs[i];
    if (a.equation != b.equation || a.flux != b.flux || a.rk != b.rk || a.scheme != b.scheme)
      return fail(ADG_E_INVALID, "all problems of a context must share equation, flux, rk and scheme");
  }
  return ADG_OK;
}

// The fused kernel's linear form: upwind advection with a > 0 on meshes of
// kLinMinElems elements or more, whatever the PEs and delays (so that a problem
// without delays and its synchronous twin agree bit for bit), no recording.
// us per step, linear form and stage by stage, Heun / RK4 / LSRK4: one mesh of 256
// elements, p = 1 1.06, 1.11 / 1.23, 1.28 / 1.62, 1.61, p = 4 1.19, 1.25 / 1.37, 1.52 / 1.83,
// 2.00; 160 of 512, p = 1 1.74, 1.25 / 2.33, 1.92 / 2.54, 2.87, p = 4 1.74, 1.55 / 2.51,
// 2.80 / 2.95, 4.31; 160 of 1024, p = 1 1.30, 1.36 / 1.84, 1.93 / 2.30, 2.77, p = 4 1.70,
// 1.94 / 2.39, 2.96 / 2.91, 4.27; 160 of 4096, p = 4 3.25, 4.08 / 4.04, 5.84 / 5.40, 8.83;
// 2^20, p = 3 RK4 4.75, 6.55, 2^24 53.9, 84.2.  From 1024 elements on it is the faster
// one for every degree and integrator, below it depends on them, and a launch is
// latency for a single mesh.  Recorded runs keep the stage form (so their states are
// an unrecorded run's to rounding only): dJ/da can be a sum that cancels down to
// rounding (a misfit without a mode in common with the state), where its value is
// that of the order of operations.
constexpr int64_t kLinMinElems = 1024;
bool lin_of(const adg_problem& p, int kernel, int64_t n_rec) {
  return kernel == ADG_KERNEL_FUSED && phys_of(p) == PHYS_ADV_UPWIND && p.speed > 0.0 && n_rec == 0 &&
         p.n_elem >= kLinMinElems;
}

// Butcher coefficients of the integrators in extended precision (a: strictly
// lower triangular, b), the 2N schemes from their published A and B.
void butcher(int rk, long double (&a)[kMaxStages][kMaxStages], long double (&b)[kMaxStages]) {
  const int S = rk_stages(rk);
  for (int i = 0; i < kMaxStages; ++i) {
    b[i] = 0.0L;
    for (int j = 0; j < kMaxStages; ++j) a[i][j] = 0.0L;
  }
  if (rk == RK_RK4) {
    a[1][0] = a[2][1] = 0.5L;
    a[3][2] = 1.0L;
    b[0] = b[3] = 1.0L / 6.0L;
    b[1] = b[2] = 1.0L / 3.0L;
  } else if (rk == RK_SSP3) {
    a[1][0] = 1.0L;
    a[2][0] = a[2][1] = 0.25L;
    b[0] = b[1] = 1.0L / 6.0L;
    b[2] = 2.0L / 3.0L;
  } else if (rk == RK_HEUN) {
    a[1][0] = 1.0L;
    b[0] = b[1] = 0.5L;
  } else {
    // y_{s+1} = u + dt sum_{j<=s} beta_sj k_j, beta_sj = sum_{l=j..s} B_l prod_{m=j+1..l} A_m
    for (int s = 0; s < S; ++s)
      for (int j = 0; j <= s; ++j) {
        long double acc = 0.0L, prod = 1.0L;
        for (int l = j; l <= s; ++l) {
          if (l > j) prod *= (long double)ls_a(rk, l);
          acc += (long double)ls_b(rk, l) * prod;
        }
        (s + 1 < S ? a[s + 1][j] : b[j]) = acc;
      }
  }
}

// Table of the linear form (layout in adg_common.hpp): the stages of one step as
// linear maps of the element's nodes, of the fluxes F_j at its left face and
// of the differences delta_j at its right face, in extended precision, from
// the folded operators Kdu, Kl, Kr.
void lin_table(const DevProblem& d, int rk, double* out) {
  const int S = rk_stages(rk), np = d.np;
  long double A[kMaxStages][kMaxStages], B[kMaxStages];
  butcher(rk, A, B);
  const long double dt = d.dt, a = d.speed;
  // columns of a stage value y_s: np of u, then S of F, then S of delta
  constexpr int kCols = kMaxNp + 2 * kMaxStages;
  const int cols = np + 2 * S;
  long double y[kMaxStages + 1][kMaxNp][kCols] = {}, k[kMaxStages][kMaxNp][kCols] = {};
  for (int s = 0; s <= S; ++s) {
    for (int i = 0; i < np; ++i) {
      y[s][i][i] = 1.0L;
      for (int j = 0; j < s; ++j)
        for (int c = 0; c < cols; ++c) y[s][i][c] += (s < S ? A[s][j] : B[j]) * k[j][i][c];
    }
    if (s == S) break;
    for (int i = 0; i < np; ++i) {
      for (int j = 0; j < np; ++j)
        for (int c = 0; c < cols; ++c) k[s][i][c] += dt * (long double)d.Kdu[i * kMaxNp + j] * y[s][j][c];
      k[s][i][np + s] += dt * (long double)d.Kl[i];
      k[s][i][np + S + s] -= dt * (long double)d.Kr[i];
    }
  }
  for (int i = 0; i < lin_tab_size(np, S); ++i) out[i] = 0.0;
  for (int kind = 0; kind < kLinCols; ++kind)
    for (int j = 0; j < lin_cols(np, S, kind); ++j) {
      double* o = out + lin_col(np, S, kind, j);
      const int c = kind == LIN_Z || kind == LIN_A ? j : (kind == LIN_W || kind == LIN_PHI ? np : np + S) + j;
      if (kind == LIN_Z || kind == LIN_W || kind == LIN_WR)  // g_s of the stages s that the column reaches
        for (int s = kind == LIN_Z ? 1 : j + 1; s < S; ++s) *o++ = (double)(a * y[s][np - 1][c]);
      else  // u' less u
        for (int i = 0; i < np; ++i) *o++ = (double)(y[S][i][c] - (c == i ? 1.0L : 0.0L));
    }
}

// Problems with the same operators (one mesh, many delay realizations) share
// a table: key of the values it is formed from.
struct LinKey {
  uint32_t degree;
  double speed, dt, length;
  int64_t n_elem;
  bool operator<(const LinKey& o) const {
    return std::tie(degree, speed, dt, length, n_elem) < std::tie(o.degree, o.speed, o.dt, o.length, o.n_elem);
  }
};
LinKey lin_key(const adg_problem& p) { return LinKey{p.degree, p.speed, p.dt, p.length, p.n_elem}; }

// Work lists of the fused kernel, one per number of steps: a launch of K steps
// takes tiles whose halo holds K.
constexpr int kLists = 4;
static_assert(1 << (kLists - 1) == kMaxSteps, "lists of 1, 2, 4 and 8 steps");
int list_of(int K) { return __builtin_ctz((unsigned)K); }

// Launch shape of the fused kernel: elements per lane and most steps per launch.
struct Shape {
  int elems, kmax;
  int elems1 = 0, elems2 = 0;  // elements per lane of launches of one and two steps, if not elems
  bool any_face = false;  // two elements per lane although a PE size is odd (general stage form, local DG)
  bool halve4 = false, halve8 = false;  // halves_first may split a launch of four, of eight steps
  int elems_at(int K) const { return K == 1 && elems1 ? elems1 : (K == 2 && elems2 ? elems2 : elems); }
};

struct Layout {
  Shape shape;               // launch shape of the fused kernel
  Shape adj[2];              // of the fused reverse sweep, per list
  int depth_steps;           // steps per launch that the ring holds
  int64_t lin, lin_doubles;  // tables of the linear form
  int64_t probs, work_f, work_s, first_s, ctr, ring, state2, y0, y1, acc, qbuf, part, stats_out;
  int64_t groups, gstats;  // ensemble statistics: group CSR (2n+1 int32) and 4 doubles per group
  // adjoint recording (-1 if not recording)
  int64_t ckpt, useg, ybuf, lam, q, adjring, cpart, work_a[2];
  int64_t total;
  int32_t n_work_f[kLists];    // items of the fused kernel's lists,
  int32_t at_f[kLists + 1];    // where each list's room starts in work_f, and the end
  int32_t n_work_s, n_work_a[2];
  int64_t n_parts;  // partial sums of dJ/da of the fused reverse sweep
  int64_t total_doubles;
  int64_t ring_doubles;
  int64_t n_rec, ckpt_every, n_ckpt;
};

// Ring slots per (boundary, stage): when an adjoint recording horizon is given
// the whole run (every level is kept), and L + q + kmax - 2 more: a launch of K
// steps writes levels n .. n + K - 1 while waves that start later still read
// levels down to n + 2 - L - q; with that many slots no level written in a
// launch shares a slot with one that it reads.
int64_t depth_of(const adg_problem& p, int64_t n_rec, int kmax) {
  return n_rec + p.n_delays + q_of(p) + std::max(kmax, 2) - 2;
}

// Elements per lane of the fused kernel (0 if the request is invalid).
int lane_elems_of(const adg_problem* probs, int32_t n, const adg_options* opt) {
  int64_t min_pes = (int64_t)1 << 62;
  for (int32_t i = 0; i < n; ++i)
    if (async_of(probs[i])) min_pes = std::min(min_pes, probs[i].pe_size);
  const int req = opt ? opt->lane_elems : 0;
  if (req == 0) return min_pes < 2 ? 1 : 2;
  if (req != 1 && req != 2 && req != 4) return 0;
  return req <= min_pes ? req : 0;
}

// Time steps per fused launch (0 if the request is invalid).
int fused_steps_of(const adg_options* opt) {
  const int req = opt ? (int)opt->fused_steps : 0;
  if (req == 0) return 2;
  return (req == 1 || req == 2) ? req : 0;
}

// Kernel family: AUTO picks the fused kernel.
int kernel_of(const adg_problem*, const adg_options* opt) {
  if (!opt || opt->kernel == ADG_KERNEL_AUTO) return ADG_KERNEL_FUSED;
  return opt->kernel;
}

bool is_ldg(const adg_problem* probs) { return probs[0].equation == ADG_EQ_VISCOUS_BURGERS; }

// Whether the workspace holds room for window lists around the PE faces: what
// ADG_OPT_PE_SPLIT_ON and OFF still decide.  No kernel reads it: the fused kernel
// keeps waves with and without PE faces apart by itself.  By default where every
// asynchronous problem's PE size holds four windows of the longest launch of one or
// two steps and a wave two.
bool pe_split_of(const adg_problem* probs, int32_t n, const adg_options* opt) {
  const uint32_t f = opt ? opt->flags : 0u;
  if ((f & (ADG_OPT_PE_SPLIT_OFF | ADG_OPT_ONE_LAUNCH)) || kernel_of(probs, opt) != ADG_KERNEL_FUSED || is_ldg(probs))
    return false;
  const int K = fused_steps_of(opt) == 1 ? 1 : 2;
  const bool force = (f & ADG_OPT_PE_SPLIT_ON) != 0;
  if (!force && fused_windows_per_wave((int)probs[0].rk, K) < 2) return false;
  const int64_t need = (int64_t)fused_window((int)probs[0].rk, K) * (force ? 1 : 4);
  bool any = false;
  for (int32_t i = 0; i < n; ++i) {
    if (!async_of(probs[i])) continue;
    any = true;
    if (probs[i].pe_size < need) return false;
  }
  return any;
}
int64_t total_elems(const adg_problem* probs, int32_t n) {
  int64_t t = 0;
  for (int32_t i = 0; i < n; ++i) t += probs[i].n_elem;
  return t;
}

int form_of(const adg_problem& p, int kernel, int64_t n_rec) {
  return lin_of(p, kernel, n_rec) ? FORM_LIN : phys_of(p) == PHYS_ADV_UPWIND && p.speed > 0.0 ? FORM_POS : FORM_GEN;
}

// Owned elements of a work item of the list for K steps.
int tile_of(const adg_problem& p, int form, const Shape& s, int K) {
  if (p.equation == ADG_EQ_VISCOUS_BURGERS) return ldg_tile_elems((int)p.rk, s.elems_at(K), K);
  if (form == FORM_GEN) return fused_tile((int)p.rk, s.elems_at(K), K);
  return fused_tile_left((int)p.rk, s.elems_at(K), K, async_of(p));
}

// Doubles of LDS per wave for problem p in launches of K steps.
int lds_of(const adg_problem& p, int elems, int K) {
  return async_of(p) ? fused_lds_words(rk_stages((int)p.rk), K, fused_faces(elems, p.pe_size), is_ldg(&p) ? 2 : 1) : 0;
}

// Elements per lane R: the option's or the library's choice, halved until it
// divides every PE size (a PE face is then always the left face of a lane's
// first element).  Few elements per lane spread a small mesh over more waves,
// many make the halo small.  Steps per launch K: the option's, or the library's
// choice: the most, eight, as long as the halo leaves enough of the lanes (on
// small meshes, where a launch is latency, few are enough) and a workgroup's
// values at PE faces leave room for five workgroups in the 160 KB of LDS: below
// 32 KB, and with room for three, below 48, us per step at 2^22 elements, linear
// form PE 2 89, 133, PE 4 59, 72, PE 8 39, 48; central 97, 149, 66, 79, 51, 61;
// Burgers, SSP-RK3, p = 2 70, 86, 48, 50, 34, 39; local DG, Heun, p = 2 63, 79, 43, 46,
// 31, 34; dJ/du0 alone, a run and its adjoint, 2^20 103, 129, 58, 63, 37, 39, but 2^16
// 26.0, 23.5, 14.0, 12.1.
// Measured, us per step, PE 256, p = 3, RK4 unless stated (R and K in brackets):
//   linear form   2^14 elements (1,8) 1.35, (2,8) 1.50, (4,8) 1.87; 2^16 1.53,
//                 1.51, 1.90; 2^18 2.74, 2.25, 2.45; 2^19 (1,4) 4.38, (2,8) 3.38,
//                 (4,8) 3.19; 2^20 6.75, 5.22, 4.76, (4,2) 9.96
//   a > 0, stage  64 elements, p = 2 (1,8) 1.57, (2,8) 2.19, (4,8) 3.45; recorded
//                 2^20 (128 steps and their adjoint, ms) (2,4) 6.32, (2,8) 6.18,
//                 (4,4) 6.30, (4,8) 5.95
//   general, central flux   2^12 (1,4) 2.25, (2,8) 2.30, (4,8) 2.77; 2^16 2.74,
//                 2.76, 2.93; 2^18 5.01, 4.25, 4.12; 2^22 (2,4) 31.8, (4,4) 29.3,
//                 (4,8) 31.0; five stages (lsrk4, p = 2) 2^22 (4,4) 27.0, (4,8)
//                 30.6; 10^5, p = 4, lsrk4, PE 30 (2,2) 4.2, (2,4) 4.5, (2,8) 5.4
//   one and two steps per launch are bound by HBM, which two elements per lane,
//                 with more waves in flight, reach better (four for two steps only
//                 where the options ask for both): 2^20 central (2,1) 16.9, (4,1)
//                 19.1, (2,2) 11.0, (4,2) 11.7; Burgers, SSP-RK3, p = 2 14.1, 16.1,
//                 9.3, 10.0; a > 0 14.8, 17.6, 8.6, 9.6; local DG 14.4, 15.9, 9.1, 9.8
//   general, Burgers, SSP-RK3, p = 2   2^22 (2,4) 26.2, (4,4) 24.0, (4,8) 23.7
//   local DG, p = 2   Heun 2^14 (1,4) 2.02, (1,8) 1.79, (2,8) 1.85; 2^16 2.35, 2.10,
//                 1.92; 2^18 (2,8) 3.16, (4,8) 3.53; 2^20 8.11, 7.43; SSP-RK3 2^14
//                 (1,4) 2.25, (1,8) 2.14; 2^18 (2,4) 4.81, (2,8) 5.07; 2^20 (4,4)
//                 11.75, (4,8) 11.96; RK4, p = 3 2^14 (1,4) 2.63, (2,8) 2.87; 2^20
//                 (4,4) 17.8, (4,8) 18.7
constexpr int kFaceLdsBytes = 32 * 1024;
Shape shape_of(const adg_problem* probs, int32_t n, const adg_options* opt, int64_t n_rec) {
  const int kern = kernel_of(probs, opt);
  Shape s{std::max(1, lane_elems_of(probs, n, opt)), kern == ADG_KERNEL_FUSED ? std::max(1, fused_steps_of(opt)) : 1};
  if (kern != ADG_KERNEL_FUSED) return s;
  const int64_t elems = total_elems(probs, n);
  uint32_t degree = 0;
  for (int32_t i = 0; i < n; ++i) degree = std::max(degree, probs[i].degree);
  const bool one_launch = opt && (opt->flags & ADG_OPT_ONE_LAUNCH);
  bool all_lin = true, gen = false, all_gen = true, odd = false;
  int64_t least = (int64_t)1 << 62;
  for (int32_t i = 0; i < n; ++i) {
    const int f = form_of(probs[i], kern, n_rec);
    all_lin = all_lin && f == FORM_LIN;
    gen = gen || f == FORM_GEN;
    all_gen = all_gen && f == FORM_GEN;
  }
  if (one_launch)
    s.elems = 2;
  else if (!opt || opt->lane_elems == 0) {
    const bool ldg = is_ldg(probs);
    const int64_t two = all_lin || ldg ? (int64_t)1 << 16 : (gen ? 0 : (int64_t)1 << 17);
    const int64_t four = all_lin || ldg ? (int64_t)1 << 19 : (int64_t)1 << 18;
    s.elems = elems >= four ? 4 : (elems >= two ? 2 : 1);
  }
  for (int32_t i = 0; i < n; ++i)
    if (async_of(probs[i]))
      odd = odd || probs[i].pe_size % 2, least = std::min(least, probs[i].pe_size);
  // The general stage form and local DG can find a lane's PE face in any element;
  // one element per lane would leave 44 of 64 lanes to five stages and two steps, 31
  // to Heun and eight.  Odd PEs (25), us per step with one and two: 4.7e6 elements,
  // p = 4, a < 0, LSRK4 98.7, 75.2, SSP-RK3 71.7, 54.2; Burgers, RK4 82.5, 70.7; local
  // DG, p = 2, 2^22, Heun 41.2, 26.8, SSP-RK3 55.0, 36.6; 2^18 3.76, 3.03 and 5.08, 4.43.
  s.any_face = all_gen && odd && !one_launch && s.elems >= 2 && least >= 2;
  if (s.any_face)
    s.elems = 2;
  else
    for (int32_t i = 0; i < n; ++i)
      if (async_of(probs[i]))
        while (probs[i].pe_size % s.elems) s.elems >>= 1;
  s.halve8 = elems >= (int64_t)1 << 18;
  s.halve4 = s.halve8 && (elems < (int64_t)1 << 21 || is_ldg(probs) || (!all_lin && degree >= 2));
  if (!one_launch) {
    s.elems1 = std::min(s.elems, 2);
    if (!opt || opt->lane_elems == 0 || opt->fused_steps == 0) s.elems2 = s.elems1;
  }
  if ((opt && opt->fused_steps != 0) || one_launch) return s;
  const int most_halo = is_ldg(probs) ? (elems <= (int64_t)1 << 16 ? 24 : 16) / s.elems
                        : gen ? (elems <= (int64_t)1 << 16 ? 21 : 8)
                        : all_lin ? (elems <= (int64_t)1 << 18 ? 40 : 20) : (elems <= (int64_t)1 << 17 ? 40 : 16);
  auto fits = [&](int K) {
    if (fused_halo((int)probs[0].rk, s.elems, K) > most_halo) return false;
    for (int32_t i = 0; i < n; ++i)
      if (8 * kWavesPerBlock * lds_of(probs[i], s.elems, K) > kFaceLdsBytes) return false;
    return true;
  };
  int K = kMaxSteps;
  while (K > 2 && !fits(K)) K >>= 1;
  s.kmax = K;
  return s;
}

// Steps of the next launch with `left` steps to go.
int steps_within(int kmax, int64_t left) {
  int K = kmax;
  while (K > left) K >>= 1;
  return K;
}

// Whether the last m steps of a call (all of them, up to a batch), from the
// caller's buffer (in_place) or the other one, halve their first launch: an odd
// number of launches ends in the other buffer and costs a copy of the state.  One
// more launch is the cheaper one from 2^18 elements on, for eight steps always,
// for four unless they are bound by HBM, as the copy is (the linear form and p = 1
// from 2^21 on).  us per step with the copy and halved, calls of four and of
// eight steps, PE 256:
//   central, RK4, p = 3   2^17 3.58, 3.56 and 2.31, 2.32; 2^18 5.82, 4.49 and 4.07,
//                         3.65; 2^20 10.9, 10.5 and 9.1, 8.0; 2^22 36.8, 33.4 and
//                         31.0, 24.8
//   upwind, RK4, p = 3    2^18 4.62, 3.74 and 3.02, 2.53; 2^20 8.96, 8.49 and 5.92,
//                         6.01; 2^22 29.4, 30.1 and 19.0, 17.1
//   upwind, Heun, p = 1   2^17 2.29, 2.54; 2^20 6.64, 5.35 and 4.05, 3.37; 2^22 14.0,
//                         14.2 and 9.5, 8.8; 2^23 29.5, 33.1 and 18.9, 17.6
//   local DG, Heun, p = 2 2^18 4.40, 3.89 and 2.98, 2.68; 2^22 26.3, 24.1 and 20.9, 18.9
bool halves_first(const Shape& s, int32_t m, bool in_place) {
  const int K = steps_within(s.kmax, m);
  if (!(K == 8 ? s.halve8 : (K == 4 && s.halve4))) return false;
  int launches = 0;
  for (int32_t i = 0; i < m; ++launches) i += steps_within(s.kmax, m - i);
  return (launches % 2 == 1) == in_place;
}

// Lists of the fused reverse sweep: with the forward stages, and (advection
// only) without them, for dJ/du0 alone.
enum AdjList : int { ADJ_FWD = 0, ADJ_LINEAR = 1 };

// Its elements per lane R (at most the PE size) and the steps per launch K of
// the list, like the forward kernels'.  With dJ/da the two are equal, so that a
// wave owns whole tiles of the partial sums; four of either would take two
// thirds of the registers for the forward stages alone.  options.fused_steps is
// the forward launches' alone: one reverse step per launch where it is 1 took
// 71.6 us per step of a recorded run and its adjoint at 2^20 against 61.1.
// Measured, us per step of a reverse sweep of 16, PE 256 (R and K in brackets):
//   with dJ/da    p = 3, RK4, 2^20 elements (1,1) 33.1, (2,2) 23.5
//   dJ/du0 alone  p = 3, RK4 2^12 (1,4) 2.35, (2,2) 3.61, (2,8) 2.35; 2^16 2.80,
//                 3.89, 2.64; 2^18 (2,2) 6.27, (2,4) 5.04, (2,8) 5.04, (4,8) 5.26;
//                 2^20 (2,4) 12.4, (2,8) 14.9, (4,8) 12.7; 2^22 (2,4) 42.6, (4,8)
//                 42.0; central, SSP-RK3, p = 2 2^20 (2,4) 8.9, (2,8) 9.0, (4,8) 7.7;
//                 2^20, LSRK3 p = 4 (2,4) 12.8, (4,8) 11.1; LSRK4 p = 2 (2,4) 14.1,
//                 (4,4) 12.5, p = 3 (2,4) 17.0, (4,4) 18.9, p = 4 (2,2) 22.3, (2,4) 21.3
//   Burgers       SSP-RK3, p = 2 2^12 (1,4) 4.62, (2,4) 4.86, (2,8) 4.32; 2^16 5.29,
//                 5.20, 4.80; 2^18 10.3, 9.75, 9.88; 2^20 (2,2) 27.7, (2,4) 24.8,
//                 (2,8) 26.5; RK4, p = 3 2^16 (1,4) 7.39, (2,4) 6.55, (2,8) 7.32
Shape adj_shape_of(const adg_problem* probs, int32_t n, const adg_options* opt, int list) {
  const bool nl = probs[0].equation == ADG_EQ_BURGERS, speed = list == ADJ_FWD && !nl;
  const int rk = (int)probs[0].rk, lanes = opt ? (int)opt->lane_elems : 0;
  const int64_t elems = total_elems(probs, n);
  Shape s{2, 2};
  int work = 0;  // the most nodes times stages, which the registers go with
  for (int32_t i = 0; i < n; ++i) work = std::max(work, ((int)probs[i].degree + 1) * rk_stages(rk));
  s.elems = speed ? 2 : lanes != 0 ? lanes : (elems >= (int64_t)1 << 19 && work <= 15 ? 4 : 2);
  if (list == ADJ_FWD) s.elems = std::min(s.elems, 2);
  for (int32_t i = 0; i < n; ++i)
    if (async_of(probs[i]))
      while (probs[i].pe_size < s.elems) s.elems >>= 1;
  if (speed) {
    s.kmax = s.elems;
    return s;
  }
  const bool small = elems <= (int64_t)1 << 17;
  const int most_halo = nl ? (small ? 13 : 10) : (small ? 20 : 12);
  const int most_lds = small && list == ADJ_LINEAR ? 48 * 1024 : kFaceLdsBytes;
  auto fits = [&](int K) {
    if (adj_halo(rk, nl, s.elems, K) > most_halo) return false;
    for (int32_t i = 0; i < n; ++i) {
      const int faces = async_of(probs[i]) ? fused_faces(s.elems, probs[i].pe_size) : 0;
      if (8 * kWavesPerBlock * adj_lds_words(rk_stages(rk), s.elems, K, faces, list == ADJ_FWD, false) > most_lds)
        return false;
    }
    return true;
  };
  s.kmax = kMaxSteps;
  while (s.kmax > 1 && !fits(s.kmax)) s.kmax >>= 1;
  return s;
}

Layout make_layout(const adg_problem* probs, int32_t n, const adg_options* opt, int64_t n_rec) {
  Layout L{};
  const int S = rk_stages((int)probs[0].rk);
  const int kern = kernel_of(probs, opt);
  L.shape = shape_of(probs, n, opt, n_rec);
  // room as without ADG_OPT_ONE_LAUNCH (whose own shape may be another), so
  // that the workspace does not depend on it
  adg_options plain = opt ? *opt : adg_options{};
  plain.flags &= ~ADG_OPT_ONE_LAUNCH;
  const Shape rs = shape_of(probs, n, &plain, n_rec);
  L.depth_steps = std::max({2, L.shape.kmax, rs.kmax});
  std::set<LinKey> tables;
  const bool nl = probs[0].equation == ADG_EQ_BURGERS;
  int TA[2];
  for (int list = 0; list < 2; ++list) {
    L.adj[list] = adj_shape_of(probs, n, opt, list);
    TA[list] = adj_tile_elems((int)probs[0].rk, nl, L.adj[list].elems, L.adj[list].kmax);
  }
  int64_t nwf[kLists] = {}, room[kLists] = {}, nws = 0, nwa[2] = {0, 0}, tot = 0, ring = 0;
  const bool split = pe_split_of(probs, n, opt);
  for (int32_t i = 0; i < n; ++i) {
    const adg_problem& p = probs[i];
    const int form = form_of(p, kern, n_rec);
    auto tiles = [&](int T) { return (p.n_elem + T - 1) / T; };
    for (int li = 0; li < kLists; ++li) {
      const int K = 1 << li;
      const int64_t t = K <= L.shape.kmax ? tiles(tile_of(p, form, L.shape, K)) : 0;
      nwf[li] += t;
      room[li] += K <= rs.kmax ? std::max(t, tiles(tile_of(p, form, rs, K))) : t;
    }
    if (form == FORM_LIN && tables.insert(lin_key(p)).second) L.lin_doubles += lin_tab_size((int)p.degree + 1, S);
    for (int list = 0; list < 2; ++list) nwa[list] += tiles(TA[list]);
    L.n_parts += tiles(adj_part_elems((int)p.rk));
    nws += (p.n_elem + kBlock - 1) / kBlock;
    tot += ld_of(p) * (p.degree + 1);
    if (split && async_of(p))  // room for the window items of a PE-face split
      for (int K = 1; K <= 2; ++K) {
        const int64_t fw = fused_windows_per_wave((int)p.rk, K);
        room[list_of(K)] += (p.n_elem / p.pe_size + fw - 1) / fw;
      }
    if (async_of(p)) {
      // local DG keeps a second ring of the same shape for u-hat
      ring += (is_ldg(probs) ? 2 : 1) * (p.n_elem / p.pe_size) * S * depth_of(p, n_rec, L.depth_steps);
    }
  }
  for (int li = 0; li < kLists; ++li) {
    L.n_work_f[li] = (int32_t)nwf[li];
    L.at_f[li + 1] = L.at_f[li] + (int32_t)room[li];
  }
  L.n_work_s = (int32_t)nws;
  L.n_work_a[ADJ_FWD] = n_rec > 0 ? (int32_t)nwa[ADJ_FWD] : 0;
  L.n_work_a[ADJ_LINEAR] = n_rec > 0 && probs[0].equation == ADG_EQ_ADVECTION ? (int32_t)nwa[ADJ_LINEAR] : 0;
  L.total_doubles = tot;
  L.ring_doubles = ring;
  int64_t off = 0;
  auto take = [&](int64_t bytes) { const int64_t o = off; off = align_up(off + bytes, kAlign); return o; };
  L.probs = take((int64_t)sizeof(DevProblem) * n);
  L.lin = take(8 * L.lin_doubles);
  L.work_f = take((int64_t)sizeof(WorkItem) * L.at_f[kLists]);
  L.work_s = take((int64_t)sizeof(WorkItem) * nws);
  L.first_s = take((int64_t)sizeof(int32_t) * (n + 1));
  L.ctr = take(8 * sizeof(int64_t));
  L.ring = take(8 * std::max<int64_t>(ring, 1));
  const bool rec = n_rec > 0;
  L.state2 = kern == ADG_KERNEL_FUSED ? take(8 * tot) : -1;
  L.y0 = kern == ADG_KERNEL_STAGE ? take(8 * tot) : -1;
  L.y1 = kern == ADG_KERNEL_STAGE ? take(8 * tot) : -1;
  L.acc = kern == ADG_KERNEL_STAGE ? take(8 * tot) : -1;
  L.qbuf = (is_ldg(probs) && kern == ADG_KERNEL_STAGE) ? take(8 * tot) : -1;  // the fused kernel keeps q on chip
  L.part = take(3 * 8 * nws);
  L.stats_out = take(3 * 8 * (int64_t)n);
  L.groups = take(4 * (2 * (int64_t)n + 1));
  L.gstats = take(4 * 8 * (int64_t)n);
  L.n_rec = n_rec;
  L.ckpt_every = (opt && opt->ckpt_every > 0) ? opt->ckpt_every : 64;
  L.n_ckpt = rec ? (n_rec + L.ckpt_every - 1) / L.ckpt_every : 0;
  L.ckpt = L.useg = L.ybuf = L.lam = L.q = L.adjring = L.cpart = L.work_a[0] = L.work_a[1] = -1;
  if (rec) {
    // stage kernels recompute a segment into seg slots; the fused adjoint
    // reads the segment's first state from its checkpoint and needs seg - 1
    const int64_t seg = std::min<int64_t>(L.ckpt_every, n_rec);
    L.ckpt = take(8 * tot * L.n_ckpt);
    L.useg = take(8 * tot * (kern == ADG_KERNEL_STAGE ? seg : std::max<int64_t>(seg - 1, 1)));
    L.lam = take(8 * tot * 2);
    L.adjring = take(8 * std::max<int64_t>(ring, 1));
    if (kern == ADG_KERNEL_STAGE) {
      L.ybuf = take(8 * tot * (S - 1));
      L.q = take(8 * tot * (S - 1));
      L.cpart = take(8 * nws);
    } else {
      for (int list = 0; list < 2; ++list)
        if (L.n_work_a[list] > 0) L.work_a[list] = take((int64_t)sizeof(WorkItem) * L.n_work_a[list]);
      L.cpart = take(8 * L.n_parts);
    }
  }
  L.total = off;
  return L;
}

}  // namespace

struct adg_ctx {
  std::vector<adg_problem> probs;
  std::vector<DevProblem> dev;
  adg_options opt{};
  int kernel = ADG_KERNEL_FUSED;
  int rk = 0, phys = 0, S = 0;
  int fused_phys = 0;  // phys of the fused kernel (its launcher takes the a > 0 upwind form per work range)
  hipStream_t stream = nullptr;
  char* ws = nullptr;
  Layout L{};
  int64_t steps = 0;
  // adjoint recording: steps recorded by the last ADG_RUN_RECORD run (0: none)
  int64_t rec_steps = 0;
  // adg_init_scratch: the device whose static scratch array holds the
  // workspace and the generation of that use (-1: caller's workspace)
  int scratch_dev = -1;
  uint64_t scratch_gen = 0;
  // a call was captured into a caller's graph: its replays advance the device's
  // step counter alone, so launches count from that one from then on
  bool device_clock = false;
  // graph cache
  hipGraphExec_t graph = nullptr;
  const double* graph_u = nullptr;
  int graph_steps = 0;

  // fused work lists
  int32_t group[kLists][kFusedRanges + 1] = {};
  int32_t grid[kLists][kFusedRanges] = {};
  int32_t single[kLists][kFusedRanges] = {};
  FaceRange faces[kLists][kFusedRanges] = {};
  int32_t one_launch = 0;  // ADG_OPT_ONE_LAUNCH
  // fused adjoint work list (recording contexts of the fused kernel)
  AdjArgs adj[2] = {};  // per list, but for the steps of a launch

  StepArgs base_args(int64_t work_off, int32_t n_work, int K = 1) const {
    StepArgs a{};
    const int list = list_of(K);
    a.probs = (const DevProblem*)(ws + L.probs);
    a.work = (const WorkItem*)(ws + work_off);
    a.n_work = n_work;
    a.ring = (double*)(ws + L.ring);
    a.ctr = ctr();
    a.clock = StepClock{ctr() + CTR_DONE, nullptr, 0};
    for (int i = 0; i <= kFusedRanges; ++i) a.group[i] = group[list][i];
    for (int i = 0; i < kFusedRanges; ++i) a.grid[i] = grid[list][i];
    for (int i = 0; i < kFusedRanges; ++i) a.single[i] = single[list][i];
    for (int i = 0; i < kFusedRanges; ++i) a.faces[i] = faces[list][i];
    a.lin = (const double*)(ws + L.lin);
    a.elems = L.shape.elems_at(K);
    a.any_face = L.shape.any_face;
    a.steps = K;
    a.halo = fused_halo(rk, a.elems, K);
    a.halo_right = ldg_halo_right(rk, a.elems, K);
    a.one_launch = one_launch;
    a.qbuf = L.qbuf >= 0 ? (double*)(ws + L.qbuf) : nullptr;
    return a;
  }
  StepArgs fused_args(int K = 1) const {
    const int list = list_of(K);
    return base_args(L.work_f + (int64_t)sizeof(WorkItem) * L.at_f[list], L.n_work_f[list], K);
  }
  StepArgs stage_args() const { return base_args(L.work_s, L.n_work_s); }

  AdjArgs adj_args(int list, int K) const {
    AdjArgs a = adj[list];
    a.steps = K;
    return a;
  }
  int64_t* ctr() const { return (int64_t*)(ws + L.ctr); }
  double* state2() const { return (double*)(ws + L.state2); }
};

namespace {

// K fused steps uin -> uout (with K > 1 also the states after the steps before
// the last into umid, umid + total_doubles, ..., if not null).
int launch_fused(const adg_ctx* c, int K, const double* uin, double* uout, double* umid, const StepClock& clock,
                 int32_t step_offset, hipStream_t st) {
  StepArgs a = c->fused_args(K);
  a.umid = umid;
  a.mid_stride = c->L.total_doubles;
  a.clock = clock;
  ADG_HIP(launch_fused_step(c->rk, c->fused_phys, a, uin, uout, step_offset, st));
  return ADG_OK;
}

// One step with the per-stage kernels, in place on U.
int launch_stages(adg_ctx* c, const StepArgs& a, double* U, int32_t step_offset, hipStream_t st) {
  double* Y0 = (double*)(c->ws + c->L.y0);
  double* Y1 = (double*)(c->ws + c->L.y1);
  double* A = (double*)(c->ws + c->L.acc);
  for (int s = 0; s < c->S; ++s) {
    const double* yin = s == 0 ? U : ((s & 1) ? Y0 : Y1);
    double* yout = (s & 1) ? Y1 : Y0;
    if (c->phys == PHYS_BURGERS_LDG) ADG_HIP(launch_ldg_q(c->rk, s, a, yin, step_offset, st));
    ADG_HIP(launch_stage(c->rk, c->phys, s, a, yin, yout, U, A, step_offset, st));
  }
  return ADG_OK;
}

int next_steps(const adg_ctx* c, int64_t left) { return steps_within(c->L.shape.kmax, left); }

// m steps, as many per launch as the kernel allows, the step counter included.
// The state goes from *cur through `dst(i)` for each launch's result after i
// steps of the batch (mid(i): states within a launch, or null).  n0: index of
// the first step, or -1 to count from the device's counter.
// halve: the first launch takes half of its steps and a second one the others.
template <class Dst, class Mid>
int enqueue_batch(adg_ctx* c, double* cur, int32_t m, int64_t n0, hipStream_t st, Dst dst, Mid mid,
                  bool halve = false) {
  int64_t* ctr = c->ctr();
  if (c->kernel != ADG_KERNEL_FUSED) {
    const StepArgs a = c->stage_args();
    for (int32_t i = 0; i < m; ++i)
      if (int rc = launch_stages(c, a, cur, i, st)) return rc;
    ADG_HIP(launch_advance(ctr, m, st));
    return ADG_OK;
  }
  const int K0 = next_steps(c, m);
  for (int32_t i = 0; i < m;) {
    const int K = halve && i < K0 ? K0 / 2 : next_steps(c, m - i);
    const bool first = i == 0, last = i + K >= m;
    StepClock clock{ctr + (n0 >= 0 ? CTR_ZERO : (first ? CTR_DONE : CTR_BATCH)), nullptr, 0};
    if (n0 >= 0) {
      if (last) clock = StepClock{clock.from, ctr + CTR_DONE, n0 + m};
    } else if (!(first && last)) {  // the word read is never the word written
      if (first) clock.to = ctr + CTR_BATCH;
      if (last) clock = StepClock{clock.from, ctr + CTR_DONE, m};
    }
    double* out = dst(i + K);
    if (int rc = launch_fused(c, K, cur, out, K > 1 ? mid(i + 1) : nullptr, clock, (int32_t)((n0 >= 0 ? n0 : 0) + i), st))
      return rc;
    if (n0 < 0 && first && last) ADG_HIP(launch_advance(ctr, m, st));
    cur = out;
    i += K;
  }
  return ADG_OK;
}

// The same between *cur and *other, which are swapped with every launch.
int enqueue_batch(adg_ctx* c, double** cur, double** other, int32_t m, int64_t n0, hipStream_t st, bool halve = false) {
  return enqueue_batch(
      c, *cur, m, n0, st,
      [&](int32_t) {
        std::swap(*cur, *other);
        return *cur;
      },
      [](int32_t) { return (double*)nullptr; }, halve);
}

// Whether the context's stream is being captured by the caller (then, and from
// then on, steps count from the device's counter).
void note_capture(adg_ctx* c) {
  if (c->device_clock) return;
  hipStreamCaptureStatus s = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(c->stream, &s) != hipSuccess) {
    (void)hipGetLastError();
    c->device_clock = true;
  } else if (s != hipStreamCaptureStatusNone) {
    c->device_clock = true;
  }
}

int reset_device(adg_ctx* c) {
  ADG_HIP(launch_zero(c->ws + c->L.ctr, 8 * sizeof(int64_t), c->stream));
  ADG_HIP(launch_zero(c->ws + c->L.ring, 8 * std::max<int64_t>(c->L.ring_doubles, 1), c->stream));
  c->steps = 0;
  c->rec_steps = 0;
  return ADG_OK;
}

void drop_graph(adg_ctx* c) {
  if (c->graph) (void)hipGraphExecDestroy(c->graph);
  c->graph = nullptr;
  c->graph_u = nullptr;
  c->graph_steps = 0;
}

int build_graph(adg_ctx* c, double* d_u) {
  drop_graph(c);
  hipStream_t cap;
  ADG_HIP(hipStreamCreateWithFlags(&cap, hipStreamNonBlocking));
  hipGraph_t g = nullptr;
  int rc = ADG_OK;
  if (hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal) != hipSuccess) {
    (void)hipStreamDestroy(cap);
    return fail(ADG_E_HIP, "hipStreamBeginCapture failed");
  }
  double* cur = d_u;
  double* other = c->state2();
  rc = enqueue_batch(c, &cur, &other, kGraphSteps, -1, cap);
  const hipError_t e1 = hipStreamEndCapture(cap, &g);
  (void)hipStreamDestroy(cap);
  if (rc != ADG_OK) { if (g) (void)hipGraphDestroy(g); return rc; }
  if (e1 != hipSuccess) return fail(ADG_E_HIP, std::string("hipStreamEndCapture: ") + hipGetErrorString(e1));
  hipGraphExec_t ex = nullptr;
  const hipError_t e2 = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
  (void)hipGraphDestroy(g);
  if (e2 != hipSuccess) return fail(ADG_E_HIP, std::string("hipGraphInstantiate: ") + hipGetErrorString(e2));
  c->graph = ex;
  c->graph_u = d_u;
  c->graph_steps = kGraphSteps;
  return ADG_OK;
}

}  // namespace

// Workspace of adg_init_scratch, for callers that cannot allocate device
// memory: one array per GPU the library runs on, held until the process ends.
// Host code never uses this name as a device address (on the host it is a
// stand-in); its per-device address comes from hipGetSymbolAddress.
// The linear form's tables (1.4 KB at most for a problem of 1024 elements or
// more) and the work lists (longer than two elements per lane make them where odd
// PEs take one) come on top of the documented size, so that what fitted without
// them fits.
constexpr int64_t kScratchBytes = ADG_SCRATCH_BYTES;
constexpr int64_t kScratchTables = 8ll << 20;
static __device__ __align__(256) unsigned char scratch[kScratchBytes + kScratchTables];

namespace {

std::mutex g_scratch_mu;
std::vector<void*> g_scratch_ptr;       // per device: address of `scratch`
std::vector<uint64_t> g_scratch_gen;    // per device: generation of the current use

// Address of the scratch array on the current device (looked up once per
// device) and a new generation number for its next use.
int scratch_acquire(int* dev_out, void** ptr_out, uint64_t* gen_out) {
  int dev = 0;
  ADG_HIP(hipGetDevice(&dev));
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if ((int)g_scratch_ptr.size() <= dev) {
    g_scratch_ptr.resize(dev + 1, nullptr);
    g_scratch_gen.resize(dev + 1, 0);
  }
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p)
      return fail(ADG_E_HIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
    g_scratch_ptr[dev] = p;
  }
  *dev_out = dev;
  *ptr_out = g_scratch_ptr[dev];
  *gen_out = ++g_scratch_gen[dev];
  return ADG_OK;
}

// A context on the scratch array is live until a later adg_init_scratch on
// the same device takes the array over.
int check_live(const adg_ctx* c) {
  if (c->scratch_dev < 0) return ADG_OK;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (c->scratch_gen != g_scratch_gen[c->scratch_dev])
    return fail(ADG_E_STATE, "the scratch workspace was taken over by a later adg_init_scratch");
  return ADG_OK;
}

}  // namespace

extern "C" {

int adg_abi_version(void) { return ADG_ABI_VERSION; }

const char* adg_last_error(void) { return g_err.c_str(); }

#ifndef ADG_SOURCE_HASH
#error "compile with -DADG_SOURCE_HASH=\"<hash of csrc/ and include/>\" (paper_2404_03399_amd/build.py does)"
#endif
const char* adg_build_id(void) { return ADG_SOURCE_HASH; }

int adg_nodes(int32_t degree, double* xi) {
  if (degree < 1 || degree > 4 || !xi) return fail(ADG_E_INVALID, "adg_nodes: degree must be 1..4");
  long double x[kMaxNp];
  gll(degree, x);
  for (int i = 0; i <= degree; ++i) xi[i] = (double)x[i];
  return ADG_OK;
}

int adg_state_layout(const adg_problem* probs, int32_t n_probs, int64_t* offsets, int64_t* lds,
                     int64_t* total_doubles) {
  int rc = validate(probs, n_probs);
  if (rc) return rc;
  int64_t off = 0;
  for (int32_t i = 0; i < n_probs; ++i) {
    if (offsets) offsets[i] = off;
    if (lds) lds[i] = ld_of(probs[i]);
    off += ld_of(probs[i]) * (probs[i].degree + 1);
  }
  if (total_doubles) *total_doubles = off;
  return ADG_OK;
}

int adg_workspace_size(const adg_problem* probs, int32_t n_probs, const adg_options* opt, int64_t n_steps_record,
                       int64_t* bytes_out) {
  int rc = validate(probs, n_probs);
  if (rc) return rc;
  if (!bytes_out) return fail(ADG_E_INVALID, "bytes_out is null");
  if (n_steps_record < 0 || n_steps_record > (1 << 28)) return fail(ADG_E_INVALID, "n_steps_record out of range");
  if (opt && opt->ckpt_every < 0) return fail(ADG_E_INVALID, "ckpt_every < 0");
  const int k = kernel_of(probs, opt);
  if (k != ADG_KERNEL_FUSED && k != ADG_KERNEL_STAGE) return fail(ADG_E_INVALID, "unknown kernel family");
  if (lane_elems_of(probs, n_probs, opt) == 0)
    return fail(ADG_E_INVALID, "lane_elems must be 1, 2 or 4 and not exceed the PE size");
  if (fused_steps_of(opt) == 0) return fail(ADG_E_INVALID, "fused_steps must be 0, 1 or 2");
  if (opt && (opt->flags & ~(ADG_OPT_PE_SPLIT_OFF | ADG_OPT_PE_SPLIT_ON | ADG_OPT_ONE_LAUNCH)))
    return fail(ADG_E_INVALID, "unknown adg_options.flags bits");
  if (opt && (opt->flags & ADG_OPT_PE_SPLIT_OFF) && (opt->flags & ADG_OPT_PE_SPLIT_ON))
    return fail(ADG_E_INVALID, "ADG_OPT_PE_SPLIT_OFF and ADG_OPT_PE_SPLIT_ON together");
  if (opt && (opt->flags & ADG_OPT_ONE_LAUNCH)) {
    if ((opt->flags & ADG_OPT_PE_SPLIT_ON) || k != ADG_KERNEL_FUSED || lane_elems_of(probs, n_probs, opt) != 2)
      return fail(ADG_E_INVALID, "ADG_OPT_ONE_LAUNCH needs the fused kernel, two elements per lane and no PE-face split");
    if (is_ldg(probs)) return fail(ADG_E_UNSUPPORTED, "ADG_OPT_ONE_LAUNCH: the local DG kernel launches per range");
  }
  if (is_ldg(probs) && n_steps_record > 0)
    return fail(ADG_E_UNSUPPORTED, "no adjoint for viscous Burgers (local DG)");
  *bytes_out = make_layout(probs, n_probs, opt, n_steps_record).total;
  return ADG_OK;
}

int adg_launch_shape(const adg_problem* probs, int32_t n_probs, const adg_options* opt, int64_t n_steps_record,
                     int64_t n_steps, int32_t* lane_elems, int32_t* steps_per_launch) {
  int64_t need = 0;
  const int rc = adg_workspace_size(probs, n_probs, opt, n_steps_record, &need);
  if (rc) return rc;
  if (!lane_elems || !steps_per_launch || n_steps < 1) return fail(ADG_E_INVALID, "adg_launch_shape: bad arguments");
  if (kernel_of(probs, opt) != ADG_KERNEL_FUSED) {
    *lane_elems = *steps_per_launch = 1;
    return ADG_OK;
  }
  const Shape s = shape_of(probs, n_probs, opt, n_steps_record);
  int K = steps_within(s.kmax, n_steps);
  if (n_steps <= kGraphSteps && halves_first(s, (int32_t)n_steps, true)) K /= 2;
  *lane_elems = s.elems_at(K);
  *steps_per_launch = K;
  return ADG_OK;
}

int adg_init(adg_ctx** out, const adg_problem* probs, int32_t n_probs, const adg_options* opt, int64_t n_steps_record,
             void* d_workspace, int64_t workspace_bytes, void* hip_stream) {
  if (!out) return fail(ADG_E_INVALID, "out is null");
  *out = nullptr;
  int64_t need = 0;
  int rc = adg_workspace_size(probs, n_probs, opt, n_steps_record, &need);
  if (rc) return rc;
  if (!d_workspace || workspace_bytes < need) return fail(ADG_E_WORKSPACE, "workspace too small: need " + std::to_string(need));
  if (((uintptr_t)d_workspace) % kAlign) return fail(ADG_E_WORKSPACE, "workspace must be 256-byte aligned");

  adg_ctx* c = new adg_ctx();
  c->probs.assign(probs, probs + n_probs);
  if (opt) c->opt = *opt;
  c->kernel = kernel_of(probs, opt);
  c->rk = (int)probs[0].rk;
  c->phys = phys_of(probs[0]);
  c->fused_phys = c->phys;
  c->S = rk_stages(c->rk);
  c->stream = (hipStream_t)hip_stream;
  c->ws = (char*)d_workspace;
  c->L = make_layout(probs, n_probs, opt, n_steps_record);

  // descriptors
  c->dev.resize(n_probs);
  int64_t uoff = 0, roff = 0, poff = 0;
  std::vector<double> lin_tabs;
  std::map<LinKey, int64_t> lin_at;
  for (int32_t i = 0; i < n_probs; ++i) {
    const adg_problem& p = probs[i];
    DevProblem& d = c->dev[i];
    std::memset(&d, 0, sizeof(d));
    d.n_elem = p.n_elem;
    d.pe_size = p.pe_size;
    d.n_pe = p.n_elem / p.pe_size;
    d.ld = ld_of(p);
    d.u_off = uoff;
    uoff += d.ld * (p.degree + 1);
    d.np = (int)p.degree + 1;
    d.q = q_of(p);
    d.n_delays = (int)p.n_delays;
    d.depth = (int32_t)depth_of(p, n_steps_record, c->L.depth_steps);
    d.per_stage = p.delay_granularity == ADG_DELAY_PER_STAGE;
    d.caa = p.delay_granularity == ADG_DELAY_CAA;
    d.scheme = (int)p.scheme;
    d.async_faces = async_of(p) ? 1 : 0;
    d.pe_div = make_fast_div((uint32_t)p.pe_size);
    for (int64_t v : {(int64_t)0, p.pe_size - 1, p.pe_size, p.n_elem - 1, p.n_elem, p.n_elem / 2 + 1}) {
      if (v < 0) continue;
      if ((int64_t)fast_div((uint32_t)v, d.pe_div) != v / p.pe_size) {
        delete c;
        return fail(ADG_E_INVALID, "internal: division by pe_size failed self-check");
      }
    }
    d.part_off = poff;
    poff += (p.n_elem + adj_part_elems((int)p.rk) - 1) / adj_part_elems((int)p.rk);
    d.ring_off = roff;
    d.ring_stride = d.n_pe * c->S;
    if (d.async_faces) {
      const int64_t one_ring = d.n_pe * c->S * (int64_t)d.depth;
      d.ring2_off = roff + one_ring;
      roff += (is_ldg(probs) ? 2 : 1) * one_ring;
    }
    d.seed_mix = splitmix64(p.seed);
    for (int k = 0; k + 1 < kMaxL; ++k) d.thr[k] = k + 1 < d.n_delays ? p.delay_threshold[k] : ~0ull;
    const double dx = p.length / (double)p.n_elem;
    d.two_over_dx = 2.0 / dx;
    d.half_dx = 0.5 * dx;
    d.speed = p.equation == ADG_EQ_ADVECTION ? p.speed : 1.0;
    d.nu = p.viscosity;
    d.dt = p.dt;
    element_operators((int)p.degree, &d);
    {
      // Kd folds the flux constant: a (advection), 1/2 (Burgers: g = u^2), 1
      // (local DG: g = u^2/2 - nu q is formed in the kernel)
      const double fac = p.equation == ADG_EQ_ADVECTION ? p.speed
                         : (p.equation == ADG_EQ_BURGERS ? 0.5 : 1.0);
      for (int i = 0; i < kMaxNp * kMaxNp; ++i) d.Kd[i] = d.two_over_dx * fac * d.D[i];
      for (int i = 0; i < kMaxNp; ++i) {
        d.Kl[i] = d.two_over_dx * d.lift_l[i];
        d.Kr[i] = d.two_over_dx * d.lift_r[i];
      }
      for (int i = 0; i < kMaxNp * kMaxNp; ++i) d.Kdu[i] = d.Kd[i];
      const int pn = (int)p.degree;
      for (int i = 0; i <= pn; ++i) d.Kdu[i * kMaxNp + pn] -= d.Kr[i] * p.speed;
    }
    d.depth_div = make_fast_div((uint32_t)d.depth);
    d.lin_off = -1;
    if (lin_of(p, c->kernel, n_steps_record)) {
      const auto it = lin_at.emplace(lin_key(p), (int64_t)lin_tabs.size());
      if (it.second) {
        lin_tabs.resize(lin_tabs.size() + lin_tab_size(d.np, c->S));
        lin_table(d, c->rk, lin_tabs.data() + it.first->second);
      }
      d.lin_off = it.first->second;
    }
    for (int k = 0; k < d.n_delays; ++k)
      for (int j = 0; j < d.q; ++j) d.atc[k][j] = at_coefficient(d.q, k, j);
  }
  if (roff != c->L.ring_doubles || (int64_t)lin_tabs.size() != c->L.lin_doubles) {
    delete c;
    return fail(ADG_E_INVALID, "internal: ring or table layout does not match the workspace layout");
  }
  // work lists: heaviest (highest degree) problems first
  std::vector<int32_t> order(n_probs);
  for (int32_t i = 0; i < n_probs; ++i) order[i] = i;
  std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return probs[a].degree > probs[b].degree; });
  std::vector<WorkItem> wf_all(c->L.at_f[kLists]), ws_;
  std::vector<int32_t> first(n_probs + 1, 0);
  c->one_launch = (opt && (opt->flags & ADG_OPT_ONE_LAUNCH)) ? 1 : 0;
  for (int list = 0; list < kLists && 1 << list <= c->L.shape.kmax; ++list) {
    const int K = 1 << list;
    std::vector<WorkItem> wf;
    wf.reserve(c->L.n_work_f[list]);
    // ranges per degree, np = 5, 4, 3, 2 (order is sorted by degree,
    // descending), each split by form
    for (int gi = 0; gi < kFusedRanges; ++gi) {
      const int np = 5 - gi / kForms, form = gi % kForms;
      const int32_t b = c->group[list][gi] = (int32_t)wf.size();
      FaceRange& fr = c->faces[list][gi];
      int n_in = 0;
      for (int32_t i : order) {
        const adg_problem& p = probs[i];
        if ((int)p.degree + 1 != np || form_of(p, c->kernel, n_steps_record) != form) continue;
        ++n_in;
        const int T = tile_of(p, form, c->L.shape, K);
        for (int64_t t = 0; t < (p.n_elem + T - 1) / T; ++t) wf.push_back(WorkItem{i, (int32_t)t});
        if (async_of(p)) {
          fr.n_faces = std::max(fr.n_faces, fused_faces(c->L.shape.elems_at(K), p.pe_size));
          fr.lds_words = std::max(fr.lds_words, lds_of(p, c->L.shape.elems_at(K), K));
        }
      }
      c->grid[list][gi] = fused_grid((int32_t)wf.size() - b);
      // one problem, whose tiles are listed in order: the kernel forms its
      // items without loading the list
      c->single[list][gi] = n_in == 1 ? wf[b].prob : -1;
    }
    c->group[list][kFusedRanges] = (int32_t)wf.size();
    if ((int64_t)wf.size() != c->L.n_work_f[list] || (int64_t)wf.size() > c->L.at_f[list + 1] - c->L.at_f[list]) {
      delete c;
      return fail(ADG_E_INVALID, "internal: fused work list does not match the workspace layout");
    }
    std::copy(wf.begin(), wf.end(), wf_all.begin() + c->L.at_f[list]);
  }
  for (int32_t i = 0; i < n_probs; ++i) {  // stage/stats list in problem order (contiguous per problem)
    first[i] = (int32_t)ws_.size();
    const int64_t nt = (probs[i].n_elem + kBlock - 1) / kBlock;
    for (int64_t t = 0; t < nt; ++t) ws_.push_back(WorkItem{i, (int32_t)t});
  }
  first[n_probs] = (int32_t)ws_.size();
  // fused reverse sweep: ranges per degree, upwind with a > 0 first
  std::vector<WorkItem> work_a[2];
  for (int list = 0; list < 2; ++list) {
    if (c->L.work_a[list] < 0) continue;
    const Shape& sh = c->L.adj[list];
    const bool nl = probs[0].equation == ADG_EQ_BURGERS;
    const int T = adj_tile_elems(c->rk, nl, sh.elems, sh.kmax);
    std::vector<WorkItem>& wl = work_a[list];
    AdjArgs& a = c->adj[list];
    a.probs = (const DevProblem*)(c->ws + c->L.probs);
    a.work = (const WorkItem*)(c->ws + c->L.work_a[list]);
    a.elems = sh.elems;
    a.halo = adj_halo(c->rk, nl, sh.elems, sh.kmax);
    for (int gi = 0; gi < kAdjRanges; ++gi) {
      a.group[gi] = (int32_t)wl.size();
      a.single[gi] = -1;
      int n_in = 0;
      FaceRange& fr = a.faces[gi];
      for (int32_t i : order) {
        const adg_problem& p = probs[i];
        const bool pos = phys_of(p) == PHYS_ADV_UPWIND && p.speed > 0.0;
        if ((int)p.degree + 1 != 5 - gi / kAdjForms || (pos ? 0 : 1) != gi % kAdjForms) continue;
        for (int64_t t = 0; t < (p.n_elem + T - 1) / T; ++t) wl.push_back(WorkItem{i, (int32_t)t});
        a.single[gi] = n_in++ == 0 ? i : -1;
        if (async_of(p)) fr.n_faces = std::max(fr.n_faces, fused_faces(sh.elems, p.pe_size));
      }
      fr.lds_words = adj_lds_words(c->S, sh.elems, sh.kmax, fr.n_faces, list == ADJ_FWD, list == ADJ_FWD && !nl);
      a.grid[gi] = fused_grid((int32_t)wl.size() - a.group[gi]);
    }
    a.group[kAdjRanges] = (int32_t)wl.size();
    if ((int64_t)wl.size() != c->L.n_work_a[list]) {
      delete c;
      return fail(ADG_E_INVALID, "internal: adjoint work list does not match the workspace layout");
    }
  }

  auto up = [&](int64_t off, const void* src, int64_t bytes) -> int {
    ADG_HIP(hipMemcpyAsync(c->ws + off, src, bytes, hipMemcpyHostToDevice, c->stream));
    return ADG_OK;
  };
  if ((rc = up(c->L.probs, c->dev.data(), (int64_t)sizeof(DevProblem) * n_probs)) ||
      (c->L.lin_doubles > 0 && (rc = up(c->L.lin, lin_tabs.data(), 8 * c->L.lin_doubles))) ||
      (rc = up(c->L.work_f, wf_all.data(), (int64_t)sizeof(WorkItem) * wf_all.size())) ||
      (rc = up(c->L.work_s, ws_.data(), (int64_t)sizeof(WorkItem) * ws_.size())) ||
      (rc = up(c->L.first_s, first.data(), (int64_t)sizeof(int32_t) * first.size())) ||
      (c->L.work_a[0] >= 0 &&
       (rc = up(c->L.work_a[0], work_a[0].data(), (int64_t)sizeof(WorkItem) * work_a[0].size()))) ||
      (c->L.work_a[1] >= 0 &&
       (rc = up(c->L.work_a[1], work_a[1].data(), (int64_t)sizeof(WorkItem) * work_a[1].size()))) ||
      (rc = reset_device(c))) {
    delete c;
    return rc;
  }
  // host data above must stay valid until the copies ran
  if (hipStreamSynchronize(c->stream) != hipSuccess) {
    delete c;
    return fail(ADG_E_HIP, "stream synchronisation after upload failed");
  }
  *out = c;
  return ADG_OK;
}

int adg_init_scratch(adg_ctx** out, const adg_problem* probs, int32_t n_probs, const adg_options* opt,
                     void* hip_stream) {
  if (!out) return fail(ADG_E_INVALID, "out is null");
  *out = nullptr;
  int64_t need = 0;
  int rc = adg_workspace_size(probs, n_probs, opt, 0, &need);
  if (rc) return rc;
  // where the library's choice of steps per launch (longer rings and lists)
  // does not fit, two steps
  auto beside_tables = [&](const adg_options* o) {
    const Layout L = make_layout(probs, n_probs, o, 0);
    return L.total - align_up(8 * L.lin_doubles, kAlign) -
           align_up((int64_t)sizeof(WorkItem) * L.at_f[kLists], kAlign);
  };
  adg_options two = opt ? *opt : adg_options{};
  if (two.fused_steps == 0) two.fused_steps = 2;
  if (beside_tables(opt) > kScratchBytes) opt = &two;
  need = make_layout(probs, n_probs, opt, 0).total;
  if (beside_tables(opt) > kScratchBytes || need - beside_tables(opt) > kScratchTables)
    return fail(ADG_E_WORKSPACE, "adg_init_scratch: these problems need " + std::to_string(need) +
                                     " bytes of workspace; the static scratch array holds " +
                                     std::to_string(kScratchBytes));
  int dev = 0;
  void* ws = nullptr;
  uint64_t gen = 0;
  if ((rc = scratch_acquire(&dev, &ws, &gen))) return rc;
  if ((rc = adg_init(out, probs, n_probs, opt, 0, ws, need, hip_stream))) return rc;
  (*out)->scratch_dev = dev;
  (*out)->scratch_gen = gen;
  return ADG_OK;
}

int adg_reset(adg_ctx* c) {
  if (!c) return fail(ADG_E_INVALID, "null context");
  if (int rc = check_live(c)) return rc;
  note_capture(c);  // replays of a captured reset clear the device's counter alone
  return reset_device(c);
}

int adg_step_count(const adg_ctx* c, int64_t* steps) {
  if (!c || !steps) return fail(ADG_E_INVALID, "null argument");
  *steps = c->steps;
  return ADG_OK;
}

int adg_run(adg_ctx* c, double* d_u, int64_t n_steps, uint32_t flags) {
  if (!c || !d_u) return fail(ADG_E_INVALID, "null argument");
  if (int rc = check_live(c)) return rc;
  if (!state_aligned(d_u)) return fail(ADG_E_INVALID, "d_u must be 16-byte aligned");
  if (n_steps < 0) return fail(ADG_E_INVALID, "n_steps < 0");
  if (c->steps + n_steps >= ((int64_t)1 << 31)) return fail(ADG_E_INVALID, "step index would exceed 2^31 - 1");
  if (flags & ~(ADG_RUN_GRAPH | ADG_RUN_RECORD | ADG_RUN_CHECK_FINITE)) return fail(ADG_E_INVALID, "unknown flags");
  note_capture(c);
  if (flags & ADG_RUN_RECORD) {
    if (c->L.n_rec <= 0) return fail(ADG_E_STATE, "context was created without a recording horizon");
    if (c->steps != 0) return fail(ADG_E_STATE, "ADG_RUN_RECORD must start at step 0 (call adg_reset)");
    if (n_steps > c->L.n_rec) return fail(ADG_E_INVALID, "n_steps exceeds the recording horizon");
    const int64_t C = c->L.ckpt_every, tot = c->L.total_doubles;
    int64_t done = 0;
    int rc;
    if (C == 1 && c->kernel == ADG_KERNEL_FUSED) {
      // every state is kept: each step writes its result straight into the
      // next checkpoint slot (the last one into d_u), no copies; two steps per
      // launch where the context runs two, the launch writing both states
      double* ck = (double*)(c->ws + c->L.ckpt);
      ADG_HIP(hipMemcpyAsync(ck, d_u, 8 * tot, hipMemcpyDeviceToDevice, c->stream));
      // the states before a launch's last lie in consecutive slots
      while (done < n_steps) {
        const int32_t m = (int32_t)std::min<int64_t>(n_steps - done, kGraphSteps);
        if ((rc = enqueue_batch(
                 c, ck + tot * done, m, c->device_clock ? -1 : done, c->stream,
                 [&](int32_t i) { return done + i < n_steps ? ck + tot * (done + i) : d_u; },
                 [&](int32_t i) { return ck + tot * (done + i); })))
          return rc;
        done += m;
      }
      c->steps += n_steps;
      c->rec_steps = n_steps;
      if (flags & ADG_RUN_CHECK_FINITE) return adg_run(c, d_u, 0, ADG_RUN_CHECK_FINITE);
      return ADG_OK;
    }
    for (int64_t k = 0; done < n_steps; ++k) {
      ADG_HIP(hipMemcpyAsync(c->ws + c->L.ckpt + 8 * tot * k, d_u, 8 * tot, hipMemcpyDeviceToDevice, c->stream));
      const int64_t m = std::min<int64_t>(C, n_steps - done);
      if ((rc = adg_run(c, d_u, m, flags & ~(ADG_RUN_RECORD | ADG_RUN_CHECK_FINITE)))) return rc;
      done += m;
    }
    c->rec_steps = n_steps;
    if (flags & ADG_RUN_CHECK_FINITE) return adg_run(c, d_u, 0, ADG_RUN_CHECK_FINITE);
    return ADG_OK;
  }
  int rc;
  if (n_steps == 0 && (flags & ADG_RUN_GRAPH) && (c->graph_u != d_u || !c->graph)) {
    // capture only: the step graph for d_u, replayed by later runs
    if ((rc = build_graph(c, d_u))) return rc;
  }
  if (n_steps > 0) c->rec_steps = 0;  // any further step invalidates a recording
  double* cur = d_u;
  double* other = c->kernel == ADG_KERNEL_FUSED ? c->state2() : nullptr;
  int64_t left = n_steps;
  if ((flags & ADG_RUN_GRAPH) && left >= kGraphSteps) {
    if (c->graph_u != d_u || !c->graph) {
      if ((rc = build_graph(c, d_u))) return rc;
    }
    while (left >= c->graph_steps) {
      ADG_HIP(hipGraphLaunch(c->graph, c->stream));
      left -= c->graph_steps;
    }
  }
  // remaining steps in batches of at most kGraphSteps
  while (left > 0) {
    const int32_t m = (int32_t)std::min<int64_t>(left, kGraphSteps);
    const bool halve = c->kernel == ADG_KERNEL_FUSED && left == m && halves_first(c->L.shape, m, cur == d_u);
    if ((rc = enqueue_batch(c, &cur, &other, m, c->device_clock ? -1 : c->steps + n_steps - left, c->stream, halve)))
      return rc;
    left -= m;
  }
  if (cur != d_u)
    ADG_HIP(hipMemcpyAsync(d_u, cur, 8 * c->L.total_doubles, hipMemcpyDeviceToDevice, c->stream));
  c->steps += n_steps;
  if (flags & ADG_RUN_CHECK_FINITE) {
    int64_t* ctr = c->ctr();
    ADG_HIP(launch_zero(ctr + CTR_FLAG, sizeof(int64_t), c->stream));
    ADG_HIP(launch_check_finite(c->stage_args(), d_u, c->stream));
    int64_t flag = 0;
    ADG_HIP(hipMemcpyAsync(&flag, ctr + CTR_FLAG, sizeof(int64_t), hipMemcpyDeviceToHost, c->stream));
    ADG_HIP(hipStreamSynchronize(c->stream));
    if (flag) return fail(ADG_E_NONFINITE, "state contains NaN or Inf");
  }
  return ADG_OK;
}

int adg_step(adg_ctx* c, double* d_u) { return adg_run(c, d_u, 1, 0); }

namespace {

// Per-problem sums of the per-work-item dJ/da shares, in work-list order.
void sum_speed_parts(const adg_ctx* c, const std::vector<double>& part, const std::vector<WorkItem>& items,
                     double* h_grad_speed) {
  std::vector<double> acc(c->probs.size(), 0.0);
  for (size_t t = 0; t < items.size(); ++t) acc[items[t].prob] += part[t];
  for (size_t i = 0; i < c->probs.size(); ++i)
    h_grad_speed[i] = c->probs[i].equation == ADG_EQ_ADVECTION ? acc[i] : 0.0;
}

// Adjoint with the per-stage kernels: the segment is recomputed stage by
// stage, and every reverse stage is one launch with its RK registers in HBM.
int adjoint_stage(adg_ctx* c, const double* d_cot_uT, double* d_grad_u0, double* h_grad_speed) {
  const Layout& L = c->L;
  const int64_t tot = L.total_doubles, C = L.ckpt_every, N = c->rec_steps;
  const int S = c->S;
  char* ws = c->ws;
  hipStream_t st = c->stream;
  StepArgs sa = c->stage_args();
  sa.ctr = c->ctr() + CTR_ZERO;  // launches below pass absolute step indices
  double* lam = (double*)(ws + L.lam);
  double* lamu = lam + tot;
  double* Q = (double*)(ws + L.q);
  double* adjring = (double*)(ws + L.adjring);
  double* cpart = (double*)(ws + L.cpart);
  double* ring = (double*)(ws + L.ring);
  double* useg = (double*)(ws + L.useg);
  double* ybuf = (double*)(ws + L.ybuf);
  double* abuf = (double*)(ws + L.acc);
  double* y0 = (double*)(ws + L.y0);
  double* y1 = (double*)(ws + L.y1);
  const size_t bytes = 8 * (size_t)tot;

  ADG_HIP(hipMemcpyAsync(lam, d_cot_uT, bytes, hipMemcpyDeviceToDevice, st));
  ADG_HIP(launch_zero(adjring, 8 * std::max<int64_t>(L.ring_doubles, 1), st));
  ADG_HIP(launch_zero(cpart, 8 * (size_t)L.n_work_s, st));

  for (int64_t k = L.n_ckpt - 1; k >= 0; --k) {
    const int64_t n0 = k * C;
    const int64_t len = std::min<int64_t>(C, N - n0);
    if (len <= 0) continue;
    // recompute the segment's states u^{n0}, ..., u^{n0+len-1}
    ADG_HIP(hipMemcpyAsync(useg, ws + L.ckpt + 8 * tot * k, bytes, hipMemcpyDeviceToDevice, st));
    for (int64_t i = 1; i < len; ++i) {
      double* u = useg + tot * i;
      ADG_HIP(hipMemcpyAsync(u, u - tot, bytes, hipMemcpyDeviceToDevice, st));
      for (int s = 0; s < S; ++s) {
        const double* yin = s == 0 ? u : ((s & 1) ? y0 : y1);
        double* yout = (s & 1) ? y1 : y0;
        ADG_HIP(launch_stage(c->rk, c->phys, s, sa, yin, yout, u, abuf, (int32_t)(n0 + i - 1), st));
      }
    }
    for (int64_t i = len - 1; i >= 0; --i) {
      const int32_t n = (int32_t)(n0 + i);
      double* u = useg + tot * i;
      // stage inputs Y_1 = u^n, Y_2..Y_S
      for (int s = 0; s + 1 < S; ++s) {
        const double* yin = s == 0 ? u : ybuf + tot * (s - 1);
        ADG_HIP(launch_stage(c->rk, c->phys, s, sa, yin, ybuf + tot * s, u, abuf, n, st));
      }
      if (S > 1) ADG_HIP(launch_zero(Q, bytes * (S - 1), st));
      ADG_HIP(hipMemcpyAsync(lamu, lam, bytes, hipMemcpyDeviceToDevice, st));
      for (int s = S - 1; s >= 0; --s) {
        const double* Y = s == 0 ? u : ybuf + tot * (s - 1);
        ADG_HIP(launch_adj_stage(c->rk, c->phys, s, sa, Y, lam, lamu, Q, tot, ring, adjring, cpart, n, st));
      }
      std::swap(lam, lamu);
    }
  }
  ADG_HIP(hipMemcpyAsync(d_grad_u0, lam, bytes, hipMemcpyDeviceToDevice, st));
  if (h_grad_speed) {
    std::vector<double> part(L.n_work_s);
    ADG_HIP(hipMemcpyAsync(part.data(), cpart, 8 * part.size(), hipMemcpyDeviceToHost, st));
    ADG_HIP(hipStreamSynchronize(st));
    std::vector<WorkItem> items;  // stage work list: contiguous per problem, in problem order
    items.reserve(L.n_work_s);
    for (size_t i = 0; i < c->probs.size(); ++i) {
      const int64_t nt = (c->probs[i].n_elem + kBlock - 1) / kBlock;
      for (int64_t t = 0; t < nt; ++t) items.push_back(WorkItem{(int32_t)i, (int32_t)t});
    }
    sum_speed_parts(c, part, items, h_grad_speed);
  }
  return ADG_OK;
}

// Adjoint with the fused kernels: each segment is recomputed out of place by
// the fused step kernel (from the checkpointed state and the ring, which keeps
// every level, so the states are bitwise those of the recorded run), then
// reversed, several steps per launch.  Where every state is a checkpoint the
// whole run is one segment with nothing to recompute: as segments of one step,
// launches of one step on the tiles of two took 52.0 us per step (recorded run
// and adjoint, Burgers, p = 3, RK4, 2^20 elements), against 38.5.
int adjoint_fused(adg_ctx* c, const double* d_cot_uT, double* d_grad_u0, double* h_grad_speed) {
  const Layout& L = c->L;
  const int64_t tot = L.total_doubles, C = L.ckpt_every, N = c->rec_steps;
  char* ws = c->ws;
  hipStream_t st = c->stream;
  double* lam = (double*)(ws + L.lam);
  double* lamu = lam + tot;
  double* adjring = (double*)(ws + L.adjring);
  double* cpart = (double*)(ws + L.cpart);
  const double* ring = (const double*)(ws + L.ring);
  double* useg = (double*)(ws + L.useg);
  const size_t bytes = 8 * (size_t)tot;
  int rc;

  ADG_HIP(hipMemcpyAsync(lam, d_cot_uT, bytes, hipMemcpyDeviceToDevice, st));
  ADG_HIP(launch_zero(adjring, 8 * std::max<int64_t>(L.ring_doubles, 1), st));
  ADG_HIP(launch_zero(cpart, 8 * (size_t)std::max<int64_t>(L.n_parts, 1), st));

  // linear advection: the reverse sweep does not depend on the forward states;
  // they are recomputed only for dJ/da
  const bool need_fwd = c->phys == PHYS_BURGERS_LLF || h_grad_speed != nullptr;
  if (!need_fwd) {
    for (int64_t n = N; n > 0;) {
      const int K = steps_within(L.adj[ADJ_LINEAR].kmax, n);
      n -= K;
      ADG_HIP(launch_adj_fused(c->rk, c->phys, c->adj_args(ADJ_LINEAR, K), nullptr, nullptr, 0, lam, lamu, ring,
                               adjring, cpart, (int32_t)n, st));
      std::swap(lam, lamu);
    }
  }
  const bool all = C == 1;
  for (int64_t k = !need_fwd ? -1 : (all ? 0 : L.n_ckpt - 1); k >= 0; --k) {
    const int64_t n0 = k * C;
    const int64_t len = all ? N : std::min<int64_t>(C, N - n0);
    if (len <= 0) continue;
    // u^{n0+i}: the checkpoint itself for i = 0, recomputed into useg[i-1] after
    double* ck = (double*)(ws + L.ckpt) + tot * k;
    auto state = [&](int64_t i) { return all || i == 0 ? ck + tot * i : useg + tot * (i - 1); };
    for (int64_t i = all ? len : 1; i < len;) {
      // several steps per launch, each one's state written
      const int K = next_steps(c, len - i);
      if ((rc = launch_fused(c, K, state(i - 1), state(i + K - 1), K > 1 ? state(i) : nullptr,
                             StepClock{c->ctr() + CTR_ZERO, nullptr, 0}, (int32_t)(n0 + i - 1), st)))
        return rc;
      i += K;
    }
    for (int64_t i = len; i > 0;) {
      const int K = steps_within(L.adj[ADJ_FWD].kmax, i);
      i -= K;
      ADG_HIP(launch_adj_fused(c->rk, c->phys, c->adj_args(ADJ_FWD, K), state(i), state(i + 1), tot, lam, lamu, ring,
                               adjring, cpart, (int32_t)(n0 + i), st));
      std::swap(lam, lamu);
    }
  }
  ADG_HIP(hipMemcpyAsync(d_grad_u0, lam, bytes, hipMemcpyDeviceToDevice, st));
  if (h_grad_speed) {
    std::vector<double> part(L.n_parts);
    ADG_HIP(hipMemcpyAsync(part.data(), cpart, 8 * part.size(), hipMemcpyDeviceToHost, st));
    ADG_HIP(hipStreamSynchronize(st));
    std::vector<WorkItem> items;  // contiguous per problem, in problem order
    items.reserve(L.n_parts);
    const int T = adj_part_elems(c->rk);
    for (size_t i = 0; i < c->probs.size(); ++i)
      for (int64_t t = 0; t < (c->probs[i].n_elem + T - 1) / T; ++t) items.push_back(WorkItem{(int32_t)i, (int32_t)t});
    sum_speed_parts(c, part, items, h_grad_speed);
  }
  return ADG_OK;
}

}  // namespace

int adg_adjoint(adg_ctx* c, const double* d_cot_uT, double* d_grad_u0, double* h_grad_speed) {
  if (!c || !d_cot_uT || !d_grad_u0) return fail(ADG_E_INVALID, "null argument");
  if (int rc = check_live(c)) return rc;
  if (!state_aligned(d_cot_uT) || !state_aligned(d_grad_u0))
    return fail(ADG_E_INVALID, "d_cot_uT and d_grad_u0 must be 16-byte aligned");
  if (c->rec_steps <= 0) return fail(ADG_E_STATE, "adg_adjoint needs a run recorded with ADG_RUN_RECORD");
  return c->kernel == ADG_KERNEL_FUSED ? adjoint_fused(c, d_cot_uT, d_grad_u0, h_grad_speed)
                                       : adjoint_stage(c, d_cot_uT, d_grad_u0, h_grad_speed);
}

int adg_error_stats(adg_ctx* c, const double* d_u, const double* d_ref, double* h_out) {
  if (!c || !d_u || !d_ref || !h_out) return fail(ADG_E_INVALID, "null argument");
  if (!state_aligned(d_u) || !state_aligned(d_ref)) return fail(ADG_E_INVALID, "d_u and d_ref must be 16-byte aligned");
  if (int rc = check_live(c)) return rc;
  const int32_t n = (int32_t)c->probs.size();
  double* part = (double*)(c->ws + c->L.part);
  double* dout = (double*)(c->ws + c->L.stats_out);
  ADG_HIP(launch_stats(c->stage_args(), d_u, d_ref, part, (const int32_t*)(c->ws + c->L.first_s), n, dout, c->stream));
  ADG_HIP(hipMemcpyAsync(h_out, dout, 3 * sizeof(double) * n, hipMemcpyDeviceToHost, c->stream));
  ADG_HIP(hipStreamSynchronize(c->stream));
  return ADG_OK;
}

int adg_ensemble_stats(adg_ctx* c, const double* d_u, const double* d_ref, const int32_t* h_group_of,
                       int32_t n_groups, double* h_out) {
  if (!c || !d_u || !d_ref || !h_group_of || !h_out) return fail(ADG_E_INVALID, "null argument");
  if (!state_aligned(d_u) || !state_aligned(d_ref)) return fail(ADG_E_INVALID, "d_u and d_ref must be 16-byte aligned");
  if (int rc = check_live(c)) return rc;
  const int32_t n = (int32_t)c->probs.size();
  if (n_groups < 1 || n_groups > n) return fail(ADG_E_INVALID, "n_groups must be in 1..n_probs");
  std::vector<int32_t> csr(2 * (size_t)n + 1, 0);  // [gstart (n_groups+1) | members (n)]
  std::vector<int32_t> count(n_groups, 0);
  for (int32_t i = 0; i < n; ++i) {
    if (h_group_of[i] < 0 || h_group_of[i] >= n_groups) return fail(ADG_E_INVALID, "group index out of range");
    ++count[h_group_of[i]];
  }
  int32_t* gstart = csr.data();
  int32_t* members = csr.data() + n + 1;
  for (int32_t g = 0; g < n_groups; ++g) gstart[g + 1] = gstart[g] + count[g];
  std::vector<int32_t> fill(gstart, gstart + n_groups);
  for (int32_t i = 0; i < n; ++i) members[fill[h_group_of[i]]++] = i;
  int32_t* d_csr = (int32_t*)(c->ws + c->L.groups);
  double* part = (double*)(c->ws + c->L.part);
  double* pstats = (double*)(c->ws + c->L.stats_out);
  double* gout = (double*)(c->ws + c->L.gstats);
  ADG_HIP(hipMemcpyAsync(d_csr, csr.data(), 4 * csr.size(), hipMemcpyHostToDevice, c->stream));
  ADG_HIP(launch_stats(c->stage_args(), d_u, d_ref, part, (const int32_t*)(c->ws + c->L.first_s), n, pstats,
                       c->stream));
  ADG_HIP(launch_group_stats(pstats, d_csr, d_csr + n + 1, n_groups, gout, c->stream));
  ADG_HIP(hipMemcpyAsync(h_out, gout, 4 * sizeof(double) * n_groups, hipMemcpyDeviceToHost, c->stream));
  ADG_HIP(hipStreamSynchronize(c->stream));
  return ADG_OK;
}

int adg_delay_schedule(const adg_problem* p, int64_t step0, int64_t n_steps, int32_t* h_k) {
  int rc = validate(p, 1);
  if (rc) return rc;
  if (!h_k || step0 < 0 || n_steps < 0) return fail(ADG_E_INVALID, "bad schedule arguments");
  const int S = rk_stages((int)p->rk);
  const int64_t P = p->n_elem / p->pe_size;
  if (P <= 1) return ADG_OK;
  const int q = q_of(*p);
  for (int64_t i = 0; i < n_steps; ++i) {
    const int64_t n = step0 + i;
    for (int s = 0; s < S; ++s) {
      const int key = p->delay_granularity == ADG_DELAY_PER_STAGE ? s : 0;
      for (int64_t b = 0; b < P; ++b) {
        int k = 0;
        if (p->scheme != ADG_SCHEME_DG) {
          k = p->delay_granularity == ADG_DELAY_CAA
                  ? caa_delay(n)
                  : draw_delay(p->seed, n, key, b, p->delay_threshold, (int)p->n_delays);
          k = clamp_delay(k, n, q);
        }
        h_k[(i * S + s) * P + b] = k;
      }
    }
  }
  return ADG_OK;
}

int adg_destroy(adg_ctx* c) {
  if (!c) return ADG_OK;
  drop_graph(c);
  delete c;
  return ADG_OK;
}

}  // extern "C"
