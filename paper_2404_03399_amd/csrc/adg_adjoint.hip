// Discrete adjoint, stage by stage: one launch per reverse RK stage (RK
// registers in HBM).
#include "adg_device.hpp"

namespace adg {

struct AdjPtrs {
  const double* __restrict__ Y;   // forward input of this stage
  const double* __restrict__ lam; // lambda_{n+1}
  double* __restrict__ lamu;      // lambda_n accumulator (starts as lambda_{n+1})
  double* __restrict__ Q;         // Q_i = sum_{j>i} a_ji mu_j, i < S-1, stride qstride
  int64_t qstride;
  const double* __restrict__ ring;  // forward raw PE fluxes (full history)
  double* __restrict__ adjring;     // their sensitivities (full history)
  double* __restrict__ cpart;       // per-workgroup dJ/da partial sums
};

// Reverse of stage SI of step n for one element: lambda_K = dt (b_SI lam + Q_SI),
// mu = (dK/dY)^T lambda_K with the transposed volume term, transposed face
// fluxes (both neighbours' lifts), and for PE faces the transposed AT
// combination: the delayed levels' share goes to the adjoint ring, the
// level-n raw flux collects its share plus what later steps deposited.
template <int NP, int RK, int PHYS, int SI>
__device__ __forceinline__ double adj_elem(const DevProblem& P, int tile, const AdjPtrs& A, int64_t n) {
  constexpr int S = rk_stages(RK);
  const int N = (int)P.n_elem;
  const int e = tile * kBlock + (int)threadIdx.x;
  if (e >= N) return 0.0;
  const int64_t ld = P.ld, off = P.u_off;
  const double a = P.speed, dt = P.dt;
  const int em = e == 0 ? N - 1 : e - 1;
  const int e1 = e + 1 == N ? 0 : e + 1;
  const double* __restrict__ Y = A.Y + off;
  double y[NP];
#pragma unroll
  for (int j = 0; j < NP; ++j) y[j] = Y[j * ld + e];
  const double um = Y[(NP - 1) * ld + em];
  const double upr = Y[e1];

  const double bs = dt * bt_b<RK>(SI);
  const double* __restrict__ lam = A.lam + off;
  const double* __restrict__ qs = A.Q + SI * A.qstride + off;
  auto lk = [&](int x, int i) {
    double v = bs * lam[i * ld + x];
    if constexpr (SI < S - 1) v += dt * qs[i * ld + x];
    return v;
  };
  double lke[NP];
  double lf_l = 0.0, lf_r = 0.0;
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    lke[i] = lk(e, i);
    lf_l += P.Kl[i] * lke[i] - P.Kr[i] * lk(em, i);
    lf_r += P.Kl[i] * lk(e1, i) - P.Kr[i] * lke[i];
  }
  double mu[NP];
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    double v = 0.0;
#pragma unroll
    for (int i = 0; i < NP; ++i) v += P.Kd[i * kMaxNp + j] * lke[i];
    mu[j] = PHYS == PHYS_BURGERS_LLF ? 2.0 * y[j] * v : v;
  }
  double dm_l, dp_l, dm_r, dp_r;
  flux_partials<PHYS>(um, y[0], a, dm_l, dp_l);
  flux_partials<PHYS>(y[NP - 1], upr, a, dm_r, dp_r);
  double raw_l = lf_l, raw_r = lf_r;
  // forward face fluxes (for the speed gradient)
  double fl = Physics<PHYS>::fhat(um, y[0], a);
  double fr = Physics<PHYS>::fhat(y[NP - 1], upr, a);
  if (P.async_faces) {
    const uint32_t pes = P.pe_div.d;
    const int depth = P.depth;
    const int slot_n = (int)(n % (int64_t)depth);
    const uint32_t bl = fast_div((uint32_t)e, P.pe_div);
    if ((uint32_t)e == bl * pes) {
      const int64_t rb = P.ring_off + ((int64_t)bl * S + SI);
      const int kd = pe_delay(P, n, SI, bl);
      raw_l = (kd == 0 ? lf_l : 0.0) + A.adjring[rb + slot_n * P.ring_stride];
      if (kd > 0) {
        fl = at_past_sum(P, A.ring + rb, kd, slot_n);
        for (int j = 0; j < P.q; ++j)
          A.adjring[rb + ring_slot(slot_n, kd + j, depth) * P.ring_stride] += P.atc[kd][j] * lf_l;
      }
    }
    const uint32_t br = fast_div((uint32_t)e1, P.pe_div);
    if ((uint32_t)e1 == br * pes) {
      const int64_t rb = P.ring_off + ((int64_t)br * S + SI);
      const int kd = pe_delay(P, n, SI, br);
      raw_r = (kd == 0 ? lf_r : 0.0) + A.adjring[rb + slot_n * P.ring_stride];
      if (kd > 0) fr = at_past_sum(P, A.ring + rb, kd, slot_n);
    }
  }
  mu[0] += raw_l * dp_l;
  mu[NP - 1] += raw_r * dm_r;

  double* __restrict__ lu = A.lamu + off;
#pragma unroll
  for (int j = 0; j < NP; ++j) lu[j * ld + e] += mu[j];
#pragma unroll
  for (int i = 0; i < SI; ++i) {
    const double c = bt_a<RK>(SI, i);
    if (c != 0.0) {
      double* __restrict__ qi = A.Q + i * A.qstride + off;
#pragma unroll
      for (int j = 0; j < NP; ++j) qi[j * ld + e] += c * mu[j];
    }
  }
  // dJ/da through this stage with its inputs held fixed: every term of K is
  // proportional to a for linear advection, so dK/da = K / a.
  double ca = 0.0;
  if constexpr (PHYS != PHYS_BURGERS_LLF) {
    double kf[NP];
    folded_rhs<NP, PHYS>(P, y, fl, fr, kf);
#pragma unroll
    for (int i = 0; i < NP; ++i) ca += lke[i] * kf[i];
    ca /= a;
  }
  return ca;
}

template <int RK, int PHYS, int SI>
__global__ __launch_bounds__(kBlock) void k_adj_stage(const DevProblem* __restrict__ probs,
                                                      const WorkItem* __restrict__ work, AdjPtrs A, int32_t n) {
  __shared__ double red[kBlock];
  const WorkItem wi = work[blockIdx.x];
  const DevProblem& P = probs[wi.prob];
  double ca;
  switch (P.np) {
    case 2: ca = adj_elem<2, RK, PHYS, SI>(P, wi.tile, A, n); break;
    case 3: ca = adj_elem<3, RK, PHYS, SI>(P, wi.tile, A, n); break;
    case 4: ca = adj_elem<4, RK, PHYS, SI>(P, wi.tile, A, n); break;
    default: ca = adj_elem<5, RK, PHYS, SI>(P, wi.tile, A, n); break;
  }
  if constexpr (PHYS != PHYS_BURGERS_LLF) {
    red[threadIdx.x] = ca;
    __syncthreads();
    for (int w = kBlock / 2; w > 0; w >>= 1) {
      if ((int)threadIdx.x < w) red[threadIdx.x] += red[threadIdx.x + w];
      __syncthreads();
    }
    if (threadIdx.x == 0) A.cpart[blockIdx.x] += red[0];
  }
}

template <int RK, int PHYS, int SI>
static void adj_go(const StepArgs& a, const AdjPtrs& p, int32_t n, hipStream_t st) {
  hipLaunchKernelGGL((k_adj_stage<RK, PHYS, SI>), dim3(a.n_work), dim3(kBlock), 0, st, a.probs, a.work, p, n);
}

template <int RK, int PHYS>
static void adj_si(int si, const StepArgs& a, const AdjPtrs& p, int32_t n, hipStream_t st) {
  switch (si) {
    case 0: adj_go<RK, PHYS, 0>(a, p, n, st); break;
    case 1: adj_go<RK, PHYS, 1>(a, p, n, st); break;
    case 2: if constexpr (rk_stages(RK) > 2) adj_go<RK, PHYS, 2>(a, p, n, st); break;
    case 3: if constexpr (rk_stages(RK) > 3) adj_go<RK, PHYS, 3>(a, p, n, st); break;
    default: if constexpr (rk_stages(RK) > 4) adj_go<RK, PHYS, 4>(a, p, n, st); break;
  }
}

template <int RK>
static void adj_phys(int phys, int si, const StepArgs& a, const AdjPtrs& p, int32_t n, hipStream_t st) {
  switch (phys) {
    case PHYS_ADV_UPWIND: adj_si<RK, PHYS_ADV_UPWIND>(si, a, p, n, st); break;
    case PHYS_ADV_CENTRAL: adj_si<RK, PHYS_ADV_CENTRAL>(si, a, p, n, st); break;
    default: adj_si<RK, PHYS_BURGERS_LLF>(si, a, p, n, st); break;
  }
}

hipError_t launch_adj_stage(int rk, int phys, int stage, const StepArgs& a, const double* Y, const double* lam,
                            double* lamu, double* Q, int64_t qstride, const double* ring, double* adjring,
                            double* cpart, int32_t n, hipStream_t stream) {
  const AdjPtrs p{Y, lam, lamu, Q, qstride, ring, adjring, cpart};
  switch (rk) {
    case RK_HEUN: adj_phys<RK_HEUN>(phys, stage, a, p, n, stream); break;
    case RK_SSP3: adj_phys<RK_SSP3>(phys, stage, a, p, n, stream); break;
    case RK_LS3: adj_phys<RK_LS3>(phys, stage, a, p, n, stream); break;
    case RK_LS4: adj_phys<RK_LS4>(phys, stage, a, p, n, stream); break;
    default: adj_phys<RK_RK4>(phys, stage, a, p, n, stream); break;
  }
  return hipGetLastError();
}

}  // namespace adg
