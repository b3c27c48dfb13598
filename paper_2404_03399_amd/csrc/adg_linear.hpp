// Tile of the fused step of linear advection with the upwind flux and a > 0,
// in flux-sequence form (device code shared by its own launch and by the
// launch over every range).
#pragma once

#include "adg_wave.hpp"

namespace adg {

// For a constant-coefficient linear problem a whole RK step of one element is
// a fixed linear map of its own nodes u and of the S fluxes F_s applied at its
// left face (table and symbols: adg_common.hpp).  The interior right face
// (upwind, a > 0: the element's own trace) being part of the map, the stages
// exchange one number per element and stage, as the stage-by-stage form does,
// but no stage value is ever formed.  A step has two phases: the fluxes,
//   g_s = sum Z_sj d_j + sum_{j<s} W_sj f_j,  f_s = a (u_p,left - u_p) + g_s,left,
// and then each element's update u' = u + (sum A_j d_j + sum Phi_s f_s), for
// degree 3 and RK4 58 FP64 operations (3 differences, 2 of the left face, 9 Z,
// 6 W, 3 sums; 3 differences, 12 A, 16 Phi, 4 sums) where the stages take 112 (a
// flux, a 4x4 operator and a lift four times, 28 of RK updates).  Information
// travels to the right only, so a tile has its halo (K S elements, recomputed)
// on the left.
//
// Rounding: u is added last and what it is added to is built from differences,
// so that a step rounds at the size of u once, as the stages' last update does;
// against 113-bit arithmetic, 64 steps, the error is 0.9 to 1.1 times the stage
// form's (RK4, Heun) or half of it and less (SSP-RK3, low storage), at sigma 0.1
// as at 0.001.  With the fluxes added to u one by one, or coefficients on the
// nodes' own values, it was 1.7 to 6.
//
// Bound by VALU issue: at p = 3, RK4, PE 256, 2^24 elements, four per lane and eight
// steps, 2945 instructions per wave, 63 % of them FP64, and a quarter of the wave
// cycles waiting.  us per step, this form and stage by stage: 2^20 elements 4.79,
// 6.55; 2^24 53.9, 84.2.
//
// At a PE face the raw flux G_s of the element on the left is replaced by the
// AT combination of delayed levels (WaveFaces) where the drawn delay is not 0;
// the element left of the face then takes the difference delta_s between
// applied and raw flux through WR and Psi.  Waves with and without faces run
// two step loops without any further branch.
//
// Every element takes the same operations in the same order whatever the
// lanes' element count R, the steps per launch and the wave it is in (explicit
// FMAs, contraction off), so all launch shapes agree bitwise.

// Columns J .. of a kind applied to one element: a_i += coefficient times x_J,
// the columns in order.
template <int NP, int S, int KIND, int J>
__device__ __forceinline__ void lin_apply(const double (&tab)[lin_tab_size(NP, S) / 16], double x, double* v) {
  constexpr int at = lin_col(NP, S, KIND, J), M = lin_col_len(NP, S, KIND, J);
  double* a[M];
#pragma unroll
  for (int i = 0; i < M; ++i) a[i] = v + i;
  fmac_bcast<at % 16, M>(tab[at / 16], x, a);
}
template <int NP, int S, int KIND, int J>
__device__ __forceinline__ void lin_all(const double (&tab)[lin_tab_size(NP, S) / 16], const double* x, double* v) {
  if constexpr (J < lin_cols(NP, S, KIND)) {
    lin_apply<NP, S, KIND, J>(tab, x[J], v);
    lin_all<NP, S, KIND, J + 1>(tab, x, v);
  }
}

// The fluxes of one step: F[r][s] holds g_s of element r and becomes f_s.  A PE
// face is the left face of a lane's element 0 (lanes with a face), so its left
// neighbour is the last element of the lane before.  kd: the delays of this
// lane's face (byte s, 0 elsewhere); at: its AT sums; raw: where it keeps the
// raw fluxes of the step; delta[s]: applied minus raw flux at the right face of
// the last element.
template <int NP, int S, int R, bool PE, int s = 0>
__device__ __forceinline__ void lin_fluxes(const double (&tab)[lin_tab_size(NP, S) / 16], double a, double u_left,
                                           double u_last, double f_left, double (&F)[R][S], double (&delta)[S],
                                           KdWord kd, const double (&at)[S], double* __restrict__ raw) {
#pragma clang fp contract(off)
  if constexpr (s < S) {
    double g_left = 0.0;
    if constexpr (s > 0) {
      g_left = lane_from_left(F[R - 1][s]);
#pragma unroll
      for (int r = R - 1; r > 0; --r) F[r][s] = F[r][0] + F[r - 1][s];
      F[0][s] = f_left + g_left;
    }
    if constexpr (PE) {
      const double G = s > 0 ? fma(a, u_left, g_left) : a * u_left;
      raw[s] = G;
      const bool late = (kd & ((KdWord)0xff << (8 * s))) != 0;
      const double d = at[s] - G, f = fma(-a, u_last, at[s]);
      F[0][s] = late ? f : F[0][s];
      delta[s] = lane_from_right(late ? d : 0.0);
    }
    if constexpr (s + 1 < S) {
#pragma unroll
      for (int r = 0; r < R; ++r) lin_apply<NP, S, LIN_W, s>(tab, F[r][s], &F[r][s + 1]);
      if constexpr (PE) lin_apply<NP, S, LIN_WR, s>(tab, delta[s], &F[R - 1][s + 1]);
    }
    lin_fluxes<NP, S, R, PE, s + 1>(tab, a, u_left, u_last, f_left, F, delta, kd, at, raw);
  }
}

template <int NP, int S, int R>
__device__ __forceinline__ void lin_tile(const DevProblem& P, const double* __restrict__ tab_in, const WorkItem wi,
                                         double* __restrict__ ring, int64_t n, int K, int HL,
                                         const double* __restrict__ uin, double* __restrict__ uout,
                                         int n_faces_max, double* __restrict__ lds, int lane) {
#pragma clang fp contract(off)  // explicit FMAs only: rounding independent of the launch shape
  const WaveElems<R> we(P, wi.tile, HL, P.async_faces ? 1 : 0, lane);
  // the AT weights, ahead of the state in the queue of loads
  double atc = 0.0;
  if (P.async_faces && lane < kMaxL * kMaxQ) atc = P.atc[0][lane];
  double u[R][NP];
  we.load(P, uin, u);
  WaveFaces<S> wf(P, we.e[0], we.own_n > 0, atc, n, K, n_faces_max, lds, lane);
  wf.draw(P, ring, n, K, lane);

  const double a = P.speed;
  constexpr int RUNS = lin_tab_size(NP, S) / 16, Z0 = lin_col(NP, S, LIN_Z, 0), A0 = lin_col(NP, S, LIN_A, 0);
  double tab[RUNS], z0[S - 1], a0[NP];
#pragma unroll
  for (int i = 0; i < RUNS; ++i) tab[i] = tab_in[16 * i + (lane & 15)];
  // the first columns, in SGPRs
#pragma unroll
  for (int i = 0; i < S - 1; ++i) z0[i] = tab_in[Z0 + i];
#pragma unroll
  for (int i = 0; i < NP; ++i) a0[i] = tab_in[A0 + i];
  int kk = 0;
  auto steps = [&](auto with_pe, int k_end) {
    constexpr bool PE = decltype(with_pe)::value;
    for (; kk < k_end; ++kk) {
      double F[R][S], delta[S] = {};
      const double u_left = lane_from_left(u[R - 1][NP - 1]);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        double d[NP];
#pragma unroll
        for (int j = 0; j + 1 < NP; ++j) d[j] = u[r][j] - u[r][NP - 1];
        F[r][0] = a * ((r > 0 ? u[r > 0 ? r - 1 : 0][NP - 1] : u_left) - u[r][NP - 1]);
#pragma unroll
        for (int s = 1; s < S; ++s) F[r][s] = z0[s - 1] * d[0];
        lin_all<NP, S, LIN_Z, 1>(tab, d, &F[r][1]);
        // one element after the other: interleaved, their sums take R sets of registers
        __builtin_amdgcn_sched_barrier(0);
      }
      double at[S] = {};
      KdWord kd = 0;
      double* const mine = PE ? wf.sums(K, kk) : nullptr;
      if constexpr (PE) {
        kd = wf.delays(K, kk);
#pragma unroll
        for (int s = 0; s < S; ++s) at[s] = mine[s];
      }
      lin_fluxes<NP, S, R, PE>(tab, a, u_left, u[0][NP - 1], F[0][0], F, delta, kd, at, mine);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        // the differences again: kept from above they are R (NP - 1) registers more
#pragma unroll
        for (int j = 0; j < NP; ++j) asm volatile("" : "+v"(u[r][j]));
        double d[NP], v[NP];
#pragma unroll
        for (int j = 0; j + 1 < NP; ++j) d[j] = u[r][j] - u[r][NP - 1];
#pragma unroll
        for (int i = 0; i < NP; ++i) v[i] = a0[i] * d[0];
        lin_all<NP, S, LIN_A, 1>(tab, d, v);
        lin_all<NP, S, LIN_PHI, 0>(tab, F[r], v);
        if constexpr (PE)
          if (r + 1 == R) lin_all<NP, S, LIN_PSI, 0>(tab, delta, v);
#pragma unroll
        for (int i = 0; i < NP; ++i) u[r][i] += v[i];
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (PE) wf.pass_on(P, K, kk, lane);
    }
  };
  // one loop after the other, of which one takes all steps: as the two sides of
  // a branch the compiler keeps the state twice (144 registers instead of 112)
  steps(std::true_type{}, wf.m_pe ? K : 0);
  steps(std::false_type{}, K);

  we.store(P, uout, u);
  wf.keep(P, ring, K, lane);
}

}  // namespace adg
