// Tile of the fused step of linear advection with the upwind flux and a > 0,
// in flux-sequence form (device code shared by its own launch and by the
// launch over every range).
#pragma once

#include "adg_wave.hpp"

namespace adg {

// For a constant-coefficient linear problem a whole RK step of one element is
// a fixed linear map of its own nodes u and of the S fluxes F_s applied at its
// left face (LinTab, adg_common.hpp):
//   G_s   = Z_s u + sum_{j<s} W_sj F_j          the flux a y_s(x_R) that stage s
//                                               sends through the right face,
//   u'    = A0 u + sum_s Phi_s F_s,
// the interior right face (upwind, a > 0: the element's own trace) being part
// of Z, W, A0 and Phi.  So the stages exchange one number per element and
// stage, as the stage-by-stage form does, but no stage value is ever formed:
// for degree 3 and RK4 a step takes 51 FP64 operations per element (1 for a
// u_p, 12 Z, 6 W, 16 A0, 16 Phi) where the stages take 116 (a 4x4 operator, a
// lift and the RK updates four times).  Information travels to the right only,
// so a tile has its halo (K S elements, recomputed) on the left.
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

// One column of the table applied to one element: f (the S values G_s, then
// F_s) and v (its nodes) take coefficient times x.
template <int NP, int S, int KIND, int J>
__device__ __forceinline__ void lin_apply(const double (&tab)[lin_tab_size(NP, S) / 16], double x, double (&f)[S],
                                          double (&v)[NP]) {
  constexpr int at = lin_col(NP, S, KIND, J), M = lin_col_len(NP, S, KIND, J), s0 = S - (M - NP);
  double* a[M];
#pragma unroll
  for (int i = 0; i < M; ++i) a[i] = i < M - NP ? &f[s0 + i] : &v[i - (M - NP)];
  fmac_bcast<at % 16, M>(tab[at / 16], x, a);
}

// the node columns but the first, in order
template <int NP, int S, int J = 1>
__device__ __forceinline__ void lin_nodes(const double (&tab)[lin_tab_size(NP, S) / 16], const double (&u)[NP],
                                          double (&f)[S], double (&v)[NP]) {
  if constexpr (J < NP) {
    lin_apply<NP, S, LIN_U, J>(tab, u[J], f, v);
    lin_nodes<NP, S, J + 1>(tab, u, f, v);
  }
}

// The stages of one step: F_s of every element from its left neighbour's G_s
// (applied AT flux at a delayed PE face), then its column.  A PE face is the
// left face of a lane's element 0 (lanes `pe`), so its left neighbour is the
// last element of the lane before.  kd: the delays of this lane's face (byte s,
// 0 elsewhere); at: its AT sums; raw: where it keeps the raw fluxes of the step.
template <int NP, int S, int R, bool PE, int s = 0>
__device__ __forceinline__ void lin_stages(const double (&tab)[lin_tab_size(NP, S) / 16], double (&F)[R][S],
                                           double (&u)[R][NP], KdWord kd, const double (&at)[S],
                                           double* __restrict__ raw) {
#pragma clang fp contract(off)
  if constexpr (s < S) {
    const double g_left = lane_from_left(F[R - 1][s]);
#pragma unroll
    for (int r = R - 1; r > 0; --r) F[r][s] = F[r - 1][s];
    F[0][s] = g_left;
    double dl = 0.0;  // applied minus raw flux at the right face of the last element
    if constexpr (PE) {
      raw[s] = g_left;
      const bool sel = (kd & ((KdWord)0xff << (8 * s))) != 0;
      const double d = at[s] - g_left;
      F[0][s] = sel ? at[s] : g_left;
      dl = lane_from_right(sel ? d : 0.0);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) lin_apply<NP, S, LIN_F, s>(tab, F[r][s], F[r], u[r]);
    if constexpr (PE) lin_apply<NP, S, LIN_D, s>(tab, dl, F[R - 1], u[R - 1]);
    lin_stages<NP, S, R, PE, s + 1>(tab, F, u, kd, at, raw);
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
  double tab[lin_tab_size(NP, S) / 16], col0[S - 1 + NP];
#pragma unroll
  for (int i = 0; i < lin_tab_size(NP, S) / 16; ++i) tab[i] = tab_in[16 * i + (lane & 15)];
#pragma unroll
  for (int i = 0; i < S - 1 + NP; ++i) col0[i] = tab_in[i];  // the first column, in SGPRs
  int kk = 0;
  auto steps = [&](auto with_pe, int k_end) {
    constexpr bool PE = decltype(with_pe)::value;
    for (; kk < k_end; ++kk) {
      // F[r][s]: first the element's own part of G_s, then F_s
      double F[R][S];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        F[r][0] = a * u[r][NP - 1];
#pragma unroll
        for (int s = 1; s < S; ++s) F[r][s] = fma(col0[s - 1], u[r][0], F[r][0]);
        double v[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i) v[i] = col0[S - 1 + i] * u[r][0];
        lin_nodes<NP, S>(tab, u[r], F[r], v);
#pragma unroll
        for (int i = 0; i < NP; ++i) u[r][i] += v[i];
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
      lin_stages<NP, S, R, PE>(tab, F, u, kd, at, mine);
      if constexpr (PE) wf.pass_on(P, K, kk, lane);
    }
  };
  // one loop after the other, of which one takes all steps: as the two sides of
  // a branch the compiler keeps the state twice (137 registers instead of 103)
  steps(std::true_type{}, wf.m_pe ? K : 0);
  steps(std::false_type{}, K);

  we.store(P, uout, u);
  wf.keep(P, ring, K, lane);
}

}  // namespace adg
