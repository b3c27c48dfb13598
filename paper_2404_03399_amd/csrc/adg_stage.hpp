// Tile of the fused step, stage by stage: every equation, flux and integrator
// of the fused kernel but viscous Burgers.
#pragma once

#include "adg_wave.hpp"

namespace adg {

// K whole RK steps of R consecutive elements per lane, all stages on chip: one
// wave64 is a tile with halo lanes (each stage shrinks the valid range by one
// element per side; upwind with a > 0 on the left only), recomputed with the
// same instructions as by their owners, so a face shared by two waves gets a
// bitwise-identical flux on both sides.  Each lane computes the fluxes of the
// left faces of its elements; the right face of its last element is the next
// lane's first left face, received by a lane shift.  No workgroup barrier: the
// waves of a workgroup are independent.  PE faces as in WaveFaces.
//
// The kernel is bound by FP64 issue (p = 3, RK4, a > 0: 112 operations per
// element and step), so what it spends beside them counts: the operator sits
// in one or two register pairs and is read by DPP row broadcasts (as scalars
// loaded inside the stages it cost a wait per stage), and waves with and
// without PE faces run loops of their own.
//
// Every element takes the same operations in the same order whatever R, K and
// the wave it is in (explicit FMAs, contraction off): all launch shapes agree
// bitwise.

// ANY: R does not divide every PE size, so a lane's PE face (at most one) is
// the left face of any of its elements; selects find it in every stage, which
// waves with a face pay for.
template <int NP, int RK, int PHYS, int R, bool ANY = false>
__device__ __forceinline__ void stage_tile(const DevProblem& P, const WorkItem wi, double* __restrict__ ring,
                                           int64_t n, int K, int HL, const double* __restrict__ uin,
                                           double* __restrict__ uout, double* __restrict__ umid, int64_t mid_stride,
                                           int n_faces_max, double* __restrict__ lds, int lane) {
#pragma clang fp contract(off)
  constexpr int S = rk_stages(RK);
  constexpr bool POS = PHYS == PHYS_ADV_UPWIND_POS;
  static_assert(!(POS && ANY), "the correction of a right PE face knows the lane's last element only");
  const WaveElems<R> we(P, wi.tile, HL, POS ? (P.async_faces ? 1 : 0) : HL, lane);
  // the AT weights, ahead of the state in the queue of loads
  double atc = 0.0;
  if (P.async_faces && lane < kMaxL * kMaxQ) atc = P.atc[0][lane];
  double y[R][NP];
  we.load(P, uin, y);
  constexpr int CPR = NP == 5 ? 3 : NP, NOP = NP == 5 ? 2 : 1;  // columns of the operator per register pair
  double op[NOP], kl[NP], kr[NP];
#pragma unroll
  for (int c = 0; c < NOP; ++c) {
    const int x = lane & 15, j = c * CPR + x / NP, i = x % NP;
    op[c] = x < CPR * NP && j < NP ? (POS ? P.Kdu : P.Kd)[i * kMaxNp + j] : 0.0;
  }
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    kl[i] = P.Kl[i];
    kr[i] = P.Kr[i];
  }
  int at_r = 0, e_face = we.e[0];  // the element right of the lane's PE face
  lane_face<R, ANY>(P, we, at_r, e_face);
  WaveFaces<S> wf(P, e_face, at_r < we.own_n, atc, n, K, n_faces_max, lds, lane);
  wf.draw(P, ring, n, K, lane);

  const double a = P.speed, dt = P.dt;
  // upwind, a > 0: the interior right-face flux a u_p is part of Kdu; a PE face
  // on the right adds -Kr (F_right - a u_p)
  bool rpe = false;
  if (POS && P.async_faces) {
    const uint32_t e1 = (we.e[R - 1] + 1 == (int)P.n_elem) ? 0u : (uint32_t)(we.e[R - 1] + 1);
    rpe = e1 == fast_div(e1, P.pe_div) * P.pe_div.d;
  }
  int kk = 0;
  auto steps = [&](auto with_pe, int k_end) {
    constexpr bool PE = decltype(with_pe)::value;
    for (; kk < k_end; ++kk) {
      // the halo holds K steps, so the owned elements are exact after each
      if (kk > 0 && umid != nullptr) we.store(P, umid + (int64_t)(kk - 1) * mid_stride, y);
      double at[S] = {};
      KdWord kd = 0;
      double* const mine = PE ? wf.sums(K, kk) : nullptr;
      if constexpr (PE) {
        kd = wf.delays(K, kk);
#pragma unroll
        for (int s = 0; s < S; ++s) at[s] = mine[s];
      }
      double u0[R][NP], ks[R][NP];
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int j = 0; j < NP; ++j) u0[r][j] = y[r][j];
#pragma unroll
      for (int s = 0; s < S; ++s) {
        double F[R];
        F[0] = Physics<PHYS>::fhat(lane_from_left(y[R - 1][NP - 1]), y[0][0], a);
#pragma unroll
        for (int r = 1; r < R; ++r) F[r] = Physics<PHYS>::fhat(y[r - 1][NP - 1], y[r][0], a);
        if constexpr (PE) {
          const bool late = (kd & ((KdWord)0xff << (8 * s))) != 0;
          double raw = F[0];
#pragma unroll
          for (int r = 1; r < R; ++r) raw = at_r == r ? F[r] : raw;
          mine[s] = raw;
#pragma unroll
          for (int r = 0; r < (ANY ? R : 1); ++r) F[r] = late && at_r == r ? at[s] : F[r];
        }
        double f_last = 0.0;
        if constexpr (!POS || PE) f_last = lane_from_right(F[0]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          double k[NP], g[NP];
          const double fr = r + 1 < R ? F[r + 1 < R ? r + 1 : r] : f_last;
#pragma unroll
          for (int i = 0; i < NP; ++i) {
            if constexpr (POS)
              k[i] = kl[i] * F[r];
            else
              k[i] = fma(-kr[i], fr, kl[i] * F[r]);
            g[i] = PHYS == PHYS_BURGERS_LLF ? y[r][i] * y[r][i] : y[r][i];
          }
          fmac_operator<NP>(op, g, k);
          if constexpr (POS && PE) {
            if (r + 1 == R) {
              // 0 at an interior face; at a PE face the applied flux minus the
              // exact a u_p (for a synchronous one the rounding error of a u_p)
              const double corr = rpe ? fma(-a, y[r][NP - 1], fr) : 0.0;
#pragma unroll
              for (int i = 0; i < NP; ++i) k[i] = fma(-kr[i], corr, k[i]);
            }
          }
          rk_update<NP, RK>(s, dt, u0[r], y[r], ks[r], k);
          // one element after the other: interleaved, their sums take R sets of registers
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if constexpr (PE) {
        // the new state before the loop below: moved behind it, its operands
        // stay live through the loop (217 registers instead of 149 at p = 3,
        // RK4, four elements per lane)
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int j = 0; j < NP; ++j) asm volatile("" : "+v"(y[r][j]));
        wf.pass_on(P, K, kk, lane);
      }
    }
  };
  // one loop after the other, of which one takes all steps: as the two sides of
  // a branch the compiler keeps the state twice
  steps(std::true_type{}, wf.m_pe ? K : 0);
  steps(std::false_type{}, K);

  we.store(P, uout, y);
  wf.keep(P, ring, K, lane);
}

}  // namespace adg
