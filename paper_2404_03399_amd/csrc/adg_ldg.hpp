// Tile of the fused step of viscous Burgers in local DG form (Sec. 7).
#pragma once

#include "adg_wave.hpp"

namespace adg {

// K whole RK steps of R consecutive elements per lane, as stage_tile.  Per
// stage: u-hat at a face is the trace of the element on its left (alternating
// flux); q = Kr u-hat_right - Kl u-hat_left - Kd u; the total flux at a face is
// G = LLF(u-, u+) - nu q+ with q+ from the element on its right; the element
// update is Kl G_left - Kr G_right + Kd (u^2/2 - nu q).  At a PE face the AT
// combinations of past levels replace both the face's u-hat and its G where the
// drawn delay is not 0; the element on the left takes the applied u-hat from
// the next lane.  Elsewhere u-hat_right is the element's own trace, so q needs
// no data from the right and each stage depends on one element to either side;
// one element more on the right covers the last lane's PE face, whose u-hat no
// lane holds.
//
// ANY: a lane's PE face may be the left face of any of its elements (as in
// stage_tile).
//
// Bound by FP64 issue (two operator products per stage).  Heun, p = 2, AT2, PE
// 256, 2^20 elements: 11.4 us per step with two elements per lane, two steps
// per launch and the operator in SGPRs; 7.4 with four, eight and the operator
// broadcast from a register pair.
template <int NP, int RK, int R, bool ANY = false>
__device__ __forceinline__ void ldg_tile(const DevProblem& P, const WorkItem wi, double* __restrict__ ring, int64_t n,
                                         int K, int HL, int HR, const double* __restrict__ uin,
                                         double* __restrict__ uout, int n_faces_max, double* __restrict__ lds,
                                         int lane) {
#pragma clang fp contract(off)  // explicit FMAs only
  constexpr int S = rk_stages(RK);
  const WaveElems<R> we(P, wi.tile, HL, HR, lane);
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
    op[c] = x < CPR * NP && j < NP ? P.Kd[i * kMaxNp + j] : 0.0;
  }
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    kl[i] = P.Kl[i];
    kr[i] = P.Kr[i];
  }
  int at_r = 0, e_face = we.e[0];
  lane_face<R, ANY>(P, we, at_r, e_face);
  WaveFaces<S, 2> wf(P, e_face, at_r < we.own_n, atc, n, K, n_faces_max, lds, lane);
  wf.draw(P, ring, n, K, lane);

  const double nu2 = 2.0 * P.nu, dt2 = 0.5 * P.dt;
  bool rpe = false;  // the right face of the last element is a PE face
  if (P.async_faces) {
    const uint32_t e1 = (we.e[R - 1] + 1 == (int)P.n_elem) ? 0u : (uint32_t)(we.e[R - 1] + 1);
    rpe = e1 == fast_div(e1, P.pe_div) * P.pe_div.d;
  }
  int kk = 0;
  auto steps = [&](auto with_pe, int k_end) {
    constexpr bool PE = decltype(with_pe)::value;
    for (; kk < k_end; ++kk) {
      KdWord kd = 0;
      double* const mine_g = PE ? wf.sums(K, kk, 0) : nullptr;
      double* const mine_u = PE ? wf.sums(K, kk, 1) : nullptr;
      if constexpr (PE) kd = wf.delays(K, kk);
      double u0[R][NP], ks[R][NP];
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int j = 0; j < NP; ++j) u0[r][j] = y[r][j];
#pragma unroll
      for (int s = 0; s < S; ++s) {
        double um[R], G[R], v[R][NP];  // G and v = -nu q doubled: no factors of 1/2
        um[0] = lane_from_left(y[R - 1][NP - 1]);  // u- at the left face, and its u-hat
#pragma unroll
        for (int r = 1; r < R; ++r) um[r] = y[r - 1][NP - 1];
        bool late = false;
        double hl[R], at_g = 0.0, hr_last = y[R - 1][NP - 1];  // hl: the applied u-hat of the left faces
#pragma unroll
        for (int r = 0; r < R; ++r) hl[r] = um[r];
        if constexpr (PE) {
          late = (kd & ((KdWord)0xff << (8 * s))) != 0;
          const double at_u = mine_u[s];
          at_g = mine_g[s];
          double raw = um[0];
#pragma unroll
          for (int r = 1; r < R; ++r) raw = ANY && at_r == r ? um[r] : raw;
          mine_u[s] = raw;
#pragma unroll
          for (int r = 0; r < (ANY ? R : 1); ++r) hl[r] = late && at_r == r ? at_u : um[r];
          const double h = lane_from_right(hl[0]);
          hr_last = rpe ? h : hr_last;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const double hr = r + 1 < R ? hl[r + 1 < R ? r + 1 : r] : hr_last;
#pragma unroll
          for (int i = 0; i < NP; ++i) v[r][i] = fma(kl[i], hl[r], -kr[i] * hr);
          fmac_operator<NP>(op, y[r], v[r]);  // -q
#pragma unroll
          for (int i = 0; i < NP; ++i) v[r][i] *= nu2;
          const double up = y[r][0], lam = fmax(fabs(um[r]), fabs(up));
          G[r] = fma(0.5, fma(um[r], um[r], up * up), fma(lam, um[r] - up, v[r][0]));
          __builtin_amdgcn_sched_barrier(0);  // one element after the other
        }
        if constexpr (PE) {
          double raw = G[0];
#pragma unroll
          for (int r = 1; r < R; ++r) raw = ANY && at_r == r ? G[r] : raw;
          mine_g[s] = 0.5 * raw;
#pragma unroll
          for (int r = 0; r < (ANY ? R : 1); ++r) G[r] = late && at_r == r ? 2.0 * at_g : G[r];
        }
        const double g_last = lane_from_right(G[0]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          const double gr = r + 1 < R ? G[r + 1 < R ? r + 1 : r] : g_last;
          double k[NP], g[NP];
#pragma unroll
          for (int j = 0; j < NP; ++j) {
            g[j] = fma(y[r][j], y[r][j], v[r][j]);
            k[j] = fma(-kr[j], gr, kl[j] * G[r]);
          }
          fmac_operator<NP>(op, g, k);
          rk_update<NP, RK>(s, dt2, u0[r], y[r], ks[r], k);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      if constexpr (PE) {
        // the new state before the loop below (as in stage_tile)
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int j = 0; j < NP; ++j) asm volatile("" : "+v"(y[r][j]));
        wf.pass_on(P, K, kk, lane);
      }
    }
  };
  steps(std::true_type{}, wf.m_pe ? K : 0);
  steps(std::false_type{}, K);

  we.store(P, uout, y);
  wf.keep(P, ring, K, lane);
}

}  // namespace adg
