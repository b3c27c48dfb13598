// Tile of the fused reverse sweep.
#pragma once

#include "adg_wave.hpp"

namespace adg {

// PE faces of a wave over a reverse launch of K steps, from level n + K - 1
// down to n; jobs as in WaveFaces.  R is at most the PE size, so a lane holds at
// most one face, the left one of its element `at_r`.  Per (face, step, stage): the
// delay, the adjoint already collected for the step's raw flux (replaced, once
// read, by the sensitivity lf of the flux applied there) and, where the forward
// stages are recomputed, the AT sum of past levels.  A delay k spreads lf over
// the levels k, ..., k + q - 1 below its step.  Those of the launch are added in
// LDS by every wave that holds the face, those below n by its owner in the
// adjoint ring, always the latest step's first, which is the order of one step
// per launch.
//
// LDS of a wave with up to n_faces faces, behind the dJ/da values:
//   atc [kMaxL][kMaxQ]
//   lf  [job]       and S doubles more that lanes without a face write to
//   at  [job]       the same, with the forward stages only
//   kd  [face][step] word, own [face] word
template <int S, bool FWD, int R>
struct AdjFaces {
  double* atc;
  double* lf;
  double* at;
  KdWord* kd;
  KdWord* own;
  uint64_t m_pe = 0;
  bool pe = false;
  int n_faces_max, at_r = 0, n_jobs = 0, n_faces = 0, depth = 1, slot_n = 0, slot = 0;
  uint32_t b0 = 0;

  __device__ __forceinline__ AdjFaces(const DevProblem& P, const WaveElems<R>& we, double atc_lane, int64_t n, int K,
                                      int n_faces_max_, double* lds, int lane)
      : atc(lds), lf(lds + kMaxL * kMaxQ), n_faces_max(n_faces_max_) {
    const int words = n_faces_max * K * S + S;
    at = lf + words;
    kd = reinterpret_cast<KdWord*>(FWD ? at + words : at);
    own = kd + n_faces_max * K;
    if (!P.async_faces) return;
    depth = P.depth;
    const uint32_t n32 = (uint32_t)n;
    slot_n = (int)(n32 - fast_div(n32, P.depth_div) * (uint32_t)depth);
    uint32_t b = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const uint32_t br = fast_div((uint32_t)we.e[r], P.pe_div);
      if ((uint32_t)we.e[r] == br * P.pe_div.d) {
        pe = true;
        at_r = r;
        b = br;
      }
    }
    m_pe = __ballot(pe);
    slot = lane_rank(m_pe);
    b0 = (uint32_t)__builtin_amdgcn_readlane((int)b, m_pe ? __builtin_ctzll(m_pe) : 0);
    n_faces = __builtin_popcountll(m_pe);
    n_jobs = K * S * n_faces;
    if (pe) own[slot] = at_r < we.own_n ? 1 : 0;
    if (lane < kMaxL * kMaxQ) atc[lane] = atc_lane;
  }

  __device__ __forceinline__ uint32_t face(const DevProblem& P, int i) const {
    uint32_t b = b0 + (uint32_t)i;
    while (b >= (uint32_t)P.n_pe) b -= (uint32_t)P.n_pe;
    return b;
  }

  __device__ __forceinline__ void draw(const DevProblem& P, const double* __restrict__ ring,
                                       const double* __restrict__ adjring, int64_t n, int K, int lane) {
#pragma clang fp contract(off)
    const uint32_t kshift = (uint32_t)__builtin_ctz((uint32_t)K);  // K is a power of two
    for (int g0 = 0; g0 < n_jobs; g0 += kWave) {                   // uniform
      const int g = g0 + lane;
      if (g < n_jobs) {
        const int ik = g / S, s = g - ik * S, i = ik >> kshift, t = ik - (i << kshift);
        const uint32_t b = face(P, i);
        const int64_t rb = P.ring_off + (int64_t)b * S + s;
        const int k = pe_delay(P, n + t, s, b);
        int sl = slot_n + t;
        while (sl >= depth) sl -= depth;
        const double collected = adjring[rb + sl * P.ring_stride];
        if constexpr (FWD) {
          double lv[kMaxQ];
#pragma unroll
          for (int j = 0; j < kMaxQ; ++j) {
            lv[j] = 0.0;
            if (j < P.q && k > 0) lv[j] = ring[rb + ring_slot(sl, k + j, depth) * P.ring_stride];
          }
          double sum = 0.0;
#pragma unroll
          for (int j = kMaxQ - 1; j >= 0; --j)
            if (j < P.q && k > 0) sum = fma(atc[k * kMaxQ + j], lv[j], sum);
          at[g] = sum;
        }
        reinterpret_cast<uint8_t*>(kd + ik)[s] = (uint8_t)k;
        lf[g] = collected;
      }
    }
  }

  // This lane's face in step t: its S entries of lf and at, its delays (0
  // without a face).
  __device__ __forceinline__ int mine(int K, int t) const {
    return ((pe ? slot : n_faces_max) * K + (pe ? t : 0)) * S;
  }
  __device__ __forceinline__ KdWord delays(int K, int t) const {
    const KdWord w = kd[pe ? slot * K + t : 0];
    return pe ? w : 0;
  }

  // The sensitivities of step t reach the launch's earlier levels.
  __device__ __forceinline__ void pass_on(const DevProblem& P, int K, int t, int lane) {
#pragma clang fp contract(off)
    for (int g0 = 0; g0 < n_jobs && t > 0; g0 += kWave) {
      const int g = g0 + lane, ik = g / S, later = t - (ik & (K - 1));  // steps back to the job's level
      if (g < n_jobs && later > 0) {
        const int k = reinterpret_cast<const uint8_t*>(kd + ik + later)[g - ik * S], j = later - k;
        if (k > 0 && j >= 0 && j < P.q) lf[g] = fma(atc[k * kMaxQ + j], lf[g + later * S], lf[g]);
      }
    }
  }

  // Their shares of the levels n - d below the launch, d >= 1 up to
  // (L - 1) + (q - 1) at the largest L and q: one job lane per (owned face,
  // stage, level), each ring entry touched once.
  __device__ __forceinline__ void keep(const DevProblem& P, double* __restrict__ adjring, int K, int lane) const {
#pragma clang fp contract(off)
    constexpr int W = (kMaxL - 1) + (kMaxQ - 1);
    for (int g0 = 0; g0 < n_faces * S * W; g0 += kWave) {  // uniform
      const int g = g0 + lane;
      const int i = g / (S * W), x = g - i * (S * W), s = x / W, d = 1 + (x - s * W);
      if (i < n_faces && own[i] && d < depth) {
        double* __restrict__ at_d =
            adjring + P.ring_off + (int64_t)face(P, i) * S + s + ring_slot(slot_n, d, depth) * P.ring_stride;
        bool reached = false;
        double v = 0.0;
        for (int t = K - 1; t >= 0; --t) {
          const int ik = i * K + t, k = reinterpret_cast<const uint8_t*>(kd + ik)[s], j = t + d - k;
          if (k > 0 && j >= 0 && j < P.q) {
            if (!reached) v = *at_d;
            reached = true;
            v = fma(atc[k * kMaxQ + j], lf[ik * S + s], v);
          }
        }
        if (reached) *at_d = v;
      }
    }
  }
};

// The integrator's Butcher table, a constant expression also where a loop over
// its entries is not unrolled (evaluated on the device, the low-storage sums
// would round by the compiler's choice of FMAs).
template <int RK>
struct Butcher {
  double a[kMaxStages][kMaxStages] = {}, b[kMaxStages] = {};
  constexpr Butcher() {
    for (int i = 0; i < rk_stages(RK); ++i) {
      b[i] = bt_b<RK>(i);
      for (int j = 0; j < i; ++j) a[i][j] = bt_a<RK>(i, j);
    }
  }
};

// K whole reverse steps of R consecutive elements per lane, levels n + K - 1
// down to n: lambda^{n+K} in, lambda^n out.  Per step the forward stages are
// recomputed on chip from the recorded state where the reverse needs them
// (FWD: the stage operator values K_i for the speed gradient of advection, the
// stage inputs Y_i for the Burgers Jacobian), then the stages are reversed in
// Butcher form with the face terms exchanged between lanes:
//   lambda_K,i = dt (b_i lambda^{n+1} + sum_{j>i} a_ji mu_j),
//   mu_i = (dK_i/dY_i)^T lambda_K,i,   lambda^n = lambda^{n+1} + sum_i mu_i.
// Each reverse stage widens the dependence by one element per side, so K steps
// take a halo of K S elements for a constant Jacobian (linear advection).  For
// Burgers reverse stage s also reads the stage input Y_s one element further
// out, which is exact only s elements in from the wave's edge: (K + 1) S - 1.
//
// PHYS_ADV_UPWIND_POS (upwind, a > 0) transposes the folded forward operator:
// the interior flux a u_p of an element's right face sits in Kdu, so an
// element's sensitivity is Kdu^T lambda_K plus a (l_l . lambda_K of the right
// neighbour) at its last node, and the right lift (l_r . lambda_K) is formed
// only in waves that hold a PE face, where the applied flux replaces a u_p.
//
// dJ/da of advection: every term of K is proportional to a, so dK/da = K / a
// with the stage inputs held fixed.  The shares are summed over tiles of
// 64 - 2S elements, whatever R, in the order of a butterfly over one wave whose
// lane S + i holds the tile's element i, and each tile adds its steps one by
// one: R must be the launch list's number of steps (1 included), so that a wave
// owns R whole tiles.
//
// What bounds it: the waves in flight (the forward stage values of R elements
// leave three waves per SIMD at p = 3, RK4) and FP64 issue.  2^20 elements,
// p = 3, RK4, PE 256, with dJ/da: 30.2 us per step with one element per lane,
// one step per launch and the operator in SGPRs; 23.5 with two of each.  Without
// the forward stages, 2^17 elements: 3.8 us per step (two and two), 2.3 (two and
// eight).
//
// Every element takes the same operations in the same order whatever R and K
// (explicit FMAs, contraction off): all launch shapes agree bitwise.
template <int NP, int RK, int PHYS, bool FWD, int R>
__device__ __forceinline__ void adj_tile(const DevProblem& P, const WorkItem wi, int64_t n, int K, int HL,
                                         const double* __restrict__ u_n, const double* __restrict__ u_next,
                                         int64_t u_stride, const double* __restrict__ lam, double* __restrict__ lamo,
                                         const double* __restrict__ ring, double* __restrict__ adjring,
                                         double* __restrict__ cpart, int n_faces_max, double* __restrict__ lds,
                                         int lane) {
#pragma clang fp contract(off)
  constexpr int S = rk_stages(RK);
  constexpr Butcher<RK> bt;
  constexpr bool POS = PHYS == PHYS_ADV_UPWIND_POS, NL = PHYS == PHYS_BURGERS_LLF, SPEED = FWD && !NL;
  // the recomputed stages take the general form also for a > 0
  constexpr int FPHYS = POS ? (int)PHYS_ADV_UPWIND : PHYS;
  const WaveElems<R> we(P, wi.tile, HL, HL, lane);
  double atc = 0.0;
  if (P.async_faces && lane < kMaxL * kMaxQ) atc = P.atc[0][lane];
  double lu[R][NP];
  we.load(P, lam, lu);
  double un[R][NP];
  auto state = [&](int t) { return t == 0 ? u_n : u_next + (int64_t)(t - 1) * u_stride; };
  if constexpr (FWD) we.load(P, state(K - 1), un);
  constexpr int CPR = NP == 5 ? 3 : NP, NOP = NP == 5 ? 2 : 1;  // columns of the operator per register pair
  double op[NOP], opt[NOP], kl[NP], kr[NP];
#pragma unroll
  for (int c = 0; c < NOP; ++c) {
    const int x = lane & 15, j = c * CPR + x / NP, i = x % NP;
    const bool in = x < CPR * NP && j < NP;
    op[c] = FWD && in ? P.Kd[i * kMaxNp + j] : 0.0;
    opt[c] = in ? (POS ? P.Kdu : P.Kd)[j * kMaxNp + i] : 0.0;  // the transpose's column j
  }
#pragma unroll
  for (int i = 0; i < NP; ++i) {
    kl[i] = P.Kl[i];
    kr[i] = P.Kr[i];
  }
  constexpr int T1 = adj_part_elems(RK);
  double* const parts = lds;  // [R][T1], SPEED only
  double* const face_lds = lds + (SPEED ? R * kWave : 0);
  AdjFaces<S, FWD, R> wf(P, we, atc, n, K, n_faces_max, face_lds, lane);
  wf.draw(P, ring, adjring, n, K, lane);

  const double a = P.speed, dt = P.dt;
  const bool lane_owned = lane >= HL && lane < kWave - HL;
  // the tile's sum stands in the first lane of a half
  double c_sum = 0.0;
  const int part = R * wi.tile + (lane >> 5);
  const bool c_lane = SPEED && (lane & 31) == 0 && (lane >> 5) < R && (int64_t)part * T1 < P.n_elem;
  if constexpr (SPEED)
    if (c_lane) c_sum = cpart[P.part_off + part];

  int t = K - 1;
  auto steps = [&](auto with_pe, int t_end) {
    constexpr bool PE = decltype(with_pe)::value;
    for (; t >= t_end; --t) {
      KdWord kd = 0;
      double* const lf = PE ? wf.lf + wf.mine(K, t) : nullptr;
      double* const at = PE && FWD ? wf.at + wf.mine(K, t) : nullptr;
      if constexpr (PE) kd = wf.delays(K, t);
      double keep[FWD ? R : 1][FWD ? S : 1][NP];
      if constexpr (FWD) {
        double y[R][NP], ks[R][NP];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int j = 0; j < NP; ++j) y[r][j] = un[r][j];
#pragma unroll
        for (int s = 0; s < S; ++s) {
          if constexpr (NL) {
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
              for (int j = 0; j < NP; ++j) keep[r][s][j] = y[r][j];
            if (s + 1 == S) break;
          }
          double F[R];
          F[0] = Physics<FPHYS>::fhat(lane_from_left(y[R - 1][NP - 1]), y[0][0], a);
#pragma unroll
          for (int r = 1; r < R; ++r) F[r] = Physics<FPHYS>::fhat(y[r - 1][NP - 1], y[r][0], a);
          if constexpr (PE) {
            const bool late = (kd & ((KdWord)0xff << (8 * s))) != 0;
            const double f = at[s];
#pragma unroll
            for (int r = 0; r < R; ++r) F[r] = late && wf.at_r == r ? f : F[r];
          }
          const double f_last = lane_from_right(F[0]);
#pragma unroll
          for (int r = 0; r < R; ++r) {
            double k[NP], g[NP];
            const double fr = r + 1 < R ? F[r + 1 < R ? r + 1 : r] : f_last;
#pragma unroll
            for (int i = 0; i < NP; ++i) {
              k[i] = fma(-kr[i], fr, kl[i] * F[r]);
              g[i] = NL ? y[r][i] * y[r][i] : y[r][i];
            }
            fmac_operator<NP>(op, g, k);
            if constexpr (!NL)
#pragma unroll
              for (int j = 0; j < NP; ++j) keep[r][s][j] = k[j];
            if (s + 1 < S) rk_update<NP, RK>(s, dt, un[r], y[r], ks[r], k);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }

      // the mu_j take the registers that keep's stages leave, where sums
      // sum_{j>i} a_ji mu_j for every stage i ahead would come on top of them
      double lamp[R][NP], mus[R][S][NP], ca[R];
#pragma unroll
      for (int r = 0; r < R; ++r) {
        ca[r] = 0.0;
#pragma unroll
        for (int j = 0; j < NP; ++j) lamp[r][j] = lu[r][j];
      }
#pragma unroll
      for (int s = S - 1; s >= 0; --s) {
        const double bs = dt * bt.b[s];
        double lk[R][NP], cl[R], cr[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
          for (int i = 0; i < NP; ++i) {
            double q = 0.0;  // dt sum_{j>s} a_js mu_j, the last stage first (dt folded into the weights)
#pragma unroll
            for (int j = S - 1; j > s; --j) {
              const double c = bt.a[j][s];
              if (c != 0.0) q = fma(dt * c, mus[r][j][i], q);
            }
            lk[r][i] = s < S - 1 ? fma(bs, lamp[r][i], q) : bs * lamp[r][i];
          }
          cl[r] = 0.0;
          cr[r] = 0.0;
#pragma unroll
          for (int i = 0; i < NP; ++i) cl[r] = fma(kl[i], lk[r][i], cl[r]);
          if constexpr (!POS || PE)
#pragma unroll
            for (int i = 0; i < NP; ++i) cr[r] = fma(kr[i], lk[r][i], cr[r]);
        }
        // raw[r]: sensitivity of the flux applied at element r's left face (both
        // neighbours' lifts); POS: g[r], what that face gives its left element's
        // last node, over a
        double raw[R], g[R];
#pragma unroll
        for (int r = 0; r < R; ++r) g[r] = cl[r];
        if constexpr (!POS || PE) {
          double crl[R];  // the left neighbour's right lift
          crl[0] = lane_from_left(cr[R - 1]);
#pragma unroll
          for (int r = 1; r < R; ++r) crl[r] = cr[r - 1];
#pragma unroll
          for (int r = 0; r < R; ++r) raw[r] = cl[r] - crl[r];
          if constexpr (PE) {
            double lfv = raw[0];
#pragma unroll
            for (int r = 1; r < R; ++r) lfv = wf.at_r == r ? raw[r] : lfv;
            const double rp = ((kd & ((KdWord)0xff << (8 * s))) == 0 ? lfv : 0.0) + lf[s];
            lf[s] = lfv;
#pragma unroll
            for (int r = 0; r < R; ++r) {
              const bool here = wf.pe && wf.at_r == r;
              // POS: the left element's right lift, which Kdu^T took off, comes
              // back with the raw flux's sensitivity
              if constexpr (POS)
                g[r] = here ? crl[r] + rp : g[r];
              else
                raw[r] = here ? rp : raw[r];
            }
          }
        }
        double dm[R], dp[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          if constexpr (NL)
            flux_partials<PHYS>(r > 0 ? keep[r > 0 ? r - 1 : 0][s][NP - 1] : lane_from_left(keep[R - 1][s][NP - 1]),
                                keep[r][s][0], a, dm[r], dp[r]);
          else if constexpr (!POS)
            flux_partials<PHYS>(0.0, 0.0, a, dm[r], dp[r]);
        }
        // the right face of element R - 1 is the next lane's first
        const double last = lane_from_right(POS ? g[0] : raw[0] * dm[0]);
#pragma unroll
        for (int r = 0; r < R; ++r) {
          double mu[NP];
#pragma unroll
          for (int j = 0; j < NP; ++j) mu[j] = 0.0;
          fmac_operator<NP>(opt, lk[r], mu);
          if constexpr (NL)
#pragma unroll
            for (int j = 0; j < NP; ++j) mu[j] = (2.0 * keep[r][s][j]) * mu[j];
          const int rn = r + 1 < R ? r + 1 : r;
          if constexpr (POS) {
            mu[NP - 1] = fma(a, r + 1 < R ? g[rn] : last, mu[NP - 1]);
          } else {
            mu[0] = fma(raw[r], dp[r], mu[0]);
            mu[NP - 1] += r + 1 < R ? raw[rn] * dm[rn] : last;
          }
#pragma unroll
          for (int j = 0; j < NP; ++j) lu[r][j] += mu[j];
#pragma unroll
          for (int j = 0; j < NP; ++j) mus[r][s][j] = mu[j];
          if constexpr (SPEED) {
#pragma unroll
            for (int i = 0; i < NP; ++i) ca[r] = fma(lk[r][i], keep[r][s][i], ca[r]);
            // here and not, with its operands kept, in the branch that uses it
            asm volatile("" : "+v"(ca[r]));
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }

      // the next step's state: not ahead of the stages, where its registers cost
      // a wave per SIMD (as would the old one's, if it stayed after the last step)
      if constexpr (FWD) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int j = 0; j < NP; ++j) un[r][j] = 0.0;
        if (t > 0) we.load(P, state(t - 1), un);
      }
      if constexpr (SPEED) {
        if (lane_owned)
#pragma unroll
          for (int r = 0; r < R; ++r) parts[R * (lane - HL) + r] = r < we.own_n ? ca[r] : 0.0;
        // the butterfly's first exchange from LDS, then the halves apart
        const int i0 = (lane & 31) - S, i1 = i0 + 32, o = (lane >> 5) * T1;
        const bool half = (lane >> 5) < R;
        double cs = (half && i0 >= 0 ? parts[o + i0] : 0.0) + (half && i1 < T1 ? parts[o + i1] : 0.0);
#pragma unroll
        for (int x = 16; x > 0; x >>= 1) cs += __shfl_xor(cs, x, kWave);
        c_sum += cs / a;
      }
      if constexpr (PE) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
          for (int j = 0; j < NP; ++j) asm volatile("" : "+v"(lu[r][j]));
        wf.pass_on(P, K, t, lane);
      }
    }
  };
  // one loop after the other, of which one takes all steps (as in stage_tile)
  steps(std::true_type{}, wf.m_pe ? 0 : K);
  steps(std::false_type{}, 0);

  we.store(P, lamo, lu);
  if constexpr (SPEED)
    if (c_lane) cpart[P.part_off + part] = c_sum;
  wf.keep(P, adjring, K, lane);
}

}  // namespace adg
