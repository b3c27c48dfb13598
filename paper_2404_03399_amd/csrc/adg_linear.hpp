// Tile of the fused step of linear advection with the upwind flux and a > 0,
// in flux-sequence form (device code shared by its own launch and by the
// launch over every range).
#pragma once

#include <type_traits>

#include "adg_device.hpp"

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
// AT combination of delayed levels where the drawn delay is not 0; the
// element left of the face then takes the difference delta_s between applied
// and raw flux through WR and Psi.  R divides every PE size, so that a PE face
// is always the left face of a lane's first element: waves with and without
// faces run two step loops without any further branch.  Every
// wave that holds a face (its owner's and
// those with the face in their halo, which see bitwise the same raw fluxes)
// draws its delays and sums the ring levels before the launch itself, one job
// lane per (face, step, stage) while the state loads are in flight; the
// levels of the launch are added after each step from the raw fluxes kept in
// LDS.  The ring is written once, at the end, by the owner waves: with a depth
// of at least L + q + K - 2 no level that a wave of the launch reads shares a
// slot with one written in it.
//
// Every element takes the same operations in the same order whatever the
// lanes' element count R, the steps per launch and the wave it is in (explicit
// FMAs, contraction off), so all launch shapes agree bitwise.

// Per-wave LDS of a launch of K steps with up to n_faces PE faces; a job is
// g = (face K + step) S + stage:
//   atc [kMaxL][kMaxQ]     the problem's AT weights
//   at  [job]              sum over the levels before the launch, then with the
//                          launch's levels, then the raw flux of that step
//   kd  [face][step] word  delays, byte s = stage s
//   own [face] word        1 if the wave owns the element right of it
// and S doubles after the jobs that lanes without a face write to.
struct LinLds {
  double* atc;
  double* at;
  RecWord* kd;
  RecWord* own;
};

__device__ __forceinline__ int lane_rank(uint64_t mask) {  // set bits below this lane
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// a[i] += c(lane L + i of each row of 16) * x, i < M: v_fmac_f64 with the
// DPP row_newbcast control, which reads one lane's value in all lanes of a
// row, so that a table sits in one register pair per 16 entries and no
// coefficient is loaded, moved or kept in SGPRs inside the step loop.  Every
// lane of the wave must be active.  The leading s_nop covers the two wait
// states that DPP needs after a VALU write of c, should the compiler copy it
// right before the block.
template <int L, int M>
__device__ __forceinline__ void fmac_bcast(double c, double x, double* const (&a)[M]) {
#define ADG_FM(i) "v_fmac_f64_dpp %" #i ", %[c], %[x] row_newbcast:%[l" #i "] row_mask:0xf bank_mask:0xf\n\t"
#define ADG_IN [c] "v"(c), [x] "v"(x), [l0] "n"(L)
  static_assert(M >= 1 && M <= 9 && L >= 0 && L + M <= 16, "a column lies within one run of 16");
  if constexpr (M == 1)
    asm("s_nop 1\n\t" ADG_FM(0) : "+v"(*a[0]) : ADG_IN);
  else if constexpr (M == 2)
    asm("s_nop 1\n\t" ADG_FM(0) ADG_FM(1) : "+v"(*a[0]), "+v"(*a[1]) : ADG_IN, [l1] "n"(L + 1));
  else if constexpr (M == 3)
    asm("s_nop 1\n\t" ADG_FM(0) ADG_FM(1) ADG_FM(2)
        : "+v"(*a[0]), "+v"(*a[1]), "+v"(*a[2])
        : ADG_IN, [l1] "n"(L + 1), [l2] "n"(L + 2));
  else if constexpr (M == 4)
    asm("s_nop 1\n\t" ADG_FM(0) ADG_FM(1) ADG_FM(2) ADG_FM(3)
        : "+v"(*a[0]), "+v"(*a[1]), "+v"(*a[2]), "+v"(*a[3])
        : ADG_IN, [l1] "n"(L + 1), [l2] "n"(L + 2), [l3] "n"(L + 3));
  else if constexpr (M == 5)
    asm("s_nop 1\n\t" ADG_FM(0) ADG_FM(1) ADG_FM(2) ADG_FM(3) ADG_FM(4)
        : "+v"(*a[0]), "+v"(*a[1]), "+v"(*a[2]), "+v"(*a[3]), "+v"(*a[4])
        : ADG_IN, [l1] "n"(L + 1), [l2] "n"(L + 2), [l3] "n"(L + 3), [l4] "n"(L + 4));
  else if constexpr (M == 6)
    asm("s_nop 1\n\t" ADG_FM(0) ADG_FM(1) ADG_FM(2) ADG_FM(3) ADG_FM(4) ADG_FM(5)
        : "+v"(*a[0]), "+v"(*a[1]), "+v"(*a[2]), "+v"(*a[3]), "+v"(*a[4]), "+v"(*a[5])
        : ADG_IN, [l1] "n"(L + 1), [l2] "n"(L + 2), [l3] "n"(L + 3), [l4] "n"(L + 4), [l5] "n"(L + 5));
  else if constexpr (M == 7)
    asm("s_nop 1\n\t" ADG_FM(0) ADG_FM(1) ADG_FM(2) ADG_FM(3) ADG_FM(4) ADG_FM(5) ADG_FM(6)
        : "+v"(*a[0]), "+v"(*a[1]), "+v"(*a[2]), "+v"(*a[3]), "+v"(*a[4]), "+v"(*a[5]), "+v"(*a[6])
        : ADG_IN, [l1] "n"(L + 1), [l2] "n"(L + 2), [l3] "n"(L + 3), [l4] "n"(L + 4), [l5] "n"(L + 5),
          [l6] "n"(L + 6));
  else if constexpr (M == 8)
    asm("s_nop 1\n\t" ADG_FM(0) ADG_FM(1) ADG_FM(2) ADG_FM(3) ADG_FM(4) ADG_FM(5) ADG_FM(6) ADG_FM(7)
        : "+v"(*a[0]), "+v"(*a[1]), "+v"(*a[2]), "+v"(*a[3]), "+v"(*a[4]), "+v"(*a[5]), "+v"(*a[6]), "+v"(*a[7])
        : ADG_IN, [l1] "n"(L + 1), [l2] "n"(L + 2), [l3] "n"(L + 3), [l4] "n"(L + 4), [l5] "n"(L + 5),
          [l6] "n"(L + 6), [l7] "n"(L + 7));
  else
    asm("s_nop 1\n\t" ADG_FM(0) ADG_FM(1) ADG_FM(2) ADG_FM(3) ADG_FM(4) ADG_FM(5) ADG_FM(6) ADG_FM(7) ADG_FM(8)
        : "+v"(*a[0]), "+v"(*a[1]), "+v"(*a[2]), "+v"(*a[3]), "+v"(*a[4]), "+v"(*a[5]), "+v"(*a[6]), "+v"(*a[7]),
          "+v"(*a[8])
        : ADG_IN, [l1] "n"(L + 1), [l2] "n"(L + 2), [l3] "n"(L + 3), [l4] "n"(L + 4), [l5] "n"(L + 5),
          [l6] "n"(L + 6), [l7] "n"(L + 7), [l8] "n"(L + 8));
#undef ADG_FM
#undef ADG_IN
}

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
// 0 elsewhere); at: its AT sums; raw: where it keeps the raw fluxes of the step
// (lanes without a face have a place of their own, so that no branch cuts the
// stages into blocks: with one the kernel took 167 registers instead of 137).
template <int NP, int S, int R, bool PE, int s = 0>
__device__ __forceinline__ void lin_stages(const double (&tab)[lin_tab_size(NP, S) / 16], double (&F)[R][S],
                                           double (&u)[R][NP], RecWord kd, const double (&at)[S],
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
      const bool sel = (kd & ((RecWord)0xff << (8 * s))) != 0;
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
  const int N = (int)P.n_elem;
  const int HR = P.async_faces ? 1 : 0;
  const int TE = R * (kWave - HL - HR);  // owned elements of a tile
  const bool grouped = R > 1 && (N % R) == 0;
  const int64_t ld = P.ld;
  const double* __restrict__ u_g = uin + P.u_off;
  const int e0 = wi.tile * TE;
  const int teff = (N - e0) < TE ? (N - e0) : TE;
  const int xb = e0 - R * HL;  // element position of lane 0, element 0 (a multiple of R)
  const bool lane_owned = lane >= HL && lane < kWave - HR;
  int e[R];
  int own_n = 0;  // owned elements of the lane: its first own_n
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int x = xb + R * lane + r;
    e[r] = wrap_once(x, N);  // the mesh holds more elements than a wave (kLinMinElems)
    own_n += lane_owned && (x - e0) < teff ? 1 : 0;
  }
  // the AT weights, ahead of the state in the queue of loads
  double atc = 0.0;
  if (P.async_faces && lane < kMaxL * kMaxQ) atc = P.atc[0][lane];
  double u[R][NP];
  // grouped lanes: 16-byte pieces through a buffer resource (planes below 2 GiB)
  const bool buffered = grouped && (int64_t)P.np * ld < (int64_t)1 << 28;
  const int voff = e[0] * 8;
  if (buffered) {
    const __amdgpu_buffer_rsrc_t rs = plane_rsrc(u_g);
#pragma unroll
    for (int j = 0; j < NP; ++j)
#pragma unroll
      for (int r = 0; r < R; r += 2) {
        const double2 v = __builtin_bit_cast(double2,
                                             __builtin_amdgcn_raw_buffer_load_b128(rs, voff + 8 * r, (int)(8 * j * ld), 0));
        u[r][j] = v.x;
        u[r + 1 < R ? r + 1 : r][j] = v.y;  // R >= 2 here
      }
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int j = 0; j < NP; ++j) u[r][j] = u_g[j * ld + e[r]];
  }

  // PE faces: the left face of element 0 of the lanes `pe` (R divides every PE size)
  bool pe = false;
  uint32_t b = 0;
  double* const lds_at = lds + kMaxL * kMaxQ;
  const LinLds sm{lds, lds_at, (RecWord*)(lds_at + n_faces_max * K * S + S),
                  (RecWord*)(lds_at + n_faces_max * (K * S + K) + S)};
  uint64_t m_pe = 0;
  int n_jobs = 0, depth = 1, slot_n = 0, slot = 0;
  uint32_t b0 = 0;
  if (P.async_faces) {
    depth = P.depth;
    const uint32_t n32 = (uint32_t)n;  // step indices stay below 2^31
    slot_n = (int)(n32 - fast_div(n32, P.depth_div) * (uint32_t)depth);
    b = fast_div((uint32_t)e[0], P.pe_div);
    pe = (uint32_t)e[0] == b * P.pe_div.d;
    m_pe = __ballot(pe);
    slot = lane_rank(m_pe);
    // the wave's elements are consecutive on the periodic mesh, so its faces are too
    b0 = (uint32_t)__builtin_amdgcn_readlane((int)b, m_pe ? __builtin_ctzll(m_pe) : 0);
    n_jobs = K * S * __builtin_popcountll(m_pe);
    if (pe) sm.own[slot] = own_n > 0 ? 1 : 0;
    if (lane < kMaxL * kMaxQ) sm.atc[lane] = atc;
  }
  const uint32_t kshift = (uint32_t)__builtin_ctz((uint32_t)K);  // K is a power of two
  for (int g0 = 0; g0 < n_jobs; g0 += kWave) {  // uniform
    const int g = g0 + lane;
    if (g < n_jobs) {
      const int ik = g / S, s = g - ik * S, i = ik >> kshift, kk = ik - (i << kshift);
      uint32_t bo = b0 + (uint32_t)i;
      bo -= bo >= (uint32_t)P.n_pe ? (uint32_t)P.n_pe : 0u;
      const int kd = pe_delay(P, n + kk, s, bo);
      // levels n - back, back >= 1, of the sum (oldest first); the levels of
      // the launch follow after its steps
      const double* __restrict__ rb = ring + P.ring_off + ((int64_t)bo * S + s) * depth;
      double lv[kMaxQ];
#pragma unroll
      for (int j = 0; j < kMaxQ; ++j) {
        lv[j] = 0.0;
        if (j < P.q) {  // uniform
          const int back = kd + j - kk;
          if (kd > 0 && back > 0) lv[j] = rb[ring_slot(slot_n, back, depth)];
        }
      }
      reinterpret_cast<uint8_t*>(sm.kd + ik)[s] = (uint8_t)kd;
      double v = 0.0;
#pragma unroll
      for (int j = kMaxQ - 1; j >= 0; --j)
        if (j < P.q && kd > 0 && kd + j > kk) v = fma(sm.atc[kd * kMaxQ + j], lv[j], v);
      sm.at[g] = v;
    }
  }

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
      RecWord kd = 0;
      double* const mine = sm.at + ((pe ? slot : n_faces_max) * K + (pe ? kk : 0)) * S;
      if constexpr (PE) {
        kd = sm.kd[pe ? slot * K + kk : 0];
        kd = pe ? kd : 0;
#pragma unroll
        for (int s = 0; s < S; ++s) at[s] = mine[s];
      }
      lin_stages<NP, S, R, PE>(tab, F, u, kd, at, mine);
      if constexpr (PE) {
        // this step's raw fluxes enter the AT sums of the launch's later steps
        for (int g0 = 0; g0 < n_jobs && kk + 1 < K; g0 += kWave) {
          const int g = g0 + lane, ik = g / S, later = (ik & (K - 1)) - kk;  // steps to the job's own
          if (g < n_jobs && later > 0) {
            const int kd_g = reinterpret_cast<const uint8_t*>(sm.kd + ik)[g - ik * S], j = later - kd_g;
            if (kd_g > 0 && j >= 0 && j < P.q)
              sm.at[g] = fma(sm.atc[kd_g * kMaxQ + j], sm.at[g - later * S], sm.at[g]);
          }
        }
      }
    }
  };
  // one loop after the other, of which one takes all steps: as the two sides of
  // a branch the compiler keeps the state twice (137 registers instead of 103)
  steps(std::true_type{}, m_pe ? K : 0);
  steps(std::false_type{}, K);

  double* __restrict__ uo = uout + P.u_off;
  if (buffered && own_n == R) {
    const __amdgpu_buffer_rsrc_t rs = plane_rsrc(uo);
#pragma unroll
    for (int j = 0; j < NP; ++j)
#pragma unroll
      for (int r = 0; r < R; r += 2) {
        double2 v;
        v.x = u[r][j];
        v.y = u[r + 1 < R ? r + 1 : r][j];
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(BufWord4, v), rs, voff + 8 * r, (int)(8 * j * ld), 0);
      }
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (r < own_n)
#pragma unroll
        for (int j = 0; j < NP; ++j) uo[j * ld + e[r]] = u[r][j];
  }

  // the raw fluxes of the owned faces into the ring
  for (int g0 = 0; g0 < n_jobs; g0 += kWave) {
    const int g = g0 + lane;
    if (g < n_jobs) {
      const int ik = g / S, s = g - ik * S, i = ik >> kshift, kk = ik - (i << kshift);
      if (sm.own[i]) {
        uint32_t bo = b0 + (uint32_t)i;
        bo -= bo >= (uint32_t)P.n_pe ? (uint32_t)P.n_pe : 0u;
        int sl = slot_n + kk;
        while (sl >= depth) sl -= depth;
        ring[P.ring_off + ((int64_t)bo * S + s) * depth + sl] = sm.at[g];
      }
    }
  }
}

}  // namespace adg
