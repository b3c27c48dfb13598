// Fused step kernels: one wave64 per tile, all RK stages of the steps of a
// launch on chip.  Compiled once per integrator (-DADG_RK=0 .. 4) so that the
// instantiations build in parallel.
#include "adg_linear.hpp"
#include "adg_stage.hpp"

#ifndef ADG_RK
#error "compile once per integrator with -DADG_RK=0, 1, 2, 3 or 4"
#endif

namespace adg {

extern __shared__ double wave_lds[];

template <int NP, int RK, int PHYS, int R>
__global__ __launch_bounds__(kBlock) void k_fused_step(const DevProblem* __restrict__ probs,
                                                       const WorkItem* __restrict__ work,
                                                       const StepClock clock, double* __restrict__ ring,
                                                       int32_t w_begin, int32_t w_end,
                                                       const double* __restrict__ uin, double* __restrict__ uout,
                                                       double* __restrict__ umid, int64_t mid_stride,
                                                       int32_t step_offset, int32_t K, int32_t HL, int32_t n_faces_max,
                                                       int32_t lds_words, int32_t single_prob) {
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int lane = (int)(threadIdx.x % kWave);
  const int w = w_begin + xcd_block((int)blockIdx.x, (int)gridDim.x) * kWavesPerBlock + wv;
  if (w >= w_end) return;  // whole wave
  const int64_t n = clock.tick(w == w_begin) + step_offset;
  // a range holding one problem lists its tiles in order: no work-list load
  const WorkItem wi = single_prob >= 0 ? WorkItem{single_prob, w - w_begin} : work[w];
  stage_tile<NP, RK, PHYS, R>(probs[wi.prob], wi, ring, n, K, HL, uin, uout, umid, mid_stride, n_faces_max,
                              wave_lds + wv * lds_words, lane);
}

// One launch over every degree range (ADG_OPT_ONE_LAUNCH): wave w finds its
// range from the range table (ranges are contiguous in the work list, in the
// order of the per-range launches) and runs that range's tile.  A kernel's
// registers are those of its largest body, so every range runs at the
// occupancy of the degree-4 tile; one launch per range (the default) lets each
// degree keep its own.  The per-element arithmetic is that of the per-range
// kernels: the results are bitwise the same.
struct FusedRangeTable {
  int32_t group[kFusedRanges + 1];
  int32_t n_faces, lds_words;  // the most over the ranges
};

template <int RK, int PHYS, int R>
__global__ __launch_bounds__(kBlock) void k_fused_all(const DevProblem* __restrict__ probs,
                                                      const double* __restrict__ lin,
                                                      const WorkItem* __restrict__ work,
                                                      const StepClock clock, double* __restrict__ ring,
                                                      const FusedRangeTable rt, const double* __restrict__ uin,
                                                      double* __restrict__ uout, double* __restrict__ umid,
                                                      int64_t mid_stride, int32_t step_offset, int32_t K, int32_t HL) {
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int lane = (int)(threadIdx.x % kWave);
  const int w = xcd_block((int)blockIdx.x, (int)gridDim.x) * kWavesPerBlock + wv;
  if (w >= rt.group[kFusedRanges]) return;  // whole wave
  const int64_t n = clock.tick(w == 0) + step_offset;
  const WorkItem wi = work[w];
  const DevProblem& P = probs[wi.prob];
  double* lds = wave_lds + wv * rt.lds_words;
  int gi = 0;  // uniform
#pragma unroll
  for (int g = 1; g < kFusedRanges; ++g) gi += w >= rt.group[g] ? 1 : 0;
  const int form = gi % kForms;
  auto tile = [&](auto np_) {
    constexpr int NP = decltype(np_)::value;
    // the linear form and the a > 0 upwind form exist for upwind advection only
    if constexpr (PHYS == PHYS_ADV_UPWIND) {
      if (form == FORM_LIN)
        return lin_tile<NP, rk_stages(RK), R>(P, lin + P.lin_off, wi, ring, n, K, HL, uin, uout, rt.n_faces, lds, lane);
      if (form == FORM_POS)
        return stage_tile<NP, RK, PHYS_ADV_UPWIND_POS, R>(P, wi, ring, n, K, HL, uin, uout, umid, mid_stride,
                                                          rt.n_faces, lds, lane);
    }
    stage_tile<NP, RK, PHYS, R>(P, wi, ring, n, K, HL, uin, uout, umid, mid_stride, rt.n_faces, lds, lane);
  };
  switch (gi / kForms) {  // np = 5, 4, 3, 2
    case 0: tile(std::integral_constant<int, 5>{}); break;
    case 1: tile(std::integral_constant<int, 4>{}); break;
    case 2: tile(std::integral_constant<int, 3>{}); break;
    default: tile(std::integral_constant<int, 2>{}); break;
  }
}

// Viscous Burgers in local DG form (Sec. 7): K in {1, 2} time steps per
// launch, R in {1, 2, 4} consecutive elements per lane, halo of K S elements
// per side.  Per stage: u-hat at a face is the trace of the element on its
// left (alternating flux); q = Kr u-hat_right - Kl u-hat_left - Kd u; the
// total flux at a face is G = LLF(u-, u+) - nu q+ with q+ from the element on
// its right; the element update is Kl G_left - Kr G_right + Kd (u^2/2 - nu q).
// u-hat_left comes from the element on the left (the left lane's last element
// by a lane shift) and u-hat_right is the element's own trace, so q needs no
// data from the right; G_right comes from the element on the right.  Each
// stage then depends on one element to either side, as the inviscid update
// does, and every element takes the same operations whatever R.  At a PE
// face the element right of it writes the raw level-m u-hat and G to their
// rings; the element holding the face as its left face takes the AT
// combinations of past levels of both, and the element holding it as its
// right face the u-hat combination.  The levels before n were written by
// earlier launches, so these sums are formed at the start of the launch; for
// the second step a delay of 1 also needs level n, which each lane adds from
// its own raw values (the left-face u-hat and G it computes, and for the
// right face its own trace, which is that face's u-hat).  A PE size of at
// least R gives a lane at most one PE face as some element's left face and
// at most one as some element's right face, so the per-lane LDS slots below
// hold each kind once.
template <int S, int K>
struct LdgSmem {
  double atu[K][kWavesPerBlock][S][kWave];   // left face: u-hat
  double atg[K][kWavesPerBlock][S][kWave];   // left face: G
  double atur[K][kWavesPerBlock][S][kWave];  // right face: u-hat
  uint8_t kl[K][kWavesPerBlock][S][kWave];   // delays of the left face
  uint8_t kr[K][kWavesPerBlock][S][kWave];   // delays of the right face
};

template <int NP, int RK, int K, int R>
__device__ __forceinline__ void wave_tile_ldg(const DevProblem& P, const WorkItem wi, double* __restrict__ ring,
                                              int64_t n, const double* __restrict__ uin, double* __restrict__ uout,
                                              LdgSmem<rk_stages(RK), K>& sm, int wv, int lane) {
#pragma clang fp contract(off)  // explicit FMAs only
  constexpr int S = rk_stages(RK);
  constexpr int HL = fused_halo(RK, R, K);
  constexpr int T = fused_tile(RK, R, K);
  const int N = (int)P.n_elem;
  const int e0 = wi.tile * T;
  const int teff = (N - e0) < T ? (N - e0) : T;
  const int xb = e0 - R * HL;  // element position of lane 0, element 0 (a multiple of R)
  const bool lane_owned = lane >= HL && lane < kWave - HL;
  const bool tiny = N < kWave * R;  // the wave's extent may wrap more than once
  int e[R];
  bool owned[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int x = xb + R * lane + r;
    e[r] = tiny ? wrap_elem(x, N) : wrap_once(x, N);
    owned[r] = lane_owned && (x - e0) < teff;
  }
  // with N a multiple of R a lane's elements never straddle the periodic
  // wrap: its planes move as 16-byte pieces through a buffer resource
  const bool buffered = R > 1 && (N % R) == 0 && (int64_t)P.np * P.ld < (int64_t)1 << 28;
  const int voff = e[0] * 8;
  const int64_t ld = P.ld;
  const double* __restrict__ u = uin + P.u_off;
  double u0[R][NP];
  if (buffered) {
    const __amdgpu_buffer_rsrc_t rs = plane_rsrc(u);
#pragma unroll
    for (int j = 0; j < NP; ++j)
#pragma unroll
      for (int r = 0; r < R; r += 2) {
        const double2 v = __builtin_bit_cast(double2,
                                             __builtin_amdgcn_raw_buffer_load_b128(rs, voff + 8 * r, (int)(8 * j * ld), 0));
        u0[r][j] = v.x;
        u0[r + 1 < R ? r + 1 : r][j] = v.y;  // R >= 2 here
      }
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
      for (int j = 0; j < NP; ++j) u0[r][j] = u[j * ld + e[r]];
  }

  bool pe[R];    // the left face of element r is a PE face
  bool per[R];   // the right face of element r is a PE face
  bool pe_any = false, per_any = false;
  uint32_t b = 0, br = 0;  // the lane's PE face of each kind
  int depth = 1, slot_n = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) pe[r] = per[r] = false;
  if (P.async_faces) {
    depth = P.depth;
    const uint32_t n32 = (uint32_t)n;  // step indices stay below 2^31
    slot_n = (int)(n32 - fast_div(n32, P.depth_div) * (uint32_t)depth);
    const uint32_t pes = P.pe_div.d;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const uint32_t bl = fast_div((uint32_t)e[r], P.pe_div);
      pe[r] = (uint32_t)e[r] == bl * pes;
      if (pe[r]) b = bl;
      const uint32_t e1 = (e[r] + 1 == N) ? 0u : (uint32_t)(e[r] + 1);
      const uint32_t b1 = fast_div(e1, P.pe_div);
      per[r] = e1 == b1 * pes;
      if (per[r]) br = b1;
      pe_any = pe_any || pe[r];
      per_any = per_any || per[r];
    }
  }
  // The delays and the AT sums over the levels before n, one job lane per
  // (PE lane, step, stage, value): the left-face u-hat and G of each lane with
  // a PE left face, the right-face u-hat of each lane with a PE right face.
  // Each job draws its delay and sums its past levels; the target lane reads
  // both from LDS.
  constexpr int KS = K * S;
  const uint64_t m_l = __ballot(pe_any), m_r = __ballot(per_any);
  const int n_l = 2 * KS * __builtin_popcountll(m_l);
  const int n_jobs = n_l + KS * __builtin_popcountll(m_r);
  for (int g0 = 0; g0 < n_jobs; g0 += kWave) {  // uniform
    const int g = g0 + lane;
    const bool left = g < n_l;
    const int h = left ? g : g - n_l;
    const int per_face = left ? 2 * KS : KS;
    const int i = h / per_face, r = h - i * per_face;
    const int v = left ? r / KS : 2;  // 0: u-hat, 1: G (left face); 2: u-hat (right face)
    const int rr = r - (left ? v * KS : 0);
    const int kk = rr / S, s = rr - kk * S;
    const int tl = nth_set_lane(m_l, i), tr = nth_set_lane(m_r, i);
    const uint32_t fl = (uint32_t)__shfl((int)b, tl), fr = (uint32_t)__shfl((int)br, tr);  // every lane active
    if (g < n_jobs) {
      const int tgt = left ? tl : tr;
      const uint32_t face = left ? fl : fr;
      const int kd = pe_delay(P, n + kk, s, face);
      const double* __restrict__ rb = ring + (v == 1 ? P.ring_off : P.ring2_off) + ((int64_t)face * S + s) * depth;
      const double val = at_old_levels(P, rb, kk, kd, slot_n, depth);
      if (v == 0) {
        sm.atu[kk][wv][s][tgt] = val;
        sm.kl[kk][wv][s][tgt] = (uint8_t)kd;
      } else if (v == 1) {
        sm.atg[kk][wv][s][tgt] = val;
      } else {
        sm.atur[kk][wv][s][tgt] = val;
        sm.kr[kk][wv][s][tgt] = (uint8_t)kd;
      }
    }
  }

  double y[R][NP], ks[R][NP], k[NP], q[R][NP];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int j = 0; j < NP; ++j) y[r][j] = u0[r][j];
  const double nu = P.nu;
  const double dt = P.dt;
  int slot_m = slot_n;
#pragma unroll
  for (int kk = 0; kk < K; ++kk) {
    if (kk > 0) {
      slot_m = slot_m + 1 == depth ? 0 : slot_m + 1;
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int j = 0; j < NP; ++j) u0[r][j] = y[r][j];
    }
#pragma unroll
    for (int s = 0; s < S; ++s) {
      const int64_t rs = ((int64_t)b * S + s) * depth + slot_m;
      double um[R], G[R];
      const double um0 = lane_from_left(y[R - 1][NP - 1]);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        um[r] = r == 0 ? um0 : y[r - 1][NP - 1];  // u- at the left face, and its u-hat
        double hl = um[r];
        if (pe[r]) {
          if (owned[r]) ring[P.ring2_off + rs] = um[r];
          if constexpr (K == 2) {  // level n completes step n+1's u-hat sum when its delay is 1
            if (kk == 0 && sm.kl[1][wv][s][lane] == 1)
              sm.atu[1][wv][s][lane] = fma(P.atc[1][0], um[r], sm.atu[1][wv][s][lane]);
          }
          if (sm.kl[kk][wv][s][lane] != 0) hl = sm.atu[kk][wv][s][lane];
        }
        double hr = y[r][NP - 1];  // u-hat at the right face: this element's own trace
        if (per[r]) {
          if constexpr (K == 2) {
            if (kk == 0 && sm.kr[1][wv][s][lane] == 1)
              sm.atur[1][wv][s][lane] = fma(P.atc[1][0], hr, sm.atur[1][wv][s][lane]);
          }
          if (sm.kr[kk][wv][s][lane] != 0) hr = sm.atur[kk][wv][s][lane];
        }
#pragma unroll
        for (int i = 0; i < NP; ++i) {
          double v = fma(-P.Kl[i], hl, P.Kr[i] * hr);
#pragma unroll
          for (int j = 0; j < NP; ++j) v = fma(-P.Kd[i * kMaxNp + j], y[r][j], v);
          q[r][i] = v;
        }
      }
#pragma unroll
      for (int r = 0; r < R; ++r) {
        G[r] = fma(-nu, q[r][0], Physics<PHYS_BURGERS_LLF>::fhat(um[r], y[r][0], 1.0));
        if (pe[r]) {
          if (owned[r]) ring[P.ring_off + rs] = G[r];
          if constexpr (K == 2) {
            if (kk == 0 && sm.kl[1][wv][s][lane] == 1)
              sm.atg[1][wv][s][lane] = fma(P.atc[1][0], G[r], sm.atg[1][wv][s][lane]);
          }
          if (sm.kl[kk][wv][s][lane] != 0) G[r] = sm.atg[kk][wv][s][lane];
        }
      }
      const double Gr_last = lane_from_right(G[0]);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const double Gr = r + 1 < R ? G[r + 1] : Gr_last;
        double g[NP];
#pragma unroll
        for (int j = 0; j < NP; ++j) g[j] = fma(0.5 * y[r][j], y[r][j], -nu * q[r][j]);
#pragma unroll
        for (int i = 0; i < NP; ++i) {
          double v = fma(-P.Kr[i], Gr, P.Kl[i] * G[r]);
#pragma unroll
          for (int j = 0; j < NP; ++j) v = fma(P.Kd[i * kMaxNp + j], g[j], v);
          k[i] = v;
        }
        rk_update<NP, RK>(s, dt, u0[r], y[r], ks[r], k);
      }
    }
  }
  bool all_owned = true;
#pragma unroll
  for (int r = 0; r < R; ++r) all_owned = all_owned && owned[r];
  double* __restrict__ uo = uout + P.u_off;
  if (buffered && all_owned) {
    const __amdgpu_buffer_rsrc_t rs = plane_rsrc(uo);
#pragma unroll
    for (int j = 0; j < NP; ++j)
#pragma unroll
      for (int r = 0; r < R; r += 2) {
        double2 v;
        v.x = y[r][j];
        v.y = y[r + 1 < R ? r + 1 : r][j];
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(BufWord4, v), rs, voff + 8 * r, (int)(8 * j * ld), 0);
      }
  } else {
#pragma unroll
    for (int r = 0; r < R; ++r)
      if (owned[r])
#pragma unroll
        for (int j = 0; j < NP; ++j) uo[j * ld + e[r]] = y[r][j];
  }
}

template <int NP, int RK, int K, int R>
__global__ __launch_bounds__(kBlock) void k_fused_ldg(const DevProblem* __restrict__ probs,
                                                      const WorkItem* __restrict__ work,
                                                      const StepClock clock, double* __restrict__ ring,
                                                      int32_t w_begin, int32_t w_end, const double* __restrict__ uin,
                                                      double* __restrict__ uout, int32_t step_offset,
                                                      int32_t single_prob) {
  __shared__ LdgSmem<rk_stages(RK), K> sm;
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int lane = (int)(threadIdx.x % kWave);
  const int w = w_begin + xcd_block((int)blockIdx.x, (int)gridDim.x) * kWavesPerBlock + wv;
  if (w >= w_end) return;  // whole wave
  const int64_t n = clock.tick(w == w_begin) + step_offset;
  const WorkItem wi = single_prob >= 0 ? WorkItem{single_prob, w - w_begin} : work[w];
  wave_tile_ldg<NP, RK, K, R>(probs[wi.prob], wi, ring, n, uin, uout, sm, wv, lane);
}

template <int NP, int RK, int R>
static void fused_ldg_go_r(const StepArgs& a, int gi, const double* uin, double* uout, int32_t off, hipStream_t st) {
  if (a.steps == 2)
    hipLaunchKernelGGL((k_fused_ldg<NP, RK, 2, R>), dim3(a.grid[gi]), dim3(kBlock), 0, st, a.probs, a.work, a.clock,
                       a.ring, a.group[gi], a.group[gi + 1], uin, uout, off, a.single[gi]);
  else
    hipLaunchKernelGGL((k_fused_ldg<NP, RK, 1, R>), dim3(a.grid[gi]), dim3(kBlock), 0, st, a.probs, a.work, a.clock,
                       a.ring, a.group[gi], a.group[gi + 1], uin, uout, off, a.single[gi]);
}

template <int NP, int RK>
static void fused_ldg_go(const StepArgs& a, int gi, const double* uin, double* uout, int32_t off, hipStream_t st) {
  switch (a.elems) {
    case 2: fused_ldg_go_r<NP, RK, 2>(a, gi, uin, uout, off, st); break;
    case 4: fused_ldg_go_r<NP, RK, 4>(a, gi, uin, uout, off, st); break;
    default: fused_ldg_go_r<NP, RK, 1>(a, gi, uin, uout, off, st); break;
  }
}

template <int RK>
static void fused_ldg_np(const StepArgs& a, const double* uin, double* uout, int32_t off, hipStream_t st) {
  for (int gi = 0; gi < kFusedRanges; ++gi) {
    if (a.group[gi + 1] <= a.group[gi]) continue;
    switch (gi / kForms) {  // np = 5, 4, 3, 2
      case 0: fused_ldg_go<5, RK>(a, gi, uin, uout, off, st); break;
      case 1: fused_ldg_go<4, RK>(a, gi, uin, uout, off, st); break;
      case 2: fused_ldg_go<3, RK>(a, gi, uin, uout, off, st); break;
      default: fused_ldg_go<2, RK>(a, gi, uin, uout, off, st); break;
    }
  }
}

template <int NP, int RK, int PHYS, int R>
static void fused_go_r(const StepArgs& a, int gi, const double* uin, double* uout, int32_t off, hipStream_t st) {
  const FaceRange& fr = a.faces[gi];
  hipLaunchKernelGGL((k_fused_step<NP, RK, PHYS, R>), dim3(a.grid[gi]), dim3(kBlock),
                     8 * kWavesPerBlock * fr.lds_words, st, a.probs, a.work, a.clock, a.ring, a.group[gi],
                     a.group[gi + 1], uin, uout, a.umid, a.mid_stride, off, a.steps, a.halo, fr.n_faces, fr.lds_words,
                     a.single[gi]);
}

template <int NP, int RK, int PHYS>
static void fused_go(const StepArgs& a, int gi, const double* uin, double* uout, int32_t off, hipStream_t st) {
  switch (a.elems) {
    case 1: fused_go_r<NP, RK, PHYS, 1>(a, gi, uin, uout, off, st); break;
    case 4: fused_go_r<NP, RK, PHYS, 4>(a, gi, uin, uout, off, st); break;
    default: fused_go_r<NP, RK, PHYS, 2>(a, gi, uin, uout, off, st); break;
  }
}

template <int NP, int RK, int PHYS>
static void fused_form(const StepArgs& a, int gi, const double* uin, double* uout, int32_t off, hipStream_t st) {
  if constexpr (PHYS == PHYS_ADV_UPWIND) {
    if (gi % kForms == FORM_LIN) return launch_lin_s<rk_stages(RK)>(a, gi, uin, uout, off, st);
    if (gi % kForms == FORM_POS) return fused_go<NP, RK, PHYS_ADV_UPWIND_POS>(a, gi, uin, uout, off, st);
  }
  fused_go<NP, RK, PHYS>(a, gi, uin, uout, off, st);
}

template <int RK, int PHYS>
static void fused_np(const StepArgs& a, const double* uin, double* uout, int32_t off, hipStream_t st) {
  for (int gi = 0; gi < kFusedRanges; ++gi) {
    if (a.group[gi + 1] <= a.group[gi]) continue;
    switch (gi / kForms) {  // np = 5, 4, 3, 2
      case 0: fused_form<5, RK, PHYS>(a, gi, uin, uout, off, st); break;
      case 1: fused_form<4, RK, PHYS>(a, gi, uin, uout, off, st); break;
      case 2: fused_form<3, RK, PHYS>(a, gi, uin, uout, off, st); break;
      default: fused_form<2, RK, PHYS>(a, gi, uin, uout, off, st); break;
    }
  }
}

template <int RK>
static void fused_phys(int phys, const StepArgs& a, const double* uin, double* uout, int32_t off, hipStream_t st) {
  switch (phys) {
    case PHYS_ADV_UPWIND: fused_np<RK, PHYS_ADV_UPWIND>(a, uin, uout, off, st); break;
    case PHYS_ADV_CENTRAL: fused_np<RK, PHYS_ADV_CENTRAL>(a, uin, uout, off, st); break;
    case PHYS_BURGERS_LDG: fused_ldg_np<RK>(a, uin, uout, off, st); break;
    default: fused_np<RK, PHYS_BURGERS_LLF>(a, uin, uout, off, st); break;
  }
}

// ADG_OPT_ONE_LAUNCH: one launch over every range (two elements per lane, or
// one where a PE size is odd).
template <int RK, int PHYS>
static void fused_all_go(const StepArgs& a, const double* uin, double* uout, int32_t off, hipStream_t st) {
  FusedRangeTable rt;
  for (int i = 0; i <= kFusedRanges; ++i) rt.group[i] = a.group[i];
  rt.n_faces = rt.lds_words = 0;
  for (int i = 0; i < kFusedRanges; ++i) {
    rt.n_faces = a.faces[i].n_faces > rt.n_faces ? a.faces[i].n_faces : rt.n_faces;
    rt.lds_words = a.faces[i].lds_words > rt.lds_words ? a.faces[i].lds_words : rt.lds_words;
  }
  const dim3 g(fused_grid(a.group[kFusedRanges])), b(kBlock);
  const size_t lds = 8 * (size_t)(kWavesPerBlock * rt.lds_words);
  if (a.elems == 2)
    hipLaunchKernelGGL((k_fused_all<RK, PHYS, 2>), g, b, lds, st, a.probs, a.lin, a.work, a.clock, a.ring, rt, uin, uout,
                       a.umid, a.mid_stride, off, a.steps, a.halo);
  else
    hipLaunchKernelGGL((k_fused_all<RK, PHYS, 1>), g, b, lds, st, a.probs, a.lin, a.work, a.clock, a.ring, rt, uin, uout,
                       a.umid, a.mid_stride, off, a.steps, a.halo);
}

template <int RK>
hipError_t launch_fused_rk(int phys, const StepArgs& a, const double* uin, double* uout, int32_t step_offset,
                           hipStream_t stream) {
  if (a.one_launch) {
    if (a.elems > 2 || phys == PHYS_BURGERS_LDG) return hipErrorInvalidValue;
    switch (phys) {
      case PHYS_ADV_UPWIND: fused_all_go<RK, PHYS_ADV_UPWIND>(a, uin, uout, step_offset, stream); break;
      case PHYS_ADV_CENTRAL: fused_all_go<RK, PHYS_ADV_CENTRAL>(a, uin, uout, step_offset, stream); break;
      default: fused_all_go<RK, PHYS_BURGERS_LLF>(a, uin, uout, step_offset, stream); break;
    }
    return hipGetLastError();
  }
  fused_phys<RK>(phys, a, uin, uout, step_offset, stream);
  return hipGetLastError();
}

template hipError_t launch_fused_rk<ADG_RK>(int, const StepArgs&, const double*, double*, int32_t, hipStream_t);

}  // namespace adg
