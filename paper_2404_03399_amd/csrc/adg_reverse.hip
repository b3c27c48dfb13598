// Fused reverse sweep (discrete adjoint), several steps per launch.  Compiled
// once per integrator (-DADG_RK=0 .. 4).
#include "adg_reverse.hpp"

#ifndef ADG_RK
#error "compile once per integrator with -DADG_RK=0, 1, 2, 3 or 4"
#endif

namespace adg {

extern __shared__ double wave_lds[];

struct AdjPtr {
  const double *u_n, *u_next;
  int64_t u_stride;
  const double *lam, *ring;
  double *lamo, *adjring, *cpart;
};

template <int NP, int RK, int PHYS, bool FWD, int R>
__global__ __launch_bounds__(kBlock) void k_adj_fused(const DevProblem* __restrict__ probs,
                                                      const WorkItem* __restrict__ work, int32_t w_begin,
                                                      int32_t w_end, const AdjPtr p, int32_t n, int32_t K, int32_t HL,
                                                      int32_t n_faces_max, int32_t lds_words, int32_t single_prob) {
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int lane = (int)(threadIdx.x % kWave);
  const int w = w_begin + xcd_block((int)blockIdx.x, (int)gridDim.x) * kWavesPerBlock + wv;
  if (w >= w_end) return;  // whole wave
  const WorkItem wi = single_prob >= 0 ? WorkItem{single_prob, w - w_begin} : work[w];
  adj_tile<NP, RK, PHYS, FWD, R>(probs[wi.prob], wi, n, K, HL, p.u_n, p.u_next, p.u_stride, p.lam, p.lamo, p.ring,
                                 p.adjring, p.cpart, n_faces_max, wave_lds + wv * lds_words, lane);
}

template <int NP, int RK, int PHYS, bool FWD, int R>
static void adj_go(const AdjArgs& a, int gi, const AdjPtr& p, int32_t n, hipStream_t st) {
  const FaceRange& fr = a.faces[gi];
  hipLaunchKernelGGL((k_adj_fused<NP, RK, PHYS, FWD, R>), dim3(a.grid[gi]), dim3(kBlock),
                     8 * kWavesPerBlock * fr.lds_words, st, a.probs, a.work, a.group[gi], a.group[gi + 1], p, n,
                     a.steps, a.halo, fr.n_faces, fr.lds_words, a.single[gi]);
}

template <int NP, int RK, int PHYS, bool FWD>
static void adj_elems(const AdjArgs& a, int gi, const AdjPtr& p, int32_t n, hipStream_t st) {
  if constexpr (!FWD)
    if (a.elems == 4) return adj_go<NP, RK, PHYS, FWD, 4>(a, gi, p, n, st);
  if (a.elems == 2)
    adj_go<NP, RK, PHYS, FWD, 2>(a, gi, p, n, st);
  else
    adj_go<NP, RK, PHYS, FWD, 1>(a, gi, p, n, st);
}

template <int NP, int RK>
static void adj_phys(int phys, const AdjArgs& a, int gi, const AdjPtr& p, int32_t n, hipStream_t st) {
  const bool fwd = p.u_n != nullptr;
  switch (phys) {
    case PHYS_ADV_CENTRAL:
      if (fwd) adj_elems<NP, RK, PHYS_ADV_CENTRAL, true>(a, gi, p, n, st);
      else adj_elems<NP, RK, PHYS_ADV_CENTRAL, false>(a, gi, p, n, st);
      break;
    case PHYS_BURGERS_LLF: adj_elems<NP, RK, PHYS_BURGERS_LLF, true>(a, gi, p, n, st); break;
    default:
      if (gi % kAdjForms == 0) {
        if (fwd) adj_elems<NP, RK, PHYS_ADV_UPWIND_POS, true>(a, gi, p, n, st);
        else adj_elems<NP, RK, PHYS_ADV_UPWIND_POS, false>(a, gi, p, n, st);
      } else {
        if (fwd) adj_elems<NP, RK, PHYS_ADV_UPWIND, true>(a, gi, p, n, st);
        else adj_elems<NP, RK, PHYS_ADV_UPWIND, false>(a, gi, p, n, st);
      }
      break;
  }
}

template <int RK>
hipError_t launch_adj_rk(int phys, const AdjArgs& a, const double* u_n, const double* u_next, int64_t u_stride,
                         const double* lam, double* lamo, const double* ring, double* adjring, double* cpart,
                         int32_t n, hipStream_t stream) {
  if (phys == PHYS_BURGERS_LLF && !u_n) return hipErrorInvalidValue;  // its Jacobian needs the forward stages
  const AdjPtr p{u_n, u_next, u_stride, lam, ring, lamo, adjring, cpart};
  for (int gi = 0; gi < kAdjRanges; ++gi) {
    if (a.group[gi + 1] <= a.group[gi]) continue;
    switch (gi / kAdjForms) {  // np = 5, 4, 3, 2
      case 0: adj_phys<5, RK>(phys, a, gi, p, n, stream); break;
      case 1: adj_phys<4, RK>(phys, a, gi, p, n, stream); break;
      case 2: adj_phys<3, RK>(phys, a, gi, p, n, stream); break;
      default: adj_phys<2, RK>(phys, a, gi, p, n, stream); break;
    }
  }
  return hipGetLastError();
}

template hipError_t launch_adj_rk<ADG_RK>(int, const AdjArgs&, const double*, const double*, int64_t, const double*,
                                          double*, const double*, double*, double*, int32_t, hipStream_t);

}  // namespace adg
