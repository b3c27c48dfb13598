// Fused step kernels: one wave64 per tile, all RK stages of the steps of a
// launch on chip.  Compiled once per integrator (-DADG_RK=0 .. 4) so that the
// instantiations build in parallel.
#include "adg_ldg.hpp"
#include "adg_linear.hpp"
#include "adg_stage.hpp"

#ifndef ADG_RK
#error "compile once per integrator with -DADG_RK=0, 1, 2, 3 or 4"
#endif

namespace adg {

extern __shared__ double wave_lds[];

template <int NP, int RK, int PHYS, int R, bool ANY>
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
  stage_tile<NP, RK, PHYS, R, ANY>(probs[wi.prob], wi, ring, n, K, HL, uin, uout, umid, mid_stride, n_faces_max,
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

template <int NP, int RK, int R, bool ANY>
__global__ __launch_bounds__(kBlock) void k_fused_ldg(const DevProblem* __restrict__ probs,
                                                      const WorkItem* __restrict__ work, const StepClock clock,
                                                      double* __restrict__ ring, int32_t w_begin, int32_t w_end,
                                                      const double* __restrict__ uin, double* __restrict__ uout,
                                                      int32_t step_offset, int32_t K, int32_t HL, int32_t HR,
                                                      int32_t n_faces_max, int32_t lds_words, int32_t single_prob) {
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int lane = (int)(threadIdx.x % kWave);
  const int w = w_begin + xcd_block((int)blockIdx.x, (int)gridDim.x) * kWavesPerBlock + wv;
  if (w >= w_end) return;  // whole wave
  const int64_t n = clock.tick(w == w_begin) + step_offset;
  const WorkItem wi = single_prob >= 0 ? WorkItem{single_prob, w - w_begin} : work[w];
  ldg_tile<NP, RK, R, ANY>(probs[wi.prob], wi, ring, n, K, HL, HR, uin, uout, n_faces_max, wave_lds + wv * lds_words, lane);
}

template <int NP, int RK, int R, bool ANY = false>
static void fused_ldg_go_r(const StepArgs& a, int gi, const double* uin, double* uout, int32_t off, hipStream_t st) {
  const FaceRange& fr = a.faces[gi];
  hipLaunchKernelGGL((k_fused_ldg<NP, RK, R, ANY>), dim3(a.grid[gi]), dim3(kBlock), 8 * kWavesPerBlock * fr.lds_words, st,
                     a.probs, a.work, a.clock, a.ring, a.group[gi], a.group[gi + 1], uin, uout, off, a.steps, a.halo,
                     a.halo_right, fr.n_faces, fr.lds_words, a.single[gi]);
}

template <int NP, int RK>
static void fused_ldg_go(const StepArgs& a, int gi, const double* uin, double* uout, int32_t off, hipStream_t st) {
  if (a.any_face) return fused_ldg_go_r<NP, RK, 2, true>(a, gi, uin, uout, off, st);
  switch (a.elems) {
    case 1: fused_ldg_go_r<NP, RK, 1>(a, gi, uin, uout, off, st); break;
    case 4: fused_ldg_go_r<NP, RK, 4>(a, gi, uin, uout, off, st); break;
    default: fused_ldg_go_r<NP, RK, 2>(a, gi, uin, uout, off, st); break;
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

template <int NP, int RK, int PHYS, int R, bool ANY = false>
static void fused_go_r(const StepArgs& a, int gi, const double* uin, double* uout, int32_t off, hipStream_t st) {
  const FaceRange& fr = a.faces[gi];
  hipLaunchKernelGGL((k_fused_step<NP, RK, PHYS, R, ANY>), dim3(a.grid[gi]), dim3(kBlock),
                     8 * kWavesPerBlock * fr.lds_words, st, a.probs, a.work, a.clock, a.ring, a.group[gi],
                     a.group[gi + 1], uin, uout, a.umid, a.mid_stride, off, a.steps, a.halo, fr.n_faces, fr.lds_words,
                     a.single[gi]);
}

template <int NP, int RK, int PHYS>
static void fused_go(const StepArgs& a, int gi, const double* uin, double* uout, int32_t off, hipStream_t st) {
  if constexpr (PHYS != PHYS_ADV_UPWIND_POS)
    if (a.any_face) return fused_go_r<NP, RK, PHYS, 2, true>(a, gi, uin, uout, off, st);
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
