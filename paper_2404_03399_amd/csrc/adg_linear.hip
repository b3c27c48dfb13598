// Fused step of linear advection with the upwind flux and a > 0: K whole RK
// steps per launch in flux-sequence form (adg_linear.hpp).  Compiled once per
// stage count (-DADG_S=2 .. 5): every integrator with S stages runs the same
// kernel, its coefficients are in the problem's table.
#include "adg_linear.hpp"

#ifndef ADG_S
#error "compile once per stage count with -DADG_S=2, 3, 4 or 5"
#endif

namespace adg {

extern __shared__ double wave_lds[];

template <int NP, int S, int R>
__global__ __launch_bounds__(kBlock) void k_lin_step(const DevProblem* __restrict__ probs,
                                                     const double* __restrict__ lin,
                                                     const WorkItem* __restrict__ work,
                                                     const StepClock clock, double* __restrict__ ring,
                                                     int32_t w_begin, int32_t w_end, const double* __restrict__ uin,
                                                     double* __restrict__ uout, int32_t step_offset, int32_t K,
                                                     int32_t HL, int32_t n_faces_max, int32_t lds_words,
                                                     int32_t single_prob) {
  const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
  const int lane = (int)(threadIdx.x % kWave);
  const int w = w_begin + xcd_block((int)blockIdx.x, (int)gridDim.x) * kWavesPerBlock + wv;
  if (w >= w_end) return;  // whole wave
  const int64_t n = clock.tick(w == w_begin) + step_offset;
  // a range holding one problem lists its tiles in order: no work-list load
  const WorkItem wi = single_prob >= 0 ? WorkItem{single_prob, w - w_begin} : work[w];
  const DevProblem& P = probs[wi.prob];
  lin_tile<NP, S, R>(P, lin + P.lin_off, wi, ring, n, K, HL, uin, uout, n_faces_max, wave_lds + wv * lds_words, lane);
}

template <int NP, int S, int R>
static void lin_go(const StepArgs& a, int gi, const double* uin, double* uout, int32_t off, hipStream_t st) {
  const FaceRange& fr = a.faces[gi];
  hipLaunchKernelGGL((k_lin_step<NP, S, R>), dim3(a.grid[gi]), dim3(kBlock), 8 * kWavesPerBlock * fr.lds_words, st,
                     a.probs, a.lin, a.work, a.clock, a.ring, a.group[gi], a.group[gi + 1], uin, uout, off, a.steps,
                     a.halo, fr.n_faces, fr.lds_words, a.single[gi]);
}

template <int NP, int S>
static void lin_r(const StepArgs& a, int gi, const double* uin, double* uout, int32_t off, hipStream_t st) {
  switch (a.elems) {
    case 1: lin_go<NP, S, 1>(a, gi, uin, uout, off, st); break;
    case 4: lin_go<NP, S, 4>(a, gi, uin, uout, off, st); break;
    default: lin_go<NP, S, 2>(a, gi, uin, uout, off, st); break;
  }
}

template <int S>
void launch_lin_s(const StepArgs& a, int gi, const double* uin, double* uout, int32_t off, hipStream_t st) {
  switch (gi / kForms) {  // np = 5, 4, 3, 2
    case 0: lin_r<5, S>(a, gi, uin, uout, off, st); break;
    case 1: lin_r<4, S>(a, gi, uin, uout, off, st); break;
    case 2: lin_r<3, S>(a, gi, uin, uout, off, st); break;
    default: lin_r<2, S>(a, gi, uin, uout, off, st); break;
  }
}

template void launch_lin_s<ADG_S>(const StepArgs&, int, const double*, double*, int32_t, hipStream_t);

}  // namespace adg
