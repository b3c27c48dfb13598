// Internal launch interface between the C ABI layer and the HIP kernels.
#pragma once

#include "adg_common.hpp"

namespace adg {

// Work items of the fused kernel are sorted by descending np and, within a
// degree, by form: range g = kForms (5 - np) + v, [group[g], group[g + 1]),
// holds the items of degree np - 1 in form v: upwind advection with a > 0 in
// the linear form (adg_linear.hpp, tiles of its own) or stage by stage with
// the interior right-face flux folded into the volume operator, and the
// general form of the context's equation.  Each problem therefore runs the
// same kernel in a batch as in a context of its own.
enum FusedForm : int { FORM_LIN = 0, FORM_POS = 1, FORM_GEN = 2 };
constexpr int kForms = 3;
constexpr int kFusedRanges = 4 * kForms;

// The context's counter words: steps completed, the same while a batch of
// launches is under way, non-finite flag, and a word that stays 0.
enum CtrWord : int { CTR_DONE = 0, CTR_BATCH = 1, CTR_FLAG = 2, CTR_ZERO = 3 };

// Step index of a fused launch: *from + step_offset; one wave also leaves
// *from + add in *to (null: nothing), a word that no wave of the launch reads.
// A batch of launches closes itself: with the first step's index known on the
// host, its launches count from CTR_ZERO and the last one writes CTR_DONE; one
// that is replayed from a graph counts from CTR_DONE in its first launch, which
// copies it to CTR_BATCH, and from there in the others, the last of which
// writes CTR_DONE (as a kernel of its own after every batch the advance cost
// 4 us of the 30 that 16 steps of a small mesh take).
struct StepClock {
  const int64_t* from;
  int64_t* to;
  int64_t add;
#ifdef __HIPCC__
  __device__ __forceinline__ int64_t tick(bool first_wave) const {
    const int64_t base = *from;
    if (first_wave && to != nullptr && threadIdx.x == 0) *to = base + add;
    return base;
  }
#endif
};

struct FaceRange {
  int32_t n_faces;     // most PE faces that a wave of the range holds
  int32_t lds_words;   // doubles of LDS per wave
};

struct StepArgs {
  const DevProblem* probs;   // device descriptors
  const WorkItem* work;      // device work list, one item per workgroup
  int32_t n_work;
  double* ring;              // delay ring (fluxes), may be null when no PE faces
  int64_t* ctr;              // stage kernels: the word that step_offset counts from; statistics: the context's words
  StepClock clock;           // fused kernel
  int32_t group[kFusedRanges + 1];   // fused kernel: work-item ranges per degree and form
  int32_t grid[kFusedRanges];        // fused kernel: workgroups per range
  int32_t single[kFusedRanges];      // fused kernel: the only problem of a range, or -1
  FaceRange faces[kFusedRanges];     // fused kernel: PE faces per wave of a range
  int32_t elems;             // fused kernel: elements per lane (1, 2 or 4)
  int32_t steps;             // fused kernel: time steps of the launch, a power of two
  int32_t any_face;          // two elements per lane although a PE size is odd (general stage form, local DG)
  int32_t halo;              // fused kernel: halo lanes per side (upwind, a > 0: on the left)
  int32_t halo_right;        // local DG: halo lanes on the right
  double* qbuf;              // local DG: q = u_x of the current stage input (state layout)
  double* umid;              // fused kernel, several steps per launch: also write the states after
                             // the steps before the last here (state layout), or null
  int64_t mid_stride;        // distance between those states (doubles)
  const double* lin;         // linear form: tables of the problems
  int32_t one_launch;        // fused kernel: one launch over every range, else one per range
};

// Fused step kernel geometry: one wave64 per work item, R in {1, 2, 4}
// consecutive elements per lane, K time steps per launch, a halo of K S
// elements: on both sides in the general form; on the left for upwind with
// a > 0, and there one lane more on the right where a problem has PE faces (the
// element right of the last owned one, whose left face may be one).
constexpr int kWave = 64;
constexpr int kWavesPerBlock = kBlock / kWave;
constexpr int kMaxSteps = 8;  // most steps per launch
__host__ __device__ constexpr int fused_halo(int rk, int R, int K) { return (K * rk_stages(rk) + R - 1) / R; }
__host__ __device__ constexpr int fused_tile(int rk, int R, int K) { return R * (kWave - 2 * fused_halo(rk, R, K)); }
__host__ __device__ constexpr int fused_tile_left(int rk, int R, int K, bool async) {
  return R * (kWave - fused_halo(rk, R, K) - (async ? 1 : 0));
}
// Local DG: one halo element more on the right.
__host__ __device__ constexpr int ldg_halo_right(int rk, int R, int K) { return (K * rk_stages(rk) + R) / R; }
__host__ __device__ constexpr int ldg_tile_elems(int rk, int R, int K) {
  return R * (kWave - fused_halo(rk, R, K) - ldg_halo_right(rk, R, K));
}
// PE faces of a wave's 64 R elements at most, one to a lane
__host__ __device__ constexpr int fused_faces(int R, int64_t pe_size) {
  return (int)((kWave * R - 1) / pe_size) + 1;
}
// LDS of a wave in doubles (layout: WaveFaces; V values per face)
__host__ __device__ constexpr int fused_lds_words(int S, int K, int n_faces, int V) {
  return n_faces > 0 ? kMaxL * kMaxQ + V * (S + n_faces * K * S) + n_faces * (K + 1) : 0;
}
// One range of the linear form (compiled per stage count).
template <int S>
void launch_lin_s(const StepArgs& a, int gi, const double* uin, double* uout, int32_t step_offset, hipStream_t stream);

// Windows of 4 K S elements around a PE face and how many fit a wave: they size
// the room that the workspace holds with ADG_OPT_PE_SPLIT_ON, or by default on
// large PEs (part of the interface's documented effect of the flags; no kernel
// reads it).
__host__ __device__ constexpr int fused_window(int rk, int K) { return 4 * K * rk_stages(rk); }
__host__ __device__ constexpr int fused_windows_per_wave(int rk, int K) { return kWave / fused_window(rk, K); }

// Workgroups of the fused kernel for n_work items (kWavesPerBlock per group).
inline int fused_grid(int n_work) { return n_work < 1 ? 1 : (n_work + kWavesPerBlock - 1) / kWavesPerBlock; }

// a.steps full RK steps, all stages on chip: state uin -> uout
// (distinct buffers).  The first step's index is *a.clock.from + step_offset.
hipError_t launch_fused_step(int rk, int phys, const StepArgs& a, const double* uin, double* uout,
                             int32_t step_offset, hipStream_t stream);
// Its per-integrator part (one translation unit per RK scheme).
template <int RK>
hipError_t launch_fused_rk(int phys, const StepArgs& a, const double* uin, double* uout, int32_t step_offset,
                           hipStream_t stream);

// One RK stage with the RK registers in HBM.  Stage 0 reads its input from U;
// the last stage writes U in place.  yin/yout alternate between two buffers.
hipError_t launch_stage(int rk, int phys, int stage, const StepArgs& a, const double* yin, double* yout,
                        double* U, double* A, int32_t step_offset, hipStream_t stream);

// Local DG, first pass of stage `stage`: q = u_x of the stage input yin into
// a.qbuf, with the u-hat face values (AT-combined at PE faces, level-n raw
// values written to the u-hat ring).
hipError_t launch_ldg_q(int rk, int stage, const StepArgs& a, const double* yin, int32_t step_offset,
                        hipStream_t stream);

// Reverse of RK stage `stage` of step n (absolute index) for all problems:
// lamu += mu, Q_i += a_{stage,i} mu, adjoint-ring deposits for delayed AT
// levels, cpart[workgroup] += dJ/da share.  Stage work list (kBlock per item).
hipError_t launch_adj_stage(int rk, int phys, int stage, const StepArgs& a, const double* Y, const double* lam,
                            double* lamu, double* Q, int64_t qstride, const double* ring, double* adjring,
                            double* cpart, int32_t n, hipStream_t stream);

// Fused reverse sweep: R elements per lane, K steps per launch, a halo of K S
// elements per side for a constant Jacobian (linear advection) and of
// (K + 1) S - 1 where the Jacobian depends on the stage inputs (Burgers).
__host__ __device__ constexpr int adj_halo(int rk, bool nonlinear, int R, int K) {
  return ((nonlinear ? (K + 1) * rk_stages(rk) - 1 : K * rk_stages(rk)) + R - 1) / R;
}
__host__ __device__ constexpr int adj_tile_elems(int rk, bool nonlinear, int R, int K) {
  return R * (kWave - 2 * adj_halo(rk, nonlinear, R, K));
}
// Elements of a partial sum of dJ/da.
__host__ __device__ constexpr int adj_part_elems(int rk) { return kWave - 2 * rk_stages(rk); }
// LDS of a wave in doubles (layout: adj_tile, AdjFaces)
__host__ __device__ constexpr int adj_lds_words(int S, int R, int K, int n_faces, bool forward, bool speed) {
  return (speed ? R * kWave : 0) + (n_faces > 0 ? kMaxL * kMaxQ + (forward ? 2 : 1) * (n_faces * K * S + S) +
                                                      n_faces * (K + 1)
                                                : 0);
}
// Work items are grouped by descending np and, within, upwind with a > 0 first.
constexpr int kAdjForms = 2, kAdjRanges = 4 * kAdjForms;
struct AdjArgs {
  const DevProblem* probs;
  const WorkItem* work;
  int32_t group[kAdjRanges + 1];
  int32_t grid[kAdjRanges];
  int32_t single[kAdjRanges];  // the range's only problem, or -1
  FaceRange faces[kAdjRanges];
  int32_t elems, steps;  // elements per lane, steps of this launch (a power of two, at most the list's)
  int32_t halo;          // halo lanes per side of the work list
};

// Reverse of the a.steps whole RK steps n, ..., n + K - 1 (absolute indices) for
// all problems in one launch per range: lamo = lambda^n from lam = lambda^{n+K};
// adjoint-ring deposits for delayed AT levels.  With the forward states u^n at
// u_n and u^{n+1}, u^{n+2}, ... at u_next, u_next + u_stride, ... (stages
// recomputed on chip) advection adds its dJ/da shares to cpart; without them
// (u_n == nullptr, advection only) dJ/du0 alone.  Compiled per integrator.
template <int RK>
hipError_t launch_adj_rk(int phys, const AdjArgs& a, const double* u_n, const double* u_next, int64_t u_stride,
                         const double* lam, double* lamo, const double* ring, double* adjring, double* cpart,
                         int32_t n, hipStream_t stream);
hipError_t launch_adj_fused(int rk, int phys, const AdjArgs& a, const double* u_n, const double* u_next,
                            int64_t u_stride, const double* lam, double* lamo, const double* ring, double* adjring,
                            double* cpart, int32_t n, hipStream_t stream);

// Zero fill of `bytes` bytes at p (8-byte aligned, a multiple of 8).
hipError_t launch_zero(void* p, int64_t bytes, hipStream_t stream);

// ctr[CTR_DONE] += n_steps (one lane), closing a batch of stage kernels or of one fused launch.
hipError_t launch_advance(int64_t* ctr, int64_t n_steps, hipStream_t stream);

// Per-workgroup partial error sums (work list with kBlock elements per item),
// then per-problem reduction in a fixed order.
hipError_t launch_stats(const StepArgs& a, const double* u, const double* ref, double* partials,
                        const int32_t* first_item, int32_t n_probs, double* out, hipStream_t stream);

// Per-group mean / variance of the per-problem statistics (3 doubles per
// problem: mean |u-ref|, max |u-ref|, integral) -> 4 doubles per group.
hipError_t launch_group_stats(const double* pstats, const int32_t* gstart, const int32_t* gmembers, int32_t n_groups,
                              double* out, hipStream_t stream);

// Sets ctr[2] = 1 if any owned state entry is NaN or Inf.
hipError_t launch_check_finite(const StepArgs& a, const double* u, hipStream_t stream);

}  // namespace adg
