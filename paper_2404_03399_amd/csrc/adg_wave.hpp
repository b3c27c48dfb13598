// What the tiles of the fused step share: the elements of a wave, their plane
// loads and stores, the PE faces a wave holds and the coefficient broadcast.
#pragma once

#include <type_traits>

#include "adg_device.hpp"

namespace adg {

// Elements of a wave64: R consecutive ones per lane, HL halo lanes on the left
// and HR on the right of the owned ones.
template <int R>
struct WaveElems {
  int e[R];       // element indices
  int own_n;      // owned elements of the lane: its first own_n
  bool buffered;  // planes move as 16-byte pieces through a buffer resource

  __device__ __forceinline__ WaveElems(const DevProblem& P, int tile, int HL, int HR, int lane) {
    const int N = (int)P.n_elem, TE = R * (kWave - HL - HR);
    const int e0 = tile * TE, teff = (N - e0) < TE ? (N - e0) : TE;
    const bool lane_owned = lane >= HL && lane < kWave - HR;
    const bool tiny = N < kWave * R;  // the wave's extent may wrap more than once
    own_n = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int x = e0 + R * (lane - HL) + r;
      e[r] = tiny ? wrap_elem(x, N) : wrap_once(x, N);
      own_n += lane_owned && (x - e0) < teff ? 1 : 0;
    }
    // with N a multiple of R a lane's elements never straddle the periodic
    // wrap; a buffer resource spans 2 GiB
    buffered = R > 1 && (N % R) == 0 && (int64_t)P.np * P.ld < (int64_t)1 << 28;
  }

  template <int NP>
  __device__ __forceinline__ void load(const DevProblem& P, const double* __restrict__ src, double (&u)[R][NP]) const {
    const double* __restrict__ p = src + P.u_off;
    const int64_t ld = P.ld;
    if (buffered) {
      const __amdgpu_buffer_rsrc_t rs = plane_rsrc(p);
#pragma unroll
      for (int j = 0; j < NP; ++j)
#pragma unroll
        for (int r = 0; r < R; r += 2) {
          const double2 v = __builtin_bit_cast(
              double2, __builtin_amdgcn_raw_buffer_load_b128(rs, e[0] * 8 + 8 * r, (int)(8 * j * ld), 0));
          u[r][j] = v.x;
          u[r + 1 < R ? r + 1 : r][j] = v.y;  // R >= 2 here
        }
    } else {
#pragma unroll
      for (int r = 0; r < R; ++r)
#pragma unroll
        for (int j = 0; j < NP; ++j) u[r][j] = p[j * ld + e[r]];
    }
  }

  template <int NP>
  __device__ __forceinline__ void store(const DevProblem& P, double* __restrict__ dst, const double (&u)[R][NP]) const {
    double* __restrict__ p = dst + P.u_off;
    const int64_t ld = P.ld;
    if (buffered && own_n == R) {
      const __amdgpu_buffer_rsrc_t rs = plane_rsrc(p);
#pragma unroll
      for (int j = 0; j < NP; ++j)
#pragma unroll
        for (int r = 0; r < R; r += 2) {
          double2 v;
          v.x = u[r][j];
          v.y = u[r + 1 < R ? r + 1 : r][j];
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(BufWord4, v), rs, e[0] * 8 + 8 * r,
                                                 (int)(8 * j * ld), 0);
        }
    } else {
      // the elements from the first one: kept from the load they are R - 1
      // registers through every step (p = 4, RK4, four elements per lane, linear
      // form: 132 registers, three waves per SIMD, and 128, four)
      int x = e[0];
      asm volatile("" : "+v"(x));
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if (r < own_n)
#pragma unroll
          for (int j = 0; j < NP; ++j) p[j * ld + x] = u[r][j];
        x = x + 1 == (int)P.n_elem ? 0 : x + 1;
      }
    }
  }
};

// Where R does not divide every PE size (ANY) a lane's PE face, at most one, is
// the left face of its element at_r, e_face; else of its first.
template <int R, bool ANY>
__device__ __forceinline__ void lane_face(const DevProblem& P, const WaveElems<R>& we, int& at_r, int& e_face) {
  if constexpr (ANY) {
    if (P.async_faces)
#pragma unroll
      for (int r = 1; r < R; ++r)
        if ((uint32_t)we.e[r] == fast_div((uint32_t)we.e[r], P.pe_div) * P.pe_div.d) at_r = r;
#pragma unroll
    for (int r = 1; r < R; ++r) e_face = at_r == r ? we.e[r] : e_face;
  }
}

// PE faces of a wave (Secs. 3-5) over a launch of K steps, at most one to a lane,
// the left face of its first element unless the tile says otherwise.  Every
// wave that holds a face (its owner's and those with the face in their halo,
// which see bitwise the same raw fluxes) draws its delays and sums the ring
// levels before the launch itself, one job lane per (face, step, stage) while
// the state loads are in flight; the levels of the launch are added after each
// step from the raw fluxes kept in LDS, the oldest level first in either part.
// The ring is written once, at the end, by the owner waves: with a depth of at
// least L + q + K - 2 no level that a wave of the launch reads shares a slot
// with one written in it.  V values per face share its delays: the flux, and
// for local DG (V = 2) u-hat, whose ring follows the flux ring.
//
// LDS of a wave with up to n_faces PE faces; a job is g = (face K + step) S + stage:
//   atc [kMaxL][kMaxQ]     the problem's AT weights
//   at  [value][job]       sum over the levels before the launch, then with the
//                          launch's levels, then the raw value of that step;
//                          S doubles more that lanes without a face write to
//   kd  [face][step] word  delays, byte s = stage s
//   own [face] word        1 if the wave owns the element right of it
using KdWord = uint64_t;
static_assert(kMaxStages <= (int)sizeof(KdWord), "one byte per stage");

__device__ __forceinline__ int lane_rank(uint64_t mask) {  // set bits below this lane
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

template <int S, int V = 1>
struct WaveFaces {
  double* atc;
  double* at;
  KdWord* kd;
  KdWord* own;
  uint64_t m_pe = 0;  // lanes with a PE face
  bool pe = false;
  int n_faces_max, vstride, n_jobs = 0, depth = 1, slot_n = 0, slot = 0;
  uint32_t b0 = 0;  // the wave's first face; its faces are consecutive, as its elements are

  // atc_lane: P.atc[0][lane], loaded ahead of the state
  __device__ __forceinline__ WaveFaces(const DevProblem& P, int e_first, bool owns, double atc_lane, int64_t n, int K,
                                       int n_faces_max_, double* lds, int lane)
      : atc(lds), at(lds + kMaxL * kMaxQ), n_faces_max(n_faces_max_) {
    vstride = n_faces_max * K * S + S;
    kd = reinterpret_cast<KdWord*>(at + V * vstride);
    own = kd + n_faces_max * K;
    if (!P.async_faces) return;
    depth = P.depth;
    const uint32_t n32 = (uint32_t)n;  // step indices stay below 2^31
    slot_n = (int)(n32 - fast_div(n32, P.depth_div) * (uint32_t)depth);
    const uint32_t b = fast_div((uint32_t)e_first, P.pe_div);
    pe = (uint32_t)e_first == b * P.pe_div.d;
    m_pe = __ballot(pe);
    slot = lane_rank(m_pe);
    b0 = (uint32_t)__builtin_amdgcn_readlane((int)b, m_pe ? __builtin_ctzll(m_pe) : 0);
    n_jobs = K * S * __builtin_popcountll(m_pe);
    if (pe) own[slot] = owns ? 1 : 0;
    if (lane < kMaxL * kMaxQ) atc[lane] = atc_lane;
  }

  __device__ __forceinline__ uint32_t face(const DevProblem& P, int i) const {
    uint32_t b = b0 + (uint32_t)i;
    while (b >= (uint32_t)P.n_pe) b -= (uint32_t)P.n_pe;
    return b;
  }

  // Delays and the sums over the levels before the launch.
  __device__ __forceinline__ void draw(const DevProblem& P, const double* __restrict__ ring, int64_t n, int K,
                                       int lane) {
#pragma clang fp contract(off)
    const uint32_t kshift = (uint32_t)__builtin_ctz((uint32_t)K);  // K is a power of two
    for (int g0 = 0; g0 < n_jobs; g0 += kWave) {                   // uniform
      const int g = g0 + lane;
      if (g < n_jobs) {
        const int ik = g / S, s = g - ik * S, i = ik >> kshift, kk = ik - (i << kshift);
        const uint32_t b = face(P, i);
        const int k = pe_delay(P, n + kk, s, b);
        const int64_t rb = (int64_t)b * S + s;
        double lv[V][kMaxQ];
#pragma unroll
        for (int j = 0; j < kMaxQ; ++j) {
#pragma unroll
          for (int v = 0; v < V; ++v) lv[v][j] = 0.0;
          if (j < P.q) {  // uniform
            const int back = k + j - kk;  // level n - back
            if (k > 0 && back > 0)
#pragma unroll
              for (int v = 0; v < V; ++v)
                lv[v][j] = ring[(v == 0 ? P.ring_off : P.ring2_off) + rb + ring_slot(slot_n, back, depth) * P.ring_stride];
          }
        }
        reinterpret_cast<uint8_t*>(kd + ik)[s] = (uint8_t)k;
        double sum[V] = {};
#pragma unroll
        for (int j = kMaxQ - 1; j >= 0; --j)
          if (j < P.q && k > 0 && k + j > kk)
#pragma unroll
            for (int v = 0; v < V; ++v) sum[v] = fma(atc[k * kMaxQ + j], lv[v][j], sum[v]);
#pragma unroll
        for (int v = 0; v < V; ++v) at[v * vstride + g] = sum[v];
      }
    }
  }

  // This lane's face in step kk: where its AT sums stand and its raw fluxes go
  // (lanes without a face have a place of their own, so that no branch cuts the
  // stages into blocks), and its delays (0 without a face).
  __device__ __forceinline__ double* sums(int K, int kk, int v = 0) const {
    return at + v * vstride + ((pe ? slot : n_faces_max) * K + (pe ? kk : 0)) * S;
  }
  __device__ __forceinline__ KdWord delays(int K, int kk) const {
    const KdWord w = kd[pe ? slot * K + kk : 0];
    return pe ? w : 0;
  }

  // The raw fluxes of step kk enter the sums of the launch's later steps.
  __device__ __forceinline__ void pass_on(const DevProblem& P, int K, int kk, int lane) {
#pragma clang fp contract(off)
    for (int g0 = 0; g0 < n_jobs && kk + 1 < K; g0 += kWave) {
      const int g = g0 + lane, ik = g / S, later = (ik & (K - 1)) - kk;  // steps to the job's own
      if (g < n_jobs && later > 0) {
        const int k = reinterpret_cast<const uint8_t*>(kd + ik)[g - ik * S], j = later - k;
        if (k > 0 && j >= 0 && j < P.q)
#pragma unroll
          for (int v = 0; v < V; ++v) {
            double* const x = at + v * vstride + g;
            *x = fma(atc[k * kMaxQ + j], x[-later * S], *x);
          }
      }
    }
  }

  // The raw fluxes of the owned faces into the ring.
  __device__ __forceinline__ void keep(const DevProblem& P, double* __restrict__ ring, int K, int lane) const {
    const uint32_t kshift = (uint32_t)__builtin_ctz((uint32_t)K);
    for (int g0 = 0; g0 < n_jobs; g0 += kWave) {
      const int g = g0 + lane;
      if (g < n_jobs) {
        const int ik = g / S, s = g - ik * S, i = ik >> kshift, kk = ik - (i << kshift);
        if (own[i]) {
          int sl = slot_n + kk;
          while (sl >= depth) sl -= depth;
#pragma unroll
          for (int v = 0; v < V; ++v)
            ring[(v == 0 ? P.ring_off : P.ring2_off) + (int64_t)face(P, i) * S + s + sl * P.ring_stride] =
                at[v * vstride + g];
        }
      }
    }
  }
};

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
  static_assert(M >= 1 && M <= 5 && L >= 0 && L + M <= 16, "a column lies within one run of 16");
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
  else
    asm("s_nop 1\n\t" ADG_FM(0) ADG_FM(1) ADG_FM(2) ADG_FM(3) ADG_FM(4)
        : "+v"(*a[0]), "+v"(*a[1]), "+v"(*a[2]), "+v"(*a[3]), "+v"(*a[4])
        : ADG_IN, [l1] "n"(L + 1), [l2] "n"(L + 2), [l3] "n"(L + 3), [l4] "n"(L + 4));
#undef ADG_FM
#undef ADG_IN
}

// The same for a whole NP x NP operator held by columns: v_i += K_ij g_j, the
// columns in order.  Up to three columns (NP = 5) or all of them sit in one
// register pair, 16 / NP to a pair.
template <int NP>
__device__ __forceinline__ void fmac_operator(const double (&op)[NP == 5 ? 2 : 1], const double (&g)[NP],
                                              double (&v)[NP]) {
#define ADG_FM(i, c, g, l) "v_fmac_f64_dpp %[v" #i "], %[" c "], %[g" #g "] row_newbcast:" #l " row_mask:0xf bank_mask:0xf\n\t"
#define ADG_C2(j, l0, l1) ADG_FM(0, "c", j, l0) ADG_FM(1, "c", j, l1)
#define ADG_C3(j, l0, l1, l2) ADG_C2(j, l0, l1) ADG_FM(2, "c", j, l2)
#define ADG_C4(j, l0, l1, l2, l3) ADG_C3(j, l0, l1, l2) ADG_FM(3, "c", j, l3)
#define ADG_C5(c, j, l0, l1, l2, l3, l4) \
  ADG_FM(0, c, j, l0) ADG_FM(1, c, j, l1) ADG_FM(2, c, j, l2) ADG_FM(3, c, j, l3) ADG_FM(4, c, j, l4)
#define ADG_V2 [v0] "+v"(v[0]), [v1] "+v"(v[1])
#define ADG_G2 [c] "v"(op[0]), [g0] "v"(g[0]), [g1] "v"(g[1])
  if constexpr (NP == 2)
    asm("s_nop 1\n\t" ADG_C2(0, 0, 1) ADG_C2(1, 2, 3) : ADG_V2 : ADG_G2);
  else if constexpr (NP == 3)
    asm("s_nop 1\n\t" ADG_C3(0, 0, 1, 2) ADG_C3(1, 3, 4, 5) ADG_C3(2, 6, 7, 8)
        : ADG_V2, [v2] "+v"(v[2])
        : ADG_G2, [g2] "v"(g[2]));
  else if constexpr (NP == 4)
    asm("s_nop 1\n\t" ADG_C4(0, 0, 1, 2, 3) ADG_C4(1, 4, 5, 6, 7) ADG_C4(2, 8, 9, 10, 11) ADG_C4(3, 12, 13, 14, 15)
        : ADG_V2, [v2] "+v"(v[2]), [v3] "+v"(v[3])
        : ADG_G2, [g2] "v"(g[2]), [g3] "v"(g[3]));
  else
    asm("s_nop 1\n\t" ADG_C5("c", 0, 0, 1, 2, 3, 4) ADG_C5("c", 1, 5, 6, 7, 8, 9) ADG_C5("c", 2, 10, 11, 12, 13, 14)
            ADG_C5("d", 3, 0, 1, 2, 3, 4) ADG_C5("d", 4, 5, 6, 7, 8, 9)
        : ADG_V2, [v2] "+v"(v[2]), [v3] "+v"(v[3]), [v4] "+v"(v[4])
        : ADG_G2, [d] "v"(op[NP == 5 ? 1 : 0]), [g2] "v"(g[2]), [g3] "v"(g[3]), [g4] "v"(g[4]));
#undef ADG_FM
#undef ADG_C2
#undef ADG_C3
#undef ADG_C4
#undef ADG_C5
#undef ADG_V2
#undef ADG_G2
}

}  // namespace adg
