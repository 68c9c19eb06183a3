// Device code of the fused per-pixel Kronecker STAP kernels for gfx950
// (MI355X), shared by the translation units that instantiate them
// (kstap_kern_fp32.hip, kstap_kern_bf16.hip, kstap_kern_wide.hip).
//
// Narrow pixels (p*q <= 64): one 64-lane wavefront (one workgroup) carries
// one pixel at a time through the whole pass and walks a run of positions of
// the tiled pixel order.
//
//   a2  sample covariance S = (1/n) sum_m x_m x_m^H  (Sec. 1.1, Eq. (2)) as a
//       dense contraction on MFMA.  FP32 path: Re S = Xr Xr^T + Xi Xi^T and
//       Im S = Xi Xr^T - Xr Xi^T over the upper 16 x 16 tiles, on the BF16
//       pipe with every sample split exactly into three BF16 parts (scm_split;
//       v_mfma_f32_16x16x4_f32 for p q > 48 and the Doppler bank).  Mixed
//       path: three BF16 products on pre-split planes.
//       Training vectors are read through buffer resources straight into
//       MFMA operands; workgroups that are in flight together on one XCD
//       cover a compact patch, so their windows are served from its L2.
//   a3  the rearrangement of Algorithm 1 is never materialised: block S(i,j)
//       of S is row i*p + j of R in address arithmetic only.
//   a4  A_0 = block sums of S / q^2 (Sec. 4, Eqs. (18)-(19)).
//   a5  LR-Kron (Algorithm 2) on the Hermitian half of S, held in registers
//       (Slots): per iteration the residual of the previous iterate, the new
//       time factor b = R^T conj(a) / ||a||^2 and the sums R conj(b).
//       EIG_{r_a} (Eq. (17)): power iteration for r_a = 1, subspace
//       iteration otherwise, warm-started from the previous iterate.
//   a6  the final b = R^T conj(a) / ||a||^2 (Hermitian) is queued as slots
//       in LDS; every 64/q' pixels (q' = q rounded up to 8, 16 or 32) one
//       batched subspace iteration finds the top-r_b subspaces, q' lanes per
//       pixel with group-local DPP reductions (CGS2, residual stop), the rank
//       a compile-time constant (kstap_tail.h; tail_batch for the variants).
//   a8  T = ||F_A X conj(F_B b_s)||^2 / (b_s^H F_B b_s) (Sec. 5, Eq. (25);
//       Sec. 6.3, Eq. (26)); D = T > tau.
// Wide pixels (p*q > 64): one 8-wave workgroup per pixel, see below.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "kstap_internal.h"
#include "kstap_small_eig.h"

namespace kstap {
namespace {

typedef float f4 __attribute__((ext_vector_type(4)));

// ------------------------------------------------------------------ complex
__device__ __forceinline__ float2 cz() { return make_float2(0.f, 0.f); }
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cscale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }
__device__ __forceinline__ float2 cconj(float2 a) { return make_float2(a.x, -a.y); }
__device__ __forceinline__ float cabs2(float2 a) { return fmaf(a.x, a.x, a.y * a.y); }
// a*b + c
__device__ __forceinline__ float2 cfma(float2 a, float2 b, float2 c) {
  return make_float2(fmaf(a.x, b.x, fmaf(-a.y, b.y, c.x)), fmaf(a.x, b.y, fmaf(a.y, b.x, c.y)));
}
// conj(a)*b + c
__device__ __forceinline__ float2 ccfma(float2 a, float2 b, float2 c) {
  return make_float2(fmaf(a.x, b.x, fmaf(a.y, b.y, c.x)), fmaf(a.x, b.y, fmaf(-a.y, b.x, c.y)));
}
__device__ __forceinline__ float2 cmul(float2 a, float2 b) { return cfma(a, b, cz()); }

// double2 versions (FP64 eigensolves and normalisation of the mixed path)
template <typename C> __device__ __forceinline__ C czero();
template <> __device__ __forceinline__ float2 czero<float2>() { return make_float2(0.f, 0.f); }
template <> __device__ __forceinline__ double2 czero<double2>() { return make_double2(0.0, 0.0); }
__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cscale(double2 a, double s) { return make_double2(a.x * s, a.y * s); }
__device__ __forceinline__ double2 cconj(double2 a) { return make_double2(a.x, -a.y); }
__device__ __forceinline__ double cabs2(double2 a) { return fma(a.x, a.x, a.y * a.y); }
__device__ __forceinline__ double2 cfma(double2 a, double2 b, double2 c) {
  return make_double2(fma(a.x, b.x, fma(-a.y, b.y, c.x)), fma(a.x, b.y, fma(a.y, b.x, c.y)));
}
__device__ __forceinline__ double2 ccfma(double2 a, double2 b, double2 c) {
  return make_double2(fma(a.x, b.x, fma(a.y, b.y, c.x)), fma(a.x, b.y, fma(-a.y, b.x, c.y)));
}
__device__ __forceinline__ double2 cmul(double2 a, double2 b) { return cfma(a, b, czero<double2>()); }
template <typename C> __device__ __forceinline__ C cto(float2 a);
template <> __device__ __forceinline__ float2 cto<float2>(float2 a) { return a; }
template <> __device__ __forceinline__ double2 cto<double2>(float2 a) { return make_double2(a.x, a.y); }
__device__ __forceinline__ float2 tof(float2 a) { return a; }
__device__ __forceinline__ float2 tof(double2 a) { return make_float2(float(a.x), float(a.y)); }
__device__ __forceinline__ float xsqrt(float a) { return sqrtf(a); }
__device__ __forceinline__ double xsqrt(double a) { return sqrt(a); }
// Scale factors that normalise an iterate or divide by a uniform norm: the
// hardware reciprocal (square root) in FP32, within one ulp, where the scale
// only has to be consistent (the next step renormalises, a statistic or a
// subspace does not depend on it); exact in FP64.  The argument is a normal
// positive number.
__device__ __forceinline__ float xrsqrt(float a) { return __builtin_amdgcn_rsqf(a); }
__device__ __forceinline__ double xrsqrt(double a) { return 1.0 / sqrt(a); }
__device__ __forceinline__ float xrcp(float a) { return __builtin_amdgcn_rcpf(a); }
__device__ __forceinline__ float xmax(float a, float b) { return fmaxf(a, b); }
__device__ __forceinline__ double xmax(double a, double b) { return fmax(a, b); }

// ------------------------------------------------------- wavefront reductions
// Sum over the 64 lanes.  Four DPP steps reduce each 16-lane row (quad swaps,
// half-row mirror, row mirror: every lane then holds its row's sum), two
// row broadcasts (lane 15 -> next row, lane 31 -> rows 2 and 3) accumulate
// the rows into lane 63, and the total is read from lane 63 as a uniform
// value.  No LDS traffic.
template <int CTRL, int ROWS>
__device__ __forceinline__ float dpp(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, ROWS, 0xF, false));
}
__device__ __forceinline__ float wsum(float v) {
  v += dpp<0xB1, 0xF>(v);    // quad_perm [1,0,3,2]
  v += dpp<0x4E, 0xF>(v);    // quad_perm [2,3,0,1]
  v += dpp<0x141, 0xF>(v);   // row_half_mirror
  v += dpp<0x140, 0xF>(v);   // row_mirror
  v += dpp<0x142, 0xA>(v);   // row_bcast:15 into rows 1 and 3
  v += dpp<0x143, 0xC>(v);   // row_bcast:31 into rows 2 and 3
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), 63));
}
__device__ __forceinline__ float2 wsum(float2 v) { return make_float2(wsum(v.x), wsum(v.y)); }
// Sums over the 64 lanes of N values at once (N a multiple of 4), each
// returned as a uniform value.  v_permlane32_swap exchanges the upper half of
// value 2m with the lower half of value 2m + 1, so one add leaves value 2m
// summed over lanes l and l + 32 in lanes 0-31 and value 2m + 1 in lanes
// 32-63; v_permlane16_swap does the same between 16-lane rows, which leaves
// four values per register, one per row (rows 0-3: values 4m, 4m + 2,
// 4m + 1, 4m + 3), and four DPP steps finish every row.  About 3.5
// instructions per value instead of the 7 of wsum.  The compiler folds the
// sum of a swap's two results into twice its first result unless the results
// pass through an empty asm first (swap_sum).
__device__ __forceinline__ float swap_sum(unsigned r0, unsigned r1) {
  asm volatile("" : "+v"(r0), "+v"(r1));
  return __builtin_bit_cast(float, r0) + __builtin_bit_cast(float, r1);
}
template <int N>
__device__ __forceinline__ void wsum_n(float (&v)[N]) {
  static_assert(N % 4 == 0, "wsum_n sums a multiple of four values");
  float w[N / 2];
#pragma unroll
  for (int m = 0; m < N / 2; ++m) {
    const auto r = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, v[2 * m]),
                                                    __builtin_bit_cast(unsigned, v[2 * m + 1]), false, false);
    w[m] = swap_sum(r[0], r[1]);
  }
#pragma unroll
  for (int m = 0; m < N / 4; ++m) {
    const auto r = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, w[2 * m]),
                                                    __builtin_bit_cast(unsigned, w[2 * m + 1]), false, false);
    float x = swap_sum(r[0], r[1]);
    x += dpp<0xB1, 0xF>(x);    // quad_perm [1,0,3,2]
    x += dpp<0x4E, 0xF>(x);    // quad_perm [2,3,0,1]
    x += dpp<0x141, 0xF>(x);   // row_half_mirror
    x += dpp<0x140, 0xF>(x);   // row_mirror: every lane holds its row's sum
    const int xi = __builtin_bit_cast(int, x);
    v[4 * m] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 0));
    v[4 * m + 2] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 16));
    v[4 * m + 1] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 32));
    v[4 * m + 3] = __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 48));
  }
}
// A swap or mirror that every lane takes part in (ROWS 0xF) has no lanes that
// keep an old value, so none is set up: the zeros an update would start from
// were two of the five instructions of every FP64 step.
template <int CTRL, int ROWS>
__device__ __forceinline__ double dppd(double v) {
  const int2 i = __builtin_bit_cast(int2, v);
  int2 o;
  if constexpr (ROWS == 0xF) {
    o.x = __builtin_amdgcn_mov_dpp(i.x, CTRL, ROWS, 0xF, true);
    o.y = __builtin_amdgcn_mov_dpp(i.y, CTRL, ROWS, 0xF, true);
  } else {
    o.x = __builtin_amdgcn_update_dpp(0, i.x, CTRL, ROWS, 0xF, false);
    o.y = __builtin_amdgcn_update_dpp(0, i.y, CTRL, ROWS, 0xF, false);
  }
  return __builtin_bit_cast(double, o);
}
__device__ __forceinline__ double wsumd(double v) {
  v += dppd<0xB1, 0xF>(v);
  v += dppd<0x4E, 0xF>(v);
  v += dppd<0x141, 0xF>(v);
  v += dppd<0x140, 0xF>(v);
  v += dppd<0x142, 0xA>(v);
  v += dppd<0x143, 0xC>(v);
  const int2 i = __builtin_bit_cast(int2, v);
  int2 o;
  o.x = __builtin_amdgcn_readlane(i.x, 63);
  o.y = __builtin_amdgcn_readlane(i.y, 63);
  return __builtin_bit_cast(double, o);
}

__device__ __forceinline__ void wave_sync() { __syncthreads(); }   // one-wave workgroups

// LDS exchange among the lanes of one wavefront inside a workgroup of several:
// a wavefront's LDS operations are performed in issue order, so only the
// compiler has to be kept from moving accesses across this point.
__device__ __forceinline__ void lane_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
template <bool WAVE_LOCAL>
__device__ __forceinline__ void lds_sync() {
  if constexpr (WAVE_LOCAL) lane_sync();
  else wave_sync();
}

__device__ __forceinline__ float frac01(float x) { return x - floorf(x); }

// Deterministic, generic start block for subspace iteration.
__device__ __forceinline__ float2 omega(int k, int c) {
  float ph = 6.2831853f * frac01(0.6180340f * (k + 1) + 0.4142136f * (c + 1) * (k + 3));
  return make_float2(__cosf(ph), __sinf(ph));
}

// Sum over each group of QP consecutive lanes (QP = 8, 16, 32 or 64); every
// lane of a group receives its group's sum (QP = 64: a uniform value).
template <int QP>
__device__ __forceinline__ float gsum(float v) {
  if constexpr (QP == 64) {
    return wsum(v);
  } else {
    v += dpp<0xB1, 0xF>(v);
    v += dpp<0x4E, 0xF>(v);
    v += dpp<0x141, 0xF>(v);
    if constexpr (QP >= 16) v += dpp<0x140, 0xF>(v);
    if constexpr (QP == 32) v += __shfl_xor(v, 16);
    return v;
  }
}
template <int QP>
__device__ __forceinline__ float2 gsum(float2 v) { return make_float2(gsum<QP>(v.x), gsum<QP>(v.y)); }
template <int QP>
__device__ __forceinline__ double gsum(double v) {
  if constexpr (QP == 64) {
    return wsumd(v);
  } else {
    v += dppd<0xB1, 0xF>(v);
    v += dppd<0x4E, 0xF>(v);
    v += dppd<0x141, 0xF>(v);
    if constexpr (QP >= 16) v += dppd<0x140, 0xF>(v);
    if constexpr (QP == 32) v += __shfl_xor(v, 16);
    return v;
  }
}
template <int QP>
__device__ __forceinline__ double2 gsum(double2 v) { return make_double2(gsum<QP>(v.x), gsum<QP>(v.y)); }

// ------------------------------------------------- small Hermitian subspaces
// Lanes are split into groups of QP; in each group lane k (< d) holds row k of
// a d x r block W.  Orthonormalise the columns inside every group by
// classical Gram-Schmidt with one re-orthogonalisation pass (CGS2).
template <typename S> __device__ __forceinline__ S tiny();
template <> __device__ __forceinline__ float tiny<float>() { return 1e-30f; }
template <> __device__ __forceinline__ double tiny<double>() { return 1e-280; }

template <int RM, int QP, typename C>
__device__ __forceinline__ void orth_cgs2(C (&w)[RM], int r, bool act) {
  using S = decltype(C{}.x);
#pragma unroll
  for (int c = 0; c < RM; ++c) {
    if (c >= r) continue;
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      // classical GS: every projection uses the column as it entered the
      // pass (w0), applied as soon as it is known (one coefficient live)
      const C w0 = w[c];
#pragma unroll
      for (int a = 0; a < c; ++a) {
        const C h = gsum<QP>(act ? ccfma(w[a], w0, czero<C>()) : czero<C>());
        if (act) w[c] = csub(w[c], cmul(w[a], h));
      }
    }
    const S nn = gsum<QP>(act ? cabs2(w[c]) : S(0));
    const S inv = xrsqrt(xmax(nn, tiny<S>()));
    w[c] = act ? cscale(w[c], inv) : czero<C>();
  }
}

// A solve that starts from another matrix's basis V stops once M V lies in the
// span of V, and that holds for every invariant subspace: where the leading
// directions of M are orthogonal to V (training sets with exact zeros: samples
// or channels that are empty on one side of an edge), the iteration would keep
// a subspace that is not the leading one, or none at all where M V = 0.  A
// direction missing from V has at most the eigenvalue tr M - tr V^H M V (M is
// positive semidefinite), so the first step checks that this is far below every
// column's Rayleigh quotient, as it is for clutter of the plan's rank; where
// that holds nothing changes.  Where it does not, the solve goes on from M V
// with generic directions added at `mix` times each column's size: the next
// residual sees a missing direction unless its eigenvalue lies within the
// tolerance over `mix` of a kept one.  mix = 0 starts anew, from the generic
// block: LR-Kron goes on from the result of its first EIG_{r_a}, so between two
// nearly equal eigenvalues it has to be the larger one's and not the
// neighbour's that comes out ahead when the steps are used up.  Its later ones
// start from the pixel's own iterate, some 1e-2 to 1e-3 off, and mix no more.
//   Measured with and without the check (results the same bit for bit): 64 x 64,
// q = 8 92.1 / 90.8 us; 2048 x 2048, q = 16 22.70 / 22.52 ms; a batch of 12 tiles
// 4.85 / 4.77 ms; two passes of p = 6, q = 16 at 256 x 256 6.76 / 6.66 ms; noise
// alone at 512 x 512, where every start is mixed, 38.0 / 37.5 ms.
constexpr float kMixNeighbour = 1.f / 16.f, kMixOwn = 1e-3f;
constexpr float kCaptured = 64.f;   // least Rayleigh quotient over the trace outside V
// The check for lane groups whose rows lie as in group_subspace, w = M v;
// `guard` is the same in all rows of a group.  Returns whether this lane's group
// got another w.
template <int RM, int QP, int D, typename C>
__device__ __forceinline__ bool guard_start(const float2 (&mrow)[D], const C (&v)[RM], C (&w)[RM], int r, int k,
                                            bool row_ok, bool guard, float mix) {
  using S = decltype(C{}.x);
  asm volatile("" : "+v"(k));   // nothing of this is hoisted out of the iteration
  float diag = 0.f;
#pragma unroll
  for (int l = 0; l < D; ++l) diag = (l == k) ? mrow[l].x : diag;
  const S tr = gsum<QP>(S(row_ok ? diag : 0.f));
  S rest = tr, least = tr;
#pragma unroll
  for (int c = 0; c < RM; ++c) {
    if (c >= r) continue;
    const S t = gsum<QP>(row_ok ? v[c].x * w[c].x + v[c].y * w[c].y : S(0));
    rest -= t;
    least = t < least ? t : least;
  }
  const bool lost = guard && !(S(kCaptured) * rest <= least);
  if (__ballot(lost) == 0) return false;
#pragma unroll
  for (int c = 0; c < RM; ++c) {
    if (c >= r) continue;
    const S t = gsum<QP>(row_ok ? v[c].x * w[c].x + v[c].y * w[c].y : S(0));
    const C g = cto<C>(omega(k, c));
    if (lost && row_ok) w[c] = mix > 0.f ? cadd(w[c], cscale(g, S(mix) * xmax(t, tr / S(D)))) : g;
  }
  return lost;
}

// Top-r invariant subspace of one Hermitian D x D matrix per lane group by
// subspace iteration.  Lane k of a group holds row k of the matrix (mrow) and
// row k of the orthonormal basis v (CGS2 orthonormalisation).  `cold` starts from M * Omega (Omega a
// fixed generic block), except in the groups whose lanes set `keep`, which
// take M * v instead (v a neighbouring pixel's basis, which does not pass
// the test on its own); otherwise v is the warm start of every group.  A group has converged
// when ||M V - V (V^H M V)||_F <= tol ||M V||_F for the basis entering a step;
// that step's orthonormalised M V is kept and the group's basis is frozen.
// The loop runs until every group has converged or max_steps; each group's
// result is the one it would reach alone.  sV: LDS scratch of RM * D * (64 / QP) C
// for this wavefront.  WAVE_LOCAL: the wavefront shares its workgroup with
// others that run their own solves, so it synchronises only its own lanes.
// `guard`: the start block is another matrix's basis (guard_start, with `mix`).
template <int RM, int QP, int D, typename C, bool WAVE_LOCAL = false>
__device__ __forceinline__ int group_subspace(const float2 (&mrow)[D], bool row_ok, int r, C (&v)[RM],
                                              C* sV, bool cold, int max_steps, double tol, bool keep = false,
                                              bool guard = false, float mix = 0.f) {
  using S = decltype(C{}.x);
  constexpr int G = 64 / QP;
  const int lane = threadIdx.x & 63, g = lane / QP, k = lane % QP;   // lane within its wavefront
  if (cold) {
    // FP64 solves: recompute the start block on every call (an empty asm
    // makes the row index opaque); hoisted out of the pixel loop, its
    // widened values would be spilled and reloaded instead
    int kk = k;
    if constexpr (sizeof(S) == 8) asm volatile("" : "+v"(kk));
#pragma unroll
    for (int c = 0; c < RM; ++c)
      if (!keep) v[c] = (row_ok && c < r) ? cto<C>(omega(kk, c)) : czero<C>();
  }
  // a start block (Omega, or a kept v) is not tested on the first step
  bool tested = !cold;
  bool done = false;
  int step = 0;
  while (true) {
    if (row_ok) {
#pragma unroll
      for (int c = 0; c < RM; ++c)
        if (c < r) sV[(c * D + k) * G + g] = v[c];
    }
    lds_sync<WAVE_LOCAL>();
    C w[RM];
#pragma unroll
    for (int c = 0; c < RM; ++c) w[c] = czero<C>();
    if (row_ok) {
#pragma unroll
      for (int l = 0; l < D; ++l) {
        float2 m = mrow[l];
        // keep the widening of the matrix row inside the loop (an empty asm
        // makes the value opaque), so it is not hoisted into extra registers
        asm volatile("" : "+v"(m.x), "+v"(m.y));
        const C mc = cto<C>(m);
#pragma unroll
        for (int c = 0; c < RM; ++c)
          if (c < r) w[c] = cfma(mc, sV[(c * D + l) * G + g], w[c]);
      }
    }
    lds_sync<WAVE_LOCAL>();
    bool conv = false;
    if (tested) {
      // residual W - V (V^H W), one column at a time
      S rn = 0, wn = 0;
#pragma unroll
      for (int b = 0; b < RM; ++b) {
        if (b >= r) continue;
        C rr = w[b];
#pragma unroll
        for (int a = 0; a < RM; ++a) {
          if (a >= r) continue;
          const C hb = gsum<QP>(row_ok ? ccfma(v[a], w[b], czero<C>()) : czero<C>());
          rr = csub(rr, cmul(v[a], hb));
        }
        if (row_ok) {
          rn += cabs2(rr);
          wn += cabs2(w[b]);
        }
      }
      rn = gsum<QP>(rn);
      wn = gsum<QP>(wn);
      conv = rn <= S(tol * tol) * wn;
    }
    if (step == 0 && __ballot(guard)) conv = !guard_start<RM, QP, D, C>(mrow, v, w, r, k, row_ok, guard, mix) && conv;
    orth_cgs2<RM, QP, C>(w, r, row_ok);
    // a group keeps the first basis computed from a converged one and is
    // frozen from then on, so its result does not depend on its neighbours
    if (!done) {
#pragma unroll
      for (int c = 0; c < RM; ++c) v[c] = w[c];
    }
    done = done || conv;
    tested = true;
    ++step;
    if (__ballot(!done) == 0 || step >= max_steps) break;
  }
  return step;
}

// Top-r invariant subspace of a small Hermitian P x P matrix (the factor A),
// computed identically by every lane with no cross-lane traffic: the
// subspace iteration, CGS2 and stopping rule of group_subspace, on a matrix
// read through M(i, j).  V[c][i] is entry i of basis column c; `cold` starts
// from M * Omega, otherwise V is the warm start, checked as by guard_start with
// `mix`.  Returns the step count.
template <int RM, int P, typename C, typename MF>
__device__ __forceinline__ int uniform_subspace(MF M, int r, C (&V)[RM][P], bool cold, int max_steps, double tol,
                                                float mix) {
  using S = decltype(C{}.x);
  if (cold) {
#pragma unroll
    for (int c = 0; c < RM; ++c)
#pragma unroll
      for (int i = 0; i < P; ++i) V[c][i] = (c < r) ? cto<C>(omega(i, c)) : czero<C>();
  }
  bool tested = !cold;
  bool done = false;
  int step = 0;
  while (true) {
    C Wm[RM][P];
#pragma unroll
    for (int c = 0; c < RM; ++c)
#pragma unroll
      for (int i = 0; i < P; ++i) {
        C sacc = czero<C>();
        if (c < r) {
#pragma unroll
          for (int j = 0; j < P; ++j) sacc = cfma(M(i, j), V[c][j], sacc);
        }
        Wm[c][i] = sacc;
      }
    bool conv = false;
    if (tested) {
      // residual W - V (V^H W)
      S rn = 0, wn = 0;
#pragma unroll
      for (int b = 0; b < RM; ++b) {
        if (b >= r) continue;
        C hb[RM];
#pragma unroll
        for (int a = 0; a < RM; ++a) {
          C d = czero<C>();
          if (a < r) {
#pragma unroll
            for (int i = 0; i < P; ++i) d = ccfma(V[a][i], Wm[b][i], d);
          }
          hb[a] = d;
        }
#pragma unroll
        for (int i = 0; i < P; ++i) {
          C rr = Wm[b][i];
#pragma unroll
          for (int a = 0; a < RM; ++a)
            if (a < r) rr = csub(rr, cmul(V[a][i], hb[a]));
          rn += cabs2(rr);
          wn += cabs2(Wm[b][i]);
        }
      }
      conv = rn <= S(tol * tol) * wn;
    }
    if (step == 0 && !cold) {   // as guard_start
      S tr = 0, t[RM];
#pragma unroll
      for (int i = 0; i < P; ++i) tr += M(i, i).x;
      S rest = tr, least = tr;
#pragma unroll
      for (int c = 0; c < RM; ++c) {
        t[c] = 0;
        if (c >= r) continue;
#pragma unroll
        for (int i = 0; i < P; ++i) t[c] += V[c][i].x * Wm[c][i].x + V[c][i].y * Wm[c][i].y;
        rest -= t[c];
        least = t[c] < least ? t[c] : least;
      }
      if (!(S(kCaptured) * rest <= least)) {
        conv = false;
#pragma unroll
        for (int c = 0; c < RM; ++c)
#pragma unroll
          for (int i = 0; i < P; ++i) {
            int ii = i;
            asm volatile("" : "+v"(ii));   // computed here, not hoisted into every solve
            const C g = (c < r) ? cto<C>(omega(ii, c)) : czero<C>();
            Wm[c][i] = mix > 0.f ? cadd(Wm[c][i], cscale(g, S(mix) * xmax(t[c], tr / S(P)))) : g;
          }
      }
    }
    // CGS2 on the columns of W
#pragma unroll
    for (int c = 0; c < RM; ++c) {
      if (c >= r) continue;
#pragma unroll
      for (int pass = 0; pass < 2; ++pass) {
        C h[RM];
#pragma unroll
        for (int a = 0; a < RM; ++a) {
          C d = czero<C>();
          if (a < c) {
#pragma unroll
            for (int i = 0; i < P; ++i) d = ccfma(Wm[a][i], Wm[c][i], d);
          }
          h[a] = d;
        }
#pragma unroll
        for (int i = 0; i < P; ++i)
#pragma unroll
          for (int a = 0; a < RM; ++a)
            if (a < c) Wm[c][i] = csub(Wm[c][i], cmul(Wm[a][i], h[a]));
      }
      S nn = 0;
#pragma unroll
      for (int i = 0; i < P; ++i) nn += cabs2(Wm[c][i]);
      const S inv = xrsqrt(xmax(nn, tiny<S>()));
#pragma unroll
      for (int i = 0; i < P; ++i) Wm[c][i] = cscale(Wm[c][i], inv);
    }
    // as in group_subspace: keep the first basis computed from a converged one
    if (!done) {
#pragma unroll
      for (int c = 0; c < RM; ++c)
#pragma unroll
        for (int i = 0; i < P; ++i) V[c][i] = Wm[c][i];
    }
    done = done || conv;
    tested = true;
    ++step;
    if (done || step >= max_steps) break;
  }
  return step;
}

// The check of guard_start for one vector, at the first step of a solve: lam =
// u^H M u stands out from the trace of M, so no direction outside u has a larger
// eigenvalue.  Where it does not, the step's result w gives way to the cold start
// (a column of M) if u was a neighbour's (`first`: a pixel's first solve), and
// takes a generic direction: a cold start may itself be an eigenvector of a
// smaller eigenvalue.
template <typename S>
__device__ __forceinline__ bool stands_out(S lam, S tr) {
  return S(4) * (tr - lam) <= lam;
}
// the generic direction, as constants (computed, it would be hoisted into every
// solve)
__device__ constexpr float kGeneric[kMaxP][2] = {{0.80f, -0.60f}, {-0.25f, 0.86f}, {0.66f, 0.88f}, {-0.77f, -0.22f},
                                                 {0.91f, 0.27f}, {-0.45f, 0.60f}, {0.31f, -1.06f}, {-0.88f, 0.47f}};
// w, or column j (read through M(i, j)) of the largest diagonal entry, plus the
// generic direction; returns the squared norm
template <int P, typename C, typename S, typename MF>
__device__ __forceinline__ S start_anew(MF M, C (&w)[P], S lam, S tr, bool cold, bool first) {
  if (first && !cold) {
    S db = M(0, 0).x;
#pragma unroll
    for (int j = 0; j < P; ++j) {
      const bool up = j == 0 || M(j, j).x > db;
      db = up ? M(j, j).x : db;
#pragma unroll
      for (int i = 0; i < P; ++i) w[i] = up ? M(i, j) : w[i];
    }
  }
  const S mix = S(first ? kMixNeighbour : kMixOwn) * xmax(lam, tr / S(P));
  S wn = 0;
#pragma unroll
  for (int i = 0; i < P; ++i) {
    w[i] = cadd(w[i], cscale(cto<C>(make_float2(kGeneric[i][0], kGeneric[i][1])), mix));
    wn += cabs2(w[i]);
  }
  return wn;
}

// Dominant eigenvector of a Hermitian P x P matrix, the same for every lane;
// M(i, j) returns its entries (registers or LDS).  Power iteration; stop on
// ||M u - (u^H M u) u|| <= tol ||M u||.
template <int P, typename C, typename MF>
__device__ __forceinline__ void power_top(MF M, C (&u)[P], bool cold, int max_steps, double tol) {
  using S = decltype(C{}.x);
  if (cold) {
    int jb = 0;
    S db = M(0, 0).x;
#pragma unroll
    for (int j = 1; j < P; ++j)
      if (M(j, j).x > db) {
        db = M(j, j).x;
        jb = j;
      }
#pragma unroll
    for (int i = 0; i < P; ++i) {
      C s = czero<C>();
#pragma unroll
      for (int j = 0; j < P; ++j) s = (j == jb) ? M(i, j) : s;
      u[i] = s;
    }
    S nn = 0;
#pragma unroll
    for (int i = 0; i < P; ++i) nn += cabs2(u[i]);
    const S inv = nn > S(0) ? xrsqrt(xmax(nn, tiny<S>())) : S(0);
#pragma unroll
    for (int i = 0; i < P; ++i) u[i] = cscale(u[i], inv);
  }
  for (int step = 0; step < max_steps; ++step) {
    C w[P];
    S lam = 0, wn = 0;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      C s = czero<C>();
#pragma unroll
      for (int j = 0; j < P; ++j) s = cfma(M(i, j), u[j], s);
      w[i] = s;
      lam += u[i].x * s.x + u[i].y * s.y;
      wn += cabs2(s);
    }
    S rn = 0;
#pragma unroll
    for (int i = 0; i < P; ++i) rn += cabs2(csub(w[i], cscale(u[i], lam)));
    if (!(wn > S(0))) break;
    const S inv = xrsqrt(xmax(wn, tiny<S>()));
#pragma unroll
    for (int i = 0; i < P; ++i) u[i] = cscale(w[i], inv);
    if (rn <= S(tol * tol) * wn) break;
  }
}

// Hermitian P x P matrices as P*P reals: the diagonal, then (Re, Im) of each
// entry (i, j), i < j, at hoff(i, j).
template <int P>
__host__ __device__ constexpr int hoff(int i, int j) { return P + 2 * (i * P - i * (i + 1) / 2 + (j - i - 1)); }

// power_top for a matrix given by its P*P reals (half the multiplications of
// the general complex product); *lam receives u^H M u of the last iterate
// tested, whose error is the square of the stopping residual.
template <int P, typename C, typename S>
__device__ __forceinline__ void power_top_h(const S (&h)[P * P], C (&u)[P], bool cold, bool first, int max_steps,
                                            double tol, S* lam_out) {
  if (cold) {   // the column of the largest diagonal entry
    int jb = 0;
    S db = h[0];
#pragma unroll
    for (int j = 1; j < P; ++j)
      if (h[j] > db) {
        db = h[j];
        jb = j;
      }
    S nn = 0;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      C s = czero<C>();
#pragma unroll
      for (int j = 0; j < P; ++j) {
        if (j != jb) continue;
        if (j == i) s.x = h[i];
        else if (i < j) s.x = h[hoff<P>(i, j)], s.y = h[hoff<P>(i, j) + 1];
        else s.x = h[hoff<P>(j, i)], s.y = -h[hoff<P>(j, i) + 1];
      }
      u[i] = s;
      nn += cabs2(s);
    }
    const S inv = nn > S(0) ? xrsqrt(xmax(nn, tiny<S>())) : S(0);
#pragma unroll
    for (int i = 0; i < P; ++i) u[i] = cscale(u[i], inv);
  }
  S lam = 0;
  for (int step = 0; step < max_steps; ++step) {
    C w[P];
#pragma unroll
    for (int i = 0; i < P; ++i) w[i] = cscale(u[i], h[i]);
#pragma unroll
    for (int i = 0; i < P; ++i)
#pragma unroll
      for (int j = i + 1; j < P; ++j) {
        C m;
        m.x = h[hoff<P>(i, j)];
        m.y = h[hoff<P>(i, j) + 1];
        w[i] = cfma(m, u[j], w[i]);
        w[j] = ccfma(m, u[i], w[j]);
      }
    S wn = 0, rn = 0;
    lam = 0;
#pragma unroll
    for (int i = 0; i < P; ++i) {
      lam += u[i].x * w[i].x + u[i].y * w[i].y;
      wn += cabs2(w[i]);
    }
#pragma unroll
    for (int i = 0; i < P; ++i) rn += cabs2(csub(w[i], cscale(u[i], lam)));
    if (step == 0) {
      S tr = 0;
#pragma unroll
      for (int i = 0; i < P; ++i) tr += h[i];
      if (!stands_out(lam, tr))
        rn = wn = start_anew<P, C, S>(
            [&](int i, int j) __attribute__((always_inline)) {
              C m;
              m.x = i == j ? h[i] : i < j ? h[hoff<P>(i, j)] : h[hoff<P>(j, i)];
              m.y = i == j ? S(0) : i < j ? h[hoff<P>(i, j) + 1] : -h[hoff<P>(j, i) + 1];
              return m;
            },
            w, lam, tr, cold, first);
    }
    if (!(wn > S(0))) break;
    const S inv = xrsqrt(xmax(wn, tiny<S>()));
#pragma unroll
    for (int i = 0; i < P; ++i) u[i] = cscale(w[i], inv);
    if (rn <= S(tol * tol) * wn) break;
  }
  *lam_out = lam;
}

// Training-vector load.  Lanes whose element does not exist (rows past p*q,
// vectors past n) read a zero from kZeroVec instead of taking a branch, so
// every load is issued unconditionally and its value is used as loaded.
// Without branches around the loads the compiler counts the loads in flight
// exactly and waits only for the ones an MFMA is about to consume, which
// keeps the prefetch ring full.
__device__ float2 kZeroVec[1];   // never written
__device__ __forceinline__ float2 load_or_zero(const float2* p, bool keep) {
  const float2* a = keep ? p : kZeroVec;
  return *a;
}

// Training vectors of the narrow kernels are read through buffer resources:
// one record per 16-row operand block, based at the pixel's window origin in
// the channel of the block's first row.  A lane's load offset is its row
// offset (loff) plus the stencil entry's byte offset (sOffB, in LDS).  Rows
// past p*q and entries past n carry kOut, which lies beyond every record, so
// the hardware returns zeros for them: no branch, select or 64-bit address
// arithmetic per load.
constexpr uint32_t kOut = 0x80000000u;
constexpr int kOffPad = 64;   // sOffB entries past kMaxN (prefetch overrun, all kOut)
constexpr int kDeltaList = 2 * kMaxDelta + 32;   // a move's entering, then leaving vectors, then kOut

template <int Q>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t block_rsrc(const float2* xwin, int64_t plane, uint32_t rec, int I) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)(xwin + int64_t((16 * I) / Q) * plane), (short)0, int(rec),
                                           0x00020000);
}
__device__ __forceinline__ float2 bload(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}

// Narrow kernels keep S in LDS as its upper q x q blocks S(i, j), i <= j, with
// a padded row stride q + 1 (the lower blocks are their conjugate
// transposes); block (i, j) starts at sblk(i, j).
template <int P, int Q>
__device__ __forceinline__ int sblk(int i, int j) {
  return (i * P - i * (i - 1) / 2 + (j - i)) * Q * (Q + 1);
}
template <int P, int Q>
__device__ __forceinline__ float2 sget(const float2* sS, int i, int j, int k, int l) {
  if (i <= j) return sS[sblk<P, Q>(i, j) + k * (Q + 1) + l];
  const float2 v = sS[sblk<P, Q>(j, i) + l * (Q + 1) + k];
  return make_float2(v.x, -v.y);
}
// Stores element (a, b), a <= b, of the stacked pq x pq matrix (and, inside a
// diagonal block, its mirror).  Only elements with a <= b are written, so
// every position has exactly one writer.
template <int P, int Q>
__device__ __forceinline__ void sput(float2* sS, int a, int b, float2 v) {
  const int ba = a / Q, ka = a - ba * Q, bb = b / Q, kb = b - bb * Q;
  sS[sblk<P, Q>(ba, bb) + ka * (Q + 1) + kb] = v;
  if (ba == bb) sS[sblk<P, Q>(ba, bb) + kb * (Q + 1) + ka] = make_float2(v.x, -v.y);
}

// Block sums of S and the lane's part of ||S||_F^2, gathered while S is
// stored (for q a multiple of 16, where every 16 x 16 tile lies in one q x q
// block): a0[i*P + j] = sum_kl S(i,j)_kl for i <= j (a lower block's sum is
// the conjugate), each element counted with its mirror.
template <int P>
struct SSums {
  float2 a0[P * P];
  float nr;
};
// off: the element is not on the diagonal of S.
template <int P, int Q>
__device__ __forceinline__ void ssums_add(SSums<P>& ss, int I, int J, bool off, float2 v) {
  if constexpr (Q % 16 == 0) {
    const int bi = (16 * I) / Q, bj = (16 * J) / Q;   // constants once the tile loops unroll
    const float m = cabs2(v);
    if (bi != bj) {
      ss.a0[bi * P + bj] = cadd(ss.a0[bi * P + bj], v);
      ss.nr += 2.f * m;
    } else if (off) {
      ss.a0[bi * P + bi].x += 2.f * v.x;   // v + conj(v)
      ss.nr += 2.f * m;
    } else {
      ss.a0[bi * P + bi] = cadd(ss.a0[bi * P + bi], v);
      ss.nr += m;
    }
  }
}

// Element (tr, tc) of the 16 x 16 MFMA tile (I, J), I <= J: row 16 I + tr,
// column 16 J + tc of the stacked matrix, 0 <= tr, tc < 16.  Written so that
// what the tile indices fix (the tile lies inside the matrix, above its
// diagonal, inside one q x q block) folds once the tile loops unroll: only
// diagonal and ragged tiles test their lanes, and no per-lane predicate of
// an off-diagonal tile is kept live across the pixel loop.
template <int P, int Q>
__device__ __forceinline__ bool tile_in(int I, int J, int tr, int tc) {
  constexpr int PQ = P * Q;
  return (16 * I + 16 <= PQ || 16 * I + tr < PQ) && (16 * J + 16 <= PQ || 16 * J + tc < PQ);
}
// inside the matrix and on or above its diagonal (row == col iff I == J and
// tr == tc, since |tc - tr| < 16)
template <int P, int Q>
__device__ __forceinline__ bool tile_keep(int I, int J, int tr, int tc) {
  return tile_in<P, Q>(I, J, tr, tc) && (J > I || tr <= tc);
}
template <int P, int Q>
__device__ __forceinline__ float2 tile_get(const float2* sS, int I, int J, int tr, int tc) {
  if constexpr (Q % 16 == 0) {   // the tile lies in upper block ((16 I) / q, (16 J) / q)
    return sS[sblk<P, Q>((16 * I) / Q, (16 * J) / Q) + ((16 * I) % Q + tr) * (Q + 1) + (16 * J) % Q + tc];
  } else {
    const int row = 16 * I + tr, col = 16 * J + tc;
    return sget<P, Q>(sS, row / Q, col / Q, row % Q, col % Q);
  }
}
// sput of a tile element that tile_keep accepts
template <int P, int Q>
__device__ __forceinline__ void tile_put(float2* sS, int I, int J, int tr, int tc, float2 v) {
  if constexpr (Q % 16 == 0) {
    const int bi = (16 * I) / Q, bj = (16 * J) / Q;
    const int ka = (16 * I) % Q + tr, kb = (16 * J) % Q + tc;
    sS[sblk<P, Q>(bi, bj) + ka * (Q + 1) + kb] = v;
    if (bi == bj) sS[sblk<P, Q>(bi, bj) + kb * (Q + 1) + ka] = make_float2(v.x, -v.y);
  } else {
    sput<P, Q>(sS, 16 * I + tr, 16 * J + tc, v);
  }
}

// ------------------------------------------------------------ a2, FP32
// Classes where the tile row and column are made opaque, so that the S
// element addresses and the diagonal tiles' lane masks are formed where used,
// per pixel, instead of being hoisted out of the pixel loop, spilled and
// reloaded: q a multiple of 16 (one base address per lane, the tile offsets
// are constants), and the classes whose addresses do not fit in registers
// beside the rest of the pixel state.
template <int P, int Q>
constexpr bool kOpaqueStore = Q % 16 == 0 || (P == 3 && Q == 12) || (P == 4 && Q == 8) || (P == 6 && Q == 8);

// S = (1/n) sum_m x_m x_m^H of one pixel on v_mfma_f32_16x16x4_f32, written
// to LDS as the full Hermitian pq x pq matrix (row-major).
template <int P, int Q>
__device__ __forceinline__ void scm_fp32(const float2* xwin, int64_t plane, uint32_t rec, const uint32_t* sOffB,
                                         const uint32_t (&loff)[(P * Q + 15) / 16], int n, float2* sS,
                                         float* sP, SSums<P>& ss) {
  constexpr int PQ = P * Q;
  constexpr int NB = (PQ + 15) / 16;
  constexpr int NT = NB * (NB + 1) / 2;
  constexpr int NO = NB * (NB - 1) / 2;
  const int lane = threadIdx.x;
    f4 accR[NT], accI[NO > 0 ? NO : 1], accD[NB];
#pragma unroll
    for (int t = 0; t < NT; ++t) accR[t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < (NO > 0 ? NO : 1); ++t) accI[t] = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NB; ++t) accD[t] = f4{0.f, 0.f, 0.f, 0.f};

    const int nch = (n + 3) >> 2;
    // operand ring: chunk ch lives in slot ch % PF; PF - 1 chunks in flight
    constexpr int PF = 4;
    float2 ring[PF][NB];
    __amdgpu_buffer_rsrc_t rs[NB];
#pragma unroll
    for (int I = 0; I < NB; ++I) rs[I] = block_rsrc<Q>(xwin, plane, rec, I);
    auto fetch = [&](int ch, float2 (&v)[NB]) {
      const uint32_t off = sOffB[ch * 4 + (lane >> 4)];
#pragma unroll
      for (int I = 0; I < NB; ++I) v[I] = bload(rs[I], loff[I] + off);
    };
    // MFMAs of one 4-vector chunk
    auto accumulate = [&](const float2 (&v)[NB]) {
      float xr[NB], xi[NB], nxr[NB];
#pragma unroll
      for (int I = 0; I < NB; ++I) {
        xr[I] = v[I].x;
        xi[I] = v[I].y;
        nxr[I] = -v[I].x;
      }
      // first product of every accumulator, then the second: no two
      // consecutive MFMAs write the same accumulator
      {
        int t = 0, u = 0;
#pragma unroll
        for (int I = 0; I < NB; ++I)
#pragma unroll
          for (int J = I; J < NB; ++J) {
            accR[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(xr[I], xr[J], accR[t], 0, 0, 0);
            if (J > I) {
              accI[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(xi[I], xr[J], accI[u], 0, 0, 0);
              ++u;
            } else {
              accD[I] = __builtin_amdgcn_mfma_f32_16x16x4f32(xi[I], xr[I], accD[I], 0, 0, 0);
            }
            ++t;
          }
      }
      {
        int t = 0, u = 0;
#pragma unroll
        for (int I = 0; I < NB; ++I)
#pragma unroll
          for (int J = I; J < NB; ++J) {
            accR[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(xi[I], xi[J], accR[t], 0, 0, 0);
            if (J > I) {
              accI[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(nxr[I], xi[J], accI[u], 0, 0, 0);
              ++u;
            }
            ++t;
          }
      }
    };
#pragma unroll
    for (int s0 = 0; s0 < PF - 1; ++s0) {   // in order: oldest chunk's loads first
      __builtin_amdgcn_sched_barrier(0);
      fetch(s0, ring[s0]);
    }
    // whole groups of PF chunks: branch-free, so the loads of the ring are
    // waited for one chunk at a time (fetches past n read zeros)
    int ch0 = 0;
    for (; ch0 + PF <= nch; ch0 += PF) {
#pragma unroll
      for (int sl = 0; sl < PF; ++sl) {
        // keep each chunk's instructions in place: hoisting work on a slot
        // that was just fetched would wait for its load right away
        __builtin_amdgcn_sched_barrier(0);
        fetch(ch0 + sl + PF - 1, ring[(sl + PF - 1) % PF]);
        accumulate(ring[sl]);
      }
    }
    // the last nch - ch0 < PF chunks are already in ring slots 0, 1, ...
#pragma unroll
    for (int sl = 0; sl < PF - 1; ++sl)
      if (ch0 + sl < nch) accumulate(ring[sl]);

    // S to LDS (upper blocks), scaled by 1/n.  MFMA output layout: lane l,
    // register q holds row 4*(l/16) + q, column l % 16 of the 16 x 16 tile.
    // Im of a diagonal tile is P - P^T with P = Xi Xr^T: the raw P goes through
    // the scratch sP ([NB][16][16]) for the transposed element.
    const float inv_n = 1.f / float(n);
    int trow = 4 * (lane >> 4), tcol = lane & 15;
    if constexpr (kOpaqueStore<P, Q>) asm volatile("" : "+v"(trow), "+v"(tcol));
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) sP[(I * 16 + trow + q4) * 16 + tcol] = accD[I][q4];
    wave_sync();
    {
      int t = 0, u = 0;
#pragma unroll
      for (int I = 0; I < NB; ++I) {
#pragma unroll
        for (int J = I; J < NB; ++J) {
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            const int tr = trow + q4;
            if (tile_keep<P, Q>(I, J, tr, tcol)) {
              const float re = accR[t][q4] * inv_n;
              const float im = (J > I) ? accI[u][q4] * inv_n
                                       : (accD[I][q4] - sP[(I * 16 + tcol) * 16 + tr]) * inv_n;
              tile_put<P, Q>(sS, I, J, tr, tcol, make_float2(re, im));
              ssums_add<P, Q>(ss, I, J, I != J || tr != tcol, make_float2(re, im));
            }
          }
          if (J > I) ++u;
          ++t;
        }
      }
    }
    wave_sync();
}

// Sliding-window update of S (FP32): from the previous pixel's S (in LDS),
// n S += sum over entering vectors x x^H - sum over leaving ones.  sAdd /
// sRem: byte offsets (kOut past nadd / nrem and for 8 entries beyond).
// Up to three 16-row blocks (where registers allow a third accumulator per
// tile), every tile takes three real products per chunk instead of four:
// with P1 = Xr Xr^T, P2 = Xi Xi^T and P3 = (Xr + Xi)(Xr - Xi)^T, Re S =
// P1 + P2 and Im S = P3 - P1 + P2, and the diagonal of S is stored real.
// Larger classes take Re and Im of every tile with two products each (no
// transpose through LDS).
template <int P, int Q>
__device__ __forceinline__ void scm_fp32_delta(const float2* xwin, int64_t plane, uint32_t rec,
                                               const uint32_t* sAdd, int nadd, const uint32_t* sRem, int nrem,
                                               const uint32_t (&loff)[(P * Q + 15) / 16], int n, float2* sS,
                                               SSums<P>& ss) {
  constexpr int PQ = P * Q;
  constexpr int NB = (PQ + 15) / 16;
  constexpr int NT = NB * (NB + 1) / 2;
  constexpr int NO = NB * (NB - 1) / 2;
  const int lane = threadIdx.x;
  int trow = 4 * (lane >> 4), tcol = lane & 15;
  if constexpr (kOpaqueStore<P, Q>) asm volatile("" : "+v"(trow), "+v"(tcol));
  const float fn = float(n);
  constexpr bool K3 = NB <= 3;
  // accR: Re (P1 in the three-product form); accI / accD: Im of the
  // off-diagonal / diagonal tiles (four-product form); p2, p3: P2 and P3
  f4 accR[NT], accI[(K3 || NO == 0) ? 1 : NO], accD[K3 ? 1 : NB];
  f4 p2[K3 ? NT : 1], p3[K3 ? NT : 1];
  // one chunk stream: the entering vectors' chunks, then the leaving ones';
  // chunk c + 1 is fetched while chunk c is accumulated.  Fetching one chunk
  // past the end reads the leaving list's kOut entries (KD > kMaxDelta + 6),
  // i.e. zeros, and is never used.
  const int na = (nadd + 3) >> 2, nch = na + ((nrem + 3) >> 2);
  __amdgpu_buffer_rsrc_t rs[NB];
#pragma unroll
  for (int I = 0; I < NB; ++I) rs[I] = block_rsrc<Q>(xwin, plane, rec, I);
  auto fetch = [&](int c, float2 (&v)[NB]) __attribute__((always_inline)) {
    const uint32_t off = (c < na ? sAdd + 4 * c : sRem + 4 * (c - na))[lane >> 4];
#pragma unroll
    for (int I = 0; I < NB; ++I) v[I] = bload(rs[I], loff[I] + off);
  };
  float2 vc[NB], vn[NB];
  fetch(0, vc);   // in flight while the old S is reloaded
  {
    int t = 0, u = 0;
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int J = I; J < NB; ++J) {
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int tr = trow + q4;
          float2 v = make_float2(0.f, 0.f);
          if (tile_in<P, Q>(I, J, tr, tcol)) v = tile_get<P, Q>(sS, I, J, tr, tcol);
          accR[t][q4] = v.x * fn;
          if constexpr (K3) {
            p2[t][q4] = 0.f;
            p3[t][q4] = (v.x + v.y) * fn;
          } else {
            if (J > I) accI[u][q4] = v.y * fn;
            else accD[I][q4] = v.y * fn;
          }
        }
        if (J > I) ++u;
        ++t;
      }
  }
#pragma unroll 1
  for (int ch = 0; ch < nch; ++ch) {
    {
      fetch(ch + 1, vn);
      const float sg = ch < na ? 1.f : -1.f;
      float2 v[NB];
#pragma unroll
      for (int I = 0; I < NB; ++I) v[I] = vc[I];
#pragma unroll
      for (int I = 0; I < NB; ++I) vc[I] = vn[I];
      if constexpr (K3) {
        float xr[NB], xi[NB], a1[NB], a2[NB], a3[NB], b3[NB];
#pragma unroll
        for (int I = 0; I < NB; ++I) {
          xr[I] = v[I].x;
          xi[I] = v[I].y;
          a1[I] = sg * v[I].x;
          a2[I] = sg * v[I].y;
          a3[I] = sg * (v[I].x + v[I].y);
          b3[I] = v[I].x - v[I].y;
        }
        int t = 0;
#pragma unroll
        for (int I = 0; I < NB; ++I)
#pragma unroll
          for (int J = I; J < NB; ++J, ++t) {
            accR[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[I], xr[J], accR[t], 0, 0, 0);
            p2[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a2[I], xi[J], p2[t], 0, 0, 0);
            p3[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a3[I], b3[J], p3[t], 0, 0, 0);
          }
        continue;
      }
      float xr[NB], xi[NB], sxr[NB], sxi[NB], nsxr[NB];
#pragma unroll
      for (int I = 0; I < NB; ++I) {
        xr[I] = v[I].x;
        xi[I] = v[I].y;
        sxr[I] = sg * v[I].x;
        sxi[I] = sg * v[I].y;
        nsxr[I] = -sxr[I];
      }
      int t = 0, u = 0;
#pragma unroll
      for (int I = 0; I < NB; ++I)
#pragma unroll
        for (int J = I; J < NB; ++J) {
          accR[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(sxr[I], xr[J], accR[t], 0, 0, 0);
          accR[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(sxi[I], xi[J], accR[t], 0, 0, 0);
          if (J > I) {
            accI[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(sxi[I], xr[J], accI[u], 0, 0, 0);
            accI[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(nsxr[I], xi[J], accI[u], 0, 0, 0);
            ++u;
          } else {
            accD[I] = __builtin_amdgcn_mfma_f32_16x16x4f32(sxi[I], xr[I], accD[I], 0, 0, 0);
            accD[I] = __builtin_amdgcn_mfma_f32_16x16x4f32(nsxr[I], xi[I], accD[I], 0, 0, 0);
          }
          ++t;
        }
    }
  }
  wave_sync();   // every lane has reloaded its part of the old S
  const float inv_n = 1.f / fn;
  {
    int t = 0, u = 0;
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int J = I; J < NB; ++J) {
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int tr = trow + q4;
          if (tile_keep<P, Q>(I, J, tr, tcol)) {
            float2 v;
            if constexpr (K3) {
              v.x = (accR[t][q4] + p2[t][q4]) * inv_n;
              v.y = (I == J && tr == tcol) ? 0.f : ((p3[t][q4] - accR[t][q4]) + p2[t][q4]) * inv_n;
            } else {
              v = make_float2(accR[t][q4] * inv_n, ((J > I) ? accI[u][q4] : accD[I][q4]) * inv_n);
            }
            tile_put<P, Q>(sS, I, J, tr, tcol, v);
            ssums_add<P, Q>(ss, I, J, I != J || tr != tcol, v);
          }
        }
        if (J > I) ++u;
        ++t;
      }
  }
  wave_sync();
}

// ------------------------------------------- a2, FP32 in three BF16 parts
// S of FP32 samples on the BF16 matrix pipe: x = h + m + l, each part the
// BF16 rounding of what the parts before it leave, is exact (8 + 8 + 8 bits
// with signs), and x y ~ hh' + hm' + mh' + mm' + hl' + lh' drops products
// below 2^-26 |x y|, a quarter of an FP32 rounding.  Every tile takes six
// products of Re and six of Im per 16 vectors, accumulated in FP32 (six
// roundings per 16 vectors instead of eight).  FP32 MFMA runs on the FMA
// units, so its time adds to the VALU's (measured: one wave of each on a SIMD
// take the sum of their times), while BF16 MFMA hides under the other
// wavefront's VALU work (17.5 cycles per MFMA with and without FMAs beside
// it): 72 x 16 matrix-pipe cycles per 16 vectors and three 16-row blocks, off
// the critical path, against 4 x 18 x 32 on it.
//   In a 16-vector chunk, lane (g = lane / 16, r = lane % 16) holds row r of
// every block for vectors 4g .. 4g + 3, packed in pairs: a row operand is
// (re_01, im_01, re_23, im_23).  The column operand of Re S has the same
// order; that of Im S = im re' - re im' is (-im_01, re_01, -im_23, re_23).  A
// leaving vector's column operands take its sign.  A remainder of up to 8
// vectors takes a half chunk (vectors 2g, 2g + 1) on the K = 16 MFMA.
//   S is kept as n S in the accumulators, and they stay in registers from one
// pixel of a sliding-window chain to the next where there is room (kKeepAcc).
// Measured against FP32 MFMA: 2048 x 2048, p = 3, q = 16, n = 200 32.9 -> 27.7
// ms; FP32 with FP64 solves (all n vectors per pixel) 512 x 512 5.87 -> 5.08
// ms; 187 x 233, q = 12, n = 128 627 -> 501 us; errors against FP64 the same
// or smaller.  Classes of four 16-row blocks keep FP32 MFMA: their operands
// and 20 accumulators do not fit beside the pixel state.
template <int P, int Q>
constexpr bool kSplitCov = (P * Q + 15) / 16 <= 3;
template <int P, int Q>
constexpr bool kKeepAcc = kSplitCov<P, Q> && P <= 4;

template <int P, int Q>
struct SplitAcc {
  static constexpr int NB = (P * Q + 15) / 16;
  static constexpr int NT = NB * (NB + 1) / 2;
  f4 r[NT], i[NT];   // Re and Im of n S, tile (I, J) at I NB - I (I - 1) / 2 + J - I
};

typedef __bf16 bf8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf2 __attribute__((ext_vector_type(2)));
typedef float f2v __attribute__((ext_vector_type(2)));
typedef unsigned int u4 __attribute__((ext_vector_type(4)));
typedef unsigned int u2 __attribute__((ext_vector_type(2)));
typedef short s4 __attribute__((ext_vector_type(4)));

template <int V>
struct Int {   // a constant as a lambda's argument
  static constexpr int value = V;
};

// the three BF16 parts of a (low halves) and b (high halves)
__device__ __forceinline__ void split3(float a, float b, uint32_t (&part)[3]) {
#pragma unroll
  for (int e = 0; e < 3; ++e) {
    const f2v ab{a, b};
    part[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(ab, bf2));
    if (e < 2) {
      a -= __builtin_bit_cast(float, part[e] << 16);
      b -= __builtin_bit_cast(float, part[e] & 0xffff0000u);
    }
  }
}

// Raw samples of a chunk: rows of block I, vectors e of this lane.
template <int P, int Q>
struct SplitRaw {
  float2 v[(P * Q + 15) / 16][4];
};
// A list of cnt vectors takes split_full(cnt) whole chunks (a remainder of 9
// to 15 vectors fills one, zeros past cnt) and, for a remainder of 1 to 8, a
// half chunk, whose vectors lie in the list two to a group of four entries
// (4g, 4g + 1: vectors 2g, 2g + 1 of the half chunk), so that every chunk is
// fetched the same way.
__device__ __forceinline__ int split_full(int cnt) { return (cnt + 7) >> 4; }
// The vector at list entry m, or -1.
__device__ __forceinline__ int split_entry(int m, int cnt) {
  const int whole = 16 * split_full(cnt);
  if (m >= whole) m = (m & 3) < 2 ? whole + 2 * ((m - whole) >> 2) + (m & 3) : cnt;
  return m < cnt ? m : -1;
}

// n S += sum over the vectors [0, npos) - sum over [npos, cnt) of a list of
// byte offsets in LDS (entries as split_entry, kOut where there is no vector;
// the chunk past the last is fetched and unused).  PF chunks are in flight:
// one where another wavefront fills the wait and the windows are in L2 (run
// mode); three for the pixel lists of the probe, whose windows come from HBM
// (no leaving vectors there).
template <int P, int Q, int PF>
__device__ __forceinline__ void scm_split(const float2* xwin, int64_t plane, uint32_t rec, const uint32_t* list,
                                          int npos, int cnt, const uint32_t (&loff)[(P * Q + 15) / 16],
                                          SplitAcc<P, Q>& acc) {
  constexpr int NB = SplitAcc<P, Q>::NB;
  const int g = threadIdx.x >> 4;
  __amdgpu_buffer_rsrc_t rs[NB];
#pragma unroll
  for (int I = 0; I < NB; ++I) rs[I] = block_rsrc<Q>(xwin, plane, rec, I);
  auto fetch = [&](int ch, SplitRaw<P, Q>& v) __attribute__((always_inline)) {
    const uint4 o = *reinterpret_cast<const uint4*>(list + 16 * ch + 4 * g);
    const uint32_t off[4] = {o.x, o.y, o.z, o.w};
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int I = 0; I < NB; ++I) v.v[I][e] = bload(rs[I], loff[I] + off[e]);
  };
  // MFMAs of one chunk of V vectors per lane; sign[k]: sign bits of the pair k;
  // `then` runs once the raw samples are consumed
  auto accumulate = [&](auto vc, const SplitRaw<P, Q>& raw, const uint32_t (&sign)[2], auto then)
                        __attribute__((always_inline)) {
    constexpr int V = decltype(vc)::value;
    uint32_t y[NB][3][V];
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int k = 0; k < V / 2; ++k) {
        uint32_t re[3], im[3];
        split3(raw.v[I][2 * k].x, raw.v[I][2 * k + 1].x, re);
        split3(raw.v[I][2 * k].y, raw.v[I][2 * k + 1].y, im);
#pragma unroll
        for (int e = 0; e < 3; ++e) {
          y[I][e][2 * k] = re[e];
          y[I][e][2 * k + 1] = im[e];
        }
      }
    __builtin_amdgcn_sched_barrier(0);
    then();
    __builtin_amdgcn_sched_barrier(0);
    constexpr int pa[6] = {2, 0, 1, 1, 0, 0}, pb[6] = {0, 2, 1, 0, 1, 0};   // small products first
#pragma unroll
    for (int J = NB - 1; J >= 0; --J) {
      __builtin_amdgcn_sched_barrier(0);   // one block's column operands at a time
      uint32_t cr[3][V], ci[3][V];
#pragma unroll
      for (int e = 0; e < 3; ++e)
#pragma unroll
        for (int k = 0; k < V / 2; ++k) {
          cr[e][2 * k] = y[J][e][2 * k] ^ sign[k];
          cr[e][2 * k + 1] = y[J][e][2 * k + 1] ^ sign[k];
          ci[e][2 * k] = y[J][e][2 * k + 1] ^ (sign[k] ^ 0x80008000u);
          ci[e][2 * k + 1] = cr[e][2 * k];
        }
#pragma unroll
      for (int w = 0; w < 6; ++w)
#pragma unroll
        for (int I = 0; I <= J; ++I) {
          const int t = I * NB - I * (I - 1) / 2 + J - I;
          if constexpr (V == 4) {
            const bf8 row = __builtin_bit_cast(bf8, u4{y[I][pa[w]][0], y[I][pa[w]][1], y[I][pa[w]][2], y[I][pa[w]][3]});
            const bf8 c0 = __builtin_bit_cast(bf8, u4{cr[pb[w]][0], cr[pb[w]][1], cr[pb[w]][2], cr[pb[w]][3]});
            const bf8 c1 = __builtin_bit_cast(bf8, u4{ci[pb[w]][0], ci[pb[w]][1], ci[pb[w]][2], ci[pb[w]][3]});
            acc.r[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(row, c0, acc.r[t], 0, 0, 0);
            acc.i[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(row, c1, acc.i[t], 0, 0, 0);
          } else {
            const s4 row = __builtin_bit_cast(s4, u2{y[I][pa[w]][0], y[I][pa[w]][1]});
            const s4 c0 = __builtin_bit_cast(s4, u2{cr[pb[w]][0], cr[pb[w]][1]});
            const s4 c1 = __builtin_bit_cast(s4, u2{ci[pb[w]][0], ci[pb[w]][1]});
            acc.r[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(row, c0, acc.r[t], 0, 0, 0);
            acc.i[t] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(row, c1, acc.i[t], 0, 0, 0);
          }
        }
    }
  };
  const int nfull = split_full(cnt);
  const bool half = cnt > 16 * nfull;
  const uint32_t none[2] = {0u, 0u};
  if constexpr (PF > 1) {
    SplitRaw<P, Q> ring[PF], rest;   // chunk ch in ring[ch % PF], refetched as soon as its vectors are split
    fetch(nfull, rest);
#pragma unroll
    for (int sl = 0; sl < PF; ++sl) fetch(sl < nfull ? sl : nfull, ring[sl]);
#pragma unroll 1
    for (int ch0 = 0; ch0 < nfull; ch0 += PF) {
#pragma unroll
      for (int sl = 0; sl < PF; ++sl)
        if (ch0 + sl < nfull)
          accumulate(Int<4>(), ring[sl], none, [&]() __attribute__((always_inline)) {
            fetch(ch0 + sl + PF < nfull ? ch0 + sl + PF : nfull, ring[sl]);
          });
    }
    if (half) accumulate(Int<2>(), rest, none, [] {});
    return;
  }
  SplitRaw<P, Q> raw;   // the chunk in flight: refetched as soon as its vectors are split
  fetch(0, raw);
#pragma unroll 1
  for (int ch = 0; ch < nfull; ++ch) {
    auto next = [&]() __attribute__((always_inline)) { fetch(ch + 1, raw); };
    if (16 * ch + 16 <= npos) {   // uniform: only entering vectors
      accumulate(Int<4>(), raw, none, next);
    } else {
      uint32_t sign[2];
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int m = 16 * ch + 4 * g + 2 * k;
        sign[k] = (m >= npos ? 0x00008000u : 0u) | (m + 1 >= npos ? 0x80000000u : 0u);
      }
      accumulate(Int<4>(), raw, sign, next);
    }
  }
  if (half) {
    const int m = 16 * nfull + 2 * g;
    const uint32_t sign[2] = {(m >= npos ? 0x00008000u : 0u) | (m + 1 >= npos ? 0x80000000u : 0u), 0u};
    accumulate(Int<2>(), raw, sign, [] {});
  }
}

// n S from LDS (the previous pixel's S), for classes that do not keep it.
template <int P, int Q>
__device__ __forceinline__ void split_reload(const float2* sS, int n, SplitAcc<P, Q>& acc) {
  constexpr int NB = SplitAcc<P, Q>::NB;
  int trow = 4 * (threadIdx.x >> 4), tcol = threadIdx.x & 15;
  if constexpr (kOpaqueStore<P, Q>) asm volatile("" : "+v"(trow), "+v"(tcol));
  const float fn = float(n);
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int J = I; J < NB; ++J)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const int t = I * NB - I * (I - 1) / 2 + J - I;
        float2 v = make_float2(0.f, 0.f);
        if (tile_in<P, Q>(I, J, trow + q4, tcol)) v = tile_get<P, Q>(sS, I, J, trow + q4, tcol);
        acc.r[t][q4] = v.x * fn;
        acc.i[t][q4] = v.y * fn;
      }
  wave_sync();   // every lane has reloaded its part
}

// Where a pixel's S is only handed from the accumulators to its slots (the
// accumulators keep it, or the next pixel starts anew), q = 16 passes it
// through LDS in two phases, block row 0 and then the others, in half the
// space (P = 3: three of the six blocks at a time).
template <int P, int Q>
constexpr bool kPhased = kKeepAcc<P, Q> && Q == 16 && P == 3;
template <int P, int Q>
constexpr int kBlocksLds = kPhased<P, Q> ? P : P * (P + 1) / 2;
// LDS offset of block (i, j), i <= j
template <int P, int Q>
__device__ __forceinline__ int lblk(int i, int j) {
  return sblk<P, Q>(i, j) - (kPhased<P, Q> && i > 0 ? P * Q * (Q + 1) : 0);
}

// S = acc / n to LDS: the 16-row blocks [lo, hi) of its rows.
template <int P, int Q>
__device__ __forceinline__ void split_store(const SplitAcc<P, Q>& acc, int n, float2* sS, int lo, int hi) {
  constexpr int NB = SplitAcc<P, Q>::NB;
  // opaque, so that the element addresses are computed here for every pixel
  // rather than hoisted out of the caller's pixel loop and spilled
  int trow = 4 * (threadIdx.x >> 4), tcol = threadIdx.x & 15;
  if constexpr (kOpaqueStore<P, Q>) asm volatile("" : "+v"(trow), "+v"(tcol));
  const float inv_n = 1.f / float(n);
#pragma unroll
  for (int I = 0; I < NB; ++I)
#pragma unroll
    for (int J = I; J < NB; ++J)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        if (I < lo || I >= hi) continue;
        const int t = I * NB - I * (I - 1) / 2 + J - I;
        const float2 v = make_float2(acc.r[t][q4] * inv_n, acc.i[t][q4] * inv_n);
        if constexpr (Q == 16) {   // a tile is a block, stored whole (one writer per element)
          sS[lblk<P, Q>(I, J) + (trow + q4) * (Q + 1) + tcol] = v;
        } else {
          if (tile_keep<P, Q>(I, J, trow + q4, tcol)) tile_put<P, Q>(sS, I, J, trow + q4, tcol, v);
        }
      }
  wave_sync();
}

// -------------------------------------------------------- a2, split BF16
// The same S from three BF16 products per tile: x = hi + lo with
// hi = bf16(x), lo = bf16(x - hi); S ~ hi hi^H + hi lo^H + lo hi^H with FP32
// accumulation.  The split is done once per frame by split_planes into two
// planes in the layout of x, one packed BF16 pair (re, im) per complex
// sample: hi first, then lo.  The covariance kernel loads MFMA operands
// straight from them.  In a 16-vector chunk, 16-lane group g of the
// wavefront holds vectors 4g .. 4g + 3.
//   Both tiles of v_mfma_f32_16x16x32_bf16 over the 16 vectors of the chunk:
//   Re S on Y = (re, im) pairs, re_I re_J + im_I im_J; Im S with the row
//   operand (im, -re), im_I re_J - re_I im_J.  36 MFMAs per chunk and three
//   16-row blocks; Im S on single components through the 16 x 16 x 16 form
//   took 54 and a half-word gather per operand (p = 3, q = 16, 1024 x 1024
//   11.8 -> 10.3 ms with the warm starts of the solves).
__device__ __forceinline__ bf8 swap_neg(bf8 y) {
  u4 w = __builtin_bit_cast(u4, y);
#pragma unroll
  for (int e = 0; e < 4; ++e) w[e] = ((w[e] >> 16) | (w[e] << 16)) ^ 0x80000000u;
  return __builtin_bit_cast(bf8, w);
}

template <int P, int Q>
__device__ __forceinline__ void scm_bf16x3(const uint32_t* hwin, const uint32_t* lwin, int64_t plane, uint32_t rec,
                                           const uint32_t* sOffB, const uint32_t (&loff)[(P * Q + 15) / 16], int n,
                                           SplitAcc<P, Q>& acc) {
  constexpr int NB = (P * Q + 15) / 16;
  constexpr int NT = NB * (NB + 1) / 2;
  const int lane = threadIdx.x;
  f4(&accR)[NT] = acc.r;
  f4(&accI)[NT] = acc.i;
#pragma unroll
  for (int t = 0; t < NT; ++t) accR[t] = accI[t] = f4{0.f, 0.f, 0.f, 0.f};
  const int nch = (n + 15) >> 4;
  constexpr int PF = 2;
  u4 ring[PF][2][NB];   // hi / lo pairs of the lane's 4 vectors, per block
  __amdgpu_buffer_rsrc_t rh[NB], rl[NB];
#pragma unroll
  for (int I = 0; I < NB; ++I) {
    const int64_t cb = int64_t((16 * I) / Q) * plane;
    rh[I] = __builtin_amdgcn_make_buffer_rsrc((void*)(hwin + cb), (short)0, int(rec), 0x00020000);
    rl[I] = __builtin_amdgcn_make_buffer_rsrc((void*)(lwin + cb), (short)0, int(rec), 0x00020000);
  }
  auto fetch = [&](int ch, u4 (&v)[2][NB]) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t off = sOffB[ch * 16 + 4 * (lane >> 4) + e];
#pragma unroll
      for (int I = 0; I < NB; ++I) {
        v[0][I][e] = __builtin_amdgcn_raw_buffer_load_b32(rh[I], loff[I] + off, 0, 0);
        v[1][I][e] = __builtin_amdgcn_raw_buffer_load_b32(rl[I], loff[I] + off, 0, 0);
      }
    }
  };
  // MFMAs of one 16-vector chunk
  auto accumulate = [&](const u4 (&v)[2][NB]) {
    bf8 yh[NB], yl[NB], zh[NB], zl[NB];   // (re, im) and (im, -re)
#pragma unroll
    for (int I = 0; I < NB; ++I) {
      yh[I] = __builtin_bit_cast(bf8, v[0][I]);
      yl[I] = __builtin_bit_cast(bf8, v[1][I]);
      zh[I] = swap_neg(yh[I]);
      zl[I] = swap_neg(yl[I]);
    }
    int t = 0;
#pragma unroll
    for (int I = 0; I < NB; ++I)
#pragma unroll
      for (int J = I; J < NB; ++J, ++t) {
        accR[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(yh[I], yh[J], accR[t], 0, 0, 0);
        accI[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zh[I], yh[J], accI[t], 0, 0, 0);
        accR[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(yh[I], yl[J], accR[t], 0, 0, 0);
        accI[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zh[I], yl[J], accI[t], 0, 0, 0);
        accR[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(yl[I], yh[J], accR[t], 0, 0, 0);
        accI[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(zl[I], yh[J], accI[t], 0, 0, 0);
      }
  };
#pragma unroll
  for (int s0 = 0; s0 < PF - 1; ++s0) {
    __builtin_amdgcn_sched_barrier(0);
    fetch(s0, ring[s0]);
  }
  int ch0 = 0;
  for (; ch0 + PF <= nch; ch0 += PF) {   // branch-free body, as in scm_fp32
#pragma unroll
    for (int sl = 0; sl < PF; ++sl) {
      __builtin_amdgcn_sched_barrier(0);
      fetch(ch0 + sl + PF - 1, ring[(sl + PF - 1) % PF]);
      __builtin_amdgcn_sched_barrier(0);   // all loads of the next chunk go out first
      accumulate(ring[sl]);
    }
  }
#pragma unroll
  for (int sl = 0; sl < PF - 1; ++sl)
    if (ch0 + sl < nch) accumulate(ring[sl]);
}

// ------------------------------------------------------------ kernel body
template <int Q>
struct Groups {
  static constexpr int QP = (Q <= 8) ? 8 : (Q <= 16) ? 16 : (Q <= 32) ? 32 : 64;
  static constexpr int G = 64 / QP;
};

template <bool B, typename T, typename F> struct Pick { using type = T; };
template <typename T, typename F> struct Pick<false, T, F> { using type = F; };

// True when the plan asks for more than the Kron-STAP statistic of one
// temporal steering (uniform across the grid).
__host__ __device__ __forceinline__ bool has_variants(const KParams& prm) {
  return prm.filter != 0 || prm.nbank != 0 || prm.passes != 1 || prm.E != nullptr || prm.bin != nullptr;
}

// Run mode: every output of a pixel outside the valid region is zero.
__device__ __forceinline__ void write_outside(const KParams& prm, int64_t idx) {
  prm.T[idx] = 0.f;
  if (prm.D) prm.D[idx] = 0;
  if (prm.E) prm.E[idx] = 0.f;
  if (prm.bin) prm.bin[idx] = 0;
  const int64_t hw = int64_t(prm.H) * prm.W;
  for (int k = 0; k < prm.passes; ++k) {
    if (prm.Tpass) prm.Tpass[k * hw + idx] = 0.f;
    if (prm.C && k > 0) prm.C[(k - 1) * hw + idx] = 0.f;
  }
}

// ------------------------------------------------ a6 + a8, batched
// The tail of the statistic variants in run mode (the plain statistic and the
// probe take tail_rows): top-r_b time subspace, projected test vector and statistic for up to
// 64 / QP queued pixels of one wavefront: lane group `slot` (QP lanes) serves
// queue slot `slot`, whose lane k holds row k of the pixel's Hermitian time
// factor in Bq; slots >= nfill are empty.  Per slot the queue holds the pixel
// index, a flag (0 ok, 1 zero covariance, 2 non-finite) and U_A (p x RAM).
// Writes T, D and the variants' outputs.
// WAVE_LOCAL: other wavefronts of the workgroup run their own tails.
// vb: this lane's row of its slot's basis; on entry the warm start of the
// slots whose lanes set `keep` (the others start cold), on return the basis.
template <int P, int Q, int RBM, typename EC, bool WAVE_LOCAL>
__device__ __forceinline__ void tail_batch(const KParams& prm, const float2 (&Bq)[Q], int slot, int nfill,
                                           const int* sQflag, const int64_t* sQidx,
                                           const EC (*sQUA)[P * ((P < kMaxRA) ? P : kMaxRA)], EC* scratch, double tol,
                                           EC (&vb)[RBM], bool keep, bool& vb_ok) {
  using ES = decltype(EC{}.x);
  constexpr int RAM = (P < kMaxRA) ? P : kMaxRA;
  constexpr int QP = Groups<Q>::QP;
  const int tk = (threadIdx.x & 63) % QP;
  const int H = prm.H, W = prm.W;
  const int r_a = prm.r_a, r_b = prm.r_b;
  const bool slot_ok = slot < nfill;
  const bool rok = slot_ok && tk < Q;
  const int flag = slot_ok ? sQflag[slot] : 1;
  const int64_t pidx = slot_ok ? sQidx[slot] : 0;
  keep = keep && rok && flag == 0;
#pragma unroll
  for (int c = 0; c < RBM; ++c)
    if (!keep) vb[c] = czero<EC>();
  // FP64 solves iterate until converged where the r_b-th and next eigenvalues
  // of B lie close together (a ratio of 0.99 takes ~1 500 steps to 1e-10);
  // the loop exits on the step cap, so a group never runs unbounded
  constexpr int kTailSteps = sizeof(ES) == 8 ? 4000 : 200;
  if (r_b > 0)
    group_subspace<RBM, QP, Q, EC, WAVE_LOCAL>(Bq, rok && flag == 0, r_b, vb, scratch, true, kTailSteps, tol, keep,
                                               keep, kMixNeighbour);
  vb_ok = rok && flag == 0;
  // statistic
  const int pr = int(pidx / W), pc = int(pidx - int64_t(pr) * W);
  const bool use = rok && flag == 0;
  // this lane's sample of every channel of the test snapshot
  const float2* xt = prm.x + (int64_t(pr) * W + pc) * Q;
  EC xv[P];
#pragma unroll
  for (int i = 0; i < P; ++i) xv[i] = use ? cto<EC>(xt[int64_t(i) * H * W * Q + tk]) : czero<EC>();
  const EC* Uq = sQUA[slot_ok ? slot : 0];   // U_A of the queued pixel, p x RAM
  // z <- (I - U_A U_A^H) z
  auto project_a = [&](EC (&z)[P]) __attribute__((always_inline)) {
#pragma unroll
    for (int c = 0; c < RAM; ++c) {
      if (c >= r_a) continue;
      EC cw = czero<EC>();
#pragma unroll
      for (int i = 0; i < P; ++i) cw = ccfma(Uq[i * RAM + c], z[i], cw);
#pragma unroll
      for (int i = 0; i < P; ++i) z[i] = csub(z[i], cmul(Uq[i * RAM + c], cw));
    }
  };
  // fixed spatial steering: h and F_A h
  EC hs[P], fh[P];
  ES hfa = 0, hpa = 0;   // ||F_A h||^2, ||P_A h||^2
  if (prm.stat_mode != 0) {
#pragma unroll
    for (int i = 0; i < P; ++i) fh[i] = hs[i] = cto<EC>(prm.h_s[i]);
    project_a(fh);
#pragma unroll
    for (int i = 0; i < P; ++i) {
      hfa += hs[i].x * fh[i].x + hs[i].y * fh[i].y;
      const EC ph = csub(hs[i], fh[i]);
      hpa += cabs2(ph);
    }
  }
  // Temporal steering: the plan's b_s, or each bin of a Doppler bank
  // b_m[k] = exp(2 pi j ((m k) mod M) / M); the statistic is the largest over
  // the bank, the bin its first maximiser.
  const int nbank = prm.nbank;
  const int nbins = nbank > 0 ? nbank : 1;
  const int K = prm.passes, PP = K > 1 ? P / K : P;
  const int filter = prm.filter;
  float* const Eout = prm.E;
  float T = 0.f, Ebest = 0.f;
  int best = 0;
  ES ez[P];   // per-channel energy |z_i|^2 / (b^H F_B b) at the best bin (passes > 1)
#pragma unroll
  for (int i = 0; i < P; ++i) ez[i] = 0;
  for (int m = 0; m < nbins; ++m) {
    EC bsk;
    ES bn2;
    if (nbank > 0) {
      const int ph = (m * tk) % nbank;
      float sn, cs;
      sincospif(float(2 * ph) / float(nbank), &sn, &cs);
      bsk = use ? cto<EC>(make_float2(cs, sn)) : czero<EC>();
      bn2 = ES(Q);
    } else {
      bsk = use ? cto<EC>(prm.b_s[tk]) : czero<EC>();
      bn2 = ES(prm.bs_norm2);
    }
    // g = F_B b
    EC gk = bsk;
    if (r_b > 0) {
#pragma unroll
      for (int c = 0; c < RBM; ++c) {
        if (c >= r_b) continue;
        const EC coef = gsum<QP>(ccfma(vb[c], bsk, czero<EC>()));
        if (use) gk = csub(gk, cmul(vb[c], coef));
      }
    }
    // w = X conj(g), z = F_A w
    EC w[P], z[P];
#pragma unroll
    for (int i = 0; i < P; ++i) z[i] = w[i] = gsum<QP>(cmul(xv[i], cconj(gk)));
    const ES den = gsum<QP>(ES(bsk.x * gk.x + bsk.y * gk.y));   // b^H F_B b
    project_a(z);
    const bool den_ok = den > ES(1e-12) * bn2;
    // w0 = X conj(b) (the classical filter, and channel 0's SAR image)
    EC w0[P];
    const int nw0 = filter == 1 ? P : (Eout ? 1 : 0);
#pragma unroll
    for (int i = 0; i < P; ++i) w0[i] = (i < nw0) ? gsum<QP>(cmul(xv[i], cconj(bsk))) : czero<EC>();
    ES t;
    if (filter == 0) {
      // Kron-STAP, Eq. (25): ||F_A X conj(F_B b)||^2 / (b^H F_B b)
      if (prm.stat_mode == 0) {
        ES num = 0;
#pragma unroll
        for (int i = 0; i < P; ++i) num += cabs2(z[i]);
        t = den_ok ? num / den : ES(0);
      } else {
        EC hz = czero<EC>();
#pragma unroll
        for (int i = 0; i < P; ++i) hz = ccfma(hs[i], z[i], hz);
        const bool ok = den_ok && hfa > ES(1e-12) * ES(prm.h_norm2);
        t = ok ? cabs2(hz) / (hfa * den) : ES(0);
      }
    } else {
      // classical, Eq. (24): the GLRT over h reduces to
      // ||F_A X b*||^2 / ||b||^2 + ||P_A X conj(F_B b)||^2 / (b^H F_B b)
      EC z0[P];
#pragma unroll
      for (int i = 0; i < P; ++i) z0[i] = w0[i];
      project_a(z0);
      if (prm.stat_mode == 0) {
        ES n0 = 0, n1 = 0;
#pragma unroll
        for (int i = 0; i < P; ++i) {
          n0 += cabs2(z0[i]);
          n1 += cabs2(csub(w[i], z[i]));
        }
        t = n0 / bn2 + (den_ok ? n1 / den : ES(0));
      } else {
        // u = F_A X b* + P_A X conj(F_B b); h^H G h = ||F_A h||^2 ||b||^2 + ||P_A h||^2 b^H F_B b
        EC hu = czero<EC>();
#pragma unroll
        for (int i = 0; i < P; ++i) hu = ccfma(hs[i], cadd(z0[i], csub(w[i], z[i])), hu);
        const ES hgh = hfa * bn2 + hpa * (den_ok ? den : ES(0));
        t = hgh > ES(1e-12) * ES(prm.h_norm2) * bn2 ? cabs2(hu) / hgh : ES(0);
      }
    }
    if (m == 0 || float(t) > T) {
      T = float(t);
      best = m;
      if (Eout) {
        const ES isar = cabs2(w0[0]) / bn2;   // channel 0's matched-filter intensity
        Ebest = isar > ES(0) ? float(t / isar) : 0.f;
      }
      if (K > 1) {
#pragma unroll
        for (int i = 0; i < P; ++i) ez[i] = den_ok ? cabs2(z[i]) / den : ES(0);
      }
    }
  }
  if (!isfinite(T)) T = NAN;
  if (flag == 1) T = 0.f;
  if (flag == 2) T = NAN;
  if (slot_ok && tk == 0) {
    prm.T[pidx] = T;
    if (prm.D) prm.D[pidx] = (T > prm.tau) ? 1 : 0;
    const int64_t hw = int64_t(H) * W;
    if (Eout) Eout[pidx] = flag == 2 ? NAN : (flag == 1 ? 0.f : Ebest);
    if (prm.bin) prm.bin[pidx] = uint8_t(flag == 0 ? best : 0);
    // pass k's image: the energy of its channels of z (passes > 1)
    if (K > 1 && (prm.Tpass || prm.C)) {
      ES t0 = 0;
#pragma unroll
      for (int i = 0; i < P; ++i)
        if (i < PP) t0 += ez[i];
#pragma unroll
      for (int k = 0; k < P; ++k) {
        if (k >= K) continue;
        ES ts = 0;
#pragma unroll
        for (int i = 0; i < P; ++i)
          if (i / PP == k) ts += ez[i];
        if (prm.Tpass) prm.Tpass[k * hw + pidx] = flag == 2 ? NAN : (flag == 1 ? 0.f : float(ts));
        if (prm.C && k > 0)
          prm.C[(k - 1) * hw + pidx] = flag == 2 ? NAN : (flag == 1 ? 0.f : float(sqrt(ts) - sqrt(t0)));
      }
    }
  }
  lds_sync<WAVE_LOCAL>();
}

}  // namespace
}  // namespace kstap

#include "kstap_tail.h"

namespace kstap {
namespace {

// PREC 0: FP32 covariance, FP32 eigensolves and statistic.
// PREC 1: split-BF16 covariance, FP64 eigensolves and statistic.
// PREC 2: FP32 covariance (full sums, no sliding window), FP64 eigensolves
//         and statistic.
// Hermitian slots.  S is Hermitian and so is every iterate of LR-Kron: A
// because EIG_{r_a} returns U Hs U^H, and with it b = R^T conj(a), whose q x q
// matrix is sum_ij conj(A_ij) S(i,j) with S(j,i) = S(i,j)^H.  The narrow
// kernels therefore work on the q^2 real dimensions of b as q^2 / 2 slots of
// two values: slot (k, l), l = k + d mod q, holds the complex entry B_kl (its
// mirror B_lk is the conjugate, weight w = 2), and q / 2 slots hold two
// diagonal entries (B_kk, B_ll), l = k + q / 2 (weight 1).  Against a slot's b
// the P^2 blocks of R become P^2 rows of two values with real coefficients:
//   D_i = S(i,i)_kl,  U_ij = S(i,j)_kl + conj(S(i,j)_lk),
//   V_ij = -j (S(i,j)_kl - conj(S(i,j)_lk)),  i < j,
//   B_kl = sum_i A_ii D_i + sum_{i<j} (Re A_ij U_ij + Im A_ij V_ij),
//   R conj(b): A_ii = sum w D_i . b,  (Re, Im) A_ij = sum w/2 (U, V)_ij . b,
//   ||R||^2 = sum w (|D|^2 + (|U|^2 + |V|^2) / 2).
// One half of the products of the full q^2 x p^2 sweep, no conjugates, and
// the values (36 registers for p = 3, q = 16) are read from LDS once per pixel
// instead of once per sweep.  The kernels are bound by VALU issue, so this is
// what counts: sweeps over all p^2 q^2 entries took the 2048 x 2048, p = 3,
// q = 16, n = 200 frame 41.4 ms (FP32), the slots 32.9 ms; split BF16 at
// 1024 x 1024 15.15 -> 13.11 ms, FP32 with FP64 solves at 512 x 512 6.50 ->
// 5.87 ms.
template <int P, int Q>
struct Slots {
  static_assert(Q % 2 == 0, "the slots pair the diagonal entries of b");
  static constexpr int NS = Q * Q / 2;
  // q = 8 has 32 slots: the two values of a slot go to lanes l and l + 32
  static constexpr int C = NS <= 32 ? 1 : 2;        // values of a slot per lane
  static constexpr int N = (NS * (2 / C) + 63) / 64;   // slots per lane
};

// Queued time factors wait for the batched tail in LDS, as slots, where S
// leaves room for them (kKeepAcc: it is in LDS only in passing); else as one
// row per lane in registers.  In registers (32 for q = 16) they raised the
// covariance phase over the register file: it spilled, and waited for each
// chunk's loads as soon as they were issued.
template <int P, int Q>
constexpr bool kQueueLds = kKeepAcc<P, Q>;

// Row k of the Hermitian q x q matrix whose slots are qb.
template <int P, int Q>
__device__ __forceinline__ void queue_row(const float2* qb, int k, float2 (&row)[Q]) {
#pragma unroll
  for (int l = 0; l < Q; ++l) {
    int d = l - k;
    d += d < 0 ? Q : 0;
    const bool up = d < Q / 2 || (d == Q / 2 && k < Q / 2), hi = k >= Q / 2;
    const int e = d == 0 ? (Q / 2 - 1) * Q + (hi ? k : k + Q / 2) : up ? (d - 1) * Q + k : (Q - d - 1) * Q + l;
    const float2 b = qb[e];
    row[l] = make_float2(d == 0 && hi ? b.y : b.x, d == 0 ? 0.f : up ? b.y : -b.y);
  }
}

// LDS carve-out of one pixel pipeline (one workgroup), largest alignment first.
template <int P, int Q, int RBM, int PREC>
struct Lds {
  using EC = typename Pick<PREC != 0, double2, float2>::type;
  static constexpr int PQ = P * Q;
  static constexpr int RAM = (P < kMaxRA) ? P : kMaxRA;
  static constexpr int G = Groups<Q>::G;
  static constexpr int NB = (PQ + 15) / 16;
  // B / tail / transpose scratch: the time factor B (q rows of q + 2; classes
  // that queue rows), the batched tail's basis exchange, and the FP32 path's
  // diagonal-tile transpose
  static constexpr size_t kB = kQueueLds<P, Q> ? 0 : sizeof(float2) * Q * (Q + 2);
  static constexpr size_t kT = tail_scratch_bytes<RBM, Q, G, EC>;
  static constexpr size_t kP = (PREC == 1 || kSplitCov<P, Q>) ? 0 : sizeof(float) * NB * 256;
  static constexpr size_t kBT = kB > kT ? (kB > kP ? kB : kP) : (kT > kP ? kT : kP);
  static constexpr size_t oUA = 0;                                        // EC[P*RAM]
  static constexpr size_t oAh = oUA + sizeof(EC) * P * RAM;               // EC[P*P]
  static constexpr size_t oQUA = oAh + sizeof(EC) * P * P;                // EC[G][P*RAM]
  static constexpr size_t oBT = (oQUA + sizeof(EC) * G * P * RAM + 15) / 16 * 16;   // kBT bytes
  static constexpr size_t oS = (oBT + kBT + 15) / 16 * 16;                // float2[blocks][Q][Q+1]
  static constexpr size_t oA = oS + sizeof(float2) * kBlocksLds<P, Q> * Q * (Q + 1);   // float2[P*P]
  static constexpr size_t oQB = oA + sizeof(float2) * P * P;              // float2[G][NS] (kQueueLds)
  static constexpr size_t oQidx = oQB + (kQueueLds<P, Q> ? sizeof(float2) * G * Slots<P, Q>::NS : 0);   // int64[G]
  static constexpr size_t oOff = (oQidx + sizeof(int64_t) * G + 15) / 16 * 16;   // uint32[kMaxN + kOffPad]
  static constexpr size_t oDelta = oOff + sizeof(uint32_t) * (kMaxN + kOffPad);   // uint32[nDelta] (FP32)
  static constexpr int nDelta = PREC ? 0 : kSplitCov<P, Q> ? 3 * kDeltaList : 6 * (kMaxDelta + 8);
  static constexpr size_t oQflag = oDelta + sizeof(uint32_t) * nDelta;   // int[G]
  static constexpr size_t oQit = oQflag + sizeof(int) * G;                // int[G]
  static constexpr size_t oQeta = oQit + sizeof(int) * G;                 // float[G]
  static constexpr size_t bytes = ((oQeta + sizeof(float) * G) + 15) / 16 * 16;
};

// The whole per-pixel pass for `count` pixels starting at `first`: positions
// in the tiled order of the frame (run mode) or in the pixel list (probe
// mode).  One 64-lane workgroup; `lds` holds Lds<...>::bytes.
template <int P, int Q, int RBM, int MODE, int PREC, bool VAR = false>
__device__ __forceinline__ void run_pixels(const KParams& prm, int64_t first, int64_t count, char* lds) {
  using EC = typename Pick<PREC != 0, double2, float2>::type;   // eigensolver / statistic precision
  using ES = decltype(EC{}.x);
  using L = Lds<P, Q, RBM, PREC>;
  constexpr int PQ = P * Q;
  constexpr int NB = (PQ + 15) / 16;        // 16-row blocks of the pq x pq covariance
  using SL = Slots<P, Q>;
  constexpr int NS = SL::NS, NSL = SL::N, C = SL::C;
  constexpr int RAM = L::RAM;
  constexpr int QP = Groups<Q>::QP;         // lanes per pixel in the batched tail
  constexpr int G = Groups<Q>::G;           // pixels per batched tail

  float2* const sS = reinterpret_cast<float2*>(lds + L::oS);     // S, upper blocks
  float2* const sBT = reinterpret_cast<float2*>(lds + L::oBT);   // B, then tail scratch
  uint32_t* const sOffB = reinterpret_cast<uint32_t*>(lds + L::oOff);
  // sliding window: per move, the entering then the leaving vectors
  uint32_t* const sDelta = reinterpret_cast<uint32_t*>(lds + L::oDelta);
  float2* const sA = reinterpret_cast<float2*>(lds + L::oA);
  EC* const sUA = reinterpret_cast<EC*>(lds + L::oUA);
  EC* const sAh = reinterpret_cast<EC*>(lds + L::oAh);
  EC (*const sQUA)[P * RAM] = reinterpret_cast<EC (*)[P * RAM]>(lds + L::oQUA);   // queued pixels: U_A
  EC* const tail_scratch = reinterpret_cast<EC*>(sBT);
  int64_t* const sQidx = reinterpret_cast<int64_t*>(lds + L::oQidx);             //   pixel index
  int* const sQflag = reinterpret_cast<int*>(lds + L::oQflag);                   //   0 ok, 1 zero, 2 non-finite
  float* const sQeta = reinterpret_cast<float*>(lds + L::oQeta);
  int* const sQit = reinterpret_cast<int*>(lds + L::oQit);

  const int lane = threadIdx.x;
  const int n = prm.n;
  const int H = prm.H, W = prm.W;
  const int r_a = prm.r_a, r_b = prm.r_b;

  // byte offset of each stencil entry from the window origin (kOut past n);
  // samples are complex64 (8 bytes) or, on the mixed path, BF16 pairs (4)
  constexpr int kSample = PREC == 1 ? 4 : 8;
  wave_sync();
  for (int e = lane; e < kMaxN + kOffPad; e += 64) {
    const int m = (PREC != 1 && kSplitCov<P, Q>) ? split_entry(e, n) : (e < n ? e : -1);
    sOffB[e] = (m >= 0) ? uint32_t(((int(prm.st[2 * m]) * W + int(prm.st[2 * m + 1])) * Q - prm.st_min) * kSample)
                        : kOut;
  }
  // per move: one list, entering then leaving vectors (scm_split), or two
  // lists of KD (scm_fp32_delta)
  constexpr int KD = kMaxDelta + 8;
  for (int m = lane; m < L::nDelta; m += 64) {
    constexpr int per = kSplitCov<P, Q> ? kDeltaList : 2 * KD;
    const int mv = m / per;
    int e = m - mv * per;
    const int na = prm.nadd[mv], nr = prm.nrem[mv];   // each <= kMaxDelta (negative: never slides)
    if constexpr (kSplitCov<P, Q>) {
      e = na >= 0 ? split_entry(e, na + nr) : -1;
      if (e < 0) e = na + nr;   // no vector
    }
    const bool rem = kSplitCov<P, Q> ? e >= na : e >= KD;
    e -= rem ? (kSplitCov<P, Q> ? na : KD) : 0;
    uint32_t off = kOut;
    if (na >= 0 && e < (rem ? nr : na)) {
      const int dr = rem ? prm.drem[mv][2 * e] : prm.dadd[mv][2 * e];
      const int dc = rem ? prm.drem[mv][2 * e + 1] : prm.dadd[mv][2 * e + 1];
      off = uint32_t(((dr * W + dc) * Q - prm.st_min) * kSample);
    }
    sDelta[m] = off;
  }
  wave_sync();

  // Operand rows of this lane: row rho = 16*I + (lane & 15) of the stacked
  // snapshot, channel rho / q, sample rho % q; its byte offset inside block
  // I's record, which starts in channel 16*I / q.
  const int64_t plane = int64_t(H) * W * Q;
  uint32_t loff[NB];
#pragma unroll
  for (int I = 0; I < NB; ++I) {
    const int rho = 16 * I + (lane & 15);
    const int ch = rho / Q, j = rho - ch * Q;
    loff[I] = (rho < PQ) ? uint32_t(((ch - (16 * I) / Q) * plane + j) * kSample) : kOut;
  }

  // queue of pixels waiting for the batched tail: their slots in LDS, or lane
  // (g, k) holds row k of the Hermitian time factor of queued pixel g
  const int tg = lane / QP, tk = lane % QP;
  float2* const sQB = reinterpret_cast<float2*>(lds + L::oQB);
  float2 Bq[Q];
#pragma unroll
  for (int l = 0; l < Q; ++l) Bq[l] = cz();
  int nq = 0;

  // ------------------------------------------------ a6 + a8 for G pixels
  // Run mode: the queue holds the pixels of one sliding-window chain at a
  // time, and every batch of a chain but its first starts each slot from the
  // converged time-factor subspace of the previous batch's slot G-1-g, its
  // nearest pixel in the snake order of a unit (directly above it for q = 16).
  // Like the sliding window, the choice depends only on the chain, so the
  // results are the same for every decomposition of the frame.  The BF16x3 and
  // FP64 paths, which do not slide their covariance, start warm as well:
  // p=3 q=16 at 512^2 BF16x3 with the product below 2.93 -> 2.61 ms, FP64
  // solves at 256^2 3.98 -> 3.88 ms.
  constexpr bool kWarmTail = MODE == kModeRun;
  EC vbw[RBM];   // lane (g, k): row k of the basis that starts slot g
#pragma unroll
  for (int c = 0; c < RBM; ++c) vbw[c] = czero<EC>();
  bool vbw_ok = false;
  int64_t qchain = -1, bchain = -2;   // chain of the queued pixels, of the last batch
  auto tail = [&](int nfill) __attribute__((always_inline)) {
    const bool keep = kWarmTail && bchain == qchain && vbw_ok;
    bool ok = false;
    if constexpr (kQueueLds<P, Q>) {
      int lanev = lane;   // per batch: no address hoisted out of the pixel loop
      asm volatile("" : "+v"(lanev));
      const int k = lanev % QP;
      queue_row<P, Q>(sQB + (lanev / QP) * NS, k < Q ? k : 0, Bq);   // empty slots: whatever is there, unused
    }
    if constexpr (VAR) {
      tail_batch<P, Q, RBM, EC, false>(prm, Bq, tg, nfill, sQflag, sQidx, sQUA, tail_scratch, PREC ? 1e-10 : 2e-6, vbw,
                                       keep, ok);
    } else {
      with_rank<RBM>(r_b, [&](auto rank) __attribute__((always_inline)) {
        tail_rows<P, Q, RBM, decltype(rank)::value, MODE, EC, false>(
            prm, Bq, 0, nfill, sQflag, sQidx, sQeta, sQit, sQUA, reinterpret_cast<char*>(sBT), PREC ? 1e-10 : 2e-6, vbw,
            keep, ok);
      });
    }
    if constexpr (kWarmTail) {
      bchain = qchain;
      const int src = (G - 1 - tg) * QP + tk;
#pragma unroll
      for (int c = 0; c < RBM; ++c) {
        vbw[c].x = __shfl(vbw[c].x, src);
        vbw[c].y = __shfl(vbw[c].y, src);
      }
      vbw_ok = __shfl(int(ok), src) != 0;
    }
  };

  // this lane's slots: entry (sk, sl) of b, the offsets of S(i,j)_kl and
  // S(i,j)_lk inside an upper block, and whether the last slot is a diagonal one
  int sk[NSL], sl[NSL], so1[NSL], so2[NSL];
  bool diag = false;
  const int comp = (C == 1) ? lane >> 5 : 0;
#pragma unroll
  for (int t = 0; t < NSL; ++t) {
    int s = (C == 1) ? (lane & 31) : lane + 64 * t;
    if (s >= NS) s = 0;
    const int d = s / Q + 1, k = s - (d - 1) * Q;
    const bool dg = d == Q / 2 && k >= Q / 2;
    sk[t] = dg ? k - Q / 2 : k;
    sl[t] = dg ? k : (k + d) % Q;
    so1[t] = dg ? sk[t] * (Q + 1) + sk[t] : sk[t] * (Q + 1) + sl[t];
    so2[t] = dg ? sl[t] * (Q + 1) + sl[t] : sl[t] * (Q + 1) + sk[t];
    if (t == NSL - 1) diag = dg;
  }
  // weight of a slot in sums over the entries of b
  auto wgt = [&](int t) __attribute__((always_inline)) -> float { return (t == NSL - 1 && diag) ? 1.f : 2.f; };

  // Sliding window (run mode, FP32 path): every position of a chain but the
  // first is a one-pixel move from the one before it (tiled_move); such a
  // pixel updates the previous pixel's S when this workgroup has just
  // computed it from finite data.  A chain's first pixel takes the full sum,
  // and runs start on a chain, so the choice is the same for every
  // decomposition.
  bool chain = false;
  SplitAcc<P, Q> acc;   // n S of the pixel processed last (kKeepAcc)
  bool ua_ok = false;   // ua (r_a = 1) or sUA holds the U_A of the pixel processed last
  EC ua[P];
#pragma unroll
  for (int i = 0; i < P; ++i) ua[i] = czero<EC>();
  int ur = 0, uc = 0;   // first pixel of the current unit: found once per unit, not by division per pixel
  auto pixel = [&](int64_t it) __attribute__((always_inline)) {
    int64_t idx;
    int r, c;
    const bool left_ok = chain;
    chain = false;
    // position k of the unit's snake: row k / 4, alternately left to right and back
    const int k = int(first + it) & (kUnit * kUnit - 1);
    if (MODE == kModeRun) {
      if (it == 0 || k == 0) tiled_pixel(first + it - k, H, W, &ur, &uc);
      r = ur + k / kUnit;
      c = uc + ((k / kUnit & 1) ? kUnit - 1 - k % kUnit : k % kUnit);
      if (r >= H || c >= W) return;
      idx = int64_t(r) * W + c;
    } else {
      idx = first + it;
      r = prm.pix[2 * idx];
      c = prm.pix[2 * idx + 1];
    }
    const bool valid = r >= prm.r0 && r < prm.r1 && c >= prm.c0 && c < prm.c1;
    if (!valid) {
      if (lane == 0) {
        if (MODE == kModeRun) write_outside(prm, idx);
        else prm.T[idx] = 0.f;
        if (MODE == kModeProbe) {
          if (prm.eta) prm.eta[idx] = 0.f;
          if (prm.iters) prm.iters[idx] = 0;
        }
      }
      if (MODE == kModeProbe) {
        if (prm.UA)
          for (int e = lane; e < P * r_a; e += 64) prm.UA[idx * P * r_a + e] = cz();
        if (prm.UB)
          for (int e = lane; e < Q * r_b; e += 64) prm.UB[idx * Q * r_b + e] = cz();
      }
      return;
    }
    // window origin as a sample index (x and the split planes share the layout)
    const int64_t win = (int64_t(r) * W + c) * Q + prm.st_min;

    // ---------------------------------------------------------------- a2 SCM
    // (the FP64-solve paths are bound by their solves, not by the covariance
    // MFMAs, so they always take the full sum: no sliding-window residue)
    static_assert(kChainNarrow == kUnit * kUnit, "a narrow chain is one unit");
    const int mv = k % kUnit == 0 ? kMoveDown : (k / kUnit & 1) ? kMoveLeft : kMoveRight;   // tiled_move in a unit
    const bool slide = PREC == 0 && MODE == kModeRun && left_ok && k > 0 && prm.nadd[0] >= 0;
    if constexpr (PREC != 1 && kSplitCov<P, Q>) {
      if (slide) {
        if constexpr (!kKeepAcc<P, Q>) split_reload<P, Q>(sS, n, acc);
      } else {
#pragma unroll
        for (int t = 0; t < SplitAcc<P, Q>::NT; ++t) acc.r[t] = acc.i[t] = f4{0.f, 0.f, 0.f, 0.f};
      }
      scm_split<P, Q, MODE == kModeProbe ? 3 : 1>(prm.x + win, plane, prm.rec_bytes,
                                                  slide ? sDelta + mv * kDeltaList : sOffB, slide ? prm.nadd[mv] : n,
                                                  slide ? prm.nadd[mv] + prm.nrem[mv] : n, loff, acc);
    } else if constexpr (PREC != 1) {
      SSums<P> ss{};   // gathered for the Doppler bank kernels only
      if (slide)
        scm_fp32_delta<P, Q>(prm.x + win, plane, prm.rec_bytes, sDelta + 2 * mv * KD, prm.nadd[mv],
                             sDelta + (2 * mv + 1) * KD, prm.nrem[mv], loff, n, sS, ss);
      else
        scm_fp32<P, Q>(prm.x + win, plane, prm.rec_bytes, sOffB, loff, n, sS, reinterpret_cast<float*>(sBT), ss);
    } else {
      scm_bf16x3<P, Q>(prm.xs + win, prm.xs + P * plane + win, plane, prm.rec_bytes / 2, sOffB, loff, n, acc);
    }

    // -------------------------------------- this pixel's slots, from S in LDS
    float v[NSL][P * P][C];
    // the entries of block row i
    auto slots_row = [&](int i) __attribute__((always_inline)) {
#pragma unroll
      for (int t = 0; t < NSL; ++t) {
        const bool last = t == NSL - 1;   // the diagonal slots are a lane's last
        const float2 s1 = sS[lblk<P, Q>(i, i) + so1[t]];
        float y = s1.y;
        if (last) {
          const float2 s2 = sS[lblk<P, Q>(i, i) + so2[t]];
          y = diag ? s2.x : y;
        }
        if constexpr (C == 2) {
          v[t][i][0] = s1.x;
          v[t][i][1] = y;
        } else {
          v[t][i][0] = comp ? y : s1.x;
        }
#pragma unroll
        for (int j = i + 1; j < P; ++j) {
          const float2 s = sS[lblk<P, Q>(i, j) + so1[t]], u = sS[lblk<P, Q>(i, j) + so2[t]];
          float ux = s.x + u.x, uy = s.y - u.y, vx = s.y + u.y, vy = u.x - s.x;
          if (last) {
            ux = diag ? 2.f * s.x : ux;
            uy = diag ? 2.f * u.x : uy;
            vx = diag ? 2.f * s.y : vx;
            vy = diag ? 2.f * u.y : vy;
          }
          if constexpr (C == 2) {
            v[t][hoff<P>(i, j)][0] = ux;
            v[t][hoff<P>(i, j)][1] = uy;
            v[t][hoff<P>(i, j) + 1][0] = vx;
            v[t][hoff<P>(i, j) + 1][1] = vy;
          } else {
            v[t][hoff<P>(i, j)][0] = comp ? uy : ux;
            v[t][hoff<P>(i, j) + 1][0] = comp ? vy : vx;
          }
        }
      }
    };
    if constexpr (kPhased<P, Q>) {
      split_store<P, Q>(acc, n, sS, 0, 1);
      slots_row(0);
      wave_sync();
      split_store<P, Q>(acc, n, sS, 1, SplitAcc<P, Q>::NB);
#pragma unroll
      for (int i = 1; i < P; ++i) slots_row(i);
    } else {
      if constexpr (kSplitCov<P, Q>) split_store<P, Q>(acc, n, sS, 0, SplitAcc<P, Q>::NB);
#pragma unroll
      for (int i = 0; i < P; ++i) slots_row(i);
    }
#pragma unroll
    for (int t = 0; t < NSL; ++t) {
      if (NS % 64 != 0 && !(lane + 64 * t < NS * (2 / C))) {   // no such slot
#pragma unroll
        for (int e = 0; e < P * P; ++e)
#pragma unroll
          for (int c2 = 0; c2 < C; ++c2) v[t][e][c2] = 0.f;
      }
    }

    // R conj(b), given w b, as uniform values (P*P reals); `extra` is summed with it
    auto half_a = [&](const float (&wb)[NSL][C], float (&out)[P * P], float& extra) __attribute__((always_inline)) {
      constexpr int NR = (P * P + 1 + 3) / 4 * 4;
      float sums[NR];
#pragma unroll
      for (int e = 0; e < NR; ++e) sums[e] = (e == P * P) ? extra : 0.f;
#pragma unroll
      for (int t = 0; t < NSL; ++t)
#pragma unroll
        for (int c2 = 0; c2 < C; ++c2)
#pragma unroll
          for (int e = 0; e < P * P; ++e) sums[e] = fmaf(v[t][e][c2], wb[t][c2], sums[e]);
      wsum_n<NR>(sums);
#pragma unroll
      for (int e = 0; e < P * P; ++e) out[e] = (e < P) ? sums[e] : 0.5f * sums[e];
      extra = sums[P * P];
    };

    // ------------------------------------------------ a4 init, ||R||_F = ||S||_F
    float A[P * P];   // the space factor A as P*P reals (hoff)
    float anorm2;
    auto norm_a = [&]() __attribute__((always_inline)) {
      anorm2 = 0.f;
#pragma unroll
      for (int e = 0; e < P; ++e) anorm2 = fmaf(A[e], A[e], anorm2);
      float o = 0.f;
#pragma unroll
      for (int e = P; e < P * P; ++e) o = fmaf(A[e], A[e], o);
      anorm2 = fmaf(2.f, o, anorm2);
    };
    double normR2;
    {
      float nr = 0.f;
#pragma unroll
      for (int t = 0; t < NSL; ++t) {
        float nd = 0.f, no = 0.f;
#pragma unroll
        for (int c2 = 0; c2 < C; ++c2)
#pragma unroll
          for (int e = 0; e < P * P; ++e) {
            if (e < P) nd = fmaf(v[t][e][c2], v[t][e][c2], nd);
            else no = fmaf(v[t][e][c2], v[t][e][c2], no);
          }
        nr = fmaf(wgt(t), fmaf(0.5f, no, nd), nr);
      }
      normR2 = wsumd(double(nr));
      // A_0 = R 1 / q^2 (block sums): b is the all-ones matrix, or (fallback)
      // R vec(I_q): b is the identity
      float wb[NSL][C], none = 0.f;
#pragma unroll
      for (int t = 0; t < NSL; ++t) {
        if constexpr (C == 2) {
          wb[t][0] = wgt(t);
          wb[t][1] = (t == NSL - 1 && diag) ? 1.f : 0.f;
        } else {
          wb[t][0] = (comp && !diag) ? 0.f : wgt(t);
        }
      }
      half_a(wb, A, none);
#pragma unroll
      for (int e = 0; e < P * P; ++e) A[e] *= 1.f / float(Q * Q);
      norm_a();
      if (double(anorm2) <= 1e-24 * normR2) {   // uniform branch
#pragma unroll
        for (int t = 0; t < NSL; ++t)
#pragma unroll
          for (int c2 = 0; c2 < C; ++c2) wb[t][c2] = (t == NSL - 1 && diag) ? 1.f : 0.f;
        none = 0.f;
        half_a(wb, A, none);
        norm_a();
      }
    }

    float eta = 0.f;
    int iters = 0;
    const bool zero = !(normR2 > 0.0);
    const bool bad = !isfinite(normR2);
    chain = !bad;   // this S may seed the next pixel's
    float bv[NSL][C];
#pragma unroll
    for (int t = 0; t < NSL; ++t)
#pragma unroll
      for (int c2 = 0; c2 < C; ++c2) bv[t][c2] = 0.f;

    if (!zero && !bad) {
      // --------------------------------------------------------- a5 LR-Kron
      float Ap[P * P];   // A' = R conj(b) / ||b||^2, P*P reals

      // b = R^T conj(a) / ||a||^2
      auto half_b = [&]() __attribute__((always_inline)) {
        const float ainv = xrcp(anorm2);
#pragma unroll
        for (int t = 0; t < NSL; ++t)
#pragma unroll
          for (int c2 = 0; c2 < C; ++c2) {
            float s = 0.f;
#pragma unroll
            for (int e = 0; e < P * P; ++e) s = fmaf(A[e], v[t][e][c2], s);
            bv[t][c2] = s * ainv;
          }
      };
      // ||R - a b^T||_F^2: per entry in FP32, summed over the lanes in FP64
      auto residual = [&]() __attribute__((always_inline)) -> double {
        double rr = 0.0;
#pragma unroll
        for (int t = 0; t < NSL; ++t) {
          float rd = 0.f, ro = 0.f;
#pragma unroll
          for (int c2 = 0; c2 < C; ++c2)
#pragma unroll
            for (int e = 0; e < P * P; ++e) {
              const float m = (e < P) ? A[e] : 2.f * A[e];
              const float d = fmaf(-m, bv[t][c2], v[t][e][c2]);
              if (e < P) rd = fmaf(d, d, rd);
              else ro = fmaf(d, d, ro);
            }
          rr += double(wgt(t) * fmaf(0.5f, ro, rd));
        }
        return wsumd(rr);
      };
      // A' and the sum ||b||^2 from the current b
      auto half_ap = [&]() __attribute__((always_inline)) {
        float wb[NSL][C], bn2 = 0.f;
#pragma unroll
        for (int t = 0; t < NSL; ++t)
#pragma unroll
          for (int c2 = 0; c2 < C; ++c2) {
            wb[t][c2] = wgt(t) * bv[t][c2];
            bn2 = fmaf(wb[t][c2], bv[t][c2], bn2);
          }
        half_a(wb, Ap, bn2);
        const float binv = xrcp(bn2);
#pragma unroll
        for (int e = 0; e < P * P; ++e) Ap[e] *= binv;
      };

      // EIG_{r_a}: A <- U (U^H A' U) U^H with U the top-r_a subspace of Herm(A').
      // A pixel that slides from its predecessor starts from that pixel's
      // U_A (sUA): the two training sets differ in a few vectors.  The choice
      // depends only on the chain position, as the sliding window does.
      const bool warm = MODE == kModeRun && left_ok && k > 0 && ua_ok;
      // `first`: the first of this pixel.
      auto eig_a = [&](bool cold, bool first) __attribute__((always_inline)) {
        if (r_a == 1) {
          ES h[P * P], lam;
#pragma unroll
          for (int e = 0; e < P * P; ++e) h[e] = ES(Ap[e]);
          power_top_h<P, EC, ES>(h, ua, cold, first, 500, PREC ? 1e-12 : 2e-6, &lam);
#pragma unroll
          for (int i = 0; i < P; ++i) {
            A[i] = float(lam * cabs2(ua[i]));
#pragma unroll
            for (int j = i + 1; j < P; ++j) {
              const EC c2 = cmul(ua[i], cconj(ua[j]));
              A[hoff<P>(i, j)] = float(lam * c2.x);
              A[hoff<P>(i, j) + 1] = float(lam * c2.y);
            }
          }
          norm_a();
          return;
        }
        EC Ah[P * P];
#pragma unroll
        for (int i = 0; i < P; ++i) {
          Ah[i * P + i] = cto<EC>(make_float2(Ap[i], 0.f));
#pragma unroll
          for (int j = i + 1; j < P; ++j) {
            Ah[i * P + j] = cto<EC>(make_float2(Ap[hoff<P>(i, j)], Ap[hoff<P>(i, j) + 1]));
            Ah[j * P + i] = cconj(Ah[i * P + j]);
          }
        }
        // r_a > 1: the top-r_a subspace of Herm(A'), warm-started from the
        // previous U_A (in LDS).  p <= 4: every lane runs the same subspace
        // iteration with no cross-lane traffic; larger p: lane k holds row k
        // and the dot products are wave reductions (fewer registers).
        EC Vb[RAM][P];
        if (!cold) {
#pragma unroll
          for (int c = 0; c < RAM; ++c)
#pragma unroll
            for (int i = 0; i < P; ++i) Vb[c][i] = sUA[i * RAM + c];
        }
        wave_sync();
        if constexpr (P <= 4) {
          uniform_subspace<RAM, P, EC>([&](int i, int j) { return Ah[i * P + j]; }, r_a, Vb, cold, 500,
                                       PREC ? 1e-12 : 2e-6, first ? 0.f : kMixOwn);
        } else {
          if (lane == 0) {
#pragma unroll
            for (int e = 0; e < P * P; ++e) sA[e] = tof(Ah[e]);
          }
          wave_sync();
          float2 mrow[P];
#pragma unroll
          for (int j = 0; j < P; ++j) mrow[j] = sA[(lane < P ? lane : 0) * P + j];
          // this lane's row of the warm start, read from LDS (a lane-indexed
          // select over Vb would be compiled into a scratch array)
          EC va[RAM];
#pragma unroll
          for (int c = 0; c < RAM; ++c) va[c] = (!cold && lane < P) ? sUA[lane * RAM + c] : czero<EC>();
          wave_sync();   // sUA is rewritten below
          group_subspace<RAM, 64, P, EC>(mrow, lane < P, r_a, va, sAh, cold, 500, PREC ? 1e-12 : 2e-6, false, !cold,
                                         first ? 0.f : kMixOwn);
          // every lane gathers the whole basis from LDS
          if (lane < P) {
#pragma unroll
            for (int c = 0; c < RAM; ++c) sUA[lane * RAM + c] = va[c];
          }
          wave_sync();
#pragma unroll
          for (int c = 0; c < RAM; ++c)
#pragma unroll
            for (int i = 0; i < P; ++i) Vb[c][i] = sUA[i * RAM + c];
          wave_sync();
        }
        if (lane == 0) {
#pragma unroll
          for (int c = 0; c < RAM; ++c)
#pragma unroll
            for (int i = 0; i < P; ++i)
              if (c < r_a) sUA[i * RAM + c] = Vb[c][i];
        }
        // Hs = U^H Herm(A') U and A = U Hs U^H
        EC Hs[RAM][RAM];
#pragma unroll
        for (int a = 0; a < RAM; ++a)
#pragma unroll
          for (int b = 0; b < RAM; ++b) {
            EC sacc = czero<EC>();
            if (a < r_a && b < r_a) {
#pragma unroll
              for (int i = 0; i < P; ++i) {
                EC t2 = czero<EC>();
#pragma unroll
                for (int j = 0; j < P; ++j) t2 = cfma(Ah[i * P + j], Vb[b][j], t2);
                sacc = ccfma(Vb[a][i], t2, sacc);
              }
            }
            Hs[a][b] = sacc;
          }
#pragma unroll
        for (int i = 0; i < P; ++i)
#pragma unroll
          for (int j = i; j < P; ++j) {
            EC sacc = czero<EC>();
#pragma unroll
            for (int a = 0; a < RAM; ++a) {
              if (a >= r_a) continue;
              EC t2 = czero<EC>();
#pragma unroll
              for (int b = 0; b < RAM; ++b)
                if (b < r_a) t2 = cfma(Hs[a][b], cconj(Vb[b][j]), t2);
              sacc = cfma(Vb[a][i], t2, sacc);
            }
            if (i == j) {
              A[i] = float(sacc.x);
            } else {
              A[hoff<P>(i, j)] = float(sacc.x);
              A[hoff<P>(i, j) + 1] = float(sacc.y);
            }
          }
        norm_a();
        wave_sync();
      };

      // one call site per lambda: iteration 0 has no residual yet
      double eta_prev = INFINITY;
      for (int k = 0;; ++k) {
        double e = 0.0;
        if (k > 0) e = sqrt(residual() / normR2);
        half_b();
        if (k > 0) {
          eta = float(e);
          const bool stop = iters >= prm.max_iter ||
                            (prm.eps > 0.0 && iters >= prm.min_iter && fabs(e - eta_prev) <= prm.eps);
          if (stop) break;
          eta_prev = e;
        }
        half_ap();
        eig_a(k == 0 && !warm, k == 0);
        iters = k + 1;
      }
      // bv now holds the final b = R^T conj(a) / ||a||^2
    }
    ua_ok = !zero && !bad;

    // ------------------------------------------ enqueue for the batched tail
    wave_sync();   // S is dead from here on
    if constexpr (kWarmTail) qchain = (first + it) / kChainNarrow;
    if constexpr (kQueueLds<P, Q>) {
#pragma unroll
      for (int t = 0; t < NSL; ++t) {
        if (NS % 64 == 0 || lane + 64 * t < NS * (2 / C)) {
          if constexpr (C == 2) sQB[nq * NS + lane + 64 * t] = make_float2(bv[t][0], bv[t][1]);
          else reinterpret_cast<float*>(sQB)[2 * (nq * NS + (lane & 31)) + comp] = bv[t][0];
        }
      }
    } else {
      // the Hermitian B from its slots, B[k][l] at k * BS + l, then one row per lane
      constexpr int BS = Q + 2;   // 16-byte rows, spread over the banks
#pragma unroll
      for (int t = 0; t < NSL; ++t) {
        if (NS % 64 == 0 || lane + 64 * t < NS * (2 / C)) {
          const bool dg = t == NSL - 1 && diag;
          const int k1 = sk[t], l1 = sl[t];
          if constexpr (C == 2) {
            sBT[dg ? k1 * BS + k1 : k1 * BS + l1] = make_float2(bv[t][0], dg ? 0.f : bv[t][1]);
            sBT[dg ? l1 * BS + l1 : l1 * BS + k1] = make_float2(dg ? bv[t][1] : bv[t][0], dg ? 0.f : -bv[t][1]);
          } else {
            float* const f = reinterpret_cast<float*>(sBT);
            const int kk = comp ? l1 : k1;   // the diagonal entry of this lane
            f[dg ? 2 * (kk * BS + kk) : 2 * (k1 * BS + l1) + comp] = bv[t][0];
            f[dg ? 2 * (kk * BS + kk) + 1 : 2 * (l1 * BS + k1) + comp] = dg ? 0.f : (comp ? -bv[t][0] : bv[t][0]);
          }
        }
      }
      wave_sync();
      if (tg == nq && tk < Q) {
        const float4* const row = reinterpret_cast<const float4*>(sBT + tk * BS);
#pragma unroll
        for (int l = 0; l < Q / 2; ++l) {
          const float4 two = row[l];
          Bq[2 * l] = make_float2(two.x, two.y);
          Bq[2 * l + 1] = make_float2(two.z, two.w);
        }
      }
    }
    if (lane == 0) {
      sQidx[nq] = idx;
      sQflag[nq] = bad ? 2 : (zero ? 1 : 0);
      sQeta[nq] = eta;
      sQit[nq] = iters;
    }
    if (r_a == 1) {
      // one lane writes U_A with static indices (a lane-indexed select over
      // ua[] is compiled into a scratch array)
      if (lane == 0) {
#pragma unroll
        for (int i = 0; i < P; ++i) sQUA[nq][i * RAM] = (zero || bad) ? czero<EC>() : ua[i];
      }
    } else if (lane < P * RAM) {
      sQUA[nq][lane] = (zero || bad) ? czero<EC>() : sUA[lane];
    }
    wave_sync();
    ++nq;
  };

  // one call site each for the pixel body and the tail, which runs when the
  // queue is full, at the end of a chain (warm tail) and at the end of the run
  for (int64_t it = 0; it < count; ++it) {
    pixel(it);
    const bool end = it + 1 == count || (kWarmTail && (first + it + 1) % kChainNarrow == 0);
    if (nq == G || (end && nq > 0)) {
      tail(nq);
      nq = 0;
    }
  }
}

}  // namespace
}  // namespace kstap

#include "kstap_bank.h"

namespace kstap {
namespace {

// Wavefronts per SIMD that the run-mode kernels are compiled for.  The p = 3,
// q = 8 FP32 kernel needs 172 registers on its own and spills one or two (outside
// its loops) at the 168 of three: 512 x 512, n = 64 874 -> 726 us.  p = 2, q = 8
// needs 151 and runs three a SIMD either way (471 us).  p = 3, q = 8 with r_b > 4
// needs 218: 960 us with two, 993 with three.  p = 3, q = 16 needs 224: at 168 it
// spills some 60 accesses a pixel and takes the 1024 x 1024 frame 7.9 ms instead
// of 5.7.
template <int P, int Q, int RBM, int PREC, bool PLAIN>
constexpr int kWavesPerSimd = (PLAIN && PREC == 0 && P <= 3 && Q == 8 && RBM == 4) ? 3 : 2;

// Which statistic a kernel is compiled for: the plain one, its variants
// (filter, enhancement, passes), or the FP32 Doppler bank (kstap_bank.h).
enum Variant { kPlain = 0, kVariant = 1, kBank = 2 };

// Whole frame (run mode) or pixel list (probe mode).  Run mode: workgroup ids
// are remapped so each of the 8 XCDs takes a contiguous share of the frame.
// VAR: the statistic variants (filter, Doppler bank, enhancement, passes) are
// compiled into a kernel of their own, so that the plain statistic keeps its
// register budget.
template <int P, int Q, int RBM, int MODE, int PREC, int VAR = kPlain>
__global__ __launch_bounds__(64, (kWavesPerSimd<P, Q, RBM, PREC, VAR == kPlain && MODE == kModeRun>)) void kstap_kernel(const KParams prm) {
  constexpr bool kBankKernel = VAR == kBank && PREC == 0;
  __shared__ __attribute__((aligned(16))) char lds[kBankKernel ? BankLds<P, Q, RBM>::bytes : Lds<P, Q, RBM, PREC>::bytes];
  int64_t first, count;
  if (MODE == kModeRun) {
    const int per = gridDim.x >> 3;   // grid is a multiple of 8 (one share per XCD)
    const int logical = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (logical >= prm.nlogical) return;
    const int64_t total = tiled_positions(prm.H, prm.W);
    first = int64_t(logical) * prm.pix_per_block;
    count = total - first;
    if (count > prm.pix_per_block) count = prm.pix_per_block;
  } else {
    first = int64_t(blockIdx.x) * prm.pix_per_block;
    count = prm.npix - first;
    if (count > prm.pix_per_block) count = prm.pix_per_block;
  }
  if constexpr (kBankKernel) run_pixels_bank<P, Q, RBM>(prm, first, count, lds);
  else run_pixels<P, Q, RBM, MODE, PREC, VAR != kPlain>(prm, first, count, lds);
}

// Persistent batched kernel: every workgroup pops work items (runs of `ppb`
// consecutive tiled-order positions of one tile's range [range_first,
// range_end)) from a
// device counters until every queue is empty (kQueues queues, see kstap_internal.h).  Items are numbered tile after
// tile in the order of `order` (longest tiles first); prefix[j] is the first item of order[j] (prefix[nt] = total).
template <int P, int Q, int RBM, int PREC>
constexpr int resident_wgs() {   // a compute unit's share of registers and LDS (160 KB, 16 bytes beside the carve-out)
  const int waves = 4 * kWavesPerSimd<P, Q, RBM, PREC, true>;
  const int lds = int(size_t(160 * 1024) / (Lds<P, Q, RBM, PREC>::bytes + 16));
  return waves < lds ? waves : lds;
}
template <int P, int Q, int RBM, int PREC>
__global__ __launch_bounds__(64, (kWavesPerSimd<P, Q, RBM, PREC, true>)) void kstap_persistent(const KParams* __restrict__ descs,
                                                          const int32_t* __restrict__ order,
                                                          const int64_t* __restrict__ prefix, int nt,
                                                          int ppb, unsigned long long* counter) {
  __shared__ __attribute__((aligned(16))) char lds[Lds<P, Q, RBM, PREC>::bytes];
  __shared__ long long s_item;
  const int64_t total = prefix[nt];
  // queue q holds items [total q / kQueues, total (q + 1) / kQueues); start
  // with this workgroup's XCD (dispatch is round-robin over the XCDs), then
  // move on whenever a queue is empty: every workgroup leaves after finding
  // all kQueues queues empty
  int q = int(blockIdx.x % kQueues), empty = 0;
  while (true) {
    const int64_t qlo = total * q / kQueues, qhi = total * (q + 1) / kQueues;
    if (threadIdx.x == 0) s_item = (long long)atomicAdd(counter + q, 1ull);
    wave_sync();
    const int64_t item = qlo + s_item;
    wave_sync();
    if (item >= qhi) {
      if (++empty == kQueues) break;
      q = (q + 1) % kQueues;
      continue;
    }
    int lo = 0, hi = nt - 1;   // last j with prefix[j] <= item
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (prefix[mid] <= item) lo = mid; else hi = mid - 1;
    }
    const KParams& prm = descs[order[lo]];
    const int64_t first = prm.range_first + (item - prefix[lo]) * ppb;
    int64_t count = prm.range_end - first;
    if (count > ppb) count = ppb;
    run_pixels<P, Q, RBM, kModeRun, PREC>(prm, first, count, lds);
  }
}

// ====================================================================
// Wide pixels (p*q > 64): one 512-lane workgroup (8 wavefronts) per pixel.
//
// The covariance tiles (16 x 16, the upper block-triangle, some as their
// transposes) are dealt so that wave w owns row block w.  Training vectors are
// staged in LDS 16 at a time, split into BF16 parts (two for PREC 1, three for
// PREC 0: as scm_split, so that the products run on the BF16 pipe beside the
// other wave's VALU work), double-buffered: the global loads of the next chunk
// are in flight while the waves run the MFMAs of the current one.  n S stays
// in the accumulators, and S passes through LDS (its upper q x q blocks) to
// the threads that solve.  In run mode every pixel of a sliding-window chain
// but the first starts from the previous pixel's n S (a one-pixel move) and
// stages only the training vectors that enter the stencil (added) and leave
// it (subtracted), as the narrow FP32 kernels do.  LR-Kron runs on the
// Hermitian half of S (Slots), one value of a slot per thread and held in its
// registers: per iteration one FP64 pass (residual and new b), one barrier for
// the P^2 sums of R conj(b) over the waves, EIG_{r_a} on wave 0 and one
// barrier for A.  Sweeps over all blocks of S in LDS, with a pass of their own
// for the block sums and four barriers, took the 512 x 512, p = 5, q = 24,
// n = 256 frame 44.4 ms (FP32) and this 30.4 ms; p = 6, q = 16 in two passes
// at 256 x 256 14.6 -> 9.9 ms.  With the split covariance in place of FP32
// MFMA on staged FP32 (tiles dealt round-robin, S reloaded for every pixel)
// 23.3 and 9.0 ms.  The time factors are queued as slots
// in LDS and the batched tail (a6 + a8) runs 64/q' pixels per wave on waves
// 0-3 at once.  Eight waves (two per SIMD, the LDS footprint allows one
// workgroup per compute unit) hide each other's LDS, reduction and barrier
// latencies; with four, each SIMD ran a single wave.
// ====================================================================
constexpr int kWideWaves = 8;                      // waves per wide workgroup
constexpr int kWideThreads = 64 * kWideWaves;
constexpr int kTailWaves = 4;                      // waves that run the batched tail

template <int P, int Q, int RBM, int PREC>
struct WideLds {
  using EC = typename Pick<PREC == 1, double2, float2>::type;
  static constexpr int PQ = P * Q;
  static constexpr int NB = (PQ + 15) / 16;
  static constexpr int NBLK = P * (P + 1) / 2;
  static constexpr int RAM = (P < kMaxRA) ? P : kMaxRA;
  static constexpr int G = Groups<Q>::G;
  static constexpr int NQ = kTailWaves * G;                          // pixels per batched tail
  static constexpr size_t kS = sizeof(float2) * NBLK * Q * (Q + 1);  // upper blocks of S
  static constexpr int NPART = PREC ? 2 : 3;                         // BF16 parts of a staged sample
  static constexpr size_t rowb = 80;                                 // padded bytes per staged row (16 vectors)
  static constexpr size_t stage1 = NPART * NB * 16 * rowb;
  static constexpr size_t kStage = 2 * stage1;
  static constexpr size_t kTail1 = tail_scratch_bytes<RBM, Q, G, EC>;      // subspace scratch of a tail wave
  static constexpr size_t kTail = kTail1 * kTailWaves;
  static constexpr size_t kST = kStage > kTail ? kStage : kTail;
  static constexpr size_t oS = 0;
  static constexpr size_t oStage = (kS + 15) / 16 * 16;              // staging; tail scratch between pixels
  static constexpr size_t oHq = oStage + (kST + 15) / 16 * 16;       // float2[NQ][Q*Q/2]: queued B, as slots
  static constexpr size_t oQUA = oHq + sizeof(float2) * NQ * Q * Q / 2;   // EC[NQ][P*RAM]: queued U_A
  static constexpr size_t oUA = oQUA + sizeof(EC) * NQ * P * RAM;    // EC[P*RAM]
  static constexpr size_t oAh = oUA + sizeof(EC) * P * RAM;          // EC[P*P]
  static constexpr size_t oRedD = oAh + sizeof(EC) * P * P;          // double[kWideWaves]
  static constexpr size_t oQidx = oRedD + sizeof(double) * kWideWaves;   // int64[NQ]
  static constexpr size_t oRed = oQidx + sizeof(int64_t) * NQ;       // float[kWideWaves][KRED]
  static constexpr int KRED = 2 * P * P + 8;
  static constexpr size_t oA = oRed + sizeof(float) * kWideWaves * KRED;   // float2[P*P]
  static constexpr size_t oOff = oA + sizeof(float2) * P * P;        // int[kMaxN]
  static constexpr size_t oDel = oOff + sizeof(int) * kMaxN;         // int[3][2*kMaxDelta]: per move, entering, leaving
  static constexpr size_t oQflag = oDel + sizeof(int) * 6 * kMaxDelta;   // int[NQ]
  static constexpr size_t oQit = oQflag + sizeof(int) * NQ;          // int[NQ]
  static constexpr size_t oQeta = oQit + sizeof(int) * NQ;           // float[NQ]
  static constexpr size_t bytes = (oQeta + sizeof(float) * NQ + 15) / 16 * 16;
  static_assert(bytes <= 160 * 1024, "LDS of one workgroup");
};

__device__ __forceinline__ void block_sync() { __syncthreads(); }

template <int P, int Q, int RBM, int MODE, int PREC, bool VAR = false>
__device__ __forceinline__ void run_pixels_wide(const KParams& prm, int64_t first, int64_t count, char* lds) {
  using EC = typename Pick<PREC == 1, double2, float2>::type;
  using ES = decltype(EC{}.x);
  using L = WideLds<P, Q, RBM, PREC>;
  constexpr int PQ = P * Q;
  constexpr int NB = L::NB;
  constexpr int QS = Q + 1;
  constexpr int QQ = Q * Q;
  constexpr int NDT = (QQ + kWideThreads - 1) / kWideThreads;   // dimensions of b per thread
  constexpr int RAM = L::RAM;
  constexpr int MYP = NB / 2 + 1;   // tiles per wave at most
  constexpr int QP = Groups<Q>::QP;
  constexpr int G = L::G;
  constexpr int NQ = L::NQ;

  float2* const sS = reinterpret_cast<float2*>(lds + L::oS);
  char* const stage = lds + L::oStage;
  float* const red = reinterpret_cast<float*>(lds + L::oRed);
  double* const redd = reinterpret_cast<double*>(lds + L::oRedD);
  EC* const sUA = reinterpret_cast<EC*>(lds + L::oUA);
  EC* const sAh = reinterpret_cast<EC*>(lds + L::oAh);
  float2* const sA = reinterpret_cast<float2*>(lds + L::oA);
  int* const sOff = reinterpret_cast<int*>(lds + L::oOff);
  int* const sDel = reinterpret_cast<int*>(lds + L::oDel);
  float2* const sHq = reinterpret_cast<float2*>(lds + L::oHq);
  EC (*const sQUA)[P * RAM] = reinterpret_cast<EC (*)[P * RAM]>(lds + L::oQUA);
  int64_t* const sQidx = reinterpret_cast<int64_t*>(lds + L::oQidx);
  int* const sQflag = reinterpret_cast<int*>(lds + L::oQflag);
  int* const sQit = reinterpret_cast<int*>(lds + L::oQit);
  float* const sQeta = reinterpret_cast<float*>(lds + L::oQeta);

  // the wave index is uniform: keep it (and the tile pairs below) in SGPRs
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int n = prm.n, H = prm.H, W = prm.W;
  const int r_a = prm.r_a, r_b = prm.r_b;

  // sample offsets of the stencil, and per one-pixel move those of the
  // entering then the leaving vectors
  block_sync();
  for (int m = tid; m < n; m += kWideThreads) sOff[m] = (int(prm.st[2 * m]) * W + int(prm.st[2 * m + 1])) * Q;
  for (int m = tid; m < 6 * kMaxDelta; m += kWideThreads) {
    const int mv = m / (2 * kMaxDelta), e = m - mv * (2 * kMaxDelta);
    int off = 0;
    if (prm.nadd[0] >= 0) {
      const int na = prm.nadd[mv], nr = prm.nrem[mv];   // each <= kMaxDelta
      if (e < na) off = (int(prm.dadd[mv][2 * e]) * W + int(prm.dadd[mv][2 * e + 1])) * Q;
      else if (e < na + nr) off = (int(prm.drem[mv][2 * (e - na)]) * W + int(prm.drem[mv][2 * (e - na) + 1])) * Q;
    }
    sDel[m] = off;
  }
  block_sync();

  // This wave's tiles: row block `wave` against column blocks wave + u mod NB,
  // u < NB / 2, and u = NB / 2 for the first half of the waves (each tile of
  // the upper block-triangle once, some as its transpose), so that a wave
  // prepares one block's row operands for all its tiles.
  static_assert(NB % 2 == 0 && NB <= kWideWaves, "one row block per wave");
  const int nmine = wave >= NB ? 0 : NB / 2 + (wave < NB / 2 ? 1 : 0);
  auto colblk = [&](int u) __attribute__((always_inline)) { return wave + u >= NB ? wave + u - NB : wave + u; };
  f4 accR[MYP], accI[MYP];   // n S of the pixel processed last
#pragma unroll
  for (int u = 0; u < MYP; ++u) accR[u] = accI[u] = f4{0.f, 0.f, 0.f, 0.f};

  constexpr int NIT = (16 * PQ + kWideThreads - 1) / kWideThreads;
  const int64_t plane = int64_t(H) * W * Q;

  // ------------------------------------------ a6 + a8 for the queued pixels
  // wave w < kTailWaves serves queue slots w*G .. w*G + G - 1; lane k of a
  // slot's group takes row k of its Hermitian time factor
  auto tail = [&](int nfill) __attribute__((always_inline)) {
    int lanev = threadIdx.x & 63;
    asm volatile("" : "+v"(lanev));   // per call: no lane arithmetic hoisted out of the pixel loop
    const int lane = lanev;
    if (wave < kTailWaves) {   // uniform per wave; the tail syncs inside a wave only
      const int slot = wave * G + lane / QP, tk = lane % QP;
      float2 Bq[Q];
      queue_row<P, Q>(sHq + slot * (QQ / 2), tk < Q ? tk : 0, Bq);   // empty slots: whatever is there, unused
      char* const scr = stage + wave * L::kTail1;
      EC vb[RBM];
#pragma unroll
      for (int c = 0; c < RBM; ++c) vb[c] = czero<EC>();
      bool vb_ok;
      if constexpr (VAR) {
        tail_batch<P, Q, RBM, EC, true>(prm, Bq, slot, nfill, sQflag, sQidx, sQUA, reinterpret_cast<EC*>(scr),
                                        PREC ? 1e-10 : 2e-6, vb, false, vb_ok);
      } else {
        with_rank<RBM>(r_b, [&](auto rank) __attribute__((always_inline)) {
          tail_rows<P, Q, RBM, decltype(rank)::value, MODE, EC, true>(prm, Bq, wave * G, nfill, sQflag, sQidx, sQeta, sQit,
                                                                      sQUA, scr, PREC ? 1e-10 : 2e-6, vb, false, vb_ok);
        });
      }
    }
    block_sync();
  };

  int nq = 0;
  bool chain = false;   // the previous position left a usable S in LDS
  bool ua_ok = false;   // sUA holds the U_A of the pixel processed last
  auto pixel = [&](int64_t itp) __attribute__((always_inline)) {
    // Opaque per-pixel copy of the thread index: the index arithmetic below
    // (staging items, tile elements, q x q entries) is redone for every pixel
    // rather than hoisted out of the pixel loop, where at two waves per SIMD
    // it would not fit in registers.
    int tidv = threadIdx.x;
    asm volatile("" : "+v"(tidv));
    const int tid = tidv, lane = tidv & 63;
    // staging items of this thread: (vector v, row rho) = divmod(tid + 512 it, PQ)
    auto item = [&](int it, int* v, int* rho) __attribute__((always_inline)) -> bool {
      const int e = tid + kWideThreads * it;
      *v = e / PQ;
      *rho = e - *v * PQ;
      return e < 16 * PQ;
    };
    int64_t idx;
    int r, c;
    const bool left_ok = chain;
    chain = false;
    if (MODE == kModeRun) {
      if (!tiled_pixel(first + itp, H, W, &r, &c)) return;
      idx = int64_t(r) * W + c;
    } else {
      idx = first + itp;
      r = prm.pix[2 * idx];
      c = prm.pix[2 * idx + 1];
    }
    const bool valid = r >= prm.r0 && r < prm.r1 && c >= prm.c0 && c < prm.c1;
    if (!valid) {
      if (tid == 0) {
        if (MODE == kModeRun) write_outside(prm, idx);
        else prm.T[idx] = 0.f;
        if (MODE == kModeProbe) {
          if (prm.eta) prm.eta[idx] = 0.f;
          if (prm.iters) prm.iters[idx] = 0;
        }
      }
      if (MODE == kModeProbe) {
        if (prm.UA)
          for (int e = tid; e < P * r_a; e += kWideThreads) prm.UA[idx * P * r_a + e] = cz();
        if (prm.UB)
          for (int e = tid; e < Q * r_b; e += kWideThreads) prm.UB[idx * Q * r_b + e] = cz();
      }
      return;
    }
    const float2* xp = prm.x + (int64_t(r) * W + c) * Q;

    // ------------------------------------------------------------ a2 SCM
    // Full sum over the n stencil vectors, or (sliding window, a one-pixel
    // move inside a unit) the previous pixel's n*S plus the entering vectors
    // minus the leaving ones: list entries m < npos are added, the others
    // subtracted.
    const int mv = tiled_move(first + itp, H, W, kChainWide);
    const bool slide = MODE == kModeRun && left_ok && mv >= 0 && prm.nadd[0] >= 0;
    const int* const list = slide ? sDel + mv * 2 * kMaxDelta : sOff;
    // EIG_{r_a} of a pixel that slides from its predecessor starts from that
    // pixel's U_A (sUA); the choice follows the chain, as the sliding window
    const bool warm = slide && ua_ok;
    const int cnt = slide ? prm.nadd[mv] + prm.nrem[mv] : n;
    const int npos = slide ? prm.nadd[mv] : n;
    const float fn = float(n);
    if (!slide) {
#pragma unroll
      for (int u = 0; u < MYP; ++u) accR[u] = accI[u] = f4{0.f, 0.f, 0.f, 0.f};
    }
    const int nch = (cnt + 15) >> 4;
    float2 pre[NIT];
    auto gload = [&](int ch) __attribute__((always_inline)) {
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        int v, rho;
        const bool in = item(it, &v, &rho);
        const int m = ch * 16 + v;
        const bool ok = in && m < cnt;
        const int chn = rho / Q;
        pre[it] = load_or_zero(xp + chn * plane + (rho - chn * Q) + list[ok ? m : 0], ok);
      }
    };
    auto sstore = [&](int buf) __attribute__((always_inline)) {
      char* base = stage + buf * L::stage1;
#pragma unroll
      for (int it = 0; it < NIT; ++it) {
        int v, rho;
        if (!item(it, &v, &rho)) continue;
        // part e of the pair (re, im), as split3 (the first two for PREC 1)
        uint32_t part[3];
        split3(pre[it].x, pre[it].y, part);
#pragma unroll
        for (int e = 0; e < L::NPART; ++e)
          *reinterpret_cast<uint32_t*>(base + size_t(e * NB * 16 + rho) * L::rowb + 4 * v) = part[e];
      }
    };
    gload(0);
    sstore(0);
    block_sync();
    for (int ch = 0; ch < nch; ++ch) {
      const int buf = ch & 1;
      if (ch + 1 < nch) gload(ch + 1);
      const char* base = stage + buf * L::stage1;
      const int g = lane >> 4, rr = lane & 15;
      if (wave < NB) {   // uniform
        // operand of block I: row 16 I + rr, vectors 4g .. 4g + 3 (re, im) = 16
        // bytes (rows past p q hold anything: they meet no stored element);
        // the row operand of a subtracted vector is negated
        auto ld = [&](int I, int e) __attribute__((always_inline)) -> u4 {
          return *reinterpret_cast<const u4*>(base + size_t((e * NB + I) * 16 + rr) * L::rowb + g * 16);
        };
        u4 msk;
#pragma unroll
        for (int e = 0; e < 4; ++e) msk[e] = (ch * 16 + 4 * g + e >= npos) ? 0x80008000u : 0u;
        bf8 y[L::NPART], z[L::NPART];   // rows of Re and of Im
#pragma unroll
        for (int e = 0; e < L::NPART; ++e) {
          y[e] = __builtin_bit_cast(bf8, ld(wave, e) ^ msk);
          z[e] = swap_neg(y[e]);
        }
        // products of the parts: those below 2^-26 (three parts) or 2^-16 (two)
        // of the leading one are dropped
        constexpr int NPROD = L::NPART == 3 ? 6 : 3;
        constexpr int pa3[6] = {2, 0, 1, 1, 0, 0}, pb3[6] = {0, 2, 1, 0, 1, 0}, pa2[3] = {0, 0, 1}, pb2[3] = {0, 1, 0};
#pragma unroll
        for (int u = 0; u < MYP; ++u) {
          if (u >= nmine) continue;   // uniform
          const int J = colblk(u);
          bf8 c[L::NPART];
#pragma unroll
          for (int e = 0; e < L::NPART; ++e) c[e] = __builtin_bit_cast(bf8, ld(J, e));
#pragma unroll
          for (int w = 0; w < NPROD; ++w) {
            const int ea = L::NPART == 3 ? pa3[w] : pa2[w], eb = L::NPART == 3 ? pb3[w] : pb2[w];
            accR[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(y[ea], c[eb], accR[u], 0, 0, 0);
            accI[u] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(z[ea], c[eb], accI[u], 0, 0, 0);
          }
        }
      }
      if (ch + 1 < nch) sstore(buf ^ 1);
      block_sync();
    }
    // S to LDS as upper blocks: every element (a, b), a <= b, has one writer
    // (the staging barrier above also ends every wave's use of the old S)
    {
      int trow = 4 * (lane >> 4), tcol = lane & 15;
      const float inv_n = 1.f / fn;
#pragma unroll
      for (int u = 0; u < MYP; ++u) {
        if (u >= nmine) continue;   // uniform
        const int J = colblk(u);
        const bool up = J >= wave;   // uniform: the tile, or its transpose, lies above the diagonal
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const int r1 = 16 * wave + trow + q4, c1 = 16 * J + tcol;
          const int a = up ? r1 : c1, b = up ? c1 : r1;
          if (a < PQ && b < PQ && a <= b)
            sput<P, Q>(sS, a, b, make_float2(accR[u][q4] * inv_n, (up ? accI[u][q4] : -accI[u][q4]) * inv_n));
        }
      }
    }
    block_sync();

    // ------------------------- this thread's dimensions of b (Slots), from S
    // Thread e + 512 t holds value x (e < q^2 / 2) or y of one slot.  Rotating
    // the y threads' entries by -j (rot) gives both the same sums.
    float v[NDT][P * P], wgt[NDT], one[NDT];   // values, weight, and the all-ones b
    int kb[NDT], lb[NDT], comp[NDT];
    bool dgl[NDT], has[NDT];
#pragma unroll
    for (int t = 0; t < NDT; ++t) {
      const int e = tid + kWideThreads * t;
      has[t] = e < QQ;
      comp[t] = e >= QQ / 2 && has[t] ? 1 : 0;
      const int s = has[t] ? e - comp[t] * (QQ / 2) : 0;
      const int d = s / Q + 1, k = s - (d - 1) * Q;
      dgl[t] = d == Q / 2 && k >= Q / 2;
      kb[t] = dgl[t] ? k - Q / 2 : k;
      lb[t] = dgl[t] ? k : (k + d >= Q ? k + d - Q : k + d);
      wgt[t] = !has[t] ? 0.f : dgl[t] ? 1.f : 2.f;
      one[t] = (comp[t] && !dgl[t]) ? 0.f : 1.f;
      const int dk = comp[t] ? lb[t] : kb[t];   // the diagonal entry of this thread
      const int o1 = dgl[t] ? dk * QS + dk : kb[t] * QS + lb[t];
      const int o2 = dgl[t] ? o1 : lb[t] * QS + kb[t];
      const bool rot = comp[t] && !dgl[t];
      if (wave * 64 + kWideThreads * t < QQ) {   // uniform: some lane of this wavefront has one
#pragma unroll
        for (int i = 0; i < P; ++i) {
          const float2 s1 = sS[sblk<P, Q>(i, i) + o1];
          v[t][i] = rot ? s1.y : s1.x;
#pragma unroll
          for (int j = i + 1; j < P; ++j) {
            const float2 a = sS[sblk<P, Q>(i, j) + o1], u = sS[sblk<P, Q>(i, j) + o2];
            v[t][hoff<P>(i, j)] = rot ? a.y - u.y : a.x + u.x;
            v[t][hoff<P>(i, j) + 1] = rot ? u.x - a.x : a.y + u.y;
          }
        }
      } else {
#pragma unroll
        for (int e2 = 0; e2 < P * P; ++e2) v[t][e2] = 0.f;
      }
    }
    // Partial sums of R conj(b) (given w b) and of `extra` over this
    // wavefront, to red; rr (FP64) to redd
    constexpr int NR = (P * P + 1 + 3) / 4 * 4;
    constexpr int NACT = (QQ + 63) / 64 < kWideWaves ? (QQ + 63) / 64 : kWideWaves;   // wavefronts with dimensions
    auto publish = [&](const float (&wb)[NDT], float extra, double rr) __attribute__((always_inline)) {
      if (wave < NACT) {
        float sums[NR];
#pragma unroll
        for (int e = 0; e < NR; ++e) sums[e] = (e == P * P) ? extra : 0.f;
#pragma unroll
        for (int t = 0; t < NDT; ++t) {
          if (t > 0 && wave * 64 + kWideThreads * t >= QQ) continue;   // uniform
#pragma unroll
          for (int e = 0; e < P * P; ++e) sums[e] = fmaf(v[t][e], wb[t], sums[e]);
        }
        wsum_n<NR>(sums);
        rr = wsumd(rr);
        if (lane == 0) {
#pragma unroll
          for (int e = 0; e <= P * P; ++e) red[wave * L::KRED + e] = sums[e];
          redd[wave] = rr;
        }
      }
      block_sync();
    };
    // the sum over the wavefronts of entry e <= P*P (R conj(b): P*P reals)
    auto total = [&](int e) __attribute__((always_inline)) -> float {
      float s = 0.f;
#pragma unroll
      for (int w = 0; w < NACT; ++w) s += red[w * L::KRED + e];
      return e < P ? s : e < P * P ? 0.5f * s : s;
    };
    auto totald = [&]() __attribute__((always_inline)) -> double {
      double s = 0.0;
#pragma unroll
      for (int w = 0; w < NACT; ++w) s += redd[w];
      return s;
    };

    // ------------------------------------------------ a4 init, ||R||_F = ||S||_F
    // The space factor A is P*P reals (hoff) in LDS (sA), copied to registers
    // by every thread for a sweep.
    float* const sAr = reinterpret_cast<float*>(sA);
    float A[P * P], anorm2;
    auto load_a = [&]() __attribute__((always_inline)) {
      float nd = 0.f, no = 0.f;
#pragma unroll
      for (int e = 0; e < P * P; ++e) {
        A[e] = sAr[e];
        if (e < P) nd = fmaf(A[e], A[e], nd);
        else no = fmaf(A[e], A[e], no);
      }
      anorm2 = fmaf(2.f, no, nd);
    };
    double normR2;
    {
      double nr = 0.0;   // exact squares of the FP32 entries, FP64 sums
      float wb[NDT];
#pragma unroll
      for (int t = 0; t < NDT; ++t) {
        double nd = 0.0, no = 0.0;
#pragma unroll
        for (int e = 0; e < P * P; ++e) {
          const double x = v[t][e];
          if (e < P) nd = fma(x, x, nd);
          else no = fma(x, x, no);
        }
        nr = fma(double(wgt[t]), fma(0.5, no, nd), nr);
        wb[t] = wgt[t] * one[t];
      }
      publish(wb, 0.f, nr);
      normR2 = totald();
      if (tid < P * P) sAr[tid] = total(tid) * (1.f / float(QQ));
      block_sync();
      load_a();
      if (double(anorm2) <= 1e-24 * normR2) {   // fallback: partial trace R vec(I_q) (uniform)
#pragma unroll
        for (int t = 0; t < NDT; ++t) wb[t] = (has[t] && dgl[t]) ? 1.f : 0.f;
        publish(wb, 0.f, 0.0);
        if (tid < P * P) sAr[tid] = total(tid);
        block_sync();
        load_a();
      }
    }

    float eta = 0.f;
    int iters = 0;
    const bool zero = !(normR2 > 0.0);
    const bool bad = !isfinite(normR2);
    float bv[NDT];
#pragma unroll
    for (int t = 0; t < NDT; ++t) bv[t] = 0.f;
    EC ua[P];
#pragma unroll
    for (int i = 0; i < P; ++i) ua[i] = warm ? sUA[i * RAM] : czero<EC>();

    if (!zero && !bad) {
      // EIG_{r_a} of A' = R conj(b) / ||b||^2 on wave 0 (the sums over the
      // wavefronts are in red), which writes A to sA
      auto eig_a = [&](bool cold, bool first) __attribute__((always_inline)) {
        if (wave != 0) return;
        const float mine = total(lane <= P * P ? lane : P * P);
        const float binv = 1.f / __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, mine), P * P));
        if (r_a == 1) {
          ES h[P * P], lam;
#pragma unroll
          for (int e = 0; e < P * P; ++e)
            h[e] = ES(__builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, mine), e)) * binv);
          power_top_h<P, EC, ES>(h, ua, cold, first, 500, PREC == 1 ? 1e-12 : 2e-6, &lam);
          if (lane == 0) {
#pragma unroll
            for (int i = 0; i < P; ++i) {
              sAr[i] = float(lam * cabs2(ua[i]));
#pragma unroll
              for (int j = i + 1; j < P; ++j) {
                const EC c2 = cmul(ua[i], cconj(ua[j]));
                sAr[hoff<P>(i, j)] = float(lam * c2.x);
                sAr[hoff<P>(i, j) + 1] = float(lam * c2.y);
              }
            }
          }
          return;
        }
        // r_a > 1: subspace iteration with lane k < P holding row k of A' and
        // of the basis, warm-started from the previous U_A; then Hs = U^H A' U
        // (r_a x r_a) and A = U Hs U^H, entry (i, j) on lane i P + j.  The
        // staging area is free and holds the basis exchange and Hs.  FP32: a
        // group of 8 lanes (the others rows of zeros) and r_a a constant, two
        // passes of p = 6, q = 16 at 128 x 128 2.27 -> 1.68 ms against the
        // whole wave and a run-time rank, which the FP64 solves keep (their
        // unrolled bases spill: p = 5, q = 24 at 192 x 192 6.5 -> 7.3 ms).
        static_assert(P <= 8, "a row per lane of a group of 8");
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));   // nothing of this path is hoisted out of the iteration
        EC* const sHs = reinterpret_cast<EC*>(stage);                               // [RAM][RAM]
        char* const scr = stage + (sizeof(EC) * RAM * RAM + 15) / 16 * 16;           // basis exchange
        if (lane < P * P) sAr[lane] = mine * binv;
        lane_sync();
        const int ai = lane / P, aj = lane - (lane / P) * P;
        if (lane < P * P) {
          const int lo = ai < aj ? ai : aj, hi = ai < aj ? aj : ai;
          EC h;
          h.x = ai == aj ? sAr[ai] : sAr[hoff<P>(lo, hi)];
          h.y = ai == aj ? 0.f : ai < aj ? sAr[hoff<P>(lo, hi) + 1] : -sAr[hoff<P>(lo, hi) + 1];
          sAh[lane] = h;
        }
        lane_sync();
        const bool rowk = lane < P;
        float2 mrow[P];
#pragma unroll
        for (int j = 0; j < P; ++j) mrow[j] = rowk ? tof(sAh[lane * P + j]) : cz();
        if constexpr (PREC == 0) {
          auto solve = [&](auto rank) __attribute__((always_inline)) {
            constexpr int R = decltype(rank)::value;
            EC va[R];
#pragma unroll
            for (int c = 0; c < R; ++c)
              va[c] = !rowk ? czero<EC>() : cold ? cto<EC>(omega(lane, c)) : sUA[lane * RAM + c];
            rows_subspace<R, 8, P, EC, true>(mrow, lane >> 3, lane & 7, va, scr, 500, 2e-6, !cold, !cold,
                                             first ? 0.f : kMixOwn);
            if (rowk) {
#pragma unroll
              for (int c = 0; c < R; ++c) sUA[lane * RAM + c] = va[c];
            }
            lane_sync();
            // (A' U)[k][b] on lane k, then Hs[a][b] = sum_k conj(U[k][a]) (A' U)[k][b]
            EC au[R], hs[R][R];
#pragma unroll
            for (int b = 0; b < R; ++b) {
              au[b] = czero<EC>();
#pragma unroll
              for (int j = 0; j < P; ++j) au[b] = cfma(cto<EC>(mrow[j]), sUA[j * RAM + b], au[b]);
            }
#pragma unroll
            for (int a2 = 0; a2 < R; ++a2)
#pragma unroll
              for (int b = 0; b < R; ++b) hs[a2][b] = gsum<8>(ccmul(va[a2], au[b]));
            if (lane == 0) {
#pragma unroll
              for (int a2 = 0; a2 < R; ++a2)
#pragma unroll
                for (int b = 0; b < R; ++b) sHs[a2 * RAM + b] = hs[a2][b];
            }
          };
          if (r_a == 2) solve(Int<2>());
          else if (r_a == 3) solve(Int<3>());
          else solve(Int<RAM>());
          lane_sync();
        } else {
          EC va[RAM];
#pragma unroll
          for (int c = 0; c < RAM; ++c) va[c] = (!cold && rowk) ? sUA[lane * RAM + c] : czero<EC>();
          group_subspace<RAM, 64, P, EC, true>(mrow, rowk, r_a, va, reinterpret_cast<EC*>(scr), cold, 500, 1e-12, false, !cold,
                                               first ? 0.f : kMixOwn);
          lane_sync();
          if (rowk) {
#pragma unroll
            for (int c = 0; c < RAM; ++c)
              if (c < r_a) sUA[lane * RAM + c] = va[c];
          }
          lane_sync();
          // (A' U)[k][b] on lane k, then Hs[a][b] = sum_k conj(U[k][a]) (A' U)[k][b]
          EC au[RAM];
#pragma unroll
          for (int b = 0; b < RAM; ++b) {
            au[b] = czero<EC>();
            if (b < r_a && rowk) {
#pragma unroll
              for (int j = 0; j < P; ++j) au[b] = cfma(sAh[lane * P + j], sUA[j * RAM + b], au[b]);
            }
          }
#pragma unroll
          for (int a2 = 0; a2 < RAM; ++a2)
#pragma unroll
            for (int b = 0; b < RAM; ++b)
              if (a2 < r_a && b < r_a) {
                const EC hs = gsum<64>(rowk ? ccfma(va[a2], au[b], czero<EC>()) : czero<EC>());
                if (lane == 0) sHs[a2 * RAM + b] = hs;
              }
          lane_sync();
        }
        if (lane < P * P && ai <= aj) {
          EC acc2 = czero<EC>();
          for (int a2 = 0; a2 < r_a; ++a2) {
            EC t2 = czero<EC>();
            for (int b = 0; b < r_a; ++b) t2 = cfma(sHs[a2 * RAM + b], cconj(sUA[aj * RAM + b]), t2);
            acc2 = cfma(sUA[ai * RAM + a2], t2, acc2);
          }
          if (ai == aj) {
            sAr[ai] = float(acc2.x);
          } else {
            sAr[hoff<P>(ai, aj)] = float(acc2.x);
            sAr[hoff<P>(ai, aj) + 1] = float(acc2.y);
          }
        }
      };
      // Iteration k: the residual of (A, b) in FP64 (k > 0), the new b, and
      // the partial sums of R conj(b), through one barrier; then the stop rule
      // on every thread and EIG_{r_a} on wave 0.
      double eta_prev = INFINITY;
      for (int k = 0;; ++k) {
        const float ainv = xrcp(anorm2);
        double rr = 0.0;
        float wb[NDT], bb = 0.f;
#pragma unroll
        for (int t = 0; t < NDT; ++t) {
          if (t > 0 && wave * 64 + kWideThreads * t >= QQ) {   // uniform
            wb[t] = 0.f;
            continue;
          }
          float bn;
          if (k > 0) {
            const double bd = bv[t];
            double s = 0.0, rd = 0.0, ro = 0.0;
#pragma unroll
            for (int e = 0; e < P * P; ++e) {
              const double x = v[t][e], a = A[e];
              const double dlt = fma(e < P ? -a : -2.0 * a, bd, x);
              if (e < P) rd = fma(dlt, dlt, rd);
              else ro = fma(dlt, dlt, ro);
              s = fma(a, x, s);
            }
            rr = fma(double(wgt[t]), fma(0.5, ro, rd), rr);
            bn = float(s) * ainv;
          } else {
            float s = 0.f;
#pragma unroll
            for (int e = 0; e < P * P; ++e) s = fmaf(A[e], v[t][e], s);
            bn = s * ainv;
          }
          bv[t] = bn;
          wb[t] = wgt[t] * bn;
          bb = fmaf(wb[t], bn, bb);
        }
        publish(wb, bb, rr);
        if (k > 0) {
          const double e = sqrt(totald() / normR2);
          eta = float(e);
          const bool stop = iters >= prm.max_iter ||
                            (prm.eps > 0.0 && iters >= prm.min_iter && fabs(e - eta_prev) <= prm.eps);
          if (stop) break;
          eta_prev = e;
        }
        eig_a(k == 0 && !warm, k == 0);
        iters = k + 1;
        block_sync();   // publishes sA; red and redd are free again
        load_a();
      }
    }
    // U_A of this pixel (rows of the r_a = 1 power iterate, or the subspace)
    block_sync();
    if (tid == 0 && r_a == 1) {
#pragma unroll
      for (int i = 0; i < P; ++i) sUA[i * RAM] = ua[i];
    }
    chain = !bad;   // this S may seed the next pixel's
    ua_ok = !zero && !bad;
    block_sync();
    // ------------------------------------------ enqueue for the batched tail
#pragma unroll
    for (int t = 0; t < NDT; ++t) {
      const int e = tid + kWideThreads * t;
      if (e < QQ) reinterpret_cast<float*>(sHq)[nq * QQ + 2 * (e - comp[t] * (QQ / 2)) + comp[t]] = bv[t];
    }
    if (tid == 0) {
      sQidx[nq] = idx;
      sQflag[nq] = bad ? 2 : (zero ? 1 : 0);
      sQeta[nq] = eta;
      sQit[nq] = iters;
    }
    if (tid < P * RAM) sQUA[nq][tid] = (zero || bad) ? czero<EC>() : sUA[tid];
    block_sync();
    ++nq;
  };

  // one call site each for the pixel body and the tail
  for (int64_t itp = 0;; ++itp) {
    const bool more = itp < count;
    if (more) pixel(itp);
    if (nq == NQ || (!more && nq > 0)) {
      tail(nq);
      nq = 0;
    }
    if (!more) break;
  }
}

template <int P, int Q, int RBM, int MODE, int PREC, bool VAR = false>
__global__ __launch_bounds__(kWideThreads, 1) void kstap_wide_kernel(const KParams prm) {
  __shared__ __attribute__((aligned(16))) char lds[WideLds<P, Q, RBM, PREC>::bytes];
  int64_t first, count;
  if (MODE == kModeRun) {
    const int per = gridDim.x >> 3;
    const int logical = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (logical >= prm.nlogical) return;
    const int64_t total = tiled_positions(prm.H, prm.W);
    first = int64_t(logical) * prm.pix_per_block;
    count = total - first;
    if (count > prm.pix_per_block) count = prm.pix_per_block;
  } else {
    first = int64_t(blockIdx.x) * prm.pix_per_block;
    count = prm.npix - first;
    if (count > prm.pix_per_block) count = prm.pix_per_block;
  }
  run_pixels_wide<P, Q, RBM, MODE, PREC, VAR>(prm, first, count, lds);
}

// ---------------------------------------------------------------- launchers
template <int P, int Q, int RBM, int PREC>
int launch_one(int mode, const KParams& prm, hipStream_t stream) {
  int64_t units = (mode == kModeRun) ? int64_t(prm.nlogical) : (int64_t(prm.npix) + prm.pix_per_block - 1) / prm.pix_per_block;
  if (units <= 0) return hipSuccess;
  int64_t grid = (mode == kModeRun) ? ((units + 7) / 8) * 8 : units;
  if (grid > 0x7fffffff) return hipErrorInvalidValue;
  if (mode == kModeRun && has_variants(prm) && prm.nbank > 0)
    hipLaunchKernelGGL((kstap_kernel<P, Q, RBM, kModeRun, PREC, PREC == 0 ? kBank : kVariant>), dim3(unsigned(grid)),
                       dim3(64), 0, stream, prm);
  else if (mode == kModeRun && has_variants(prm))
    hipLaunchKernelGGL((kstap_kernel<P, Q, RBM, kModeRun, PREC, kVariant>), dim3(unsigned(grid)), dim3(64), 0, stream,
                       prm);
  else if (mode == kModeRun)
    hipLaunchKernelGGL((kstap_kernel<P, Q, RBM, kModeRun, PREC>), dim3(unsigned(grid)), dim3(64), 0, stream, prm);
  else
    hipLaunchKernelGGL((kstap_kernel<P, Q, RBM, kModeProbe, PREC>), dim3(unsigned(grid)), dim3(64), 0, stream, prm);
  return hipGetLastError();
}

template <int P, int Q, int RBM, int PREC>
int launch_wide(int mode, const KParams& prm, hipStream_t stream) {
  int64_t units = (mode == kModeRun) ? int64_t(prm.nlogical) : (int64_t(prm.npix) + prm.pix_per_block - 1) / prm.pix_per_block;
  if (units <= 0) return hipSuccess;
  int64_t grid = (mode == kModeRun) ? ((units + 7) / 8) * 8 : units;
  if (grid > 0x7fffffff) return hipErrorInvalidValue;
  if (mode == kModeRun && has_variants(prm))
    hipLaunchKernelGGL((kstap_wide_kernel<P, Q, RBM, kModeRun, PREC, true>), dim3(unsigned(grid)), dim3(kWideThreads), 0,
                       stream, prm);
  else if (mode == kModeRun)
    hipLaunchKernelGGL((kstap_wide_kernel<P, Q, RBM, kModeRun, PREC>), dim3(unsigned(grid)), dim3(kWideThreads), 0, stream,
                       prm);
  else
    hipLaunchKernelGGL((kstap_wide_kernel<P, Q, RBM, kModeProbe, PREC>), dim3(unsigned(grid)), dim3(kWideThreads), 0, stream,
                       prm);
  return hipGetLastError();
}

template <int P, int Q, int RBM, int PREC>
int launch_persist(const KParams* descs, const int32_t* order, const int64_t* prefix, int nt, int ppb,
                   unsigned long long* counter, int grid, hipStream_t stream) {
  hipLaunchKernelGGL((kstap_persistent<P, Q, RBM, PREC>), dim3(grid), dim3(64), 0, stream, descs, order, prefix, nt,
                     ppb, counter);
  return hipGetLastError();
}

}  // namespace
}  // namespace kstap
