// a6 + a8 of the plain statistic, batched: top-r_b time
// subspace, projected test vector and statistic of up to 64 / QP queued pixels
// of one wavefront (the statistic variants take tail_batch, which has the
// Doppler bank, the filters and the passes).
//
// Bound by VALU issue, a third of it lane-group reductions.  Against
// tail_batch, whose loops run to a run-time rank and mask absent rows at every
// step:
//   * R is the plan's r_b as a constant (the caller switches on it once per
//     batch), so the loops over columns have no branches;
//   * absent rows (lanes past q, empty or flagged slots) are rows of zeros in
//     the matrix and the basis, and everything computed from them is zero, so
//     nothing is masked;
//   * V^H M V is Hermitian: the residual takes R (R + 1) / 2 lane-group dot
//     products instead of R^2;
//   * the basis exchange through LDS keeps a row's columns together, so two
//     columns come in one 16-byte read.
// With the queued factors in LDS (kQueueLds) no class of the headline shapes
// spills.  Measured, tail_batch and a register queue against this:
// 2048 x 2048, p = 3, q = 16, n = 200 27.5 -> 22.6 ms; FP32 with FP64 solves
// 512 x 512 5.08 -> 4.03 ms; split BF16 1024 x 1024 13.1 -> 11.9 ms;
// 187 x 233, q = 12, r_b = 6 509 -> 390 us; 64 x 64, q = 8, r_b = 3 109 -> 91 us.
#pragma once

namespace kstap {
namespace {

// c - a b
__device__ __forceinline__ float2 cfms(float2 a, float2 b, float2 c) {
  return make_float2(fmaf(-a.x, b.x, fmaf(a.y, b.y, c.x)), fmaf(-a.x, b.y, fmaf(-a.y, b.x, c.y)));
}
__device__ __forceinline__ double2 cfms(double2 a, double2 b, double2 c) {
  return make_double2(fma(-a.x, b.x, fma(a.y, b.y, c.x)), fma(-a.x, b.y, fma(-a.y, b.x, c.y)));
}
// conj(a) b
template <typename C>
__device__ __forceinline__ C ccmul(C a, C b) {
  C r;
  r.x = a.x * b.x + a.y * b.y;
  r.y = a.x * b.y - a.y * b.x;
  return r;
}

// orth_cgs2 for rows that are zero where absent.
template <int R, int QP, typename C>
__device__ __forceinline__ void orth_rows(C (&w)[R]) {
  using S = decltype(C{}.x);
#pragma unroll
  for (int c = 0; c < R; ++c) {
#pragma unroll
    for (int pass = 0; pass < 2; ++pass) {
      C h[R];   // every projection of a pass uses the column as it entered it
#pragma unroll
      for (int a = 0; a < c; ++a) h[a] = ccmul(w[a], w[c]);
#pragma unroll
      for (int a = 0; a < c; ++a) h[a] = gsum<QP>(h[a]);
#pragma unroll
      for (int a = 0; a < c; ++a) w[c] = cfms(w[a], h[a], w[c]);
    }
    const S inv = xrsqrt(xmax(gsum<QP>(cabs2(w[c])), tiny<S>()));
    w[c] = cscale(w[c], inv);
  }
}

// Bytes of the basis exchange of a wavefront: per group D rows of R columns,
// padded by one 16-byte access so that the groups' reads fall on other banks.
template <int R, int D, int G, typename C>
constexpr size_t tail_scratch_bytes = size_t(G) * (sizeof(C) * R * D + 16);

// group_subspace for exactly R columns and zero rows: the top-R invariant
// subspace of one Hermitian D x D matrix per lane group.  v enters as the
// start block (tested at the first step if `tested`) and leaves as the basis;
// `guard` where it is another matrix's (guard_start, with `mix`).  Same iteration,
// stopping rule and freezing.
template <int R, int QP, int D, typename C, bool WAVE_LOCAL>
__device__ __forceinline__ void rows_subspace(const float2 (&mrow)[D], int g, int k, C (&v)[R], char* scratch,
                                              int max_steps, double tol, bool tested, bool guard, float mix) {
  using S = decltype(C{}.x);
  C* const sV = reinterpret_cast<C*>(scratch + g * (sizeof(C) * R * D + 16));
  bool done = false;
  for (int step = 0; step < max_steps; ++step) {
    if (k < D) {
#pragma unroll
      for (int c = 0; c < R; ++c) sV[k * R + c] = v[c];
    }
    lds_sync<WAVE_LOCAL>();
    C w[R];
#pragma unroll
    for (int c = 0; c < R; ++c) w[c] = czero<C>();
    // rows of the basis come two at a time (one for wide or FP64 bases), the
    // next ones in flight while the current ones are used; without the
    // scheduling barriers all D rows are loaded at once and spill
    constexpr int GR = (sizeof(C) * R <= 32 && D % 2 == 0) ? 2 : 1, NG = D / GR;
    static_assert(D % GR == 0, "rows in groups");
    C buf[2][GR][R];
    auto load = [&](int gi, C (&to)[GR][R]) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < GR; ++e)
#pragma unroll
        for (int c = 0; c < R; ++c) to[e][c] = sV[(gi * GR + e) * R + c];
    };
    load(0, buf[0]);
#pragma unroll
    for (int gi = 0; gi < NG; ++gi) {
      if (gi + 1 < NG) load(gi + 1, buf[(gi + 1) & 1]);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int e = 0; e < GR; ++e) {
        float2 m = mrow[gi * GR + e];
        // the widening of the matrix row stays inside the loop (an empty asm
        // makes the value opaque), so it is not hoisted into extra registers
        if constexpr (sizeof(S) == 8) asm volatile("" : "+v"(m.x), "+v"(m.y));
        const C mc = cto<C>(m);
#pragma unroll
        for (int c = 0; c < R; ++c) w[c] = cfma(mc, buf[gi & 1][e][c], w[c]);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // keeps the products here: the compiler otherwise sinks all but the first
    // column's past the test below, and holds (spills) all rows until then
#pragma unroll
    for (int c = 0; c < R; ++c) asm volatile("" : "+v"(w[c].x), "+v"(w[c].y));
    lds_sync<WAVE_LOCAL>();
    bool conv = false;
    if (tested) {
      // residual W - V (V^H W), V^H W Hermitian: one row of it at a time
      C rr[R];
      S rn = 0, wn = 0;
#pragma unroll
      for (int b = 0; b < R; ++b) {
        rr[b] = w[b];
        wn += cabs2(w[b]);
      }
#pragma unroll
      for (int a = 0; a < R; ++a) {
        S hd = v[a].x * w[a].x + v[a].y * w[a].y;
        C h[R];
#pragma unroll
        for (int b = a + 1; b < R; ++b) h[b] = ccmul(v[a], w[b]);
        hd = gsum<QP>(hd);
#pragma unroll
        for (int b = a + 1; b < R; ++b) h[b] = gsum<QP>(h[b]);
        rr[a].x -= v[a].x * hd;
        rr[a].y -= v[a].y * hd;
#pragma unroll
        for (int b = a + 1; b < R; ++b) {
          rr[b] = cfms(v[a], h[b], rr[b]);
          rr[a] = cfms(v[b], cconj(h[b]), rr[a]);
        }
      }
#pragma unroll
      for (int b = 0; b < R; ++b) rn += cabs2(rr[b]);
      rn = gsum<QP>(rn);
      wn = gsum<QP>(wn);
      conv = rn <= S(tol * tol) * wn;
    }
    if (step == 0 && __ballot(guard)) conv = !guard_start<R, QP, D, C>(mrow, v, w, R, k, k < D, guard, mix) && conv;
    orth_rows<R, QP, C>(w);
    // a group keeps the first basis computed from a converged one and is
    // frozen from then on, so its result does not depend on its neighbours
    if (!done) {
#pragma unroll
      for (int c = 0; c < R; ++c) v[c] = w[c];
    }
    done = done || conv;
    tested = true;
    if (__ballot(!done) == 0) break;
  }
}

// The batched tail for r_b = R.  Arguments as tail_batch: lane group g of this
// wavefront serves queue slot slot0 + g, whose lane k holds row k of the pixel's Hermitian
// time factor in Bq (cleared here in empty and flagged slots); vb: this lane's
// row of its slot's basis, on entry the start of the slots whose lanes set
// `keep`, on return the basis.
template <int P, int Q, int RBM, int R, int MODE, typename EC, bool WAVE_LOCAL>
__device__ __forceinline__ void tail_rows(const KParams& prm, float2 (&Bq)[Q], int slot0, int nfill, const int* sQflag,
                                          const int64_t* sQidx, const float* sQeta, const int* sQit,
                                          const EC (*sQUA)[P * ((P < kMaxRA) ? P : kMaxRA)], char* scratch, double tol,
                                          EC (&vb)[RBM], bool keep, bool& vb_ok) {
  using ES = decltype(EC{}.x);
  constexpr int RAM = (P < kMaxRA) ? P : kMaxRA;
  constexpr int QP = Groups<Q>::QP;
  constexpr int RR = R > 0 ? R : 1;
  // opaque lane and slot: the tail's per-lane addresses, start block and
  // steering entries are formed here, once per batch, instead of being hoisted
  // out of the pixel loop, where they would be spilled (187 x 233, q = 12,
  // r_b = 6 takes 966 us with them hoisted)
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const int tk = lane % QP, slot = slot0 + lane / QP;
  const int H = prm.H, W = prm.W;
  const int r_a = prm.r_a;
  const bool slot_ok = slot < nfill;
  const int flag = slot_ok ? sQflag[slot] : 1;
  const int64_t pidx = slot_ok ? sQidx[slot] : 0;
  const bool use = flag == 0 && tk < Q;
  vb_ok = use;
  EC v[RR];
  if constexpr (R > 0) {
    if (__ballot(!use)) {
#pragma unroll
      for (int l = 0; l < Q; ++l) Bq[l] = use ? Bq[l] : cz();
    }
    keep = keep && use;
#pragma unroll
    for (int c = 0; c < R; ++c) v[c] = vb[c];
    if (__ballot(!keep)) {
#pragma unroll
      for (int c = 0; c < R; ++c)
        if (!keep) v[c] = use ? cto<EC>(omega(tk, c)) : czero<EC>();
    }
    // FP64 solves iterate until converged where the r_b-th and next eigenvalues
    // of B lie close together (a ratio of 0.99 takes ~1 500 steps to 1e-10);
    // the loop exits on the step cap, so a group never runs unbounded
    rows_subspace<R, QP, Q, EC, WAVE_LOCAL>(Bq, lane / QP, tk, v, scratch, sizeof(ES) == 8 ? 4000 : 200, tol, false,
                                            keep, kMixNeighbour);
#pragma unroll
    for (int c = 0; c < R; ++c) vb[c] = v[c];
  }
  // this lane's sample of every channel of the test snapshot
  int pr, pc;
  if (MODE == kModeRun) {
    pr = int(pidx / W);
    pc = int(pidx - int64_t(pr) * W);
  } else {
    pr = prm.pix[2 * pidx];
    pc = prm.pix[2 * pidx + 1];
  }
  const float2* xt = prm.x + (int64_t(pr) * W + pc) * Q + (tk < Q ? tk : 0);
  EC xv[P];
#pragma unroll
  for (int i = 0; i < P; ++i) xv[i] = use ? cto<EC>(xt[int64_t(i) * H * W * Q]) : czero<EC>();
  const EC* Uq = sQUA[slot_ok ? slot : 0];   // U_A of the queued pixel, p x RAM
  // z <- (I - U_A U_A^H) z
  auto project_a = [&](EC (&z)[P]) __attribute__((always_inline)) {
#pragma unroll 1
    for (int c = 0; c < r_a; ++c) {
      EC cw = czero<EC>();
#pragma unroll
      for (int i = 0; i < P; ++i) cw = ccfma(Uq[i * RAM + c], z[i], cw);
#pragma unroll
      for (int i = 0; i < P; ++i) z[i] = cfms(Uq[i * RAM + c], cw, z[i]);
    }
  };
  // g = F_B b_s
  const EC bsk = use ? cto<EC>(prm.b_s[tk < Q ? tk : 0]) : czero<EC>();
  EC gk = bsk;
  if constexpr (R > 0) {
    EC coef[R];
#pragma unroll
    for (int c = 0; c < R; ++c) coef[c] = ccmul(v[c], bsk);
#pragma unroll
    for (int c = 0; c < R; ++c) coef[c] = gsum<QP>(coef[c]);
#pragma unroll
    for (int c = 0; c < R; ++c) gk = cfms(v[c], coef[c], gk);
  }
  // z = F_A X conj(g), den = b^H F_B b
  EC z[P];
#pragma unroll
  for (int i = 0; i < P; ++i) z[i] = ccmul(gk, xv[i]);
  ES den = bsk.x * gk.x + bsk.y * gk.y;
#pragma unroll
  for (int i = 0; i < P; ++i) z[i] = gsum<QP>(z[i]);
  den = gsum<QP>(den);
  project_a(z);
  const bool den_ok = den > ES(1e-12) * ES(prm.bs_norm2);
  // Kron-STAP, Eq. (25): ||F_A X conj(F_B b)||^2 / (b^H F_B b), or its value
  // for one spatial steering h
  ES t;
  if (prm.stat_mode == 0) {
    ES num = 0;
#pragma unroll
    for (int i = 0; i < P; ++i) num += cabs2(z[i]);
    t = den_ok ? num / den : ES(0);
  } else {
    EC hs[P], fh[P], hz = czero<EC>();
    ES hfa = 0;   // ||F_A h||^2
#pragma unroll
    for (int i = 0; i < P; ++i) fh[i] = hs[i] = cto<EC>(prm.h_s[i]);
    project_a(fh);
#pragma unroll
    for (int i = 0; i < P; ++i) {
      hfa += hs[i].x * fh[i].x + hs[i].y * fh[i].y;
      hz = ccfma(hs[i], z[i], hz);
    }
    const bool ok = den_ok && hfa > ES(1e-12) * ES(prm.h_norm2);
    t = ok ? cabs2(hz) / (hfa * den) : ES(0);
  }
  float T = float(t);
  if (!isfinite(T) || flag == 2) T = NAN;
  if (flag == 1) T = 0.f;
  if (slot_ok && tk == 0) {
    prm.T[pidx] = T;
    if (MODE == kModeRun && prm.D) prm.D[pidx] = (T > prm.tau) ? 1 : 0;
    if (MODE == kModeProbe) {
      if (prm.eta) prm.eta[pidx] = sQeta[slot];
      if (prm.iters) prm.iters[pidx] = sQit[slot];
    }
  }
  if (MODE == kModeProbe && slot_ok) {
    if (prm.UA && tk < P) {
#pragma unroll
      for (int c = 0; c < RAM; ++c)
        if (c < r_a) prm.UA[(pidx * P + tk) * r_a + c] = (flag != 0) ? cz() : tof(sQUA[slot][tk * RAM + c]);
    }
    if (R > 0 && prm.UB && tk < Q) {
#pragma unroll
      for (int c = 0; c < R; ++c) prm.UB[(pidx * Q + tk) * R + c] = (flag != 0) ? cz() : tof(v[c]);
    }
  }
  lds_sync<WAVE_LOCAL>();
}

// f(Int<r_b>()): r_b as a constant (r_b > 4 takes the RBM = 8 classes).
template <int RBM, typename F>
__device__ __forceinline__ void with_rank(int r_b, F f) {
  if constexpr (RBM == 4) {
    if (r_b == 4) f(Int<4>());
    else if (r_b == 3) f(Int<3>());
    else if (r_b == 2) f(Int<2>());
    else if (r_b == 1) f(Int<1>());
    else f(Int<0>());
  } else {
    if (r_b == 8) f(Int<8>());
    else if (r_b == 7) f(Int<7>());
    else if (r_b == 6) f(Int<6>());
    else f(Int<5>());
  }
}

}  // namespace
}  // namespace kstap
