// Narrow FP32 kernels of the Doppler bank (nbank > 0).
//
// A bank's bin map is the argmax of the statistic over M steerings, and on
// noise the two best bins of one pixel in about 5 10^5 lie within one part in
// 10^6 of each other, the size of any change of rounding: with the split
// covariance and the Hermitian sweeps of run_pixels, one bin of a 768 x 768
// frame with 16 bins came out as its neighbour in the tie, and the enhancement
// image with it.  So that the bins of a frame stay what they were, the bank
// keeps the arithmetic its results were first computed with: FP32 MFMA
// covariance and sweeps of LR-Kron over all of R in LDS (6.9 ms on that frame
// against 4.9 ms).  The batched tail, and with it the bank loop, is shared.
// This holds for the narrow FP32 classes (p q <= 64) alone: a bank in the other
// precisions or on the wide kernels shares the arithmetic of the plain statistic,
// and bins of theirs that tie within its rounding may move with it.
#pragma once

namespace kstap {
namespace {

// LDS carve-out, largest alignment first.
template <int P, int Q, int RBM>
struct BankLds {
  using EC = float2;
  static constexpr int PQ = P * Q;
  static constexpr int RAM = (P < kMaxRA) ? P : kMaxRA;
  static constexpr int G = Groups<Q>::G;
  static constexpr int NB = (PQ + 15) / 16;
  // B / tail / transpose scratch: the raw time factor B (q x q), the batched
  // tail's basis exchange, and the FP32 path's diagonal-tile transpose
  static constexpr size_t kB = sizeof(float2) * Q * Q;
  static constexpr size_t kT = sizeof(EC) * RBM * Q * G;
  static constexpr size_t kP = sizeof(float) * NB * 256;
  static constexpr size_t kBT = kB > kT ? (kB > kP ? kB : kP) : (kT > kP ? kT : kP);
  static constexpr size_t oUA = 0;                                        // EC[P*RAM]
  static constexpr size_t oAh = oUA + sizeof(EC) * P * RAM;               // EC[P*P]
  static constexpr size_t oQUA = oAh + sizeof(EC) * P * P;                // EC[G][P*RAM]
  static constexpr size_t oBT = oQUA + sizeof(EC) * G * P * RAM;          // kBT bytes
  static constexpr size_t oS = (oBT + kBT + 15) / 16 * 16;                // float2[P(P+1)/2][Q][Q+1]
  static constexpr size_t oA = oS + sizeof(float2) * (P * (P + 1) / 2) * Q * (Q + 1);   // float2[P*P]
  static constexpr size_t oQidx = oA + sizeof(float2) * P * P;            // int64[G]
  static constexpr size_t oOff = oQidx + sizeof(int64_t) * G;             // uint32[kMaxN + kOffPad]
  static constexpr size_t oDelta = oOff + sizeof(uint32_t) * (kMaxN + kOffPad);   // uint32[3][2][kMaxDelta + 8]
  static constexpr size_t oQflag = oDelta + sizeof(uint32_t) * 6 * (kMaxDelta + 8);   // int[G]
  static constexpr size_t bytes = ((oQflag + sizeof(int) * G) + 15) / 16 * 16;
};

// The whole per-pixel pass of run mode for `count` positions starting at
// `first` of the tiled order.  One 64-lane workgroup; `lds` holds
// BankLds<...>::bytes.
template <int P, int Q, int RBM>
__device__ __forceinline__ void run_pixels_bank(const KParams& prm, int64_t first, int64_t count, char* lds) {
  using EC = float2;
  using ES = decltype(EC{}.x);
  using L = BankLds<P, Q, RBM>;
  constexpr int PQ = P * Q;
  constexpr int NB = (PQ + 15) / 16;        // 16-row blocks of the pq x pq covariance
  constexpr int QQ = Q * Q;
  constexpr int NE = (QQ + 63) / 64;        // q x q entries per lane
  constexpr int RAM = L::RAM;
  constexpr int QP = Groups<Q>::QP;         // lanes per pixel in the batched tail
  constexpr int G = Groups<Q>::G;           // pixels per batched tail

  float2* const sS = reinterpret_cast<float2*>(lds + L::oS);     // S, upper blocks
  float2* const sBT = reinterpret_cast<float2*>(lds + L::oBT);   // raw B, then tail scratch
  uint32_t* const sOffB = reinterpret_cast<uint32_t*>(lds + L::oOff);
  // sliding window: per move, the entering then the leaving vectors
  uint32_t* const sDelta = reinterpret_cast<uint32_t*>(lds + L::oDelta);
  constexpr int KD = kMaxDelta + 8;
  float2* const sA = reinterpret_cast<float2*>(lds + L::oA);
  EC* const sUA = reinterpret_cast<EC*>(lds + L::oUA);
  EC* const sAh = reinterpret_cast<EC*>(lds + L::oAh);
  EC (*const sQUA)[P * RAM] = reinterpret_cast<EC (*)[P * RAM]>(lds + L::oQUA);   // queued pixels: U_A
  EC* const tail_scratch = reinterpret_cast<EC*>(sBT);
  int64_t* const sQidx = reinterpret_cast<int64_t*>(lds + L::oQidx);             //   pixel index
  int* const sQflag = reinterpret_cast<int*>(lds + L::oQflag);                   //   0 ok, 1 zero, 2 non-finite

  const int lane = threadIdx.x;
  const int n = prm.n;
  const int H = prm.H, W = prm.W;
  const int r_a = prm.r_a, r_b = prm.r_b;

  // byte offset of each stencil entry from the window origin (kOut past n);
  // samples are complex64 (8 bytes) or, on the mixed path, BF16 pairs (4)
  constexpr int kSample = 8;
  wave_sync();
  for (int m = lane; m < kMaxN + kOffPad; m += 64)
    sOffB[m] = (m < n) ? uint32_t(((int(prm.st[2 * m]) * W + int(prm.st[2 * m + 1])) * Q - prm.st_min) * kSample)
                       : kOut;
  for (int m = lane; m < 6 * KD; m += 64) {
    const int t = m / KD, e = m - t * KD, mv = t >> 1;
    const int cnt = (t & 1) ? prm.nrem[mv] : prm.nadd[mv];
    uint32_t off = kOut;
    if (e < cnt) {   // cnt <= kMaxDelta
      const int dr = (t & 1) ? prm.drem[mv][2 * e] : prm.dadd[mv][2 * e];
      const int dc = (t & 1) ? prm.drem[mv][2 * e + 1] : prm.dadd[mv][2 * e + 1];
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

  // queue of pixels waiting for the batched tail: lane (g, k) holds row k of
  // the Hermitian time factor of queued pixel g
  const int tg = lane / QP, tk = lane % QP;
  float2 Bq[Q];
#pragma unroll
  for (int l = 0; l < Q; ++l) Bq[l] = cz();
  int nq = 0;

  // ------------------------------------------------ a6 + a8 for G pixels
  // FP32 run mode: the queue holds the pixels of one sliding-window chain at
  // a time, and every batch of a chain but its first starts each slot from
  // the converged time-factor subspace of the previous batch's slot G-1-g,
  // its nearest pixel in the snake order of a unit (directly above it for
  // q = 16).  Like the sliding window, the choice depends only on the chain,
  // so the results are the same for every decomposition of the frame.
  EC vbw[RBM];   // lane (g, k): row k of the basis that starts slot g
#pragma unroll
  for (int c = 0; c < RBM; ++c) vbw[c] = czero<EC>();
  bool vbw_ok = false;
  int64_t qchain = -1, bchain = -2;   // chain of the queued pixels, of the last batch
  auto tail = [&](int nfill) __attribute__((always_inline)) {
    const bool keep = bchain == qchain && vbw_ok;
    bool ok;
    tail_batch<P, Q, RBM, EC, false>(prm, Bq, tg, nfill, sQflag, sQidx, sQUA, tail_scratch, 2e-6, vbw, keep, ok);
    bchain = qchain;
    const int src = (G - 1 - tg) * QP + tk;
#pragma unroll
    for (int c = 0; c < RBM; ++c) {
      vbw[c].x = __shfl(vbw[c].x, src);
      vbw[c].y = __shfl(vbw[c].y, src);
    }
    vbw_ok = __shfl(int(ok), src) != 0;
  };

  // Sliding window (run mode, FP32 path): every position of a chain but the
  // first is a one-pixel move from the one before it (tiled_move); such a
  // pixel updates the previous pixel's S when this workgroup has just
  // computed it from finite data.  A chain's first pixel takes the full sum,
  // and runs start on a chain, so the choice is the same for every
  // decomposition.
  bool chain = false;
  bool ua_ok = false;   // sUA holds the U_A of the pixel processed last
  for (int64_t it = 0; it < count; ++it) {
    int64_t idx;
    int r, c;
    const bool left_ok = chain;
    chain = false;
    if (!tiled_pixel(first + it, H, W, &r, &c)) continue;
    idx = int64_t(r) * W + c;
    const bool valid = r >= prm.r0 && r < prm.r1 && c >= prm.c0 && c < prm.c1;
    if (!valid) {
      if (lane == 0) write_outside(prm, idx);
      continue;
    }
    // window origin as a sample index (x and the split planes share the layout)
    const int64_t win = (int64_t(r) * W + c) * Q + prm.st_min;

    // ---------------------------------------------------------------- a2 SCM
    const int mv = tiled_move(first + it, H, W, kChainNarrow);
    const bool slide = left_ok && mv >= 0 && prm.nadd[0] >= 0;
    // q a multiple of 16: the block sums and ||S||^2 of a4 are gathered while
    // S is stored
    constexpr bool kSums = Q % 16 == 0;
    SSums<P> ss;
#pragma unroll
    for (int e = 0; e < P * P; ++e) ss.a0[e] = cz();
    ss.nr = 0.f;
    if (slide)
      scm_fp32_delta<P, Q>(prm.x + win, plane, prm.rec_bytes, sDelta + 2 * mv * KD, prm.nadd[mv],
                           sDelta + (2 * mv + 1) * KD, prm.nrem[mv], loff, n, sS, ss);
    else
      scm_fp32<P, Q>(prm.x + win, plane, prm.rec_bytes, sOffB, loff, n, sS, reinterpret_cast<float*>(sBT), ss);

    // ------------------------------------------------ a4 init, ||R||_F = ||S||_F
    float2 A[P * P];
    double normR2;
    {
      float2 a0[P * P];
      if constexpr (kSums) {
        normR2 = wsumd(double(ss.nr));
        // the upper block sums in one multi-value reduction
        constexpr int NU = P * (P + 1) / 2, NS = (2 * NU + 3) / 4 * 4;
        float sums[NS];
        {
          int e = 0;
#pragma unroll
          for (int i = 0; i < P; ++i)
#pragma unroll
            for (int j = i; j < P; ++j, e += 2) {
              sums[e] = ss.a0[i * P + j].x;
              sums[e + 1] = ss.a0[i * P + j].y;
            }
#pragma unroll
          for (int f = 2 * NU; f < NS; ++f) sums[f] = 0.f;
        }
        wsum_n<NS>(sums);
        {
          int e = 0;
#pragma unroll
          for (int i = 0; i < P; ++i)
#pragma unroll
            for (int j = i; j < P; ++j, e += 2) {
              a0[i * P + j] = cscale(make_float2(sums[e], sums[e + 1]), 1.f / float(QQ));
              if (j > i) a0[j * P + i] = cconj(a0[i * P + j]);
            }
        }
      } else {
#pragma unroll
        for (int e = 0; e < P * P; ++e) a0[e] = cz();
        float nr = 0.f;
#pragma unroll
        for (int t = 0; t < NE; ++t) {
          const int e = lane + 64 * t;
          if (e < QQ) {
            const int k = e / Q, l = e - (e / Q) * Q;
#pragma unroll
            for (int i = 0; i < P; ++i)
#pragma unroll
              for (int j = 0; j < P; ++j) {
                const float2 s = sget<P, Q>(sS, i, j, k, l);
                a0[i * P + j] = cadd(a0[i * P + j], s);
                nr += cabs2(s);
              }
          }
        }
        normR2 = wsumd(double(nr));
        constexpr int NS = (2 * P * P + 3) / 4 * 4;
        float sums[NS];
#pragma unroll
        for (int f = 0; f < NS; ++f) sums[f] = (f < 2 * P * P) ? ((f & 1) ? a0[f / 2].y : a0[f / 2].x) : 0.f;
        wsum_n<NS>(sums);
#pragma unroll
        for (int e = 0; e < P * P; ++e) a0[e] = cscale(make_float2(sums[2 * e], sums[2 * e + 1]), 1.f / float(QQ));
      }
      float an = 0.f;
#pragma unroll
      for (int e = 0; e < P * P; ++e) {
        A[e] = a0[e];
        an += cabs2(a0[e]);
      }
      if (double(an) <= 1e-24 * normR2) {   // fallback: partial trace R vec(I_q) (uniform branch)
        float2 pt[P * P];
#pragma unroll
        for (int e = 0; e < P * P; ++e) pt[e] = cz();
#pragma unroll
        for (int t = 0; t < NE; ++t) {
          const int e = lane + 64 * t;
          if (e < QQ && e / Q == e - (e / Q) * Q) {
#pragma unroll
            for (int i = 0; i < P; ++i)
#pragma unroll
              for (int j = 0; j < P; ++j) pt[i * P + j] = cadd(pt[i * P + j], sget<P, Q>(sS, i, j, e / Q, e / Q));
          }
        }
#pragma unroll
        for (int e = 0; e < P * P; ++e) A[e] = wsum(pt[e]);
      }
    }

    int iters = 0;
    const bool zero = !(normR2 > 0.0);
    const bool bad = !isfinite(normR2);
    chain = !bad;   // this S may seed the next pixel's
    float2 bv[NE];
#pragma unroll
    for (int t = 0; t < NE; ++t) bv[t] = cz();

    if (!zero && !bad) {
      // --------------------------------------------------------- a5 LR-Kron
      float2 Ap[P * P];
      float bn2;
      double resid = 0.0;
      float anorm2 = 0.f;
#pragma unroll
      for (int e = 0; e < P * P; ++e) anorm2 += cabs2(A[e]);

      // one sweep over S: residual of (A, bv) if RES, then the new b and the
      // partial sums of R conj(b)
      auto sweep = [&](bool res) __attribute__((always_inline)) {
        const float ainv = xrcp(anorm2);
        float2 ap[P * P];
#pragma unroll
        for (int e = 0; e < P * P; ++e) ap[e] = cz();
        float bb = 0.f;
        double rr = 0.0;
#pragma unroll
        for (int t = 0; t < NE; ++t) {
          const int e = lane + 64 * t;
          if (QQ % 64 == 0 || e < QQ) {
            const int k = e / Q, l = e - (e / Q) * Q;
            float2 s[P * P];
#pragma unroll
            for (int i = 0; i < P; ++i)
#pragma unroll
              for (int j = 0; j < P; ++j) s[i * P + j] = sget<P, Q>(sS, i, j, k, l);
            if (res) {
              float acc = 0.f;
#pragma unroll
              for (int ij = 0; ij < P * P; ++ij) acc += cabs2(csub(s[ij], cmul(A[ij], bv[t])));
              rr += double(acc);
            }
            float2 bn = cz();
#pragma unroll
            for (int ij = 0; ij < P * P; ++ij) bn = ccfma(A[ij], s[ij], bn);
            bn = cscale(bn, ainv);
            bv[t] = bn;
            bb += cabs2(bn);
#pragma unroll
            for (int ij = 0; ij < P * P; ++ij) ap[ij] = ccfma(bn, s[ij], ap[ij]);
          } else {
            bv[t] = cz();
          }
        }
        // the 2 p^2 sums of R conj(b) and ||b||^2 in one multi-value reduction
        constexpr int NS = (2 * P * P + 1 + 3) / 4 * 4;
        float sums[NS];
#pragma unroll
        for (int ij = 0; ij < P * P; ++ij) {
          sums[2 * ij] = ap[ij].x;
          sums[2 * ij + 1] = ap[ij].y;
        }
#pragma unroll
        for (int e = 2 * P * P; e < NS; ++e) sums[e] = (e == 2 * P * P) ? bb : 0.f;
        wsum_n<NS>(sums);
        bn2 = sums[2 * P * P];
        const float binv = xrcp(bn2);
#pragma unroll
        for (int ij = 0; ij < P * P; ++ij) Ap[ij] = cscale(make_float2(sums[2 * ij], sums[2 * ij + 1]), binv);
        if (res) resid = wsumd(rr);
      };

      // EIG_{r_a}: A <- U (U^H A' U) U^H with U the top-r_a subspace of Herm(A').
      // A pixel that slides from its predecessor starts from that pixel's
      // U_A (sUA): the two training sets differ in a few vectors.  The choice
      // depends only on the chain position, as the sliding window does.
      const bool warm = slide && ua_ok;
      EC ua[P];
#pragma unroll
      for (int i = 0; i < P; ++i) ua[i] = warm ? sUA[i * RAM] : czero<EC>();
      auto eig_a = [&](bool cold, bool first) __attribute__((always_inline)) {
        EC Ah[P * P];
#pragma unroll
        for (int i = 0; i < P; ++i)
#pragma unroll
          for (int j = 0; j < P; ++j)
            Ah[i * P + j] = cscale(cadd(cto<EC>(Ap[i * P + j]), cconj(cto<EC>(Ap[j * P + i]))), ES(0.5));
        if (r_a == 1) {
          // The check of a start that power_top_h makes at its first step comes
          // after the solve here, which leaves the rounding of every step, and
          // with it the bins, as it was.
          const auto Af = [&](int i, int j) { return Ah[i * P + j]; };
          ES lam;
          for (bool again = false;; again = true) {
            power_top<P, EC>(Af, ua, cold && !again, 500, 2e-6);
            ES tr = 0;
            EC s[P];
            lam = 0;
#pragma unroll
            for (int i = 0; i < P; ++i) {
              s[i] = czero<EC>();
#pragma unroll
              for (int j = 0; j < P; ++j) s[i] = cfma(Ah[i * P + j], ua[j], s[i]);
              lam += ua[i].x * s[i].x + ua[i].y * s[i].y;
              tr += Ah[i * P + i].x;
            }
            if (again || stands_out(lam, tr)) break;
            const ES inv = xrsqrt(xmax(start_anew<P, EC, ES>(Af, s, lam, tr, cold, first), tiny<ES>()));
#pragma unroll
            for (int i = 0; i < P; ++i) ua[i] = cscale(s[i], inv);
          }
          anorm2 = 0.f;
#pragma unroll
          for (int i = 0; i < P; ++i)
#pragma unroll
            for (int j = 0; j < P; ++j) {
              A[i * P + j] = tof(cscale(cmul(ua[i], cconj(ua[j])), lam));
              anorm2 += cabs2(A[i * P + j]);
            }
          // one lane writes U_A with static indices (a lane-indexed select
          // over ua[] is compiled into a scratch array)
          if (lane == 0) {
#pragma unroll
            for (int i = 0; i < P; ++i) sUA[i * RAM] = ua[i];
          }
          wave_sync();
          return;
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
                                       2e-6, first ? 0.f : kMixOwn);
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
          group_subspace<RAM, 64, P, EC>(mrow, lane < P, r_a, va, sAh, cold, 500, 2e-6, false, !cold, first ? 0.f : kMixOwn);
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
        anorm2 = 0.f;
#pragma unroll
        for (int i = 0; i < P; ++i)
#pragma unroll
          for (int j = 0; j < P; ++j) {
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
            A[i * P + j] = tof(sacc);
            anorm2 += cabs2(A[i * P + j]);
          }
        wave_sync();
      };

      sweep(false);
      eig_a(!warm, true);
      iters = 1;
      double eta_prev = INFINITY;
      while (true) {
        sweep(true);
        const double e = sqrt(resid / normR2);
        const bool stop = iters >= prm.max_iter ||
                          (prm.eps > 0.0 && iters >= prm.min_iter && fabs(e - eta_prev) <= prm.eps);
        if (stop) break;
        eta_prev = e;
        eig_a(false, false);
        ++iters;
      }
      // bv now holds the final b = R^T conj(a) / ||a||^2
    }
    ua_ok = !zero && !bad;

    // ------------------------------------------ enqueue for the batched tail
    // A full queue, or (warm tail) one that holds another chain's pixels,
    // runs its batch here, before this pixel joins: the queued pixels wait in
    // Bq and their own LDS slots, which this pixel's work does not touch, and
    // the tail is inlined at one place in the loop.
    wave_sync();   // S is dead from here on
    {
      bool flush = nq == G;
      const int64_t cid = (first + it) / kChainNarrow;
      flush = flush || (nq > 0 && cid != qchain);
      if (flush) {
        tail(nq);
        nq = 0;
      }
      qchain = cid;
    }
#pragma unroll
    for (int t = 0; t < NE; ++t) {
      const int e = lane + 64 * t;
      if (QQ % 64 == 0 || e < QQ) sBT[e] = bv[t];   // B[k][l] at k*q + l
    }
    wave_sync();
    if (tg == nq && tk < Q) {
#pragma unroll
      for (int l = 0; l < Q; ++l) Bq[l] = cscale(cadd(sBT[tk * Q + l], cconj(sBT[l * Q + tk])), 0.5f);
    }
    if (lane == 0) {
      sQidx[nq] = idx;
      sQflag[nq] = bad ? 2 : (zero ? 1 : 0);
    }
    if (lane < P * RAM) sQUA[nq][lane] = (zero || bad) ? czero<EC>() : sUA[lane];
    wave_sync();
    ++nq;
  }
  if (nq > 0) tail(nq);
}


}  // namespace
}  // namespace kstap
