// The P1 / P2 / Lambda update as device code: a kernel of its own (dense.hip) and the last
// workgroups of the sweep's launch (sweep.hip).
#pragma once
#include "nlpr_internal.h"

namespace nlpr {
namespace {

// Work item = 256 pixels.  A pixel has NC threads (1, or 4 when the launch covers few pixels in
// all, so that it still fills the GPU), each owning a contiguous share of the bands; with 4 a
// workgroup takes a quarter of the item's pixels, one wave per share, so that the exchange of
// the shares holds up four waves instead of sixteen.
// With E = I:
//   P1 = (rho BX + Y_l - rho Lambda1) / (1 + rho)  on sampled pixels (S^T S = 1)
//   P1 = BX - Lambda1                              elsewhere            (eq. (Qh_update))
//   P2 = (X - Lambda2 + lambda1/rho Y_h R^T) F,  F = (I + lambda1/rho R R^T)^{-1}
//                                                                       (eq. (Qm_update))
// P2 is evaluated as  P2 = A0 + (Y_h - A0 R) G R^T  with A0 = X - Lambda2 and
// G = (rho/lambda1 I + R^T R)^{-1}: Woodbury gives F = I - R G R^T and the push-through
// identity R^T F = (I + lambda1/rho R^T R)^{-1} R^T turns lambda1/rho Y_h R^T F into
// Y_h G R^T.  The rearrangement is exact and keeps every FP32 term O(|X|) instead of
// O(lambda1/rho |Y_h|), which avoids a large cancellation.  The contraction A0 R over
// bands is summed per band share and the parts are added in share order (through LDS when a
// pixel has several threads).
//   Lambda1 -= BX - P1,  Lambda2 -= X - P2;  W1 = P1 + Lambda1,  W2 = P2 + Lambda2
// Off the sampled pixels P1 = BX - Lambda1 gives Lambda1 = Lambda1 - (BX - P1) = 0 and W1 = BX,
// exactly, from Lambda1 = 0 at the start: so when B X arrives in W1 (slots bx == w1) only the
// sampled pixels, one in d^2, have a P1 to update.  Per pixel and band that leaves 16 bytes (X
// and Lambda2 read, Lambda2 and W2 written) of 32: a 12-scene batch, whose P-update runs beside
// the sweep, 16.6 -> 15.7 ms per 10-iteration solve; 256 x 256 x 31, where the launch is bound by
// latency, 15.1 -> 14.7 us.
// Band shares of the contraction A0 R in the P-update: fixed, so that the sum is the same
// whichever number of threads a pixel has.
constexpr int kPuShares = 4;

// rp += sum over bands [c0, c1) of (X - Lambda2)_c R_c, one fused multiply-add per term.
template <int LHM>
__device__ __forceinline__ void pupdate_share(const gfloat* __restrict__ X,
                                              const gfloat* __restrict__ L2,
                                              cfloat* R, float (&rp)[LHM],
                                              size_t plane, int Lh, int c0, int c1, int j) {
  for (int c = c0; c < c1; ++c) {
    const float a0 = X[c * plane + j] - L2[c * plane + j];
#pragma unroll
    for (int h = 0; h < LHM; ++h)
      if (h < Lh) rp[h] = __builtin_fmaf(a0, R[c * Lh + h], rp[h]);
  }
}

// Bands [c0, c1) of one pixel: P2, Lambda2, W2 and, where p1, P1, Lambda1 and W1.  Lambda is
// read through L1, L2 and written through L1o, L2o, which may be the same buffers, and BX may
// be W1 (no restrict on those six); BXo, if not null, also takes B X where p1.  R and G are read
// through the constant address space, so that they stay scalar loads in the sweep's launch too
// (as vector loads there, 256 x 256 x 31 took 1995 instead of 1922 us).
template <int LHM>
__device__ __forceinline__ void pupdate_write(
    const gfloat* __restrict__ X, const gfloat* BX, const gfloat* __restrict__ Yl,
    const gfloat* L1, const gfloat* L2, gfloat* L1o, gfloat* L2o, gfloat* W1,
    gfloat* __restrict__ W2, gfloat* BXo, cfloat* R, const float (&u)[LHM],
    size_t plane, size_t lplane, size_t lj, bool sampled, bool p1, int Lh, float rho,
    float inv_1prho, int c0, int c1, int j) {
  for (int c = c0; c < c1; ++c) {
    const size_t o = c * plane + j;
    float corr = 0.f;
#pragma unroll
    for (int h = 0; h < LHM; ++h)
      if (h < Lh) corr += u[h] * R[c * Lh + h];
    const float x = X[o], l2 = L2[o];
    const float p2 = (x - l2) + corr;
    const float l2n = l2 - (x - p2);
    L2o[o] = l2n;
    W2[o] = p2 + l2n;
    if (!p1) continue;
    const float bx = BX[o], l1 = L1[o];
    const float p1v = sampled ? (rho * bx + Yl[c * lplane + lj] - rho * l1) * inv_1prho : bx - l1;
    const float l1n = l1 - (bx - p1v);
    L1o[o] = l1n;
    W1[o] = p1v + l1n;
    if (BXo) BXo[o] = bx;
  }
}

// With at most kPuKeep bands per thread, X and Lambda2 are read once: the contraction pass
// keeps them in registers for the write pass (32 bytes per pixel and band instead of 40).
// Same operations in the same order as the two functions above.
constexpr int kPuKeep = 16;

// All loads of the thread's bands up front (X, Lambda2, and for P1 BX and Lambda1), so that
// their latencies overlap: the contraction pass then only waits for X and Lambda2.
template <int LHM>
__device__ __forceinline__ void pupdate_load_keep(const gfloat* __restrict__ X,
                                                  const gfloat* __restrict__ L2,
                                                  const gfloat* BX, const gfloat* L1,
                                                  const gfloat* __restrict__ Yl, bool p1,
                                                  bool sampled, size_t plane, size_t lplane,
                                                  size_t lj, int c0, int c1, int j,
                                                  float (&xs)[kPuKeep], float (&l2s)[kPuKeep],
                                                  float (&bxs)[kPuKeep], float (&l1s)[kPuKeep],
                                                  float (&yls)[kPuKeep]) {
#pragma unroll
  for (int i = 0; i < kPuKeep; ++i) {
    const int c = c0 + i;
    if (c < c1) {
      xs[i] = X[c * plane + j];
      l2s[i] = L2[c * plane + j];
    }
  }
  if (!p1) return;
#pragma unroll
  for (int i = 0; i < kPuKeep; ++i) {
    const int c = c0 + i;
    if (c < c1) {
      bxs[i] = BX[c * plane + j];
      l1s[i] = L1[c * plane + j];
      if (sampled) yls[i] = Yl[c * lplane + lj];
    }
  }
}

// rp += sum over bands [cs, ce) of (X - Lambda2)_c R_c, from the kept values (band c at
// register c - c0)
template <int LHM>
__device__ __forceinline__ void pupdate_share_kept(const float (&xs)[kPuKeep],
                                                   const float (&l2s)[kPuKeep],
                                                   cfloat* R,
                                                   float (&rp)[LHM], int Lh, int c0, int cs,
                                                   int ce) {
#pragma unroll
  for (int i = 0; i < kPuKeep; ++i) {
    const int c = c0 + i;
    if (c >= cs && c < ce) {
      const float a0 = xs[i] - l2s[i];
#pragma unroll
      for (int h = 0; h < LHM; ++h)
        if (h < Lh) rp[h] = __builtin_fmaf(a0, R[c * Lh + h], rp[h]);
    }
  }
}

template <int LHM>
__device__ __forceinline__ void pupdate_write_kept(
    const float (&xs)[kPuKeep], const float (&l2s)[kPuKeep], const float (&bxs)[kPuKeep],
    const float (&l1s)[kPuKeep], const float (&yls)[kPuKeep], gfloat* L1o, gfloat* L2o,
    gfloat* __restrict__ W1, gfloat* __restrict__ W2, gfloat* BXo, cfloat* R,
    const float (&u)[LHM], size_t plane, bool sampled, bool p1, int Lh, float rho,
    float inv_1prho, int c0, int c1, int j) {
#pragma unroll
  for (int i = 0; i < kPuKeep; ++i) {
    const int c = c0 + i;
    if (c >= c1) continue;
    const size_t o = c * plane + j;
    float corr = 0.f;
#pragma unroll
    for (int h = 0; h < LHM; ++h)
      if (h < Lh) corr += u[h] * R[c * Lh + h];
    const float x = xs[i], l2 = l2s[i];
    const float p2 = (x - l2) + corr;
    const float l2n = l2 - (x - p2);
    L2o[o] = l2n;
    W2[o] = p2 + l2n;
    if (!p1) continue;
    const float bx = bxs[i], l1 = l1s[i];
    const float p1v = sampled ? (rho * bx + yls[i] - rho * l1) * inv_1prho : bx - l1;
    const float l1n = l1 - (bx - p1v);
    L1o[o] = l1n;
    W1[o] = p1v + l1n;
    if (BXo) BXo[o] = bx;
  }
}

// LDS of a workgroup: the shares' parts of A0 R
constexpr int pupdate_lds_floats(int lhm, int nc) { return nc > 1 ? 256 * lhm : 1; }

template <int LHM, int PU_NC, bool KEEP>
__device__ __forceinline__ void pupdate_body(const SceneDesc& S, int item, int quarter,
                                             const PuSlots& sl, float* part) {
  constexpr int PX = 256 / PU_NC;          // pixels of the workgroup
  const int p = S.p, q = S.q, L = S.L, Lh = S.Lh, d = S.d;
  // the band share is uniform over a wave; readfirstlane lets the band loops index R and G
  // with scalar loads
  const int pix = threadIdx.x & (PX - 1);
  const int ch = PU_NC == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x / PX);
  const int j = item * 256 + quarter * PX + pix;
  const size_t plane = (size_t)p * q;
  const bool act = j < (int)plane;
  const int c0 = (L * ch) / PU_NC, c1 = (L * (ch + 1)) / PU_NC;   // this thread's bands
  const gfloat* __restrict__ X = gslot<const gfloat>(S, sl.x);
  const gfloat* L2 = gslot<const gfloat>(S, sl.l2);
  cfloat* R = as_constant(S.R);
  cfloat* G = as_constant(S.G);
  const gfloat* __restrict__ Yh = gslot<const gfloat>(S, sl.yh);
  // res = Y_h - A0 R.  The bands form kPuShares contiguous shares; each share's part of A0 R
  // is summed on its own and the parts are added in share order, so the result does not
  // depend on how many threads a pixel has.
  float res[LHM];
  // KEEP: every scene of the launch has at most kPuKeep bands per thread
  const int i1 = j / q, i2 = j - i1 * q;
  const bool sampled = (i1 % d == 0) && (i2 % d == 0);
  // no P1 with the fused-S splitting; with a basis p1_subspace_kernel updates the sampled
  // pixels; and with W1 in place of B X the others hold their W1 (see launch_pupdate)
  const bool p1 = !S.fused && (sampled ? !S.subspace : sl.bx != sl.w1);
  const size_t lplane = (size_t)(p / d) * (q / d), lj = (size_t)(i1 / d) * (q / d) + i2 / d;
  float xs[KEEP ? kPuKeep : 1], l2s[KEEP ? kPuKeep : 1], bxs[KEEP ? kPuKeep : 1],
      l1s[KEEP ? kPuKeep : 1], yls[KEEP ? kPuKeep : 1], yh[LHM];
  if constexpr (KEEP)
    if (act)
    pupdate_load_keep<LHM>(X, L2, gslot<const gfloat>(S, sl.bx), gslot<const gfloat>(S, sl.l1),
                           gslot<const gfloat>(S, sl.yl), p1, sampled, plane, lplane, lj, c0, c1,
                           j, xs, l2s, bxs, l1s, yls);
  if (act) {
#pragma unroll
    for (int h = 0; h < LHM; ++h) yh[h] = (h < Lh) ? Yh[h * plane + j] : 0.f;
  }
  if constexpr (PU_NC == 1) {
    // one thread per pixel: the parts are added in registers, and no barrier sits between
    // the two band loops (with one the memory-bound loops of different waves do not overlap)
    if (!act) return;
    float a[LHM];
#pragma unroll
    for (int h = 0; h < LHM; ++h) a[h] = 0.f;
    for (int k = 0; k < kPuShares; ++k) {
      float rp[LHM];
#pragma unroll
      for (int h = 0; h < LHM; ++h) rp[h] = 0.f;
      if constexpr (KEEP)
        pupdate_share_kept<LHM>(xs, l2s, R, rp, Lh, c0, (L * k) / kPuShares,
                                (L * (k + 1)) / kPuShares);
      else
        pupdate_share<LHM>(X, L2, R, rp, plane, Lh, (L * k) / kPuShares,
                           (L * (k + 1)) / kPuShares, j);
#pragma unroll
      for (int h = 0; h < LHM; ++h) a[h] += rp[h];
    }
#pragma unroll
    for (int h = 0; h < LHM; ++h) res[h] = (h < Lh) ? yh[h] - a[h] : 0.f;
  } else {
    static_assert(PU_NC == kPuShares, "one share per thread");
    float rp[LHM];
#pragma unroll
    for (int h = 0; h < LHM; ++h) rp[h] = 0.f;
    if (act) {
      if constexpr (KEEP) pupdate_share_kept<LHM>(xs, l2s, R, rp, Lh, c0, c0, c1);
      else pupdate_share<LHM>(X, L2, R, rp, plane, Lh, c0, c1, j);
    }
#pragma unroll
    for (int h = 0; h < LHM; ++h) part[(ch * LHM + h) * PX + pix] = rp[h];
    __syncthreads();
    if (!act) return;
#pragma unroll
    for (int h = 0; h < LHM; ++h) {
      float a = 0.f;
#pragma unroll
      for (int k = 0; k < PU_NC; ++k) a += part[(k * LHM + h) * PX + pix];
      res[h] = (h < Lh) ? yh[h] - a : 0.f;
    }
  }
  float u[LHM];                           // u = res G
#pragma unroll
  for (int h2 = 0; h2 < LHM; ++h2) {
    float sum = 0.f;
#pragma unroll
    for (int h = 0; h < LHM; ++h)
      if (h < Lh && h2 < Lh) sum += res[h] * G[h * Lh + h2];
    u[h2] = sum;
  }
  if constexpr (KEEP)
    pupdate_write_kept<LHM>(xs, l2s, bxs, l1s, yls, gslot<gfloat>(S, sl.l1o),
                            gslot<gfloat>(S, sl.l2o), gslot<gfloat>(S, sl.w1),
                            gslot<gfloat>(S, sl.w2), gslot<gfloat>(S, sl.bxo), R, u, plane,
                            sampled, p1, Lh, S.rho, S.inv_1prho, c0, c1, j);
  else
    pupdate_write<LHM>(X, gslot<const gfloat>(S, sl.bx), gslot<const gfloat>(S, sl.yl),
                       gslot<const gfloat>(S, sl.l1), L2, gslot<gfloat>(S, sl.l1o),
                       gslot<gfloat>(S, sl.l2o), gslot<gfloat>(S, sl.w1), gslot<gfloat>(S, sl.w2),
                       gslot<gfloat>(S, sl.bxo), R, u, plane, lplane, lj, sampled, p1, Lh, S.rho,
                       S.inv_1prho, c0, c1, j);
}

}  // namespace
}  // namespace nlpr
