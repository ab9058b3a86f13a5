// X-update of the ADMM iteration: X_c = IDFT2(DFT2(C_c) / den) for every band c
// (Sec. "Optimization", eqs. (xupdateoper), (inv)).
//
// Two real bands a = 2m, b = 2m+1 are packed into one complex image C_a + i C_b.  The
// spectral weight 1/den is real and even (den(-w) = den(w)), so filtering the packed image
// and splitting real / imaginary parts gives the two filtered bands exactly; one complex
// 2-D transform pair serves two bands.
//
// The 2-D transform runs as three passes over a complex [pairs][p][q] buffer:
//   rows_fwd   : pack two bands, forward DFT along every row
//   cols_solve : forward DFT along columns, multiply by 1/(den p q), inverse DFT along
//                columns (between the two transforms the points stay in registers at powers of
//                2, in LDS else)
//   rows_inv   : inverse DFT along rows, unpack the two bands
// Every pass runs over a batch of scenes (see nlpr_internal.h).  Lines per block and columns per
// block are picked per image size: for a scene alone by timing candidates when its plan is
// created, for the scenes of a batch by rule (batch_fft_shape).
// Each 1-D transform is a Stockham autosort FFT (mixed radix 2/3/4/8): every stage reads R
// values strided by n/R, twiddles them, does an R-point DFT and writes them to their
// natural-order position, so no bit reversal is needed.  The first stage reads global memory
// and the last one writes it (both touch points n/R apart per thread, neighbouring threads
// neighbouring points), so LDS only carries the exchanges between stages.  Twiddles come from
// a table computed in FP64.
//
// The passes are bound by the latency of their requests and barriers (8 MB planes live in the
// caches).  Per launch at 256 x 256 x 31 / 1024 x 1024 x 4, against passes that staged every
// line through LDS on the way in and out, with two block barriers per stage: rows 9.3 -> 7.3 /
// 15.1 -> 11.9 us, columns 17.0 -> 13.7 / 39 -> 20 us (half of that from the order of the
// workgroups); columns of fused-S at 192 x 256 x 31, whose groups one thread each solved:
// 29 -> 17 us; 12-scene batch: rows 24.6 -> 13.5, columns 38 -> 27 us.
#include <algorithm>
#include <map>
#include <mutex>
#include <tuple>

#include "nlpr_internal.h"

namespace nlpr {
namespace {

__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cscale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }
// a * (-i) for the forward transform, a * (+i) for the inverse
template <bool INV>
__device__ __forceinline__ float2 rot90(float2 a) {
  return INV ? make_float2(-a.y, a.x) : make_float2(a.y, -a.x);
}

template <int R, bool INV> struct Dft;

template <bool INV> struct Dft<2, INV> {
  __device__ __forceinline__ static void run(float2* v) {
    float2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  }
};

template <bool INV> struct Dft<4, INV> {
  __device__ __forceinline__ static void run(float2* v) {
    float2 t0 = cadd(v[0], v[2]), t1 = csub(v[0], v[2]);
    float2 t2 = cadd(v[1], v[3]), t3 = rot90<INV>(csub(v[1], v[3]));
    v[0] = cadd(t0, t2);
    v[1] = cadd(t1, t3);
    v[2] = csub(t0, t2);
    v[3] = csub(t1, t3);
  }
};

template <bool INV> struct Dft<8, INV> {
  __device__ __forceinline__ static void run(float2* v) {
    float2 e[4] = {v[0], v[2], v[4], v[6]};
    float2 o[4] = {v[1], v[3], v[5], v[7]};
    Dft<4, INV>::run(e);
    Dft<4, INV>::run(o);
    const float c = 0.70710678118654752440f;
    // w8^s, w8 = exp(-+ 2 pi i / 8)
    const float2 w1 = INV ? make_float2(c, c) : make_float2(c, -c);
    const float2 w3 = INV ? make_float2(-c, c) : make_float2(-c, -c);
    float2 o1 = cmul(o[1], w1), o2 = rot90<INV>(o[2]), o3 = cmul(o[3], w3);
    v[0] = cadd(e[0], o[0]);
    v[4] = csub(e[0], o[0]);
    v[1] = cadd(e[1], o1);
    v[5] = csub(e[1], o1);
    v[2] = cadd(e[2], o2);
    v[6] = csub(e[2], o2);
    v[3] = cadd(e[3], o3);
    v[7] = csub(e[3], o3);
  }
};

template <bool INV> struct Dft<3, INV> {
  __device__ __forceinline__ static void run(float2* v) {
    const float s3 = 0.86602540378443864676f;  // sqrt(3)/2
    float2 a = v[0], b = v[1], c = v[2];
    float2 t1 = cadd(b, c);
    float2 t2 = csub(a, cscale(t1, 0.5f));
    float2 t3 = cscale(rot90<INV>(csub(b, c)), s3);
    v[0] = cadd(a, t1);
    v[1] = cadd(t2, t3);
    v[2] = csub(t2, t3);
  }
};

// One Stockham stage of radix R on a line of n points.  Ns is the product of the radices of
// the earlier stages; tw holds the line's n twiddles, staged in LDS.  Threads t < tpl of the
// line take part; tpl >= ceil(n/8) keeps every thread at <= ceil(8/R) butterflies.
// rd(u, r, i) gives point i, wr(u, r, i, v) takes it (butterfly u of the thread, leg r).
// IN_LDS / OUT_LDS: rd reads / wr writes the line's LDS buffer; between a read and a write of
// it, and after a write, sync() orders the threads of a line.  Every thread of the block
// calls it.
template <int R, bool INV, bool IN_LDS, bool OUT_LDS, class RD, class WR, class SYNC>
__device__ __forceinline__ void fft_stage(int n, int Ns, int step, const float2* tw, int t,
                                          int tpl, RD rd, WR wr, SYNC sync) {
  constexpr int MAXB = (8 + R - 1) / R;
  const int nb = n / R;
  float2 v[MAXB][R];
#pragma unroll
  for (int u = 0; u < MAXB; ++u) {
    const int j = t + u * tpl;
    if (t < tpl && j < nb) {
#pragma unroll
      for (int r = 0; r < R; ++r) v[u][r] = rd(u, r, j + r * nb);
    }
  }
  if (IN_LDS && OUT_LDS) sync();
#pragma unroll
  for (int u = 0; u < MAXB; ++u) {
    const int j = t + u * tpl;
    if (t < tpl && j < nb) {
      const int k = (Ns & (Ns - 1)) == 0 ? j & (Ns - 1) : j % Ns;
      if constexpr (IN_LDS) {            // the twiddles of a transform's first stage are 1
#pragma unroll
        for (int r = 1; r < R; ++r) {
          float2 w = tw[r * k * step];
          if (INV) w.y = -w.y;
          v[u][r] = cmul(v[u][r], w);
        }
      }
      Dft<R, INV>::run(v[u]);
      // the values as they are here: a part computed in a branch of wr would round other
      // products into its additions
      if constexpr (!OUT_LDS) {
#pragma unroll
        for (int r = 0; r < R; ++r) asm volatile("" : "+v"(v[u][r].x), "+v"(v[u][r].y));
      }
      const int base = (j - k) * R + k;
#pragma unroll
      for (int r = 0; r < R; ++r) wr(u, r, base + r * Ns, v[u][r]);
    }
  }
  if (OUT_LDS) sync();
}

template <bool INV, bool IN_LDS, bool OUT_LDS, class RD, class WR, class SYNC>
__device__ __forceinline__ void fft_stage_r(int R, int n, int Ns, int step, const float2* tw,
                                            int t, int tpl, RD rd, WR wr, SYNC sync) {
  if (R == 8) fft_stage<8, INV, IN_LDS, OUT_LDS>(n, Ns, step, tw, t, tpl, rd, wr, sync);
  else if (R == 4) fft_stage<4, INV, IN_LDS, OUT_LDS>(n, Ns, step, tw, t, tpl, rd, wr, sync);
  else if (R == 2) fft_stage<2, INV, IN_LDS, OUT_LDS>(n, Ns, step, tw, t, tpl, rd, wr, sync);
  else fft_stage<3, INV, IN_LDS, OUT_LDS>(n, Ns, step, tw, t, tpl, rd, wr, sync);
}

// Twiddles of a line length, copied from the FP64-computed table to LDS, so that the stages
// read them without global latency (a barrier follows before the second stage).
__device__ __forceinline__ void stage_twiddles(float2* twl, const LineFFT& f) {
  const gfloat* tw = (const gfloat*)f.tw;
  for (int e = threadIdx.x; e < f.n; e += blockDim.x) twl[e] = ldg2(tw + 2 * e);
}

// A line transform from `first` (points of global memory) to `last`, through the line's LDS
// buffer (brd, bwr).  sync() orders the threads of a line, and its first call also orders the
// staged twiddles, so it is made a block barrier by the caller (sync0).  Transforms of one
// stage (n = 8) exchange nothing.
template <bool INV, class RD, class WR, class BR, class BW, class SYNC0, class SYNC>
__device__ __forceinline__ void fft_line(const LineFFT& f, int t, int tpl, const float2* tw,
                                         RD first, WR last, BR brd, BW bwr, SYNC0 sync0,
                                         SYNC sync) {
  const int nf = f.nfac;
  if (nf == 1) {                         // n = 8: the only length of one factor
    fft_stage<8, INV, false, false>(8, 1, 1, tw, t, tpl, first, last, sync);
    return;
  }
  int Ns = f.fac[0], step = f.n / f.fac[0];
  fft_stage_r<INV, false, true>(f.fac[0], f.n, 1, step, tw, t, tpl, first, bwr, sync0);
  for (int s = 1; s < nf - 1; ++s) {
    const int R = f.fac[s];
    step /= R;
    fft_stage_r<INV, true, true>(R, f.n, Ns, step, tw, t, tpl, brd, bwr, sync);
    Ns *= R;
  }
  fft_stage_r<INV, true, false>(f.fac[nf - 1], f.n, Ns, 1, tw, t, tpl, brd, last, sync);
}

// Order the LDS accesses of a line's threads.  Where they are lanes of one wave (tpl divides
// 64) the LDS pipe does it, since a wave's accesses execute in order: only the compiler has to
// keep them in place.  Else a block barrier.
__device__ __forceinline__ void line_sync(bool in_wave) {
  if (in_wave) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  } else {
    __syncthreads();
  }
}

// LDS position of point i of a row line: one point of padding per 8, so that the stages'
// stores, 8 points apart at first, spread over the banks.
__device__ __forceinline__ int row_pos(int i) { return i + (i >> 3); }

// Pack bands (2m, 2m+1) of C, forward DFT along rows.  Local block = (pair, row block).
__global__ void fft_rows_fwd(const SceneDesc* __restrict__ sd, const int2* __restrict__ items,
                             int c_s, int f_s) {
  extern __shared__ float2 sh[];
  const int2 it = work_item_xcd(items);
  const SceneDesc& S = sd[it.x];
  const int p = S.p, q = S.q, L = S.L, lpb = S.fq_lpb, tpl = S.fq_tpl;
  const int nrb = ceil_div(p, lpb);
  const int m = it.y / nrb, row0 = (it.y - m * nrb) * lpb;
  const size_t plane = (size_t)p * q;
  const int g = threadIdx.x / tpl, r = row0 + g;
  const bool act = g < lpb && r < p;
  const int t = act ? threadIdx.x - g * tpl : tpl;
  const bool two = 2 * m + 1 < L;
  const gfloat* Ca = gslot<const gfloat>(S, c_s) + (size_t)(2 * m) * plane;
  const gfloat* Cb = Ca + (two ? plane : 0);
  gfloat* Fm = gslot<gfloat>(S, f_s) + 2 * (size_t)m * plane;   // complex, interleaved
  const unsigned ro = (unsigned)r * q;
  float2* buf = sh + (act ? g : 0) * row_pos(q);
  float2* twl = sh + lpb * row_pos(q);
  stage_twiddles(twl, S.fq);
  const bool in_wave = 64 % tpl == 0;
  fft_line<false>(
      S.fq, t, tpl, twl,
      [&](int, int, int i) { return make_float2(Ca[ro + i], two ? Cb[ro + i] : 0.f); },
      [&](int, int, int i, float2 v) { stg2(Fm + 2 * (ro + i), v); },
      [&](int, int, int i) { return buf[row_pos(i)]; },
      [&](int, int, int i, float2 v) { buf[row_pos(i)] = v; }, [] { __syncthreads(); },
      [&] { line_sync(in_wave); });
}

// Forward DFT along columns, multiply by invden, inverse DFT along columns.
// Local block = (pair, column block); LDS holds cb columns of p points, point i of column l at
// i cb + l.  Thread = (column l, thread t of the line), columns fastest: a stage's accesses to
// global memory and to LDS are runs of cb neighbouring columns.  The weights 1/den of the
// thread's last-stage points are requested before the forward transform.  At a power of 2 the
// last forward stage leaves a thread the points its first inverse stage reads (p = 8 tpl, first
// radix 8, last 8, 4 or 2): they stay in registers.
//
// Fused-S scenes solve, per aliasing group of d^2 frequencies, the system of
// fused_tables_kernel instead of the division: line l of the block holds column
// b0 + (l % cbb) + (l / cbb) q/d (cbb = cb / d base columns and their d - 1 column aliases),
// so each group's d^2 entries (rows i1 + m1 p/d of those d columns) are in LDS.  All lines
// are transformed forward, the group solves run, then all lines are transformed back.  A group
// is solved by d threads, one per column: each sums the d entries of its column, the d sums
// are added through LDS in the order of the columns, and each thread updates its d entries.
template <int RL>
__device__ __forceinline__ void cols_plain(const SceneDesc& S, int t, int tpl, int cb, int l,
                                           int col, float2* sh, const float2* twl, gfloat* Fm) {
  const int p = S.p, q = S.q, nf = S.fp.nfac;
  constexpr int MAXB = (8 + RL - 1) / RL;
  constexpr bool KEEP = RL != 3;         // with p = 8 tpl, checked by the caller's choice of RL
  const gfloat* invden = as_global(S.invden);
  const int nb = p / RL;
  auto brd = [&](int, int, int i) { return sh[i * cb + l]; };
  auto bwr = [&](int, int, int i, float2 v) { sh[i * cb + l] = v; };
  auto sync = [] { __syncthreads(); };
  auto gin = [&](int, int, int i) { return ldg2(Fm + 2 * (unsigned)(i * q + col)); };
  auto gout = [&](int, int, int i, float2 v) { stg2(Fm + 2 * (unsigned)(i * q + col), v); };
  // the points of the last forward stage: i = t + u tpl + r nb
  float sv[MAXB][RL];
#pragma unroll
  for (int u = 0; u < MAXB; ++u)
#pragma unroll
    for (int r = 0; r < RL; ++r)
      sv[u][r] = t < tpl && t + u * tpl < nb ? invden[(unsigned)((t + u * tpl + r * nb) * q + col)] : 0.f;
  float2 keep[KEEP ? 8 : 1];
  auto scaled = [&](int u, int r, int i, float2 v) {
    v = cscale(v, sv[u][r]);
    if constexpr (KEEP) keep[u + MAXB * r] = v;    // point t + (u + MAXB r) tpl
    else bwr(u, r, i, v);
  };
  // forward
  const int R0 = S.fp.fac[0];
  int Ns = R0, step = p / R0;
  if (nf == 1) {                         // p = 8
    fft_stage<RL, false, false, !KEEP>(p, 1, 1, twl, t, tpl, gin, scaled, sync);
  } else {
    fft_stage_r<false, false, true>(R0, p, 1, step, twl, t, tpl, gin, bwr, sync);
    for (int s = 1; s < nf - 1; ++s) {
      const int R = S.fp.fac[s];
      step /= R;
      fft_stage_r<false, true, true>(R, p, Ns, step, twl, t, tpl, brd, bwr, sync);
      Ns *= R;
    }
    fft_stage<RL, false, true, !KEEP>(p, Ns, 1, twl, t, tpl, brd, scaled, sync);
    if (KEEP) sync();                    // the last reads of the buffer before it is rewritten
  }
  // inverse
  if constexpr (KEEP) {
    auto kin = [&](int, int r, int) { return keep[r]; };
    if (nf == 1) {
      fft_stage<8, true, false, false>(p, 1, 1, twl, t, tpl, kin, gout, sync);
      return;
    }
    fft_stage<8, true, false, true>(p, 1, p / 8, twl, t, tpl, kin, bwr, sync);
  } else {
    fft_stage_r<true, true, true>(R0, p, 1, p / R0, twl, t, tpl, brd, bwr, sync);
  }
  Ns = R0;
  step = p / R0;
  for (int s = 1; s < nf - 1; ++s) {
    const int R = S.fp.fac[s];
    step /= R;
    fft_stage_r<true, true, true>(R, p, Ns, step, twl, t, tpl, brd, bwr, sync);
    Ns *= R;
  }
  fft_stage_r<true, true, false>(S.fp.fac[nf - 1], p, Ns, 1, twl, t, tpl, brd, gout, sync);
}


// The forward transform of a line into its LDS buffer, and the inverse one out of it.
template <class RD, class BR, class BW, class SYNC>
__device__ __forceinline__ void cols_to_lds(const SceneDesc& S, int t, int tpl,
                                            const float2* twl, RD gin, BR brd, BW bwr,
                                            SYNC sync) {
  const int p = S.p, nf = S.fp.nfac, R0 = S.fp.fac[0];
  int Ns = R0, step = p / R0;
  fft_stage_r<false, false, true>(R0, p, 1, step, twl, t, tpl, gin, bwr, sync);
  for (int s = 1; s < nf; ++s) {
    const int R = S.fp.fac[s];
    step /= R;
    fft_stage_r<false, true, true>(R, p, Ns, step, twl, t, tpl, brd, bwr, sync);
    Ns *= R;
  }
}
template <class BR, class BW, class WR, class SYNC>
__device__ __forceinline__ void cols_from_lds(const SceneDesc& S, int t, int tpl,
                                              const float2* twl, BR brd, BW bwr, WR gout,
                                              SYNC sync) {
  const int p = S.p, nf = S.fp.nfac;
  int Ns = 1, step = p;
  for (int s = 0; s < nf - 1; ++s) {
    const int R = S.fp.fac[s];
    step /= R;
    fft_stage_r<true, true, true>(R, p, Ns, step, twl, t, tpl, brd, bwr, sync);
    Ns *= R;
  }
  fft_stage_r<true, true, false>(S.fp.fac[nf - 1], p, Ns, 1, twl, t, tpl, brd, gout, sync);
}

__global__ void fft_cols_solve(const SceneDesc* __restrict__ sd, const int2* __restrict__ items,
                               int f_s) {
  extern __shared__ float2 sh[];
  const int2 it = work_item_xcd(items);
  const SceneDesc& S = sd[it.x];
  const int p = S.p, q = S.q, cb = S.fp_cb, tpl = S.fp_tpl;
  const int ncb = ceil_div(q, cb);
  const int m = it.y / ncb, cblk = it.y - m * ncb;
  const size_t plane = (size_t)p * q;
  gfloat* Fm = gslot<gfloat>(S, f_s) + 2 * (size_t)m * plane;   // complex, interleaved
  float2* twl = sh + cb * p;
  stage_twiddles(twl, S.fp);
  const int t0 = threadIdx.x / cb, l = threadIdx.x - t0 * cb;
  const int d = S.d, cbb = S.fused ? cb / d : cb, qd = q / d;
  // column of line l (-1: past the image)
  int col;
  if (!S.fused) {
    col = cblk * cb + l;
    if (col >= q) col = -1;
  } else {
    const int bc = cblk * cbb + l % cbb;
    col = bc < qd ? bc + (l / cbb) * qd : -1;
  }
  const int t = t0 < tpl && col >= 0 ? t0 : tpl;
  if (!S.fused) {
    // (a length with a factor 3 ends on radix 3; the others are powers of 2, p = 8 tpl, and
    // start on radix 8)
    const int RL = S.fp.fac[S.fp.nfac - 1];
    if (RL == 3) cols_plain<3>(S, t, tpl, cb, l, col, sh, twl, Fm);
    else if (RL == 8) cols_plain<8>(S, t, tpl, cb, l, col, sh, twl, Fm);
    else if (RL == 4) cols_plain<4>(S, t, tpl, cb, l, col, sh, twl, Fm);
    else cols_plain<2>(S, t, tpl, cb, l, col, sh, twl, Fm);
    return;
  }
  auto brd = [&](int, int, int i) { return sh[i * cb + l]; };
  auto bwr = [&](int, int, int i, float2 v) { sh[i * cb + l] = v; };
  auto gin = [&](int, int, int i) { return ldg2(Fm + 2 * (unsigned)(i * q + col)); };
  auto gout = [&](int, int, int i, float2 v) { stg2(Fm + 2 * (unsigned)(i * q + col), v); };
  auto sync = [] { __syncthreads(); };
  cols_to_lds(S, t, tpl, twl, gin, brd, bwr, sync);
  const int pd = p / d;
  const gfloat* ia = as_global(S.fia);
  const gfloat* fu = (const gfloat*)S.fu;
  const gfloat* fv = (const gfloat*)S.fv;
  float2* part = twl + p;                // [pd][cb]
  for (int e = threadIdx.x; e < pd * cb; e += blockDim.x) {
    const int i1 = e / cb, le = e - i1 * cb, bc = cblk * cbb + le % cbb;
    if (bc >= qd) continue;
    const int ce = bc + (le / cbb) * qd;
    float tr = 0.f, ti = 0.f;            // sum over the column's entries of u c
    for (int m1 = 0; m1 < d; ++m1) {
      const int i = i1 + m1 * pd;
      const float2 u = ldg2(fu + 2 * (unsigned)(i * q + ce)), c = sh[i * cb + le];
      tr += u.x * c.x - u.y * c.y;
      ti += u.x * c.y + u.y * c.x;
    }
    part[e] = make_float2(tr, ti);
  }
  __syncthreads();
  for (int e = threadIdx.x; e < pd * cb; e += blockDim.x) {
    const int i1 = e / cb, le = e - i1 * cb, bl = le % cbb, bc = cblk * cbb + bl;
    if (bc >= qd) continue;
    const int ce = bc + (le / cbb) * qd;
    float tr = 0.f, ti = 0.f;
    for (int m2 = 0; m2 < d; ++m2) {
      const float2 s2 = part[i1 * cb + m2 * cbb + bl];
      tr += s2.x;
      ti += s2.y;
    }
    for (int m1 = 0; m1 < d; ++m1) {
      const int i = i1 + m1 * pd;
      const float a = ia[(unsigned)(i * q + ce)];
      const float2 v = ldg2(fv + 2 * (unsigned)(i * q + ce)), c = sh[i * cb + le];
      sh[i * cb + le] =
          make_float2(a * c.x - (v.x * tr - v.y * ti), a * c.y - (v.x * ti + v.y * tr));
    }
  }
  __syncthreads();
  cols_from_lds(S, t, tpl, twl, brd, bwr, gout, sync);
}

// Inverse DFT along rows, unpack bands (2m, 2m+1) into X.
// ADD: plus a [L][p][q] slot.
template <bool ADD>
__global__ void fft_rows_inv(const SceneDesc* __restrict__ sd, const int2* __restrict__ items,
                             int f_s, int x_s, int add_s) {
  extern __shared__ float2 sh[];
  const int2 it = work_item_xcd(items);
  const SceneDesc& S = sd[it.x];
  const int p = S.p, q = S.q, L = S.L, lpb = S.fq_lpb, tpl = S.fq_tpl;
  const int nrb = ceil_div(p, lpb);
  const int m = it.y / nrb, row0 = (it.y - m * nrb) * lpb;
  const size_t plane = (size_t)p * q;
  const int g = threadIdx.x / tpl, r = row0 + g;
  const bool act = g < lpb && r < p;
  const int t = act ? threadIdx.x - g * tpl : tpl;
  const bool two = 2 * m + 1 < L;
  const gfloat* Fm = gslot<const gfloat>(S, f_s) + 2 * (size_t)m * plane;   // complex
  const unsigned ro = (unsigned)r * q;
  gfloat* Xa = gslot<gfloat>(S, x_s) + (size_t)(2 * m) * plane;
  gfloat* Xb = Xa + (two ? plane : 0);
  const gfloat* Aa = gslot<const gfloat>(S, ADD ? add_s : f_s) + (ADD ? (size_t)(2 * m) * plane : 0);
  const gfloat* Ab = Aa + (two ? plane : 0);
  float2* buf = sh + (act ? g : 0) * row_pos(q);
  float2* twl = sh + lpb * row_pos(q);
  stage_twiddles(twl, S.fq);
  const bool in_wave = 64 % tpl == 0;
  fft_line<true>(
      S.fq, t, tpl, twl, [&](int, int, int i) { return ldg2(Fm + 2 * (ro + i)); },
      [&](int, int, int i, float2 v) {
        Xa[ro + i] = ADD ? v.x + Aa[ro + i] : v.x;
        if (two) Xb[ro + i] = ADD ? v.y + Ab[ro + i] : v.y;
      },
      [&](int, int, int i) { return buf[row_pos(i)]; },
      [&](int, int, int i, float2 v) { buf[row_pos(i)] = v; }, [] { __syncthreads(); },
      [&] { line_sync(in_wave); });
}

// LDS of a row workgroup: the lines (padded) and a line of twiddles; of a column workgroup: the
// lines, a line of twiddles and, for fused-S, the partial sums of the group solves
constexpr size_t kFftLds = 65536;
size_t rows_bytes(int q, int lpb) {
  return ((size_t)lpb * (q + q / 8) + q) * sizeof(float2);
}
size_t cols_bytes(int p, int cb, int d_fused) {
  return ((size_t)(cb + 1) * p + (d_fused > 0 ? (size_t)cb * (p / d_fused) : 0)) * sizeof(float2);
}
// one line with its padding takes more than 64 KiB from q = 3888 on
size_t rows_max(int q) { return std::max(kFftLds, rows_bytes(q, 1)); }
// a column group of fused-S is at least d columns: beyond 64 KiB by its partial sums at most
size_t cols_max(int p, int d_fused) {
  return std::max(kFftLds, d_fused > 0 ? cols_bytes(p, d_fused, d_fused) : 0);
}

int launch_rows(const Batch& B, bool inv, int a, int b, int add, hipStream_t s) {
  for (const Group& g : B.groups[KD_ROWS]) {
    if (!g.nitems) continue;
    if (inv && add >= 0)
      hipLaunchKernelGGL(fft_rows_inv<true>, dim3(g.nitems), dim3(g.block), g.lds, s, B.d_desc,
                         items_of(B, g), a, b, add);
    else if (inv)
      hipLaunchKernelGGL(fft_rows_inv<false>, dim3(g.nitems), dim3(g.block), g.lds, s, B.d_desc,
                         items_of(B, g), a, b, -1);
    else
      hipLaunchKernelGGL(fft_rows_fwd, dim3(g.nitems), dim3(g.block), g.lds, s, B.d_desc,
                         items_of(B, g), a, b);
    NLPR_LAUNCH_CHECK(inv ? "fft_rows_inv" : "fft_rows_fwd");
  }
  return NLPR_OK;
}

int launch_cols(const Batch& B, int f, hipStream_t s) {
  for (const Group& g : B.groups[KD_COLS]) {
    if (!g.nitems) continue;
    hipLaunchKernelGGL(fft_cols_solve, dim3(g.nitems), dim3(g.block), g.lds, s, B.d_desc,
                       items_of(B, g), f);
    NLPR_LAUNCH_CHECK("fft_cols_solve");
  }
  return NLPR_OK;
}

}  // namespace

int fft_block(int tpl) {
  int b = 256;
  while (b < tpl) b *= 2;
  return b;
}

// Workgroup size for `lines` lines of tpl threads each (at most 1024 in all): at least
// fft_block(tpl), and every line of the block has its threads.
static int lines_block(int tpl, int lines) {
  int b = fft_block(tpl);
  while (b < lines * tpl && b < 1024) b *= 2;
  return b;
}

int rows_blocks(const Plan& P) {
  return ceil_div(P.prm.p, P.fft.q_lpb) * ((P.Lx + 1) / 2);
}
int cols_blocks(const Plan& P) {
  return ceil_div(P.prm.q, P.fft.p_cb) * ((P.Lx + 1) / 2);
}
size_t rows_lds(const Plan& P) { return rows_bytes(P.prm.q, P.fft.q_lpb); }
size_t cols_lds(const Plan& P) {
  return cols_bytes(P.prm.p, P.fft.p_cb, P.d_fia ? P.prm.d : 0);
}

// d_fused > 0: the columns per block must be a multiple of d (a base column and its aliases)
FftShape default_fft_shape(int p, int q, int d_fused) {
  FftShape f{};
  f.q_tpl = ceil_div(q, 8);
  f.p_tpl = ceil_div(p, 8);
  f.q_lpb = fft_block(f.q_tpl) / f.q_tpl;
  while (f.q_lpb > 1 && rows_bytes(q, f.q_lpb) > kFftLds) --f.q_lpb;
  const int unit = d_fused > 0 ? d_fused : 1;
  f.p_cb = unit;
  while (f.p_cb * 2 <= std::max(16, unit) && f.p_cb * 2 * f.p_tpl <= 1024 &&
         cols_bytes(p, f.p_cb * 2, d_fused) <= kFftLds)
    f.p_cb *= 2;
  f.q_bs = fft_block(f.q_tpl);
  f.p_bs = lines_block(f.p_tpl, f.p_cb);
  return f;
}

// A launch over scenes of several sizes has one workgroup size; threads without a line of their
// scene would only wait.  So a scene of a batch takes as many lines as fill workgroups of about
// the same size: 256 threads for the rows, 512 for the columns (more where one line, or one
// column group of fused-S, needs it).
void batch_fft_shape(Plan& P) {
  const int p = P.prm.p, q = P.prm.q, dfu = P.d_fia ? P.prm.d : 0;
  FftShape f = default_fft_shape(p, q, dfu);
  f.q_bs = fft_block(f.q_tpl);
  f.q_lpb = f.q_bs / f.q_tpl;
  const int unit = dfu > 0 ? dfu : 1;
  f.p_cb = unit;
  while (f.p_cb * 2 <= std::max(32, unit) && f.p_cb * 2 * f.p_tpl <= 512 &&
         cols_bytes(p, f.p_cb * 2, dfu) <= kFftLds)
    f.p_cb *= 2;
  f.p_bs = lines_block(f.p_tpl, f.p_cb);
  P.fft = f;
}

int launch_xsolve(const Batch& B, int c, int x, int f, int add, hipStream_t s) {
  int rc;
  if ((rc = launch_rows(B, false, c, f, -1, s))) return rc;
  if ((rc = launch_cols(B, f, s))) return rc;
  return launch_rows(B, true, f, x, add, s);
}

// Allow the passes of an image size more dynamic LDS than the default limit where a single line
// or column group needs it; before their launches and outside graph capture.
int fft_prepare(const Plan& P) {
  const void* kern[4] = {};
  if (rows_max(P.prm.q) > kFftLds) {
    kern[0] = reinterpret_cast<const void*>(fft_rows_fwd);
    kern[1] = reinterpret_cast<const void*>(fft_rows_inv<false>);
    kern[2] = reinterpret_cast<const void*>(fft_rows_inv<true>);
  }
  if (cols_max(P.prm.p, P.d_fia ? P.prm.d : 0) > kFftLds)
    kern[3] = reinterpret_cast<const void*>(fft_cols_solve);
  for (const void* k : kern)
    if (k)
      NLPR_HIP_TRY(hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)kMaxSweepLds));
  return NLPR_OK;
}

// Autotuner: time the row and column passes of one band pair for every admissible lines-
// per-block / columns-per-block choice and keep the fastest; results are cached per
// (device, p, q) for the life of the process.
int autotune_fft(Plan& P) {
  static std::mutex mtx;
  static std::map<std::tuple<int, int, int, int>, FftShape> cache;
  const int p = P.prm.p, q = P.prm.q;
  const int dfu = P.d_fia ? P.prm.d : 0;
  int dev = 0;
  NLPR_HIP_TRY(hipGetDevice(&dev));
  const auto key = std::make_tuple(dev, p, q, dfu);
  {
    std::lock_guard<std::mutex> lk(mtx);
    auto hit = cache.find(key);
    if (hit != cache.end()) {
      P.fft = hit->second;
      return NLPR_OK;
    }
  }
  FftShape best = default_fft_shape(p, q, dfu);
  const size_t plane = (size_t)p * q;
  // time on up to 16 band pairs so the launch fills the GPU like the real one
  const int tp = std::max(1, std::min((P.Lx + 1) / 2, 16));
  float* d_real = nullptr;
  float2* d_cplx = nullptr;
  SceneDesc* d_sd = nullptr;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  int rc = NLPR_OK;
  auto cleanup = [&]() {
    hipFree(d_real);
    hipFree(d_cplx);
    hipFree(d_sd);
    if (e0) hipEventDestroy(e0);
    if (e1) hipEventDestroy(e1);
  };
  if (hipMalloc(&d_real, 2 * tp * plane * sizeof(float)) != hipSuccess ||
      hipMalloc(&d_cplx, tp * plane * sizeof(float2)) != hipSuccess ||
      hipMalloc(&d_sd, sizeof(SceneDesc)) != hipSuccess ||
      hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
    cleanup();
    set_error("autotune: allocation failed");
    return NLPR_ERR_HIP;
  }
  hipMemset(d_real, 0, 2 * tp * plane * sizeof(float));
  // no work-item table, as in a solve of one scene: the workgroups run in its order (work_item_xcd)
  const int2* const items = nullptr;
  SceneDesc h{};
  h.p = p;
  h.q = q;
  h.L = 2 * tp;
  h.fp = P.fp;
  h.fq = P.fq;
  h.invden = P.d_invden;
  h.d = P.prm.d;
  h.fused = dfu > 0 ? 1 : 0;
  h.fia = P.d_fia;
  h.fu = P.d_fu;
  h.fv = P.d_fv;
  h.buf[B_C] = d_real;
  h.buf[B_Z] = d_real;
  h.buf[B_F] = d_cplx;
  // best of three runs of 5 launches each (single runs flip between near-equal candidates)
  auto time_it = [&](auto launch) -> float {
    launch();
    float best_ms = 1e30f;
    for (int trial = 0; trial < 3; ++trial) {
      hipEventRecord(e0, nullptr);
      for (int r = 0; r < 5; ++r) launch();
      hipEventRecord(e1, nullptr);
      hipEventSynchronize(e1);
      float ms = 0.f;
      hipEventElapsedTime(&ms, e0, e1);
      best_ms = std::min(best_ms, ms);
    }
    return best_ms;
  };
  // rows: lines per block from 1 up to what LDS holds, on a workgroup of lines_block threads
  {
    const int tpl = best.q_tpl;
    float tbest = 1e30f;
    for (int lpb = 1; lpb * tpl <= 1024; lpb *= 2) {
      if (rows_bytes(q, lpb) > rows_max(q)) break;
      const int bs = lines_block(tpl, lpb);
      h.fq_tpl = tpl;
      h.fq_lpb = lpb;
      hipMemcpy(d_sd, &h, sizeof(SceneDesc), hipMemcpyHostToDevice);
      const int nb = ceil_div(p, lpb) * tp;
      const size_t lds = rows_bytes(q, lpb);
      const float ms = time_it([&]() {
        hipLaunchKernelGGL(fft_rows_fwd, dim3(nb), dim3(bs), lds, nullptr, d_sd, items, (int)B_C,
                           (int)B_F);
        hipLaunchKernelGGL(fft_rows_inv<false>, dim3(nb), dim3(bs), lds, nullptr, d_sd, items, (int)B_F,
                           (int)B_Z, -1);
      });
      if (hipGetLastError() != hipSuccess) { rc = NLPR_ERR_HIP; break; }
      if (ms < tbest) { tbest = ms; best.q_lpb = lpb; best.q_bs = bs; }
    }
  }
  // columns: the same over columns per block
  if (rc == NLPR_OK) {
    const int tpl = best.p_tpl;
    float tbest = 1e30f;
    for (int cb = std::max(dfu, 1); cb <= std::max(32, dfu) && cb * tpl <= 1024; cb *= 2) {
      if (cols_bytes(p, cb, dfu) > cols_max(p, dfu)) break;
      const int bs = lines_block(tpl, cb);
      h.fp_tpl = tpl;
      h.fp_cb = cb;
      hipMemcpy(d_sd, &h, sizeof(SceneDesc), hipMemcpyHostToDevice);
      const int nb = ceil_div(q, cb) * tp;
      const size_t lds = cols_bytes(p, cb, dfu);
      const float ms = time_it([&]() {
        hipLaunchKernelGGL(fft_cols_solve, dim3(nb), dim3(bs), lds, nullptr, d_sd, items,
                           (int)B_F);
      });
      if (hipGetLastError() != hipSuccess) { rc = NLPR_ERR_HIP; break; }
      if (ms < tbest) { tbest = ms; best.p_cb = cb; best.p_bs = bs; }
    }
  }
  cleanup();
  if (rc != NLPR_OK) {
    set_error("autotune: a timing launch failed");
    return rc;
  }
  P.fft = best;
  std::lock_guard<std::mutex> lk(mtx);
  cache[key] = best;
  return NLPR_OK;
}

}  // namespace nlpr
