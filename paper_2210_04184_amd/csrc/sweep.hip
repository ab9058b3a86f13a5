// The regulariser sweep: the Q-update (eq. (Qj_main)), the Sigma-update (eq. (dualvar3_main))
// and the regulariser part of the next right-hand side (after eq. (x_linear_system_main)),
// fused into one pass over the dual state.  This is where nearly all HBM traffic of an
// iteration goes: every Sigma value is read once and written once.
//
// Reduced form used here (all identities are exact):
//  * Q-elimination.  With V = D_{tau k} X - Sigma_{tau k}, the soft-threshold gives
//    Q+ = V - clip(V, +-mu) and then Sigma+ = Sigma - (D X - Q+) = -clip(V, +-mu), so Q
//    need not be stored and Q+ + Sigma+ = V - 2 clip(V, +-mu).
//  * Half window.  omega_{i-tau,-tau} = omega_{i tau} and D_{-tau,k} X(i - tau) = -D_{tau k} X(i),
//    so from Sigma = 0 the duals of -tau stay minus those of tau (shifted by tau) and the
//    adjoint terms of tau and -tau are equal; tau = 0 contributes nothing.  Only the half
//    window W+ is visited and its adjoint terms count twice.
//  * Source alignment.  D_{tau k} X(i) = g_tau(i - k) with g_tau = X - X(. - tau) (the shift
//    property of the difference filters).  Storing Sigma'_{tau k}(j) = Sigma_{tau k}(j + k)
//    makes every update at j read g_tau(j) and the threshold mu(j + k, tau), and turns
//    sum_k D_{tau k}^T U_{tau k} into A_tau(j) - A_tau(j + tau) with A_tau = sum_k U'_{tau k}.
// So, per band and pixel j:   Creg(j) = 2 sum_{tau in W+} [A_tau(j) - A_tau(j + tau)].
//
// Work decomposition.  A workgroup owns a tile of `rows` full image rows of one band and
// loops over tau in W+.  Per tau it stages the thresholds mu(., tau) of the tile plus a K
// halo in LDS, forms g_tau from the X tile in LDS, then streams the (2K+1)^2 planes of
// Sigma' for its tile with 16-byte loads and stores, issuing all loads of one patch row
// before any compute.  A_tau is added to the thread's own pixels in registers and
// subtracted at j - tau in an LDS accumulator that spans the tile plus `halo` rows above
// it; since j -> j - tau is one-to-one, the LDS updates of one tau never collide.  The rows
// above the tile go to a small halo buffer that the right-hand-side assembly folds in, so
// the result is deterministic (no atomics).
//
// Split.  A scene with fewer (tile, band) pairs than the GPU has CUs would leave most of it
// idle, so each pair is then served by `psplit` workgroups, part j taking the contiguous
// shifts [j Npairs / psplit, (j+1) Npairs / psplit) of W+.  Part 0 writes the regulariser
// plane and its halo rows as above, part j > 0 its own plane (slot B_CSPLIT) and halo rows;
// the assembly adds the parts in a fixed order, so results stay bit-for-bit repeatable.
#include "nlpr_internal.h"
#include "pupdate.h"

namespace nlpr {
namespace {


// Sigma' is touched once per iteration: stream it with non-temporal loads and stores so it
// does not evict X and mu from the caches.
#ifndef NLPR_SWEEP_NT
#define NLPR_SWEEP_NT 1
#endif
__device__ __forceinline__ float4 ld_nt(const gfloat* p) {
#if NLPR_SWEEP_NT
  const v4f_t v = __builtin_nontemporal_load((const gv4f*)p);
#else
  const v4f_t v = *(const gv4f*)p;
#endif
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void st_nt(gfloat* p, float4 v) {
  v4f_t w = {v.x, v.y, v.z, v.w};
#if NLPR_SWEEP_NT
  __builtin_nontemporal_store(w, (gv4f*)p);
#else
  *(gv4f*)p = w;
#endif
}
__device__ __forceinline__ float clampf(float v, float m) { return fminf(fmaxf(v, -m), m); }

// ---- sweep kernel begin (the traffic record of the benchmark is keyed to this text)
// Storage of Sigma' (coded).  Every new dual value is -clip(V, +-mu), so an element that
// reached the threshold (|V| >= mu) holds exactly -mu (V > 0) or +mu (V < 0): its value
// follows from the threshold, which the sweep has at hand, and one sign bit.  Per float4
// item of a plane the state keeps a code byte, for element e:
//   bit e     the sign bit of V (set: the value is +mu when on the threshold, else -mu);
//   bit 4 + e off the threshold: the sign bit of |V| - mu, i.e. |V| < mu (a NaN V gives a
//             NaN with the sign of |V|, so it counts as on; the NaN reaches C through A).
// The bits are shifted in one at a time with alignbit.  An item with any element off the
// threshold (byte >= 16) is "open": its four values are stored as a float4, as
// clip(V, +-mu) = -Sigma' (so the next sweep adds them: V = g - Sigma').  Open items are
// packed per wave: the 64 items a wave owns in a plane (one 1 KB
// segment of the plane) keep the float4s of their open items at the start of that segment,
// in lane order, so a wave reads and writes only as many 16-byte slots as it has open
// items (mbcnt of the ballot gives each open lane its slot).  The last 64 bytes of a run are
// written whole: up to three lanes without an open item write what they hold into the slots
// after it, which nothing reads.  A part of a 64-byte block costs HBM a read of the rest
// (first sweep of 512 x 512 x 16, write only: 2.77 ms with runs that end anywhere, 1.82 ms
// with whole 64-byte blocks, 1.88 ms with whole 128-byte lines).  A wave reads its whole old
// run before it writes the new one, and each segment belongs to one wave, so the update is
// in place.  Decoding is exact: the stored values are the values, and -mu, +mu are the
// thresholds that produced the on-threshold ones.
// CODES (differentiated form): also record, per dual element, which branch of the
// threshold it took, which is all the sweep's adjoint needs of this iteration: 2 bits, 0 for
// |V| < mu, 1 for V >= mu, 2 for V <= -mu, 3 for V = 0 with mu = 0 (or V not a number).  The
// four elements of a float4 item share one byte, at the item's float offset / 4.
// count, if not null: add the number of open items written by each wave to one of the
// kCountSlots counters there (kCountStride apart); their sum is the launch's count.
// POLICY: which part of the dual state passes the caches by (sweep_policy).
template <int K, int ITEMS, int NT, bool FIRST, bool CODES, int POLICY>
__device__ __forceinline__ void
sweep_body(const SceneDesc* __restrict__ sd, const int2* __restrict__ items, int block, int x_s,
           int mu_s, int sig_s, int code_s, int creg_s, int halo_s, uint8_t* codes,
           unsigned long long* count) {
  const int2 it_ = items[block];
  const SceneDesc& S = sd[it_.x];
  const int p = S.p, q = S.q, L = S.L, npairs = S.npairs, R = S.rows, ntiles = S.ntiles,
            H = S.halo, split = S.psplit;
  const gfloat* __restrict__ X = gslot<const gfloat>(S, x_s);
  const gfloat* __restrict__ mu = gslot<const gfloat>(S, mu_s);
  gfloat* sig = gslot<gfloat>(S, sig_s);   // updated in place
  gu8* scode = gslot<gu8>(S, code_s);      // updated in place
  constexpr int KW = 2 * K + 1;
  constexpr int NP = KW * KW;
  extern __shared__ float4 lds4[];
  float* lds = reinterpret_cast<float*>(lds4);
  const int q4 = q >> 2;
  float* Ms = lds;                      // (R + 2K) x q        mu(., tau), rows r0-K .. r0+R+K-1
  float* Xs = Ms + (R + 2 * K) * q;     // (R + H) x q         X rows r0-H .. r0+R-1
  float* Cs = Xs + (R + H) * q;         // (R + H) x q         adjoint accumulator

  // work item y = (tile * split + part) * L + band: bands fastest, so that the workgroups
  // resident together share the tile's thresholds in L2
  const int tp = it_.y / L;
  const int c = it_.y - tp * L;
  const int tile = tp / split;
  const int part = tp - tile * split;
  const int n_begin = part * npairs / split, n_end = (part + 1) * npairs / split;
  const int r0 = tile * R;
  const int rows = min(R, p - r0);
  const size_t plane = (size_t)p * q;
  gfloat* creg = part == 0 ? gslot<gfloat>(S, creg_s)
                           : gslot<gfloat>(S, B_CSPLIT) + (size_t)(part - 1) * L * plane;
  gfloat* halo = gslot<gfloat>(S, halo_s) + (size_t)part * L * ntiles * H * q;
  const gfloat* Xc = X + (size_t)c * plane;

  int row[ITEMS], col[ITEMS], seg[ITEMS];
  bool ok[ITEMS];
  float4 xv[ITEMS], cp[ITEMS];
#pragma unroll
  for (int m = 0; m < ITEMS; ++m) {
    const int it = threadIdx.x + NT * m;
    row[m] = it / q4;
    col[m] = (it - row[m] * q4) * 4;
    seg[m] = 4 * (it & ~63);            // float offset of the wave's segment in a plane
    ok[m] = row[m] < rows;
    cp[m] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
  unsigned open_written = 0;            // open items this wave wrote (wave-uniform)

  // Sigma' as [L][tiles][Npairs][|P|][R][q]: the whole state of one workgroup is one
  // contiguous stream, each (tau, k) slab of it R*q floats.
  const size_t kstride = (size_t)R * q;             // between patch offsets
  const size_t tstride = (size_t)NP * kstride;      // between shifts
  const size_t tile_off = ((size_t)c * ntiles + tile) * (size_t)npairs * tstride;
  // without the pipeline below (several items per thread): code bytes of the next patch
  // row to process, requested one row ahead
  unsigned cbn[KW][ITEMS];
  auto load_codes = [&](size_t row_off) {
#pragma unroll
    for (int k2 = 0; k2 < KW; ++k2) {
      const gu8* cbp = scode + ((row_off + (size_t)k2 * kstride) >> 2);
#pragma unroll
      for (int m = 0; m < ITEMS; ++m)
        cbn[k2][m] = __builtin_nontemporal_load(cbp + (threadIdx.x + NT * m));
    }
  };
  // the open items' float4s of a patch row, from the waves' packed runs: a wave with open
  // items loads on every lane (lanes past the tile from the start of the segment): the closed
  // lanes' slots lie inside the open run, so no extra line is read and no lane branches
  auto load_open = [&](size_t row_off, const unsigned (&cbx)[KW][ITEMS],
                       float4 (&sx)[KW][ITEMS]) {
#pragma unroll
    for (int k2 = 0; k2 < KW; ++k2) {
      const gfloat* vb = sig + row_off + (size_t)k2 * kstride;
#pragma unroll
      for (int m = 0; m < ITEMS; ++m) {
        const bool open = ok[m] && cbx[k2][m] >= 16u;
        const unsigned long long bal = __builtin_amdgcn_ballot_w64(open);
        const unsigned slot = __builtin_amdgcn_mbcnt_hi(
            (unsigned)(bal >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0u));
        if (bal) sx[k2][m] = ld_nt(vb + (seg[m] + 4u * (ok[m] ? slot : 0u)));
      }
    }
  };

  // the shifts of this workgroup, one per lane, 64 at a time, packed as (tau1 << 16 | tau2):
  // read before the planes' requests, since a load inside the shift loop would wait for
  // every request issued before it
  int tau_lane = 0;
  auto tau_fetch = [&](int n0) {
    const int j = n0 + (int)(threadIdx.x & 63);
    const int2 tj = j < n_end ? tau_at(S, j) : make_int2(0, 0);
    tau_lane = (tj.x << 16) | (tj.y & 0xffff);
  };

  // With one item per thread the planes are software-pipelined.  The planes of a workgroup
  // form one contiguous sequence over its shifts (plane x at base + x kstride); while plane x
  // is updated, the open float4s of plane x + D and the code bytes of plane x + D + E are in
  // flight.  These requests are issued on every path (a wave with no open item reads the
  // start of its segment; past the last plane the last plane is read again, unused), so the
  // number of memory operations after each is fixed and the wait for plane x leaves the later
  // ones in flight.  A plane is read only before it is written: its own requests come D and
  // D + E planes earlier, repeats of the last plane up to its own update.
  // A request that is still in flight at the end of a shift must land in the register its
  // plane is read from in the next one: a copy there would wait for the request (and, the
  // counter being in order, for all before it).  The registers turn over once per shift of NP
  // planes, so this needs D + E <= NP; at 3 x 3 D = E = 6 (12 > 9) drained the pipeline at
  // the end of every shift.
  constexpr bool PIPE = !FIRST && ITEMS == 1;
  constexpr int D = K == 0 ? 6 : K == 1 ? 4 : 5, E = D;
  const int nplanes = (n_end - n_begin) * NP;
  const size_t base = tile_off + (size_t)n_begin * tstride;
  // The ring's indices are constants only where the planes of a shift are unrolled, which is
  // past the compiler's limit for the 81 planes of 9 x 9 with branch codes: there the registers
  // move on by one per plane (as a ring they lay in scratch memory: gradient of 256 x 256 x 16,
  // 9x9/3x3, 6 iterations, 6.83 ms, like this 3.13 ms).
  constexpr bool RING = NP > D + E && !(CODES && K > 3);
  uint8_t cq[RING ? NP : D + E + 1];   // code bytes of planes x .. x + D + E (kept as bytes: a
                                       // widening at the loop's back edge would wait)
  float4 sb[RING ? NP : D + 1];        // open float4s of planes x .. x + D
  unsigned long long oq[RING ? NP : D + 1];   // and their ballots
  // With one item per thread the workgroup's code bytes and its packed values are one buffer
  // each, plane x at byte x * cstride and 16 x * cstride (at most 11 664 planes of 4 KB: 32
  // bits): a lane's address is the plane offset (a scalar that grows by one stride per plane)
  // plus a 32-bit lane offset, with no 64-bit arithmetic.  Accesses past the range are
  // dropped and read zero, which is what the lanes past the tile get (coff).
  constexpr bool BUF = ITEMS == 1;
  constexpr int POL = POLICY != kSweepCached ? kCacheNT : 0;    // packed values
  constexpr int CPOL = POLICY == kSweepStream ? kCacheNT : 0;   // code bytes
  const unsigned cstride = (unsigned)(kstride >> 2);
  const unsigned clast = (unsigned)max(nplanes - 1, 0) * cstride;   // the last plane
  const __amdgpu_buffer_rsrc_t crs = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(uint8_t*)(scode + (base >> 2)), (short)0, BUF ? nplanes * (int)cstride : 0,
      kRawBufferFlags);
  const __amdgpu_buffer_rsrc_t vrs = __builtin_amdgcn_make_buffer_rsrc(
      (void*)(float*)(sig + base), (short)0, BUF ? 16 * nplanes * (int)cstride : 0,
      kRawBufferFlags);
  const __amdgpu_buffer_rsrc_t brs = __builtin_amdgcn_make_buffer_rsrc(
      CODES ? (void*)(codes + (base >> 2)) : nullptr, (short)0,
      BUF && CODES ? nplanes * (int)cstride : 0, kRawBufferFlags);
  const unsigned coff = ok[0] ? threadIdx.x : 0x7fffffffu;
  // requests of the plane at code offset co, or of the last plane if that is before it
  auto pipe_codes = [&](unsigned co) -> uint8_t {
    return __builtin_amdgcn_raw_buffer_load_b8(crs, coff, min(co, clast), CPOL);
  };
  // each lane without an open item reads the slot after the open lanes below it, inside the
  // segment
  const unsigned segb = 4u * (unsigned)seg[0];  // byte offset of the wave's segment
  auto pipe_open = [&](unsigned co, unsigned cx, unsigned long long& bal) -> float4 {
    bal = __builtin_amdgcn_ballot_w64(cx >= 16u);
    const unsigned slot = __builtin_amdgcn_mbcnt_hi(
        (unsigned)(bal >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0u));
    const v4u_t v = __builtin_amdgcn_raw_buffer_load_b128(vrs, segb + 16u * slot,
                                                          16u * min(co, clast), POL);
    return make_float4(__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z),
                       __uint_as_float(v.w));
  };
  // what the lane's wave may store of the segment of item it: its items in the plane, and the
  // position of the workgroup's first item in a 64-byte block
  const unsigned okn = (unsigned)(R * q4), a0 = (unsigned)(base >> 2) & 3u;
  auto seg_cap = [&](int m) -> unsigned {
    const unsigned s0 = __builtin_amdgcn_readfirstlane(threadIdx.x + NT * m) & ~63u;
    return s0 < okn ? min(64u, okn - s0) : 0u;
  };
  unsigned cap[ITEMS];
  unsigned long long okmask[ITEMS];
#pragma unroll
  for (int m = 0; m < ITEMS; ++m) {
    cap[m] = seg_cap(m);
    okmask[m] = __builtin_amdgcn_ballot_w64(ok[m]);
  }
  const unsigned lane = threadIdx.x & 63u;

  // thresholds mu(., tau) of the tile rows and their K halo, (R + 2K) q4 float4s per shift.
  // When they fit MUR per thread their offsets in a mu plane are computed once (no integer
  // division per shift), and for patches of at most 3 x 3 they are requested one shift ahead
  // into registers, so their latency hides behind the previous shift (at 5 x 5 the extra
  // registers would cost a wave per SIMD).
  constexpr int MUR = K <= 1 ? 2 : 3;
  constexpr bool MU_AHEAD = K <= 1;
  const int mu_n4 = (R + 2 * K) * q4;
  const bool mu_hoist = mu_n4 <= MUR * NT;
  int mu_off[MUR];
  float4 mv[MU_AHEAD ? MUR : 1];
#pragma unroll
  for (int u = 0; u < MUR; ++u) {
    const int e = threadIdx.x + u * NT;
    const int rr = e / q4, c4 = e - rr * q4;
    int gr = (r0 - K + rr) % p;
    if (gr < 0) gr += p;
    mu_off[u] = e < mu_n4 ? gr * q + 4 * c4 : -1;
  }
  auto mu_fetch = [&](int n) {
    const gfloat* mun = mu + (size_t)n * plane;
#pragma unroll
    for (int u = 0; u < MUR; ++u)
      if (mu_off[u] >= 0) mv[MU_AHEAD ? u : 0] = ldg4(mun + mu_off[u]);
  };
  // All first requests before the first wait: the codes of the first planes, the shifts, the
  // first thresholds and the tile of X; then the values that the codes place.
  if constexpr (PIPE) {
    if (nplanes > 0) {
#pragma unroll
      for (int i = 0; i < D + E; ++i) cq[i] = pipe_codes(i * cstride);
    }
  } else if (!FIRST && n_begin < n_end) {
    load_codes(tile_off + (size_t)n_begin * tstride);
  }
  tau_fetch(n_begin);
  if (MU_AHEAD && mu_hoist && n_begin < n_end) mu_fetch(n_begin);
  constexpr int XU = 4;
  for (int e0 = threadIdx.x; e0 < (R + H) * q4; e0 += XU * NT) {
    float4 t[XU];
#pragma unroll
    for (int u = 0; u < XU; ++u) {
      const int e = min(e0 + u * NT, (R + H) * q4 - 1);
      const int rr = e / q4, c4 = e - rr * q4;
      int gr = (r0 - H + rr) % p;
      if (gr < 0) gr += p;
      t[u] = ldg4(Xc + (size_t)gr * q + 4 * c4);
    }
#pragma unroll
    for (int u = 0; u < XU; ++u) {
      const int e = e0 + u * NT;
      if (e < (R + H) * q4) {
        reinterpret_cast<float4*>(Xs)[e] = t[u];
        reinterpret_cast<float4*>(Cs)[e] = make_float4(0.f, 0.f, 0.f, 0.f);
      }
    }
  }
  if constexpr (PIPE) {
    if (nplanes > 0) {
#pragma unroll
      for (int i = 0; i < D; ++i) sb[i] = pipe_open(i * cstride, cq[i], oq[i]);
    }
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < ITEMS; ++m)
    xv[m] = ok[m] ? *reinterpret_cast<const float4*>(Xs + (row[m] + H) * q + col[m])
                  : make_float4(0.f, 0.f, 0.f, 0.f);

  unsigned co = 0;                      // code offset of the current plane
  for (int n = n_begin; n < n_end; ++n) {
    if (n > n_begin && ((n - n_begin) & 63) == 0) tau_fetch(n);
    const int tpk = __builtin_amdgcn_readlane(tau_lane, (n - n_begin) & 63);
    const int2 t = make_int2(tpk >> 16, (int)(short)(tpk & 0xffff));
    __syncthreads();  // the previous shift's reads of Ms and updates of Cs are done
    if (MU_AHEAD && mu_hoist) {
#pragma unroll
      for (int u = 0; u < MUR; ++u)
        if (mu_off[u] >= 0) reinterpret_cast<float4*>(Ms)[threadIdx.x + u * NT] = mv[u];
      if (n + 1 < n_end) mu_fetch(n + 1);
    } else if (mu_hoist) {
      // all of a thread's requests first (lanes without a float4 read the plane's first),
      // then the stores: one wait per shift
      const gfloat* mun = mu + (size_t)n * plane;
      float4 mt[MUR];
#pragma unroll
      for (int u = 0; u < MUR; ++u) mt[u] = ldg4(mun + max(mu_off[u], 0));
#pragma unroll
      for (int u = 0; u < MUR; ++u)
        if (mu_off[u] >= 0) reinterpret_cast<float4*>(Ms)[threadIdx.x + u * NT] = mt[u];
    } else {
      const gfloat* mun = mu + (size_t)n * plane;
      for (int e = threadIdx.x; e < mu_n4; e += NT) {
        const int rr = e / q4, c4 = e - rr * q4;
        int gr = (r0 - K + rr) % p;
        if (gr < 0) gr += p;
        reinterpret_cast<float4*>(Ms)[e] = ldg4(mun + (size_t)gr * q + 4 * c4);
      }
    }
    __syncthreads();

    float4 g[ITEMS], A[ITEMS];
#pragma unroll
    for (int m = 0; m < ITEMS; ++m) {
      const float* xr = Xs + (row[m] + H - t.x) * q;
      float sh[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        int cc = col[m] + e - t.y;
        cc = cc < 0 ? cc + q : (cc >= q ? cc - q : cc);
        sh[e] = xr[cc];
      }
      g[m] = make_float4(xv[m].x - sh[0], xv[m].y - sh[1], xv[m].z - sh[2], xv[m].w - sh[3]);
      A[m] = make_float4(0.f, 0.f, 0.f, 0.f);
    }

    const size_t n_off = tile_off + (size_t)n * tstride;
#pragma unroll
    for (int k1 = -K; k1 <= K; ++k1) {
      // thresholds mu(j + k, tau) for k2 in [-K, K]: columns col-4 .. col+7 of row + k1, the
      // float4 before and after wrapped around the full-width row (no padding columns, so
      // four workgroups fit a CU's LDS at q = 512)
      float mw[ITEMS][12];
#pragma unroll
      for (int m = 0; m < ITEMS; ++m) {
        const float4* mr = reinterpret_cast<const float4*>(Ms + (row[m] + K + k1) * q);
        const int c4 = col[m] >> 2;
        const float4 a = mr[c4 == 0 ? q4 - 1 : c4 - 1], b = mr[c4],
                     d = mr[c4 + 1 == q4 ? 0 : c4 + 1];
        mw[m][0] = a.x; mw[m][1] = a.y; mw[m][2] = a.z; mw[m][3] = a.w;
        mw[m][4] = b.x; mw[m][5] = b.y; mw[m][6] = b.z; mw[m][7] = b.w;
        mw[m][8] = d.x; mw[m][9] = d.y; mw[m][10] = d.z; mw[m][11] = d.w;
      }
      const size_t row_off = n_off + (size_t)((k1 + K) * KW) * kstride;
      // without the pipeline (several items per thread), the old state of this patch row's
      // planes: the code bytes (loaded with the previous row), then the open items' float4s
      // from the waves' packed runs; the next row's code bytes (or the next shift's first
      // row) are requested before this row's values
      unsigned cb[KW][ITEMS];
      float4 s[KW][ITEMS];
      if (!FIRST && !PIPE) {
#pragma unroll
        for (int k2 = 0; k2 < KW; ++k2)
#pragma unroll
          for (int m = 0; m < ITEMS; ++m) cb[k2][m] = cbn[k2][m];
        if (k1 < K || n + 1 < n_end) load_codes(row_off + (size_t)KW * kstride);
        load_open(row_off, cb, s);
      }
#pragma unroll
      for (int k2 = 0; k2 < KW; ++k2) {
        const size_t pl_off = row_off + (size_t)k2 * kstride;
        gfloat* vb = sig + pl_off;
        gu8* cbp = scode + (pl_off >> 2);
#pragma unroll
        for (int m = 0; m < ITEMS; ++m) {
          const int o = 4 + (k2 - K);  // window index of column col + (k2 - K)
          const float mu4[4] = {mw[m][o + 0], mw[m][o + 1], mw[m][o + 2], mw[m][o + 3]};
          float sv[4];
          unsigned cbv = 0;  // this plane's old code byte and open float4
          float4 s4 = make_float4(0.f, 0.f, 0.f, 0.f);
          bool open = false;
          if constexpr (PIPE) {
            if constexpr (RING) {
              const int kk = (k1 + K) * KW + k2;   // plane of the shift: known when unrolled
              cq[(kk + D + E) % NP] = pipe_codes(co + (D + E) * cstride);
              sb[(kk + D) % NP] =
                  pipe_open(co + D * cstride, cq[(kk + D) % NP], oq[(kk + D) % NP]);
              cbv = cq[kk];
              s4 = sb[kk];
              open = __builtin_amdgcn_inverse_ballot_w64(oq[kk]);
            } else {
              cq[D + E] = pipe_codes(co + (D + E) * cstride);
              sb[D] = pipe_open(co + D * cstride, cq[D], oq[D]);
              cbv = cq[0];
              s4 = sb[0];
              open = __builtin_amdgcn_inverse_ballot_w64(oq[0]);
#pragma unroll
              for (int i = 0; i < D + E; ++i) cq[i] = cq[i + 1];
#pragma unroll
              for (int i = 0; i < D; ++i) {
                sb[i] = sb[i + 1];
                oq[i] = oq[i + 1];
              }
            }
          } else if (!FIRST) {
            cbv = cb[k2][m];
            s4 = s[k2][m];
            open = ok[m] && cbv >= 16u;
          }
          if (FIRST) {
            sv[0] = sv[1] = sv[2] = sv[3] = 0.f;
          } else {
            // sv = -Sigma' = clip(V_old, +-mu): the stored value, or on the threshold mu with
            // the sign of V_old (bit e), i.e. mu's magnitude under that sign bit
            const float st[4] = {s4.x, s4.y, s4.z, s4.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              const float on = __uint_as_float((cbv >> e) << 31 | __float_as_uint(mu4[e]));
              sv[e] = open ? st[e] : on;
            }
          }
          const float gv[4] = {g[m].x, g[m].y, g[m].z, g[m].w};
          float nv[4], acc[4];
          unsigned code = 0, branch = 0;
          float vv[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float v = gv[e] + sv[e];
            const float cl = __builtin_amdgcn_fmed3f(v, -mu4[e], mu4[e]);
            vv[e] = v;
            acc[e] = __builtin_fmaf(-2.f, cl, v);
            nv[e] = cl;
          }
          // the code byte, shifted in one bit at a time (alignbit(c, x, 31) = c << 1 | x >> 31):
          // the off flags (sign bits of |V| - mu) of elements 3..0, then the signs of V
#pragma unroll
          for (int e = 3; e >= 0; --e)
            code = __builtin_amdgcn_alignbit(code, __float_as_uint(fabsf(vv[e]) - mu4[e]), 31);
#pragma unroll
          for (int e = 3; e >= 0; --e)
            code = __builtin_amdgcn_alignbit(code, __float_as_uint(vv[e]), 31);
          if (CODES) {
            // the branches from the code byte: on the threshold with the sign clear (1) or set
            // (2), bits e spread to bits 2e.  A wave with a V or a mu that is not a number (mu from
            // a NaN in Y_h), or with both 0, takes them from the comparisons
            unsigned w = (~code >> 4 & ~code & 15u) | (~code >> 4 & code & 15u) << 16;
            w = (w | w << 2) & 0x00330033u;
            w = (w | w << 1) & 0x00550055u;
            branch = w | w >> 15;
            bool odd = false;
#pragma unroll
            for (int e = 0; e < 4; ++e) odd |= !(fabsf(vv[e]) > -mu4[e]);
            if (__builtin_amdgcn_ballot_w64(odd)) {
              branch = 0;
#pragma unroll
              for (int e = 0; e < 4; ++e)
                branch |= (fabsf(vv[e]) < mu4[e] ? 0u : (vv[e] > 0.f ? 1u : (vv[e] < 0.f ? 2u : 3u)))
                          << (2 * e);
            }
          }
          A[m].x += acc[0];   // lanes past the tile too: they never use it
          A[m].y += acc[1];
          A[m].z += acc[2];
          A[m].w += acc[3];
          // (in place: the additions must not sink to their use at the end of the shift)
          asm volatile("" : "+v"(A[m].x), "+v"(A[m].y), "+v"(A[m].z), "+v"(A[m].w));
          const unsigned long long bal = __builtin_amdgcn_ballot_w64(code >= 16u) & okmask[m];
          const unsigned nopen = (unsigned)__builtin_popcountll(bal);
          open_written += nopen;
          if (bal) {
            // the open lanes in lane order, then lanes without an open item up to the end of
            // the last 64-byte block (at most the segment's items)
            const unsigned slot = __builtin_amdgcn_mbcnt_hi(
                (unsigned)(bal >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0u));
            const unsigned at = BUF ? co + a0 : (unsigned)(pl_off >> 2);
            const unsigned lim = min(((at + nopen + 3u) & ~3u) - at, cap[m]);
            const unsigned to =
                __builtin_amdgcn_inverse_ballot_w64(bal) ? slot : nopen + lane - slot;
            if (to < lim) {
              if constexpr (BUF) {
                const v4u_t w = {__float_as_uint(nv[0]), __float_as_uint(nv[1]),
                                 __float_as_uint(nv[2]), __float_as_uint(nv[3])};
                __builtin_amdgcn_raw_buffer_store_b128(w, vrs, segb + 16u * to, 16u * co, POL);
              } else {
                st_nt(vb + (seg[m] + 4u * to), make_float4(nv[0], nv[1], nv[2], nv[3]));
              }
            }
          }
          if constexpr (BUF) {
            __builtin_amdgcn_raw_buffer_store_b8((uint8_t)code, crs, coff, co, CPOL);
            if (CODES)
              __builtin_amdgcn_raw_buffer_store_b8((uint8_t)branch, brs, coff, co, 0);
          } else if (ok[m]) {
            __builtin_nontemporal_store((uint8_t)code, cbp + (threadIdx.x + NT * m));
          }
          co += cstride;
        }
      }
    }

#pragma unroll
    for (int m = 0; m < ITEMS; ++m) {
      if (!ok[m]) continue;
      cp[m].x += A[m].x; cp[m].y += A[m].y; cp[m].z += A[m].z; cp[m].w += A[m].w;
      float* cr = Cs + (row[m] + H - t.x) * q;
      const float a4[4] = {A[m].x, A[m].y, A[m].z, A[m].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        int cc = col[m] + e - t.y;
        cc = cc < 0 ? cc + q : (cc >= q ? cc - q : cc);
        cr[cc] -= a4[e];
      }
    }
  }
  if (count && (threadIdx.x & 63) == 0) {
    // spread over kCountSlots counters a cache line apart: waves that end together on one
    // address would queue behind each other at the L2
    const unsigned slot = (block * (NT / 64) + threadIdx.x / 64) % kCountSlots;
    atomicAdd(count + (size_t)slot * kCountStride, (unsigned long long)open_written);
  }
  __syncthreads();

  gfloat* cregc = creg + (size_t)c * plane + (size_t)r0 * q;
#pragma unroll
  for (int m = 0; m < ITEMS; ++m) {
    if (!ok[m]) continue;
    const float4 acc = *reinterpret_cast<const float4*>(Cs + (row[m] + H) * q + col[m]);
    stg4(cregc + (size_t)row[m] * q + col[m],
         make_float4(2.f * (cp[m].x + acc.x), 2.f * (cp[m].y + acc.y), 2.f * (cp[m].z + acc.z),
                     2.f * (cp[m].w + acc.w)));
  }
  if (H > 0) {
    gfloat* hb = halo + ((size_t)c * ntiles + tile) * H * q;
    for (int e = threadIdx.x; e < H * q4; e += NT) {
      const float4 v = reinterpret_cast<const float4*>(Cs)[e];
      stg4(hb + 4 * e, make_float4(2.f * v.x, 2.f * v.y, 2.f * v.z, 2.f * v.w));
    }
  }
}

template <int K, int ITEMS, int NT, bool FIRST, bool CODES, int POLICY>
__global__ void __launch_bounds__(NT)
sweep_kernel(const SceneDesc* __restrict__ sd, const int2* __restrict__ items, int x_s, int mu_s,
             int sig_s, int code_s, int creg_s, int halo_s, uint8_t* codes,
             unsigned long long* count) {
  sweep_body<K, ITEMS, NT, FIRST, CODES, POLICY>(sd, items, blockIdx.x, x_s, mu_s, sig_s, code_s,
                                                 creg_s, halo_s, codes, count);
}

// The sweep (the first nsw workgroups) and the P-update (the rest), which read X and write
// disjoint buffers.  A P-update of its own is bound by latency up to 256 x 256 (13.9 us for 40 MB at
// 31 bands) and costs a launch; here its workgroups fill the end of the sweep, whose last
// workgroups leave CUs idle.  At K = 1, 2 and 3 it stays within the sweep's registers, so the sweep's
// occupancy is the same; at K = 0 it takes 97 where the sweep alone takes 94, four waves per SIMD
// instead of five, and is still the faster.  Per iteration of a solve, two launches and one:
// 64 x 64 x 8 (graph) 36.2 and 32.2 us, 128 x 128 x 31 65 and 58, 192 x 256 x 31 fused-S 88 and 80,
// 256 x 256 x 31 103 and 96; with K = 0, 3x3 window, 128 x 128 x 31 50 and 43, 256 x 256 x 31 85 and
// 81; with K = 3 105 and 96, 249 and 238.  With the P-update's workgroups first, 88 -> 90 and
// 103 -> 102.
template <int K, bool CODES, int POLICY>
__global__ void __launch_bounds__(256)
sweep_pu_kernel(const SceneDesc* __restrict__ sd, const int2* __restrict__ items, int x_s,
                int mu_s, int sig_s, int code_s, int creg_s, int halo_s, uint8_t* codes,
                PuSlots sl, int nsw, int lhm) {
  const int b = (int)blockIdx.x - nsw;
  if (b >= 0) {
    extern __shared__ float4 lds4[];
    float* part = reinterpret_cast<float*>(lds4);
    if (lhm == 1) pupdate_body<1, 4, true>(sd[0], b / 4, b % 4, sl, part);
    else pupdate_body<4, 4, true>(sd[0], b / 4, b % 4, sl, part);
    return;
  }
  sweep_body<K, 1, 256, false, CODES, POLICY>(sd, items, blockIdx.x, x_s, mu_s, sig_s, code_s,
                                              creg_s, halo_s, codes, nullptr);
}

// ---- sweep kernel end

// Tiles and launch shapes.  A tile is 1024 * items pixels (items = 1, 2 or 4: the fewest with
// one full image row per tile), i.e. 256 * items float4 items, on a workgroup of 256 threads
// with `items` items each; the layout of Sigma' and of its codes depends on the tile only
// (segments of 64 items).  For 3 x 3 patches at 256 x 256 x 31 this shape was faster than
// 128 threads with two items each (89 against 154 VGPRs at the time: five waves per SIMD
// instead of three; 20-iteration solve 2.88 against 3.16 ms).

template <int K, int ITEMS, int NT, bool FIRST, bool CODES, int POLICY>
int launch_k(const Batch& B, const Group& g, int x, int mu, int sig, int creg, int halo,
             uint8_t* codes, unsigned long long* count, hipStream_t s) {
  auto kern = sweep_kernel<K, ITEMS, NT, FIRST, CODES, POLICY>;
  hipLaunchKernelGGL(kern, dim3(g.nitems), dim3(NT), g.lds, s, B.d_desc, g.d_items, x, mu,
                     sig, (int)B_SCODE, creg, halo, codes, count);
  NLPR_LAUNCH_CHECK("sweep_kernel");
  return NLPR_OK;
}

// Allow the sweep's dynamic LDS beyond the default limit (done when a batch is built, not
// during graph capture).  The branch-recording variant exists for single-item tiles.
template <typename Kern>
int lds_limit(Kern kern) {
  NLPR_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                   hipFuncAttributeMaxDynamicSharedMemorySize,
                                   (int)kMaxSweepLds));
  return NLPR_OK;
}

template <int K, int ITEMS, int NT, int POLICY>
int set_lds_limit() {
  int rc;
  if ((rc = lds_limit(sweep_kernel<K, ITEMS, NT, true, false, POLICY>)) ||
      (rc = lds_limit(sweep_kernel<K, ITEMS, NT, false, false, POLICY>)))
    return rc;
  if constexpr (ITEMS == 1)
    if ((rc = lds_limit(sweep_kernel<K, ITEMS, NT, true, true, POLICY>)) ||
        (rc = lds_limit(sweep_kernel<K, ITEMS, NT, false, true, POLICY>)))
      return rc;
  if constexpr (K <= 3 && ITEMS == 1)
    if ((rc = lds_limit(sweep_pu_kernel<K, false, POLICY>)) ||
        (rc = lds_limit(sweep_pu_kernel<K, true, POLICY>)))
      return rc;
  return NLPR_OK;
}

template <int K>
int set_lds_limit_items(int items) {
  constexpr int NT = kSweepThreads;
  int rc;
  switch (items) {
    case 1:
      if ((rc = set_lds_limit<K, 1, NT, kSweepCached>()) ||
          (rc = set_lds_limit<K, 1, NT, kSweepCodesCached>()))
        return rc;
      return set_lds_limit<K, 1, NT, kSweepStream>();
    case 2: return set_lds_limit<K, 2, NT, kSweepStream>();
    default: return set_lds_limit<K, 4, NT, kSweepStream>();
  }
}

// g.key1 = tile items; the cache policy of single-item tiles
inline int policy_of(const Group& g, const uint8_t* codes) { return codes ? g.grad_policy : g.policy; }
template <int K, bool FIRST, int POLICY>
int launch_single(const Batch& B, const Group& g, int x, int mu, int sig, int creg, int halo,
                  uint8_t* codes, unsigned long long* count, hipStream_t s) {
  constexpr int NT = kSweepThreads;
  return codes ? launch_k<K, 1, NT, FIRST, true, POLICY>(B, g, x, mu, sig, creg, halo, codes, count, s)
               : launch_k<K, 1, NT, FIRST, false, POLICY>(B, g, x, mu, sig, creg, halo, codes, count, s);
}

template <int K, bool FIRST>
int launch_items(const Batch& B, const Group& g, int x, int mu, int sig, int creg, int halo,
                 uint8_t* codes, unsigned long long* count, hipStream_t s) {
  constexpr int NT = kSweepThreads;
  if (codes && g.key1 != 1) {
    set_error("sweep: branch codes need single-item tiles");
    return NLPR_ERR_UNSUPPORTED_SHAPE;
  }
  switch (g.key1) {
    case 1:
      switch (policy_of(g, codes)) {
        case kSweepCached:
          return launch_single<K, FIRST, kSweepCached>(B, g, x, mu, sig, creg, halo, codes, count, s);
        case kSweepCodesCached:
          return launch_single<K, FIRST, kSweepCodesCached>(B, g, x, mu, sig, creg, halo, codes, count, s);
        default:
          return launch_single<K, FIRST, kSweepStream>(B, g, x, mu, sig, creg, halo, codes, count, s);
      }
    case 2:
      return launch_k<K, 2, NT, FIRST, false, kSweepStream>(B, g, x, mu, sig, creg, halo, nullptr, count, s);
    default:
      return launch_k<K, 4, NT, FIRST, false, kSweepStream>(B, g, x, mu, sig, creg, halo, nullptr, count, s);
  }
}

template <int K, bool CODES, int POLICY>
int launch_kpu(const Batch& B, const Group& g, const Group& gp, const PuSlots& sl, int x, int mu,
               int sig, int creg, int halo, uint8_t* codes, hipStream_t s) {
  auto kern = sweep_pu_kernel<K, CODES, POLICY>;
  const size_t lds = std::max(g.lds, sizeof(float) * pupdate_lds_floats(4, 4));
  hipLaunchKernelGGL(kern, dim3(g.nitems + 4 * gp.nitems), dim3(256), lds, s, B.d_desc, g.d_items, x, mu,
                     sig, (int)B_SCODE, creg, halo, codes, sl, g.nitems, gp.key0);
  NLPR_LAUNCH_CHECK("sweep_pu_kernel");
  return NLPR_OK;
}

template <int K>
int launch_pu_k(const Batch& B, const Group& g, const Group& gp, const PuSlots& sl, int x, int mu,
                int sig, int creg, int halo, uint8_t* codes, hipStream_t s) {
  switch (policy_of(g, codes)) {
    case kSweepCached:
      return codes ? launch_kpu<K, true, kSweepCached>(B, g, gp, sl, x, mu, sig, creg, halo, codes, s)
                   : launch_kpu<K, false, kSweepCached>(B, g, gp, sl, x, mu, sig, creg, halo, codes, s);
    case kSweepCodesCached:
      return codes ? launch_kpu<K, true, kSweepCodesCached>(B, g, gp, sl, x, mu, sig, creg, halo, codes, s)
                   : launch_kpu<K, false, kSweepCodesCached>(B, g, gp, sl, x, mu, sig, creg, halo, codes, s);
    default:
      return codes ? launch_kpu<K, true, kSweepStream>(B, g, gp, sl, x, mu, sig, creg, halo, codes, s)
                   : launch_kpu<K, false, kSweepStream>(B, g, gp, sl, x, mu, sig, creg, halo, codes, s);
  }
}

}  // namespace

// One scene without a second stream (kForkPixelBands), tiles of one item per thread, and bands
// that four threads per pixel can hold; timing keeps the stages apart.
bool sweep_pu(const Batch& B) {
  if (B.scenes.size() != 1 || B.side || B.timing) return false;
  const auto &gs = B.groups[KD_SWEEP], &gp = B.groups[KD_PIXEL];
  return gs.size() == 1 && gs[0].nitems && gs[0].key1 == 1 && gs[0].key0 <= 3 &&
         gp.size() == 1 && gp[0].key0 <= 4 && B.scenes[0]->Lx <= 4 * kPuKeep;
}

int launch_sweep_pu(const Batch& B, const PuSlots& sl, int x, int mu, int sig, int creg, int halo,
                    hipStream_t s, uint8_t* codes) {
  const Group &g = B.groups[KD_SWEEP][0], &gp = B.groups[KD_PIXEL][0];
  if (const int rc = check_table(g)) return rc;
  switch (g.key0) {
    case 0: return launch_pu_k<0>(B, g, gp, sl, x, mu, sig, creg, halo, codes, s);
    case 1: return launch_pu_k<1>(B, g, gp, sl, x, mu, sig, creg, halo, codes, s);
    case 2: return launch_pu_k<2>(B, g, gp, sl, x, mu, sig, creg, halo, codes, s);
    default: return launch_pu_k<3>(B, g, gp, sl, x, mu, sig, creg, halo, codes, s);
  }
}

SweepShape choose_sweep_shape(int p, int q, int K, int halo) {
  SweepShape sh{};
  int items = 1;
  while (items < 4 && kSweepThreads * items * 4 < q) items *= 2;
  sh.items = items;
  const int per_block = kSweepThreads * items * 4;  // pixels per workgroup
  sh.rows = std::max(1, std::min(p, per_block / q));
  sh.ntiles = ceil_div(p, sh.rows);
  sh.halo = halo;
  sh.lds = (size_t)((sh.rows + 2 * K) * q + 2 * (sh.rows + halo) * q) * sizeof(float);
  return sh;
}

size_t sweep_sigma_bytes(const SweepShape& sh, int q, int L, int npairs, int npatch) {
  return (size_t)L * sh.ntiles * npairs * npatch * sh.rows * q * sizeof(float);
}

// Workgroups per (tile, band): 1 unless the scene has fewer (tile, band) pairs than the GPU
// has CUs, then enough parts of W+ (at most one shift each) for about one workgroup per CU.
int choose_pair_split(int blocks, int npairs) {
  constexpr int kCus = 256;
  if (blocks <= 0 || blocks >= kCus || npairs <= 1) return 1;
  return std::min(npairs, (kCus + blocks - 1) / blocks);
}

// Cache policy of a sweep launch over `state` bytes of dual state (capacity) with `planes` planes
// per band, in a batch with `all` bytes of state and `pbands` pixel-bands.  The lines lie where they
// are measured, on an MI355X:
// - up to 384 MB, of which an iteration touches about half, the state stays in the 256 MB
//   Infinity Cache from one sweep to the next when it is not streamed; sweep per launch:
//   256 x 256 x 31 3x3/3x3 (312 MB) 65 us streamed, 54 us cached; 192 x 256 x 31 (233 MB) 51 and
//   40 us; but 256 x 256 x 46 (461 MB) 3.74 and 3.79 ms per 20-iteration solve, and
//   1024 x 1024 x 4 with a 5x5 window (1.9 GB) 597 and 727 us.  The launches of a batch share that
//   cache: 24 scenes with 3x3 and 5x5 patches, 294 and 310 MB in two launches, 2.27 ms per solve
//   streamed, 2.77 cached.
// - below 2^19 pixel-bands the ten planes that the other stages pass on stay in the 32 MB of L2,
//   from which a cached state, read or written, pushes them.  Solves of 10 iterations there, streamed
//   and cached, in us: 64 x 64 x 8 5x5/7x7 (80 MB) 496 and 563, 128 x 128 x 31 3x3/3x3 (74 MB) 500
//   and 534, 96 x 96 x 8 9x9/3x3 (97 MB) 621 and 702; from about 192 MB of state on cached is the
//   better as often as not: 192 x 192 x 8 5x5/5x5 (359 MB) 1282 and 1229, 16 x 512 x 6 7x7/7x7
//   (234 MB) 1110 and 937, 64 x 64 x 8 9x9/7x7 (258 MB) 970 and 1001.  Above 2^19:
//   256 x 256 x 16 3x3/3x3 (153 MB) 734 and 713, 512 x 512 x 3 3x3/3x3 (115 MB) 818 and 789.
// - otherwise the values are streamed.  The code bytes (1/17 of the state, read and written
//   64 bytes per wave) gain from the caches, which also join stores that are not whole 64-byte
//   blocks: 108 x 144 x 31 5x5/5x5 151 us streamed, 139 us cached; 512 x 512 x 16 5x5/11x11
//   2.91 and 2.83 ms.  But they push the dense planes out of the caches, which counts where the
//   sweep does not carry the iteration: 256 x 256 x 124 3x3/3x3 (1.2 GB) 9.1 ms per solve
//   streamed, 9.5 ms cached.  So the codes are streamed for more than 1 GB of state in planes
//   so few (under 200) that the other stages matter.
int sweep_policy(size_t state, int planes, size_t all, size_t pbands) {
  const bool l2 = pbands < (size_t)1 << 19;
  if (all <= (size_t)384 << 20 && (!l2 || all >= (size_t)192 << 20)) return kSweepCached;
  if (state <= (size_t)1 << 30 || planes >= 200) return kSweepCodesCached;
  return kSweepStream;
}

int sweep_blocks(const Plan& P) { return P.sweep.ntiles * P.Lx * P.sweep.split; }

int sweep_prepare(int K, int items) {
  switch (K) {
    case 0: return set_lds_limit_items<0>(items);
    case 1: return set_lds_limit_items<1>(items);
    case 2: return set_lds_limit_items<2>(items);
    case 3: return set_lds_limit_items<3>(items);
    case 4: return set_lds_limit_items<4>(items);
    default: set_error("sweep: unsupported patch radius"); return NLPR_ERR_UNSUPPORTED_SHAPE;
  }
}

int launch_sweep(const Batch& B, int x, int mu, int sig, int creg, int halo, bool first,
                 hipStream_t s, uint8_t* codes, unsigned long long* count) {
  for (const Group& g : B.groups[KD_SWEEP]) {
    if (!g.nitems) continue;
    int rc = check_table(g);
    if (rc) return rc;
    switch (g.key0) {
#define NLPR_SW(KK)                                                                            \
  case KK:                                                                                     \
    rc = first ? launch_items<KK, true>(B, g, x, mu, sig, creg, halo, codes, count, s)        \
               : launch_items<KK, false>(B, g, x, mu, sig, creg, halo, codes, count, s);      \
    break;
      NLPR_SW(0)
      NLPR_SW(1)
      NLPR_SW(2)
      NLPR_SW(3)
      NLPR_SW(4)
#undef NLPR_SW
      default:
        set_error("sweep: unsupported patch radius");
        return NLPR_ERR_UNSUPPORTED_SHAPE;
    }
    if (rc) return rc;
  }
  return NLPR_OK;
}

// ------------------------------------------------------------------ decoding Sigma'
namespace {
// Dense Sigma' of bands [c0, c0 + nb) from the coded state: out[c - c0][n][k][i1][i2] =
// Sigma'_{tau_n, k}(i1, i2) of band c (image rows, not tiles).  One thread per float4 item of a
// plane, in the sweep's order (ITEMS * NT items per plane, 64 per wave), so every wave sees
// the packed run of the segment the sweep's wave wrote.
__global__ void __launch_bounds__(256)
sigma_expand_kernel(const SceneDesc* __restrict__ sd, const gfloat* __restrict__ sig,
                    const gu8* __restrict__ scode, const gfloat* __restrict__ mu, int c0, int nb,
                    int per_plane, gfloat* __restrict__ out) {
  const SceneDesc& S = sd[0];
  const int p = S.p, q = S.q, K = S.K, npairs = S.npairs, npatch = S.npatch, R = S.rows,
            ntiles = S.ntiles, q4 = q >> 2, KW = 2 * K + 1;
  const size_t g = (size_t)blockIdx.x * 256 + threadIdx.x;
  const size_t planes = (size_t)nb * ntiles * npairs * npatch;
  const bool live = g < planes * per_plane;        // whole waves are live or not
  const size_t pi = live ? g / per_plane : 0;
  const int it = (int)(g - pi * per_plane);
  // plane index pi = ((cl * ntiles + tile) * npairs + n) * npatch + k
  const int k = (int)(pi % npatch);
  const size_t r1 = pi / npatch;
  const int n = (int)(r1 % npairs);
  const size_t r2 = r1 / npairs;
  const int tile = (int)(r2 % ntiles);
  const int cl = (int)(r2 / ntiles);
  const int r0 = tile * R, rows = min(R, p - r0);
  const int row = it / q4, col = (it - row * q4) * 4;
  const bool ok = live && row < rows;
  const size_t pl_off = (((size_t)(c0 + cl) * ntiles + tile) * npairs + n) * npatch * ((size_t)R * q) +
                        (size_t)k * R * q;
  const unsigned cb = ok ? scode[(pl_off >> 2) + it] : 0u;
  const bool open = ok && cb >= 16u;
  const unsigned long long bal = __builtin_amdgcn_ballot_w64(open);
  const unsigned slot = __builtin_amdgcn_mbcnt_hi((unsigned)(bal >> 32),
                                                  __builtin_amdgcn_mbcnt_lo((unsigned)bal, 0u));
  if (!ok) return;
  float v[4];
  if (open) {
    const float4 t = ldg4(sig + pl_off + 4 * (it & ~63) + 4 * slot);   // clip(V) = -Sigma'
    v[0] = -t.x; v[1] = -t.y; v[2] = -t.z; v[3] = -t.w;
  } else {
    const int k1 = k / KW - K, k2 = k % KW - K;
    const int mr = (r0 + row + k1 + p) % p;
    const gfloat* mun = mu + (size_t)n * p * q + (size_t)mr * q;
    for (int e = 0; e < 4; ++e) {
      const float m = mun[(col + e + k2 + q) % q];
      v[e] = (cb >> e) & 1u ? m : -m;
    }
  }
  const size_t o = ((((size_t)cl * npairs + n) * npatch + k) * p + (r0 + row)) * q + col;
  stg4(out + o, make_float4(v[0], v[1], v[2], v[3]));
}
}  // namespace

int launch_sigma_expand(const Batch& B, const float* sig, const uint8_t* codes, const float* mu,
                        int c0, int nb, float* out, hipStream_t s) {
  const Plan& P = *B.scenes[0];
  const int per_plane = kSweepThreads * P.sweep.items;
  const size_t total = (size_t)nb * P.sweep.ntiles * P.npairs * P.npatch * per_plane;
  if (total == 0) return NLPR_OK;
  const size_t blocks = (total + 255) / 256;
  if (blocks > 0x7fffffffu) {
    set_error("sigma expand: too many bands at once");
    return NLPR_ERR_INVALID_ARG;
  }
  hipLaunchKernelGGL(sigma_expand_kernel, dim3((unsigned)blocks), dim3(256), 0, s, B.d_desc,
                     (const gfloat*)sig, (const gu8*)codes, (const gfloat*)mu, c0, nb, per_plane,
                     (gfloat*)out);
  NLPR_LAUNCH_CHECK("sigma_expand_kernel");
  return NLPR_OK;
}

}  // namespace nlpr
