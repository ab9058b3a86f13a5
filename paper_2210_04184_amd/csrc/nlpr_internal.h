// Internal declarations of libnlpr: scene plans, the batch every launch runs over, device
// scene descriptors and kernel launchers.
//
// Every kernel runs over a batch of scenes.  Block b of a launch has a work item (scene, local
// block), takes the scene's sizes, tables and buffers from the device descriptor sd[scene] and
// does the work of that local block.  The items of a batch of several scenes are read from a
// table, items[b]; a single-scene plan is a batch of one, whose items follow from b (work_item),
// the sweep's and its adjoint's excepted.  Kernels reach buffers through slots
// (SceneDesc::buf[slot]), so the same kernel serves the solve and the per-stage entry
// points with different buffers.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <string>
#include <vector>

#include "nlpr.h"

namespace nlpr {

constexpr int kMaxLh = 16;
constexpr int kMaxK = 4;
constexpr int kMaxSw = 8;
constexpr int kMaxBlurRadius = 16;
constexpr int kMaxFFTFactors = 24;
constexpr int kMaxFFTLen = 4096;
constexpr size_t kMaxSweepLds = 160 * 1024;  // LDS per workgroup on gfx950
constexpr int kMaxLs = 32;                    // bands of X with a subspace basis

// One-dimensional FFT of length n = product of fac[] (each 2, 3, 4 or 8).
// tw[m] = exp(-2 pi i m / n), m in [0, n).
struct LineFFT {
  int n;
  int nfac;
  int fac[kMaxFFTFactors];
  const float2* tw;
};

// Buffer slots of a scene descriptor.
enum Slot {
  B_YL = 0, B_YH, B_Z, B_SIGMA, B_MU, B_C, B_L1, B_L2, B_BX, B_W1, B_W2, B_F, B_HALO, B_TMP,
  B_OUT,     // Z = X E when a subspace basis is used (B_Z is then the X iterate)
  B_YLE,     // Y_l E^T, [Ls][p/d][q/d]
  B_YLP,     // Y_l E^+, [Ls][p/d][q/d]
  B_L1O, B_L2O,   // where the P-update writes Lambda1, Lambda2 when not in place (checkpoints)
  B_CSPLIT,  // regulariser planes of sweep parts 1 .. psplit-1, [psplit-1][L][p][q]
  B_SCODE,   // Sigma' codes: one byte per float4 item of Sigma' (sweep.hip)
  // reverse mode (single scene): adjoints of the iteration's variables and the outputs
  B_GZ,      // Z' (input)
  B_GC,      // C'
  B_GCP,     // C' of the backward step before (the sweep adjoint rebuilds Sigma'' from it)
  B_GL1,     // Lambda1'' (sampled pixels)
  B_GSIG,    // Sigma'' (coded: float4 items with an element inside the threshold, packed)
  B_GX,      // X'
  B_GW1,     // W1' = B C', then BX' (they differ on the sampled pixels)
  B_GXP,     // X' of the P-update, which is also -Lambda2''
  B_GXR,     // X' of the sweep (+ halo rows in B_GHALO)
  B_GHALO,
  B_GMUP,    // mu' partial tiles [L][ntiles][Npairs][R + 2K][q]
  B_GMU,     // mu' [Npairs][p][q]
  B_GE,      // e' [Npairs][p][q]
  B_GYL, B_GYH,   // Y_l', Y_h' (outputs)
  B_GPART,   // FP64 partial sums
  B_COUNT
};

// Everything a kernel needs to know about one scene.  Lives in device memory.
struct SceneDesc {
  int p, q, L, Lh, d, r, K, npairs, npatch;
  int rows, ntiles, halo;          // sweep tiling
  int psplit;                      // sweep workgroups per (tile, band), each over a part of W+
  int fq_tpl, fq_lpb;              // row FFT: threads per line, lines per block
  int fp_tpl, fp_cb;               // column FFT: threads per line, columns per block
  int init_zero, unweighted;
  int subspace, Lz;                // basis in use; bands of Z (L is the number of X bands)
  int fused;                       // S inside the X-system (no P1)
  float rho, inv_1prho, mu_scale, inv_h2;
  LineFFT fp, fq;
  const int2* taus;
  const float* invden;
  const float* blur;
  const float* bsep;               // u then v (2r+1 each) of a rank-one blur b = u v^T, else null
  const float* R;
  const float* G;
  const float* E;                  // [Ls][Lz]
  const float* Ep;                 // E^+ = E^T (E E^T)^{-1}, [Lz][Ls]
  const float* M;                  // (E E^T + rho I)^{-1}, [Ls][Ls]
  // fused-S X-update tables, [p][q]: 1/(a p q), b^/a, gamma conj(b^)/(a p q)
  const float* fia;
  const float2* fu;
  const float2* fv;
  // monitor: partial sums [mon_npix][4] (data_l, data_h, r1^2, r2^2 per pixel block), then
  // [mon_nreg] (regulariser per (shift, tile) block), then the trace [points][8]
  double* mon;
  int mon_npix, mon_nreg;
  double rho_d, lam1_d, lam_d;
  void* buf[B_COUNT];
};

constexpr int kXcds = 8;             // workgroup b of a launch runs on XCD b % kXcds
constexpr int kSweepThreads = 256;   // workgroup size of the sweep
// Batches of at least this many pixel-bands (summed over scenes) run the P-side of each
// iteration on a second stream, concurrently with the sweep.  Below it the two cross-stream
// waits of an iteration (about 6 and 11 us on MI355X) and the sweep's hold on the CUs cost
// more than the overlap gains (256 x 256 x 31: 2.77 -> 2.90 ms per solve; 512 x 512 x 128:
// 3.03 -> 2.98 s).
constexpr size_t kForkPixelBands = (size_t)1 << 22;
// A single scene above it that can have both in one launch (sweep_pu) does without the second
// stream below this many pixels, unless it has a basis, whose P1 is a launch of its own.  Per
// iteration, second stream and one launch: 512 x 512 x 24 5x5/5x5 1010 and 910 us, 512 x 512 x 31 3x3/3x3
// 345 and 323, 512 x 512 x 16 5x5/11x11 2705 and 2595, 768 x 768 x 8 5x5/5x5 940 and 908; but
// 1024 x 1024 x 4 3x3/3x3 291 and 303, 1024 x 1024 x 8 3x3/5x5 833 and 838, and 512 x 512 with a
// 20-band basis 2491 and 2497 (there the second stream hides the blur too).  These are wall times
// without a tracer.  Under a kernel trace the 1024 x 1024 x 4 scene runs in 450 us per iteration
// with the P-side inside the sweep, so some of the second stream's cost lies outside the kernels; the
// line holds as long as that does.
constexpr size_t kForkPixels = (size_t)1 << 20;
// Cache policies of the sweep's dual state: nothing, the packed values, or all of it bypass
// the caches (non-temporal).
enum SweepPolicy { kSweepCached = 0, kSweepCodesCached = 1, kSweepStream = 2 };
// open-item counters of one sweep launch (timing plans): kCountSlots, kCountStride apart
constexpr int kCountSlots = 64;
constexpr int kCountStride = 16;

struct SweepShape {
  int rows;      // tile height R
  int items;     // tile size in units of 256 float4 items (1024 pixels): 1, 2 or 4
  int ntiles;    // ceil(p / R)
  int halo;      // rows above the tile reached by the adjoint scatter (max tau1)
  int split;     // workgroups per (tile, band), each over a contiguous part of W+
  size_t lds;    // dynamic LDS bytes
};

struct FftShape {
  int q_tpl, q_lpb, q_bs;   // row passes: threads per line, lines per block, block size
  int p_tpl, p_cb, p_bs;    // column pass: threads per line, columns per block, block size
};

// One scene: parameters, device tables and its part of the workspace.
struct Plan {
  nlpr_params prm{};
  void* arena = nullptr;          // the device tables below, one allocation
  int npairs = 0;
  int npatch = 0;
  std::vector<int32_t> taus;      // W+ (tau1, tau2 pairs)
  int2* d_taus = nullptr;
  float* d_invden = nullptr;      // [p][q], 1 / (den * p * q)
  float2* d_tw_p = nullptr;
  float2* d_tw_q = nullptr;
  LineFFT fp{}, fq{};
  FftShape fft{};
  float* d_blur = nullptr;          // (2r+1)^2 taps, then u and v when blur_separable
  bool blur_separable = false;
  float* d_R = nullptr;
  float* d_G = nullptr;
  int Lx = 0;                     // bands of X: Ls with a basis, else L
  float* d_E = nullptr;           // [Ls][L]
  float* d_Ep = nullptr;          // [L][Ls]
  float* d_M = nullptr;           // [Ls][Ls]
  float* d_Rt = nullptr;          // E R, [Ls][Lh]
  double* d_mon = nullptr;        // monitor partials and trace (monitor_every > 0)
  float* d_fia = nullptr;         // fused-S tables (NLPR_FUSED_S)
  float2* d_fu = nullptr;
  float2* d_fv = nullptr;
  int mon_points = 0;             // records per solve
  SweepShape sweep{};
  // workspace layout relative to the scene's base
  size_t off[B_COUNT] = {};
  size_t sz[B_COUNT] = {};
  size_t ws_bytes = 0;
};

// A launch: the work items of the scenes that share its template parameters.
constexpr size_t kNoTable = ~size_t(0);
struct Group {
  const int2* d_items = nullptr;   // the work items, in the batch's arena
  size_t table = kNoTable;         // and where they start there
  int nitems = 0;
  int block = 256;
  size_t lds = 0;
  int key0 = 0, key1 = 0;   // sweep: K, items per thread
  int policy = 0;           // sweep: cache policy of the dual state
  int grad_policy = 0;      // the same in reverse mode: branch-recording sweep and its adjoint
};

enum Kind { KD_WEIGHTS = 0, KD_PLANE, KD_CONV, KD_PIXEL, KD_SWEEP, KD_ROWS, KD_COLS,
            KD_LOWRES,   // one thread per low-resolution pixel of scenes with a basis
            KD_COMPOSE,  // one thread per pixel of scenes with a basis
            KD_MONREG,   // monitor regulariser: (shift, 32 x 64 tile) of scenes with a window
            KD_SCENE,    // one workgroup per scene
            KD_MUPLANE,  // one thread per (shift, pixel): single-scene reverse mode
            KD_WBWD,     // weights adjoint: (shift, 16 x 64 tile), single-scene reverse mode
            KD_COUNT };

struct Batch {
  int device = 0;
  uint32_t flags = 0;              // flags shared by every scene (INIT_ZERO, STATE_IN, ...)
  int iters = 0;
  int monitor_every = 0;           // shared by every scene
  int mon_last = 0;                // monitor records written by the last solve
  hipEvent_t done_ev = nullptr;    // recorded after each solve
  // second stream of the iteration (large batches only): the P-side (blur, P-update and the
  // part of the right-hand side that does not wait for the sweep) runs on it while the sweep
  // runs on the solve's stream
  hipStream_t side = nullptr;
  hipEvent_t fork_ev = nullptr, join_ev = nullptr;
  std::vector<Plan*> scenes;       // owned
  std::vector<size_t> base;        // workspace base of each scene
  size_t ws_bytes = 0;
  void* arena = nullptr;           // work-item tables, descriptors, flag, counters
  std::vector<int2> tables;        // the tables while the batch is built
  SceneDesc* d_desc = nullptr;     // device descriptors, one per scene (and kDescRing more)
  SceneDesc* h_desc = nullptr;     // pinned staging copy (more than one scene)
  std::vector<SceneDesc> uploaded; // what d_desc holds
  bool desc_valid = false;
  hipEvent_t upload_ev = nullptr;
  std::vector<Group> groups[KD_COUNT];
  unsigned long long* d_counts = nullptr;  // open Sigma' items written per sweep (timing)
  int* d_flag = nullptr;           // finite check: first checked iteration with NaN / Inf
  int nonfinite_iter = -1;         // what the last checked solve found (-1: nothing)
  // graph
  bool use_graph = false;
  hipGraphExec_t graph = nullptr;
  uint32_t graph_key = 0;
  // timing
  bool timing = false;
  std::vector<hipEvent_t> ev_pool;
  size_t ev_used = 0;
  struct Rec { int stage; size_t a, b; };
  std::vector<Rec> recs;
  double acc_ms[NLPR_STAGE_COUNT] = {};
  int64_t acc_n[NLPR_STAGE_COUNT] = {};
};

// The work-item table a launch passes (work_item): none for a single scene.
inline const int2* items_of(const Batch& B, const Group& g) {
  return B.scenes.size() == 1 ? nullptr : g.d_items;
}

// ---- error plumbing (api.hip)
void set_error(const std::string& msg);
#define NLPR_HIP_TRY(expr)                                                          \
  do {                                                                              \
    hipError_t e_ = (expr);                                                         \
    if (e_ != hipSuccess) {                                                         \
      ::nlpr::set_error(std::string(#expr) + ": " + hipGetErrorString(e_));         \
      return NLPR_ERR_HIP;                                                          \
    }                                                                               \
  } while (0)
#define NLPR_LAUNCH_CHECK(what)                                                     \
  do {                                                                              \
    hipError_t e_ = hipGetLastError();                                              \
    if (e_ != hipSuccess) {                                                         \
      ::nlpr::set_error(std::string("launch of ") + (what) + ": " + hipGetErrorString(e_)); \
      return NLPR_ERR_HIP;                                                          \
    }                                                                               \
  } while (0)

// The sweep and its adjoint index their table whatever it is: their items are in an order that
// the workgroup index does not give (sweep_items).
inline int check_table(const Group& g) {
  if (g.d_items) return NLPR_OK;
  set_error("sweep: no work-item table");
  return NLPR_ERR_HIP;
}

__host__ __device__ inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

// Pointers read from a descriptor are generic (flat); kernels convert them to the global
// address space so the compiler emits global loads, and scalar loads for uniform addresses.
// Vector elements move through clang ext-vector types (HIP's vector structs cannot be
// copied out of an address-space-qualified object).
typedef __attribute__((address_space(1))) float gfloat;
typedef __attribute__((address_space(1))) uint8_t gu8;
typedef __attribute__((address_space(1))) double gdouble;
// small tables read at wave-uniform addresses: scalar loads whatever stores surround them
typedef __attribute__((address_space(4))) const float cfloat;
typedef float v2f_t __attribute__((ext_vector_type(2)));
typedef float v4f_t __attribute__((ext_vector_type(4)));
typedef int v2i_t __attribute__((ext_vector_type(2)));
typedef unsigned v4u_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(1))) v2f_t gv2f;
typedef __attribute__((address_space(1))) v4f_t gv4f;
typedef __attribute__((address_space(1))) v2i_t gv2i;
// cache policy of a buffer access: non-temporal
constexpr int kCacheNT = 2;
// last word of a raw byte-addressed buffer resource: 32-bit data format (bits 15-18 = 4),
// no stride, no swizzle; offsets are bytes from the base
constexpr int kRawBufferFlags = 0x00020000;
__device__ __forceinline__ const gfloat* as_global(const float* p) { return (const gfloat*)p; }
__device__ __forceinline__ cfloat* as_constant(const float* p) { return (cfloat*)p; }
__device__ __forceinline__ gfloat* as_global(float* p) { return (gfloat*)p; }
template <typename G>
__device__ __forceinline__ G* gslot(const SceneDesc& S, int k) {
  return k < 0 ? nullptr : (G*)(S.buf[k]);
}
__device__ __forceinline__ float2 ldg2(const gfloat* p) {
  const v2f_t v = *(const gv2f*)p;
  return make_float2(v.x, v.y);
}
__device__ __forceinline__ void stg2(gfloat* p, float2 a) {
  const v2f_t v = {a.x, a.y};
  *(gv2f*)p = v;
}
__device__ __forceinline__ float4 ldg4(const gfloat* p) {
  const v4f_t v = *(const gv4f*)p;
  return make_float4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void stg4(gfloat* p, float4 a) {
  const v4f_t v = {a.x, a.y, a.z, a.w};
  *(gv4f*)p = v;
}
// A workgroup's work item.  The launches of a single scene need no table (items is null): the
// scene is 0 and the local block is the workgroup index, or, where the table is ordered by
// XCD, the same position of that order (xcd_append from position 0).  A table costs a dependent
// load in front of everything a kernel does, which is most of a microsecond of a launch.
__device__ __forceinline__ int2 work_item(const int2* items, unsigned b) {
  return items ? items[b] : make_int2(0, (int)b);
}
__device__ __forceinline__ int2 work_item_xcd(const int2* items) {
  const unsigned b = blockIdx.x, n = gridDim.x, x = b & 7u;
  return items ? items[b] : make_int2(0, (int)(x * (n >> 3) + min(x, n & 7u) + (b >> 3)));
}
__device__ __forceinline__ int2 tau_at(const SceneDesc& S, int n) {
  const v2i_t v = ((const gv2i*)S.taus)[n];
  return make_int2(v.x, v.y);
}

// ---- plan precompute (dense.hip); runs once per scene on the null stream
int launch_precompute(Plan& P);

// ---- local work-item counts per scene for each kind of launch
int weights_blocks(const Plan& P);
int plane_blocks(const Plan& P);      // elementwise over [L][p][q], 256 elements per block
int conv_blocks(const Plan& P);
int pixel_blocks(const Plan& P);      // one thread per pixel
int rows_blocks(const Plan& P);
int cols_blocks(const Plan& P);
int sweep_blocks(const Plan& P);
size_t weights_lds(const Plan& P);
size_t conv_lds(const Plan& P);
int conv_class(int r);                // template bound of a blur radius: 1, 2, 4, 8 or 16
size_t rows_lds(const Plan& P);
size_t cols_lds(const Plan& P);

// ---- batched kernels: each launches the groups of one kind with buffer slots (< 0: none)
int launch_weights(const Batch& B, int yh, int mu, hipStream_t s);
int launch_init(const Batch& B, int yl, int ylp, int x0, int l1, int l2, int w2, hipStream_t s);
// reg_mask: bit 0 / 1 mark add1 / add2 as regulariser terms (skipped, like the halo, for
// scenes without a search window); bit 2 marks them as the forward sweep's output, whose
// parts 1 .. psplit-1 (slot B_CSPLIT) and halo parts are then added as well
int launch_conv(const Batch& B, int in, int out, bool transpose, int add1, int add2, int halo,
                int reg_mask, hipStream_t s);
// Buffer slots of the P-update.  Lambda1, Lambda2 are read from slots l1, l2 and written to
// l1o, l2o (the same slots for an update in place).  bx == w1: B X lies in W1 and only the
// sampled pixels' P1, Lambda1 and W1 are updated, the others being P1 + Lambda1 = B X; the caller
// knows their Lambda1 to be zero (a solve that started from zero keeps it so).  bxo >= 0: the
// slot that also takes B X where P1 is updated.
struct PuSlots {
  int x, bx, yl, yh, l1, l2, w1, w2, l1o, l2o, bxo;
};
int launch_pupdate(const Batch& B, const PuSlots& sl, hipStream_t s);
// Descriptors for the iterations of a reverse-mode pass, which moves through its checkpoints by
// re-pointing buffer slots: copies of the descriptor of scene 0, each with its own pointers in
// up to six slots, kDescRing at a time behind it.  (A launch before each iteration that
// re-pointed the slots of the one descriptor took 4.5 us and its place in the queue twice per
// iteration: gradient of 256 x 256 x 31 5.15 -> 5.04 ms.)
constexpr int kDescRing = 32;
struct SlotTable {
  int n = 0, count = 0;            // slots, descriptors
  int slot[6];
  void* ptr[kDescRing][6];
};
int launch_desc_ring(const Batch& B, const SlotTable& t, hipStream_t s);
int launch_set_desc(const Batch& B, const SceneDesc& d, hipStream_t s);   // scene 0's descriptor
int lh_class(int Lh);                // pupdate template class of a guide-band count: 1, 4 or 16
// threads per pixel of a P-update launch over `pixels` pixels in all: 4 (bands split) below
// 131072, where one thread per pixel would leave most of the GPU idle, else 1
inline int pixel_split(size_t pixels) { return pixels < 131072 ? 4 : 1; }
int lowres_blocks(const Plan& P);
// in-place negation of n4 float4 values with non-temporal 16-byte accesses (reference stream)
int launch_stream_rmw(float* buf, size_t n4, hipStream_t s);
int launch_stream_chunks(float* buf, size_t chunk4, int nchunks, int bands, int planes,
                         size_t lds, hipStream_t s);
// with a subspace basis: Y_l E^T and Y_l E^+ (once per solve), the P1-update on sampled
// pixels, and Z = X E
int launch_project(const Batch& B, int yl, int yle, int ylp, hipStream_t s);
int launch_p1_subspace(const Batch& B, int bx, int yle, int l1, int w1, hipStream_t s);
int launch_compose(const Batch& B, int x, int z, hipStream_t s);
// monitor (monitor.hip): objective terms and primal residuals after iteration `iter`,
// written to record `point` of each scene's trace
int monreg_blocks(const Plan& P);
size_t monreg_lds(const Plan& P);
int monitor_points(int iters, int every);
int launch_monitor(const Batch& B, int point, int iter, hipStream_t s);
// reverse mode (adjoint.hip); single-scene batches
size_t sweep_bwd_lds(const Plan& P);
size_t weights_bwd_lds(const Plan& P);
int weights_bwd_blocks(const Plan& P);
size_t mubar_partial_elems(const Plan& P);
int sweep_bwd_prepare(int K);
// codes: the forward sweep's threshold branches of the iteration (launch_sweep's codes);
// pcodes, cbp: those of the iteration whose backward step ran last and its C' (null on the
// first backward step, whose incoming Sigma'' is zero)
struct PbSlots {                   // buffer slots of the P-update's adjoint
  int x, bx, yl, yh, l1, l2, w1b, w2b, l1b, xp, gyl, gyh, part;
};
int launch_sweep_bwd(const Batch& B, int cb, const uint8_t* codes, int sb, int xr, int halo,
                     int mup, const uint8_t* pcodes, int cbp, const PbSlots& sl, hipStream_t s);
int pupdate_bwd_split(const Plan& P);
int launch_mubar_reduce(const Batch& B, int mup, int mub, hipStream_t s);
int launch_pupdate_bwd(const Batch& B, const PbSlots& sl, hipStream_t s);
int launch_weights_bwd(const Batch& B, int yh, int mub, int eb, int part, int w0, hipStream_t s);
int launch_yh_bwd(const Batch& B, int yh, int eb, int gyh, hipStream_t s);
int launch_upsample_bwd(const Batch& B, int x0b, int gyl, hipStream_t s);
int launch_grad_scalars(const Batch& B, int part, int npix, int nw, double* out, hipStream_t s);
// Finite check every kFiniteEvery iterations (and after the last) with NLPR_CHECK_FINITE.
constexpr int kFiniteEvery = 8;
int launch_finite_clear(int* flag, hipStream_t s);
int launch_finite(const Batch& B, int z, int* flag, int iter, hipStream_t s);
int launch_fill(const Batch& B, int slot, hipStream_t s);   // zero a [L][p][q] slot
int launch_upsample_zero(const Batch& B, int yl, int t, hipStream_t s);   // S^T Y_l / rho
// X = solve(C) (+ add, a [L][p][q] slot, when add >= 0); the fused-S system for fused scenes
int launch_xsolve(const Batch& B, int c, int x, int f, int add, hipStream_t s);
// Sigma' (coded: values in slot `sigma`, code bytes in slot B_SCODE) is updated in place.
// codes (differentiated form, one item per thread): also write each dual element's 2-bit
// threshold branch there, one byte per float4 of Sigma'.  count: if not null, add the
// number of open items written (float4s stored) to *count.
int launch_sweep(const Batch& B, int x, int mu, int sigma, int creg, int halo, bool first,
                 hipStream_t s, uint8_t* codes = nullptr, unsigned long long* count = nullptr);
// the P-update and a sweep but the first in one launch, for batches where sweep_pu
bool sweep_pu(const Batch& B);
int launch_sweep_pu(const Batch& B, const PuSlots& sl, int x, int mu, int sigma, int creg,
                    int halo, hipStream_t s, uint8_t* codes);
// Dense Sigma' of bands [c0, c0 + nb) of scene 0: [nb][Npairs][|P|][p][q]
int launch_sigma_expand(const Batch& B, const float* sig, const uint8_t* codes, const float* mu,
                        int c0, int nb, float* out, hipStream_t s);
// zero n 64-bit counters
int launch_zero_u64(unsigned long long* p, int n, hipStream_t s);
int sweep_prepare(int K, int items);   // kernel attributes; before launches or capture

// ---- shapes and tuning
SweepShape choose_sweep_shape(int p, int q, int K, int halo);
int sweep_policy(size_t state, int planes, size_t all, size_t pbands);
int choose_pair_split(int blocks, int npairs);   // SweepShape.split for `blocks` (tile, band) pairs
size_t sweep_sigma_bytes(const SweepShape& sh, int q, int L, int npairs, int npatch);
int fft_block(int tpl);             // workgroup size of a line FFT with tpl threads per line
int fft_prepare(const Plan& P);     // kernel attributes of the X-update; before its launches
int autotune_fft(Plan& P);          // picks P.fft by timing candidates (cached per (p, q, d if fused))
FftShape default_fft_shape(int p, int q, int d_fused);
void batch_fft_shape(Plan& P);      // P.fft of a scene of a batch of several

}  // namespace nlpr
