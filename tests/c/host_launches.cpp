// The host side of libnlpr without a GPU: this program defines the HIP runtime functions that the
// library calls (its symbols come before those of the HIP library), so that a plan is made and
// used as ever, but memory is host memory and a kernel launch only prints a line:
//   PHASE kernel GRID BLOCK DYNAMIC_LDS LIMIT TABLE
// LIMIT: the dynamic LDS that the kernel may be launched with, 65536 or what hipFuncSetAttribute
// raised it to.  TABLE: whether the kernel's work-item table is null ("-": it takes none).
// PHASE: create, solve, forward or backward; each ends with a line "PHASE status N".
//   host_launches N P Q L LH D R K SW ITERS FLAGS [no-table]
// N > 1: a batch of N such scenes.  no-table: the sweep's table is taken away after create.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "nlpr_internal.h"

namespace {
const char* phase = "load";
std::map<const void*, std::string>& names() {
  static std::map<const void*, std::string> m;
  return m;
}
std::map<const void*, int> limits;
struct Config { dim3 grid, block; size_t lds; hipStream_t stream; } config;
char dummy[64];
template <typename T> T handle() { return reinterpret_cast<T>(dummy); }
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* module = dummy; return &module; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*,
                           void*, void*, void*, int*) {
  names()[host] = name;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  config = {grid, block, lds, stream};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, hipStream_t* stream) {
  *grid = config.grid; *block = config.block; *lds = config.lds; *stream = config.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* host, dim3 grid, dim3 block, void** args, size_t lds,
                           hipStream_t) {
  const int limit = limits.count(host) ? limits[host] : 65536;
  const std::string& name = names()[host];
  const bool items = name.find("9SceneDescEPK15HIP_vector_type") != std::string::npos;
  std::printf("%s %s %u %u %zu %d %s\n", phase, name.c_str(), grid.x, block.x, lds, limit,
              !items ? "-" : *static_cast<void**>(args[1]) ? "table" : "null");
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void* host, hipFuncAttribute attr, int value) {
  if (attr == hipFuncAttributeMaxDynamicSharedMemorySize) limits[host] = value;
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { *p = std::calloc(n, 1); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::calloc(n, 1); return hipSuccess; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void* to, const void* from, size_t n, hipMemcpyKind) {
  std::memcpy(to, from, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* to, const void* from, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(to, from, n);
  return hipSuccess;
}
hipError_t hipMemset(void*, int, size_t) { return hipSuccess; }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void*) {
  *a = {};
  a->type = hipMemoryTypeDevice;
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetSymbolAddress(void** p, const void*) { *p = dummy; return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = handle<hipEvent_t>(); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = handle<hipStream_t>();
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
}

int main(int argc, char** argv) {
  if (argc < 12) return 2;
  int a[11];
  for (int i = 0; i < 11; ++i) a[i] = std::atoi(argv[1 + i]);
  const int n = a[0], w = 2 * a[6] + 1;
  nlpr_params prm{};
  prm.p = a[1]; prm.q = a[2]; prm.L = a[3]; prm.Lh = a[4]; prm.d = a[5]; prm.blur_radius = a[6];
  prm.K = a[7]; prm.Sw = a[8]; prm.iters = a[9]; prm.flags = (uint32_t)a[10];
  prm.lambda = 1e-3; prm.lambda1 = 1.0; prm.rho = 1e-2; prm.h = 0.5;
  const std::vector<float> blur(w * w, 1.f / (w * w)), R(prm.L * prm.Lh, 1.f);
  // device pointers: the library hands them on to kernels only
  char* mem = reinterpret_cast<char*>(uintptr_t(1) << 40);
  float* f = reinterpret_cast<float*>(mem);
  size_t ws = 0;
  phase = "create";
  if (n > 1) {
    const std::vector<nlpr_params> ps(n, prm);
    const std::vector<const float*> bs(n, blur.data()), rs(n, R.data()), in(n, f);
    const std::vector<float*> out(n, f);
    nlpr_batch* b = nullptr;
    std::printf("create status %d\n", nlpr_batch_create(n, ps.data(), bs.data(), rs.data(), nullptr, &b));
    if (!b) return 0;
    nlpr_batch_workspace_size(b, &ws);
    phase = "solve";
    std::printf("solve status %d\n", nlpr_batch_solve(b, in.data(), in.data(), out.data(), mem, ws, nullptr));
    nlpr_batch_destroy(b);
    return 0;
  }
  nlpr_plan* p = nullptr;
  std::printf("create status %d\n", nlpr_plan_create(&prm, blur.data(), R.data(), nullptr, &p));
  if (!p) return 0;
  if (argc > 12 && !std::strcmp(argv[12], "no-table"))
    for (nlpr::Group& g : reinterpret_cast<nlpr::Batch*>(p)->groups[nlpr::KD_SWEEP]) g.d_items = nullptr;
  nlpr_workspace_size(p, &ws);
  phase = "solve";
  std::printf("solve status %d\n", nlpr_solve(p, f, f, f, mem, ws, nullptr));
  size_t ck = 0, gws = 0;
  if (nlpr_grad_sizes(p, &ck, &gws) == NLPR_OK) {
    phase = "forward";
    std::printf("forward status %d\n", nlpr_forward(p, f, f, f, mem, ws, mem, ck, nullptr));
    phase = "backward";
    std::printf("backward status %d\n", nlpr_backward(p, f, f, f, mem, ws, mem, ck, mem, gws, f, f,
                                                      reinterpret_cast<double*>(mem), nullptr));
  }
  nlpr_plan_destroy(p);
  return 0;
}
