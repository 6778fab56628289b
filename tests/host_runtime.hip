// A HIP runtime of the host alone, for tests of the library's host code
// without a GPU: device memory is host memory, kernels do not run, and every
// launch is recorded with its kernel's name, shape and dynamic LDS.  Linked
// with the host objects of the library in place of the real runtime
// (host_runtime.py).
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <utility>
#include <vector>

#include "cosmo_internal.h"

namespace {

struct Launch {
  std::string name;
  dim3 grid, block;
  size_t lds;
  int allowed;   // dynamic LDS the kernel had been allowed on the device, -1: the default
  cosmo::TeamView team;
  cosmo::View<double> view;   // (a float32 View is laid out the same)
};

std::map<const void *, std::string> &names() {   // (kernels are registered before this file's globals exist)
  static std::map<const void *, std::string> n;
  return n;
}
std::map<std::pair<const void *, int>, int> allowed;
std::vector<Launch> launches;
std::vector<float> elapsed;
size_t elapsed_at = 0;
int device = 0;
struct Config {
  dim3 grid, block;
  size_t lds;
  hipStream_t st;
} config;

hipError_t record(const void *f, dim3 grid, dim3 block, void **args, size_t lds) {
  Launch l{names()[f], grid, block, lds, -1, {}, {}};
  const auto a = allowed.find({f, device});
  if (a != allowed.end()) l.allowed = a->second;
  if (l.name.find("k_pcg_team") != std::string::npos) {
    std::memcpy(static_cast<void *>(&l.view), args[0], sizeof l.view);
    l.team = *static_cast<const cosmo::TeamView *>(args[1]);
  }
  launches.push_back(l);
  return hipSuccess;
}

}  // namespace

extern "C" {

// ---- what the tests read ---------------------------------------------------------

void host_runtime_reset() { launches.clear(); }
void host_runtime_device(int d) { device = d; }
void host_runtime_elapsed(const float *ms, int n) {   // the event pairs' times, in turn
  elapsed.assign(ms, ms + n);
  elapsed_at = 0;
}
int host_runtime_launches() { return (int)launches.size(); }
const char *host_runtime_launch(int i, long long *out) {   // grid, block, dynamic LDS, allowed dynamic LDS
  const Launch &l = launches[i];
  out[0] = l.grid.x;
  out[1] = l.block.x;
  out[2] = (long long)l.lds;
  out[3] = l.allowed;
  return l.name.c_str();
}
void host_runtime_team(int i, long long *out) {   // the team tables of a k_pcg_team launch
  const cosmo::TeamView &t = launches[i].team;
  const cosmo::View<double> &v = launches[i].view;
  const auto at = [](const void *p) { return (long long)reinterpret_cast<uintptr_t>(p); };
  const long long f[] = {v.B, v.n_tot, t.slices, t.max_n, t.cap_off, t.cap, at(t.colcut), at(v.dcol),
                         at(t.dense_cut), at(t.dense_list), at(t.dense_slot), t.dense_slots,
                         at(t.used), at(t.uses), at(t.At_loc), at(v.At_rowptr), at(v.At_col), at(t.sliceA), at(v.rowsA),
                         v.m_tot};
  std::memcpy(out, f, sizeof f);
}

// ---- the runtime -----------------------------------------------------------------

struct {
  int x;
} dummy_module;
void **__hipRegisterFatBinary(const void *) { return reinterpret_cast<void **>(&dummy_module); }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned int, void *, void *, dim3 *, dim3 *,
                           int *) {
  names()[f] = name;
}
void __hipRegisterVar(void **, void *, char *, const char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t st) {
  config = {grid, block, lds, st};
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *st) {
  *grid = config.grid;
  *block = config.block;
  *lds = config.lds;
  *st = config.st;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t) {
  return record(f, grid, block, args, lds);
}
hipError_t hipLaunchCooperativeKernel(const void *f, dim3 grid, dim3 block, void **args, unsigned int lds, hipStream_t) {
  return record(f, grid, block, args, lds);
}
hipError_t hipFuncSetAttribute(const void *f, hipFuncAttribute, int value) {
  allowed[{f, device}] = value;
  return hipSuccess;
}
hipError_t hipFuncGetAttributes(hipFuncAttributes *a, const void *) {
  *a = {};
  a->sharedSizeBytes = 5632;
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) {
  *n = 4;
  return hipSuccess;
}
hipError_t hipMalloc(void **p, size_t n) {
  *p = std::calloc(1, n ? n : 1);
  return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void *p) {
  std::free(p);
  return hipSuccess;
}
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind, hipStream_t) {
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void **, const void *) { return hipErrorInvalidValue; }
hipError_t hipGetDevice(int *d) {
  *d = device;
  return hipSuccess;
}
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 1;
  return hipSuccess;
}
hipError_t hipGetDeviceProperties(hipDeviceProp_t *p, int) {   // (a macro names the current version)
  std::memset(static_cast<void *>(p), 0, sizeof *p);
  std::strcpy(p->gcnArchName, "gfx950:sramecc+:xnack-");
  p->multiProcessorCount = 256;
  return hipSuccess;
}
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned int) {
  *s = nullptr;
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned int) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
  *g = reinterpret_cast<hipGraph_t>(&dummy_module);
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t, hipGraphNode_t *, char *, size_t) {
  *e = reinterpret_cast<hipGraphExec_t>(&dummy_module);
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) {
  *e = nullptr;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned int) {
  *e = nullptr;
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) {
  *ms = elapsed.empty() ? 1.f : elapsed[elapsed_at++ % elapsed.size()];
  return hipSuccess;
}

}  // extern "C"
