// A stand-in for the HIP runtime that has no device: memory is the host's, kernels do not
// run.  With it the library's host code (which kernels it launches, with which grids, what it
// does when a call fails) runs where there is no GPU.  The test's process sees every call it
// asks about through `hook`, which may write to a kernel's memory in the kernel's place.
#include <hip/hip_runtime_api.h>

#include <cstdlib>
#include <cstring>
#include <cxxabi.h>
#include <map>
#include <string>

namespace {
std::map<const void*, std::string> kernels;
std::multimap<size_t, void*> freed;     // blocks given back
std::map<void*, size_t> sizes;
dim3 cfg_grid, cfg_block;
size_t cfg_lds;
hipStream_t cfg_stream;
bool capturing = false;
long events = 0;
// hook(what, detail, args): `what` is a runtime call's name, `detail` a kernel's.  Nonzero:
// the call fails with that error.
typedef int (*hook_t)(const char*, const char*, const long long*, void**);
hook_t hook = nullptr;
hipError_t call(const char* what, const char* detail = "", const long long* dims = nullptr, void** args = nullptr) {
  return hook ? (hipError_t)hook(what, detail, dims, args) : hipSuccess;
}
}  // namespace

extern "C" {
void stub_set_hook(hook_t h) { hook = h; }

hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceSynchronize() { return call("hipDeviceSynchronize"); }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  switch (a) {
    case hipDeviceAttributeMultiprocessorCount: *v = 256; break;
    case hipDeviceAttributeMaxGridDimX: *v = 2147483647; break;
    case hipDeviceAttributeMaxGridDimY:
    case hipDeviceAttributeMaxGridDimZ: *v = 65536; break;
    case hipDeviceAttributeMaxSharedMemoryPerBlock: *v = 163840; break;
    default: *v = 1024;
  }
  return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
  std::memset(p, 0, sizeof *p);
  std::strcpy(p->gcnArchName, "gfx950");
  p->multiProcessorCount = 256;
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
  const hipError_t e = call("hipMalloc");
  if (e != hipSuccess) return e;
  // the smallest block given back that is large enough comes at the same address again
  auto it = freed.lower_bound(n);
  if (it != freed.end()) {
    *p = it->second;
    sizes[*p] = it->first;
    freed.erase(it);
  } else {
    sizes[*p = std::aligned_alloc(4096, (n + 4095) & ~(size_t)4095)] = n;   // untouched pages take no memory
  }
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!p) return hipSuccess;
  auto it = sizes.find(p);
  if (it == sizes.end()) return hipErrorInvalidValue;
  freed.insert({it->second, p});
  sizes.erase(it);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { *p = std::calloc(1, n); return hipSuccess; }
hipError_t hipHostFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  const hipError_t e = call("hipMemcpy");
  if (e == hipSuccess) std::memcpy(d, s, n);
  return e;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) {
  const hipError_t e = call("hipMemcpyAsync");
  if (e == hipSuccess) std::memcpy(d, s, n);
  return e;
}
hipError_t hipMemset(void* d, int v, size_t n) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipPointerGetAttributes(hipPointerAttribute_t* a, const void*) {
  std::memset(a, 0, sizeof *a);
  a->type = hipMemoryTypeDevice;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* mem = std::aligned_alloc(4096, 64 << 20);
  *p = mem;
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "error of the stand-in runtime"; }
hipError_t hipGetLastError() { return call("hipGetLastError"); }

hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = (hipStream_t)std::malloc(8); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t s) { std::free(s); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return call("hipStreamSynchronize"); }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
  const hipError_t e = call("hipStreamBeginCapture");
  capturing = e == hipSuccess;
  return e;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  capturing = false;
  *g = (hipGraph_t)std::malloc(8);
  return call("hipStreamEndCapture");
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  *e = (hipGraphExec_t)std::malloc(8);
  return call("hipGraphInstantiate");
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return call("hipGraphLaunch"); }
hipError_t hipGraphDestroy(hipGraph_t g) { std::free(g); return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t e) { std::free(e); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)++events; return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipFuncGetAttributes(hipFuncAttributes* a, const void*) {
  std::memset(a, 0, sizeof *a);
  a->maxThreadsPerBlock = 1024;
  return hipSuccess;
}

void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*,
                           int*) {
  int status = 0;
  char* text = abi::__cxa_demangle(name, nullptr, nullptr, &status);
  kernels[host] = status == 0 ? text : name;
  std::free(text);
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s) {
  cfg_grid = g;
  cfg_block = b;
  cfg_lds = lds;
  cfg_stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s) {
  *g = cfg_grid;
  *b = cfg_block;
  *lds = cfg_lds;
  *s = cfg_stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t, hipStream_t) {
  const long long dims[5] = {g.x, g.y, g.z, b.x, capturing};
  return call("launch", kernels[f].c_str(), dims, args);
}
}
