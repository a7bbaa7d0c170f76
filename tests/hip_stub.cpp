// A HIP runtime without a device, for tests of the solver's host code on the CPU: device memory is host
// memory, copies are made, kernels are only noted by name. Built as a shared library that carries the
// runtime's soname, so the library under test binds to it (see hip_stub.py).
#include <hip/hip_runtime_api.h>

#include <cstring>
#include <map>
#include <string>
#include <vector>

namespace {
std::map<const void *, std::string> g_names;  // host stub of a kernel -> its mangled name
std::string g_log;                            // launches since the last clear, one a line
std::vector<std::string> g_graph;             // launches of the capture under way
bool g_capturing = false;
int g_uploads = 0, g_fail_upload = -1, g_lds = 160 << 10;
struct Config {
  dim3 grid, block;
  size_t shmem;
  hipStream_t stream;
};
std::vector<Config> g_config;
}  // namespace

extern "C" {

// controls
const char *stub_log() { return g_log.c_str(); }
void stub_clear() { g_log.clear(); }
void stub_fail_upload(int k) {  // the k-th host-to-device copy from now on fails (-1: none)
  g_uploads = 0;
  g_fail_upload = k;
}
int stub_uploads() { return g_uploads; }
void stub_set_lds(int bytes) { g_lds = bytes; }

// what the compiler's host code registers and calls
void **__hipRegisterFatBinary(const void *) {
  static void *h = nullptr;
  return &h;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *fn, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *, int *) {
  g_names[fn] = name;
}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shmem, hipStream_t stream) {
  g_config.push_back({grid, block, shmem, stream});
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shmem, hipStream_t *stream) {
  const Config c = g_config.back();
  g_config.pop_back();
  *grid = c.grid;
  *block = c.block;
  *shmem = c.shmem;
  *stream = c.stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void *fn, dim3, dim3, void **, size_t shmem, hipStream_t) {
  if (shmem > size_t(g_lds)) return hipErrorInvalidValue;
  if (g_capturing) g_graph.push_back(g_names[fn]);
  else g_log += g_names[fn] + "\n";
  return hipSuccess;
}

hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMaxSharedMemoryPerBlock ? g_lds : 256;
  return hipSuccess;
}
hipError_t hipPointerGetAttributes(hipPointerAttribute_t *a, const void *p) {
  std::memset(a, 0, sizeof *a);
  a->type = hipMemoryTypeDevice;
  a->devicePointer = const_cast<void *>(p);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void *dst, const void *src, size_t n, hipMemcpyKind kind, hipStream_t) {
  if (kind == hipMemcpyHostToDevice && g_uploads++ == g_fail_upload) return hipErrorInvalidValue;
  std::memmove(dst, src, n);
  return hipSuccess;
}
hipError_t hipGetDevice(int *d) { return *d = 0, hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "stub error"; }
hipError_t hipGetSymbolAddress(void **p, const void *) { return *p = nullptr, hipErrorInvalidValue; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t) { return *n = 4, hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { return *e = nullptr, hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return *e = nullptr, hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 1.0f, hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return *s = nullptr, hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) {
  g_capturing = true;
  g_graph.clear();
  return hipSuccess;
}
// graphs: an executable is its list of launches, noted when it is replayed
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
  g_capturing = false;
  *g = reinterpret_cast<hipGraph_t>(new std::vector<std::string>(g_graph));
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t *e, hipGraph_t g, hipGraphNode_t *, char *, size_t) {
  *e = reinterpret_cast<hipGraphExec_t>(new std::vector<std::string>(*reinterpret_cast<std::vector<std::string> *>(g)));
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t) {
  for (const std::string &n : *reinterpret_cast<std::vector<std::string> *>(e)) g_log += n + "\n";
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
  delete reinterpret_cast<std::vector<std::string> *>(g);
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t e) {
  delete reinterpret_cast<std::vector<std::string> *>(e);
  return hipSuccess;
}

}  // extern "C"
