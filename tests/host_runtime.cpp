// A stand-in for the HIP runtime library in host-only tests of the library's control flow: memory is the host's, kernels do
// nothing, and every call on a stream or graph is noted.  A call named to host_runtime_fail returns an error once.  Asked about a
// stream, it first reports the next round as the kernels would (HostReport in common.h), while host_runtime_rounds lasts.
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <string>
#include <vector>

namespace {
std::string notes, failing;
uint64_t (*report)[3];          // the last pinned allocation
std::vector<int> seen;          // of every round to report: the second ring's entry
uint32_t reported;
char symbol[1 << 16];
int call(const char* name) {
  notes += name;
  notes += '\n';
  if (failing != name) return 0;
  failing.clear();
  return 2;   // hipErrorOutOfMemory
}
int handle(void** out) {
  *out = std::malloc(1);
  return 0;
}
}  // namespace

extern "C" {
const char* host_runtime_notes() { return notes.c_str(); }
void host_runtime_clear() { notes.clear(); }
void host_runtime_fail(const char* name) { failing = name; }
void host_runtime_rounds(const int* values, int n) { seen.assign(values, values + n), reported = 0; }

int hipMalloc(void** p, size_t n) { return *p = std::calloc(1, n ? n : 1), 0; }
int hipHostMalloc(void** p, size_t n, unsigned) {
  hipMalloc(p, n);
  report = static_cast<uint64_t(*)[3]>(*p);
  return 0;
}
int hipHostGetDevicePointer(void** d, void* h, unsigned) { return *d = h, 0; }
int hipFree(void* p) { return std::free(p), 0; }
int hipHostFree(void* p) { return std::free(p), 0; }
int hipMemcpy(void* d, const void* s, size_t n, int) { return std::memcpy(d, s, n), 0; }
int hipMemset(void* d, int v, size_t n) { return std::memset(d, v, n), 0; }
int hipGetSymbolAddress(void** p, const void*) { return *p = symbol, 0; }
int hipGetDevice(int* d) { return *d = 0, 0; }
int hipSetDevice(int) { return 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "an error"; }
int hipFuncSetAttribute(const void*, int, int) { return 0; }
int hipDeviceSynchronize() { return 0; }
int hipEventCreate(void** e) { return handle(e); }
int hipEventCreateWithFlags(void** e, unsigned) { return handle(e); }
int hipEventDestroy(void* e) { return std::free(e), 0; }
int hipEventElapsedTime(float* ms, void*, void*) { return *ms = 0.f, 0; }
int hipEventRecord(void*, void*) { return 0; }
int hipStreamCreateWithFlags(void** s, unsigned) { return handle(s); }
int hipStreamDestroy(void* s) { return std::free(s), 0; }
int hipStreamWaitEvent(void*, void*, unsigned) { return 0; }
int hipStreamQuery(void*) {
  if (reported < seen.size()) {
    const uint32_t r = reported++, v[3] = {reported < seen.size(), (uint32_t)seen[r], reported};
    for (int i = 0; i < 3; ++i) report[r % 8][i] = (uint64_t)(r + 1) << 32 | v[i];
  }
  return call("query");
}
int hipStreamSynchronize(void*) { return call("synchronize"); }
int hipStreamBeginCapture(void*, int) { return call("begin"); }
int hipStreamEndCapture(void*, void** g) { return handle(g), call("end"); }
int hipGraphInstantiate(void** e, void*, void*, char*, size_t) { return handle(e), call("instantiate"); }
int hipGraphDestroy(void* g) { return std::free(g), 0; }
int hipGraphExecDestroy(void* e) { return std::free(e), 0; }
int hipGraphLaunch(void*, void*) { return call("launch graph"); }
struct Dim { uint32_t x, y, z; };
int hipLaunchKernel(const void*, Dim, Dim, void**, size_t, void*) { return call("launch"); }
int __hipPushCallConfiguration(Dim, Dim, size_t, void*) { return 0; }
int __hipPopCallConfiguration(Dim* g, Dim* b, size_t* n, void** s) { return *g = *b = Dim{1, 1, 1}, *n = 0, *s = nullptr, 0; }
void** __hipRegisterFatBinary(const void*) { return new void*[1](); }
void __hipUnregisterFatBinary(void** m) { delete[] m; }
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
}
