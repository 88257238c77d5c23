// A HIP runtime for tests of the library's host code on a machine without a
// GPU: "device" memory is host memory, kernels are recorded and do nothing.
// The library's own sources, compiled for the host only, are linked with it.
//
// What it observes and what a test can make happen:
//   - every kernel launch with the set of its pointer operands that are NULL;
//   - the n-th device allocation of the library fails (fake_fail_alloc), the
//     runtime's own hipMalloc fails (fake_device_bytes), a synchronisation
//     fails (fake_fail_sync), a host allocation fails (fake_fail_new);
//   - work is pending on a stream from a launch or asynchronous copy until the
//     stream or the device is synchronised; memory that the library gives up
//     while work is pending is counted (fake_early_frees);
//   - a stream is being captured (fake_capture): allocations and
//     synchronisations are refused, launches on it are recorded.
#include <cxxabi.h>
#include <stdlib.h>
#include <string.h>

#include <sys/mman.h>

#include <chrono>
#include <condition_variable>
#include <map>
#include <mutex>
#include <new>
#include <set>
#include <string>
#include <vector>

#include "merbit_host.hpp"

namespace {

struct Arg {
  std::string type;
  bool pointer;
};
struct Kernel {
  std::string name;  // without parameters
  std::vector<Arg> args;
};
struct State {
  std::map<const void*, Kernel> kernels;
  std::map<void*, size_t> live;
  size_t live_bytes = 0, device_bytes = (size_t)1 << 40;
  long mallocs = 0, frees = 0, early_frees = 0;
  long held = 0;     // library blocks allocated and not yet given up
  int32_t fill = 0;  // what new device memory holds
  std::set<hipStream_t> pending;
  hipStream_t capturing = nullptr;
  bool any_capture = false;
  std::string log;  // one line per launch
  dim3 grid, block;
  size_t shmem = 0;
  hipStream_t stream = nullptr;
  int fail_alloc = 0;  // 1: the next library allocation fails; n: the n-th
  int fail_sync = 0;   // the same for synchronisations
  int fail_graph = 0;  // the same for graph instantiations
  void* spmv_y = nullptr;  // what the last SpMV launch wrote
};
State& st() {
  static State* s = new State();
  return *s;
}
std::recursive_mutex& mu() {
  static std::recursive_mutex* m = new std::recursive_mutex();
  return *m;
}
typedef std::lock_guard<std::recursive_mutex> Lock;
std::mutex& gate_mu() {
  static std::mutex* m = new std::mutex();
  return *m;
}
std::condition_variable& gate_cv() {
  static std::condition_variable* c = new std::condition_variable();
  return *c;
}
bool g_gate = false;
long g_gate_timeouts = 0, g_gate_waiting = 0;
thread_local long g_fail_new = 0;

bool countdown(int& n) {
  if (n <= 0) return false;
  return --n == 0;
}

// "void merbit::f<float>(float const*, merbit::SpmmArgs, int)" -> name, types
Kernel parse(const char* mangled) {
  Kernel k;
  int status = 0;
  char* d = abi::__cxa_demangle(mangled, nullptr, nullptr, &status);
  std::string s = status == 0 ? d : mangled;
  free(d);
  const size_t ns = s.find("merbit::");
  if (ns != std::string::npos) s = s.substr(ns + 8);
  int depth = 0;
  size_t open = std::string::npos;
  for (size_t i = 0; i < s.size(); ++i) {
    if (s[i] == '<') ++depth;
    if (s[i] == '>') --depth;
    if (s[i] == '(' && depth == 0) {
      open = i;
      break;
    }
  }
  k.name = s.substr(0, open);
  if (open == std::string::npos) return k;
  std::string cur;
  depth = 0;
  for (size_t i = open + 1; i < s.size(); ++i) {
    const char c = s[i];
    if ((c == ',' && depth == 0) || i + 1 == s.size()) {
      while (!cur.empty() && cur[0] == ' ') cur.erase(0, 1);
      if (!cur.empty()) k.args.push_back({cur, cur.find('*') != std::string::npos});
      cur.clear();
      continue;
    }
    if (c == '<' || c == '(') ++depth;
    if (c == '>' || c == ')') --depth;
    cur += c;
  }
  return k;
}

}  // namespace

extern "C" {

// ------------------------------------------------------------- control --

void fake_reset_log() {
  Lock l(mu());
  st().log.clear();
}
const char* fake_log() { return st().log.c_str(); }
void fake_fail_alloc(int n) { st().fail_alloc = n; }
void fake_fail_graph(int n) { st().fail_graph = n; }
void* fake_spmv_y() { return st().spmv_y; }
void fake_fail_sync(int n) { st().fail_sync = n; }
// returns what was left of the count before: > 0 if the failure did not come
long fake_fail_new(long n) {
  const long left = g_fail_new;
  g_fail_new = n;
  return left;
}
void fake_device_bytes(size_t n) { st().device_bytes = n; }
size_t fake_live_bytes() { return st().live_bytes; }
long fake_mallocs() { return st().mallocs; }
long fake_frees() { return st().frees; }
long fake_early_frees() { return st().early_frees; }
void fake_gate(int on) {
  std::lock_guard<std::mutex> g(gate_mu());
  g_gate = on != 0;
  gate_cv().notify_all();
}
long fake_gate_waiting() { return g_gate_waiting; }
long fake_gate_timeouts() { return g_gate_timeouts; }
long fake_held() { return st().held; }
void fake_fill(int v) { st().fill = v; }
void fake_capture(void* stream, int on) {
  st().any_capture = on != 0;
  st().capturing = static_cast<hipStream_t>(stream);
}

// ------------------------------------------------- registration, launch --

void** __hipRegisterFatBinary(const void*) {
  static void* h = nullptr;
  return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* handle, char*, const char* name, unsigned, void*,
                           void*, void*, void*, int*) {
  Lock l(mu());
  st().kernels[handle] = parse(name);
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t s, hipStream_t q) {
  Lock l(mu());
  st().grid = g;
  st().block = b;
  st().shmem = s;
  st().stream = q;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* s, hipStream_t* q) {
  Lock l(mu());
  *g = st().grid;
  *b = st().block;
  *s = st().shmem;
  *q = st().stream;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t, hipStream_t q) {
  Lock l(mu());
  const Kernel& k = st().kernels[f];
  std::string line = k.name + " null:";
  for (size_t i = 0; i < k.args.size(); ++i) {
    if (k.args[i].pointer && *static_cast<void**>(args[i]) == nullptr)
      line += " " + std::to_string(i);
    if (k.args[i].type == "merbit::SpmmArgs") {
      const merbit::SpmmArgs& a = *static_cast<const merbit::SpmmArgs*>(args[i]);
      const void* p[] = {a.X, a.Y, a.Z, a.Xn, a.src, a.sums_in, a.dmask, a.part};
      for (size_t j = 0; j < sizeof p / sizeof p[0]; ++j)
        if (p[j] == nullptr) line += " m" + std::to_string(j);
    }
    if (k.args[i].type == "merbit::SpmvArgs") {
      const merbit::SpmvArgs& a = *static_cast<const merbit::SpmvArgs*>(args[i]);
      st().spmv_y = a.y;
      const void* p[] = {a.x, a.y, a.z, a.row_start};
      for (size_t j = 0; j < sizeof p / sizeof p[0]; ++j)
        if (p[j] == nullptr) line += " m" + std::to_string(j);
    }
  }
  line += " block: " + std::to_string(b.x) + " grid: " + std::to_string(g.x);
  st().log += line + "\n";
  if (!(st().any_capture && q == st().capturing)) st().pending.insert(q);
  return hipSuccess;
}

// -------------------------------------------------------------- memory --

hipError_t hipMalloc(void** p, size_t n) {
  Lock l(mu());
  *p = nullptr;
  if (st().any_capture) return hipErrorStreamCaptureUnsupported;
  if (n == 0) return hipSuccess;
  ++st().mallocs;
  if (st().live_bytes + n > st().device_bytes) return hipErrorOutOfMemory;
  *p = mmap(nullptr, n, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
  if (*p == MAP_FAILED) abort();
  for (size_t i = 0; st().fill != 0 && i < n / 4; ++i) static_cast<int32_t*>(*p)[i] = st().fill;
  st().live[*p] = n;
  st().live_bytes += n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  {
    // a device that is busy until fake_gate(0) (or for five seconds)
    std::unique_lock<std::mutex> g(gate_mu());
    if (g_gate) ++g_gate_waiting;
    if (g_gate && !gate_cv().wait_for(g, std::chrono::seconds(5), [] { return !g_gate; }))
      ++g_gate_timeouts;
  }
  Lock l(mu());
  if (st().any_capture) return hipErrorStreamCaptureUnsupported;
  auto it = st().live.find(p);
  if (it == st().live.end()) return hipErrorInvalidValue;
  st().pending.clear();  // waits for the device
  st().live_bytes -= it->second;
  ++st().frees;
  munmap(p, it->second);
  st().live.erase(it);
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  Lock l(mu());
  if (st().any_capture) return hipErrorStreamCaptureUnsupported;
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t q) {
  Lock l(mu());
  if (!d || !s) return hipErrorInvalidValue;
  memcpy(d, s, n);
  st().pending.insert(q);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t q) {
  Lock l(mu());
  memset(d, v, n);
  st().pending.insert(q);
  return hipSuccess;
}
hipError_t hipMemsetD32Async(hipDeviceptr_t, int, size_t, hipStream_t q) {
  Lock l(mu());
  st().pending.insert(q);
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
  static void* scratch = calloc(1, MERBIT_NOALLOC_SCRATCH_BYTES);
  *p = scratch;
  return hipSuccess;
}

// ------------------------------------------- streams, events, the device --

hipError_t hipStreamSynchronize(hipStream_t q) {
  Lock l(mu());
  if (countdown(st().fail_sync)) return hipErrorUnknown;
  if (st().any_capture) return hipErrorStreamCaptureUnsupported;
  st().pending.erase(q);
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
  Lock l(mu());
  if (countdown(st().fail_sync)) return hipErrorUnknown;
  if (st().any_capture) return hipErrorStreamCaptureUnsupported;
  st().pending.clear();
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t q, hipStreamCaptureStatus* s) {
  Lock l(mu());
  *s = st().any_capture && q == st().capturing ? hipStreamCaptureStatusActive
                                               : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamCreateWithFlags(hipStream_t* q, unsigned) {
  *q = reinterpret_cast<hipStream_t>(malloc(8));
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t q) {
  free(q);
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t q, hipGraph_t* g) {
  Lock l(mu());
  st().pending.erase(q);
  *g = reinterpret_cast<hipGraph_t>(malloc(8));
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  if (countdown(st().fail_graph)) return hipErrorOutOfMemory;
  *e = reinterpret_cast<hipGraphExec_t>(malloc(8));
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t q) {
  Lock l(mu());
  st().pending.insert(q);
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t g) {
  free(g);
  return hipSuccess;
}
hipError_t hipGraphExecDestroy(hipGraphExec_t g) {
  free(g);
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = reinterpret_cast<hipEvent_t>(malloc(8));
  return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
  free(e);
  return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}
hipError_t hipGetDevice(int* d) {
  *d = 0;
  return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 160 * 1024;  // or LDS bytes
  return hipSuccess;
}
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int threads, size_t) {
  *n = 1024 / threads;  // 16 wavefronts per CU
  return hipSuccess;
}
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "fake error"; }

// ------------------------------------- the library's own memory functions --
// (linked with --wrap: the library's calls arrive here first)

hipError_t __real__ZN6merbit15dev_alloc_bytesEPPvm(void** out, size_t bytes);
hipError_t __wrap__ZN6merbit15dev_alloc_bytesEPPvm(void** out, size_t bytes) {
  {
    Lock l(mu());
    if (countdown(st().fail_alloc)) {
      *out = nullptr;
      return hipErrorOutOfMemory;
    }
  }
  const hipError_t e = __real__ZN6merbit15dev_alloc_bytesEPPvm(out, bytes);
  Lock l(mu());
  if (e == hipSuccess) ++st().held;
  return e;
}
void __real__ZN6merbit8dev_freeEPv(void* p) noexcept;
void __wrap__ZN6merbit8dev_freeEPv(void* p) noexcept {
  {
    Lock l(mu());
    if (p) --st().held;
    if (p && !st().pending.empty()) ++st().early_frees;
  }
  __real__ZN6merbit8dev_freeEPv(p);
}
void __real__ZN6merbit14dev_free_afterE10hipError_tPv(hipError_t waited, void* p) noexcept;
void __wrap__ZN6merbit14dev_free_afterE10hipError_tPv(hipError_t waited, void* p) noexcept {
  {
    Lock l(mu());
    if (p) --st().held;
    if (p && waited == hipSuccess && !st().pending.empty()) ++st().early_frees;
  }
  __real__ZN6merbit14dev_free_afterE10hipError_tPv(waited, p);
}

}  // extern "C"

// A host allocation of this thread fails (operator new of the library only:
// it is linked with its own symbols bound first).
void* operator new(size_t n) {
  if (g_fail_new > 0 && --g_fail_new == 0) throw std::bad_alloc();
  void* p = malloc(n ? n : 1);
  if (!p) throw std::bad_alloc();
  return p;
}
void operator delete(void* p) noexcept { free(p); }
void operator delete(void* p, size_t) noexcept { free(p); }
