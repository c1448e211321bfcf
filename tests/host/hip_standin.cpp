// A stand-in for the HIP runtime, for tests of the library's host code without a GPU: several devices, memory that knows
// its device, and a log of what the library asks for.  Kernels are not run, so whatever they would write keeps the zeros
// that memory starts with.
#include <hip/hip_runtime.h>

#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <sstream>
#include <string>

namespace {
std::mutex mu;
// (made on first use: the library's kernels are registered while it is loaded)
std::map<const void*, std::string>& kernels() {
  static auto* k = new std::map<const void*, std::string>;
  return *k;
}
std::map<const void*, size_t>& vars() {
  static auto* v = new std::map<const void*, size_t>;
  return *v;
}
std::map<char*, std::pair<size_t, int>> memory;  // start -> size, device
std::map<std::pair<const void*, int>, void*> symbols;
std::string text;
thread_local int device = 0;
thread_local dim3 grid, block;
thread_local size_t shmem;
thread_local hipStream_t stream;
hipStream_t capturing = reinterpret_cast<hipStream_t>(~uintptr_t(0));
uintptr_t next_event = 0x1000;

template <typename... A>
void note(const A&... a) {
  std::ostringstream o;
  (void)std::initializer_list<int>{(o << a << ' ', 0)...};
  std::lock_guard<std::mutex> lk(mu);
  text += o.str() + "\n";
}
unsigned long long num(const void* p) { return reinterpret_cast<unsigned long long>(p); }
void* take(size_t n) {
  char* p = static_cast<char*>(calloc(n ? n : 1, 1));
  std::lock_guard<std::mutex> lk(mu);
  memory[p] = {n, device};
  return p;
}
}  // namespace

extern "C" {
// What the tests ask for.
const char* standin_log() {  // what happened since the last call
  static thread_local std::string out;
  std::lock_guard<std::mutex> lk(mu);
  out.swap(text);
  text.clear();
  return out.c_str();
}
int standin_device_of(const void* q) {  // -1: nobody's
  std::lock_guard<std::mutex> lk(mu);
  auto it = memory.upper_bound(static_cast<char*>(const_cast<void*>(q)));
  if (it == memory.begin()) return -1;
  --it;
  return static_cast<const char*>(q) < it->first + it->second.first ? it->second.second : -1;
}
void standin_set_device(int d) { device = d; }
void standin_capture(void* s) { capturing = static_cast<hipStream_t>(s); }

// What the compiler's host code calls.
void** __hipRegisterFatBinary(const void*) {
  static void* h;
  return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* f, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
  std::lock_guard<std::mutex> lk(mu);
  kernels()[f] = name;
}
void __hipRegisterVar(void**, void* var, char*, char*, int, size_t size, int, int) { vars()[var] = size; }
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t m, hipStream_t s) {
  grid = g, block = b, shmem = m, stream = s;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* m, hipStream_t* s) {
  *g = grid, *b = block, *m = shmem, *s = stream;
  return hipSuccess;
}
// (the ninth argument is logged as well: the bins' totals of the sort's count pass)
hipError_t hipLaunchKernel(const void* f, dim3, dim3, void** args, size_t, hipStream_t s) {
  std::string name;
  {
    std::lock_guard<std::mutex> lk(mu);
    name = kernels().at(f);
  }
  const bool count = name.find("bs_count_kernel") != std::string::npos;
  note("launch", device, num(s), name, count ? *static_cast<unsigned long long*>(args[8]) : 0ull);
  return hipSuccess;
}

// What the library calls.
hipError_t hipGetDevice(int* d) {
  *d = device;
  return hipSuccess;
}
hipError_t hipSetDevice(int d) {
  device = d;
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) {
  *p = take(n);
  note("malloc", device, num(*p));
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  note("free", device, num(p));
  std::lock_guard<std::mutex> lk(mu);
  memory.erase(static_cast<char*>(p));
  free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) {
  *p = calloc(n, 1);
  return hipSuccess;
}
hipError_t hipHostFree(void* p) {
  free(p);
  return hipSuccess;
}
hipError_t hipHostGetDevicePointer(void** d, void* h, unsigned) {
  *d = h;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void* var) {
  void*& at = symbols[{var, device}];
  if (!at) at = take(vars().at(var));
  *p = at;
  return hipSuccess;
}
hipError_t hipDeviceSynchronize() {
  note("drain", device);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t s) {
  note("sync", device, num(s));
  return hipSuccess;
}
hipError_t hipStreamQuery(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  *st = s == capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
  std::lock_guard<std::mutex> lk(mu);
  *e = reinterpret_cast<hipEvent_t>(next_event += 16);
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  note("record", device, num(s), num(e));
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* t, hipEvent_t, hipEvent_t) {
  *t = 1.f;
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  note("wait", device, num(s), num(e));
  return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) {
  memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipMemsetAsync(void*, int, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
int hipGetStreamDeviceId(hipStream_t) { return device; }
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600*, int) { return hipErrorInvalidValue; }
}
