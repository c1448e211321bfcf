// Stands in for the HIP runtime's header where a kernel is compiled for the CPU: emulator.cpp runs a workgroup's threads as fibres that
// change over at barriers and at the operations of a wave.  What is here is what the sort uses.
#pragma once
#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>

#define __HIPCC__ 1
#define __device__
#define __host__
#define __global__ static
#define __shared__ static  // one workgroup runs at a time
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __HIP_MEMORY_SCOPE_SYSTEM 0

struct int2 { int x, y; };
struct int4 { int x, y, z, w; };
struct uint4 { unsigned x, y, z, w; };
inline int2 make_int2(int x, int y) { return {x, y}; }
inline int4 make_int4(int x, int y, int z, int w) { return {x, y, z, w}; }
struct dim3 {
  unsigned x, y, z;
  dim3(unsigned x_ = 1, unsigned y_ = 1, unsigned z_ = 1) : x(x_), y(y_), z(z_) {}
};
using hipStream_t = void*;
using hipEvent_t = void*;
using hipError_t = int;
enum { hipSuccess = 0, hipFuncAttributeMaxDynamicSharedMemorySize = 1 };
inline hipError_t hipGetLastError() { return hipSuccess; }
inline const char* hipGetErrorString(hipError_t) { return ""; }
inline hipError_t hipFuncSetAttribute(const void*, int, int) { return hipSuccess; }
inline hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
inline hipError_t hipSetDevice(int) { return hipSuccess; }
inline hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }

namespace emu {
extern unsigned dynamic_lds[];
int thread();
uint64_t* exchange(uint64_t mine);  // what every lane of the wave has brought
void launch(const char* kernel, dim3 grid, dim3 block, std::function<void()> body);
void before_launch(const char* kernel);  // (the test's)
template <typename T>
T from_lane(T v, int lane) {
  uint64_t bits = 0;
  memcpy(&bits, &v, sizeof v);
  bits = exchange(bits)[lane & 63];
  memcpy(&v, &bits, sizeof v);
  return v;
}
template <typename K, typename... A>
void go(const char* name, dim3 grid, dim3 block, K kernel, A... args) {
  launch(name, grid, block, [=] { kernel(args...); });
}
inline int readlane(int v, int lane) { return from_lane(v, lane); }
inline int readfirstlane(int v) { return v; }  // (the sort's are the same in all lanes)
inline int update_dpp(int old, int v, int ctrl, int row_mask, int, bool zeros) {
  const uint64_t* all = exchange(static_cast<uint32_t>(v));
  const int lane = thread() & 63, row = lane / 16;
  if (!((row_mask >> row) & 1)) return old;
  int from = -1;  // row_shr:n, row_bcast:15, row_bcast:31
  if (ctrl > 0x110 && ctrl < 0x120) from = lane % 16 >= ctrl - 0x110 ? lane - (ctrl - 0x110) : -1;
  else if (ctrl == 0x142) from = 16 * row - 1;
  else if (ctrl == 0x143) from = row >= 2 ? 31 : -1;
  else abort();
  return from >= 0 ? static_cast<int>(all[from]) : zeros ? 0 : old;
}
}  // namespace emu

extern dim3 blockIdx, gridDim;
static struct {
  struct {
    operator unsigned() const { return emu::thread(); }
  } x;
} threadIdx;
void __syncthreads();
inline unsigned long long __ballot(bool p) {
  const uint64_t* all = emu::exchange(p);
  unsigned long long m = 0;
  for (int i = 0; i < 64; ++i) m |= static_cast<unsigned long long>(all[i] & 1) << i;
  return m;
}
template <typename T>
T __shfl(T v, int lane, int) { return emu::from_lane(v, lane); }
template <typename T>
T __shfl_up(T v, int d, int) { return emu::from_lane(v, std::max((emu::thread() & 63) - d, 0)); }
inline int __clz(unsigned x) { return x ? __builtin_clz(x) : 32; }
inline int __popc(unsigned x) { return __builtin_popcount(x); }
inline int __popcll(unsigned long long x) { return __builtin_popcountll(x); }
template <typename T, typename U>
T atomicAdd(T* p, U v) {
  const T before = *p;
  *p = before + static_cast<T>(v);
  return before;
}
template <typename T, typename U>
T atomicOr(T* p, U v) {
  const T before = *p;
  *p = before | v;
  return before;
}
#define __hip_atomic_fetch_add(p, v, order, scope) atomicAdd(p, v)
#define __hip_atomic_store(p, v, order, scope) (*(p) = (v))
using std::max;
using std::min;
#define hipLaunchKernelGGL(kernel, grid, block, lds, stream, ...) emu::go(#kernel, grid, block, kernel, __VA_ARGS__)
