// Test-only: the HIP subset that csrc/contact.hip uses, for a build on the CPU
// in which every lane of a workgroup is a fiber (contact_lanes.cpp).  A launch
// runs its workgroups one after another; a barrier or a cross-lane operation
// hands over to the next lane until all of the wavefront (workgroup) have come
// to it.  Between two of those the lanes run one by one from the first, so a
// lane that reads what a later one has still to write gets wrong numbers.
// Dynamic LDS starts as NaNs, and writes past the size of the launch are
// counted.
#pragma once
#define __HIPCC__

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <string>

#define __host__
#define __device__
#define __shared__ thread_local  // one per workgroup: they run one by one
#define __global__
#define __forceinline__ inline
#define __launch_bounds__(...)
#define __align__(n) __attribute__((aligned(n)))

struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};
typedef int hipError_t;
typedef void* hipStream_t;
typedef void* hipEvent_t;
enum { hipSuccess = 0, hipErrorInvalidValue = 1 };
enum { hipDeviceAttributeMaxSharedMemoryPerBlock, hipDeviceAttributeMultiprocessorCount };

namespace lanes {
struct Index { unsigned x; };
extern Index thread, block, block_size;
extern int compute_units;
constexpr size_t kLds = 160 * 1024;
void run(const char* kernel, const std::function<void()>& body, dim3 grid, dim3 threads, size_t lds);
void wave_barrier();
void block_barrier();
int lane();
// posts the lane's value; the 64 lanes' values, 16 bytes apart
const unsigned char* post(const void* p, size_t n);
template <typename T>
T of(T v, int lane) {
  const unsigned char* s = post(&v, sizeof v);
  std::memcpy(&v, s + 16 * lane, sizeof v);
  return v;
}
}  // namespace lanes

#define threadIdx lanes::thread
#define blockIdx lanes::block
#define blockDim lanes::block_size
#define hipLaunchKernelGGL(k, g, b, l, st, a) lanes::run(#k, [&] { k(a); }, g, b, l)

// ---- runtime
inline hipError_t hipGetLastError() { return 0; }
inline const char* hipGetErrorString(hipError_t) { return ""; }
inline hipError_t hipGetDevice(int* d) { return *d = 0; }
inline hipError_t hipDeviceGetAttribute(int* v, int a, int) {
  *v = a == hipDeviceAttributeMultiprocessorCount ? lanes::compute_units : (int)lanes::kLds;
  return 0;
}
template <typename T>
hipError_t hipMalloc(T** p, size_t n) {
  *p = (T*)std::malloc(n ? n : 1);
  return 0;
}
inline hipError_t hipFree(void* p) { std::free(p); return 0; }
inline hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return 0; }
inline hipError_t hipStreamSynchronize(hipStream_t) { return 0; }
inline hipError_t hipEventCreate(hipEvent_t* e) { *e = nullptr; return 0; }
inline hipError_t hipEventDestroy(hipEvent_t) { return 0; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return 0; }
inline hipError_t hipEventSynchronize(hipEvent_t) { return 0; }
inline hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1; return 0; }

// ---- device functions
#define __builtin_amdgcn_fence(order, scope) ((void)0)
inline void __builtin_amdgcn_wave_barrier() { lanes::wave_barrier(); }
inline void __syncthreads() { lanes::block_barrier(); }
inline int __builtin_amdgcn_readfirstlane(int x) { return x; }
// DPP: whole-wavefront shifts, broadcast and rotation in a row of 16, quads
template <typename T>
T __builtin_amdgcn_update_dpp(T old, T x, int c, int, int, bool) {
  const int l = lanes::lane();
  int s = -1;
  if (c == 0x130) s = l == 63 ? -1 : l + 1;
  else if (c == 0x138) s = l - 1;
  else if (c >= 0x150) s = (l & 48) | (c & 15);
  else if (c > 0x120) s = (l & 48) | ((l - (c & 15)) & 15);
  else s = (l & 60) | (c >> 2 * (l & 3) & 3);
  const T v = lanes::of(x, s < 0 ? 0 : s);
  return s < 0 ? old : v;
}
template <typename T>
T __shfl(T x, int s, int w = 64) {
  return lanes::of(x, (lanes::lane() & ~(w - 1)) | (s & (w - 1)));
}
inline unsigned long long __ballot(bool p) {
  const unsigned char* s = lanes::post(&p, 1);
  unsigned long long r = 0;
  for (int i = 0; i < 64; ++i) r |= (unsigned long long)(s[16 * i] & 1) << i;
  return r;
}
inline int __popc(unsigned x) { return __builtin_popcount(x); }
inline int __ffs(int x) { return __builtin_ffs(x); }
using std::fma;
using std::max;
using std::min;
using std::sqrt;
