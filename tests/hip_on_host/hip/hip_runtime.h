// The library's kernels on the CPU, for tests of what a GPU's scheduling may do:
// every thread of a workgroup is a fiber, and threads and workgroups run in
// ascending, descending or shuffled order (emu_order), so that the arrival order of
// atomics is the test's choice.  A fiber runs until it ends or waits: at __syncthreads for
// every live thread of its workgroup, at a wave operation (shuffle, ballot,
// wave barrier) for every lane of its wave that can still come to the same place.
// Only what the library's sources use is here.  x86-64.
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <memory>
#include <vector>

using std::max;
using std::min;

#define __device__
#define __host__
#define __global__
#define __forceinline__ inline
#define __noinline__ __attribute__((noinline)) inline
#define __align__(x) __attribute__((aligned(x)))
#define __launch_bounds__(...)
#define __restrict__
#define __shared__ static  // (dynamic LDS: see the build)

struct int2 { int x, y; };
struct __align__(16) int4 { int x, y, z, w; };
struct uint2 { unsigned x, y; };
struct __align__(16) uint4 { unsigned x, y, z, w; };
struct __align__(16) ulonglong2 { unsigned long long x, y; };
struct float2 { float x, y; };
struct float3 { float x, y, z; };
struct __align__(16) float4 { float x, y, z, w; };
inline int2 make_int2(int a, int b) { return {a, b}; }
inline int4 make_int4(int a, int b, int c, int d) { return {a, b, c, d}; }
inline uint2 make_uint2(unsigned a, unsigned b) { return {a, b}; }
inline uint4 make_uint4(unsigned a, unsigned b, unsigned c, unsigned d) { return {a, b, c, d}; }
inline float2 make_float2(float a, float b) { return {a, b}; }
inline float3 make_float3(float a, float b, float c) { return {a, b, c}; }
inline float4 make_float4(float a, float b, float c, float d) { return {a, b, c, d}; }

struct dim3 {
  unsigned x, y, z;
  dim3(unsigned a = 1, unsigned b = 1, unsigned c = 1) : x(a), y(b), z(c) {}
};

// ---- runtime calls -------------------------------------------------------
typedef int hipError_t;
typedef void* hipStream_t;
typedef void* hipEvent_t;
enum { hipSuccess = 0 };
enum { hipDeviceAttributeMaxSharedMemoryPerBlock = 0 };
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
inline hipError_t hipDeviceGetAttribute(int* v, int, int) { *v = 163840; return hipSuccess; }
inline hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
#define HIP_SYMBOL(x) (x)
template <class T>
inline hipError_t hipGetSymbolAddress(void** p, T& x) { *p = (void*)&x; return hipSuccess; }

// ---- fibers --------------------------------------------------------------
namespace emu {

enum Wait { kNone, kBlock, kWave };
struct Fiber {
  void* sp = nullptr;
  std::unique_ptr<char[]> stack;
  int thread = -1;  // the thread it runs, -1: idle
  Wait wait = kNone;
  const void* site = nullptr;  // wave operations: the place in the code
  int group = 64;              // ... lanes that take part together
  unsigned long long in = 0, out[64];
  unsigned long long peers = 0;
};
struct State {
  std::function<void()> body;
  std::vector<std::unique_ptr<Fiber>> pool;
  std::vector<Fiber*> of;  // fiber of a thread that has started and not ended
  Fiber* cur = nullptr;
  void* main_sp = nullptr;
  int next = 0, threads = 0;  // threads started, of how many
  int order = 0;  // 0 ascending, 1 descending, 2 shuffled
  std::vector<int> shuffle;  // of the workgroup's threads
  dim3 block_idx, grid, block;
  int thread_of(int k) const { return order == 2 ? shuffle[k] : (order ? threads - 1 - k : k); }
};
extern State g;
extern "C" void emu_switch(void** save, void* to);
void wait_block();
Fiber* wait_wave(const void* site, unsigned long long x, int group);
void launch(dim3 grid, dim3 block, size_t lds, std::function<void()> body, const char* name);

struct ThreadIdx {
  struct X {
    operator unsigned() const { return (unsigned)g.cur->thread; }
  } x;
};
struct BlockIdx {
  struct X {
    operator unsigned() const { return g.block_idx.x; }
  } x;
  struct Y {
    operator unsigned() const { return g.block_idx.y; }
  } y;
};

template <class T>
inline unsigned long long bits(T x) {
  unsigned long long u = 0;
  memcpy(&u, &x, sizeof x);
  return u;
}
template <class T>
inline T value(unsigned long long u) {
  T x;
  memcpy(&x, &u, sizeof x);
  return x;
}
// x of lane src (within the wave); its own where src takes no part
template <class T>
__attribute__((noinline)) T lane_value(const void* site, T x, int group, int src) {
  const int lane = g.cur->thread & 63;
  Fiber* f = wait_wave(site, bits(x), group);
  return (f->peers >> (src & 63)) & 1 ? value<T>(f->out[src & 63]) : value<T>(f->out[lane]);
}
}  // namespace emu

static const emu::ThreadIdx threadIdx;
static const emu::BlockIdx blockIdx;
#define gridDim emu::g.grid
#define blockDim emu::g.block
#define EMU_SITE __builtin_return_address(0)
#define EMU_OP __attribute__((noinline))

#define hipLaunchKernelGGL(k, grid, block, lds, stream, ...) \
  emu::launch(dim3(grid), dim3(block), lds, [=] { (k)(__VA_ARGS__); }, #k)

// ---- wave and workgroup operations ---------------------------------------
inline void __syncthreads() { emu::wait_block(); }
EMU_OP inline unsigned long long __ballot(bool b) {
  emu::Fiber* f = emu::wait_wave(EMU_SITE, b, 64);
  unsigned long long m = 0;
  for (int l = 0; l < 64; ++l)
    if ((f->peers >> l) & 1) m |= (f->out[l] & 1) << l;
  return m;
}
template <class T>
EMU_OP T __shfl(T x, int src, int width = 64) {
  const int lane = threadIdx.x & 63;
  return emu::lane_value(EMU_SITE, x, width, (lane & ~(width - 1)) | (src & (width - 1)));
}
template <class T>
EMU_OP T __shfl_up(T x, int d, int width = 64) {
  const int lane = threadIdx.x & 63, r = lane & (width - 1);
  return emu::lane_value(EMU_SITE, x, width, r >= d ? lane - d : lane);
}
template <class T>
EMU_OP T __shfl_down(T x, int d, int width = 64) {
  const int lane = threadIdx.x & 63, r = lane & (width - 1);
  return emu::lane_value(EMU_SITE, x, width, r + d < width ? lane + d : lane);
}
template <class T>
EMU_OP T __shfl_xor(T x, int d, int width = 64) {
  const int lane = threadIdx.x & 63;
  return emu::lane_value(EMU_SITE, x, width, lane ^ d);
}
EMU_OP inline void emu_wave_barrier() { (void)emu::wait_wave(EMU_SITE, 0, 64); }
EMU_OP inline int emu_first_lane(int x) {
  emu::Fiber* f = emu::wait_wave(EMU_SITE, emu::bits(x), 64);
  return emu::value<int>(f->out[__builtin_ctzll(f->peers)]);
}
EMU_OP inline int emu_read_lane(int x, int src) { return emu::lane_value(EMU_SITE, x, 64, src); }
EMU_OP inline int emu_dpp(int x, int ctrl) {  // quad permutation, half-row mirror
  const int lane = threadIdx.x & 63;
  const int src = ctrl == 0x141 ? (lane ^ 7) : ((lane & ~3) | ((ctrl >> (2 * (lane & 3))) & 3));
  return emu::lane_value(EMU_SITE, x, 64, src);
}
#define __builtin_amdgcn_fence(...) ((void)0)
#define __threadfence_block() ((void)0)
#define __builtin_amdgcn_wave_barrier() emu_wave_barrier()
#define __builtin_amdgcn_readfirstlane(x) emu_first_lane(x)
#define __builtin_amdgcn_readlane(x, l) emu_read_lane(x, l)
#define __builtin_amdgcn_update_dpp(o, x, ctrl, ...) emu_dpp(x, ctrl)
// estimates with errors of the instructions' size
inline double emu_estimate(double y) {
  static unsigned k = 1;
  k = k * 1664525u + 1013904223u;
  return y * (1.0 + ((int)(k >> 8) % 1000 - 500) / 500.0 * 0x1p-23);
}
#define __builtin_amdgcn_rcp(x) emu_estimate(1.0 / (x))
#define __builtin_amdgcn_rsq(x) emu_estimate(1.0 / std::sqrt(x))

// ---- scalar functions ----------------------------------------------------
inline float __int_as_float(int x) { return emu::value<float>((unsigned)x); }
inline float __uint_as_float(unsigned x) { return emu::value<float>(x); }
inline unsigned __float_as_uint(float x) { return (unsigned)emu::bits(x); }
inline long long __double_as_longlong(double x) { return (long long)emu::bits(x); }
inline double __longlong_as_double(long long x) { return emu::value<double>((unsigned long long)x); }
inline int __popcll(unsigned long long x) { return __builtin_popcountll(x); }
inline int __popc(unsigned x) { return __builtin_popcount(x); }
inline int __ffsll(unsigned long long x) { return __builtin_ffsll((long long)x); }

template <class T, class U>
inline T atomicAdd(T* p, U v) { T o = *p; *p = (T)(o + v); return o; }
template <class T, class U>
inline T atomicSub(T* p, U v) { T o = *p; *p = (T)(o - v); return o; }
template <class T, class U>
inline T atomicMin(T* p, U v) { T o = *p; if ((T)v < o) *p = (T)v; return o; }
template <class T, class U>
inline T atomicMax(T* p, U v) { T o = *p; if ((T)v > o) *p = (T)v; return o; }
template <class T, class U>
inline T atomicOr(T* p, U v) { T o = *p; *p = (T)(o | (T)v); return o; }
template <class T, class U, class V>
inline T atomicCAS(T* p, U c, V v) { T o = *p; if (o == (T)c) *p = (T)v; return o; }
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __HIP_MEMORY_SCOPE_WORKGROUP 0
#define __hip_atomic_load(p, ...) (*(p))
#define __hip_atomic_store(p, v, ...) (*(p) = (v))
