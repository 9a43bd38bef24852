// Volume and surface area of hull surfaces, and their gradients with respect
// to float point positions on a fixed face set, batched over clouds.
//
// For the outward faces (a, b, d) of a closed surface and a reference point c
// (here the cloud's point 0, inside the hull, so every term is >= 0):
//   V = 1/6 sum_f (a - c) . ((b - c) x (d - c)),  A = 1/2 sum_f |n_f|,
//   n_f = (b - a) x (d - a)  (the same for every rotation of the face).
// Gradients (c drops out on a closed surface):
//   dV/dp = 1/6 sum_{f containing p} n_f,
//   dA/da = 1/2 (b - d) x n_f / |n_f| for the corner a of f = (a, b, d)
//           (0 for a face of zero area).
#include <stddef.h>

#include "common.hpp"

namespace hull {

constexpr int kVolThreads = 1024;

struct Kahan {
  float s = 0.f, c = 0.f;
  __device__ __forceinline__ void add(float x) {
    float y = x - c;
    float t = s + y;
    c = (t - s) - y;
    s = t;
  }
};

__device__ __forceinline__ float3 sub3(float3 a, float3 b) {
  return make_float3(a.x - b.x, a.y - b.y, a.z - b.z);
}
__device__ __forceinline__ float3 cross3(float3 a, float3 b) {
  return make_float3(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}
__device__ __forceinline__ float dot3(float3 a, float3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ __forceinline__ float3 ld3(const float* p, int64_t i) {
  return make_float3(p[3 * i], p[3 * i + 1], p[3 * i + 2]);
}

// Deterministic block reduction of two floats (wave shuffles, then LDS).
__device__ __forceinline__ float2 block_sum2(float x, float y) {
  __shared__ float sx[kVolThreads / 64], sy[kVolThreads / 64];
  for (int o = 32; o > 0; o >>= 1) {
    x += __shfl_down(x, o);
    y += __shfl_down(y, o);
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
    sx[wave] = x;
    sy[wave] = y;
  }
  __syncthreads();
  float tx = 0.f, ty = 0.f;
  if (threadIdx.x == 0)
    for (int w = 0; w < kVolThreads / 64; ++w) {
      tx += sx[w];
      ty += sy[w];
    }
  return make_float2(tx, ty);
}

// One workgroup per cloud (blockIdx.x).
__global__ void __launch_bounds__(kVolThreads)
    k_vol_area_fwd(const float* __restrict__ p, const int64_t* __restrict__ pt_off,
                   const int32_t* __restrict__ faces, const int64_t* __restrict__ face_off,
                   float* __restrict__ V, float* __restrict__ A) {
  const int h = blockIdx.x;
  const int64_t po = pt_off[h], pn = pt_off[h + 1] - po;
  const int64_t f0 = face_off[h], f1 = face_off[h + 1];
  Kahan kv, ka;
  if (pn > 0) {
    const float3 c = ld3(p, po);
    for (int64_t f = f0 + threadIdx.x; f < f1; f += kVolThreads) {
      const int ia = faces[3 * f], ib = faces[3 * f + 1], id = faces[3 * f + 2];
      const float3 a = ld3(p, po + ia), b = ld3(p, po + ib), d = ld3(p, po + id);
      kv.add(dot3(sub3(a, c), cross3(sub3(b, c), sub3(d, c))));
      const float3 n = cross3(sub3(b, a), sub3(d, a));
      ka.add(sqrtf(dot3(n, n)));
    }
  }
  float2 t = block_sum2(kv.s - kv.c, ka.s - ka.c);
  if (threadIdx.x == 0) {
    V[h] = t.x / 6.f;
    A[h] = t.y * 0.5f;
  }
}

// The backward pass adds nine floats per face into the gradient rows of its
// corners.  As global atomics on scattered rows these run at about 20 G/s
// (1.84 ms for 256 clouds of 15,970 points and 15,936 faces).  So a cloud of
// up to kVolMaxLds points is cut into ranges of kVolRange points, one
// workgroup each: it reads the cloud's face rows, adds the corners inside its
// range into LDS and writes the range's rows once, coalesced, with no clearing
// pass.  Larger clouds would read their faces too many times and keep the
// global atomics.  The cloud is the grid's fast dimension: the ranges of one
// cloud then mostly share an XCD's L2 (with the range fast, a multiple of 8
// ranges apart, the same kernel took 2.5 times as long), and the range size
// hardly matters (2,048 to 13,000 points: within 5%).
constexpr int kVolRange = 4096;  // points: 48 KiB of LDS
constexpr int kVolRanges = 16;   // workgroups per cloud
constexpr int kVolBwdThreads = 512;
constexpr int kVolFaces = 4;     // faces a thread has in flight
constexpr int64_t kVolMaxLds = (int64_t)kVolRanges * kVolRange;

// Clears what the range workgroups do not write: the rows of the clouds too
// large for them and any before the first cloud.
__global__ void __launch_bounds__(256) k_vol_area_zero(float* __restrict__ g,
                                                       const int64_t* __restrict__ pt_off,
                                                       const int64_t* __restrict__ face_off,
                                                       int32_t H) {
  for (int32_t h = blockIdx.y; h < H; h += gridDim.y) {
    const int64_t o = pt_off[h], e = pt_off[h + 1];
    const bool big = e - o > kVolMaxLds || face_off[h + 1] - face_off[h] >= (int64_t(1) << 29);
    const int64_t first = h == 0 ? 0 : o, last = big ? e : (h == 0 ? o : first);
    for (int64_t q = 3 * first + blockIdx.x * (int64_t)blockDim.x + threadIdx.x; q < 3 * last;
         q += (int64_t)gridDim.x * blockDim.x)
      g[q] = 0.f;
  }
}

// What one face adds to the gradient rows of its corners a, b, d.
struct FaceGrad {
  float3 a, b, d;
};
__device__ __forceinline__ FaceGrad face_grad(float3 a, float3 b, float3 d, float sv, float sa) {
  const float3 n = cross3(sub3(b, a), sub3(d, a));
  const float nn = sqrtf(dot3(n, n));
  const float inv = nn > 0.f ? sa / nn : 0.f;
  const float3 m = make_float3(n.x * inv, n.y * inv, n.z * inv);  // gA/2 * unit normal
  const float3 v = make_float3(n.x * sv, n.y * sv, n.z * sv);    // gV/6 * n
  const float3 ga = cross3(sub3(b, d), m), gb = cross3(sub3(d, a), m), gd = cross3(sub3(a, b), m);
  FaceGrad r;
  r.a = make_float3(v.x + ga.x, v.y + ga.y, v.z + ga.z);
  r.b = make_float3(v.x + gb.x, v.y + gb.y, v.z + gb.z);
  r.d = make_float3(v.x + gd.x, v.y + gd.y, v.z + gd.z);
  return r;
}
__device__ __forceinline__ void add3(float* p, float3 v) {
  atomicAdd(p + 0, v.x);
  atomicAdd(p + 1, v.y);
  atomicAdd(p + 2, v.z);
}

// Cloud blockIdx.x: range blockIdx.y of its points (or, too large a cloud, a share of its faces).
__global__ void __launch_bounds__(kVolBwdThreads)
    k_vol_area_bwd(const float* __restrict__ p, const int64_t* __restrict__ pt_off,
                   const int32_t* __restrict__ faces, const int64_t* __restrict__ face_off,
                   const float* __restrict__ gV, const float* __restrict__ gA,
                   float* __restrict__ grad) {
  constexpr int T = kVolBwdThreads;
  __shared__ float acc[3 * kVolRange];
  const int h = blockIdx.x, tid = threadIdx.x;
  const int64_t po = pt_off[h], pn = pt_off[h + 1] - po;
  const int64_t f0 = face_off[h], f1 = face_off[h + 1];
  const float sv = gV ? gV[h] / 6.f : 0.f, sa = gA ? gA[h] * 0.5f : 0.f;
  if (pn > kVolMaxLds || f1 - f0 >= (int64_t(1) << 29)) {
    for (int64_t f = f0 + blockIdx.y * (int64_t)T + tid; f < f1; f += (int64_t)gridDim.y * T) {
      const int64_t ia = po + faces[3 * f], ib = po + faces[3 * f + 1], id = po + faces[3 * f + 2];
      const FaceGrad g = face_grad(ld3(p, ia), ld3(p, ib), ld3(p, id), sv, sa);
      add3(&grad[3 * ia], g.a);
      add3(&grad[3 * ib], g.b);
      add3(&grad[3 * id], g.d);
    }
    return;
  }
  const int F = (int)(f1 - f0);
  const int32_t* fc = faces + 3 * f0;
  const float* pc = p + 3 * po;
  const int64_t r0 = (int64_t)blockIdx.y * kVolRange;
  if (r0 < pn) {
    const int rn = (int)(pn - r0 < kVolRange ? pn - r0 : kVolRange);
    const int base = (int)r0;
    const auto inside = [=](int i) { return (unsigned)(i - base) < (unsigned)rn; };
    for (int q = tid; q < 3 * rn; q += T) acc[q] = 0.f;
    __syncthreads();
    for (int f = tid; f < F; f += T * kVolFaces) {
      int ia[kVolFaces], ib[kVolFaces], id[kVolFaces];
      bool use[kVolFaces];
      float3 a[kVolFaces], b[kVolFaces], d[kVolFaces];
#pragma unroll
      for (int j = 0; j < kVolFaces; ++j) {
        const int x = f + j * T < F ? f + j * T : f;
        ia[j] = fc[3 * x];
        ib[j] = fc[3 * x + 1];
        id[j] = fc[3 * x + 2];
      }
#pragma unroll
      for (int j = 0; j < kVolFaces; ++j) {
        use[j] = f + j * T < F && (inside(ia[j]) || inside(ib[j]) || inside(id[j]));
        if (use[j]) {
          a[j] = ld3(pc, ia[j]);
          b[j] = ld3(pc, ib[j]);
          d[j] = ld3(pc, id[j]);
        }
      }
#pragma unroll
      for (int j = 0; j < kVolFaces; ++j) {
        if (!use[j]) continue;
        const FaceGrad g = face_grad(a[j], b[j], d[j], sv, sa);
        if (inside(ia[j])) add3(&acc[3 * (ia[j] - base)], g.a);
        if (inside(ib[j])) add3(&acc[3 * (ib[j] - base)], g.b);
        if (inside(id[j])) add3(&acc[3 * (id[j] - base)], g.d);
      }
    }
    __syncthreads();
    for (int q = tid; q < 3 * rn; q += T) grad[3 * (po + r0) + q] = acc[q];
  }
}

}  // namespace hull

extern "C" {

int32_t hull_volume_area_fwd(const float* d_p, const int64_t* d_pt_off, const int32_t* d_faces,
                             const int64_t* d_face_off, int32_t H, float* d_V, float* d_A,
                             void* stream) {
  if (H < 0 || (H > 0 && (!d_p || !d_pt_off || !d_faces || !d_face_off || !d_V || !d_A)))
    return HULL_EINVAL;
  if (H == 0) return HULL_OK;
  hull::clear_stale_hip_error();
  hipLaunchKernelGGL(hull::k_vol_area_fwd, dim3(H), dim3(hull::kVolThreads), 0,
                     (hipStream_t)stream, d_p, d_pt_off, d_faces, d_face_off, d_V, d_A);
  HULL_LAUNCH_CHECK();
  return HULL_OK;
}

int32_t hull_volume_area_bwd(const float* d_p, const int64_t* d_pt_off, const int32_t* d_faces,
                             const int64_t* d_face_off, int32_t H, const float* d_gV,
                             const float* d_gA, float* d_grad_p, void* stream) {
  if (H < 0 || (H > 0 && (!d_p || !d_pt_off || !d_faces || !d_face_off || !d_grad_p)))
    return HULL_EINVAL;
  if (H == 0) return HULL_OK;
  hull::clear_stale_hip_error();
  hipStream_t s = (hipStream_t)stream;
  hipLaunchKernelGGL(hull::k_vol_area_zero, dim3(32, H < 64 ? H : 64), dim3(256), 0, s, d_grad_p,
                     d_pt_off, d_face_off, H);
  hipLaunchKernelGGL(hull::k_vol_area_bwd, dim3(H, hull::kVolRanges), dim3(hull::kVolBwdThreads), 0,
                     s, d_p, d_pt_off, d_faces, d_face_off, d_gV, d_gA, d_grad_p);
  HULL_LAUNCH_CHECK();
  return HULL_OK;
}

}  // extern "C"
