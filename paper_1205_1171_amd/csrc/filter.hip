// Interior points leave before the sort.  A point strictly inside the hull of
// other input points is no vertex of the hull, whatever the symbolic
// perturbation (it moves points by infinitesimals), and taking it away
// changes neither the faces nor their order (ranks keep their order, and the
// perturbation goes by the input index a point carries).
//
// The certificate is a star of tetrahedra around a centre c, the mean of 256
// input points (so c lies in their hull):
//   - directions from c are cut into G x G cells (the octahedral map: the
//     sphere's directions unfolded onto a square); every cell's representative
//     is its point farthest from c;
//   - the representatives of four adjacent cells give two triangles, and with c
//     two tetrahedra of points of the hull;
//   - a point strictly inside one of the eight tetrahedra around its cell (which
//     hold the cell's directions whatever the representatives' places in their
//     cells) is dropped.
// A tetrahedron that is flat or misses a corner drops nothing, so any input is
// safe.  Most points need no tetrahedron: when every one of a grid's is
// positively oriented, their triangles are a closed surface around c that
// meets every direction (its signed solid angles are all positive, so it winds
// around c at least once), and the ball up to its nearest plane lies inside.
// Kept: 13,400 of 2^20 points of a ball (whose hull has 4,600 vertices), 13,700
// of a cube, all of a sphere; of 2^24 points, 1% on a sphere around a Gaussian,
// the sphere's.  That cloud's hull took 26.6 ms with every point, 3.1 with the
// filter (0.28 of them the filter's).
//
// Arithmetic: coordinates relative to c, each axis scaled by a power of two to
// |q| <= 1 (exact in double: 256 samples add 8 bits to at most 43), rounded to
// float.  Every tetrahedron is stored as four planes with unit normals, made in
// double and rounded to float; a dot product of such a normal with q is
// within 2^-21 |q|_1 (2^-24 each for the normal, for q and for three products
// and sums), and the tests ask for a margin of 2^-20 |q|_1.  A tetrahedron's
// orientation is taken from a determinant in double, and those below 2^-24 (in
// units where |q| <= 1) are not used.
#include <algorithm>
#include <limits>

#include "common.hpp"
#include "predicates.hpp"

namespace hull {

constexpr int kCoarse = 8;       // cells per side of the first test (its tetrahedra in LDS)
constexpr int kFilterTile = 1024;  // points per block of the mask and the compaction
constexpr double kMinDet = 0x1p-24;

struct FilterArgs {
  int64_t n;
  Header* h;
  unsigned long long* reps;  // [G * G] (|q|^2 as float bits, point), 0: empty
  float4* quads;             // [(kCoarse + 1)^2 + (G + 1)^2] x 8
  unsigned long long* mask;  // [ceil(n / 1024) * 16] points kept
  int32_t* tcnt;             // [ceil(n / 1024)] points kept per tile, then their offsets
  uint32_t* keys;            // kept points: x - min x
  int32_t* vals;             //              index
  int64_t* off1;             // [1] receives the number of points kept
  int G;
};

struct Frame {
  double c[3], s[3];
};
// A power of two that takes a span to 1 at most.
__device__ __forceinline__ double scale_of(double span) {
  int e = 0;
  (void)frexp(span > 1.0 ? span : 1.0, &e);  // span <= 2^e
  return ldexp(1.0, -e);
}
__device__ __forceinline__ Frame frame_of(const Header* h) {
  Frame f;
  for (int a = 0; a < 3; ++a) {
    f.c[a] = h->csum[a] * (1.0 / 256.0);
    f.s[a] = scale_of((double)(h->hi[a] - h->lo[a]));
  }
  return f;
}
template <class InT>
__device__ __forceinline__ void rel(const Frame& f, const InT c[3], double q[3]) {
  for (int a = 0; a < 3; ++a) q[a] = ((double)c[a] - f.c[a]) * f.s[a];
}
template <class InT>
__device__ __forceinline__ void rel(const Frame& f, const InT* xyz, int64_t i, double q[3]) {
  for (int a = 0; a < 3; ++a) q[a] = ((double)xyz[3 * i + a] - f.c[a]) * f.s[a];
}
__device__ __forceinline__ float abs1(float x, float y, float z) { return fabsf(x) + fabsf(y) + fabsf(z); }

// The direction of q on the unit square (any rounding will do: the square only
// says which tetrahedra to try).
__device__ __forceinline__ void square_of(float x, float y, float z, float& u, float& v) {
  const float l = 1.0f / fmaxf(abs1(x, y, z), 1e-30f);
  u = x * l;
  v = y * l;
  if (z < 0) {
    const float a = copysignf(1.0f - fabsf(v), u), b = copysignf(1.0f - fabsf(u), v);
    u = a;
    v = b;
  }
  u = u * 0.5f + 0.5f;
  v = v * 0.5f + 0.5f;
}
__device__ __forceinline__ int cell_at(float u, int G) {
  const int i = (int)(u * (float)G);
  return i < 0 ? 0 : (i > G - 1 ? G - 1 : i);
}

// Extent of each axis, the range check, and (block 0) the sum of 256 samples.
// Clears the representatives.
template <class InT>
__global__ void __launch_bounds__(256) k_extent(const InT* __restrict__ xyz, int64_t n, Header* h,
                                                unsigned long long* reps, int nreps) {
  __shared__ long long smin[3][256], smax[3][256];
  __shared__ int sbad[256];
  const int t = threadIdx.x;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + t; i < nreps; i += (int64_t)gridDim.x * blockDim.x)
    reps[i] = 0;
  InT lo[3], hi[3];
  for (int a = 0; a < 3; ++a) {
    lo[a] = std::numeric_limits<InT>::max();
    hi[a] = std::numeric_limits<InT>::lowest();
  }
  int bad = 0;
  for (int64_t p = blockIdx.x * (int64_t)blockDim.x + t; p < n; p += (int64_t)gridDim.x * blockDim.x) {
    const InT c[3] = {xyz[3 * p], xyz[3 * p + 1], xyz[3 * p + 2]};
    const bool b = pt_out_of_range(c[0], c[1], c[2]);
    bad |= b;
    for (int a = 0; a < 3; ++a) {  // rows out of range count as zero
      const InT v = b ? 0 : c[a];
      lo[a] = v < lo[a] ? v : lo[a];
      hi[a] = v > hi[a] ? v : hi[a];
    }
  }
  for (int a = 0; a < 3; ++a) {
    smin[a][t] = lo[a];
    smax[a][t] = hi[a];
  }
  sbad[t] = bad;
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (t < s) {
      for (int a = 0; a < 3; ++a) {
        smin[a][t] = min(smin[a][t], smin[a][t + s]);
        smax[a][t] = max(smax[a][t], smax[a][t + s]);
      }
      sbad[t] |= sbad[t + s];
    }
    __syncthreads();
  }
  if (t < 3) {
    // the device's rows only narrow an extent that others have widened
    atomicMin(&h->lo[t], smin[t][0]);
    atomicMax(&h->hi[t], smax[t][0]);
  }
  if (t == 0 && sbad[0]) atomicCAS(&h->err, 0, HULL_ERANGE);
  if (blockIdx.x != 0) return;
  __syncthreads();
  for (int a = 0; a < 3; ++a) smin[a][t] = (long long)xyz[3 * ((int64_t)t * n / 256) + a];
  __syncthreads();
  for (int s = 128; s > 0; s >>= 1) {
    if (t < s)
      for (int a = 0; a < 3; ++a) smin[a][t] += smin[a][t + s];
    __syncthreads();
  }
  if (t < 3) h->csum[t] = (double)smin[t][0];
}

template <class InT>
__global__ void __launch_bounds__(256) k_reps(const InT* __restrict__ xyz, FilterArgs F) {
  extern __shared__ unsigned long long best[];
  const int cells = F.G * F.G;
  if (F.h->err) return;
  for (int q = threadIdx.x; q < cells; q += blockDim.x) best[q] = 0;
  __syncthreads();
  const Frame f = frame_of(F.h);
  for (int64_t p = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; p < F.n;
       p += (int64_t)gridDim.x * blockDim.x) {
    double q[3];
    rel(f, xyz, p, q);
    const float x = (float)q[0], y = (float)q[1], z = (float)q[2];
    float u, v;
    square_of(x, y, z, u, v);
    const int c = cell_at(v, F.G) * F.G + cell_at(u, F.G);
    const unsigned long long key =
        ((unsigned long long)__float_as_uint(x * x + y * y + z * z) << 32) | (unsigned)p;
    if (key > best[c]) atomicMax(&best[c], key);
  }
  __syncthreads();
  for (int q = threadIdx.x; q < cells; q += blockDim.x)
    if (best[q] > __hip_atomic_load(&F.reps[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(&F.reps[q], best[q]);
}

// Cells across the edges of the square: the octahedron's edges there fold onto
// themselves.
__device__ __forceinline__ void wrap_cell(int& i, int& j, int G) {
  if (i < 0) { i = 0; j = G - 1 - j; }
  else if (i >= G) { i = G - 1; j = G - 1 - j; }
  if (j < 0) { j = 0; i = G - 1 - i; }
  else if (j >= G) { j = G - 1; i = G - 1 - i; }
}

__device__ double det3(const double* a, const double* b, const double* d) {
  return (a[1] * b[2] - a[2] * b[1]) * d[0] + (a[2] * b[0] - a[0] * b[2]) * d[1] +
         (a[0] * b[1] - a[1] * b[0]) * d[2];
}

// The tetrahedron (c, a, b, d) as three planes through c and the outer one;
// left zero when it is flat.  Returns the outer plane's distance from c, 0
// unless the tetrahedron is positively oriented.
__device__ float tetra(const double* a, const double* b, const double* d, float4* out) {
  auto cross = [](const double* p, const double* q, double* r) {
    r[0] = p[1] * q[2] - p[2] * q[1];
    r[1] = p[2] * q[0] - p[0] * q[2];
    r[2] = p[0] * q[1] - p[1] * q[0];
  };
  // (the normals are not zero: the determinant is not; two Newton steps on the
  // estimate of the reciprocal root, relative error below 2^-44)
  auto unit = [](double* r, double sg) {
    const double l2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2];
    double y = __builtin_amdgcn_rsq(l2);
    y = y * (1.5 - 0.5 * l2 * y * y);
    y = y * (1.5 - 0.5 * l2 * y * y) * sg;
    for (int k = 0; k < 3; ++k) r[k] *= y;
  };
  double ab[3], bd[3], da[3], n[3], e[3], g[3];
  cross(a, b, ab);
  const double det = ab[0] * d[0] + ab[1] * d[1] + ab[2] * d[2];
  if (!(fabs(det) > kMinDet)) {
    for (int k = 0; k < 4; ++k) out[k] = make_float4(0, 0, 0, 0);
    return 0.0f;
  }
  const double sg = det > 0 ? 1.0 : -1.0;
  cross(b, d, bd);
  cross(d, a, da);
  for (int k = 0; k < 3; ++k) {
    e[k] = b[k] - a[k];
    g[k] = d[k] - a[k];
  }
  cross(e, g, n);
  unit(ab, sg);
  unit(bd, sg);
  unit(da, sg);
  unit(n, sg);
  const double h = n[0] * a[0] + n[1] * a[1] + n[2] * a[2];
  out[0] = make_float4((float)ab[0], (float)ab[1], (float)ab[2], (float)n[0]);
  out[1] = make_float4((float)bd[0], (float)bd[1], (float)bd[2], (float)n[1]);
  out[2] = make_float4((float)da[0], (float)da[1], (float)da[2], (float)n[2]);
  const float dist = (float)(h * (1.0 - 0x1p-22));
  out[3] = make_float4(dist, 0, 0, 0);
  return det > 0 ? dist : 0.0f;
}

// The two tetrahedra of the 2 x 2 block of adjacent cells at corner (qi, qj) of a
// grid of g cells per side, from the cells' representatives rep(i, j) (0: none).
// Returns the distance of their nearest outer plane, 0 if one is not positively
// oriented, and a large number for a block that folds onto one edge.
template <class InT, class REP>
__device__ float quad(const InT* xyz, const Frame& f, int g, int qi, int qj, const REP& rep, float4* out) {
  double v[4][3];
  int cell[4];
  bool ok = true;
  for (int k = 0; k < 4; ++k) {
    int i = qi - (k == 0 || k == 3), j = qj - (k < 2);
    wrap_cell(i, j, g);
    cell[k] = j * g + i;
    const unsigned long long key = rep(i, j);
    ok = ok && key != 0;
    rel(f, xyz, (int64_t)(unsigned)key, v[k]);
  }
  if (!ok)
    for (int k = 0; k < 3; ++k) v[1][k] = v[3][k] = 0.0;
  // the diagonal that leaves both triangles positively oriented, if one does
  const double d02 = fmin(det3(v[0], v[1], v[2]), det3(v[0], v[2], v[3]));
  const double d13 = fmin(det3(v[1], v[2], v[3]), det3(v[1], v[3], v[0]));
  const bool swap = d13 > d02;
  const double *a = swap ? v[1] : v[0], *b = swap ? v[2] : v[1], *c = swap ? v[3] : v[2],
               *d = swap ? v[0] : v[3];
  const float r0 = tetra(a, b, c, out), r1 = tetra(a, c, d, out + 4);
  // in the middle of the square's edges a block folds onto one edge of the
  // surface
  return cell[0] != cell[2] && cell[1] != cell[3] ? fminf(r0, r1) : 3e38f;
}

// Every block's tetrahedra, at kCoarse cells per side (a coarse cell's
// representative: the farthest of its cells') and at G.
template <class InT>
__global__ void __launch_bounds__(64) k_mesh(const InT* __restrict__ xyz, FilterArgs F) {
  if (F.h->err) return;
  const int nc = (kCoarse + 1) * (kCoarse + 1), nf = (F.G + 1) * (F.G + 1);
  int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t >= nc + nf) return;
  float4* out = F.quads + 8 * (int64_t)t;
  const int grid = t >= nc;  // 0: the coarse cells, 1: the fine ones
  const int g = grid ? F.G : kCoarse, per = F.G / g;
  if (grid) t -= nc;
  const Frame f = frame_of(F.h);
  const auto rep = [&](int i, int j) {
    unsigned long long key = 0;
    for (int y = 0; y < per; ++y)
      for (int x = 0; x < per; ++x) {
        const unsigned long long c = F.reps[(j * per + y) * F.G + i * per + x];
        key = c > key ? c : key;
      }
    return key;
  };
  const float r = quad(xyz, f, g, t % (g + 1), t / (g + 1), rep, out);
  atomicMin(&F.h->rho[grid], __float_as_uint(r));
}

__device__ __forceinline__ bool inside(const float4* T, float x, float y, float z, float l1) {
  const float tol = 0x1p-20f * l1;
  bool in = false;
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const float4 a = T[4 * k], b = T[4 * k + 1], c = T[4 * k + 2];
    const float d = T[4 * k + 3].x;
    const float p = a.x * x + a.y * y + a.z * z, q = b.x * x + b.y * y + b.z * z,
                r = c.x * x + c.y * y + c.z * z, o = a.w * x + b.w * y + c.w * z;
    in = in || (p > tol && q > tol && r > tol && o < d - tol);
  }
  return in;
}

// The tetrahedra at the four corners of the cell of (u, v).
__device__ __forceinline__ bool inside_around(const float4* quads, int G, float u, float v, float x,
                                              float y, float z, float l1) {
  const int i = cell_at(u, G), j = cell_at(v, G);
  bool in = false;
  for (int k = 0; k < 4 && !in; ++k)
    in = inside(quads + 8 * ((j + (k >> 1)) * (G + 1) + i + (k & 1)), x, y, z, l1);
  return in;
}

// Points kept, as bits, and their number per tile.  The ball decides most; the
// others are listed in LDS, so that the tetrahedra are tested by full wavefronts.
template <class InT>
__global__ void __launch_bounds__(256) k_mask(const InT* __restrict__ xyz, FilterArgs F) {
  constexpr int nc = (kCoarse + 1) * (kCoarse + 1);
  __shared__ float4 coarse[8 * nc];
  __shared__ unsigned short list[kFilterTile];
  __shared__ unsigned mask[kFilterTile / 32];
  __shared__ int listed, count;
  if (F.h->err) return;
  const int t = threadIdx.x;
  for (int q = t; q < 8 * nc; q += 256) coarse[q] = F.quads[q];
  if (t < kFilterTile / 32) mask[t] = 0;
  if (t == 0) listed = count = 0;
  __syncthreads();
  const Frame f = frame_of(F.h);
  const float rho = fmaxf(__uint_as_float(F.h->rho[0]), __uint_as_float(F.h->rho[1]));
  const float rr = rho * rho * (1.0f - 0x1p-18f);
  const int64_t base = (int64_t)blockIdx.x * kFilterTile;
  const int64_t left = F.n - base;
  for (int j = t; j < kFilterTile && j < left; j += 256) {
    double q[3];
    rel(f, xyz, base + j, q);
    const float x = (float)q[0], y = (float)q[1], z = (float)q[2];
    if (!(x * x + y * y + z * z < rr)) list[atomicAdd(&listed, 1)] = (unsigned short)j;
  }
  __syncthreads();
  int kept = 0;
  for (int k = t; k < listed; k += 256) {
    const int j = list[k];
    double q[3];
    rel(f, xyz, base + j, q);
    const float x = (float)q[0], y = (float)q[1], z = (float)q[2], l1 = abs1(x, y, z);
    float u, v;
    square_of(x, y, z, u, v);
    if (inside_around(coarse, kCoarse, u, v, x, y, z, l1)) continue;
    if (F.G > kCoarse && inside_around(F.quads + 8 * nc, F.G, u, v, x, y, z, l1)) continue;
    atomicOr(&mask[j >> 5], 1u << (j & 31));
    ++kept;
  }
  if (kept) atomicAdd(&count, kept);
  __syncthreads();
  if (t < kFilterTile / 64)
    F.mask[(base >> 6) + t] = mask[2 * t] | ((unsigned long long)mask[2 * t + 1] << 32);
  if (t == 0) F.tcnt[blockIdx.x] = count;
}

// The kept points in input order: keys and indices for the sort.
template <class InT>
__global__ void __launch_bounds__(256) k_compact(const InT* __restrict__ xyz, FilterArgs F) {
  constexpr int words = kFilterTile / 64;
  __shared__ int before[words];
  const int t = threadIdx.x;
  if (F.h->err) {  // no merge runs
    if (blockIdx.x == 0 && t == 0) {
      F.off1[1] = 0;
      F.h->radix_len = 0;
    }
    return;
  }
  const int64_t base = (int64_t)blockIdx.x * kFilterTile;
  if (t < words) {
    const int c = __popcll(F.mask[(base >> 6) + t]);
    int incl = c;
    for (int o = 1; o < words; o <<= 1) {
      const int y = __shfl_up(incl, o, words);
      if (t >= o) incl += y;
    }
    before[t] = F.tcnt[blockIdx.x] + incl - c;
  }
  __syncthreads();
  const long long minx = F.h->lo[0];
  for (int j = 0; j < kFilterTile / 256; ++j) {
    const int w = j * 4 + (t >> 6);
    const unsigned long long m = F.mask[(base >> 6) + w];
    if (!((m >> (t & 63)) & 1)) continue;
    const int64_t p = base + j * 256 + t;
    const int at = before[w] + __popcll(m & ((1ull << (t & 63)) - 1));
    F.keys[at] = (uint32_t)((long long)xyz[3 * p] - minx);
    F.vals[at] = (int32_t)p;
  }
  if (blockIdx.x == 0 && t == 0) {
    F.off1[1] = F.h->kept;
    F.h->radix_len = (F.h->kept + kTile - 1) / kTile * kBuckets;
  }
}

// ---------------------------------------------------------------------------
// Batches: the same, one workgroup per cloud, with the grid in LDS.
// ---------------------------------------------------------------------------
struct CloudArgs {
  const int64_t* off;  // [H + 1] the clouds' points
  int64_t H;
  const Header* h;
  int32_t* list;       // [n] cloud h's kept points from off[h] on
  int32_t* kept;       // [H + 1] their number
  int64_t lo, hi;      // clouds of lo <= points < hi
};

constexpr int kCloudThreads = 512;
constexpr int64_t kCloudMin = 256;  // smaller clouds keep every point

// The points of a cloud for a block of NT threads: point p = threadIdx.x + j NT of
// every pass is read from memory, or (PER > 0, at most PER NT points) was
// loaded into registers once, all loads in flight together.
template <int NT, int PER, class InT>
struct CloudPoints {
  const InT* P;
  int n;
  InT c[PER > 0 ? PER : 1][3];
  __device__ __forceinline__ CloudPoints(const InT* points, int count) : P(points), n(count) {
    if constexpr (PER > 0) {
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        const int p = threadIdx.x + j * NT;
        for (int a = 0; a < 3; ++a) c[j][a] = p < n ? P[3 * (int64_t)p + a] : 0;
      }
    }
  }
  template <class FN>
  __device__ __forceinline__ void each(const FN& fn) const {
    if constexpr (PER > 0) {
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        const int p = threadIdx.x + j * NT;
        if (p < n) fn(p, c[j]);
      }
    } else {
      for (int p = threadIdx.x; p < n; p += NT) {
        const InT x[3] = {P[3 * (int64_t)p], P[3 * (int64_t)p + 1], P[3 * (int64_t)p + 2]};
        fn(p, x);
      }
    }
  }
};

// Extent, range check and frame of a cloud (red: 10 words).
template <int NT, class PTS, class InT>
__device__ __forceinline__ Frame cloud_frame(const PTS& pts, const InT* P, int n, long long* red, long long& minx,
                                             bool& bad) {
  const int t = threadIdx.x;
  __syncthreads();  // earlier readers of red
  if (t < 10) red[t] = t < 3 ? 0x7fffffffffffffffll : (t < 6 ? -0x7fffffffffffffffll - 1 : 0);
  InT lo[3], hi[3], sample[3];
  for (int a = 0; a < 3; ++a) {
    lo[a] = std::numeric_limits<InT>::max();
    hi[a] = std::numeric_limits<InT>::lowest();
    sample[a] = t < 256 ? P[3 * ((int64_t)t * n / 256) + a] : 0;
  }
  int out = 0;
  pts.each([&](int, const InT* c) {
    for (int a = 0; a < 3; ++a) {
      lo[a] = c[a] < lo[a] ? c[a] : lo[a];
      hi[a] = c[a] > hi[a] ? c[a] : hi[a];
    }
    out |= pt_out_of_range(c[0], c[1], c[2]);
  });
  __syncthreads();
  // by wavefront first: atomics of many lanes on one word take their turns
  long long sum[3] = {sample[0], sample[1], sample[2]};
  for (int a = 0; a < 3; ++a) {
    for (int o = 32; o > 0; o >>= 1) {
      const InT l = __shfl_xor(lo[a], o), u = __shfl_xor(hi[a], o);
      lo[a] = l < lo[a] ? l : lo[a];
      hi[a] = u > hi[a] ? u : hi[a];
    }
    if (t < 256)
      for (int o = 32; o > 0; o >>= 1) sum[a] += __shfl_xor(sum[a], o);
  }
  const bool any = __ballot(out) != 0;
  if ((t & 63) == 0 && t < n) {
    for (int a = 0; a < 3; ++a) {
      atomicMin(&red[a], (long long)lo[a]);
      atomicMax(&red[3 + a], (long long)hi[a]);
    }
    if (any) atomicOr((unsigned long long*)&red[9], 1ull);
  }
  if ((t & 63) == 0 && t < 256)
    for (int a = 0; a < 3; ++a) atomicAdd((unsigned long long*)&red[6 + a], (unsigned long long)sum[a]);
  __syncthreads();
  Frame f;
  for (int a = 0; a < 3; ++a) {
    f.c[a] = (double)red[6 + a] * (1.0 / 256.0);
    f.s[a] = scale_of((double)(red[3 + a] - red[a]));
  }
  minx = red[0];
  bad = red[9] != 0;
  return f;
}

// Representatives and tetrahedra of a cloud in LDS; returns the square of the
// ball's radius.
template <int NT, int G, class PTS, class InT>
__device__ __forceinline__ float cloud_grid(const PTS& pts, const InT* P, const Frame& f, unsigned long long* reps,
                                            float4* quads, unsigned* rho) {
  constexpr int nq = (G + 1) * (G + 1);
  const int t = threadIdx.x;
  for (int q = t; q < G * G; q += NT) reps[q] = 0;
  if (t == 0) *rho = 0x7f7fffffu;
  __syncthreads();
  pts.each([&](int p, const InT* xyz) {
    double q[3];
    rel(f, xyz, q);
    const float x = (float)q[0], y = (float)q[1], z = (float)q[2];
    float u, v;
    square_of(x, y, z, u, v);
    const int c = cell_at(v, G) * G + cell_at(u, G);
    const unsigned long long key =
        ((unsigned long long)__float_as_uint(x * x + y * y + z * z) << 32) | (unsigned)p;
    if (key > reps[c]) atomicMax(&reps[c], key);
  });
  __syncthreads();
  for (int k = t; k < nq; k += NT) {
    const float r = quad(P, f, G, k % (G + 1), k / (G + 1), [&](int i, int j) { return reps[j * G + i]; },
                         quads + 8 * k);
    atomicMin(rho, __float_as_uint(r));
  }
  __syncthreads();
  const float radius = __uint_as_float(*rho);
  return radius * radius * (1.0f - 0x1p-18f);
}

// May a point be a vertex, as far as the grid can tell?
template <int G, class InT>
__device__ __forceinline__ bool cloud_keeps(const InT* xyz, const Frame& f, const float4* quads, float rr) {
  double q[3];
  rel(f, xyz, q);
  const float x = (float)q[0], y = (float)q[1], z = (float)q[2];
  if (x * x + y * y + z * z < rr) return false;
  float u, v;
  square_of(x, y, z, u, v);
  return !inside_around(quads, G, u, v, x, y, z, abs1(x, y, z));
}

template <class InT, int G>
__global__ void __launch_bounds__(kCloudThreads) k_cloud_filter(const InT* __restrict__ xyz, CloudArgs A) {
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  constexpr int nq = (G + 1) * (G + 1), T = kCloudThreads;
  float4* quads = (float4*)dyn_lds;                                    // [8 nq]
  unsigned long long* reps = (unsigned long long*)(quads + 8 * nq);    // [G * G]
  __shared__ long long red[10];
  __shared__ unsigned rho;
  __shared__ int wcnt[2][T / 64];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  for (int64_t h = blockIdx.x; h < A.H; h += gridDim.x) {
    const int64_t o = A.off[h];
    const int64_t n64 = A.off[h + 1] - o;
    if (n64 < A.lo || n64 >= A.hi) continue;  // the same for the whole block
    const int n = (int)n64;
    const InT* P = xyz + 3 * o;
    int32_t* list = A.list + o;
    // (A.h->err was settled by an earlier launch: the same for the whole block)
    if (A.h->err || n < kCloudMin) {
      for (int p = t; p < n; p += T) list[p] = (int32_t)(o + p);
      if (t == 0) A.kept[h] = n;
      continue;
    }
    long long minx;
    bool bad;  // (the range was checked by an earlier launch)
    const CloudPoints<T, 0, InT> pts(P, n);
    const Frame f = cloud_frame<T>(pts, P, n, red, minx, bad);
    const float rr = cloud_grid<T, G>(pts, P, f, reps, quads, &rho);
    // kept points in input order
    int done = 0;
    for (int p0 = 0, turn = 0; p0 < n; p0 += T, turn ^= 1) {
      const int p = p0 + t;
      const bool keep = p < n && cloud_keeps<G>(P + 3 * (int64_t)p, f, quads, rr);
      const unsigned long long m = __ballot(keep);
      if (lane == 0) wcnt[turn][wave] = __popcll(m);
      __syncthreads();  // (two sets of counts: one barrier a turn)
      int before = 0, all = 0;
      for (int w = 0; w < T / 64; ++w) {
        const int c = wcnt[turn][w];
        before += w < wave ? c : 0;
        all += c;
      }
      if (keep) list[done + before + __popcll(m & ((1ull << lane) - 1))] = (int32_t)(o + p);
      done += all;
    }
    if (t == 0) A.kept[h] = done;
    __syncthreads();  // the next cloud rewrites the grid
  }
}

// The clouds' kept points one after the other: their offsets, and the sort's
// list (key, index) with the hull of each.
template <class InT>
__global__ void __launch_bounds__(256) k_cloud_list(const InT* __restrict__ xyz, CloudArgs A,
                                                    const int32_t* __restrict__ before, Header* h,
                                                    int64_t* off2, uint32_t* keys, int32_t* vals, int32_t* hid) {
  const int64_t i0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x, step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t q = i0; q <= A.H; q += step) off2[q] = before[q];
  const int total = before[A.H];
  const long long minx = h->lo[0];
  for (int64_t r = i0; r < total; r += step) {
    int64_t lo = 0, hi = A.H;  // largest cloud with before <= r
    while (hi - lo > 1) {
      const int64_t mid = (lo + hi) >> 1;
      if (before[mid] <= r) lo = mid;
      else hi = mid;
    }
    const int32_t p = A.list[A.off[lo] + (r - before[lo])];
    keys[r] = (uint32_t)((long long)xyz[3 * (int64_t)p] - minx);
    vals[r] = p;
    hid[p] = (int32_t)lo;
  }
  if (i0 == 0) h->radix_len = (int32_t)(((int64_t)total + kTile - 1) / kTile * kBuckets);
}

// Cells per side: finer cells follow the surface closer but take more
// representatives, and a cell should hold tens of points for its farthest to
// be near the surface.
static int filter_cells(int64_t n) { return n >= (1 << 17) ? 32 : (n >= (1 << 13) ? 16 : kCoarse); }

template <class InT>
int32_t extent_and_filter(const InT* d_xyz, int64_t n, bool filter, char* ws, const Plan& pl,
                          hipStream_t s) {
  Header* h = (Header*)(ws + pl.header);
  FilterArgs F{};
  F.n = n;
  F.h = h;
  F.G = filter_cells(n);
  // in the space of the merge levels' event places (32 bytes per point)
  char* o = ws + pl.pos[0];
  auto take = [&](size_t bytes) {
    char* q = o;
    o += (bytes + 255) & ~(size_t)255;
    return q;
  };
  const int64_t tiles = (n + kFilterTile - 1) / kFilterTile;
  const int quads = (kCoarse + 1) * (kCoarse + 1) + (F.G + 1) * (F.G + 1);
  F.reps = (unsigned long long*)take((size_t)F.G * F.G * 8);
  F.quads = (float4*)take((size_t)quads * 8 * sizeof(float4));
  F.mask = (unsigned long long*)take((size_t)tiles * (kFilterTile / 64) * 8);
  F.tcnt = (int32_t*)take((size_t)(tiles + 1) * 4);
  // (kFilterMin points have room)
  if (filter && (size_t)(o - (ws + pl.pos[0])) > 2 * (size_t)n * sizeof(int4)) return HULL_EINTERNAL;
  F.keys = (uint32_t*)(ws + pl.keys1);
  F.vals = (int32_t*)(ws + pl.vals1);
  F.off1 = (int64_t*)(ws + pl.off1);
  const unsigned eg = (unsigned)std::max<int64_t>(1, std::min<int64_t>((n + 255) / 256, 1024));
  hipLaunchKernelGGL(k_extent<InT>, dim3(eg), dim3(256), 0, s, d_xyz, n, h, F.reps,
                     filter ? F.G * F.G : 0);
  if (!filter) return HULL_OK;
  hipLaunchKernelGGL(k_reps<InT>, dim3(std::min(eg, 512u)), dim3(256), (size_t)F.G * F.G * 8, s, d_xyz, F);
  hipLaunchKernelGGL(k_mesh<InT>, dim3((quads + 63) / 64), dim3(64), 0, s, d_xyz, F);
  hipLaunchKernelGGL(k_mask<InT>, dim3((unsigned)tiles), dim3(256), 0, s, d_xyz, F);
  ScanJobs J{};
  J.j[0] = ScanJob{F.tcnt, F.tcnt, nullptr, &h->kept};
  J.count = 1;
  const int32_t rc = exclusive_scan_chained(J, 0, tiles, (unsigned long long*)(ws + pl.chain_words),
                                            pl.chain_stride, kChainEpochFilter, h, s);
  if (rc) return rc;
  hipLaunchKernelGGL(k_compact<InT>, dim3((unsigned)tiles), dim3(256), 0, s, d_xyz, F);
  HULL_LAUNCH_CHECK();
  return HULL_OK;
}

// ---------------------------------------------------------------------------
// Small single hulls: the call's setup, the filter and the sort in one launch of
// one workgroup.
// ---------------------------------------------------------------------------
// Nineteen launches (six of them the filter's) took 61 us for 97 points and 93 for
// 4,096 cube points, 7 and 37 in this one.  The kept points' (x, index) pairs are
// sorted in LDS: chunks of 128 by counting smaller keys (one barrier), then merged
// pair by pair, every key finding its place in the other chunk by binary search
// (a bitonic network takes 28 barriers for 97 points, 78 for 4,096).  The order
// is total, so the points need not arrive in order.
constexpr int kSmallChunk = 128;
constexpr int kSmallGrid = 8;
constexpr size_t kSmallQuads = (size_t)(kSmallGrid + 1) * (kSmallGrid + 1) * 8 * sizeof(float4);

template <class InT, class PT, int T, int PER>
__global__ void __launch_bounds__(T)
    k_small_sort(const InT* __restrict__ xyz, int n, int filter, int cap, Header* h, int64_t* off1,
                 unsigned long long* words, int64_t nwords, PT* __restrict__ out, RunInitPair I) {
  constexpr int G = kSmallGrid, C = kSmallChunk;
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  unsigned long long* keys = (unsigned long long*)dyn_lds;  // [cap], cap >= n + 1, even
  unsigned long long* ordered = keys + cap;                 // [cap] the same, sorted by chunk
  float4* quads = (float4*)(ordered + cap);                 // the filter's grid, if wanted
  unsigned long long* reps = (unsigned long long*)((unsigned char*)quads + kSmallQuads);
  __shared__ long long red[10];
  __shared__ unsigned rho;
  __shared__ int kept;
  const int t = threadIdx.x;
  for (int64_t q = t; q < nwords; q += T) words[q] = 0;
  if (t == 0) kept = 0;
  long long minx;
  bool bad;
  const CloudPoints<T, PER, InT> pts(xyz, n);
  const Frame f = cloud_frame<T>(pts, xyz, n, red, minx, bad);
  if (t == 0) {
    h->err = bad ? HULL_ERANGE : 0;
    off1[0] = 0;
    off1[1] = n;
  }
  for (int q = t; q < kCtrSlots; q += T)
    for (int r = 0; r < 2; ++r)
      if (I.r[r].pv0) I.r[r].ctr[q] = 0;
  if (bad) return;
  if (filter) {
    const float rr = cloud_grid<T, G>(pts, xyz, f, reps, quads, &rho);
    pts.each([&](int p, const InT* c) {
      if (cloud_keeps<G>(c, f, quads, rr))
        keys[atomicAdd(&kept, 1)] = ((unsigned long long)((long long)c[0] - minx) << 32) | (unsigned)p;
    });
    __syncthreads();
  } else {
    pts.each([&](int p, const InT* c) {
      keys[p] = ((unsigned long long)((long long)c[0] - minx) << 32) | (unsigned)p;
    });
  }
  const int m = filter ? kept : n;
  if (t == 0) keys[m] = ~0ull;  // chunks are read in pairs
  __syncthreads();
  for (int p = t; p < m; p += T) {
    const unsigned long long key = keys[p];
    const int base = p / C * C, pairs = (min(C, m - base) + 1) / 2;
    const ulonglong2* c = (const ulonglong2*)(keys + base);
    int r = 0;
#pragma unroll 8
    for (int q = 0; q < pairs; ++q) {
      const ulonglong2 x = c[q];
      r += (x.x < key) + (x.y < key);
    }
    ordered[base + r] = key;
  }
  __syncthreads();
  for (int run = C; run < m; run *= 2) {
    for (int p = t; p < m; p += T) {
      const unsigned long long key = ordered[p];
      const int mine = p / run * run, pair = mine & ~run, other = pair + (mine == pair ? run : 0);
      int lo = 0, hi = max(0, min(run, m - other));
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (ordered[other + mid] < key) lo = mid + 1;
        else hi = mid;
      }
      keys[pair + (p - mine) + lo] = key;
    }
    __syncthreads();
    unsigned long long* x = keys;
    keys = ordered;
    ordered = x;
  }
  for (int r = t; r < m; r += T) {
    const unsigned long long key = ordered[r];
    const int i = (int)(unsigned)key;
    out[r] = make_pt(xyz, i, i);
    for (int q = 0; q < 2; ++q) {
      if (!I.r[q].pv0) continue;
      I.r[q].pv0[r] = kNil;
      I.r[q].nx0[r] = kNil;
      I.r[q].len[r] = 0;
    }
  }
  if (t == 0) off1[1] = m;
}

template <class InT, class PT>
int32_t small_setup_and_sort(const InT* d_xyz, int64_t n, bool filter, char* ws, const Plan& pl,
                             const RunInit* runs, hipStream_t s) {
  const int cap = (int)(n + 2) & ~1;
  const size_t lds = (size_t)cap * 16 + (filter ? kSmallQuads + (size_t)kSmallGrid * kSmallGrid * 8 : 0);
#define HULL_SMALL(T, PER)                                                                                 \
  hipLaunchKernelGGL((k_small_sort<InT, PT, T, PER>), dim3(1), dim3(T), lds, s, d_xyz, (int)n, (int)filter, cap, \
                     (Header*)(ws + pl.header), (int64_t*)(ws + pl.off1),                               \
                     (unsigned long long*)(ws + pl.chain_words), kChainJobs * pl.chain_stride,          \
                     (PT*)(ws + pl.pts), RunInitPair{{runs[0], runs[1]}})
  if (n <= 512) HULL_SMALL(256, 2);
  else if (n <= 4096) HULL_SMALL(1024, 4);
  else HULL_SMALL(1024, 8);
#undef HULL_SMALL
  HULL_LAUNCH_CHECK();
  return HULL_OK;
}

template int32_t small_setup_and_sort<int32_t, int4>(const int32_t*, int64_t, bool, char*, const Plan&,
                                                     const RunInit*, hipStream_t);
template int32_t small_setup_and_sort<int64_t, WPt>(const int64_t*, int64_t, bool, char*, const Plan&,
                                                    const RunInit*, hipStream_t);

// Clouds by size: 8, 16 or 32 cells per side (10, 39 or 148 KB of LDS).  The
// clouds of a batch are small enough for one workgroup each (kCloudMax).
int32_t filter_clouds(const int32_t* d_xyz, int64_t n, const int64_t* d_off, int64_t H, int64_t longest,
                      char* ws, const Plan& pl, hipStream_t s) {
  Header* h = (Header*)(ws + pl.header);
  CloudArgs A{};
  A.off = d_off;
  A.H = H;
  A.h = h;
  A.list = (int32_t*)(ws + pl.pos[0]);
  A.kept = (int32_t*)(ws + pl.mcnt);
  const unsigned grid = (unsigned)std::min<int64_t>(H, 16384);
  const auto lds = [](int G) { return (size_t)(G + 1) * (G + 1) * 8 * sizeof(float4) + (size_t)G * G * 8; };
  A.lo = 0;
  A.hi = 2048;
  hipLaunchKernelGGL((k_cloud_filter<int32_t, 8>), dim3(grid), dim3(kCloudThreads), lds(8), s, d_xyz, A);
  A.lo = 2048;
  A.hi = 8192;
  if (longest >= A.lo)
    hipLaunchKernelGGL((k_cloud_filter<int32_t, 16>), dim3(grid), dim3(kCloudThreads), lds(16), s, d_xyz, A);
  A.lo = 8192;
  A.hi = INT64_MAX;
  if (longest >= A.lo)
    hipLaunchKernelGGL((k_cloud_filter<int32_t, 32>), dim3(grid), dim3(kCloudThreads), lds(32), s, d_xyz, A);
  int32_t* before = (int32_t*)(ws + pl.moff);
  ScanJobs J{};  // entry H is not a cloud: the scan only writes its place
  J.j[0] = ScanJob{A.kept, before, nullptr, nullptr};
  J.count = 1;
  const int32_t rc = exclusive_scan_chained(J, 0, H + 1, (unsigned long long*)(ws + pl.chain_words),
                                            pl.chain_stride, kChainEpochFilter, h, s);
  if (rc) return rc;
  hipLaunchKernelGGL(k_cloud_list<int32_t>, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 4096)), dim3(256),
                     0, s, d_xyz, A, before, h, (int64_t*)(ws + pl.off2), (uint32_t*)(ws + pl.keys1),
                     (int32_t*)(ws + pl.vals1), (int32_t*)(ws + pl.hid));
  HULL_LAUNCH_CHECK();
  return HULL_OK;
}

template int32_t extent_and_filter<int32_t>(const int32_t*, int64_t, bool, char*, const Plan&, hipStream_t);
template int32_t extent_and_filter<int64_t>(const int64_t*, int64_t, bool, char*, const Plan&, hipStream_t);

}  // namespace hull
