// Face adjacency of hull surfaces: for every face and each of its three
// directed edges, the face across that edge (the half-edge twin) -- the
// connectivity of an edge-list structure, which the paper names as the
// prerequisite for further algorithms (Sec. "Conclusion", future work; Sec.
// "Introduction" on the missing doubly connected edge list).
//
// A hash table of undirected edges in the caller's workspace: a slot holds the
// id 3f + k of the first half-edge of its edge to arrive; the second, which
// runs the other way, writes both twins and marks the slot.  The table holds
// ids alone (4 bytes a slot): the key of a slot is read back from the face
// rows.  Clouds of a batch never match each other (a slot's face must lie in
// the same cloud).  Open addressing, linear probing, at least 3.5 slots per
// face for at most 3 entries (every probe sequence ends at an empty slot or
// its edge).  The kernel is bound by its atomics on scattered slots (one
// compare-and-swap per half-edge): 2.1 million faces, 0.67 ms with a table of
// directed edges (16-byte slots, one pass to insert and one to look up),
// 0.41 ms with this one.
#include <algorithm>

#include "common.hpp"

namespace hull {

// Half-edge ids 3f + k are stored as int32: at most this many faces.
constexpr int64_t kMaxAdjFaces = (int64_t(INT32_MAX) - 2) / 3;

constexpr unsigned kMatched = 1u << 31;  // flag of a slot whose edge has both half-edges

__device__ __forceinline__ int64_t owner64(const int64_t* off, int64_t count, int64_t x) {
  int64_t lo = 0, hi = count;
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (off[mid] <= x) lo = mid;
    else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ uint64_t slot_of(unsigned long long key, int bits) {
  return (key * 0x9E3779B97F4A7C15ull) >> (64 - bits);
}

struct AdjArgs {
  const int32_t* faces;
  int64_t F;
  const int64_t* face_off;  // [H + 1] or null (one surface)
  const int64_t* pt_off;    // [H + 1] or null
  int64_t H;
  unsigned* table;  // half-edge id + 1 (0: empty) | kMatched
  int bits;
  int32_t* adj;
  int64_t* info;
  int* err;    // device status word (in the workspace)
  int* open;   // half-edges without a twin
};

__global__ void __launch_bounds__(256) k_adj_clear(AdjArgs A) {
  const int64_t quads = int64_t(1) << (A.bits - 2);
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < quads;
       i += (int64_t)gridDim.x * blockDim.x)
    ((uint4*)A.table)[i] = make_uint4(0, 0, 0, 0);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *A.err = 0;
    *A.open = 0;
  }
}

// One face per thread: its three half-edges inserted or matched.  After an
// error some rows are left as they were; k_adj_finish writes them.
__global__ void __launch_bounds__(256) k_adj_match(AdjArgs A) {
  const int64_t size = int64_t(1) << A.bits, mask = size - 1;
  for (int64_t f = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; f < A.F;
       f += (int64_t)gridDim.x * blockDim.x) {
    int v[3];
    for (int k = 0; k < 3; ++k) v[k] = A.faces[3 * f + k];
    int64_t p0 = 0, f0 = 0, f1 = A.F;  // the cloud's first point and its face rows
    bool ok = v[0] >= 0 && v[1] >= 0 && v[2] >= 0;
    if (A.face_off) {
      const int64_t h = owner64(A.face_off, A.H, f);
      p0 = A.pt_off[h];
      const int64_t np = A.pt_off[h + 1] - p0;
      // (owner64 gives rows before or past all offsets to the first or last cloud)
      if (h > 0) f0 = A.face_off[h];
      if (h + 1 < A.H) f1 = A.face_off[h + 1];
      ok = ok && v[0] < np && v[1] < np && v[2] < np;
    }
    if (!ok) {
      atomicCAS(A.err, 0, HULL_ERANGE);
      continue;
    }
    for (int k = 0; k < 3; ++k) {
      const int a = v[k], b = v[k == 2 ? 0 : k + 1];
      const unsigned id = (unsigned)(3 * f + k) + 1;
      const unsigned long long lo = (unsigned long long)(p0 + (a < b ? a : b)),
                               hi = (unsigned long long)(p0 + (a < b ? b : a));
      int64_t i = (int64_t)slot_of((lo << 32) | hi, A.bits);
      for (int64_t probe = 0; probe < size; ++probe, i = (i + 1) & mask) {
        // a cached value may be out of date, but only as an empty or an
        // unmarked slot, and the swaps below see the current one
        unsigned cur =
            __hip_atomic_load(&A.table[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (cur == 0) {
          // an edge from a point to itself is its own twin
          cur = atomicCAS(&A.table[i], 0u, a == b ? id | kMatched : id);
          if (cur == 0) {
            if (a == b) A.adj[3 * f + k] = (int)f;
            break;
          }
        }
        const unsigned other = (cur & ~kMatched) - 1;
        const int64_t g = other / 3u;
        const int m = (int)(other - 3u * (unsigned)g);
        if (g < f0 || g >= f1) continue;
        const int x = A.faces[3 * g + m], y = A.faces[3 * g + (m == 2 ? 0 : m + 1)];
        if (x == b && y == a) {
          const unsigned want = cur & ~kMatched;
          if (atomicCAS(&A.table[i], want, want | kMatched) != want) {
            atomicCAS(A.err, 0, HULL_EINTERNAL);  // a third half-edge of this edge
          } else {
            A.adj[3 * f + k] = (int)g;
            A.adj[other] = (int)f;
          }
          break;
        }
        if (x == a && y == b) {  // the same directed edge twice: not a 2-manifold
          atomicCAS(A.err, 0, HULL_EINTERNAL);
          break;
        }
      }
    }
  }
}

// Half-edges left without a twin; every row after an error.
__global__ void __launch_bounds__(256) k_adj_finish(AdjArgs A) {
  if (*A.err) {
    for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < 3 * A.F;
         e += (int64_t)gridDim.x * blockDim.x)
      A.adj[e] = -1;
    return;
  }
  const int64_t quads = int64_t(1) << (A.bits - 2);
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < quads;
       i += (int64_t)gridDim.x * blockDim.x) {
    const uint4 q = ((const uint4*)A.table)[i];
    const unsigned s[4] = {q.x, q.y, q.z, q.w};
    for (int j = 0; j < 4; ++j)
      if (s[j] != 0 && !(s[j] & kMatched)) {
        A.adj[s[j] - 1] = -1;
        atomicAdd(A.open, 1);
      }
  }
}

__global__ void k_adj_info(AdjArgs A) {
  if (threadIdx.x == 0) {
    A.info[0] = *A.err;
    A.info[1] = *A.err ? 0 : *A.open;
  }
}

static int table_bits(int64_t F) {
  int bits = 4;
  while (2 * (int64_t(1) << bits) < 7 * F) ++bits;
  return bits;
}

// The workspace asked for stays what it was with a table of 16-byte slots, at
// least 6 per face (callers size buffers by it); the table takes the front of it.
static size_t adj_ws_bytes(int64_t F) {
  int bits = 4;
  while ((int64_t(1) << bits) < 6 * F) ++bits;
  return 256 + (size_t(16) << bits);
}

}  // namespace hull

extern "C" {

int32_t hull_adjacency_workspace_bytes(int64_t F, size_t* bytes) {
  if (!bytes || F < 0 || F > hull::kMaxAdjFaces) return HULL_EINVAL;
  *bytes = hull::adj_ws_bytes(F);
  return HULL_OK;
}

int32_t hull_face_adjacency(const int32_t* d_faces, int64_t F, const int64_t* d_face_off,
                            const int64_t* d_pt_off, int64_t H, int32_t* d_adj, int64_t* d_info,
                            void* d_ws, size_t ws_bytes, void* stream) {
  if (F < 0 || F > hull::kMaxAdjFaces || !d_info || !d_ws || (F > 0 && (!d_faces || !d_adj)) ||
      (d_face_off && (!d_pt_off || H < 1)) || (!d_face_off && d_pt_off))
    return HULL_EINVAL;
  if (ws_bytes < hull::adj_ws_bytes(F)) return HULL_EWORKSPACE;
  hull::clear_stale_hip_error();
  hipStream_t s = (hipStream_t)stream;
  char* ws = (char*)d_ws;
  hull::AdjArgs A{};
  A.faces = d_faces;
  A.F = F;
  A.face_off = d_face_off;
  A.pt_off = d_pt_off;
  A.H = d_face_off ? H : 1;
  A.err = (int*)ws;
  A.open = (int*)(ws + 64);
  A.table = (unsigned*)(ws + 256);
  A.bits = hull::table_bits(F);
  A.adj = d_adj;
  A.info = d_info;
  const int64_t quads = int64_t(1) << (A.bits - 2);
  const unsigned gt = (unsigned)std::min<int64_t>((quads + 255) / 256, 2048);
  const unsigned gf = (unsigned)std::max<int64_t>(1, std::min<int64_t>((F + 255) / 256, 8192));
  hipLaunchKernelGGL(hull::k_adj_clear, dim3(gt), dim3(256), 0, s, A);
  hipLaunchKernelGGL(hull::k_adj_match, dim3(gf), dim3(256), 0, s, A);
  hipLaunchKernelGGL(hull::k_adj_finish, dim3(gt), dim3(256), 0, s, A);
  hipLaunchKernelGGL(hull::k_adj_info, dim3(1), dim3(64), 0, s, A);
  HULL_LAUNCH_CHECK();
  return HULL_OK;
}

}  // extern "C"
