// One merge per group of lanes with its time axis cut into segments (walk.hpp),
// everything the walks touch in LDS: the points, the -inf links, both child
// movies (8 bytes an event: three child-local ranks of 10 bits, the kind and
// the time) and the lists of link-changing events of every point.
//
// The lane-serial and lane-group merges run a chain of one step per event
// (0.4-0.8 us each, so a merge of 1,024 points takes about 0.6-1 ms however
// idle the chip is).  Here the chain is a tangent search and the steps of one
// segment of a few events, whatever the block's size.
#pragma once
#include "common.hpp"
#include "events.hpp"
#include "walk.hpp"

namespace hull {

constexpr int kTileRankBits = 10;
constexpr int kListScan = 12;    // longest list kept unsorted
constexpr int kListSerial = 32;  // longest list sorted by one lane
constexpr int kTileKeep = 8;   // bridge events a lane puts aside per segment
constexpr int kTileMaxWidth = 2 << kTileRankBits;  // two children of 1,024 points

// LDS of one merge of up to W points (W even) by a group of GS lanes.
template <class PT>
struct TileLds {
  PT* pts;
  uint2* ev;             // [2W] child events, left movie first
  int* off;              // [2W + 1] list bounds: next links at p, prev links at W + p
  LinkPair<short>* lk;   // [W] -inf links
  unsigned short* ent;   // [6W] list entries: positions in ev
  uint2* keep;           // [kTileKeep * GS] bridge events put aside
  unsigned short* cut;   // [2 W + 2] segment bounds in the left movie (W + 2 at most), then
                         // from W + 2 on the number of long lists (an int) and their keys
  __host__ __device__ static constexpr size_t bytes(int W, int GS) {
    const size_t b = (size_t)W * (sizeof(PT) + 16 + 8 + 4 + 12) + 16 +
                     (size_t)kTileKeep * GS * sizeof(uint2) + (size_t)(2 * W + 2) * 2;
    return (b + 15) & ~(size_t)15;
  }
  __device__ __forceinline__ TileLds(unsigned char* lds, int W, int GS) {
    pts = (PT*)lds;
    ev = (uint2*)(pts + W);
    keep = ev + 2 * W;
    off = (int*)(keep + kTileKeep * GS);
    lk = (LinkPair<short>*)(off + 2 * W + 4);
    ent = (unsigned short*)(lk + W);
    cut = ent + 6 * W;
  }
};

template <class PT>
struct TileCtx {
  const PT* pts;
  const uint2* evs;
  const int* off;
  const LinkPair<short>* lk;
  const unsigned short* ent;
  int nL, half, W, zs;
  __device__ __forceinline__ WalkEv ev(bool left, int i) const { return at(left ? i : nL + i, left); }
  __device__ __forceinline__ WalkEv at(int c, bool left) const {
    const uint2 x = evs[c];
    const int o = left ? 0 : half;
    constexpr unsigned M = (1u << kTileRankBits) - 1;
    WalkEv e;
    e.a = (int)(x.x & M) + o;
    e.w = (int)((x.x >> kTileRankBits) & M) + o;
    e.b = (int)((x.x >> (2 * kTileRankBits)) & M) + o;
    e.kind = (int)(x.x >> 31);
    e.t = (double)__uint_as_float(x.y);
    return e;
  }
  // position in ev of the last event among the list [lo, hi) before position
  // `cur`, -1 if none: a list of up to kListScan entries is not sorted and read
  // whole, four independent reads at a time; a longer one by binary search
  __device__ __forceinline__ int last_before(int lo, int hi, int cur) const {
    int best = -1;
    if (hi - lo > kListScan) {
      const int first = lo;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if ((int)ent[mid] < cur) lo = mid + 1;
        else hi = mid;
      }
      return lo > first ? (int)ent[lo - 1] : -1;
    }
    for (; lo < hi; lo += 4) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int c = (int)ent[lo + k < hi ? lo + k : lo];
        best = c < cur && c > best ? c : best;
      }
    }
    return best;
  }
  __device__ __forceinline__ int resolve(int c, int p, bool nx, bool left, LinkPair<short> l) const {
    const WalkEv e = at(c < 0 ? 0 : c, left);
    const int n = next_after(e.a, e.w, e.b, e.kind, p), q = prev_after(e.a, e.w, e.b, e.kind, p);
    return c < 0 ? (nx ? l.nx : l.pv) : (nx ? n : q);
  }
  __device__ __forceinline__ int link(int p, bool nx, bool left, int cursor) const {
    const int key = nx ? p : W + p;
    const LinkPair<short> l = lk[p];
    return resolve(last_before(off[key], off[key + 1], left ? cursor : nL + cursor), p, nx, left, l);
  }
  __device__ __forceinline__ void links(int p, bool left, int cursor, int& nx, int& pv) const {
    const int n0 = off[p], n1 = off[p + 1], p0 = off[W + p], p1 = off[W + p + 1];
    const int cur = left ? cursor : nL + cursor;
    const LinkPair<short> l = lk[p];
    const int cn = last_before(n0, n1, cur), cp = last_before(p0, p1, cur);
    nx = resolve(cn, p, true, left, l);
    pv = resolve(cp, p, false, left, l);
  }
};

// The outcomes of a counting walk: its steps, and its first kTileKeep bridge
// events put aside in LDS (an event's three ranks in 32 bits: the outer two
// child-local, the middle one with its side).
struct TileCount {
  WalkNote note;
  uint2* keep;  // the lane's column: entry q at keep[q * stride]
  int stride, half;
  __device__ __forceinline__ void child(bool left, bool kept, int, int, int, int, double) {
    note.child(left, kept);
  }
  __device__ __forceinline__ void bridge(int a, int w, int b, int kind, double t) {
    constexpr int B = kTileRankBits;
    const unsigned side = w >= half;
    if (note.nbridge < kTileKeep)
      keep[note.nbridge * stride] =
          make_uint2((unsigned)a | ((unsigned)(b - half) << B) | ((unsigned)(w - (side ? half : 0)) << (2 * B)) |
                         (side << (3 * B)) | ((unsigned)kind << 31),
                     __float_as_uint((float)t));
    ++note.nbridge;
    note.step(kStepBridge, true);
  }
  __device__ __forceinline__ bool complete() const {
    return note.nsteps <= kWalkSteps && note.nbridge <= kTileKeep;
  }
};

// Writes a walk's output events, in global ranks.
struct TileWrite {
  Event* out;
  int base;
  __device__ __forceinline__ void put(int a, int w, int b, int kind, double t) {
    *out++ = make_event(a + base, w + base, b + base, kind, t);
  }
  __device__ __forceinline__ void child(bool, bool kept, int a, int w, int b, int kind, double t) {
    if (kept) put(a, w, b, kind, t);
  }
  __device__ __forceinline__ void bridge(int a, int w, int b, int kind, double t) {
    put(a, w, b, kind, t);
  }
};

// Sorts a short list of positions (Shell's method).
__device__ __forceinline__ void sort_positions(unsigned short* a, int k) {
  int gap = 1;
  while (gap < k / 3) gap = 3 * gap + 1;
  for (; gap > 0; gap /= 3)
    for (int i = gap; i < k; ++i) {
      const unsigned short x = a[i];
      int j = i;
      while (j >= gap && a[j - gap] > x) {
        a[j] = a[j - gap];
        j -= gap;
      }
      a[j] = x;
    }
}

// Sorts a list of up to 4 x the group's size by the whole group (a vertex of high
// degree has one as long as the movie; the positions differ, so an entry's place is
// the number of smaller ones).  A cone over 1,024 points 0.51 ms, a moment curve of as
// many 2.5; by one lane, with Shell's method, 0.83 and 3.8.
template <class GRP>
__device__ __forceinline__ void sort_positions_by(const GRP& g, unsigned short* a, int k) {
  unsigned short x[4];
  int r[4] = {0, 0, 0, 0};
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int i = g.rank() + e * g.size();
    x[e] = a[i < k ? i : 0];
  }
  for (int j = 0; j < k; ++j) {
    const unsigned short y = a[j];
#pragma unroll
    for (int e = 0; e < 4; ++e) r[e] += y < x[e];
  }
  g.sync();
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (g.rank() + e * g.size() < k) a[r[e]] = x[e];
}

// The merge of [s, m) and [m, e), e - s <= W, by the group g (rank, size,
// sync, exclusive scan); the same arguments on every lane of the group.
template <class PT, class GRP>
__device__ __forceinline__ void tile_merge(const GRP& g, unsigned char* lds, int W,
                                           const RunPtrs& R, Header* h, int64_t s, int64_t m,
                                           int64_t e, int seg) {
  const int nL = R.left_len(s), nR = R.right_len(m, e);
  const Event* Lev = R.left_ev(s);
  const Event* Rev = R.right_ev(m, e);
  const int w = (int)(e - s), half = (int)(m - s);
  if (nL < 0 || nR < 0 || nL > 2 * half || nR > 2 * (w - half) || w > W || half > (1 << kTileRankBits) ||
      w - half > (1 << kTileRankBits)) {
    if (g.rank() == 0) {
      atomicCAS(&h->err, 0, HULL_EINTERNAL);
      R.out_len(s) = 0;
    }
    return;
  }
  const TileLds<PT> L(lds, W, g.size());
  const int N = nL + nR, S = segments_for(N, seg);
  const PT* pts = (const PT*)R.pts + s;
  for (int q = g.rank(); q < 2 * W + 1; q += g.size()) L.off[q] = 0;
  for (int q = g.rank(); q < w; q += g.size()) {
    L.pts[q] = pts[q];
    const int pv = R.pv0[s + q], nx = R.nx0[s + q];
    LinkPair<short> k;
    k.pv = (short)(pv == kNil ? -1 : pv - (int)s);
    k.nx = (short)(nx == kNil ? -1 : nx - (int)s);
    L.lk[q] = k;
  }
  g.sync();
  // events, and the lengths of the points' lists: an event sets next(a) and
  // prev(b), an insertion both links of w too
  for (int c = g.rank(); c < N; c += g.size()) {
    const bool left = c < nL;
    const int64_t o = left ? s : m;
    const int4 x = *(const int4*)(left ? Lev + c : Rev + (c - nL));
    const int a = (int)(x.x - o), ww = (int)((x.y & 0x7fffffff) - o), b = (int)(x.z - o);
    const unsigned kind = (unsigned)x.y >> 31;
    L.ev[c] = make_uint2((unsigned)a | ((unsigned)ww << kTileRankBits) |
                             ((unsigned)b << (2 * kTileRankBits)) | (kind << 31),
                         (unsigned)x.w);
    const int d = left ? 0 : half;
    atomicAdd(&L.off[a + d], 1);
    atomicAdd(&L.off[W + b + d], 1);
    if (kind) {
      atomicAdd(&L.off[ww + d], 1);
      atomicAdd(&L.off[W + ww + d], 1);
    }
  }
  g.sync();
  // list ends, then (as the fill counts them down) starts
  int total = 0;
  for (int q0 = 0; q0 < 2 * W; q0 += 4 * g.size()) {
    int v[4], sum = 0;
    const int q = q0 + 4 * g.rank();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      if (q + j < 2 * W) sum += L.off[q + j];
      v[j] = sum;
    }
    int all;
    const int before = total + g.scan(sum, all);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (q + j < 2 * W) L.off[q + j] = before + v[j];
    total += all;
  }
  if (g.rank() == 0) L.off[2 * W] = total;
  g.sync();
  if (total > 6 * W) {
    if (g.rank() == 0) {
      atomicCAS(&h->err, 0, HULL_EINTERNAL);
      R.out_len(s) = 0;
    }
    return;
  }
  TileCtx<PT> X;
  X.pts = L.pts;
  X.evs = L.ev;
  X.off = L.off;
  X.lk = L.lk;
  X.ent = L.ent;
  X.nL = nL;
  X.half = half;
  X.W = W;
  X.zs = R.zs;
  for (int c = g.rank(); c < N; c += g.size()) {
    const WalkEv x = X.at(c, c < nL);
    L.ent[atomicSub(&L.off[x.a], 1) - 1] = (unsigned short)c;
    L.ent[atomicSub(&L.off[W + x.b], 1) - 1] = (unsigned short)c;
    if (x.kind) {
      L.ent[atomicSub(&L.off[x.w], 1) - 1] = (unsigned short)c;
      L.ent[atomicSub(&L.off[W + x.w], 1) - 1] = (unsigned short)c;
    }
  }
  for (int i = g.rank(); i < S; i += g.size())
    L.cut[i] = (unsigned short)segment_split<PT>(X, nL, nR, i, S);
  int* longs = (int*)(L.cut + W + 2);
  unsigned short* long_key = L.cut + W + 4;  // (at most 6 W / 32 of them)
  if (g.rank() == 0) {
    L.cut[S] = (unsigned short)nL;
    *longs = 0;
  }
  g.sync();
  for (int q = g.rank(); q < 2 * W; q += g.size()) {
    const int first = L.off[q], k = L.off[q + 1] - first;
    if (k > kListSerial) long_key[atomicAdd(longs, 1)] = (unsigned short)q;
    else if (k > kListScan) sort_positions(L.ent + first, k);
  }
  g.sync();
  if (*longs) {
    for (int i = 0; i < *longs; ++i) {
      const int q = long_key[i];
      sort_positions_by(g, L.ent + L.off[q], L.off[q + 1] - L.off[q]);
    }
    g.sync();
  }
  const int64_t cap = 2 * (e - s);
  const int limit = 4 * w + N + 16;
  int done = 0, u00 = 0, v00 = 0;
  bool bad = false;
  for (int i0 = 0; i0 < S; i0 += g.size()) {
    const int i = i0 + g.rank();
    TileCount cnt;
    cnt.keep = L.keep + g.rank();
    cnt.stride = g.size();
    cnt.half = half;
    int jL = 0, jR = 0, kL = 0, kR = 0, u = 0, v = 0;
    Cand T;
    T.t = Tri{-1, -1, -1};
    T.st = 0.0;
    T.kind = 0;
    if (i < S) {
      jL = L.cut[i];
      jR = (int)((int64_t)i * N / S) - jL;
      kL = L.cut[i + 1];
      kR = (int)((int64_t)(i + 1) * N / S) - kL;
      if (i > 0) {  // the last event before the segment: the later of its two movies' last
        if (jL == 0) T = walk_cand(X.ev(false, jR - 1));
        else if (jR == 0) T = walk_cand(X.ev(true, jL - 1));
        else {
          const Cand x = walk_cand(X.ev(true, jL - 1)), y = walk_cand(X.ev(false, jR - 1));
          T = ev_cmp(X.pts, x, y, X.zs) > 0 ? x : y;
        }
      }
      bad |= !bridge_at<PT>(X, half, jL, jR, i > 0, T, limit, u, v);
      if (i == 0) {
        u00 = u;
        v00 = v;
      }
      if (!bad) bad |= !walk<PT>(X, u, v, jL, kL, jR, kR, i + 1 == S, i > 0, T, limit, cnt);
    }
    int all;
    const int pos = done + g.scan(bad ? 0 : cnt.note.nout, all);
    if (done + all > cap) {  // uniform in the group
      bad = true;
      break;
    }
    if (i < S && !bad && cnt.note.nout > 0) {
      Event* out = R.out_ev(s) + pos;
      TileWrite wr{out, (int)s};
      if (cnt.complete()) {
        int nb = 0;
        for (int q = 0; q < cnt.note.nsteps; ++q) {
          const unsigned code = (unsigned)(cnt.note.steps >> (3 * q)) & 7u;
          constexpr unsigned M = (1u << kTileRankBits) - 1;
          if (code == kStepBridge) {
            const uint2 x = L.keep[nb++ * g.size() + g.rank()];
            const unsigned side = (x.x >> (3 * kTileRankBits)) & 1u;
            wr.put((int)(x.x & M), (int)((x.x >> (2 * kTileRankBits)) & M) + (side ? half : 0),
                   (int)((x.x >> kTileRankBits) & M) + half, (int)(x.x >> 31), (double)__uint_as_float(x.y));
          } else {
            const bool left = code == kStepL || code == kStepHideL;
            const int c = left ? jL++ : jR++;
            if (code == kStepL || code == kStepR) {
              const WalkEv x = X.ev(left, c);
              wr.put(x.a, x.w, x.b, x.kind, x.t);
            }
          }
        }
      } else {
        (void)walk<PT>(X, u, v, jL, kL, jR, kR, i + 1 == S, i > 0, T, limit, wr);
      }
    }
    done += all;
  }
  if (bad) atomicCAS(&h->err, 0, HULL_EINTERNAL);
  if (g.rank() == 0) {
    R.out_len(s) = bad ? 0 : done;
    if (!bad) {
      // splice the -inf chains
      R.nx0[s + u00] = (int)s + v00;
      R.pv0[s + v00] = (int)s + u00;
    }
  }
}

// GL lanes of a wavefront (GL = 16, 32 or 64).
template <int GL>
struct LaneGroup {
  __device__ __forceinline__ int rank() const { return threadIdx.x & (GL - 1); }
  __device__ __forceinline__ int size() const { return GL; }
  __device__ __forceinline__ void sync() const {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
  __device__ __forceinline__ int scan(int x, int& total) const {
    int incl = x;
    for (int o = 1; o < GL; o <<= 1) {
      const int y = __shfl_up(incl, o, GL);
      if (rank() >= o) incl += y;
    }
    total = __shfl(incl, GL - 1, GL);
    return incl - x;
  }
};

// A workgroup of T threads (wsum: T / 64 words of LDS).
template <int T>
struct BlockGroup {
  int* wsum;
  __device__ __forceinline__ int rank() const { return threadIdx.x; }
  __device__ __forceinline__ int size() const { return T; }
  __device__ __forceinline__ void sync() const { __syncthreads(); }
  __device__ __forceinline__ int scan(int x, int& total) const {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int incl = x;
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(incl, o);
      if (lane >= o) incl += y;
    }
    __syncthreads();  // wsum's earlier readers
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    int before = 0;
    total = 0;
    for (int q = 0; q < T / 64; ++q) {
      const int t = wsum[q];
      if (q < wave) before += t;
      total += t;
    }
    return before + incl - x;
  }
};

// GS lanes per merge: GS <= 64 lanes of a wavefront, 64 / GS merges per
// workgroup of one wavefront; more: one merge per workgroup of GS threads.
// Dynamic LDS: the block's merges x TileLds::bytes(A.width, GS).
template <class PT, int GS>
__global__ void __launch_bounds__(GS < 64 ? 64 : GS) k_merge_tile(LevelArgs A, int seg) {
  extern __shared__ __align__(16) unsigned char dyn_lds[];
  __shared__ int wsum[GS > 64 ? GS / 64 : 1];
  __shared__ int stop;
  constexpr int per = GS < 64 ? 64 / GS : 1;
  const RunPtrs& R = A.run[blockIdx.y];
  if (!R.pts || !selected(A.S, A.sel)) return;
  const int grp = GS < 64 ? (int)threadIdx.x / GS : 0;
  const int W = (int)A.width;
  const int64_t M = A.S.merges();
  unsigned char* lds = dyn_lds + grp * TileLds<PT>::bytes(W, GS);
  // t is the same on every lane of the group
  for (int64_t t = blockIdx.x * (int64_t)per + grp; t < M; t += (int64_t)gridDim.x * per) {
    const int2 se = A.S.merge(t);
    const int64_t s = se.x, m = s + A.half, e = se.y;
    if constexpr (GS <= 64) {
      const LaneGroup<GS> g;
      g.sync();  // the merge before still reads the group's LDS
      if (A.h->err) {
        if (g.rank() == 0) R.out_len(s) = 0;
        continue;
      }
      tile_merge<PT>(g, lds, W, R, A.h, s, m, e, seg);
    } else {
      const BlockGroup<GS> g{wsum};
      g.sync();
      if (g.rank() == 0) stop = A.h->err;  // one reading for the whole group
      g.sync();
      if (stop) {
        if (g.rank() == 0) R.out_len(s) = 0;
        continue;
      }
      tile_merge<PT>(g, lds, W, R, A.h, s, m, e, seg);
    }
  }
}

}  // namespace hull
