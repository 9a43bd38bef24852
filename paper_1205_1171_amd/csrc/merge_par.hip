// Parallel merge strategy for large blocks: the merge of two movies (Sec. 2, the
// merge step) with its time axis cut into segments (walk.hpp) and the lists of
// link-changing events in global memory.
//
// Per level, over the child events of all merges (nothing per merge is serial):
//   1. the events are enumerated and every event takes its places in the lists
//      of the points whose links it changes (one atomic per change; its value
//      is the place);
//   2. list bounds by a scan over the points, then the entries: the event's
//      position in its child movie and the link after it.  Lists of up to
//      kParScan entries stay in arrival order (a lookup reads them whole);
//      longer ones are sorted by position;
//   3. a counting walk per segment, a scan, and a writing walk that replays
//      the counted steps.  A segment's output is in order, so the level needs
//      no classification of the child events and no ranks of events in other
//      lists.
// A level is nine launches.  Claiming lists by events, filling and sorting
// 16-byte entries, a separate bridge list, survival flags and three more scans
// took 1.70-2.25 ms a level on the 2^20-point sphere,
// this 0.70-1.05 ms.
#include <algorithm>
#include <initializer_list>

#include "common.hpp"
#include "events.hpp"
#include "walk.hpp"

namespace hull {

// Longest list kept unsorted.  Sorting is one thread's chain of dependent global
// accesses: with 12, k_par_sort took 170 us a level on the 2^20-point sphere
// (mean length 3, a few lists of 13-25), 6 with 32.
constexpr int kParScan = 32;
constexpr unsigned long long kStepsLost = ~0ull;  // a segment to be walked again

template <class PT>
struct ParCtx {
  const PT* pts;
  const Event* evL;
  const Event* evR;
  const int* off;
  const int2* ent;
  const int* nx0;
  const int* pv0;
  int64_t np1;  // points + 1: prev lists start there
  int zs;
  __device__ __forceinline__ WalkEv ev(bool left, int i) const {
    const int4 x = *(const int4*)((left ? evL : evR) + i);
    WalkEv e;
    e.a = x.x;
    e.w = x.y & 0x7fffffff;
    e.b = x.z;
    e.kind = (int)((unsigned)x.y >> 31);
    e.t = (double)__int_as_float(x.w);
    return e;
  }
  // the link after the last event of the list [lo, hi) before position
  // `cursor`, `none` if there is none
  __device__ __forceinline__ int last_before(int lo, int hi, int cursor, int none) const {
    if (hi - lo > kParScan) {
      const int first = lo;
      while (lo < hi) {
        const int mid = (lo + hi) >> 1;
        if (ent[mid].x < cursor) lo = mid + 1;
        else hi = mid;
      }
      return lo > first ? ent[lo - 1].y : none;
    }
    int best = -1, l = none;
    for (; lo < hi; lo += 4) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int2 c = ent[lo + k < hi ? lo + k : lo];
        const bool later = c.x < cursor && c.x > best;
        best = later ? c.x : best;
        l = later ? c.y : l;
      }
    }
    return l;
  }
  __device__ __forceinline__ int link(int p, bool nx, bool, int cursor) const {
    const int64_t key = nx ? p : np1 + p;
    return last_before(off[key], off[key + 1], cursor, nx ? nx0[p] : pv0[p]);
  }
  __device__ __forceinline__ void links(int p, bool, int cursor, int& nx, int& pv) const {
    const int n0 = off[p], n1 = off[p + 1], p0 = off[np1 + p], p1 = off[np1 + p + 1];
    const int ln = nx0[p], lp = pv0[p];
    nx = last_before(n0, n1, cursor, ln);
    pv = last_before(p0, p1, cursor, lp);
  }
};

template <class PT>
__device__ __forceinline__ ParCtx<PT> ctx_of(const ParLevel& P, int r, int64_t s, int64_t m) {
  const RunPtrs& R = P.run[r];
  ParCtx<PT> X;
  X.pts = (const PT*)R.pts;
  X.evL = R.left_ev(s);
  X.evR = R.ev[(P.S.k - 1) & 1] + 2 * m;  // k_par_prep settled it there
  X.off = P.par[r].off;
  X.ent = P.par[r].ent;
  X.nx0 = R.nx0;
  X.pv0 = R.pv0;
  X.np1 = P.S.off[P.S.H] + 1;
  X.zs = R.zs;
  return X;
}

// Sorts a list by position (Shell's method; only lists above kParScan).
__device__ void sort_entries(int2* a, int k) {
  int gap = 1;
  while (gap < k / 3) gap = 3 * gap + 1;
  for (; gap > 0; gap /= 3)
    for (int i = gap; i < k; ++i) {
      const int2 x = a[i];
      int j = i;
      while (j >= gap && a[j - gap].x > x.x) {
        a[j] = a[j - gap];
        j -= gap;
      }
      a[j] = x;
    }
}

#define GRID_STRIDE(i, n) \
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < (n); \
       i += (int64_t)gridDim.x * blockDim.x)

// Per merge: child event count and walk segments; the list bounds cleared;
// short right blocks moved out of the buffer the level writes; and the splices of the level before (its walks, which read the -inf links, have
// ended; nothing here reads them).
__global__ void __launch_bounds__(256) k_par_prep(ParLevel P) {
  const RunPtrs& R = P.run[blockIdx.y];
  const ParRun& Q = P.par[blockIdx.y];
  if (!R.pts) return;
  const int64_t merges = selected(P.S, P.sel) ? P.S.merges() : 0, half = int64_t(1) << (P.S.k - 1);
  const int64_t keys = merges ? 2 * (P.S.off[P.S.H] + 1) : 0;
  const bool err = P.h->err != 0;
  GRID_STRIDE(g, (int64_t)(err ? 0 : Q.ctr[kCtrSplice + ((P.S.k - 1) & 1)])) {
    const int2 b = Q.uv0[g];
    R.nx0[b.x] = b.y;
    R.pv0[b.y] = b.x;
  }
  GRID_STRIDE(g, merges + 1) {
    if (g == 0) {
      Q.ctr[kCtrMerges] = (int)merges;
      Q.ctr[kCtrKeys] = (int)keys;
      Q.ctr[kCtrSplice + (P.S.k & 1)] = (int)merges;
    }
    if (g < merges && !err) {
      const int2 se = P.S.merge(g);
      const int64_t m = se.x + half;
      const int nL = R.left_len(se.x), nR = R.right_len(m, se.y);
      Q.ecnt[g] = nL + nR;
      Q.segS[g] = segments_for(nL + nR, P.seg_events);
    } else {
      Q.ecnt[g] = 0;
      Q.segS[g] = 0;
    }
  }
  GRID_STRIDE(q, keys) Q.off[q] = 0;
  if (err) return;
  for (int64_t g = blockIdx.x; g < merges; g += gridDim.x) {  // one block per merge
    const int2 se = P.S.merge(g);
    const int64_t m = se.x + half, e = se.y;
    if (R.right_waits_in_output(m, e))
      (void)R.settle_right(m, e, R.right_len(m, e), threadIdx.x, blockDim.x);
  }
}

// The child events take their places in the lists; then, past the events, the
// segment table: per walk segment its merge and the left events before it.
template <class PT>
__global__ void __launch_bounds__(256) k_par_enum(ParLevel P) {
  const RunPtrs& R = P.run[blockIdx.y];
  const ParRun& Q = P.par[blockIdx.y];
  if (!R.pts) return;
  const int merges = Q.ctr[kCtrMerges], E = Q.ctr[kCtrEvents], Sg = Q.ctr[kCtrSegments];
  if (!merges) return;
  const int64_t half = int64_t(1) << (P.S.k - 1), np1 = P.S.off[P.S.H] + 1;
  GRID_STRIDE(c, (int64_t)E + Sg) {
    const bool seg = c >= E;
    const int64_t t = seg ? c - E : c;
    const int g = find_owner(seg ? Q.segBase : Q.eoff, merges, t);
    const int2 se = P.S.merge(g);
    const int64_t s = se.x, m = s + half, e = se.y;
    const ParCtx<PT> X = ctx_of<PT>(P, blockIdx.y, s, m);
    const int nL = R.left_len(s);
    if (seg) {
      const int nR = R.right_len(m, e);
      Q.segMerge[t] = g;
      Q.segJ[t] = segment_split<PT>(X, nL, nR, (int)(t - Q.segBase[g]), Q.segS[g]);
      continue;
    }
    const int i = (int)(t - Q.eoff[g]);
    const WalkEv x = X.ev(i < nL, i < nL ? i : i - nL);
    Q.cmerge[c] = g;
    int4 at = make_int4(0, 0, 0, 0);
    at.x = atomicAdd(&Q.off[x.a], 1);
    at.y = atomicAdd(&Q.off[np1 + x.b], 1);
    if (x.kind) {
      at.z = atomicAdd(&Q.off[x.w], 1);
      at.w = atomicAdd(&Q.off[np1 + x.w], 1);
    }
    Q.pos[c] = at;
  }
}

// An event sets next(a) and prev(b), an insertion both links of w too.
template <class PT>
__global__ void __launch_bounds__(256) k_par_fill(ParLevel P) {
  const RunPtrs& R = P.run[blockIdx.y];
  const ParRun& Q = P.par[blockIdx.y];
  if (!R.pts) return;
  const int E = Q.ctr[kCtrEvents], keys = Q.ctr[kCtrKeys];
  if (E <= 0 || keys <= 0) return;
  const int64_t half = int64_t(1) << (P.S.k - 1), np1 = P.S.off[P.S.H] + 1;
  // capacity: 6 entries per point (the last bound is the entries of all but
  // the last key, whose list is empty)
  if (Q.off[keys - 1] > 6 * P.n) {
    if (blockIdx.x == 0 && threadIdx.x == 0) atomicCAS(&P.h->err, 0, HULL_EINTERNAL);
    return;
  }
  GRID_STRIDE(c, (int64_t)E) {
    const int g = Q.cmerge[c];
    const int2 se = P.S.merge(g);
    const int64_t s = se.x, m = s + half, e = se.y;
    const ParCtx<PT> X = ctx_of<PT>(P, blockIdx.y, s, m);
    const int nL = R.left_len(s), i = (int)(c - Q.eoff[g]);
    const int j = i < nL ? i : i - nL;
    const WalkEv x = X.ev(i < nL, j);
    const int4 at = Q.pos[c];
    Q.ent[Q.off[x.a] + at.x] = make_int2(j, x.kind ? x.w : x.b);
    Q.ent[Q.off[np1 + x.b] + at.y] = make_int2(j, x.kind ? x.w : x.a);
    if (x.kind) {
      Q.ent[Q.off[x.w] + at.z] = make_int2(j, x.b);
      Q.ent[Q.off[np1 + x.w] + at.w] = make_int2(j, x.a);
    }
  }
}

__global__ void __launch_bounds__(256) k_par_sort(ParLevel P) {
  const ParRun& Q = P.par[blockIdx.y];
  if (!P.run[blockIdx.y].pts || P.h->err) return;
  GRID_STRIDE(q, (int64_t)Q.ctr[kCtrKeys] - 1) {
    const int first = Q.off[q], k = Q.off[q + 1] - first;
    if (k > kParScan) sort_entries(Q.ent + first, k);
  }
}

// A counting walk: its steps, and its first kSegKeep bridge events put aside.
struct ParCount {
  WalkNote note;
  Event* keep;
  __device__ __forceinline__ void child(bool left, bool kept, int, int, int, int, double) {
    note.child(left, kept);
  }
  __device__ __forceinline__ void bridge(int a, int w, int b, int kind, double t) {
    if (note.nbridge < kSegKeep) keep[note.nbridge] = make_event(a, w, b, kind, t);
    ++note.nbridge;
    note.step(kStepBridge, true);
  }
};

struct ParWrite {
  Event* out;
  __device__ __forceinline__ void child(bool, bool kept, int a, int w, int b, int kind, double t) {
    if (kept) *out++ = make_event(a, w, b, kind, t);
  }
  __device__ __forceinline__ void bridge(int a, int w, int b, int kind, double t) {
    *out++ = make_event(a, w, b, kind, t);
  }
};

// One segment's place: its merge, its child events and the last event before
// it.
template <class PT>
struct ParSeg {
  int64_t s, m, e;
  ParCtx<PT> X;
  int i, S, jL, jR, kL, kR, limit;
  Cand T;
  __device__ __forceinline__ ParSeg(const ParLevel& P, int r, int64_t t, int g) {
    const RunPtrs& R = P.run[r];
    const ParRun& Q = P.par[r];
    const int2 se = P.S.merge(g);
    s = se.x;
    m = s + (int64_t(1) << (P.S.k - 1));
    e = se.y;
    X = ctx_of<PT>(P, r, s, m);
    i = (int)(t - Q.segBase[g]);
    S = Q.segS[g];
    const int nL = R.left_len(s), nR = R.right_len(m, e);
    const int64_t N = (int64_t)nL + nR;
    jL = Q.segJ[t];
    jR = (int)(i * N / S) - jL;
    kL = i + 1 < S ? Q.segJ[t + 1] : nL;
    kR = (int)((i + 1) * N / S) - kL;
    const int64_t lim = 4 * (e - s) + N + 16;
    limit = (int)(lim < 0x7fffffff ? lim : 0x7ffffffe);
    T.t = Tri{-1, -1, -1};
    T.st = 0.0;
    T.kind = 0;
    if (i > 0) {
      if (jL == 0) T = walk_cand(X.ev(false, jR - 1));
      else if (jR == 0) T = walk_cand(X.ev(true, jL - 1));
      else {
        const Cand x = walk_cand(X.ev(true, jL - 1)), y = walk_cand(X.ev(false, jR - 1));
        T = ev_cmp(X.pts, x, y, X.zs) > 0 ? x : y;
      }
    }
  }
};

template <class PT>
__global__ void __launch_bounds__(64) k_par_walk(ParLevel P) {
  const ParRun& Q = P.par[blockIdx.y];
  if (!P.run[blockIdx.y].pts) return;
  const int total = Q.ctr[kCtrSegments];
  if (!Q.ctr[kCtrMerges]) return;
  const bool err = P.h->err != 0;
  GRID_STRIDE(t, (int64_t)total + 1) {
    if (t == total || err) {  // the scan reads one entry past the last segment
      Q.segCnt[t] = 0;
      continue;
    }
    const int g = Q.segMerge[t];
    const ParSeg<PT> Z(P, blockIdx.y, t, g);
    int u = 0, v = 0;
    ParCount cnt;
    cnt.keep = Q.segKeep + t * kSegKeep;
    bool ok = bridge_at<PT>(Z.X, (int)Z.m, Z.jL, Z.jR, Z.i > 0, Z.T, Z.limit, u, v);
    if (ok)
      ok = walk<PT>(Z.X, u, v, Z.jL, Z.kL, Z.jR, Z.kR, Z.i + 1 == Z.S, Z.i > 0, Z.T, Z.limit, cnt);
    if (!ok) {
      atomicCAS(&P.h->err, 0, HULL_EINTERNAL);
      Q.segCnt[t] = 0;
      continue;
    }
    if (Z.i == 0) Q.uv0[g] = make_int2(u, v);
    Q.segUV[t] = make_int2(u, v);
    Q.segCnt[t] = cnt.note.nout;
    Q.segSteps[t] = cnt.note.nsteps <= kWalkSteps && cnt.note.nbridge <= kSegKeep ? cnt.note.steps
                                                                                  : kStepsLost;
  }
}

// Every segment's events to their place in the merged movie.
template <class PT>
__global__ void __launch_bounds__(64) k_par_write(ParLevel P) {
  const RunPtrs& R = P.run[blockIdx.y];
  const ParRun& Q = P.par[blockIdx.y];
  if (!R.pts || !Q.ctr[kCtrMerges]) return;
  const bool err = P.h->err != 0;
  GRID_STRIDE(t, (int64_t)Q.ctr[kCtrSegments]) {
    const int g = Q.segMerge[t];
    const int first = Q.segBase[g];
    if (err) {  // every merge writes its length, also after an error
      if (t == first) R.out_len(P.S.merge(g).x) = 0;
      continue;
    }
    const ParSeg<PT> Z(P, blockIdx.y, t, g);
    const int len = Q.segOff[first + Z.S] - Q.segOff[first];
    const int64_t cap = 2 * (Z.e - Z.s);
    if (t == first) R.out_len(Z.s) = len <= cap ? len : 0;
    if (len > cap) {
      atomicCAS(&P.h->err, 0, HULL_EINTERNAL);
      continue;
    }
    ParWrite wr{R.out_ev(Z.s) + (Q.segOff[t] - Q.segOff[first])};
    unsigned long long steps = Q.segSteps[t];
    if (steps == kStepsLost) {
      const int2 uv = Q.segUV[t];
      (void)walk<PT>(Z.X, uv.x, uv.y, Z.jL, Z.kL, Z.jR, Z.kR, Z.i + 1 == Z.S, Z.i > 0, Z.T, Z.limit, wr);
      continue;
    }
    int jL = Z.jL, jR = Z.jR;
    const Event* keep = Q.segKeep + t * kSegKeep;
    for (; steps; steps >>= 3) {
      const unsigned code = (unsigned)steps & 7u;
      if (code == kStepBridge) {
        *wr.out++ = *keep++;
      } else {
        const bool left = code == kStepL || code == kStepHideL;
        const Event* x = left ? Z.X.evL + jL++ : Z.X.evR + jR++;
        if (code == kStepL || code == kStepR) *wr.out++ = *x;
      }
    }
  }
}

// Scans of the same arrays of both runs in one launch.  kinds: 0 child events
// and 1 walk segments per merge (their totals are the level's), 2 the lists'
// lengths by key, 3 events put out per segment.
static ScanJobs jobs_of(const ParLevel& P, std::initializer_list<int> kinds) {
  ScanJobs J{};
  for (int r = 0; r < 2; ++r) {
    if (!P.run[r].pts) continue;
    const ParRun& Q = P.par[r];
    for (int f : kinds) {
      ScanJob& j = J.j[J.count++];
      switch (f) {
        case 0: j = ScanJob{Q.ecnt, Q.eoff, Q.ctr + kCtrMerges, Q.ctr + kCtrEvents}; break;
        case 1: j = ScanJob{Q.segS, Q.segBase, Q.ctr + kCtrMerges, Q.ctr + kCtrSegments}; break;
        case 2: j = ScanJob{Q.off, Q.off, Q.ctr + kCtrKeys, nullptr}; break;
        default: j = ScanJob{Q.segCnt, Q.segOff, Q.ctr + kCtrSegments, nullptr}; break;
      }
    }
  }
  return J;
}

// The level's three scans, on job slots of their own; the epoch (level and
// scan) tells their status words from those of earlier levels of the call.
static int32_t chained(const ParLevel& P, const ScanJobs& J, int slot, int site, int add, int64_t cap,
                       hipStream_t s) {
  return exclusive_scan_chained(J, add, cap, P.chain_words + slot * P.chain_stride, P.chain_stride,
                                (unsigned)(P.S.k * 8 + site), P.h, s);
}

template <class PT>
int32_t parallel_level(const ParLevel& P, hipStream_t s) {
  const dim3 g2(kStrideBlocks, 2), b256(256);
  hipLaunchKernelGGL(k_par_prep, g2, b256, 0, s, P);
  int32_t rc = chained(P, jobs_of(P, {0, 1}), 0, 1, 1, P.mcap + 1, s);
  if (rc) return rc;
  hipLaunchKernelGGL(k_par_enum<PT>, g2, b256, 0, s, P);
  rc = chained(P, jobs_of(P, {2}), 4, 2, 0, 2 * P.n + 2, s);
  if (rc) return rc;
  hipLaunchKernelGGL(k_par_fill<PT>, g2, b256, 0, s, P);
  hipLaunchKernelGGL(k_par_sort, g2, b256, 0, s, P);
  const dim3 gw(16384, 2), b64(64);
  hipLaunchKernelGGL(k_par_walk<PT>, gw, b64, 0, s, P);
  rc = chained(P, jobs_of(P, {3}), 6, 3, 1, P.seg_cap + 1, s);
  if (rc) return rc;
  hipLaunchKernelGGL(k_par_write<PT>, gw, b64, 0, s, P);
  HULL_LAUNCH_CHECK();
  return HULL_OK;
}

template int32_t parallel_level<int4>(const ParLevel&, hipStream_t);
template int32_t parallel_level<WPt>(const ParLevel&, hipStream_t);

}  // namespace hull
