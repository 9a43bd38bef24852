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
//      longer ones are sorted by position, the longest by a whole workgroup;
//   3. a counting walk per segment, a scan, and a writing walk that replays
//      the counted steps.  A segment's output is in order, so the level needs
//      no classification of the child events and no ranks of events in other
//      lists.
// Where many points take part, steps 1 and 2 run per range of points in LDS instead
// (k_list_count, k_list_fill; the largest blocks: k_bin, k_bin_lists).
// A level is 10 launches with lists by atomics or by ranges and 11 by bins; where only
// the device knows the number of points, the last two have those of the atomics (3)
// as well.  Claiming lists by events, filling and sorting
// 16-byte entries, a separate bridge list, survival flags and three more scans
// took 1.70-2.25 ms a level on the 2^20-point sphere,
// this 0.36-0.55 ms.
#include <algorithm>
#include <initializer_list>

#include "common.hpp"
#include "events.hpp"
#include "merge_tile.hpp"
#include "walk.hpp"

namespace hull {

// Longest list kept unsorted.  Sorting is one thread's chain of dependent global
// accesses: with 12, k_par_sort took 170 us a level on the 2^20-point sphere
// (mean length 3, a few lists of 13-25), 6 with 32.
constexpr int kParScan = 32;
constexpr int kWave = 64;
constexpr unsigned long long kStepsLost = ~0ull;  // a segment to be walked again

// Lists built range by range in LDS rather than by global atomics: calls of many
// points, whose changes are enough to be bound by the atomics (they run at about
// 37 G/s and write one sector each), in blocks of up to 8 ranges (every range reads
// the child events of its whole merge).  Levels 12 to 16 of the 2^20 sphere took
// 872, 772, 711, 668 and 644 us by atomics, 551, 468, 427, 416 and 435 by ranges; the
// 10,000 ragged clouds of 1.3e8 points, 165 and 127 ms a pass.
constexpr int kRangeLog = 13;
constexpr int kRange = 1 << kRangeLog;  // points: two counts each, 64 KiB of LDS
constexpr int64_t kRangesFrom = int64_t(1) << 19;
__host__ __device__ constexpr bool lists_by_range(int64_t n, int k) {
  return n >= kRangesFrom && k >= kRangesFromLevel && k <= kRangeLog + 3;
}
// Above those levels, and at every level of calls of fewer points (whose ranges would
// be too few blocks), the changes are first sorted into bins of points (the
// levels' walk scratch, idle until then, holds them), then a block per bin builds its
// lists.  Levels 17 to 20 of the 2^20 sphere: 635, 623, 640 and 657 us by atomics,
// 387, 360, 369 and 373 by bins (counting 5, placing 14, lists 23 us a level, both runs).
// Delaunay of 262,139 points (levels 11 to 18, one run): 622 + 157 us a pass by atomics
// (k_par_enum, k_par_fill), 163 + 491 by bins with the segment table; 5.47 and 5.27 ms.
constexpr int64_t kBinsFrom = int64_t(1) << 17;
constexpr int64_t kBinsMax = 4096;  // a count of each in LDS
constexpr int kBinThreads = 512, kBinEvents = 8;
__host__ __device__ constexpr int64_t bins_of(int64_t n, int log) { return (n + (1 << log) - 1) >> log; }
// The bins' size (log), 0 for none: the host's rule.  The device builds lists by bins
// where this gives a size and it counts kBinsFrom points.
static int bin_log(const ParLevel& P) {
  const int log = P.n >= kRangesFrom ? kRangeLog : kRangeLog - 2, k = P.S.k;
  // records of the bins: 8 + 2 bytes each, up to 6 per point
  const bool room = bins_of(P.n, log) <= kBinsMax &&
                    (P.seg_cap + 1) * kSegKeep * (int64_t)sizeof(Event) >= 60 * P.n;
  const bool on = P.n >= kRangesFrom ? k > kRangeLog + 3 : P.n >= kBinsFrom && k >= kRangesFromLevel;
  return room && on ? log : 0;
}
__host__ __device__ constexpr int ranges_of(int k) { return k <= kRangeLog ? 1 : 1 << (k - kRangeLog); }
__host__ __device__ constexpr int range_points(int k) { return k <= kRangeLog ? 1 << k : kRange; }
// Threads per range: about 8 points each, so that blocks of small merges are many and
// their barriers cheap.
static int range_threads(int k) { return std::min(std::max(range_points(k) / 8, 64), 512); }

// A point's two lists lie side by side (their bounds are then one 8-byte load and the
// word after it, their entries often one cache line).
__device__ __forceinline__ int64_t key_of(int p, int prev) { return 2 * (int64_t)p + prev; }

template <class PT>
struct ParCtx {
  const PT* pts;
  const Event* evL;
  const Event* evR;
  const int* off;
  const int2* ent;
  const int* nx0;
  const int* pv0;
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
    const int64_t key = key_of(p, !nx);
    return last_before(off[key], off[key + 1], cursor, nx ? nx0[p] : pv0[p]);
  }
  __device__ __forceinline__ void links(int p, bool, int cursor, int& nx, int& pv) const {
    const int2 b = *(const int2*)(off + key_of(p, 0));
    const int end = off[key_of(p, 2)];
    const int ln = nx0[p], lp = pv0[p];
    nx = last_before(b.x, b.y, cursor, ln);
    pv = last_before(b.y, end, cursor, lp);
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
  X.zs = R.zs;
  return X;
}

// Sorts a list by position (Shell's method; only lists above kParScan, up to
// kParSerial).
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

// Longer lists (a vertex of high degree has one as long as the movie) are noted in LDS
// and sorted by the whole workgroup, one after the other: a cone over 16,384 points
// 1.8 ms, a moment curve 31; by one thread each 21 and 84.
constexpr int kParSerial = 128;
constexpr int kParRank = 1024;   // longest list whose entries count the smaller ones
constexpr int kLongLists = 64;   // noted at a time
struct LongLists {
  int count;
  int2 list[kLongLists];  // first entry, length
};
constexpr int sort_words(int T) { return 5 * T; }  // LDS of sort_long, lists above kParRank

// By rank up to kParRank entries.  Above, by windows of 128 T positions: the
// positions differ, so a bit each says which are there, and an entry's place is the
// number of bits before its own.  tmp: space for the list; the positions are below
// `limit`.
template <int T, class G>
__device__ void sort_long(const G& g, unsigned* lds, int2* a, int2* tmp, int k, int limit) {
  const int t = threadIdx.x;
  if (k <= kParRank) {
    for (int i = t; i < k; i += T) {
      const int2 x = a[i];
      int r = 0;
#pragma unroll 8
      for (int j = 0; j < k; ++j) r += a[j].x < x.x;
      tmp[r] = x;
    }
  } else {
    constexpr int window = 128 * T;
    unsigned* bits = lds;             // [4 T]
    int* before = (int*)(lds + 4 * T);  // [T]
    int done = 0;
    for (int lo = 0; done < k && lo < limit; lo += window) {
      for (int q = t; q < 4 * T; q += T) bits[q] = 0;
      __syncthreads();
      for (int i = t; i < k; i += T) {
        const unsigned x = (unsigned)(a[i].x - lo);
        if (x < (unsigned)window) atomicOr(&bits[x >> 5], 1u << (x & 31));
      }
      __syncthreads();
      int sum = 0, all;
      for (int q = 0; q < 4; ++q) sum += __popc(bits[4 * t + q]);
      before[t] = done + g.scan(sum, all);
      __syncthreads();
      for (int i = t; i < k; i += T) {
        const int2 e = a[i];
        const unsigned x = (unsigned)(e.x - lo);
        if (x >= (unsigned)window) continue;
        const int w = x >> 5;
        int r = before[w >> 2] + __popc(bits[w] & ((1u << (x & 31)) - 1));
        for (int q = w & ~3; q < w; ++q) r += __popc(bits[q]);
        tmp[r] = e;
      }
      done += all;
      __syncthreads();
    }
  }
  __syncthreads();
  for (int i = t; i < k; i += T) a[i] = tmp[i];
}

// Sorts the lists q, q + step, ... below `keys`: list(q) gives its first entry and its
// length.  S.count is 0, cleared before a barrier; it is again after the next one.
// The walk scratch takes the sorted entries (idle until the walks; 6 entries per point
// fit, and a bin's records there have been read to the end by its own block).
template <int T, class G, class LIST>
__device__ __forceinline__ void sort_lists(const G& g, LongLists& S, unsigned* lds, const ParLevel& P,
                                           const ParRun& Q, int q, int step, int keys,
                                           const LIST& list) {
  int2 *ent = Q.ent, *tmp = (int2*)Q.segKeep;
  for (;;) {
    for (; q < keys; q += step) {
      const int2 l = list(q);
      if (l.y > kParSerial) {
        const int at = atomicAdd(&S.count, 1);
        if (at >= kLongLists) break;  // the next round's
        S.list[at] = l;
      } else if (l.y > kParScan) {
        sort_entries(ent + l.x, l.y);
      }
    }
    __syncthreads();
    const int count = S.count;
    for (int i = 0; i < count && i < kLongLists; ++i)
      sort_long<T>(g, lds, ent + S.list[i].x, tmp + S.list[i].x, S.list[i].y, 2 * (int)P.n);
    __syncthreads();
    if (threadIdx.x == 0) S.count = 0;
    if (count <= kLongLists) return;
    __syncthreads();
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
  const int64_t n = P.S.off[P.S.H];
  const int64_t keys = merges ? 2 * n + 1 : 0;
  const bool bins = P.bin_log && n >= kBinsFrom, ranges = bins || lists_by_range(n, P.S.k);
  const bool err = P.h->err != 0;
  GRID_STRIDE(g, (int64_t)(err ? 0 : Q.ctr[kCtrSplice + ((P.S.k - 1) & 1)])) {
    const int2 b = Q.uv0[g];
    R.nx0[b.x] = b.y;
    R.pv0[b.y] = b.x;
  }
  GRID_STRIDE(g, merges + 1) {
    if (g == 0) {
      Q.ctr[kCtrMerges] = (int)merges;
      Q.ctr[kCtrKeys] = ranges ? 0 : (int)keys;
      const int count = err || !ranges || !merges ? 0 : (int)(bins ? bins_of(n, P.bin_log) : merges * P.ranges);
      Q.ctr[kCtrRanges] = count;
      // (no word at all without ranges: pos then holds the events' places)
      Q.ctr[kCtrTotals] = count ? count + 1 : 0;
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
  if (!ranges) GRID_STRIDE(q, keys) Q.off[q] = 0;
  if (bins) GRID_STRIDE(q, bins_of(n, P.bin_log)) ((int*)Q.pos)[q] = 0;
  if (err) return;
  if (merges <= gridDim.x) {  // one block per merge
    if (blockIdx.x >= merges) return;
    const int2 se = P.S.merge(blockIdx.x);
    const int64_t m = se.x + half, e = se.y;
    if (R.right_waits_in_output(m, e))
      (void)R.settle_right(m, e, R.right_len(m, e), threadIdx.x, blockDim.x);
    return;
  }
  // many merges (so short ones): few have a block to move, a wave looks at 64
  const int lane = threadIdx.x % kWave;
  for (int64_t g0 = blockIdx.x * (int64_t)blockDim.x + threadIdx.x - lane; g0 < merges;
       g0 += (int64_t)gridDim.x * blockDim.x) {
    const int64_t g = g0 + lane < merges ? g0 + lane : merges - 1;
    const int2 se = P.S.merge(g);
    unsigned long long todo = __ballot(g0 + lane < merges && R.right_waits_in_output(se.x + half, se.y));
    for (; todo; todo &= todo - 1) {
      const int q = __ffsll(todo) - 1;
      const int64_t m = __shfl(se.x, q) + half, e = __shfl(se.y, q);
      (void)R.settle_right(m, e, R.right_len(m, e), lane, kWave);
    }
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
  const int64_t half = int64_t(1) << (P.S.k - 1);
  const int events = Q.ctr[kCtrKeys] ? E : 0;  // (else the lists are built by range)
  GRID_STRIDE(c, (int64_t)events + Sg) {
    const bool seg = c >= events;
    const int64_t t = seg ? c - events : c;
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
    at.x = atomicAdd(&Q.off[key_of(x.a, 0)], 1);
    at.y = atomicAdd(&Q.off[key_of(x.b, 1)], 1);
    if (x.kind) {
      at.z = atomicAdd(&Q.off[key_of(x.w, 0)], 1);
      at.w = atomicAdd(&Q.off[key_of(x.w, 1)], 1);
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
  const int64_t half = int64_t(1) << (P.S.k - 1);
  // capacity: 6 entries per point (the last bound is all entries)
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
    Q.ent[Q.off[key_of(x.a, 0)] + at.x] = make_int2(j, x.kind ? x.w : x.b);
    Q.ent[Q.off[key_of(x.b, 1)] + at.y] = make_int2(j, x.kind ? x.w : x.a);
    if (x.kind) {
      Q.ent[Q.off[key_of(x.w, 0)] + at.z] = make_int2(j, x.b);
      Q.ent[Q.off[key_of(x.w, 1)] + at.w] = make_int2(j, x.a);
    }
  }
}

// One range of points of one merge.
struct Range {
  int64_t s, m, e, p0;
  int pn, nL, N;
  bool closes;  // the points after it belong to no merge: it ends its lists itself
  const Event* evL;
  const Event* evR;
  __device__ __forceinline__ Range(const ParLevel& P, const RunPtrs& R, int64_t pair, int64_t merges) {
    const int64_t g = pair / P.ranges;
    const int r = (int)(pair - g * P.ranges);
    const int2 se = P.S.merge(g);
    s = se.x;
    m = s + (int64_t(1) << (P.S.k - 1));
    e = se.y;
    p0 = s + (int64_t)r * kRange;
    pn = p0 >= e ? 0 : (int)(e - p0 < kRange ? e - p0 : kRange);
    closes = pn > 0 && p0 + pn == e && (g + 1 == merges || P.S.merge(g + 1).x != e);
    nL = R.left_len(s);
    N = nL + R.right_len(m, e);
    evL = R.left_ev(s);
    evR = R.ev[(P.S.k - 1) & 1] + 2 * m;
  }
  // fn(point within the range, which list, position in the child movie, link
  // after) for every link that the merge's child events change in the range
  template <int T, class FN>
  __device__ __forceinline__ void changes(const FN& fn) const {
    constexpr int U = 4;  // events in flight per thread
    for (int c0 = threadIdx.x; c0 < N; c0 += U * T) {
      int4 x[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = c0 + u * T;
        if (c < N) x[u] = *(const int4*)(c < nL ? evL + c : evR + (c - nL));
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int c = c0 + u * T;
        if (c >= N) continue;
        const int j = c < nL ? c : c - nL, w = x[u].y & 0x7fffffff;
        const bool ins = x[u].y < 0;
        const unsigned a = (unsigned)(x[u].x - (int)p0), i = (unsigned)(w - (int)p0),
                       b = (unsigned)(x[u].z - (int)p0);
        if (a < (unsigned)pn) fn((int)a, 0, j, ins ? w : x[u].z);
        if (b < (unsigned)pn) fn((int)b, 1, j, ins ? w : x[u].x);
        if (ins && i < (unsigned)pn) {
          fn((int)i, 0, j, x[u].z);
          fn((int)i, 1, j, x[u].x);
        }
      }
    }
  }
};

// Offsets of the lists of counted lengths in LDS (keys of them), in order from `first`
// on; returns their total.
template <int T, class G>
__device__ __forceinline__ int lists_scan(const G& g, const int* cnt, int keys, int* off, int first) {
  int total = 0;
  for (int q0 = 0; q0 < keys; q0 += 4 * T) {
    const int q = q0 + 4 * threadIdx.x;
    int v[4], sum = 0, all;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      v[j] = sum;
      if (q + j < keys) sum += cnt[q + j];
    }
    const int before = first + total + g.scan(sum, all);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (q + j < keys) off[q + j] = before + v[j];
    total += all;
  }
  return total;
}
// Lengths of a range's lists, as offsets within the range, and their total.
template <int T>
__global__ void __launch_bounds__(T) k_list_count(ParLevel P) {
  extern __shared__ int range_lds[];
  __shared__ int wsum[T / 64];
  int* cnt = range_lds;
  const RunPtrs& R = P.run[blockIdx.y];
  const ParRun& Q = P.par[blockIdx.y];
  if (!R.pts) return;
  const int64_t pairs = Q.ctr[kCtrRanges], merges = Q.ctr[kCtrMerges];
  int* totals = (int*)Q.pos;
  const BlockGroup<T> g{wsum};
  for (int64_t pair = blockIdx.x; pair < pairs; pair += gridDim.x) {
    const Range X(P, R, pair, merges);
    const int keys = 2 * X.pn;
    __syncthreads();
    for (int q = threadIdx.x; q < keys; q += T) cnt[q] = 0;
    __syncthreads();
    if (X.pn) X.template changes<T>([&](int p, int l, int, int) { atomicAdd(&cnt[2 * p + l], 1); });
    __syncthreads();
    const int total = lists_scan<T>(g, cnt, keys, Q.off + key_of((int)X.p0, 0), 0);
    if (threadIdx.x == 0) totals[pair] = total;
  }
}

// The lists' bounds and entries, once the totals are scanned; long lists sorted.
template <int T>
__global__ void __launch_bounds__(T) k_list_fill(ParLevel P) {
  extern __shared__ int range_lds[];
  __shared__ LongLists S;
  __shared__ int wsum[T / 64];
  int* cur = range_lds;
  const BlockGroup<T> g{wsum};
  if (threadIdx.x == 0) S.count = 0;
  const RunPtrs& R = P.run[blockIdx.y];
  const ParRun& Q = P.par[blockIdx.y];
  if (!R.pts) return;
  const int64_t pairs = Q.ctr[kCtrRanges], merges = Q.ctr[kCtrMerges];
  const int* before = (const int*)Q.pos;
  if (pairs > 0 && before[pairs] > 6 * P.n) {
    if (blockIdx.x == 0 && threadIdx.x == 0) atomicCAS(&P.h->err, 0, HULL_EINTERNAL);
    return;
  }
  for (int64_t pair = blockIdx.x; pair < pairs; pair += gridDim.x) {
    const Range X(P, R, pair, merges);
    int* off = Q.off + key_of((int)X.p0, 0);
    const int keys = 2 * X.pn, base = before[pair];
    __syncthreads();
    for (int q = threadIdx.x; q < keys; q += T) {
      const int v = off[q] + base;
      cur[q] = v;
      off[q] = v;
    }
    if (threadIdx.x == 0 && X.closes) off[keys] = before[pair + 1];
    __syncthreads();
    if (!X.pn) continue;
    X.template changes<T>([&](int p, int l, int j, int link) {
      Q.ent[atomicAdd(&cur[2 * p + l], 1)] = make_int2(j, link);
    });
    __syncthreads();  // (also makes the block's entries visible to all of it)
    // (longer lists than kParRank come from level 11 on, whose ranges have 16 T words)
    static_assert(16 * T >= sort_words(T) && kParRank >= 1 << 10, "");
    const int end = before[pair + 1];
    sort_lists<T>(g, S, (unsigned*)range_lds, P, Q, threadIdx.x, T, keys, [&](int q) {
      return make_int2(off[q], (q + 1 < keys ? off[q + 1] : end) - off[q]);
    });
  }
}

// A link change on its way to its bin: the list (2 x point within the bin + prev),
// the event's position in its child movie and the link after it.
struct BinRecords {
  int2* rec;
  unsigned short* list;
  __device__ __forceinline__ BinRecords(const ParLevel& P, const ParRun& Q)
      : rec((int2*)Q.segKeep), list((unsigned short*)((int2*)Q.segKeep + 6 * P.n)) {}
};

// fn(point, prev, position, link) for the changes of the events of a block's chunk.
template <class FN>
__device__ __forceinline__ void bin_changes(const int4* x, const int* j, const FN& fn) {
#pragma unroll
  for (int u = 0; u < kBinEvents; ++u) {
    if (j[u] < 0) continue;
    const int w = x[u].y & 0x7fffffff;
    const bool ins = x[u].y < 0;
    fn(x[u].x, 0, j[u], ins ? w : x[u].z);
    fn(x[u].z, 1, j[u], ins ? w : x[u].x);
    if (ins) {
      fn(w, 0, j[u], x[u].z);
      fn(w, 1, j[u], x[u].x);
    }
  }
}

// The bins' counts (PLACE: their records, at the counts scanned), chunk by chunk of
// the level's child events.
template <bool PLACE>
__global__ void __launch_bounds__(kBinThreads) k_bin(ParLevel P) {
  extern __shared__ int range_lds[];
  int* cnt = range_lds;
  const RunPtrs& R = P.run[blockIdx.y];
  const ParRun& Q = P.par[blockIdx.y];
  if (!R.pts) return;
  const int bins = Q.ctr[kCtrRanges], merges = Q.ctr[kCtrMerges], E = Q.ctr[kCtrEvents];
  int* total = (int*)Q.pos;
  if (!bins || (PLACE && total[bins] > 6 * P.n)) return;  // (k_bin_lists reports it)
  const BinRecords B(P, Q);
  constexpr int kChunk = kBinThreads * kBinEvents;
  for (int64_t c0 = (int64_t)blockIdx.x * kChunk; c0 < E; c0 += (int64_t)gridDim.x * kChunk) {
    __syncthreads();
    for (int q = threadIdx.x; q < bins; q += kBinThreads) cnt[q] = 0;
    __syncthreads();
    int4 x[kBinEvents];
    int j[kBinEvents];
#pragma unroll
    for (int u = 0; u < kBinEvents; ++u) {
      const int64_t c = c0 + u * kBinThreads + threadIdx.x;
      j[u] = -1;
      if (c >= E) continue;
      const int g = find_owner(Q.eoff, merges, c);
      const int64_t s = P.S.merge(g).x, m = s + (int64_t(1) << (P.S.k - 1));
      const int nL = R.left_len(s), i = (int)(c - Q.eoff[g]);
      const bool left = i < nL;
      j[u] = left ? i : i - nL;
      x[u] = *(const int4*)((left ? R.left_ev(s) : R.ev[(P.S.k - 1) & 1] + 2 * m) + j[u]);
    }
    bin_changes(x, j, [&](int p, int, int, int) { atomicAdd(&cnt[p >> P.bin_log], 1); });
    __syncthreads();
    for (int q = threadIdx.x; q < bins; q += kBinThreads)
      if (cnt[q]) cnt[q] = atomicAdd(&total[q], cnt[q]);
    if (!PLACE) continue;
    __syncthreads();
    bin_changes(x, j, [&](int p, int prev, int pos, int link) {
      const int at = atomicAdd(&cnt[p >> P.bin_log], 1);
      B.rec[at] = make_int2(pos, link);
      B.list[at] = (unsigned short)(2 * (p & ((1 << P.bin_log) - 1)) + prev);
    });
  }
}

// The lists of a bin's points: counted, their bounds, filled, the long ones sorted.
template <int T>
__global__ void __launch_bounds__(T) k_bin_lists(ParLevel P) {
  extern __shared__ int range_lds[];
  __shared__ int wsum[T / 64];
  __shared__ LongLists S;
  if (threadIdx.x == 0) S.count = 0;
  int* cnt = range_lds;
  const ParRun& Q = P.par[blockIdx.y];
  if (!P.run[blockIdx.y].pts) return;
  const int bins = Q.ctr[kCtrRanges];
  const int* ends = (const int*)Q.pos;  // where k_bin left its cursors
  if (bins && ends[bins] > 6 * P.n) {
    if (blockIdx.x == 0 && threadIdx.x == 0) atomicCAS(&P.h->err, 0, HULL_EINTERNAL);
    return;
  }
  const int64_t n = P.S.off[P.S.H];
  const BinRecords B(P, Q);
  const BlockGroup<T> g{wsum};
  for (int b = blockIdx.x; b < bins; b += gridDim.x) {
    const int first = b ? ends[b - 1] : 0, end = ends[b];
    const int64_t p0 = (int64_t)b << P.bin_log;
    const int64_t most = int64_t(1) << P.bin_log;
    const int keys = 2 * (int)(n - p0 < most ? n - p0 : most);
    int* off = Q.off + key_of((int)p0, 0);
    __syncthreads();
    for (int q = threadIdx.x; q < keys; q += T) cnt[q] = 0;
    __syncthreads();
    for (int q = first + threadIdx.x; q < end; q += T) atomicAdd(&cnt[B.list[q]], 1);
    __syncthreads();
    (void)lists_scan<T>(g, cnt, keys, off, first);
    if (threadIdx.x == 0 && b + 1 == bins) off[keys] = end;
    __syncthreads();
    for (int q = threadIdx.x; q < keys; q += T) cnt[q] = off[q];
    __syncthreads();
    for (int q = first + threadIdx.x; q < end; q += T) Q.ent[atomicAdd(&cnt[B.list[q]], 1)] = B.rec[q];
    __syncthreads();
    sort_lists<T>(g, S, (unsigned*)range_lds, P, Q, threadIdx.x, T, keys, [&](int q) {
      return make_int2(off[q], (q + 1 < keys ? off[q + 1] : end) - off[q]);
    });
  }
}

// Sorts the long lists of k_par_fill (lists built by range: no keys).
__global__ void __launch_bounds__(256) k_par_sort(ParLevel P) {
  __shared__ LongLists S;
  __shared__ int wsum[4];
  __shared__ unsigned lds[sort_words(256)];
  const ParRun& Q = P.par[blockIdx.y];
  if (!P.run[blockIdx.y].pts) return;
  if (threadIdx.x == 0) S.count = P.h->err ? -1 : 0;  // (one reading for the whole block)
  __syncthreads();
  if (S.count < 0) return;
  sort_lists<256>(BlockGroup<256>{wsum}, S, lds, P, Q, blockIdx.x * 256 + threadIdx.x, gridDim.x * 256,
                  Q.ctr[kCtrKeys] - 1, [&](int q) { return make_int2(Q.off[q], Q.off[q + 1] - Q.off[q]); });
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

// Every counted segment's events to their place in the merged movie.  A lane
// decodes its segment's steps into references in LDS, then the wave copies the
// events of its 64 segments in output order, so that writes are whole lines and
// reads nearly.  10,000 ragged clouds, levels 10 to 16: 3.3 ms
// a pass, and 1.6 for the segments walked again; a lane writing its own segment's
// events, in one kernel with the walks (150 VGPRs), took 25.3 over levels 8 to 16.
template <class PT>
__global__ void __launch_bounds__(kWave) k_par_write(ParLevel P) {
  __shared__ unsigned short ref[kWave * kWalkSteps];  // lane, source, event of the source
  __shared__ const int4* src[3][kWave];               // left and right child, bridge events
  __shared__ int4* dst[kWave];
  const RunPtrs& R = P.run[blockIdx.y];
  const ParRun& Q = P.par[blockIdx.y];
  if (!R.pts || !Q.ctr[kCtrMerges]) return;
  const bool err = P.h->err != 0;
  const int64_t total = Q.ctr[kCtrSegments];
  const int lane = threadIdx.x;
  for (int64_t t0 = (int64_t)blockIdx.x * kWave; t0 < total; t0 += (int64_t)gridDim.x * kWave) {
    const int64_t t = t0 + lane;
    unsigned long long steps = 0;
    int count = 0, jL = 0, jR = 0;
    int64_t s = 0, m = 0;
    Event* out = nullptr;
    if (t < total) {
      const int g = Q.segMerge[t], first = Q.segBase[g], S = Q.segS[g];
      const int2 se = P.S.merge(g);
      s = se.x;
      m = s + (int64_t(1) << (P.S.k - 1));
      const int before = Q.segOff[first], len = Q.segOff[first + S] - before;
      const bool fits = !err && len <= 2 * (se.y - s);
      if (t == first) R.out_len(s) = fits ? len : 0;  // also after an error
      if (!fits) {
        if (!err) atomicCAS(&P.h->err, 0, HULL_EINTERNAL);
      } else if (Q.segSteps[t] != kStepsLost) {
        steps = Q.segSteps[t];
        count = Q.segOff[t + 1] - Q.segOff[t];
        jL = Q.segJ[t];
        jR = (int)((t - first) * (R.left_len(s) + (int64_t)R.right_len(m, se.y)) / S) - jL;
        out = R.out_ev(s) + (Q.segOff[t] - before);
      }
    }
    int end = count;
    for (int o = 1; o < kWave; o <<= 1) {
      const int y = __shfl_up(end, o);
      if (lane >= o) end += y;
    }
    const int all = __shfl(end, kWave - 1);
    int p = end - count;
    __syncthreads();  // the earlier segments' copies
    if (count) {
      src[0][lane] = (const int4*)(R.left_ev(s) + jL);
      src[1][lane] = (const int4*)(R.ev[(P.S.k - 1) & 1] + 2 * m + jR);
      src[2][lane] = (const int4*)(Q.segKeep + t * kSegKeep);
      dst[lane] = (int4*)out - p;
    }
    int nL = 0, nR = 0, nB = 0;
    for (; steps; steps >>= 3) {
      const int code = (int)steps & 7;
      const bool left = code == kStepL || code == kStepHideL, bridge = code == kStepBridge;
      const int i = bridge ? nB : (left ? nL : nR);
      if (bridge || code == kStepL || code == kStepR)
        ref[p++] = (unsigned short)(lane | (bridge ? 2 : !left) << 6 | i << 8);
      nB += bridge;
      nL += !bridge && left;
      nR += !bridge && !left;
    }
    __syncthreads();
    for (int q = lane; q < all; q += kWave) {
      const int r = ref[q], o = r & 63;
      dst[o][q] = src[(r >> 6) & 3][o][r >> 8];
    }
  }
}

// The segments whose steps were too many to note, walked again.
template <class PT>
__global__ void __launch_bounds__(64) k_par_rewalk(ParLevel P) {
  const RunPtrs& R = P.run[blockIdx.y];
  const ParRun& Q = P.par[blockIdx.y];
  if (!R.pts || !Q.ctr[kCtrMerges] || P.h->err) return;
  GRID_STRIDE(t, (int64_t)Q.ctr[kCtrSegments]) {
    if (Q.segSteps[t] != kStepsLost) continue;
    const int g = Q.segMerge[t];
    const ParSeg<PT> Z(P, blockIdx.y, t, g);
    const int first = Q.segBase[g];
    ParWrite wr{R.out_ev(Z.s) + (Q.segOff[t] - Q.segOff[first])};
    const int2 uv = Q.segUV[t];
    (void)walk<PT>(Z.X, uv.x, uv.y, Z.jL, Z.kL, Z.jR, Z.kR, Z.i + 1 == Z.S, Z.i > 0, Z.T, Z.limit, wr);
  }
}

// Scans of the same arrays of both runs in one launch.  kinds: 0 child events
// and 1 walk segments per merge (their totals are the level's), 2 the lists'
// lengths by key, 3 events put out per segment, 4 entries per range or bin.
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
        case 4: j = ScanJob{(int*)Q.pos, (int*)Q.pos, Q.ctr + kCtrTotals, nullptr}; break;
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
int32_t parallel_level(const ParLevel& level, hipStream_t s) {
  ParLevel P = level;
  P.ranges = ranges_of(P.S.k);
  P.bin_log = bin_log(P);
  // The device may have few segments, and an empty block costs its dispatch (2^24
  // points, 1% on a sphere: 3.14 ms with 16384 blocks a run, 3.06 with 4096; 2^20 sphere:
  // 7.64 and 7.61, 7.98 with 2048).  Calls of more points keep the finer split, and
  // enough blocks for their segments walked again (10,000 ragged clouds: 114.2 ms
  // with 4096, 117.1 with 512).  The same for the blocks of the lists (2^24: 3.05 and
  // 3.01 ms).
  const bool huge = P.n >= int64_t(1) << 25;
  const dim3 g2(kStrideBlocks, 2), b256(256);
  hipLaunchKernelGGL(k_par_prep, g2, b256, 0, s, P);
  int32_t rc = chained(P, jobs_of(P, {0, 1}), 0, 1, 1, P.mcap + 1, s);
  if (rc) return rc;
  hipLaunchKernelGGL(k_par_enum<PT>, g2, b256, 0, s, P);
  if (lists_by_range(P.n, P.S.k)) {  // the device's number of points may say otherwise
    // (a merge at level k has more than 2^(k-1) points)
    const int64_t pairs = ((P.n >> (P.S.k - 1)) + 1) * P.ranges;
    const int T = range_threads(P.S.k);
    const dim3 gr((unsigned)std::min<int64_t>(pairs, (int64_t)(huge ? 2048 : 1024) * 512 / T), 2);
    const size_t lds = 2 * sizeof(int) * range_points(P.S.k);
#define HULL_RANGES(KERNEL)                                                            \
  if (T == 512) hipLaunchKernelGGL(KERNEL<512>, gr, dim3(512), lds, s, P);             \
  else if (T == 256) hipLaunchKernelGGL(KERNEL<256>, gr, dim3(256), lds, s, P);        \
  else if (T == 128) hipLaunchKernelGGL(KERNEL<128>, gr, dim3(128), lds, s, P);        \
  else hipLaunchKernelGGL(KERNEL<64>, gr, dim3(64), lds, s, P);
    HULL_RANGES(k_list_count)
    rc = chained(P, jobs_of(P, {4}), 8, 4, 0, pairs + 1, s);
    if (rc) return rc;
    HULL_RANGES(k_list_fill)
#undef HULL_RANGES
  }
  if (P.bin_log) {
    const int64_t nb = bins_of(P.n, P.bin_log);
    const size_t lds = nb * sizeof(int);
    const dim3 gb((unsigned)std::min<int64_t>((2 * P.n) / (kBinThreads * kBinEvents) + 1, 512), 2);
    hipLaunchKernelGGL(k_bin<false>, gb, dim3(kBinThreads), lds, s, P);
    rc = chained(P, jobs_of(P, {4}), 8, 4, 0, nb + 1, s);
    if (rc) return rc;
    hipLaunchKernelGGL(k_bin<true>, gb, dim3(kBinThreads), lds, s, P);
    hipLaunchKernelGGL(k_bin_lists<1024>, dim3((unsigned)std::min<int64_t>(nb, 512), 2), dim3(1024),
                       sizeof(int) * std::max(2 << P.bin_log, sort_words(1024)), s, P);
  }
  if (!(P.bin_log || lists_by_range(P.n, P.S.k)) || P.device_n) {
    rc = chained(P, jobs_of(P, {2}), 4, 2, 0, 2 * P.n + 1, s);
    if (rc) return rc;
    hipLaunchKernelGGL(k_par_fill<PT>, g2, b256, 0, s, P);
    hipLaunchKernelGGL(k_par_sort, g2, b256, 0, s, P);
  }
  const dim3 gw((unsigned)std::min<int64_t>(P.seg_cap / 64 + 1, huge ? 16384 : 4096), 2), b64(64);
  hipLaunchKernelGGL(k_par_walk<PT>, gw, b64, 0, s, P);
  rc = chained(P, jobs_of(P, {3}), 6, 3, 1, P.seg_cap + 1, s);
  if (rc) return rc;
  hipLaunchKernelGGL(k_par_write<PT>, gw, b64, 0, s, P);
  hipLaunchKernelGGL(k_par_rewalk<PT>, dim3(std::min(gw.x, huge ? 4096u : 1024u), 2), b64, 0, s, P);
  HULL_LAUNCH_CHECK();
  return HULL_OK;
}

template int32_t parallel_level<int4>(const ParLevel&, hipStream_t);
template int32_t parallel_level<WPt>(const ParLevel&, hipStream_t);

}  // namespace hull
