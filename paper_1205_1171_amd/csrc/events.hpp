// Events of a movie as comparison candidates, and their exact order.
#pragma once
#include "common.hpp"
#include "predicates.hpp"

namespace hull {

struct Cand {
  Tri t;
  double st;  // standard part of tau (NaN: not covered by the fast path)
  int kind;   // 1 insertion, 0 deletion
};

// Levels of merges that a block of n points has behind it.
__host__ __device__ inline int levels_of(int64_t n) {
  return n <= 1 ? 0 : 64 - __builtin_clzll((unsigned long long)(n - 1));
}

// Pointers of one run (lower or upper).
// pts: the points by rank, int4 (x, y, z, w) on the standard range or WPt on
// the wide range (the kernels are instantiated for each).
// A block's movie sits in the buffer of the last level that merged it: level
// k writes buffer k & 1, and a block of n points was last merged at level
// levels_of(n) (an unpaired trailing block waits there for as many levels as
// it takes).
struct RunPtrs {
  const void* pts;
  int* pv0;
  int* nx0;
  int2* lk;  // working links of the level: (pv, nx) of each point
  Event* ev[2];
  int* len[2];
  int k;  // the level
  int zs;
  // The left block of a merge at this level is always a full one.
  __device__ __forceinline__ const Event* left_ev(int64_t s) const { return ev[(k - 1) & 1] + 2 * s; }
  __device__ __forceinline__ int left_len(int64_t s) const { return len[(k - 1) & 1][s]; }
  __device__ __forceinline__ const Event* right_ev(int64_t m, int64_t e) const {
    return ev[levels_of(e - m) & 1] + 2 * m;
  }
  __device__ __forceinline__ int right_len(int64_t m, int64_t e) const {
    return len[levels_of(e - m) & 1][m];
  }
  // Where the right block waits in the buffer that this level writes, its movie
  // would be overwritten while it is read (the merged movie covers its slots):
  // it moves to the other buffer first, copied by a group of `size` threads.
  // The caller's threads must see each other's stores before they read it.
  __device__ __forceinline__ bool right_waits_in_output(int64_t m, int64_t e) const {
    return ((levels_of(e - m) ^ k) & 1) == 0;
  }
  __device__ __forceinline__ const Event* settle_right(int64_t m, int64_t e, int nR, int rank,
                                                       int size) const {
    if (right_waits_in_output(m, e)) {
      const Event* src = ev[k & 1] + 2 * m;
      Event* dst = ev[(k - 1) & 1] + 2 * m;
      for (int q = rank; q < nR; q += size) dst[q] = src[q];
    }
    return ev[(k - 1) & 1] + 2 * m;
  }
  __device__ __forceinline__ Event* out_ev(int64_t s) const { return ev[k & 1] + 2 * s; }
  __device__ __forceinline__ int& out_len(int64_t s) const { return len[k & 1][s]; }
};

// Working links (pv, nx) of a merge's points, in one of three places.  The
// merge kernels read and write them only through get / set_pv / set_nx /
// set, so one merge loop serves all three.
//
// In global memory: one int2 per point, indexed like the point array.
struct GlobalLinks {
  int2* p;
  __device__ __forceinline__ int2 get(int i) const { return p[i]; }
  __device__ __forceinline__ void set_pv(int i, int v) const { p[i].x = v; }
  __device__ __forceinline__ void set_nx(int i, int v) const { p[i].y = v; }
  __device__ __forceinline__ void set(int i, int pv, int nx) const { p[i] = make_int2(pv, nx); }
};

// In LDS, as block-local ranks (kNil stays -1) in a narrow signed type: one
// lane's merge of up to kLinkLdsLane points in int8, a lane group's merge in
// int16 while the block's groups need at most kLinkLdsGroupBytes.  Entry i
// sits at p[i * STRIDE] (STRIDE 64: the entries of a wave's 64 lanes
// interleaved, so that a wave-wide access spans consecutive banks).  Indices
// and link values are block-local.
constexpr int kLinkLdsLane = 128;
constexpr int kLinkLdsGroupBytes = 32768;
template <class T>
struct __align__(2 * sizeof(T)) LinkPair {
  T pv, nx;
};
template <class T, int STRIDE>
struct LdsLinks {
  LinkPair<T>* p;
  __device__ __forceinline__ int2 get(int i) const {
    const LinkPair<T> e = p[i * STRIDE];
    return make_int2(e.pv, e.nx);
  }
  __device__ __forceinline__ void set_pv(int i, int v) const { p[i * STRIDE].pv = (T)v; }
  __device__ __forceinline__ void set_nx(int i, int v) const { p[i * STRIDE].nx = (T)v; }
  __device__ __forceinline__ void set(int i, int pv, int nx) const {
    LinkPair<T> e;
    e.pv = (T)pv;
    e.nx = (T)nx;
    p[i * STRIDE] = e;
  }
};

// In LDS as above, for a merge loop that works in global ranks: indices and
// link values are shifted by the block start on the way in and out.
template <class T>
struct LdsLinksShifted {
  LinkPair<T>* p;
  int base;
  __device__ __forceinline__ int2 get(int i) const {
    const LinkPair<T> e = p[i - base];
    return make_int2(e.pv < 0 ? kNil : e.pv + base, e.nx < 0 ? kNil : e.nx + base);
  }
  __device__ __forceinline__ void set_pv(int i, int v) const {
    p[i - base].pv = (T)(v == kNil ? -1 : v - base);
  }
  __device__ __forceinline__ void set_nx(int i, int v) const {
    p[i - base].nx = (T)(v == kNil ? -1 : v - base);
  }
  __device__ __forceinline__ void set(int i, int pv, int nx) const {
    LinkPair<T> e;
    e.pv = (T)(pv == kNil ? -1 : pv - base);
    e.nx = (T)(nx == kNil ? -1 : nx - base);
    p[i - base] = e;
  }
};

// The hulls of a call (rank offsets) and the merges of a level: pairs of
// adjacent blocks inside a hull.  A single hull's follow from its number of
// points; a batch's are listed on the device for every level.
struct Sched {
  const int64_t* off;  // [H + 1] rank offsets of the hulls
  int64_t H;
  int* moff;           // [H + 1] merges before each hull; moff[H] = merges of the level
  int2* mlist;         // [mcap] (s, e) of each merge, m = s + half
  int k;               // the level
  __device__ __forceinline__ int64_t merges() const {
    if (H != 1) return moff[H];
    return ((off[1] + (int64_t(1) << (k - 1)) - 1) >> (k - 1)) >> 1;
  }
  __device__ __forceinline__ int2 merge(int64_t g) const {
    if (H != 1) return mlist[g];
    const int64_t s = g << k, e = s + (int64_t(1) << k), n = off[1];
    return make_int2((int)s, (int)(e < n ? e : n));
  }
};

// A level's merges run either way (kernels' `sel`: 1, only if the level counts as
// many merges; 2, only if it does not; 0, always).  The host cannot tell once
// interior points have been taken out, so both kernels are launched and the
// device's number of points decides.  Many: enough merges to fill the chip one
// lane or lane group each, or a block's points mostly not vertices.
constexpr int64_t kTileMerges = 49152;
constexpr int64_t kTilePoints = int64_t(1) << 21;
__host__ __device__ inline bool many_merges(int64_t merges, int64_t n) {
  return 2 * merges >= kTileMerges || n > kTilePoints;
}
__device__ __forceinline__ bool selected(const Sched& S, int sel) {
  return sel == 0 || many_merges(S.merges(), S.off[S.H]) == (sel == 1);
}

struct LevelArgs {
  RunPtrs run[2];
  int* perm[2];   // per run: merge of each lane (nullptr: lane g takes merge g)
  int* wbins[2];  // per run: histogram, then cursors, of the work order
  Header* h;
  Sched S;
  int64_t half;   // size of a left block
  int64_t width;  // size of a merged block
  int sel;
};
// Exact (time, rank triple) order of two events (cold path).  Arguments
// go by value so that callers keep their candidates in registers.  lead: what
// lead_cmp gave (its three coefficients are not taken again where they vanish).
constexpr int kLeadOpen = 2;
template <class PT>
__device__ __noinline__ int tri_cmp_exact(const PT* pts, Tri A, Tri B, int zs, int lead) {
  Coef ca, cb;
  coef_of(pts[A.a], pts[A.w], pts[A.b], zs, ca);
  coef_of(pts[B.a], pts[B.w], pts[B.b], zs, cb);
  int s = tau_cmp_exact(ca, cb, lead == 0 ? 3 : 0);
  if (s) return s;
  if (A.a != B.a) return A.a < B.a ? -1 : 1;
  if (A.w != B.w) return A.w < B.w ? -1 : 1;
  if (A.b != B.b) return A.b < B.b ? -1 : 1;
  return 0;
}

// Leading terms of D and N of a triple, exact in int64: D0, N0 (the
// unperturbed orientations) and D1, N1 (their e1 coefficients).
struct Lead {
  int64_t d0, n0, d1, n1;
};

__device__ __forceinline__ Lead lead_of(int4 P, int4 Q, int4 R, int zs) {
  const int dx1 = dif32(Q.x, P.x), dx2 = dif32(R.x, P.x);
  const int dy1 = dif32(Q.y, P.y), dy2 = dif32(R.y, P.y);
  const int dz1 = dif32(Q.z, P.z), dz2 = dif32(R.z, P.z);
  const int di1 = Q.w - P.w, di2 = R.w - P.w;
  Lead L;
  L.d0 = mul32(dx1, dy2) - mul32(dx2, dy1);
  L.n0 = zs * (mul32(dx1, dz2) - mul32(dx2, dz1));
  L.d1 = mul32(di1, dy2) - mul32(di2, dy1);
  L.n1 = zs * (mul32(di1, dz2) - mul32(di2, dz1));
  return L;
}

// Exact order when the double filter cannot decide.  The first three
// coefficients of N_A D_B - N_B D_A (monomials 1, e1, e1^2) fit int128:
//   N0a D0b - N0b D0a,  N0a D1b + N1a D0b - N0b D1a - N1b D0a,  N1a D1b - N1b D1a.
// They decide every tie of the standard parts that comes from a pair of
// points with equal x (all triples on such a pair share a standard part),
// with no 256-bit arithmetic; only when all three vanish (or D0 = D1 = 0)
// does the full cascade run.
// Sign of tau_A - tau_B from coefficients 1-3 of both leading terms; 0 when all
// three vanish, kLeadOpen when they cannot be taken (D0 = D1 = 0 on a side).
__device__ __forceinline__ int lead_cmp(const Lead& a, const Lead& b) {
  const int sa = a.d0 ? (a.d0 > 0 ? 1 : -1) : (a.d1 > 0) - (a.d1 < 0);
  const int sb = b.d0 ? (b.d0 > 0 ? 1 : -1) : (b.d1 > 0) - (b.d1 < 0);
  if (sa && sb) {
    i128 p = (i128)a.n0 * b.d0 - (i128)b.n0 * a.d0;
    if (!p) {
      p = (i128)a.n0 * b.d1 + (i128)a.n1 * b.d0 - (i128)b.n0 * a.d1 - (i128)b.n1 * a.d0;
      if (!p) p = (i128)a.n1 * b.d1 - (i128)b.n1 * a.d1;
    }
    return p ? (p > 0 ? 1 : -1) * sa * sb : 0;
  }
  return kLeadOpen;
}

__device__ __forceinline__ int tri_cmp_mid_body(const int4* pts, Tri A, Tri B, int zs) {
  const int s = lead_cmp(lead_of(pts[A.a], pts[A.w], pts[A.b], zs),
                         lead_of(pts[B.a], pts[B.w], pts[B.b], zs));
  return s == 1 || s == -1 ? s : tri_cmp_exact(pts, A, B, zs, s);
}

// The same on the wide range, where D0, N0, D1, N1 need int128 and their
// products may not fit it (N0 D0 up to 2^138): the three coefficients are
// taken in int128 when every leading term's bit length leaves the products
// below 2^124 (so that no sum of four overflows), which covers, for
// instance, all lifted points of |x|, |y| <= 2^20 (N up to 2^70, D up to
// 2^48); otherwise the full cascade decides.
struct WLead {
  i128 d0, n0, d1, n1;
};

__device__ __forceinline__ WLead lead_of(const WPt& P, const WPt& Q, const WPt& R, int zs) {
  const int64_t dx1 = (int64_t)Q.x - P.x, dx2 = (int64_t)R.x - P.x;
  const int64_t dy1 = (int64_t)Q.y - P.y, dy2 = (int64_t)R.y - P.y;
  const int64_t dz1 = Q.z - P.z, dz2 = R.z - P.z;
  const int64_t di1 = Q.w - P.w, di2 = R.w - P.w;
  WLead L;
  L.d0 = (i128)dx1 * dy2 - (i128)dx2 * dy1;
  L.n0 = zs * ((i128)dx1 * dz2 - (i128)dx2 * dz1);
  L.d1 = (i128)di1 * dy2 - (i128)di2 * dy1;
  L.n1 = zs * ((i128)di1 * dz2 - (i128)di2 * dz1);
  return L;
}

__device__ __forceinline__ int bits128(i128 v) {
  const u128 u = v < 0 ? (u128)(-v) : (u128)v;
  const uint64_t hi = (uint64_t)(u >> 64), lo = (uint64_t)u;
  return hi ? 128 - __builtin_clzll(hi) : (lo ? 64 - __builtin_clzll(lo) : 0);
}

__device__ __forceinline__ int lead_cmp(const WLead& a, const WLead& b) {
  const int sa = a.d0 ? (a.d0 > 0 ? 1 : -1) : (a.d1 > 0) - (a.d1 < 0);
  const int sb = b.d0 ? (b.d0 > 0 ? 1 : -1) : (b.d1 > 0) - (b.d1 < 0);
  const int mn = max(max(bits128(a.n0), bits128(a.n1)), max(bits128(b.n0), bits128(b.n1)));
  const int md = max(max(bits128(a.d0), bits128(a.d1)), max(bits128(b.d0), bits128(b.d1)));
  if (sa && sb && mn + md <= 124) {
    i128 p = a.n0 * b.d0 - b.n0 * a.d0;
    if (!p) {
      p = a.n0 * b.d1 + a.n1 * b.d0 - b.n0 * a.d1 - b.n1 * a.d0;
      if (!p) p = a.n1 * b.d1 - b.n1 * a.d1;
    }
    return p ? (p > 0 ? 1 : -1) * sa * sb : 0;
  }
  return kLeadOpen;
}

__device__ __forceinline__ int tri_cmp_mid_body(const WPt* pts, Tri A, Tri B, int zs) {
  const int s = lead_cmp(lead_of(pts[A.a], pts[A.w], pts[A.b], zs),
                         lead_of(pts[B.a], pts[B.w], pts[B.b], zs));
  return s == 1 || s == -1 ? s : tri_cmp_exact(pts, A, B, zs, s);
}

// Order of two events that the filter on stored times cannot tell apart:
// 0 for the same triple, else the standard parts once more in double (a stored
// time is a float), then the mid tier.  A call: kernels with many live
// registers.
template <class PT>
__device__ __noinline__ int tri_cmp_near(const PT* pts, Tri A, Tri B, int zs) {
  if (A.a == B.a && A.w == B.w && A.b == B.b) return 0;
  const int s = std_cmp_fine(tau_std(pts[A.a], pts[A.w], pts[A.b], zs),
                             tau_std(pts[B.a], pts[B.w], pts[B.b], zs));
  return s ? s : tri_cmp_mid_body(pts, A, B, zs);
}

// Order of two events: the standard-part filter, then (rare) tri_cmp_near, or
// with kInlineMid the mid tier inline (the lane-serial merge, where exact
// standard-part ties are frequent and a call costs more than the registers).
template <bool kInlineMid = false, class PT>
__device__ __forceinline__ int ev_cmp(const PT* pts, const Cand& A, const Cand& B, int zs) {
  const int s = std_cmp(A.st, B.st);
  if (s) return s;
  if (!kInlineMid) return tri_cmp_near(pts, A.t, B.t, zs);
  if (A.t.a == B.t.a && A.t.w == B.t.w && A.t.b == B.t.b) return 0;
  return tri_cmp_mid_body(pts, A.t, B.t, zs);
}

// The same for a candidate A whose points the caller holds (a0, a1, a2) against
// an event B: a tie loads only B's points.
template <class PT>
__device__ __forceinline__ int ev_cmp_half(const PT* pts, const Cand& A, const PT& a0, const PT& a1,
                                           const PT& a2, const Cand& B, int zs) {
  const int s = std_cmp(A.st, B.st);
  if (s) return s;
  if (A.t.a == B.t.a && A.t.w == B.t.w && A.t.b == B.t.b) return 0;
  const int m = lead_cmp(lead_of(a0, a1, a2, zs), lead_of(pts[B.t.a], pts[B.t.w], pts[B.t.b], zs));
  return m == 1 || m == -1 ? m : tri_cmp_exact(pts, A.t, B.t, zs, m);
}

// Perturbed sign of D when D0 = D1 = 0 (cold path).
template <class PT>
__device__ __noinline__ int d_sign_slow(PT P, PT Q, PT R) {
  Coef c;
  coef_of(P, Q, R, 1, c);
  return c.dsign;
}

// Perturbed sign of D(a, b, c) (xy orientation).
template <class PT>
__device__ __forceinline__ int d_sign(const PT& P, const PT& Q, const PT& R) {
  const Dif q = dif_of(P, Q), r = dif_of(P, R);
  const double D0 = det2(q.x, r.y, r.x, q.y);
  if (D0 != 0) return D0 > 0 ? 1 : -1;
  const double D1 = det2((double)(Q.w - P.w), r.y, (double)(R.w - P.w), q.y);
  if (D1 != 0) return D1 > 0 ? 1 : -1;
  return d_sign_slow<PT>(P, Q, R);
}

template <class PT>
__device__ __forceinline__ Cand make_cand(const PT* pts, int a, int w, int b, const PT& A,
                                          const PT& W, const PT& B, int kind, int zs) {
  Cand c;
  c.t = Tri{a, w, b};
  c.kind = kind;
  c.st = tau_std(A, W, B, zs);
  return c;
}

// Largest i in [0, count) with off[i] <= x (off non-decreasing, off[0] <= x).
__device__ __forceinline__ int find_owner(const int* off, int count, int64_t x) {
  int lo = 0, hi = count;
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (off[mid] <= x) lo = mid;
    else hi = mid;
  }
  return lo;
}

// Workspace of one run for the parallel strategy (merge_par.hip).
struct ParRun {
  int* off;       // [2n + 1] bounds of the link-change lists: next links of point p at 2p,
                  // prev links at 2p + 1
  int2* ent;      // list entries: (position in the child movie, the link after it)
  int4* pos;      // per child event: its places in the lists of a, b, w, w
  int* cmerge;    // per child event: its merge
  int* ctr;       // [kCtrSlots]: level totals
  int* ecnt;      // per merge: child events (mcap + 1)
  int* eoff;      // exclusive scan of ecnt
  int* segS;      // per merge: # time segments of its walk
  int* segBase;   // exclusive scan of segS
  int* segMerge;  // per segment: its merge
  int* segJ;      // per segment: left events before it
  int* segCnt;    // per segment: # events it puts out
  int* segOff;    // exclusive scan of segCnt
  int2* segUV;    // per segment: the bridge at its start
  unsigned long long* segSteps;  // per segment: outcomes of its steps (kStepsLost: not kept)
  Event* segKeep;                // per segment: its first kSegKeep bridge events
  int2* uv0;      // per merge: the bridge at -inf
};

constexpr int kRangesFromLevel = 7;  // lists by ranges of points: from this level on
struct ParLevel {
  RunPtrs run[2];
  ParRun par[2];
  Header* h;
  Sched S;
  int64_t n;        // bound on the points
  int sel;
  bool device_n;    // n is a bound, the device knows the number
  int bin_log;      // log of the bins' points (0: no lists by bins)
  int ranges;       // ranges of points per merge (lists built in LDS)
  int seg_events;   // child events per walk segment
  int64_t seg_cap;  // bound on the walk segments of a level
  int64_t mcap;     // bound on the merges of a level
  unsigned long long* chain_words;  // status words of the level's one-launch scans
  int64_t chain_stride;             // (kChainJobs slots), zeroed once per call
};

template <class PT>
int32_t parallel_level(const ParLevel& P, hipStream_t s);

}  // namespace hull
