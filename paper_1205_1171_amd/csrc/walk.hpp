// One time segment of a merge (the merge step of Sec. 2), for the strategies
// that cut a merge's time axis into segments walked in parallel.
//
// The child events of a merge, both movies together in time order, are cut
// into S segments of about the same number (segment_split: positions jL of
// the left movie and jR of the right one at each cut, by a co-rank search).
// A segment's walk is the lane-serial merge loop over its own child events,
// with two differences:
//   - it starts from the bridge just after the last event before it, found by
//     walking to the lower common tangent of the two chains at that time;
//   - the chains' links are not replayed.  The links of u and v follow the
//     child events the walk itself passes, and the links of a point the
//     bridge moves to come from the point's list of link-changing events: the
//     cursors say which of them have happened, so the lists are searched by
//     integer positions and never by time.
// Every child event is met in time order with the bridge of its time at hand,
// so its survival costs one comparison, and the segment's output is already
// in the merged movie's order: a segment needs only the number of events the
// segments before it put out.
//
// A context CX names the merge's data: its points (pts, by the rank the walk
// uses), its child events in time order (ev(left, i)), the links of a point
// after the first `cursor` events of its child movie (link(p, next, left,
// cursor): its next or previous link; links(...): both), and zs.
//
// The loops are written as straight-line code with selects.  A wavefront runs
// the union of its lanes' branches anyway, and a step is a chain of dependent
// LDS reads and double operations: branch by branch its four candidates cost
// four such chains (8,000 cycles a step on the 60,001-point sphere), computed
// together they overlap.  Only what is rare branches: exact comparisons when
// the filter cannot decide, and D0 = 0.
#pragma once
#include "common.hpp"
#include "events.hpp"

namespace hull {

// A child event in the walk's ranks.
struct WalkEv {
  int a, w, b, kind;
  double t;
};

__device__ __forceinline__ Cand walk_cand(const WalkEv& e) {
  Cand c;
  c.t = Tri{e.a, e.w, e.b};
  c.kind = e.kind;
  c.st = e.t;
  return c;
}

// Links of p after an event that changes them.
__device__ __forceinline__ int next_after(int a, int w, int b, int kind, int p) {
  return p == a && kind ? w : b;
}
__device__ __forceinline__ int prev_after(int a, int w, int b, int kind, int p) {
  return p == b && kind ? w : a;
}

__device__ __forceinline__ int segments_for(int n, int G) { return 1 + n / G; }

// # of left-movie events among the first k = floor(i N / S) child events of
// the merge in time order: the first j at which L[j] comes after R[k-1-j].
template <class PT, class CX>
__device__ __forceinline__ int segment_split(const CX& X, int nL, int nR, int i, int S) {
  const int k = (int)((int64_t)i * (nL + nR) / S);
  int lo = k - nR > 0 ? k - nR : 0, hi = k < nL ? k : nL;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (ev_cmp(X.pts, walk_cand(X.ev(true, mid)), walk_cand(X.ev(false, k - 1 - mid)), X.zs) < 0)
      lo = mid + 1;
    else
      hi = mid;
  }
  return lo;
}

// What a counting walk notes for the writing pass: the outcome of every step
// (3 bits each) and how many bridge events it put aside, so that a segment of
// few steps is written without walking it again.
constexpr int kWalkSteps = 21;
enum { kStepL = 1, kStepR = 2, kStepHideL = 3, kStepHideR = 4, kStepBridge = 5 };
struct WalkNote {
  unsigned long long steps = 0;
  int nsteps = 0, nbridge = 0, nout = 0;
  __device__ __forceinline__ void step(unsigned code, bool out) {
    if (nsteps < kWalkSteps) steps |= (unsigned long long)code << (3 * nsteps);
    ++nsteps;
    nout += out;
  }
  __device__ __forceinline__ void child(bool left, bool kept) {
    step(kept ? (left ? kStepL : kStepR) : (left ? kStepHideL : kStepHideR), kept);
  }
};

template <class PT>
__device__ __noinline__ double tau_std_call(const PT* pts, Tri t, double n, int zs) {
  return tau_std_flat(pts[t.a], pts[t.w], pts[t.b], n, zs);
}

// Orientation of the rank-ordered triple (a, b, c) just after the event T,
// exactly: before the triple's own event sign(D), after it the opposite.
template <class PT>
__device__ __noinline__ int orient_exact(const PT* pts, int a, int b, int c, Tri t, double st, int zs) {
  Cand T;
  T.t = t;
  T.st = st;
  T.kind = 0;
  const PT A = pts[a], B = pts[b], C = pts[c];
  const Cand e = make_cand(pts, a, b, c, A, B, C, 0, zs);
  const int ds = d_sign(A, B, C);
  return ev_cmp(pts, e, T, zs) > 0 ? ds : -ds;
}

// The bridge (u, v) just after the event T (haveT; else at t = -inf) with iL
// and iR child events past: from the inner ends of the blocks, one endpoint
// at a time, to the lower common tangent.  The orientation of a triple just
// after T is the sign of f = N - tau_T D (at -inf: of D); with tau_T within
// 2^-24 and N0, D0 within 2^-52 relative, f decides beyond 2^-22 (|N0| +
// |t D0|).  limit bounds the steps (false: not reached, an internal error).
template <class PT, class CX>
__device__ __forceinline__ bool bridge_at(const CX& X, int m, int iL, int iR, bool haveT,
                                          const Cand& T, int limit, int& u, int& v) {
  const PT* pts = X.pts;
  u = m - 1;
  v = m;
  int vn = X.link(v, true, false, iR), up = X.link(u, false, true, iL);
  PT Pu = pts[u], Pv = pts[v], Pn = pts[vn < 0 ? v : vn], Pp = pts[up < 0 ? u : up];
  for (int guard = 0; guard <= limit; ++guard) {
    const Dif q = dif_of(Pu, Pv), r1 = dif_of(Pu, Pn), r2 = dif_of(Pu, Pp);
    const double d1 = det2(q.x, r1.y, r1.x, q.y), d2 = det2(q.x, r2.y, r2.x, q.y);
    double f1 = d1, f2 = d2, tol1 = 0.0, tol2 = 0.0;
    if (haveT) {
      const double n1 = X.zs * det2(q.x, r1.z, r1.x, q.z), n2 = X.zs * det2(q.x, r2.z, r2.x, q.z);
      const double x1 = T.st * d1, x2 = T.st * d2;
      f1 = n1 - x1;
      f2 = n2 - x2;
      tol1 = 0x1p-22 * (fabs(n1) + fabs(x1));
      tol2 = 0x1p-22 * (fabs(n2) + fabs(x2));
    }
    bool mv = vn >= 0 && f1 < 0, mu = up >= 0 && f2 < 0;
    const bool amb1 = vn >= 0 && !(fabs(f1) > tol1);  // true for NaN
    if (amb1)
      mv = (haveT ? orient_exact<PT>(pts, u, v, vn, T.t, T.st, X.zs) : d_sign_slow<PT>(Pu, Pv, Pn)) < 0;
    const bool amb2 = !mv && up >= 0 && !(fabs(f2) > tol2);
    if (amb2)
      mu = (haveT ? orient_exact<PT>(pts, up, u, v, T.t, T.st, X.zs) : d_sign_slow<PT>(Pp, Pu, Pv)) < 0;
    if (!mv && !mu) return true;
    // v moves to vn, else u to up
    const int p = mv ? vn : up;
    const int l = X.link(p, mv, !mv, mv ? iR : iL);
    const PT Pl = pts[l < 0 ? p : l];
    if (mv) {
      v = vn;
      vn = l;
      Pv = Pn;
      Pn = Pl;
    } else {
      u = up;
      up = l;
      Pu = Pp;
      Pp = Pl;
    }
  }
  return false;
}

// The walk of one segment from the bridge (u, v): left events [i, iE), right
// events [j, jE), and the bridge moves among them (after them too in the
// `last` segment).  out.child(left, kept, event) is called for every child
// event and out.bridge(a, w, b, kind, st) for every bridge move, in time
// order.  False: more than `limit` steps (an internal error).
template <class PT, class CX, class OUT>
__device__ __forceinline__ bool walk(const CX& X, int u, int v, int i, int iE, int j, int jE,
                                     bool last, bool haveT, Cand T, int limit, OUT& out) {
  const PT* pts = X.pts;
  const int zs = X.zs;
  PT Pu = pts[u], Pv = pts[v];
  int nu, pu, nv, pvv;
  X.links(u, true, i, nu, pu);
  X.links(v, false, j, nv, pvv);
  WalkEv EL = X.ev(true, i < iE ? i : 0), ER = X.ev(false, j < jE ? j : 0);
  for (int it = 0; it <= limit; ++it) {
    if (!last && i >= iE && j >= jE) return true;
    // The four bridge moves: nx(u) enters (u, nu, v), u leaves (pu, u, v),
    // pv(v) enters (u, pvv, v), v leaves (u, v, nv).  tau does not depend on the
    // order of its triple, so all four are taken from u.
    const int lk[4] = {nu, pu, pvv, nv};
    Tri tr[4] = {Tri{u, nu, v}, Tri{pu, u, v}, Tri{u, pvv, v}, Tri{u, v, nv}};
    double st[4], dd[4], nn[4];
    bool ok[4];
    const Dif q = dif_of(Pu, Pv);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const Dif r = dif_of(Pu, pts[lk[k] < 0 ? u : lk[k]]);
      dd[k] = det2(q.x, r.y, r.x, q.y);
      nn[k] = zs * det2(q.x, r.z, r.x, q.z);
      st[k] = quotient(nn[k], dd[k]);
    }
    // What needs a call is gathered first: a wavefront then calls as often as its
    // lane with the most, not once for each of the four.  Points on lattices, where
    // ties are everywhere: 300 points of 60^3 911 -> 897 us, flat 30,000 the same,
    // duplicates 19.5 -> 18.1 ms; 2^20 sphere 7.64 -> 7.60 (four registers fewer).
    const auto move = [&](int k) {
      return Tri{k == 1 ? pu : u, k == 0 ? nu : (k == 1 ? u : (k == 2 ? pvv : v)), k == 3 ? nv : v};
    };
    unsigned flat = 0, amb = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      ok[k] = lk[k] >= 0;
      flat |= (unsigned)(ok[k] && dd[k] == 0) << k;
    }
    for (; flat; flat &= flat - 1) {
      const int f = __builtin_ctz(flat);
      const double x = tau_std_call(pts, move(f), f == 0 ? nn[0] : (f == 1 ? nn[1] : (f == 2 ? nn[2] : nn[3])), zs);
#pragma unroll
      for (int k = 0; k < 4; ++k) st[k] = f == k ? x : st[k];
    }
    if (haveT) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const int c = std_cmp(st[k], T.st);
        const bool same = T.t.a == tr[k].a && T.t.w == tr[k].w && T.t.b == tr[k].b;
        amb |= (unsigned)(ok[k] && c == 0 && !same) << k;
        ok[k] = ok[k] && c > 0;
      }
      for (; amb; amb &= amb - 1) {
        const int f = __builtin_ctz(amb);
        const bool after = tri_cmp_near(pts, move(f), T.t, zs) > 0;
#pragma unroll
        for (int k = 0; k < 4; ++k) ok[k] = f == k ? after : ok[k];
      }
    }
    // the earliest valid one
    int bi = ok[0] ? 0 : -1;
    Cand B;
    B.t = tr[0];
    B.st = st[0];
    B.kind = 1;
#pragma unroll
    for (int k = 1; k < 4; ++k) {
      const int c = std_cmp(st[k], B.st);
      bool take = ok[k] && (bi < 0 || c < 0);
      if (ok[k] && bi >= 0 && c == 0) take = tri_cmp_near(pts, tr[k], B.t, zs) < 0;
      bi = take ? k : bi;
      B.t.a = take ? tr[k].a : B.t.a;
      B.t.w = take ? tr[k].w : B.t.w;
      B.t.b = take ? tr[k].b : B.t.b;
      B.st = take ? st[k] : B.st;
    }
    // the child events before it, up to one that changes a link of u or v
    bool dirty = false;
    while (i < iE || j < jE) {
      int c = std_cmp(EL.t, ER.t);
      if (i < iE && j < jE && c == 0)
        c = tri_cmp_near(pts, Tri{EL.a, EL.w, EL.b}, Tri{ER.a, ER.w, ER.b}, zs);
      const bool left = i < iE && (j >= jE || c < 0);
      const WalkEv E = left ? EL : ER;
      const Tri t = Tri{E.a, E.w, E.b};
      if (bi >= 0) {
        int o = std_cmp(E.t, B.st);
        if (o == 0) o = tri_cmp_near(pts, t, B.t, zs);
        if (o > 0) break;
      }
      T.t = t;
      T.st = E.t;
      haveT = true;
      out.child(left, left ? E.w < u : E.w > v, E.a, E.w, E.b, E.kind, E.t);
      i += left;
      j += !left;
      const WalkEv Z = X.ev(left, left ? (i < iE ? i : 0) : (j < jE ? j : 0));
      if (left) EL = Z;
      else ER = Z;
      // it sets next(a) and prev(b) (w is never u or v when inserted)
      const int na = E.kind ? E.w : E.b, pb = E.kind ? E.w : E.a;
      dirty = E.a == u || E.b == u || E.a == v || E.b == v;
      nu = E.a == u ? na : nu;
      pu = E.b == u ? pb : pu;
      nv = E.a == v ? na : nv;
      pvv = E.b == v ? pb : pvv;
      if (dirty) break;
    }
    if (dirty) continue;
    if (bi < 0 || (!last && i >= iE && j >= jE)) return true;
    T = B;
    haveT = true;
    out.bridge(B.t.a, B.t.w, B.t.b, bi == 0 || bi == 2, B.st);
    const bool left = bi <= 1;
    const int p = bi == 0 ? nu : (bi == 1 ? pu : (bi == 2 ? pvv : nv));
    const PT Pp = pts[p];
    int nx, pv;
    X.links(p, left, left ? i : j, nx, pv);
    if (left) {
      u = p;
      Pu = Pp;
      nu = nx;
      pu = pv;
    } else {
      v = p;
      Pv = Pp;
      nv = nx;
      pvv = pv;
    }
  }
  return false;
}

}  // namespace hull
