// gdp_cdt_dev.hip -- Line 1 of Algorithm 1 on the GPU: the constrained
// Delaunay triangulation of the input PSLG built by kernels, so that a mesh
// can go from its PSLG to the refinement loop without the host builder.
//
// The result is the same triangulation as the host builder's, element for
// element: the CDT is unique once cocircular ties are broken by the symbolic
// perturbation of the lifting map with the smaller vertex id dominant, and
// the canonical form (each triangle rotated so its smallest vertex comes
// first, triangles sorted) fixes the slot order.
//
// Stages, all on one stream:
//   1. Delaunay triangulation of the points and a large enclosing triangle by
//      rounds of insertion and flips.  The points are renumbered along a
//      Morton curve (the ids decide ties and the final order only), so that
//      neighbouring lanes work on neighbouring triangles.  Each pending point
//      walks to the triangle holding it; each triangle takes one point
//      (largest key), splits 1-3 (2-4 for a point on an edge, which needs
//      both triangles), and edges that are not locally Delaunay are flipped
//      in passes until none is left.  Every triangle that holds points is
//      split in every round, so the points of each triangle fall to a third
//      per round.  An evenly spread sample of the points goes first, in one
//      workgroup.
//   2. Segment recovery by rounds: a segment whose edge is missing walks the
//      triangles it crosses and stamps them and their outer neighbours; a
//      segment that keeps every stamp replaces the crossed triangles by the
//      constrained Delaunay triangulations of the two pseudo-polygons on its
//      sides (recursive choice of the apex whose circle holds no other
//      polygon vertex).  Crossed regions of different winners are disjoint,
//      so the result is the one sequential insertion gives.
//   3. Triangles with an enclosing vertex are dropped; every dropped/kept
//      boundary must be a segment, every vertex used, the kept region a
//      convex disk; the survivors are rotated, sorted by (v0, v1) with a
//      radix sort of this file and renumbered into the refinement's mesh
//      layout.
#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>
#include <vector>

#include "gdp_internal.h"

namespace gdp {
namespace {

constexpr int kBlk = 256;        // block of the plain kernels
constexpr int kWalkCap = 1 << 20;   // steps of one walk or rotation
constexpr int kSeedMax = 4096;      // points of the sample
constexpr uint64_t kPassMax = 1ull << 23;  // flip passes of a build (24 bits of a claim)
constexpr int kPassBatch = 6;       // flip passes between two host reads (even: the worklist ends where it began)

enum CdtErr : int {
  kEOk = 0, kEDup, kEWalk, kERepeat, kEOnSeg, kECross, kELeave, kEDir, kEHull, kEUnused,
  kEDisk, kEInternal = 100  // + the site that found an inconsistency
};

const char *cdt_err_text(int e) {
  switch (e) {
    case kEDup: return "duplicate point";
    case kEWalk: return "point location failed";
    case kERepeat: return "repeated segment";
    case kEOnSeg: return "a vertex lies in the interior of a segment";
    case kECross: return "segments cross";
    case kELeave: return "segment leaves the domain";
    case kEDir: return "segment direction not found";
    case kEHull: return "a convex hull edge is not covered by a segment";
    case kEUnused: return "a convex hull edge is not covered by a segment";
    case kEDisk: return "the kept region is not a disk";
    default: return "device CDT builder: internal error";
  }
}

std::string cdt_err_string(int e) {
  if (e >= kEInternal) return "device CDT builder: internal error at site " + std::to_string(e - kEInternal);
  return cdt_err_text(e);
}

// Round counters, read back after each round.
struct Ctr {
  int npend;   // entries appended to the next pending list
  int nwin;    // insertions this round
  int pool;    // ints of the per-round pool taken
  int err;     // first error code
  int nkeep;   // kept triangles (final stage)
  int nhull;   // boundary edges of the kept region
  int ntri;    // triangles so far
  int nlist[2];  // flip worklists (one read, one built per pass)
  int ncand[2];  // flip candidates (by the parity of the pass)
  int first_stamp, first_pass;  // after the sample: the last stamp and pass used
};

struct Bld {
  const double2 *P;    // nv + 3 points along the Morton curve, then the enclosing triangle
  const int *id;       // their ids (nv .. nv + 2: the enclosing triangle)
  int nv;
  int4 *tv, *tn, *ts;  // triangle slots: vertices, neighbours, segment id per edge (-1 none)
  int capT;
  uint64_t *pick;      // per slot: key of the point that splits it, then of the segment that crosses it (round << 32 | key)
  uint64_t *mark;      // per slot: claim of a flip (pass << 40 | edge), then stamp of a segment (round << 32 | key)
  int *loc, *state;    // per point: 4 * (last triangle) + edge it lies on (3: inside); per segment: start triangle
  int *vt;             // per vertex: an incident triangle
  // flips
  int4 *grp;           // slots that replaced a split triangle (shares fc0's memory: no flips then)
  int *sstamp;         // round in which the slot was split
  int *wstamp;         // pass stamp: on the worklist
  int *list[2];
  int4 *fc0, *fc1;     // candidates: (t, e, o, j) and the four outer slots
  uint64_t *fprio;
  int *pool;           // per-round scratch of the segment recovery
  int pool_cap;
  Ctr *c;
};

__device__ __forceinline__ void set_err(Ctr *c, int e) { atomicCAS(&c->err, 0, e); }

__device__ __forceinline__ int comp(const int4 &v, int i) { return i == 0 ? v.x : (i == 1 ? v.y : v.z); }
__device__ __forceinline__ int *comp_ptr(int4 *a, int t, int i) { return reinterpret_cast<int *>(a + t) + i; }

// A fixed bijection of 32-bit ids (MurmurHash3 finalizer of id + 1) makes
// the election keys distinct and spread.
__device__ __forceinline__ uint32_t mix32(uint32_t x) {
  uint32_t h = x + 1u;
  h ^= h >> 16;
  h *= 0x85ebca6bu;
  h ^= h >> 13;
  h *= 0xc2b2ae35u;
  h ^= h >> 16;
  return h;
}

__device__ __forceinline__ int orient_ids(const double2 *P, int a, int b, int c) {
  const double2 A = P[a], B = P[b], C = P[c];
  return orient2d(A.x, A.y, B.x, B.y, C.x, C.y);
}

// incircle with the symbolic perturbation of the lifting map (gdp_exact.h)
// by the ids of the points; equal ids (a chain vertex repeated around a
// slit) keep their argument order.
__device__ __forceinline__ int incircle_sos(const Bld &bl, int a, int b, int c, int d) {
  const double2 A = bl.P[a], B = bl.P[b], C = bl.P[c], D = bl.P[d];
  const int f = incircle_filter(A.x, A.y, B.x, B.y, C.x, C.y, D.x, D.y);
  if (f != kUndecided) return f;
  return gdp::incircle_sos(A.x, A.y, B.x, B.y, C.x, C.y, D.x, D.y, bl.id[a], bl.id[b], bl.id[c], bl.id[d]);
}

__device__ __forceinline__ int eidx(const int4 &v, int u, int w) {
  if (v.x == u && v.y == w) return 0;
  if (v.y == u && v.z == w) return 1;
  if (v.z == u && v.x == w) return 2;
  return -1;
}

__device__ __forceinline__ int vidx(const int4 &v, int a) { return v.x == a ? 0 : (v.y == a ? 1 : (v.z == a ? 2 : -1)); }

// Variable-size allocation by a whole wave: one atomic per wave.
__device__ __forceinline__ int wave_take(int *counter, int n) {
  const int lane = __lane_id();
  int x = n;
  for (int d = 1; d < 64; d <<= 1) {
    int y = __shfl_up(x, d);
    if (lane >= d) x += y;
  }
  const int total = __shfl(x, 63);
  int base = 0;
  if (lane == 63 && total > 0) base = atomicAdd(counter, total);
  base = __shfl(base, 63);
  return base + x - n;
}

// The same by a whole workgroup of kBlk threads: one atomic per workgroup.
// Atomics on one address are served about 12 ns apart, so with one per wave a
// pass over a million elements would wait 190 us for each counter.
__device__ __forceinline__ int block_take(int *counter, int n) {
  __shared__ int s_part[kBlk / 64], s_base;
  const int lane = __lane_id(), wid = threadIdx.x >> 6;
  int x = n;
  for (int d = 1; d < 64; d <<= 1) {
    const int y = __shfl_up(x, d);
    if (lane >= d) x += y;
  }
  if (lane == 63) s_part[wid] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    int acc = 0;
    for (int i = 0; i < kBlk / 64; i++) {
      const int t = s_part[i];
      s_part[i] = acc;
      acc += t;
    }
    s_base = acc ? atomicAdd(counter, acc) : 0;
  }
  __syncthreads();
  x += s_base + s_part[wid] - n;
  __syncthreads();
  return x;
}
// Space from a counter in memory (BLOCK: by every thread of the workgroup) or
// in LDS (by every lane of the wave).
template <bool BLOCK>
__device__ __forceinline__ int take(int *counter, int n) {
  return BLOCK ? block_take(counter, n) : wave_take(counter, n);
}

// ---------------------------------------------------------------------------
// Stage 1: Delaunay triangulation by insertion rounds and flip passes
// ---------------------------------------------------------------------------
// Bounding box of the points, each block's extremes by atomics on the
// monotone integer image of a double.
__device__ __forceinline__ unsigned long long ord_of(double x) {
  const unsigned long long b = (unsigned long long)__double_as_longlong(x);
  return (b >> 63) ? ~b : (b | (1ull << 63));
}
double ord_to(unsigned long long o) {
  const unsigned long long b = (o >> 63) ? (o & ~(1ull << 63)) : ~o;
  double x;
  memcpy(&x, &b, sizeof x);
  return x;
}
// box: max of x, y and of -x, -y (all zero bits at first: below every double)
__global__ __launch_bounds__(kBlk) void k_box(const double2 *xy, int nv, unsigned long long *box) {
  unsigned long long m[4] = {0, 0, 0, 0};
  const int stride = gridDim.x * blockDim.x;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nv; i += stride) {
    const double2 p = xy[i];
    m[0] = max(m[0], ord_of(p.x));
    m[1] = max(m[1], ord_of(p.y));
    m[2] = max(m[2], ord_of(-p.x));
    m[3] = max(m[3], ord_of(-p.y));
  }
  for (int k = 0; k < 4; k++) {
    for (int d = 32; d >= 1; d >>= 1) {
      const unsigned long long o = (unsigned long long)__shfl_xor((long long)m[k], d);
      m[k] = max(m[k], o);
    }
    if (__lane_id() == 0) atomicMax(&box[k], m[k]);
  }
}

// 16-bit cells of the box per axis, interleaved.
__device__ __forceinline__ uint32_t morton_of(double2 p, double x0, double y0, double sc) {
  uint32_t c[2] = {(uint32_t)min(max((p.x - x0) * sc, 0.0), 65535.0), (uint32_t)min(max((p.y - y0) * sc, 0.0), 65535.0)};
  for (int k = 0; k < 2; k++) {
    uint32_t x = c[k];
    x = (x | (x << 8)) & 0x00ff00ffu;
    x = (x | (x << 4)) & 0x0f0f0f0fu;
    x = (x | (x << 2)) & 0x33333333u;
    x = (x | (x << 1)) & 0x55555555u;
    c[k] = x;
  }
  return c[0] | (c[1] << 1);
}
__global__ __launch_bounds__(kBlk) void k_morton(const double2 *xy, int nv, double x0, double y0, double sc,
                                                 uint64_t *keys, int *vals) {
  const int stride = gridDim.x * blockDim.x;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nv; i += stride) {
    keys[i] = morton_of(xy[i], x0, y0, sc);
    vals[i] = i;
  }
}

__device__ __forceinline__ void first_triangle(const Bld &b, double2 *P, int *id, double L) {
  P[b.nv] = make_double2(-4 * L, -4 * L);
  P[b.nv + 1] = make_double2(8 * L, -4 * L);
  P[b.nv + 2] = make_double2(-4 * L, 8 * L);
  for (int k = 0; k < 3; k++) id[b.nv + k] = b.nv + k;
  b.tv[0] = make_int4(b.nv, b.nv + 1, b.nv + 2, 0);
  b.tn[0] = make_int4(-1, -1, -1, 0);
}

// The points along the curve, their ids, the inverse permutation and the
// first triangle.
__global__ __launch_bounds__(kBlk) void k_reorder(Bld b, const double2 *xy, double2 *P, const int *vals, int *id,
                                                  int *rank, double L) {
  const int stride = gridDim.x * blockDim.x;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < b.nv; i += stride) {
    const int v = vals[i];
    P[i] = xy[v];
    id[i] = v;
    rank[v] = i;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    first_triangle(b, P, id, L);
    b.c->ntri = 1;
  }
}

__device__ __forceinline__ uint64_t point_key(int p, uint32_t round) { return ((uint64_t)round << 32) | mix32((uint32_t)p); }

// Walks point p (act) from its last triangle to the one holding it and
// claims that (and the one across the edge it lies on) for the round's
// split.  All lanes of the wave take part: lanes that share a triangle
// combine their keys before the atomic while such groups are large.
__device__ __forceinline__ void dt_locate(const Bld &b, int p, bool act, uint32_t round) {
  const int lane = __lane_id();
  int t = 0, e = 3, o = -1;
  uint64_t key = 0;
  if (act) {
    t = b.loc[p] >> 2;
    key = point_key(p, round);
    int from = -1;
    const double2 q = b.P[p];
    for (int steps = 0;; steps++) {
      const int4 v = b.tv[t], n = b.tn[t];
      const double2 A = b.P[v.x], B = b.P[v.y], C = b.P[v.z];
      const int s0 = orient2d(A.x, A.y, B.x, B.y, q.x, q.y), s1 = orient2d(B.x, B.y, C.x, C.y, q.x, q.y),
                s2 = orient2d(C.x, C.y, A.x, A.y, q.x, q.y);
      const int m = (s0 < 0 && n.x != from) ? 0 : ((s1 < 0 && n.y != from) ? 1 : ((s2 < 0 && n.z != from) ? 2 : -1));
      if (m < 0) {
        if ((s0 == 0) + (s1 == 0) + (s2 == 0) >= 2) {
          set_err(b.c, kEDup);  // on a vertex
          act = false;
        }
        e = s0 == 0 ? 0 : (s1 == 0 ? 1 : (s2 == 0 ? 2 : 3));
        o = e < 3 ? comp(n, e) : -1;
        break;
      }
      const int nx = comp(n, m);
      if (nx < 0 || steps > kWalkCap) {
        set_err(b.c, kEWalk);
        act = false;
        break;
      }
      from = t;
      t = nx;
    }
    b.loc[p] = 4 * t + e;
  }
  if (act && o >= 0) atomicMax((unsigned long long *)&b.pick[o], (unsigned long long)key);
  uint64_t left = __ballot(act);
  for (int it = 0; it < 64 && left; it++) {
    const int leader = __ffsll((unsigned long long)left) - 1;
    const int tl = __shfl(t, leader);
    const bool same = act && t == tl;
    const uint64_t m = __ballot(same);
    if (it > 0 && __popcll(m) < 3) break;
    long long best = same ? (long long)key : 0;
    for (int d = 32; d >= 1; d >>= 1) {
      long long x = __shfl_xor(best, d);
      best = (unsigned long long)x > (unsigned long long)best ? x : best;
    }
    if (lane == leader) atomicMax((unsigned long long *)&b.pick[tl], (unsigned long long)best);
    if (same) act = false;
    left &= ~m;
  }
  if (act) atomicMax((unsigned long long *)&b.pick[t], (unsigned long long)key);
}

// Splits the triangle(s) of point p if it holds them; returns whether it did.
// A new triangle is (x, y, p): edge 0 is the outer one, which still names the
// old neighbour (dt_fix follows).  The new triangles go to the worklist.
template <bool BLOCK>
__device__ __forceinline__ bool dt_split(const Bld &b, int p, bool act, uint32_t round, int wst, int *ntri, int *nlist) {
  int t0 = 0, e0 = 3, t1 = -1;
  bool own = false;
  if (act) {
    const uint64_t key = point_key(p, round);
    t0 = b.loc[p] >> 2;
    e0 = b.loc[p] & 3;
    own = b.pick[t0] == key;
    if (own && e0 < 3) {
      t1 = comp(b.tn[t0], e0);
      own = t1 >= 0 && b.pick[t1] == key;
    }
  }
  const int base = take<BLOCK>(ntri, own ? 2 : 0);
  const int lb = take<BLOCK>(nlist, own ? (e0 < 3 ? 4 : 3) : 0);
  if (!own) return false;
  if (base + 2 > b.capT) {  // not reached: 2 nv + 1 triangles in the end
    set_err(b.c, kEInternal + 1);
    for (int i = 0; i < (e0 < 3 ? 4 : 3); i++) b.list[0][lb + i] = t0;
    return false;
  }
  const int4 v = b.tv[t0], n = b.tn[t0];
  int slot[4], x[4], out[4], k = 3;
  if (e0 == 3) {
    slot[0] = t0; slot[1] = base; slot[2] = base + 1; slot[3] = -1;
    x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = -1;
    out[0] = n.x; out[1] = n.y; out[2] = n.z; out[3] = -1;
    b.grp[t0] = make_int4(t0, base, base + 1, -1);
  } else {
    // edge (u, v) of t0 = (u, v, w) and t1 = (v, u, x): around p the quad u, x, v, w
    const int4 v1 = b.tv[t1], n1 = b.tn[t1];
    const int u = comp(v, e0), vv = comp(v, (e0 + 1) % 3), w = comp(v, (e0 + 2) % 3);
    const int e1 = v1.x == vv ? 0 : (v1.y == vv ? 1 : 2);
    k = 4;
    slot[0] = t1; slot[1] = base; slot[2] = t0; slot[3] = base + 1;
    x[0] = u; x[1] = comp(v1, (e1 + 2) % 3); x[2] = vv; x[3] = w;
    out[0] = comp(n1, (e1 + 1) % 3); out[1] = comp(n1, (e1 + 2) % 3);
    out[2] = comp(n, (e0 + 1) % 3); out[3] = comp(n, (e0 + 2) % 3);
    const int4 g = make_int4(slot[0], slot[1], slot[2], slot[3]);
    b.grp[t0] = g;
    b.grp[t1] = g;
    b.sstamp[t1] = (int)round;
  }
  b.sstamp[t0] = (int)round;
#pragma unroll
  for (int i = 0; i < 4; i++) {
    if (i >= k) continue;
    const bool last = i == k - 1;
    const int s = slot[i];
    b.tv[s] = make_int4(x[i], last ? x[0] : x[(i + 1) & 3], p, 0);
    b.tn[s] = make_int4(out[i], last ? slot[0] : slot[(i + 1) & 3], i == 0 ? slot[k - 1] : slot[(i + 3) & 3], 0);
    b.wstamp[s] = wst;
    b.list[0][lb + i] = s;
  }
  return true;
}

// The outer edge of a new triangle: the neighbour it names was split too (the
// edge is the outer edge of one of its replacements) or has its pointer set.
__device__ __forceinline__ void dt_fix(const Bld &b, int s, uint32_t round) {
  const int o = b.tn[s].x;
  if (o < 0) return;
  const int4 v = b.tv[s];
  if (b.sstamp[o] == (int)round) {
    const int4 g = b.grp[o];
    const int c[4] = {g.x, g.y, g.z, g.w};
    int found = -1;
#pragma unroll
    for (int k = 0; k < 4; k++) {
      if (c[k] < 0) continue;
      const int4 w = b.tv[c[k]];
      if (w.x == v.y && w.y == v.x) found = c[k];
    }
    if (found < 0) set_err(b.c, kEInternal + 2);
    else *comp_ptr(b.tn, s, 0) = found;
  } else {
    const int j = eidx(b.tv[o], v.y, v.x);
    if (j < 0) set_err(b.c, kEInternal + 3);
    else *comp_ptr(b.tn, o, j) = s;
  }
}

// Flip check of one worklist triangle (act): every edge that is not locally
// Delaunay claims its two triangles and the four around them with one 64-bit
// atomicMax of (pass, edge).
template <bool BLOCK>
__device__ __forceinline__ void dt_check(const Bld &b, int t, bool act, int in_stamp, uint64_t pass, int *ncand) {
  int4 a = make_int4(0, 0, 0, 0), na = make_int4(-1, -1, -1, 0);
  int j[3] = {0, 0, 0};
  int flip = 0;  // bits: the edges to flip
  if (act) {
    a = b.tv[t];
    na = b.tn[t];
    // the three neighbours and their far vertices, loaded together
    int d[3];
    int4 v[3];
    int st[3];
#pragma unroll
    for (int e = 0; e < 3; e++) {
      const int o = max(comp(na, e), 0);
      v[e] = b.tv[o];
      st[e] = b.wstamp[o];
    }
    const double2 P[3] = {b.P[a.x], b.P[a.y], b.P[a.z]};
    double2 D[3];
#pragma unroll
    for (int e = 0; e < 3; e++) {
      const int u = comp(a, e);
      // the edge runs the other way in the neighbour: its end u comes second
      j[e] = v[e].y == u ? 0 : (v[e].z == u ? 1 : 2);
      d[e] = j[e] == 0 ? v[e].z : (j[e] == 1 ? v[e].x : v[e].y);
      D[e] = b.P[d[e]];
    }
#pragma unroll
    for (int e = 0; e < 3; e++) {
      const int o = comp(na, e);
      if (o < 0 || (o < t && st[e] == in_stamp)) continue;  // the lower slot on the list checks the edge
      const double2 U = P[e], W = P[e == 2 ? 0 : e + 1], C = P[e == 0 ? 2 : e - 1], Q = D[e];
      int in = incircle_filter(U.x, U.y, W.x, W.y, C.x, C.y, Q.x, Q.y);
      if (in == kUndecided) {
        const int u = comp(a, e), w = comp(a, e == 2 ? 0 : e + 1), c = comp(a, e == 0 ? 2 : e - 1);
        in = gdp::incircle_sos(U.x, U.y, W.x, W.y, C.x, C.y, Q.x, Q.y, b.id[u], b.id[w], b.id[c], b.id[d[e]]);
      }
      if (in > 0) flip |= 1 << e;
    }
  }
  // (a triangle has at most three edges to flip and an edge enters once, so
  // there are at most 3/2 candidates per slot; the lists hold two)
  int idx = take<BLOCK>(ncand, __popc(flip));
#pragma unroll
  for (int e = 0; e < 3; e++) {
    if (!(flip & (1 << e))) continue;
    const int o = comp(na, e), je = j[e];
    const int4 nb = b.tn[o];
    const int4 f1 = make_int4(comp(na, e == 2 ? 0 : e + 1), comp(na, e == 0 ? 2 : e - 1), comp(nb, je == 2 ? 0 : je + 1),
                              comp(nb, je == 0 ? 2 : je - 1));
    const uint64_t prio = (pass << 40) | (uint64_t)(t < o ? 4 * (int64_t)t + e : 4 * (int64_t)o + je);
    b.fc0[idx] = make_int4(t, e, o, je);
    b.fc1[idx] = f1;
    b.fprio[idx] = prio;
    idx++;
    atomicMax((unsigned long long *)&b.mark[t], (unsigned long long)prio);
    atomicMax((unsigned long long *)&b.mark[o], (unsigned long long)prio);
    if (f1.x >= 0) atomicMax((unsigned long long *)&b.mark[f1.x], (unsigned long long)prio);
    if (f1.y >= 0) atomicMax((unsigned long long *)&b.mark[f1.y], (unsigned long long)prio);
    if (f1.z >= 0) atomicMax((unsigned long long *)&b.mark[f1.z], (unsigned long long)prio);
    if (f1.w >= 0) atomicMax((unsigned long long *)&b.mark[f1.w], (unsigned long long)prio);
  }
}

// A candidate (act) whose six claims hold is flipped: it is the only writer of
// the six triangles in the pass.  The triangles of the others are checked
// again.  Each triangle enters the next worklist once.
template <bool BLOCK>
__device__ __forceinline__ void dt_apply(const Bld &b, int i, bool act, int wst, int *out, int *nout) {
  int t = 0, o = 0;
  bool win = false;
  if (act) {
    const int4 f = b.fc0[i], g = b.fc1[i];
    const uint64_t prio = b.fprio[i];
    const int e = f.y, j = f.w;
    t = f.x;
    o = f.z;
    const uint64_t m0 = b.mark[t], m1 = b.mark[o], m2 = b.mark[max(g.x, 0)], m3 = b.mark[max(g.y, 0)],
                   m4 = b.mark[max(g.z, 0)], m5 = b.mark[max(g.w, 0)];
    win = m0 == prio && m1 == prio && (g.x < 0 || m2 == prio) && (g.y < 0 || m3 == prio) &&
          (g.z < 0 || m4 == prio) && (g.w < 0 || m5 == prio);
    if (win) {
      // t = (u, v, w) with edge e = (u, v), o = (v, u, d) with edge j: (u, v)
      // gives way to (d, w): (u, d, w) in t, (d, v, w) in o
      const int4 a = b.tv[t], bv = b.tv[o];
      const int u = comp(a, e), v = comp(a, (e + 1) % 3), w = comp(a, (e + 2) % 3), d = comp(bv, (j + 2) % 3);
      b.tv[t] = make_int4(u, d, w, 0);
      b.tn[t] = make_int4(g.z, o, g.y, 0);
      b.tv[o] = make_int4(d, v, w, 0);
      b.tn[o] = make_int4(g.w, g.x, t, 0);
      if (g.z >= 0) {
        const int q = eidx(b.tv[g.z], d, u);
        if (q < 0) set_err(b.c, kEInternal + 4);
        else *comp_ptr(b.tn, g.z, q) = t;
      }
      if (g.x >= 0) {
        const int q = eidx(b.tv[g.x], w, v);
        if (q < 0) set_err(b.c, kEInternal + 5);
        else *comp_ptr(b.tn, g.x, q) = o;
      }
    }
  }
  const bool pt = act && atomicExch(&b.wstamp[t], wst) != wst;
  const bool po = win && atomicExch(&b.wstamp[o], wst) != wst;
  int at = take<BLOCK>(nout, (pt ? 1 : 0) + (po ? 1 : 0));
  if (pt) out[at++] = t;
  if (po) out[at] = o;
}

__global__ __launch_bounds__(kBlk) void k_dt_locate(Bld b, const int *pend, int np, uint32_t round) {
  const int stride = gridDim.x * blockDim.x;
  for (int base = blockIdx.x * blockDim.x; base < np; base += stride) {
    const int i = base + threadIdx.x;
    dt_locate(b, i < np ? pend[i] : 0, i < np, round);
  }
}

__global__ __launch_bounds__(kBlk) void k_dt_split(Bld b, const int *pend, int np, uint32_t round, int wst, int *pend_out) {
  const int stride = gridDim.x * blockDim.x;
  for (int base = blockIdx.x * blockDim.x; base < np; base += stride) {
    const int i = base + threadIdx.x;
    const int p = i < np ? pend[i] : 0;
    const bool done = dt_split<true>(b, p, i < np, round, wst, &b.c->ntri, &b.c->nlist[0]);
    const int po = block_take(&b.c->npend, i < np && !done ? 1 : 0);
    if (i < np && !done) pend_out[po] = p;
  }
}

__global__ __launch_bounds__(kBlk) void k_dt_fix(Bld b, uint32_t round) {
  const int n = b.c->nlist[0], stride = gridDim.x * blockDim.x;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) dt_fix(b, b.list[0][i], round);
}

// A flip pass is these two launches; worklists and candidate counts
// alternate, each emptied by a launch that does not use it.  Bound by latency:
// a check is three dependent gathers (list, triangle, neighbours and points),
// an apply the same, and most passes hold few entries.  A million points take
// 212 passes of 20 + 11 us; with one atomic per wave and list instead of one per
// workgroup the two kernels took 40 + 31 us.
__global__ __launch_bounds__(kBlk) void k_dt_check(Bld b, int cur, int in_stamp, uint64_t pass) {
  const int n = b.c->nlist[cur], stride = gridDim.x * blockDim.x;
  if (blockIdx.x == 0 && threadIdx.x == 0) b.c->nlist[cur ^ 1] = 0;
  for (int base = blockIdx.x * blockDim.x; base < n; base += stride) {
    const int i = base + threadIdx.x;
    dt_check<true>(b, i < n ? b.list[cur][i] : 0, i < n, in_stamp, pass, &b.c->ncand[pass & 1]);
  }
}
__global__ __launch_bounds__(kBlk) void k_dt_apply(Bld b, int cur, int wst, uint64_t pass) {
  const int n = b.c->ncand[pass & 1], stride = gridDim.x * blockDim.x;
  if (blockIdx.x == 0 && threadIdx.x == 0) b.c->ncand[(pass + 1) & 1] = 0;
  for (int base = blockIdx.x * blockDim.x; base < n; base += stride) {
    const int i = base + threadIdx.x;
    dt_apply<true>(b, i, i < n, wst, b.list[cur ^ 1], &b.c->nlist[cur ^ 1]);
  }
}

// Passes over a short worklist inside one workgroup (two barriers instead of
// two launches each), until it is empty: list s_n[cur] entries in b.list[cur].
// The waves of a workgroup run on one compute unit, so its barrier, a release
// and an acquire at workgroup scope, is enough for a phase's plain loads to see
// what the phases before stored or changed by atomics (here and in all the
// one-workgroup kernels of this file).
struct SeedShared {
  int n[2], ncand;
};
__device__ __forceinline__ void dt_flips(const Bld &b, SeedShared &sh, int &cur, int &stamp, uint64_t &pass) {
  for (;;) {
    __syncthreads();
    const int n = sh.n[cur];
    if (n == 0 || pass > kPassMax) break;
    __syncthreads();
    if (threadIdx.x == 0) {
      sh.n[cur ^ 1] = 0;
      sh.ncand = 0;
    }
    __syncthreads();
    pass++;
    for (int base = 0; base < n; base += blockDim.x) {
      const int i = base + threadIdx.x;
      dt_check<false>(b, i < n ? b.list[cur][i] : 0, i < n, stamp, pass, &sh.ncand);
    }
    __syncthreads();
    const int nc = sh.ncand;
    stamp++;
    for (int base = 0; base < nc; base += blockDim.x) {
      const int i = base + threadIdx.x;
      dt_apply<false>(b, i, i < nc, stamp, b.list[cur ^ 1], &sh.n[cur ^ 1]);
    }
    cur ^= 1;
  }
}

// A grid pass costs two launches, about 10 us; a pass of this over n
// entries about 3 us per 1,024.
constexpr int kTailMax = 2048;
constexpr int kSeedBlk = 1024;
// stamp / pass: the last ones used; the kernel may use as many as it needs
// (the host leaves a gap of kTailGap).
constexpr int kTailGap = 1 << 12;
__global__ __launch_bounds__(kSeedBlk) void k_dt_tail(Bld b, int cur, int stamp, uint64_t pass) {
  __shared__ SeedShared sh;
  const int n0 = b.c->nlist[cur];
  if (n0 == 0 || n0 > kTailMax) return;
  if (threadIdx.x == 0) sh.n[cur] = n0;
  const int cur0 = cur;
  // (bounded by the gap: what is left goes on with the next launch)
  int passes = 0;
  for (; passes < kTailGap; passes++) {
    __syncthreads();
    const int n = sh.n[cur];
    if (n == 0 || (n > kTailMax && cur == cur0)) break;
    __syncthreads();
    if (threadIdx.x == 0) {
      sh.n[cur ^ 1] = 0;
      sh.ncand = 0;
    }
    __syncthreads();
    pass++;
    for (int base = 0; base < n; base += blockDim.x) {
      const int i = base + threadIdx.x;
      dt_check<false>(b, i < n ? b.list[cur][i] : 0, i < n, stamp, pass, &sh.ncand);
    }
    __syncthreads();
    const int nc = sh.ncand;
    stamp++;
    for (int base = 0; base < nc; base += blockDim.x) {
      const int i = base + threadIdx.x;
      dt_apply<false>(b, i, i < nc, stamp, b.list[cur ^ 1], &sh.n[cur ^ 1]);
    }
    cur ^= 1;
  }
  __syncthreads();
  // an even number of passes leaves the list where the host expects it; else
  // it is copied there
  const int n = sh.n[cur];
  if (cur != cur0)
    for (int i = threadIdx.x; i < n; i += blockDim.x) b.list[cur0][i] = b.list[cur][i];
  // the next pass takes these entries as written with this stamp
  for (int i = threadIdx.x; i < n; i += blockDim.x) b.wstamp[b.list[cur][i]] = stamp;
  if (threadIdx.x == 0) {
    b.c->nlist[cur0] = n;
    b.c->ncand[0] = 0;
    b.c->ncand[1] = 0;
    b.c->nwin = stamp;
  }
}

// Inserts the np points of pend[0] (b.loc: a triangle to start from, times 4, +
// 3) round by round in one workgroup, where a round costs barriers instead of
// launches.  Returns the points left (0).
struct InsertState {
  int stamp = 0;
  uint32_t round = 0;
  uint64_t pass = 0;
};
__device__ __forceinline__ int wg_insert(const Bld &b, SeedShared &sh, int *s_ntri, int *pend0, int *pend1, int np,
                                         InsertState &st) {
  __shared__ int s_left, s_err;
  int *pend[2] = {pend0, pend1};
  int pc = 0, cur = 0;
  while (np > 0) {
    st.round++;
    if (threadIdx.x == 0) {
      s_left = 0;
      sh.n[0] = 0;
      s_err = b.c->err;
    }
    __syncthreads();
    if (s_err) break;
    for (int base = 0; base < np; base += blockDim.x) {
      const int i = base + threadIdx.x;
      dt_locate(b, i < np ? pend[pc][i] : 0, i < np, st.round);
    }
    __syncthreads();
    st.stamp++;
    for (int base = 0; base < np; base += blockDim.x) {
      const int i = base + threadIdx.x;
      const int p = i < np ? pend[pc][i] : 0;
      const bool done = dt_split<false>(b, p, i < np, st.round, st.stamp, s_ntri, &sh.n[0]);
      const int po = wave_take(&s_left, i < np && !done ? 1 : 0);
      if (i < np && !done) pend[pc ^ 1][po] = p;
    }
    __syncthreads();
    const int nl = sh.n[0];
    for (int i = threadIdx.x; i < nl; i += blockDim.x) dt_fix(b, b.list[0][i], st.round);
    __syncthreads();
    cur = 0;
    dt_flips(b, sh, cur, st.stamp, st.pass);
    __syncthreads();
    // every round inserts at least the point of the largest key
    if (s_left >= np || st.pass > kPassMax) {
      if (threadIdx.x == 0) set_err(b.c, kEInternal + 6);
      np = s_left;
      break;
    }
    np = s_left;
    pc ^= 1;
    __syncthreads();
  }
  return np;
}

// The sample: every step-th point along the curve, in one workgroup (4,096
// points 3.0 ms; with samples of 512, 1,024 or 2,048 and more rounds on the grid
// a build of 60,013 points took 15.3, 14.7, 14.6 ms against 15.1 and one of a
// million 38.6, 39.4, 38.7 against 37.6).  pend: two lists of ns entries.
// Leaves the rounds in nwin and the remaining points (0) in npend.
__global__ __launch_bounds__(kSeedBlk) void k_dt_seed(Bld b, int ns, int step, int *pend0, int *pend1) {
  __shared__ SeedShared sh;
  __shared__ int s_ntri;
  for (int i = threadIdx.x; i < ns; i += blockDim.x) {
    pend0[i] = i * step;
    b.loc[i * step] = 3;
  }
  if (threadIdx.x == 0) s_ntri = 1;
  InsertState st;
  const int np = wg_insert(b, sh, &s_ntri, pend0, pend1, ns, st);
  if (threadIdx.x == 0) {
    b.c->ntri = s_ntri;
    b.c->npend = np;
    b.c->nwin = (int)st.round;
    b.c->first_stamp = st.stamp;
    b.c->first_pass = (int)st.pass;
  }
}

// Every other point starts at a triangle of the sample point before it.
__device__ __forceinline__ void start_one(const Bld &b, int ns, int step, int *pend, int i) {
  const int s = min(i / step, ns - 1), k = i - s * step;
  if (k == 0) return;
  b.loc[i] = 4 * b.vt[s * step] + 3;
  pend[i - s - 1] = i;
}
__global__ __launch_bounds__(kBlk) void k_dt_start(Bld b, int ns, int step, int *pend) {
  if (b.c->err) return;  // (see k_vt_seed)
  const int stride = gridDim.x * blockDim.x;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < b.nv; i += stride) start_one(b, ns, step, pend, i);
}

// ---------------------------------------------------------------------------
// Stage 2: segment recovery
// ---------------------------------------------------------------------------
__device__ __forceinline__ void vt_one(const Bld &b, int t) {
  const int4 v = b.tv[t];
  b.vt[v.x] = t;
  b.vt[v.y] = t;
  b.vt[v.z] = t;
}
__global__ void k_vt(Bld b, int nt) {
  const int stride = gridDim.x * blockDim.x;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < nt; t += stride) vt_one(b, t);
}
// The sample's triangles, queued before the host has read how many there are:
// a sample that an error cut short (points that coincide) leaves fewer than
// its points call for, and the slots beyond them hold whatever the scratch
// memory held.
__global__ void k_vt_seed(Bld b) {
  if (b.c->err) return;
  const int nt = b.c->ntri, stride = gridDim.x * blockDim.x;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < nt; t += stride) vt_one(b, t);
}

// Around vertex a: the edge a-b (returns 1 with t, i of edge a->b or b->a),
// else the triangle whose wedge at a holds the direction to b (returns 0,
// t = that triangle), else an error code < 0.
__device__ int around(const Bld &b, int a, int bb, int &tout, int &iout) {
  const int start = b.vt[a];
  int cur = start, found = -1, onseg = 0;
  const double2 A = b.P[a], Bp = b.P[bb];
  for (int guard = 0; guard < kWalkCap; guard++) {
    const int4 v = b.tv[cur];
    const int k = vidx(v, a);
    if (k < 0) return -(kEInternal + 3);
    const int u = comp(v, (k + 1) % 3), w = comp(v, (k + 2) % 3);
    if (u == bb) { tout = cur; iout = k; return 1; }
    if (w == bb) { tout = cur; iout = (k + 2) % 3; return 1; }
    if (found < 0) {
      const double2 U = b.P[u], W = b.P[w];
      const int ou = orient2d(A.x, A.y, U.x, U.y, Bp.x, Bp.y);
      const int ow = orient2d(A.x, A.y, W.x, W.y, Bp.x, Bp.y);
      if (ou == 0 && (U.x - A.x) * (Bp.x - A.x) + (U.y - A.y) * (Bp.y - A.y) > 0) onseg = 1;
      if (ou > 0 && ow < 0) found = cur;
    }
    const int nx = comp(b.tn[cur], (k + 2) % 3);
    if (nx < 0) return -(kEInternal + 4);
    if (nx == start) break;
    cur = nx;
  }
  if (found < 0) return onseg ? -kEOnSeg : -kEDir;
  tout = found;
  return 0;
}

// Outputs of one walk along segment a->b from the triangle at a.
struct WalkOut {
  int *crossed;        // k
  int *lc, *lo, *lcn;  // left chain L_1..L_m; out tri / segment id of edge L_{i+1}->L_i (m + 1)
  int *rc, *ro, *rcn;  // right chain R_1..R_n; out of edge R_i->R_{i+1} (n + 1)
};

// Walks the triangles crossed by a->b.  mode 0: stamp the crossed triangles
// and their outer neighbours; mode 1: require the stamp before reading a
// triangle; mode 2: as mode 1 and fill w.  Returns the number of crossed
// triangles, or -2 for a foreign stamp, or -(error code + 16).
__device__ int seg_walk(const Bld &b, int a, int bb, int t0, uint64_t key, int mode, const WalkOut &w,
                        int &m_out, int &n_out) {
  auto stamp = [&](int t) -> bool {
    if (t < 0) return true;
    if (mode == 0) { atomicMax((unsigned long long *)&b.mark[t], (unsigned long long)key); return true; }
    return __hip_atomic_load(&b.mark[t], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == key;
  };
  if (!stamp(t0)) return -2;
  int4 v = b.tv[t0];
  int4 nb = b.tn[t0];
  int4 sg = b.ts[t0];
  const int k0 = vidx(v, a);
  if (k0 < 0) return -(kEInternal + 5 + 16);
  int R = comp(v, (k0 + 1) % 3), L = comp(v, (k0 + 2) % 3);
  int m = 0, n = 0, kc = 0;
  {
    const int ol = comp(nb, (k0 + 2) % 3), orr = comp(nb, k0);
    if (!stamp(ol) || !stamp(orr)) return -2;
    if (mode == 2) {
      w.lo[0] = ol; w.lcn[0] = comp(sg, (k0 + 2) % 3);
      w.ro[0] = orr; w.rcn[0] = comp(sg, k0);
      w.lc[0] = L; w.rc[0] = R;
      w.crossed[0] = t0;
    }
    m = 1; n = 1; kc = 1;
  }
  int cur = t0;
  const double2 A = b.P[a], Bp = b.P[bb];
  for (int guard = 0;; guard++) {
    if (guard > kWalkCap) return -(kEInternal + 6 + 16);
    const int e = eidx(v, R, L);
    if (e < 0) return -(kEInternal + 7 + 16);
    if (comp(sg, e) >= 0) return -(kECross + 16);
    const int nx = comp(nb, e);
    if (nx < 0) return -(kELeave + 16);
    if (!stamp(nx)) return -2;
    v = b.tv[nx];
    nb = b.tn[nx];
    sg = b.ts[nx];
    const int j = eidx(v, L, R);
    if (j < 0) return -(kEInternal + 8 + 16);
    const int wv = comp(v, (j + 2) % 3);
    if (mode == 2) w.crossed[kc] = nx;
    kc++;
    if (wv == bb) {
      const int orr = comp(nb, (j + 1) % 3), ol = comp(nb, (j + 2) % 3);
      if (!stamp(orr) || !stamp(ol)) return -2;
      if (mode == 2) {
        w.ro[n] = orr; w.rcn[n] = comp(sg, (j + 1) % 3);
        w.lo[m] = ol; w.lcn[m] = comp(sg, (j + 2) % 3);
      }
      break;
    }
    const double2 W = b.P[wv];
    const int o = orient2d(A.x, A.y, Bp.x, Bp.y, W.x, W.y);
    if (o == 0) return -(kEOnSeg + 16);
    if (o > 0) {
      const int ol = comp(nb, (j + 2) % 3);
      if (!stamp(ol)) return -2;
      if (mode == 2) { w.lo[m] = ol; w.lcn[m] = comp(sg, (j + 2) % 3); w.lc[m] = wv; }
      m++;
      L = wv;
    } else {
      const int orr = comp(nb, (j + 1) % 3);
      if (!stamp(orr)) return -2;
      if (mode == 2) { w.ro[n] = orr; w.rcn[n] = comp(sg, (j + 1) % 3); w.rc[n] = wv; }
      n++;
      R = wv;
    }
    cur = nx;
  }
  (void)cur;
  m_out = m;
  n_out = n;
  return kc;
}

__global__ void k_seg_rank(const int2 *seg, int ns, const int *rank, int2 *out) {
  const int stride = gridDim.x * blockDim.x;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < ns; i += stride) out[i] = make_int2(rank[seg[i].x], rank[seg[i].y]);
}

// A segment whose edge is there constrains it; another stamps what it crosses.
__device__ __forceinline__ void seg_mark_one(const Bld &b, const int2 *seg, int s, uint32_t round, int *sstart) {
  const int2 ab = seg[s];
  int t = -1, e = -1;
  const int r = around(b, ab.x, ab.y, t, e);
  if (r < 0) { set_err(b.c, -r); sstart[s] = -1; return; }
  if (r == 1) {
    // the edge is there: constrain both sides
    const int o = comp(b.tn[t], e);
    const int prev = atomicCAS(comp_ptr(b.ts, t, e), -1, s);
    if (prev != -1 && prev != s) set_err(b.c, kERepeat);
    if (o >= 0) {
      const int4 vt = b.tv[t];
      const int oe = eidx(b.tv[o], comp(vt, (e + 1) % 3), comp(vt, e));
      if (oe < 0) { set_err(b.c, kEInternal + 9); sstart[s] = -1; return; }
      const int p2 = atomicCAS(comp_ptr(b.ts, o, oe), -1, s);
      if (p2 != -1 && p2 != s) set_err(b.c, kERepeat);
    }
    sstart[s] = -1;
    return;
  }
  const uint64_t key = ((uint64_t)round << 32) | mix32((uint32_t)s);
  int m, n;
  const int kc = seg_walk(b, ab.x, ab.y, t, key, 0, WalkOut{}, m, n);
  if (kc < -2) { set_err(b.c, -kc - 16); sstart[s] = -1; return; }
  sstart[s] = t;
}
__global__ void k_seg_mark(Bld b, const int2 *seg, const int *list, int nl, uint32_t round, int *sstart) {
  const int stride = gridDim.x * blockDim.x;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < nl; i += stride)
    seg_mark_one(b, seg, list[i], round, sstart);
}

constexpr int kSegGrp = 8;

// Constrained Delaunay triangulation of the pseudo-polygon with base p->q
// and chain c[0..m) (from the p side to the q side, left of p->q); out[i] is
// the outer triangle / segment id across the polygon edge E[i+1]->E[i] of
// E = (p, c_0, .., c_{m-1}, q).  New triangles take the slots slot[*next..].
// Returns the slot of the triangle on the base.  Run by kSegGrp lanes: all of
// them keep the same state and store the same values; the scan for the apex is
// shared out, each step taking the first of kSegGrp vertices that is inside
// the circle of the best one so far, as a scan of one by one would.
__device__ int tri_poly(const Bld &b, int p, int q, const int *c, int m, const int *out, const int *outcn,
                        const int *slot, int &next, int *stk) {
  auto E = [&](int i) { return i == 0 ? p : (i == m + 1 ? q : c[i - 1]); };
  auto link_out = [&](int s, int ei, int x, int y, int oi) {
    // edge ei of s runs x->y; the outer triangle sees it as y->x
    const int o = out[oi];  // -2: a slit edge, linked inside the region afterwards
    *comp_ptr(b.tn, s, ei) = o;
    *comp_ptr(b.ts, s, ei) = outcn[oi];
    if (o >= 0) {
      const int oe = eidx(b.tv[o], y, x);
      if (oe >= 0) *comp_ptr(b.tn, o, oe) = s;
      else set_err(b.c, kEInternal + 10);
    }
  };
  const int gl = __lane_id() & (kSegGrp - 1), g0 = __lane_id() - gl;
  int sp = 0, root = -1;
  stk[0] = 0; stk[1] = m; stk[2] = -1; stk[3] = 0;
  sp = 1;
  while (sp > 0) {
    sp--;
    const int lo = stk[4 * sp], hi = stk[4 * sp + 1], ps = stk[4 * sp + 2], pe = stk[4 * sp + 3];
    const int u = E(lo), w = E(hi + 1);
    int best = lo, cb = c[lo];
    for (int k = lo + 1; k < hi;) {
      const int x = k + gl, cx = x < hi ? c[x] : -1;
      const int in = x < hi && incircle_sos(b, u, w, cb, cx) > 0;
      const unsigned hit = (unsigned)(__ballot(in) >> g0) & ((1u << kSegGrp) - 1);
      if (!hit) {
        k += kSegGrp;
        continue;
      }
      const int f = __ffs(hit) - 1;
      best = k + f;
      cb = __shfl(cx, g0 + f);
      k = best + 1;
    }
    const int s = slot[next++];
    b.tv[s] = make_int4(u, w, cb, 0);
    b.tn[s] = make_int4(ps, -1, -1, 0);
    b.ts[s] = make_int4(-1, -1, -1, 0);
    if (ps >= 0) *comp_ptr(b.tn, ps, pe) = s;
    else root = s;
    b.vt[u] = s; b.vt[w] = s; b.vt[cb] = s;
    // edge 1: w -> cb; the sub-polygon (best + 1, hi) or the polygon edge E[hi+1] -> E[hi]
    if (best + 1 < hi) { stk[4 * sp] = best + 1; stk[4 * sp + 1] = hi; stk[4 * sp + 2] = s; stk[4 * sp + 3] = 1; sp++; }
    else link_out(s, 1, w, cb, hi);
    // edge 2: cb -> u; the sub-polygon (lo, best) or the polygon edge E[lo+1] -> E[lo]
    if (best > lo) { stk[4 * sp] = lo; stk[4 * sp + 1] = best; stk[4 * sp + 2] = s; stk[4 * sp + 3] = 2; sp++; }
    else link_out(s, 2, cb, u, lo);
  }
  return root;
}

// Entry i of the list (act: i < nl) by its group of kSegGrp lanes, if it keeps
// every stamp of its walk; else it goes to the next list.  All lanes of the
// wave take part.
__device__ __forceinline__ void seg_insert_group(const Bld &b, const int2 *seg, const int *list, int i, bool act,
                                                 uint32_t round, const int *sstart, int *list_out, int *pool,
                                                 int *npend, int *nwin) {
  const int gl = __lane_id() & (kSegGrp - 1), g0 = __lane_id() - gl;
  int s = -1, kc = -2, m = 0, n = 0, t0 = -1;
  int2 ab = make_int2(0, 0);
  uint64_t key = 0;
  if (act) {
    s = list[i];
    t0 = sstart[s];
    if (t0 < 0) act = false;  // constrained in place (or failed)
  }
  if (act) {
    ab = seg[s];
    key = ((uint64_t)round << 32) | mix32((uint32_t)s);
    kc = seg_walk(b, ab.x, ab.y, t0, key, 1, WalkOut{}, m, n);
    if (kc < -2) { set_err(b.c, -kc - 16); act = false; }
  }
  const bool win = act && kc > 0;
  const int need = win ? kc + 3 * (m + 1) + 3 * (n + 1) + 4 * (kc + 2) + (m + n + 2) : 0;
  const int po = __shfl(wave_take(pool, gl == 0 ? need : 0), g0);
  const int lo = wave_take(npend, gl == 0 && act && !win ? 1 : 0);
  if (gl == 0 && act && !win) list_out[lo] = s;
  if (!win) return;
  if (po < 0 || (int64_t)po + need > b.pool_cap) { set_err(b.c, kEInternal + 11); return; }
  int *q = b.pool + po;
  WalkOut w;
  w.crossed = q; q += kc;
  w.lc = q; q += m + 1;
  w.lo = q; q += m + 1;
  w.lcn = q; q += m + 1;
  w.rc = q; q += n + 1;
  w.ro = q; q += n + 1;
  w.rcn = q; q += n + 1;
  int *stk = q; q += 4 * (kc + 2);
  int *rev = q;  // right chain reversed
  int m2, n2;
  if (seg_walk(b, ab.x, ab.y, t0, key, 2, w, m2, n2) != kc || m2 != m || n2 != n) { set_err(b.c, kEInternal + 12); return; }
  // Where the crossed region wraps around a vertex, an edge of a chain has
  // crossed triangles on both sides (a slit): it stays an edge of the new
  // triangulation, linked between the two new triangles that carry it.
  for (int x = gl; x < kc; x += kSegGrp) b.pick[w.crossed[x]] = key;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  bool slit = false;
  for (int k = gl; k <= m + n + 1; k += kSegGrp) {
    int *op = k <= m ? &w.lo[k] : &w.ro[k - m - 1];
    if (*op >= 0 && b.pick[*op] == key) {
      *op = -2;
      slit = true;
    }
  }
  slit = ((__ballot(slit) >> g0) & ((1u << kSegGrp) - 1)) != 0;
  // right side: base b->a, chain R_n..R_1, out[i] = edge R_{n-i} -> R_{n+1-i}
  for (int k = gl; k < n; k += kSegGrp) rev[k] = w.rc[n - 1 - k];
  for (int k = gl; k <= n / 2; k += kSegGrp) {
    const int x = n - k;
    int t1 = w.ro[k]; w.ro[k] = w.ro[x]; w.ro[x] = t1;
    int t2 = w.rcn[k]; w.rcn[k] = w.rcn[x]; w.rcn[x] = t2;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  if (gl == 0) atomicAdd(nwin, 1);
  int next = 0;
  const int rl = tri_poly(b, ab.x, ab.y, w.lc, m, w.lo, w.lcn, w.crossed, next, stk);
  const int rr = tri_poly(b, ab.y, ab.x, rev, n, w.ro, w.rcn, w.crossed, next, stk);
  if (next != kc) { set_err(b.c, kEInternal + 13); return; }
  *comp_ptr(b.tn, rl, 0) = rr;
  *comp_ptr(b.tn, rr, 0) = rl;
  *comp_ptr(b.ts, rl, 0) = s;
  *comp_ptr(b.ts, rr, 0) = s;
  for (int x = 0; x < kc && slit; x++) {
    const int t = w.crossed[x];
    const int4 tv = b.tv[t];
    for (int e = 0; e < 3; e++) {
      if (*comp_ptr(b.tn, t, e) != -2) continue;
      const int u = comp(tv, e), v = comp(tv, (e + 1) % 3);
      int found = -1;
      for (int y = 0; y < kc && found < 0; y++) {
        const int ye = eidx(b.tv[w.crossed[y]], v, u);
        if (ye >= 0) { found = y; *comp_ptr(b.tn, w.crossed[y], ye) = t; }
      }
      if (found < 0) { set_err(b.c, kEInternal + 15); continue; }
      *comp_ptr(b.tn, t, e) = w.crossed[found];
    }
  }
}

// The segments of a round, kSegGrp lanes to each.  Bound by the dependent loads
// of the longest segment (about one microsecond for each triangle it crosses
// and walk).  One thread per segment, which compared every chain edge with
// every crossed triangle for the slits and scanned for each apex alone, took
// 1.83 ms a round of a million points against 0.51 here.
__global__ __launch_bounds__(kBlk) void k_seg_insert(Bld b, const int2 *seg, const int *list, int nl, uint32_t round,
                                                     const int *sstart, int *list_out) {
  const int per = kBlk / kSegGrp, stride = gridDim.x * per;
  for (int base = blockIdx.x * per; base < nl; base += stride) {
    const int i = base + (int)threadIdx.x / kSegGrp;
    seg_insert_group(b, seg, list, i, i < nl, round, sstart, list_out, &b.c->pool, &b.c->npend, &b.c->nwin);
  }
}

// ---------------------------------------------------------------------------
// Stage 3: outside removal, checks, canonical order
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool is_out(const Bld &b, int t) {
  if (t < 0) return true;
  const int4 v = b.tv[t];
  return v.x >= b.nv || v.y >= b.nv || v.z >= b.nv;
}

// Whether triangle t stays; its sort key and hull edges.
__device__ __forceinline__ bool keep_one(const Bld &b, int t, int *used, uint64_t &key, int &hull) {
  if (is_out(b, t)) return false;
  const int4 v = b.tv[t], n = b.tn[t], sg = b.ts[t];
  used[v.x] = 1; used[v.y] = 1; used[v.z] = 1;
  for (int e = 0; e < 3; e++) {
    if (!is_out(b, comp(n, e))) continue;
    hull++;
    if (comp(sg, e) < 0) { set_err(b.c, kEHull); continue; }
    // the boundary must turn left at its end vertex
    const int u = comp(v, e), x = comp(v, (e + 1) % 3);
    int cur = t, ce = (e + 1) % 3;
    for (int guard = 0; guard < kWalkCap; guard++) {
      const int o = comp(b.tn[cur], ce);
      if (is_out(b, o)) break;
      cur = o;
      ce = vidx(b.tv[o], x);
      if (ce < 0) { set_err(b.c, kEInternal + 14); ce = 0; break; }
    }
    const int y = comp(b.tv[cur], (ce + 1) % 3);
    if (orient_ids(b.P, u, x, y) < 0) set_err(b.c, kEDisk);
  }
  const int4 w = make_int4(b.id[v.x], b.id[v.y], b.id[v.z], 0);
  const int r = (w.y < w.x && w.y < w.z) ? 1 : ((w.z < w.x && w.z < w.y) ? 2 : 0);
  key = ((uint64_t)(uint32_t)comp(w, r) << 32) | (uint32_t)comp(w, (r + 1) % 3);
  return true;
}

__global__ __launch_bounds__(kBlk) void k_keep(Bld b, int nt, int *used, uint64_t *keys, int *vals) {
  const int stride = gridDim.x * blockDim.x;
  for (int base = blockIdx.x * blockDim.x; base < nt; base += stride) {
    const int t = base + threadIdx.x;
    int hull = 0;
    uint64_t key = 0;
    const bool keep = t < nt && keep_one(b, t, used, key, hull);
    const int slot = block_take(&b.c->nkeep, keep ? 1 : 0);
    if (hull) atomicAdd(&b.c->nhull, hull);
    if (keep) { keys[slot] = key; vals[slot] = t; }
  }
}

__global__ void k_used(Bld b, const int *used) {
  const int stride = gridDim.x * blockDim.x;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < b.nv; i += stride)
    if (!used[i]) set_err(b.c, kEUnused);
}

__global__ void k_newid(int nk, const int *vals, int *newid) {
  const int stride = gridDim.x * blockDim.x;
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < nk; k += stride) newid[vals[k]] = k;
}

__device__ __forceinline__ void emit_one(const Bld &b, int k, const int *vals, const int *newid, int4 *otv, int4 *otn,
                                         int4 *ots) {
  const int t = vals[k];
  const int4 vr = b.tv[t], n = b.tn[t], sg = b.ts[t];
  const int4 v = make_int4(b.id[vr.x], b.id[vr.y], b.id[vr.z], 0);
  const int r = (v.y < v.x && v.y < v.z) ? 1 : ((v.z < v.x && v.z < v.y) ? 2 : 0);
  int vv[3], nn[3], ss[3];
  for (int i = 0; i < 3; i++) {
    const int src = (r + i) % 3;
    vv[i] = comp(v, src);
    const int o = comp(n, src);
    nn[i] = is_out(b, o) ? -1 : newid[o];
    ss[i] = comp(sg, src);
  }
  const int mask = (ss[0] >= 0 ? 1 : 0) | (ss[1] >= 0 ? 2 : 0) | (ss[2] >= 0 ? 4 : 0);
  otv[k] = make_int4(vv[0], vv[1], vv[2], mask);
  otn[k] = make_int4(nn[0], nn[1], nn[2], 0);
  ots[k] = make_int4(ss[0], ss[1], ss[2], 0);
}
__global__ void k_emit(Bld b, int nk, const int *vals, const int *newid, int4 *otv, int4 *otn, int4 *ots) {
  const int stride = gridDim.x * blockDim.x;
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < nk; k += stride) emit_one(b, k, vals, newid, otv, otn, ots);
}

// ---------------------------------------------------------------------------
// Canonical order: least-significant-digit radix sort of (key, value) pairs
// by 8-bit digits, one stable counting pass per digit that varies:
//   1. tile histograms (a tile is kSortThreads x kSortItems keys), written
//      digit-major, so that
//   2. one exclusive scan gives every (digit, tile) its output offset;
//   3. each tile scatters its keys in their input order: items are taken
//      kSortThreads at a time; inside a wave, lanes with the same digit find
//      each other by eight ballots (one per digit bit) and rank themselves by
//      the lanes below; the waves' digit counts, taken in wave order, and the
//      running count of the tile's earlier items complete the rank.
// ---------------------------------------------------------------------------
constexpr int kSortThreads = 256;
constexpr int kSortItems = 8;
constexpr int kSortTile = kSortThreads * kSortItems;
constexpr int kSortWaves = kSortThreads / 64;

__global__ __launch_bounds__(kSortThreads) void k_sort_hist(const uint64_t *keys, int n, int shift, int ntiles,
                                                            int *hist) {
  __shared__ int h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const int base = blockIdx.x * kSortTile;
  for (int j = 0; j < kSortItems; j++) {
    const int i = base + j * kSortThreads + threadIdx.x;
    if (i < n) atomicAdd(&h[(keys[i] >> shift) & 0xff], 1);
  }
  __syncthreads();
  hist[threadIdx.x * ntiles + blockIdx.x] = h[threadIdx.x];
}

// Exclusive scan of hist[0..m) in place by one workgroup: kScanPer entries per
// thread and step, read and written as vectors (m is a multiple of 256).
constexpr int kSortScanThreads = 1024;
__global__ __launch_bounds__(kSortScanThreads) void k_sort_scan(int *hist, int m) {
  __shared__ int part[kSortScanThreads / 64];
  __shared__ int s_carry;
  const int lane = __lane_id(), wid = threadIdx.x >> 6;
  int carry = 0;
  for (int base = 0; base < m; base += kSortScanThreads * 16) {
    const int i0 = base + (int)threadIdx.x * 16;
    int4 v[4];
    int sum = 0;
#pragma unroll
    for (int k = 0; k < 4; k++) {
      v[k] = i0 + 4 * k < m ? *reinterpret_cast<const int4 *>(hist + i0 + 4 * k) : make_int4(0, 0, 0, 0);
      sum += v[k].x + v[k].y + v[k].z + v[k].w;
    }
    int x = sum;
    for (int d = 1; d < 64; d <<= 1) {
      const int y = __shfl_up(x, d);
      if (lane >= d) x += y;
    }
    if (lane == 63) part[wid] = x;
    __syncthreads();
    if (threadIdx.x < kSortScanThreads / 64) {
      int y = part[threadIdx.x];
      for (int d = 1; d < kSortScanThreads / 64; d <<= 1) {
        const int z = __shfl_up(y, d);
        if ((int)threadIdx.x >= d) y += z;
      }
      part[threadIdx.x] = y;
      if (threadIdx.x == kSortScanThreads / 64 - 1) s_carry = y;
    }
    __syncthreads();
    int run = carry + x - sum + (wid ? part[wid - 1] : 0);
#pragma unroll
    for (int k = 0; k < 4; k++) {
      int4 o;
      o.x = run; run += v[k].x;
      o.y = run; run += v[k].y;
      o.z = run; run += v[k].z;
      o.w = run; run += v[k].w;
      if (i0 + 4 * k < m) *reinterpret_cast<int4 *>(hist + i0 + 4 * k) = o;
    }
    carry += s_carry;
    __syncthreads();
  }
}

__global__ __launch_bounds__(kSortThreads) void k_sort_scatter(const uint64_t *keys, const int *vals,
                                                               uint64_t *keys_out, int *vals_out, int n, int shift,
                                                               int ntiles, const int *offs) {
  __shared__ int run[256];       // items of the tile ranked so far, per digit
  __shared__ int wcnt[kSortWaves][256];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  run[threadIdx.x] = offs[threadIdx.x * ntiles + blockIdx.x];
  for (int w = 0; w < kSortWaves; w++) wcnt[w][threadIdx.x] = 0;
  __syncthreads();
  const int base = blockIdx.x * kSortTile;
  const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
  for (int j = 0; j < kSortItems; j++) {
    const int i = base + j * kSortThreads + threadIdx.x;
    const bool act = i < n;
    const uint64_t k = act ? keys[i] : 0ull;
    const int v = act ? vals[i] : 0;
    const int d = (int)((k >> shift) & 0xff);
    uint64_t peers = __ballot(act);
    for (int bit = 0; bit < 8; bit++) {
      const uint64_t m = __ballot((d >> bit) & 1);
      peers &= ((d >> bit) & 1) ? m : ~m;
    }
    const int rank = __popcll(peers & below);
    if (act && rank == 0) wcnt[wave][d] = __popcll(peers);
    __syncthreads();
    if (act) {
      int pos = run[d] + rank;
      for (int w = 0; w < wave; w++) pos += wcnt[w][d];
      keys_out[pos] = k;
      vals_out[pos] = v;
    }
    __syncthreads();
    int add = 0;
    for (int w = 0; w < kSortWaves; w++) {
      add += wcnt[w][threadIdx.x];
      wcnt[w][threadIdx.x] = 0;
    }
    run[threadIdx.x] += add;
    __syncthreads();
  }
}

// Sorts n pairs by the low vbits of each 32-bit half of the key (halves: 1:
// the low half only, else a key is (a << 32) | b with a, b < 2^vbits); the
// result ends in (k1, v1).  hist holds 256 * ceil(n / kSortTile) ints.
hipError_t radix_sort_pairs(hipStream_t stream, uint64_t *k0, int *v0, uint64_t *k1, int *v1, int n, int vbits,
                            int *hist, int halves = 2) {
  if (n <= 0) return hipSuccess;
  const int ntiles = (n + kSortTile - 1) / kSortTile;
  int shifts[16], ns = 0;
  for (int half = 0; half < halves; half++)
    for (int b = 0; b < vbits; b += 8) shifts[ns++] = 32 * half + b;
  uint64_t *kin = k0, *kout = k1;
  int *vin = v0, *vout = v1;
  for (int p = 0; p < ns; p++) {
    k_sort_hist<<<ntiles, kSortThreads, 0, stream>>>(kin, n, shifts[p], ntiles, hist);
    k_sort_scan<<<1, kSortScanThreads, 0, stream>>>(hist, 256 * ntiles);
    k_sort_scatter<<<ntiles, kSortThreads, 0, stream>>>(kin, vin, kout, vout, n, shifts[p], ntiles, hist);
    std::swap(kin, kout);
    std::swap(vin, vout);
  }
  // after an odd number of passes the result is in (k1, v1); else copy it there
  if (kin != k1) {
    hipError_t e = hipMemcpyAsync(k1, kin, sizeof(uint64_t) * n, hipMemcpyDeviceToDevice, stream);
    if (e == hipSuccess) e = hipMemcpyAsync(v1, vin, sizeof(int) * n, hipMemcpyDeviceToDevice, stream);
    if (e != hipSuccess) return e;
  }
  return hipGetLastError();
}

__global__ void k_iota(int n, int *a) {
  const int stride = gridDim.x * blockDim.x;
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) a[i] = i;
}

int grid_for(int n, int blk) { return std::max(1, std::min((n + blk - 1) / blk, 4096)); }

// The scratch of a build and its view; some arrays lie where another stage's
// will be: the lists of the flip passes in the pool of the segment recovery
// and in the sort buffers of the last stage, the points' walks under the
// segments' starts, the split stamps under the new ids, the ranks under the
// used marks, the renumbered segments in the sort keys (when they fit: a
// planar set has fewer than 3 nv segments).  Returns the bytes (base may be
// null).
struct Scratch {
  Bld b;
  double2 *P;
  int *id, *rank, *pl[2], *used, *vals, *vals2, *newid, *hist;
  uint64_t *keys, *keys2;
  unsigned long long *box;
  int2 *sseg;
};
size_t cdt_scratch(int nv, int ns, char *base, Scratch &S) {
  const int capT = 2 * nv + 8;
  // (ints; from 67 million vertices on more than an int counts, of which the
  // segment recovery uses what it can count)
  const int64_t pool_ints = 16 * (int64_t)capT + 4096;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += (bytes + 255) & ~(size_t)255; return base + o; };
  Bld &b = S.b;
  b.nv = nv;
  b.capT = capT;
  b.pool_cap = (int)std::min<int64_t>(pool_ints, 0x7fffffff);
  b.tv = (int4 *)take(sizeof(int4) * capT);
  b.tn = (int4 *)take(sizeof(int4) * capT);
  b.ts = (int4 *)take(sizeof(int4) * capT);
  b.pick = (uint64_t *)take(8 * (size_t)capT);
  b.mark = (uint64_t *)take(8 * (size_t)capT);
  b.loc = b.state = (int *)take(4 * (size_t)std::max(nv, ns));
  b.vt = (int *)take(4 * (size_t)(nv + 3));
  b.wstamp = (int *)take(4 * (size_t)capT);
  b.pool = (int *)take(4 * (size_t)pool_ints);
  S.P = (double2 *)take(sizeof(double2) * (size_t)(nv + 3));
  S.id = (int *)take(4 * (size_t)(nv + 3));
  S.pl[0] = (int *)take(4 * (size_t)std::max(nv, ns));
  S.pl[1] = (int *)take(4 * (size_t)std::max(nv, ns));
  b.c = (Ctr *)take(sizeof(Ctr));
  S.box = (unsigned long long *)take(4 * 8);
  S.used = S.rank = (int *)take(4 * (size_t)nv);
  S.keys = (uint64_t *)take(8 * (size_t)capT);
  S.keys2 = (uint64_t *)take(8 * (size_t)capT);
  S.vals = (int *)take(4 * (size_t)capT);
  S.vals2 = (int *)take(4 * (size_t)capT);
  S.newid = (int *)take(4 * (size_t)capT);
  S.hist = (int *)take(4 * 256 * (size_t)((capT + kSortTile - 1) / kSortTile));
  S.sseg = ns <= 2 * (int64_t)capT ? (int2 *)S.keys : (int2 *)take(sizeof(int2) * (size_t)ns);
  b.P = S.P;
  b.id = S.id;
  b.sstamp = S.newid;
  b.fc0 = (int4 *)b.pool;
  b.fc1 = b.fc0 + 2 * (size_t)capT;
  b.grp = b.fc0;
  b.fprio = S.keys;
  b.list[0] = S.vals;
  b.list[1] = S.vals2;
  return off;
}

// ---------------------------------------------------------------------------
// Many small builds at once: one workgroup to a mesh, all stages in it.
// ---------------------------------------------------------------------------
struct MeshJob {
  Scratch S;
  DevCdtJob j;
};

// Radix sort by the 8-bit digits at the given shifts, as k_sort_*: the digit
// counts of all pairs, then the pairs in their order, a workgroup's worth at a
// time.  Returns whether the result is in (k1, v1) (else (k0, v0)).
struct SortShared {
  int run[256], wcnt[kSeedBlk / 64][256];
};
__device__ bool wg_sort(SortShared &S, uint64_t *k0, int *v0, uint64_t *k1, int *v1, int n, int vbits, int halves) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t below = lane ? (~0ull >> (64 - lane)) : 0ull;
  bool odd = false;
  for (int half = 0; half < halves; half++)
    for (int bit0 = 0; bit0 < vbits; bit0 += 8, odd = !odd) {
      const uint64_t *kin = odd ? k1 : k0;
      const int *vin = odd ? v1 : v0;
      uint64_t *kout = odd ? k0 : k1;
      int *vout = odd ? v0 : v1;
      const int shift = 32 * half + bit0;
      if (tid < 256) S.run[tid] = 0;
      for (int i = tid; i < 256 * (kSeedBlk / 64); i += kSeedBlk) (&S.wcnt[0][0])[i] = 0;
      __syncthreads();
      for (int i = tid; i < n; i += kSeedBlk) atomicAdd(&S.run[(kin[i] >> shift) & 0xff], 1);
      __syncthreads();
      if (wave == 0) {  // exclusive scan, four digits to a lane
        int c[4], sum = 0;
        for (int q = 0; q < 4; q++) {
          c[q] = S.run[4 * lane + q];
          sum += c[q];
        }
        int x = sum;
        for (int d = 1; d < 64; d <<= 1) {
          const int y = __shfl_up(x, d);
          if (lane >= d) x += y;
        }
        x -= sum;
        for (int q = 0; q < 4; q++) {
          S.run[4 * lane + q] = x;
          x += c[q];
        }
      }
      __syncthreads();
      for (int base = 0; base < n; base += kSeedBlk) {
        const int i = base + tid;
        const bool act = i < n;
        const uint64_t k = act ? kin[i] : 0ull;
        const int v = act ? vin[i] : 0;
        const int d = (int)((k >> shift) & 0xff);
        uint64_t peers = __ballot(act);
        for (int bit = 0; bit < 8; bit++) {
          const uint64_t m = __ballot((d >> bit) & 1);
          peers &= ((d >> bit) & 1) ? m : ~m;
        }
        const int rank = __popcll(peers & below);
        if (act && rank == 0) S.wcnt[wave][d] = __popcll(peers);
        __syncthreads();
        if (act) {
          int pos = S.run[d] + rank;
          for (int w = 0; w < wave; w++) pos += S.wcnt[w][d];
          kout[pos] = k;
          vout[pos] = v;
        }
        __syncthreads();
        if (tid < 256) {
          int add = 0;
          for (int w = 0; w < kSeedBlk / 64; w++) {
            add += S.wcnt[w][tid];
            S.wcnt[w][tid] = 0;
          }
          S.run[tid] += add;
        }
        __syncthreads();
      }
    }
  return odd;
}

// Whether a stage of the workgroup's mesh found an error (uniform).
__device__ __forceinline__ bool wg_failed(const Ctr *c) {
  __shared__ int s_err;
  __syncthreads();
  if (threadIdx.x == 0) s_err = c->err;
  __syncthreads();
  const int e = s_err;
  __syncthreads();
  return e != 0;
}

// The stages are a launch each, a workgroup to a mesh, the scratch zero at
// first; an error (c->err) skips the later ones.  Bound by the largest mesh:
// 40,000 vertices take 25 ms of insertion (latency while the lists are short,
// then the one workgroup's issue rate) and 5 ms of the rest, 128 meshes of 100
// to 40,000 side by side no more.  All stages in one kernel kept more pointers
// and spilled more: 36 ms for 50,004 points, of which the sample took 8 instead
// of 3 (k_mesh_insert and k_mesh_segs spill 90 and 138 registers still, at the
// 128 that a lane of 1,024 threads gets).  With 512 or 256 threads a batch of
// 128 takes 74 or 92 ms instead of 68.
__global__ __launch_bounds__(kSeedBlk) void k_mesh_sort(const MeshJob *jobs) {
  __shared__ SortShared so;
  __shared__ unsigned long long s_box[4];
  const MeshJob &J = jobs[blockIdx.x];
  const Bld b = J.S.b;
  const int nv = b.nv, tid = threadIdx.x;
  const double2 *xy = J.j.xy;
  if (tid < 4) s_box[tid] = 0;
  __syncthreads();
  {
    unsigned long long m[4] = {0, 0, 0, 0};
    for (int i = tid; i < nv; i += kSeedBlk) {
      const double2 p = xy[i];
      m[0] = max(m[0], ord_of(p.x));
      m[1] = max(m[1], ord_of(p.y));
      m[2] = max(m[2], ord_of(-p.x));
      m[3] = max(m[3], ord_of(-p.y));
    }
    for (int k = 0; k < 4; k++) {
      for (int d = 32; d >= 1; d >>= 1) {
        const unsigned long long o = (unsigned long long)__shfl_xor((long long)m[k], d);
        m[k] = max(m[k], o);
      }
      if (__lane_id() == 0) atomicMax(&s_box[k], m[k]);
    }
  }
  __syncthreads();
  double ext[4];
  for (int k = 0; k < 4; k++) {
    const unsigned long long o = s_box[k], u = (o >> 63) ? (o & ~(1ull << 63)) : ~o;
    ext[k] = __longlong_as_double((long long)u);
  }
  const double x0 = -ext[2], y0 = -ext[3], side = max(max(ext[0] - x0, ext[1] - y0), 0x1p-100);
  const double mx = max(max(max(1.0, fabs(x0)), fabs(ext[0])), max(fabs(y0), fabs(ext[1])));
  int ex;
  (void)frexp(mx, &ex);
  const double L = ldexp(1.0, ex + 1);
  for (int i = tid; i < nv; i += kSeedBlk) {
    J.S.keys[i] = morton_of(xy[i], x0, y0, 65536.0 / side);
    J.S.vals[i] = i;
  }
  __syncthreads();
  (void)wg_sort(so, J.S.keys, J.S.vals, J.S.keys2, J.S.vals2, nv, 32, 1);  // (an even number of digits)
  for (int i = tid; i < nv; i += kSeedBlk) {
    const int v = J.S.vals[i];
    J.S.P[i] = xy[v];
    J.S.id[i] = v;
    J.S.rank[v] = i;
  }
  if (tid == 0) first_triangle(b, J.S.P, J.S.id, L);
}

// Insertion: bound by latency while lists are short, then by the one
// workgroup's issue rate.
__global__ __launch_bounds__(kSeedBlk) void k_mesh_insert(const MeshJob *jobs) {
  __shared__ SeedShared sh;
  __shared__ int s_ntri;
  const Bld b = jobs[blockIdx.x].S.b;
  int *pl0 = jobs[blockIdx.x].S.pl[0], *pl1 = jobs[blockIdx.x].S.pl[1];
  const int nv = b.nv, tid = threadIdx.x;
  const int step = (nv + kSeedMax - 1) / kSeedMax, n_seed = (nv + step - 1) / step;
  if (tid == 0) s_ntri = 1;
  for (int i = tid; i < n_seed; i += kSeedBlk) {
    pl0[i] = i * step;
    b.loc[i * step] = 3;
  }
  __syncthreads();
  InsertState st;
  // the sample, then the other points
  for (int part = 0; part < (n_seed < nv ? 2 : 1); part++) {
    if (part == 1) {
      __syncthreads();
      for (int t = tid; t < s_ntri; t += kSeedBlk) vt_one(b, t);
      __syncthreads();
      for (int i = tid; i < nv; i += kSeedBlk) start_one(b, n_seed, step, pl0, i);
      __syncthreads();
    }
    (void)wg_insert(b, sh, &s_ntri, pl0, pl1, part == 0 ? n_seed : nv - n_seed, st);
  }
  __syncthreads();
  if (tid == 0) {
    if (s_ntri != 2 * nv + 1) set_err(b.c, kEInternal + 16);
    b.c->ntri = s_ntri;
    b.c->nwin = (int)st.round;
  }
}

__global__ __launch_bounds__(kSeedBlk) void k_mesh_segs(const MeshJob *jobs, DevCdtResult *res) {
  __shared__ int s_pool, s_npend, s_nwin;
  const MeshJob &J = jobs[blockIdx.x];
  const Bld b = J.S.b;
  const int ns = J.j.ns, tid = threadIdx.x, nt = b.c->ntri, dt_rounds = b.c->nwin;
  if (wg_failed(b.c)) {
    if (tid == 0) res[blockIdx.x] = DevCdtResult{b.c->err, 0, 0, dt_rounds, 0};
    return;
  }
  int seg_rounds = 0;
  for (int t = tid; t < nt; t += kSeedBlk) {
    vt_one(b, t);
    b.ts[t] = make_int4(-1, -1, -1, -1);
    b.mark[t] = 0;
  }
  for (int i = tid; i < ns; i += kSeedBlk) {
    const int2 sg = J.j.seg[i];
    J.S.sseg[i] = make_int2(J.S.rank[sg.x], J.S.rank[sg.y]);
    J.S.pl[0][i] = i;
  }
  __syncthreads();
  uint32_t round = (uint32_t)dt_rounds;
  for (int nl = ns, cur = 0; nl > 0; cur ^= 1) {
    round++;
    seg_rounds++;
    if (tid == 0) s_pool = s_npend = s_nwin = 0;
    for (int i = tid; i < nl; i += kSeedBlk) seg_mark_one(b, J.S.sseg, J.S.pl[cur][i], round, b.state);
    __syncthreads();
    constexpr int per = kSeedBlk / kSegGrp;
    for (int base = 0; base < nl; base += per) {
      const int i = base + tid / kSegGrp;
      seg_insert_group(b, J.S.sseg, J.S.pl[cur], i, i < nl, round, b.state, J.S.pl[cur ^ 1], &s_pool, &s_npend, &s_nwin);
    }
    __syncthreads();
    const int left = s_npend;
    if (tid == 0 && left > 0 && s_nwin == 0 && left == nl) set_err(b.c, kEInternal + 17);
    if (wg_failed(b.c)) break;
    nl = left;
  }
  if (tid == 0)
    res[blockIdx.x] = DevCdtResult{b.c->err, 1, 0, dt_rounds, seg_rounds};
}

// Outside removal and canonical order.
__global__ __launch_bounds__(kSeedBlk) void k_mesh_final(const MeshJob *jobs, DevCdtResult *res) {
  __shared__ SortShared so;
  __shared__ int s_npend, s_nwin;
  const MeshJob &J = jobs[blockIdx.x];
  const Bld b = J.S.b;
  const int nv = b.nv, ns = J.j.ns, tid = threadIdx.x, nt = b.c->ntri;
  if (wg_failed(b.c)) return;
  for (int i = tid; i < nv; i += kSeedBlk) J.S.used[i] = 0;
  if (tid == 0) s_npend = s_nwin = 0;  // kept triangles, hull edges
  __syncthreads();
  for (int base = 0; base < nt; base += kSeedBlk) {
    const int t = base + tid;
    int hull = 0;
    uint64_t key = 0;
    const bool keep = t < nt && keep_one(b, t, J.S.used, key, hull);
    const int slot = wave_take(&s_npend, keep ? 1 : 0);
    if (hull) atomicAdd(&s_nwin, hull);
    if (keep) { J.S.keys[slot] = key; J.S.vals[slot] = t; }
  }
  __syncthreads();
  for (int i = tid; i < nv; i += kSeedBlk)
    if (!J.S.used[i]) set_err(b.c, kEUnused);
  const int nk = s_npend;
  if (!wg_failed(b.c) && tid == 0) {
    if ((int64_t)nk != 2 * (int64_t)nv - s_nwin - 2) set_err(b.c, kEDisk);
    else if (nk > J.j.cap_out) set_err(b.c, kEInternal + 18);
  }
  if (wg_failed(b.c)) {
    if (tid == 0) {
      res[blockIdx.x].stage = 2;
      res[blockIdx.x].err = b.c->err;
    }
    return;
  }
  int vbits = 1;
  while (vbits < 31 && (1 << vbits) < nv + 3) vbits++;
  const int *vals = wg_sort(so, J.S.keys, J.S.vals, J.S.keys2, J.S.vals2, nk, vbits, 2) ? J.S.vals2 : J.S.vals;
  for (int k = tid; k < nk; k += kSeedBlk) J.S.newid[vals[k]] = k;
  __syncthreads();
  for (int k = tid; k < nk; k += kSeedBlk) emit_one(b, k, vals, J.S.newid, J.j.tv, J.j.tn, J.j.ts);
  for (int i = tid; i < nv; i += kSeedBlk) J.j.vxy[i] = J.j.xy[i];
  for (int i = tid; i < ns; i += kSeedBlk) {
    J.j.sv[i] = J.j.seg[i];
    J.j.spar[i] = i;
  }
  if (tid == 0) {
    DevState *d = J.j.st;
    d->nV = nv;
    d->nT = nk;
    d->nS = ns;
    d->wT = nk / 32 + 1;
    d->wS = ns / 32 + 1;
    d->full = 1;
    res[blockIdx.x].nt = nk;
  }
}

}  // namespace

size_t dev_cdt_batch_bytes(const DevCdtJob *jobs, size_t n) {
  auto up = [](size_t b) { return (b + 255) & ~(size_t)255; };
  size_t bytes = 0;
  Scratch S;
  for (size_t i = 0; i < n; i++) bytes += up(cdt_scratch(jobs[i].nv, jobs[i].ns, nullptr, S));
  return bytes + up(sizeof(MeshJob) * n) + up(sizeof(DevCdtResult) * n);
}

// Queues the builds of jobs (scratch: dev_cdt_batch_bytes bytes of device
// memory); *res is their results in it, valid once the stream has finished.
int dev_cdt_batch(hipStream_t stream, const DevCdtJob *jobs, size_t n, void *scratch, DevCdtResult **res) {
  std::vector<MeshJob> d(n);
  char *at = (char *)scratch;
  for (size_t i = 0; i < n; i++) {
    d[i].j = jobs[i];
    at += (cdt_scratch(jobs[i].nv, jobs[i].ns, at, d[i].S) + 255) & ~(size_t)255;
  }
  MeshJob *dj = (MeshJob *)at;
  *res = (DevCdtResult *)(at + ((sizeof(MeshJob) * n + 255) & ~(size_t)255));
  if (hipMemsetAsync(scratch, 0, (size_t)(at - (char *)scratch), stream) != hipSuccess ||
      hipMemcpyAsync(dj, d.data(), sizeof(MeshJob) * n, hipMemcpyHostToDevice, stream) != hipSuccess ||
      hipStreamSynchronize(stream) != hipSuccess)  // d is a local
    return GDP_E_DEVICE;
  k_mesh_sort<<<(unsigned)n, kSeedBlk, 0, stream>>>(dj);
  k_mesh_insert<<<(unsigned)n, kSeedBlk, 0, stream>>>(dj);
  k_mesh_segs<<<(unsigned)n, kSeedBlk, 0, stream>>>(dj, *res);
  k_mesh_final<<<(unsigned)n, kSeedBlk, 0, stream>>>(dj, *res);
  return hipGetLastError() == hipSuccess ? GDP_OK : GDP_E_DEVICE;
}

int dev_cdt_result(const DevCdtResult &r, std::string &err) {
  if (!r.err) return GDP_OK;
  err = std::string(r.stage == 0 ? "points: " : (r.stage == 1 ? "segments: " : "final: ")) + cdt_err_string(r.err);
  return r.err >= kEInternal ? GDP_E_DEVICE : GDP_E_INPUT;
}

// Sorts n (64-bit key, int) pairs by the whole key (8 digit passes); the
// result ends in (k1, v1).  hist holds 256 * ceil(n / 2048) ints.
static_assert(kSortPairsTile == kSortTile, "the sort's tile as declared in gdp_internal.h");
hipError_t sort_pairs_u64(hipStream_t stream, uint64_t *k0, int *v0, uint64_t *k1, int *v1, int n, int *hist) {
  return radix_sort_pairs(stream, k0, v0, k1, v1, n, 32, hist);
}

void dev_cdt_work_free(DevCdtWork &ws) {
  if (ws.mem) (void)hipFree(ws.mem);
  if (ws.hctr) (void)hipHostFree(ws.hctr);
  ws = DevCdtWork();
}

// Builds the CDT of the PSLG whose nv vertices (d_xy) and segments (d_seg) are
// on the device; writes the canonical triangles to otv / otn / ots (capacity
// cap_out) and their count to *n_tri.  Coordinates and segment endpoints are
// checked by the caller.  Returns GDP_OK, GDP_E_INPUT (invalid PSLG, err set),
// GDP_E_NOMEM or GDP_E_DEVICE.
int dev_cdt_build(hipStream_t stream, int32_t nv, double2 *d_xy, int32_t ns, const int2 *d_seg, int4 *otv,
                  int4 *otn, int4 *ots, int32_t cap_out, int32_t *n_tri, DevCdtStats *stats, std::string &err,
                  DevCdtWork *ws) {
  if (nv < 3) { err = "bad arguments"; return GDP_E_ARG; }
  void *mem = nullptr;
  Scratch S;
  const size_t off = cdt_scratch(nv, ns, nullptr, S);
  static_assert(sizeof(Ctr) <= sizeof(DevCounters), "lent pinned memory holds the counters of a round");
  Ctr *hctr = nullptr;
  if (ws && ws->lent) {
    if (ws->bytes < off) {
      ws = nullptr;
    } else {
      mem = ws->mem;
      hctr = (Ctr *)ws->hctr;
    }
  }
  if (mem) {
  } else if (ws) {
    // every earlier build on the workspace has finished (each one ends with
    // a stream synchronisation), so its scratch can be replaced
    if (ws->bytes < off) {
      if (ws->mem) (void)hipFree(ws->mem);
      ws->mem = nullptr;
      ws->bytes = 0;
      if (hipMalloc(&ws->mem, off) != hipSuccess) { ws->mem = nullptr; err = "device allocation failed"; return GDP_E_NOMEM; }
      ws->bytes = off;
    }
    if (!ws->hctr && hipHostMalloc(&ws->hctr, sizeof(Ctr)) != hipSuccess) { ws->hctr = nullptr; err = "host allocation failed"; return GDP_E_NOMEM; }
    mem = ws->mem;
    hctr = (Ctr *)ws->hctr;
  } else {
    if (hipMalloc(&mem, off) != hipSuccess) { err = "device allocation failed"; return GDP_E_NOMEM; }
    if (hipHostMalloc((void **)&hctr, sizeof(Ctr)) != hipSuccess) { (void)hipFree(mem); err = "host allocation failed"; return GDP_E_NOMEM; }
  }
  char *base = (char *)mem;
  auto done = [&](int rc) {
    (void)hipStreamSynchronize(stream);
    if (!ws) {
      (void)hipFree(mem);
      (void)hipHostFree(hctr);
    }
    return rc;
  };
  (void)cdt_scratch(nv, ns, base, S);
  const Bld b = S.b;
  const int capT = b.capT;
  double2 *P = S.P;
  int *id = S.id, *rank = S.rank;
  unsigned long long *box = S.box;
  int *pl[2] = {S.pl[0], S.pl[1]};
  auto dev_err = [&](const char *what) { err = what; return done(GDP_E_DEVICE); };
  if (hipMemsetAsync(b.pick, 0, 8 * (size_t)capT, stream) != hipSuccess ||
      hipMemsetAsync(b.mark, 0, 8 * (size_t)capT, stream) != hipSuccess ||
      hipMemsetAsync(b.sstamp, 0, 4 * (size_t)capT, stream) != hipSuccess ||
      hipMemsetAsync(b.wstamp, 0, 4 * (size_t)capT, stream) != hipSuccess ||
      hipMemsetAsync(box, 0, 4 * 8, stream) != hipSuccess ||
      hipMemsetAsync(b.c, 0, sizeof(Ctr), stream) != hipSuccess)
    return dev_err("device call failed");
  auto round_trip = [&]() -> bool {
    if (hipMemcpyAsync(hctr, b.c, sizeof(Ctr), hipMemcpyDeviceToHost, stream) != hipSuccess) return false;
    return hipStreamSynchronize(stream) == hipSuccess;
  };
  // the points along a Morton curve of their box, and the enclosing triangle
  // (placed as the host builder places it)
  k_box<<<std::min(grid_for(nv, kBlk), 256), kBlk, 0, stream>>>(d_xy, nv, box);
  unsigned long long hbox[4];
  if (hipMemcpyAsync(hbox, box, sizeof hbox, hipMemcpyDeviceToHost, stream) != hipSuccess ||
      hipStreamSynchronize(stream) != hipSuccess)
    return dev_err("copy failed");
  const double x1 = ord_to(hbox[0]), y1 = ord_to(hbox[1]), x0 = -ord_to(hbox[2]), y0 = -ord_to(hbox[3]);
  const double mx = std::max({1.0, std::fabs(x0), std::fabs(x1), std::fabs(y0), std::fabs(y1)});
  const double Lb = std::exp2(std::ceil(std::log2(mx)) + 1.0);
  const double side = std::max({x1 - x0, y1 - y0, 0x1p-100});
  uint64_t *keys = S.keys, *keys2 = S.keys2;
  int *vals = S.vals, *vals2 = S.vals2, *newid = S.newid;
  k_morton<<<grid_for(nv, kBlk), kBlk, 0, stream>>>(d_xy, nv, x0, y0, 65536.0 / side, keys, vals);
  if (radix_sort_pairs(stream, keys, vals, keys2, vals2, nv, 32, S.hist, 1) != hipSuccess)
    return dev_err("sort failed");
  k_reorder<<<grid_for(nv, kBlk), kBlk, 0, stream>>>(b, d_xy, P, vals2, id, rank, Lb);
  // the sample in one workgroup, then every other point round by round
  const int step = (nv + kSeedMax - 1) / kSeedMax, n_seed = (nv + step - 1) / step;
  k_dt_seed<<<1, kSeedBlk, 0, stream>>>(b, n_seed, step, pl[0], pl[1]);
  if (n_seed < nv) {
    k_vt_seed<<<grid_for(2 * n_seed + 1, kBlk), kBlk, 0, stream>>>(b);
    k_dt_start<<<grid_for(nv, kBlk), kBlk, 0, stream>>>(b, n_seed, step, pl[0]);
  }
  if (!round_trip()) return dev_err("device call failed");
  int dt_rounds = hctr->nwin, seg_rounds = 0;
  auto points_failed = [&]() {
    err = std::string("points (round " + std::to_string(dt_rounds) + "): ") + cdt_err_string(hctr->err);
    return done(hctr->err >= kEInternal ? GDP_E_DEVICE : GDP_E_INPUT);
  };
  if (hctr->err) return points_failed();
  int np = nv - n_seed, cur = 0, stamp = hctr->first_stamp;
  uint64_t pass = (uint64_t)hctr->first_pass;
  uint32_t round = (uint32_t)dt_rounds;
  while (np > 0) {
    round++;
    dt_rounds++;
    if (hipMemsetAsync(&b.c->npend, 0, 2 * sizeof(int), stream) != hipSuccess ||  // npend, nwin
        hipMemsetAsync(&b.c->nlist[0], 0, 4 * sizeof(int), stream) != hipSuccess)
      return dev_err("device call failed");
    stamp++;
    k_dt_locate<<<grid_for(np, kBlk), kBlk, 0, stream>>>(b, pl[cur], np, round);
    k_dt_split<<<grid_for(np, kBlk), kBlk, 0, stream>>>(b, pl[cur], np, round, stamp, pl[cur ^ 1]);
    // at most one point per triangle, three new triangles each (four for the
    // rare one on an edge)
    int64_t est = 4 * std::min<int64_t>(np, hctr->ntri);
    k_dt_fix<<<grid_for((int)std::min<int64_t>(est, 1 << 30), kBlk), kBlk, 0, stream>>>(b, round);
    for (;;) {
      if (pass > kPassMax) return dev_err("device CDT builder: flip passes did not converge");
      for (int q = 0; q < kPassBatch; q++) {
        pass++;
        const unsigned g = grid_for((int)std::min<int64_t>(est, 1 << 30), kBlk);
        k_dt_check<<<g, kBlk, 0, stream>>>(b, q & 1, stamp, pass);
        stamp++;
        k_dt_apply<<<g, kBlk, 0, stream>>>(b, q & 1, stamp, pass);
      }
      k_dt_tail<<<1, kSeedBlk, 0, stream>>>(b, 0, stamp, pass);
      if (!round_trip()) return dev_err("device call failed");
      if (hctr->err) return points_failed();
      // (the tail sets nwin to the stamp of what it leaves, if it ran)
      if (hctr->nlist[0] == 0) {
        stamp += kTailGap;
        pass += kTailGap;
        break;
      }
      if (hctr->nwin > stamp) {
        stamp = hctr->nwin;
        pass += kTailGap;
      }
      est = hctr->nlist[0];
      if (stamp > (1 << 30)) return dev_err("device CDT builder: flip passes did not converge");
    }
    if (hctr->npend >= np) { err = "device CDT builder: no insertion progress"; return done(GDP_E_DEVICE); }
    np = hctr->npend;
    cur ^= 1;
  }
  const int nt = hctr->ntri;
  if (nt != 2 * nv + 1) { err = "device CDT builder: triangle count"; return done(GDP_E_DEVICE); }
  // segments, between the points' places along the curve
  int2 *sseg = S.sseg;
  k_vt<<<grid_for(nt, kBlk), kBlk, 0, stream>>>(b, nt);
  if (hipMemsetAsync(b.ts, 0xff, sizeof(int4) * (size_t)nt, stream) != hipSuccess ||
      hipMemsetAsync(b.mark, 0, 8 * (size_t)nt, stream) != hipSuccess)
    return dev_err("device call failed");
  if (ns > 0) k_seg_rank<<<grid_for(ns, kBlk), kBlk, 0, stream>>>(d_seg, ns, rank, sseg);
  int *sstart = b.state;
  int nl = ns;
  cur = 0;
  if (ns > 0) k_iota<<<grid_for(ns, kBlk), kBlk, 0, stream>>>(ns, pl[0]);
  while (nl > 0) {
    round++;
    seg_rounds++;
    if (hipMemsetAsync(b.c, 0, 3 * sizeof(int), stream) != hipSuccess) { err = "device call failed"; return done(GDP_E_DEVICE); }
    k_seg_mark<<<grid_for(nl, kBlk), kBlk, 0, stream>>>(b, sseg, pl[cur], nl, round, sstart);
    k_seg_insert<<<grid_for((int)std::min<int64_t>((int64_t)nl * kSegGrp, 1 << 30), kBlk), kBlk, 0, stream>>>(b, sseg, pl[cur], nl, round, sstart, pl[cur ^ 1]);
    if (!round_trip()) { err = "device call failed"; return done(GDP_E_DEVICE); }
    if (hctr->err) { err = std::string("segments (round " + std::to_string(seg_rounds) + "): ") + cdt_err_string(hctr->err); return done(hctr->err >= kEInternal ? GDP_E_DEVICE : GDP_E_INPUT); }
    if (hctr->npend > 0 && hctr->nwin == 0 && hctr->npend == nl) { err = "device CDT builder: no segment progress"; return done(GDP_E_DEVICE); }
    nl = hctr->npend;
    cur ^= 1;
  }
  // outside removal and canonical order
  int *used = S.used;
  if (hipMemsetAsync(used, 0, 4 * (size_t)nv, stream) != hipSuccess || hipMemsetAsync(b.c, 0, sizeof(Ctr), stream) != hipSuccess)
    { err = "device call failed"; return done(GDP_E_DEVICE); }
  k_keep<<<grid_for(nt, kBlk), kBlk, 0, stream>>>(b, nt, used, keys, vals);
  k_used<<<grid_for(nv, kBlk), kBlk, 0, stream>>>(b, used);
  if (!round_trip()) { err = "device call failed"; return done(GDP_E_DEVICE); }
  if (hctr->err) { err = std::string("final: ") + cdt_err_string(hctr->err); return done(hctr->err >= kEInternal ? GDP_E_DEVICE : GDP_E_INPUT); }
  const int nk = hctr->nkeep;
  if ((int64_t)nk != 2 * (int64_t)nv - hctr->nhull - 2) { err = "the kept region is not a disk"; return done(GDP_E_INPUT); }
  if (nk > cap_out) { err = "output capacity"; return done(GDP_E_NOMEM); }
  int vbits = 1;
  while (vbits < 31 && (1 << vbits) < nv + 3) vbits++;
  if (radix_sort_pairs(stream, keys, vals, keys2, vals2, nk, vbits, S.hist) != hipSuccess)
    { err = "sort failed"; return done(GDP_E_DEVICE); }
  k_newid<<<grid_for(nk, kBlk), kBlk, 0, stream>>>(nk, vals2, newid);
  k_emit<<<grid_for(nk, kBlk), kBlk, 0, stream>>>(b, nk, vals2, newid, otv, otn, ots);
  if (hipStreamSynchronize(stream) != hipSuccess || hipGetLastError() != hipSuccess)
    { err = "device call failed"; return done(GDP_E_DEVICE); }
  *n_tri = nk;
  if (stats) { stats->dt_rounds = dt_rounds; stats->seg_rounds = seg_rounds; }
  return done(GDP_OK);
}

}  // namespace gdp
