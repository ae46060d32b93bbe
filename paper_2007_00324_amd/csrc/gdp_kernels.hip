// gdp_kernels.hip -- gfx950 kernels of one refinement round (Algorithm 1,
// Lines 3-8 of gDP2d, with cavity insertion as in Section 5.2).
//
// Every kernel works on a slot-indexed structure-of-arrays mesh in HBM.  The
// round is deterministic: candidate lists are built with atomics in any
// order, but every decision depends only on the mesh at the start of the
// round, on 64-bit priority keys (unique per element) and on atomicMax,
// which is order independent; vertex ids, triangle slots and subsegment ids
// of the inserted points come from prefix sums over element-indexed bitmaps.
#include "gdp_kernels.h"

namespace gdp {

// ---------------------------------------------------------------------------
// Priorities (Section 4.3: midpoints before circumcenters, then larger
// length / area first; the element id, mixed by a fixed bijection, makes
// every key unique).
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t perm32(uint32_t x) {
  // MurmurHash3 32-bit finalizer applied to id + 1 (never 0)
  uint32_t h = x + 1u;
  h ^= h >> 16;
  h *= 0x85ebca6bu;
  h ^= h >> 13;
  h *= 0xc2b2ae35u;
  h ^= h >> 16;
  return h;
}

__device__ __forceinline__ uint32_t perm32_inv(uint32_t h) {
  h ^= h >> 16;
  h *= 0x7ed1b41du;  // inverse of 0xc2b2ae35 mod 2^32
  h ^= (h >> 13) ^ (h >> 26);
  h *= 0xa5cb9243u;  // inverse of 0x85ebca6b mod 2^32
  h ^= h >> 16;
  return h - 1u;
}

__device__ __forceinline__ uint32_t q31(double x) {
  uint64_t b = (uint64_t)__double_as_longlong(x);
  return (uint32_t)((b >> 32) & 0x7fffffffu);
}

__device__ __forceinline__ int comp(const int4 &v, int i) { return i == 0 ? v.x : (i == 1 ? v.y : v.z); }

struct SplitPt {
  double px, py;
  uint64_t key;
  int bad;
  double d;  // doubled area by the fixed formula (triangles)
};

// Circumcenter / radius-edge test / key of triangle t, in one fixed FP64
// operation order (vertices rotated so the smallest id comes first); a
// needle (non-positive FP64 doubled area, or a circumcenter beyond 2^20)
// is bad, has measure 0 and splits at the midpoint of its longest edge.
__device__ SplitPt tri_split(const DevMesh &m, int t, int4 tri, double B2, double L2, int pm) {
  int v0 = tri.x, v1 = tri.y, v2 = tri.z, ia, ib, ic;
  if (v0 < v1 && v0 < v2) { ia = v0; ib = v1; ic = v2; }
  else if (v1 < v2) { ia = v1; ib = v2; ic = v0; }
  else { ia = v2; ib = v0; ic = v1; }
  double2 A = m.vxy[ia], B = m.vxy[ib], C = m.vxy[ic];
  double ax = A.x, ay = A.y;
  double bx = B.x - ax, by = B.y - ay;
  double cx = C.x - ax, cy = C.y - ay;
  double b2 = bx * bx + by * by;
  double c2 = cx * cx + cy * cy;
  double d = bx * cy - by * cx;
  double ex = C.x - B.x, ey = C.y - B.y;
  double e2 = ex * ex + ey * ey;
  SplitPt r;
  uint64_t q = 0;
  bool needle = true;
  if (d > 0.0) {
    double den = d + d;
    double ux = (cy * b2 - by * c2) / den;
    double uy = (bx * c2 - cx * b2) / den;
    double px = ax + ux, py = ay + uy;
    if (fabs(px) <= 0x1p20 && fabs(py) <= 0x1p20) {
      needle = false;
      r.px = px;
      r.py = py;
      double r2 = ux * ux + uy * uy;
      double lmin2 = b2;
      if (c2 < lmin2) lmin2 = c2;
      if (e2 < lmin2) lmin2 = e2;
      r.bad = r2 > B2 * lmin2 ? 1 : 0;
      if (L2 > 0.0) {
        // edge-length bound (Section 4.1): the longest edge against l^2
        double lmax2 = b2;
        if (c2 > lmax2) lmax2 = c2;
        if (e2 > lmax2) lmax2 = e2;
        if (lmax2 > L2) r.bad = 1;
      }
      q = q31(d);
    }
  }
  if (needle) {
    double2 U = A, W = B;
    double best = b2;
    if (c2 > best) { best = c2; U = A; W = C; }
    if (e2 > best) { best = e2; U = B; W = C; }
    r.px = (U.x + W.x) * 0.5;
    r.py = (U.y + W.y) * 0.5;
    r.bad = 1;
    q = 0;
  }
  if (pm == 1) q = 0;
  // mode 2: a tie-break that does not depend on the slot (the first two ids
  // of the rotation that starts at the smallest id, 22 bits each), above it
  // the measure reduced to 19 bits
  if (pm == 2) r.key = ((q >> 12) << 44) | ((uint64_t)ia << 22) | (uint64_t)ib;
  else r.key = (q << 32) | (uint64_t)perm32((uint32_t)t);
  r.d = d;
  return r;
}

// Splitting point of subsegment k: its midpoint, or with split_mode 1
// (concentric shells) when exactly one endpoint c is an input vertex, the
// point at distance 2^j from c, 2^j the power of two nearest to half the
// length (2^e if len/2 = f 2^e with f > 3/4, else 2^(e-1)), so that
// subsegments meeting at a small input angle are cut on common circles.
__device__ SplitPt seg_split(const DevMesh &m, int k, int pm, int split_mode) {
  int2 s = m.sv[k];
  double2 A = m.vxy[s.x], B = m.vxy[s.y];
  SplitPt r;
  double dx = B.x - A.x, dy = B.y - A.y;
  double len2 = dx * dx + dy * dy;
  const bool ina = split_mode == 1 && m.vkind[s.x] == 0, inb = split_mode == 1 && m.vkind[s.y] == 0;
  if (ina != inb) {
    const double2 C = ina ? A : B, O = ina ? B : A;
    const double len = sqrt(len2);
    int e;
    const double f = frexp(len * 0.5, &e);
    const double d = f > 0.75 ? ldexp(1.0, e) : ldexp(1.0, e - 1);
    const double t = d / len;
    r.px = C.x + (O.x - C.x) * t;
    r.py = C.y + (O.y - C.y) * t;
  } else {
    r.px = (A.x + B.x) * 0.5;
    r.py = (A.y + B.y) * 0.5;
  }
  uint64_t q = pm == 1 ? 0 : (uint64_t)q31(len2);
  r.key = (1ull << 63) | (q << 32) | (uint64_t)perm32((uint32_t)k);
  r.bad = 1;
  return r;
}

// ---------------------------------------------------------------------------
// Small helpers
// ---------------------------------------------------------------------------
// A variable-size allocation by one wave (all 64 lanes take part): one
// atomic per wave instead of one per lane.
__device__ __forceinline__ int wave_alloc(int *counter, int n) {
  int lane = __lane_id();
  int x = n;
  for (int d = 1; d < 64; d <<= 1) {
    int y = __shfl_up(x, d);
    if (lane >= d) x += y;
  }
  int total = __shfl(x, 63);
  int base = 0;
  if (lane == 63 && total > 0) base = atomicAdd(counter, total);
  base = __shfl(base, 63);
  return base + x - n;
}

// Encroachment of subsegment ab by p under the round's mode (circle or lens).
__device__ __forceinline__ bool encroached(const Work &w, double2 a, double2 b, double2 p) {
  return encroaches(w.enc_mode, a.x, a.y, b.x, b.y, p.x, p.y, w.tally);
}

// Entry idx of the midpoint list: subsegment k.
__device__ __forceinline__ void put_mid(const Work &w, int idx, int k) {
  w.mid.elem[idx] = k;
  w.mid.state[idx] = 0;
  w.cidx_s[k] = idx;
}

// Flags subsegment k; the first flag of the round appends it to the list.
// (One lane at a time: used where flags are rare; the collection gathers its
// flags and appends them per workgroup, see push_mids.)
__device__ __forceinline__ void flag_mid(const Work &w, int k) {
  if (atomicOr(&w.mflag[k], 1u) == 0u) put_mid(w, atomicAdd(&w.cnt->nmk, 1), k);
}

// Round statistics: a wave-wide sum (every lane of the wave takes part)
// added by one lane to the stat line of the wave.
__device__ __forceinline__ StatLine *stat_line(const Work &w) {
  const unsigned wave = (blockIdx.x * blockDim.x + threadIdx.x) >> 6;
  return w.stat + (wave & (kStatStripes - 1));
}
__device__ __forceinline__ void stat_add(const Work &w, int f, uint64_t v) {
  for (int d = 32; d > 0; d >>= 1) v += __shfl_xor(v, d);
  if (__lane_id() == 0 && v) atomicAdd((unsigned long long *)&stat_line(w)->v[f], (unsigned long long)v);
}
// Two statistics summed at once whose wave sums fit 32 bits.
__device__ __forceinline__ void stat_add2(const Work &w, int f0, int f1, uint32_t a, uint32_t b) {
  uint64_t v = (uint64_t)a | ((uint64_t)b << 32);
  for (int k = 32; k > 0; k >>= 1) v += __shfl_xor(v, k);
  if (__lane_id() == 0 && v) {
    StatLine *l = stat_line(w);
    if (v & 0xffffffffu) atomicAdd((unsigned long long *)&l->v[f0], (unsigned long long)(v & 0xffffffffu));
    if (v >> 32) atomicAdd((unsigned long long *)&l->v[f1], (unsigned long long)(v >> 32));
  }
}
__device__ __forceinline__ void stat_max(const Work &w, int f, uint64_t v) {
  for (int d = 32; d > 0; d >>= 1) v = max(v, (uint64_t)__shfl_xor(v, d));
  if (__lane_id() == 0 && v) atomicMax((unsigned long long *)&stat_line(w)->v[f], (unsigned long long)v);
}

__device__ __forceinline__ bool bit_get(const uint32_t *bm, int i) { return (bm[i >> 5] >> (i & 31)) & 1u; }
__device__ __forceinline__ void bit_set(uint32_t *bm, int i) { atomicOr(&bm[i >> 5], 1u << (i & 31)); }

// Rank of bit i among the set bits of bm: the scanned popcounts of the words
// before it (word prefix + tile prefix) and the set bits below it in its word.
__device__ __forceinline__ int bit_rank(const uint32_t *bm, const int32_t *words_prefix, const int32_t *tiles, int i) {
  uint32_t w = bm[i >> 5];
  uint32_t below = (i & 31) ? (w & ((1u << (i & 31)) - 1u)) : 0u;
  return words_prefix[i >> 5] + tiles[(i >> 5) / kScanTileSize] + __popc(below);
}

__device__ __forceinline__ int orient_pts(const Work &w, double2 a, double2 b, double2 c) {
  return orient2d(a.x, a.y, b.x, b.y, c.x, c.y, w.tally);
}

__device__ __forceinline__ int incircle_tri(const DevMesh &m, const Work &w, int4 tri, double2 p) {
  double2 A = m.vxy[tri.x], B = m.vxy[tri.y], C = m.vxy[tri.z];
  return incircle(A.x, A.y, B.x, B.y, C.x, C.y, p.x, p.y, w.tally);
}

__device__ __forceinline__ bool in_sorted(const int32_t *a, int n, int v) {
  int lo = 0, hi = n - 1;
  while (lo <= hi) {
    int mid = (lo + hi) >> 1;
    int x = a[mid];
    if (x == v) return true;
    if (x < v) lo = mid + 1; else hi = mid - 1;
  }
  return false;
}

// Work distribution of a phase: item = base + threadIdx.x for base = base0,
// base0 + stride, ...  A grid kernel spreads the items over all workgroups;
// the single-workgroup engine takes them all.  The loops are uniform over a
// workgroup, as the wave-wide operations require.
// blk: every thread of the workgroup runs the loop (grid kernels), so list
// space can be taken once per workgroup; otherwise once per wave (the
// engine, whose waves share one compute unit and see no contention).
struct Lanes {
  int base0, stride, blk;
};
__device__ __forceinline__ Lanes grid_lanes() {
  return {(int)(blockIdx.x * blockDim.x), (int)(gridDim.x * blockDim.x), 1};
}
__device__ __forceinline__ Lanes block_lanes() { return {0, (int)blockDim.x, 0}; }

// n entries per lane from a shared counter: returns this lane's first offset.
// One atomic per workgroup (L.blk) or per wave; the loops that call it are
// uniform over the workgroup.
constexpr int kMaxWaves = 16;
__device__ __forceinline__ int group_alloc(int *counter, int n, const Lanes &L) {
  if (!L.blk) return wave_alloc(counter, n);
  __shared__ int s_part[kMaxWaves];
  __shared__ int s_base;
  const int lane = __lane_id(), wid = threadIdx.x >> 6;
  int x = n;
  for (int d = 1; d < 64; d <<= 1) {
    int y = __shfl_up(x, d);
    if (lane >= d) x += y;
  }
  if (lane == 63) s_part[wid] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    int acc = 0;
    for (int i = 0; i < (int)(blockDim.x >> 6); i++) {
      int t = s_part[i];
      s_part[i] = acc;
      acc += t;
    }
    s_base = acc ? atomicAdd(counter, acc) : 0;
  }
  __syncthreads();
  const int r = s_base + s_part[wid] + x - n;
  __syncthreads();
  return r;
}

// The midpoint entries a lane flagged (up to 4), appended together (kept in
// named registers: an indexed array would go to scratch memory).
struct MidFlags {
  int k0 = -1, k1 = -1, k2 = -1, k3 = -1;
  int n = 0;
  __device__ __forceinline__ void push(int k) {
    k3 = n == 3 ? k : k3;
    k2 = n == 2 ? k : k2;
    k1 = n == 1 ? k : k1;
    k0 = n == 0 ? k : k0;
    n++;
  }
};
__device__ __forceinline__ void push_mids(const Work &w, const MidFlags &f, const Lanes &L) {
  const int off = group_alloc(&w.cnt->nmk, f.n, L);
  if (f.n > 0) put_mid(w, off, f.k0);
  if (f.n > 1) put_mid(w, off + 1, f.k1);
  if (f.n > 2) put_mid(w, off + 2, f.k2);
  if (f.n > 3) put_mid(w, off + 3, f.k3);
}
// the first lane of the whole distribution (single writes)
__device__ __forceinline__ bool first_lane(const Lanes &L) { return L.base0 == 0 && threadIdx.x == 0; }

// ---------------------------------------------------------------------------
// R1: collect encroached subsegments and bad triangles (Line 3)
// ---------------------------------------------------------------------------
// Tests one triangle: subsegment sides + encroaching apex, and badness.
__device__ __forceinline__ bool scan_triangle(const DevMesh &m, const Work &w, int i, double B2, int pm,
                                              SplitPt &r, MidFlags &fl) {
  int4 tri = m.tv[i];
  if (tri.w) {
    int4 s = m.ts[i];
    for (int e = 0; e < 3; e++) {
      if (!((tri.w >> e) & 1)) continue;
      int k = comp(s, e);
      int u = comp(tri, e), v = comp(tri, (e + 1) % 3), c = comp(tri, (e + 2) % 3);
      int side = (u == m.sv[k].x) ? 0 : 1;
      w.sadj[2 * k + side] = i * 4 + e;
      double2 U = m.vxy[u], V = m.vxy[v], Cc = m.vxy[c];
      if (encroached(w, U, V, Cc) && atomicOr(&w.mflag[k], 1u) == 0u) fl.push(k);
    }
  }
  r = tri_split(m, i, tri, B2, w.L2, pm);
  return r.bad != 0;
}

__device__ __forceinline__ void append_cc(const Work &w, bool bad, int t, const SplitPt &r, const Lanes &L) {
  int idx = group_alloc(&w.cnt->ncc, bad ? 1 : 0, L);
  if (bad) {
    w.cc.elem[idx] = t;
    w.cc.key[idx] = r.key;
    w.cc.p[idx] = make_double2(r.px, r.py);
    w.cc.state[idx] = 0;
    w.cidx_t[t] = idx;
  }
}

// Full collection over every triangle and subsegment (first round of a call).
__device__ __forceinline__ void scan_part(const DevMesh &m, const Work &w, double B2, int pm, const Lanes &L) {
  const int nT = w.st->nT, nS = w.st->nS, n = max(nT, nS);
  for (int base = L.base0; base < n; base += L.stride) {
    int i = base + threadIdx.x;
    bool bad = false;
    SplitPt r;
    MidFlags fl;
    if (i < nT) bad = scan_triangle(m, w, i, B2, pm, r, fl);
    append_cc(w, bad, i, r, L);
    if (i < nS && m.spend[i] && atomicOr(&w.mflag[i], 1u) == 0u) fl.push(i);
    push_mids(w, fl, L);
  }
}

__global__ void k_scan(DevMesh m, Work w, double B2, int pm) {
  if (w.st->halt) return;
  scan_part(m, w, B2, pm, grid_lanes());
}

// Incremental collection, later rounds.  A triangle that no winner rewrote
// keeps its vertices, so its badness and split point are unchanged: the bad
// triangles of the previous round that were not rewritten are carried over.
// (The carried list and the rewritten slots are collected by one kernel, one
// grid-stride loop each; each loop is uniform over the grid, as the wave-wide
// appends require.)
__device__ __forceinline__ void carry_part(const Work &w, const Lanes &L) {
  const int n_prev = w.st->prev_ncc, prev_serial = w.st->serial - 1;
  for (int base = L.base0; base < n_prev; base += L.stride) {
    int c = base + threadIdx.x;
    bool keep = false;
    int t = 0;
    if (c < n_prev) {
      t = w.prev_cc_elem[c];
      keep = w.tstamp[t] != prev_serial;
    }
    int idx = group_alloc(&w.cnt->ncc, keep ? 1 : 0, L);
    if (keep) {
      w.cc.elem[idx] = t;
      w.cc.key[idx] = w.prev_cc_key[c];
      w.cc.p[idx] = w.prev_cc_p[c];
      w.cc.state[idx] = 0;
      w.cidx_t[t] = idx;
    }
  }
}

// ... and every slot written last round (the fan records) is tested afresh;
// an encroaching apex can only appear on a rewritten triangle.
__device__ __forceinline__ void dirty_part(const DevMesh &m, const Work &w, double B2, int pm, const Lanes &L) {
  const int n_dirty = w.st->prev_fan;
  for (int base = L.base0; base < n_dirty; base += L.stride) {
    int c = base + threadIdx.x;
    bool bad = false;
    SplitPt r;
    MidFlags fl;
    int t = 0;
    if (c < n_dirty) {
      t = w.fan[c].slot;
      bad = scan_triangle(m, w, t, B2, pm, r, fl);
    }
    append_cc(w, bad, t, r, L);
    push_mids(w, fl, L);
  }
}

// ... and last round's flagged subsegments are tested again: pending, or an
// apex still inside the diametric circle (a flagged subsegment the candidate
// cap left out is not pending, and its sides may be unchanged).  The side
// slots are current: rewritten sides were re-scanned just before.
// Returns true if subsegment k is flagged anew.
__device__ __forceinline__ bool pending_one(const DevMesh &m, const Work &w, int k) {
  if (m.spend[k]) return atomicOr(&w.mflag[k], 1u) == 0u;
  for (int side = 0; side < 2; side++) {
    int a = w.sadj[2 * k + side];
    if (a < 0) continue;
    int t = a >> 2, e = a & 3;
    int4 tri = m.tv[t];
    double2 U = m.vxy[comp(tri, e)], V = m.vxy[comp(tri, (e + 1) % 3)], C = m.vxy[comp(tri, (e + 2) % 3)];
    if (encroached(w, U, V, C)) return atomicOr(&w.mflag[k], 1u) == 0u;
  }
  return false;
}

__device__ __forceinline__ void pending_part(const DevMesh &m, const Work &w, const Lanes &L) {
  const int n_prev = w.st->prev_nmk;
  for (int base = L.base0; base < n_prev; base += L.stride) {
    int c = base + threadIdx.x;
    MidFlags fl;
    if (c < n_prev) {
      const int k = w.prev_mid_elem[c];
      if (pending_one(m, w, k)) fl.push(k);
    }
    push_mids(w, fl, L);
  }
}

__global__ void k_collect(DevMesh m, Work w, double B2, int pm) {
  if (w.st->halt) return;
  carry_part(w, grid_lanes());
  dirty_part(m, w, B2, pm, grid_lanes());
}

// Separate launch: it reads side slots that k_collect rewrites.
__global__ void k_pending(DevMesh m, Work w) {
  if (w.st->halt) return;
  pending_part(m, w, grid_lanes());
}

// After the collection: stop if nothing is left (Algorithm 1, the loop ends
// when L is empty) or if the round cap is reached with work left.
// One workgroup.  At the round cap this round's flags are dropped before
// leaving.  Returns the halt code it set (0: the round goes on).
__device__ __forceinline__ int gate_part(const Work &w, int max_rounds) {
  __shared__ int s_h;
  DevState *st = w.st;
  DevCounters *c = w.cnt;
  if (threadIdx.x == 0) {
    s_h = 0;
    if (!st->halt) {
      const int ncc = c->ncc, nmk = c->nmk;
      c->nmk0 = nmk;
      if (ncc == 0 && nmk == 0) s_h = kHaltDone;
      else if (max_rounds > 0 && st->rounds >= max_rounds) s_h = kHaltCap;
      if (s_h) st->halt = s_h;
    }
  }
  __syncthreads();
  const int h = s_h;
  if (h == kHaltCap) {
    const int nmk = c->nmk;
    for (int i = threadIdx.x; i < nmk; i += blockDim.x) w.mflag[w.mid.elem[i]] = 0u;
  }
  return h;
}

__global__ void k_gate(Work w, int max_rounds) { (void)gate_part(w, max_rounds); }

// ---------------------------------------------------------------------------
// R3 (optional): keep the K largest keys.  Keys of both classes are placed in
// one array; a radix select finds the K-th largest (keys are unique).
// ---------------------------------------------------------------------------
__device__ __forceinline__ void gather_part(const DevMesh &m, const Work &w, int pm, const Lanes &L) {
  const int ncc = w.cnt->ncc, nmk = w.cnt->nmk;
  if (first_lane(L)) {
    w.sel[0] = 0;  // prefix
    w.sel[1] = 0;  // prefix mask
  }
  for (int base = L.base0; base < ncc + nmk; base += L.stride) {
    int c = base + threadIdx.x;
    if (c >= ncc + nmk) break;
    if (c < ncc) {
      w.keys[c] = w.cc.key[c];
    } else {
      int j = c - ncc;
      SplitPt r = seg_split(m, w.mid.elem[j], pm, w.split_mode);
      w.mid.key[j] = r.key;
      w.mid.p[j] = make_double2(r.px, r.py);
      w.keys[c] = r.key;
    }
  }
}

__global__ void k_gather_keys(DevMesh m, Work w, int pm) {
  if (w.st->halt) return;
  gather_part(m, w, pm, grid_lanes());
}

// Histogram of 8-bit digit `shift` over keys whose higher digits equal the
// prefix chosen so far.
__global__ void k_radix_hist(Work w, int shift) {
  __shared__ int h[256];
  if (w.st->halt) return;
  const int n = w.cnt->ncc + w.cnt->nmk;
  const uint64_t prefix = w.sel[0], pmask = w.sel[1];
  for (int i = threadIdx.x; i < 256; i += blockDim.x) h[i] = 0;
  __syncthreads();
  for (int c = blockIdx.x * blockDim.x + threadIdx.x; c < n; c += gridDim.x * blockDim.x) {
    uint64_t k = w.keys[c];
    if ((k & pmask) == prefix) atomicAdd(&h[(k >> shift) & 255u], 1);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 256; i += blockDim.x)
    if (h[i]) atomicAdd(&w.rhist[i], h[i]);
}

// Picks the digit of the K-th largest key (keys are unique) and clears the
// histogram for the next digit.  With no more than K keys the threshold is 0
// and every key is kept.
__device__ __forceinline__ void radix_pick_part(const Work &w, int shift, int K) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    const int n = w.cnt->ncc + w.cnt->nmk;
    if (shift == 56) w.sel[2] = (uint64_t)K;
    if (n > K) {
      int64_t remaining = (int64_t)w.sel[2];
      int64_t cum = 0;
      int d = 255;
      for (; d > 0; d--) {
        if (cum + w.rhist[d] >= remaining) break;
        cum += w.rhist[d];
      }
      w.sel[2] = (uint64_t)(remaining - cum);
      w.sel[0] |= (uint64_t)d << shift;
      w.sel[1] |= (uint64_t)0xff << shift;
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 256; i += blockDim.x) w.rhist[i] = 0;
}

__global__ void k_radix_pick(Work w, int shift, int K) {
  if (w.st->halt) return;
  radix_pick_part(w, shift, K);
}

__device__ __forceinline__ void apply_part(const Work &w, const Lanes &L) {
  const int ncc = w.cnt->ncc, nmk = w.cnt->nmk;
  const uint64_t th = w.sel[0];
  for (int base = L.base0; base < ncc + nmk; base += L.stride) {
    int c = base + threadIdx.x;
    if (c >= ncc + nmk) break;
    if (c < ncc) {
      if (w.cc.key[c] < th) w.cc.state[c] = kStDone | kStSkip;
      else atomicAdd(&w.cnt->n_kept_cc, 1);
    } else {
      int j = c - ncc;
      if (w.mid.key[j] < th) {
        w.mid.state[j] = kStSkip;
        w.mflag[w.mid.elem[j]] = 0u;
      } else {
        atomicAdd(&w.cnt->n_kept_mid, 1);
      }
    }
  }
}

__global__ void k_apply_cap(Work w) {
  if (w.st->halt) return;
  apply_part(w, grid_lanes());
}

// ---------------------------------------------------------------------------
// R4: locate circumcenters by a visibility walk (Line 6); a walk stopped only
// by subsegments turns into the midpoint candidate of the first one.
// ---------------------------------------------------------------------------
// Returns 1 for a coincident point, 2 for a walk blocked by a subsegment.
// The walk length is kept in bits 16-30 of the state of a located point (at
// most 0x7fff) and added to *nsteps.
constexpr int kStepShift = 16;
__device__ __forceinline__ int locate_one(const DevMesh &m, const Work &w, int c, int nS, int &nsteps) {
  if (w.cc.state[c] & kStSkip) return 0;
  int cur = w.cc.elem[c];
  double2 p = w.cc.p[c];
  for (int steps = 1;; steps++) {
    nsteps++;
    if (steps > (1 << 20)) {
      atomicOr(&w.cnt->err, kErrWalk);
      w.cc.state[c] = kStDone;
      return 0;
    }
    // the neighbours are loaded with the vertices (needed unless p is found here)
    int4 tri = m.tv[cur];
    const int4 nb = m.tn[cur];
    double2 A = m.vxy[tri.x], B = m.vxy[tri.y], C = m.vxy[tri.z];
    int s0 = orient_pts(w, A, B, p), s1 = orient_pts(w, B, C, p), s2 = orient_pts(w, C, A, p);
    if (s0 >= 0 && s1 >= 0 && s2 >= 0) {
      int nz = (s0 == 0) + (s1 == 0) + (s2 == 0);
      if (nz >= 2) {
        w.cc.state[c] = kStDone;
        return 1;
      }
      w.cc.loc[c] = cur;
      w.cc.state[c] = kStFound | (min(steps, 0x7fff) << kStepShift);
      return 0;
    }
    int s[3] = {s0, s1, s2};
    int first_neg = -1, next = -1;
    for (int e = 0; e < 3; e++) {
      if (s[e] >= 0) continue;
      if (first_neg < 0) first_neg = e;
      int o = comp(nb, e);
      if (!((tri.w >> e) & 1) && o >= 0) { next = o; break; }
    }
    if (next < 0) {
      int k = comp(m.ts[cur], first_neg);
      if (k < 0 || k >= nS) {  // a hull edge that is not a subsegment
        atomicOr(&w.cnt->err, kErrInput);
        w.cc.state[c] = kStDone;
        return 0;
      }
      flag_mid(w, k);
      w.cc.state[c] = kStDone;
      return 2;
    }
    cur = next;
  }
}

__device__ __forceinline__ void locate_part(const DevMesh &m, const Work &w, const Lanes &L) {
  const int ncc = w.cnt->ncc, nS = w.st->nS;
  int n_coin = 0, n_blk = 0, n_steps = 0;
  for (int base = L.base0; base < ncc; base += L.stride) {
    int c = base + threadIdx.x;
    if (c < ncc) {
      const int r = locate_one(m, w, c, nS, n_steps);
      n_coin += r == 1;
      n_blk += r == 2;
    }
  }
  stat_add(w, kStCoincident, n_coin);
  stat_add(w, kStBlocked, n_blk);
  stat_add(w, kStOrTests, 3 * (uint64_t)n_steps);
}

__global__ void k_locate(DevMesh m, Work w) {
  if (w.st->halt) return;
  locate_part(m, w, grid_lanes());
}

// ---------------------------------------------------------------------------
// Optional semantic prefilters on located circumcenters.
//   F1 (Line 6): one circumcenter per located triangle, the largest key.
//   F2 (Line 7): the first n triangles of the cavity growth order (seed, then
//   breadth first across non-subsegment edges whose far circumcircle strictly
//   holds the point, edges in index order, stopping as soon as n are taken)
//   are marked with atomicMax; a point that does not hold all of them is
//   dropped.  Marks are cleared before the real cavities are grown.
// mode: 0 F1 mark, 1 F1 filter, 2 F1 clear, 3 F2 mark, 4 F2 filter, 5 F2 clear
// ---------------------------------------------------------------------------
constexpr int kApproxMax = 16;
constexpr int kPreBlock = 128;

__device__ __forceinline__ void prefilter_one(const DevMesh &m, const Work &w, int32_t *lds, int ls, int tid, int c, int mode,
                              int n) {
  int st = w.cc.state[c];
  if (!(st & kStFound)) return;
  int loc = w.cc.loc[c];
  uint64_t key = w.cc.key[c];
  if (mode <= 2) {
    if (mode == 0) {
      if (!(st & kStDone)) atomicMax((unsigned long long *)&w.mark[loc], (unsigned long long)key);
    } else if (mode == 1) {
      if (!(st & kStDone) && w.mark[loc] != key) {
        w.cc.state[c] = st | kStDone;
        atomicAdd(&w.cnt->n_f1_drop, 1);
      }
    } else {
      w.mark[loc] = 0ull;
    }
    return;
  }
  if (mode != 5 && (st & kStDone)) return;
  double2 p = w.cc.p[c];
  int len = 0;
  lds[tid] = loc;
  len = 1;
  for (int h = 0; h < len && len < n; h++) {
    int t = lds[h * ls + tid];
    int4 tri = m.tv[t];
    int4 nb = m.tn[t];
    for (int e = 0; e < 3 && len < n; e++) {
      if ((tri.w >> e) & 1) continue;
      int o = comp(nb, e);
      if (o < 0) continue;
      bool in = false;
      for (int q = 0; q < len; q++)
        if (lds[q * ls + tid] == o) { in = true; break; }
      if (in) continue;
      if (incircle_tri(m, w, m.tv[o], p) > 0) lds[(len++) * ls + tid] = o;
    }
  }
  if (mode == 3) {
    for (int j = 0; j < len; j++)
      atomicMax((unsigned long long *)&w.mark[lds[j * ls + tid]], (unsigned long long)key);
  } else if (mode == 4) {
    bool own = true;
    for (int j = 0; j < len && own; j++) own = w.mark[lds[j * ls + tid]] == key;
    if (!own) {
      w.cc.state[c] = st | kStDone;
      atomicAdd(&w.cnt->n_f2_drop, 1);
    }
  } else {
    for (int j = 0; j < len; j++) w.mark[lds[j * ls + tid]] = 0ull;
  }
}

// lds: kApproxMax slices of blockDim.x entries
__device__ __forceinline__ void prefilter_part(const DevMesh &m, const Work &w, int mode, int n, int32_t *lds, const Lanes &L) {
  const int ncc = w.cnt->ncc;
  for (int base = L.base0; base < ncc; base += L.stride) {
    int c = base + threadIdx.x;
    if (c < ncc) prefilter_one(m, w, lds, blockDim.x, threadIdx.x, c, mode, n);
  }
}

__global__ __launch_bounds__(kPreBlock) void k_prefilter(DevMesh m, Work w, int mode, int n) {
  __shared__ int32_t lds[kApproxMax * kPreBlock];
  if (w.st->halt) return;
  prefilter_part(m, w, mode, n, lds, grid_lanes());
}

// ---------------------------------------------------------------------------
// R5 / R6: Bowyer-Watson cavities, each grown by a group of kGrp lanes; a
// cavity larger than the group's list goes to the cooperative kernel below.
//
// The unit of work is a boundary edge, not a triangle: the queue holds the
// edges of the cavity found so far that have not been tested, and the lanes
// of the group take the next kGrp of them.  A lane tests the triangle across
// its edge; one whose circle holds the point joins the cavity and queues its
// two other edges; any other edge is a boundary edge of the finished cavity.
// The cavity of a point has no vertex inside, so its triangles form a tree
// and every edge is tested once: 2 |C| + 1 edges, in about as many steps as
// the tree is deep.
//
// What bounds it: each step is two dependent levels of gathers (the records
// of the triangle across and the edge's end points, then the far vertex)
// and one FP64 circle test, so a round lasts as long as its longest chain of
// steps until the candidates fill the chip, and then as long as the lines it
// gathers.  One lane per cavity (three circle tests per step, a step per
// triangle, the wave waiting for its largest of 64 cavities) took 4.3 ms of a
// refinement of the benchmark's mesh of 1,000,000 points (30 launches of 144
// us); this takes 2.9 (38 launches of 77).  Eight lanes: most steps of a
// cavity of 8 triangles (the average) keep under eight edges waiting; four
// lanes and twice the cavities took 59 and 124 us a launch on meshes of 50,000
// and 1,000,000 points against 53 and 117.
// ---------------------------------------------------------------------------
constexpr int kGrp = 8;         // lanes per cavity
constexpr int kRing = 64;       // queue entries (at most len + 4 wait at once)
constexpr int kListMax = 56;    // cavity triangles a group can list
constexpr int kGrpWords = 3 * kRing + kListMax;  // LDS of a group; = 56 mod 64 banks, so that the eight
                                                 // groups of a wave start in different banks
constexpr int kCap = kCavCapDefault;
static_assert(kCap <= kListMax && kListMax + 4 <= kRing, "cavity list and queue of a group");
constexpr int kCavBlock = kCavBlockSize;

__device__ __forceinline__ int grp_lane() { return __lane_id() & (kGrp - 1); }
__device__ __forceinline__ int grp_first() { return __lane_id() & ~(kGrp - 1); }
// The lanes of the caller's group for which p holds.
__device__ __forceinline__ unsigned grp_ballot(bool p) {
  return (unsigned)(__ballot(p) >> grp_first()) & ((1u << kGrp) - 1u);
}
// Orders the LDS accesses of a wave's lanes (one wave: the hardware keeps
// them in program order; this keeps the compiler from moving them).
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

struct CavCheck {
  int nbnd;
  bool fan_bad;
  bool enc;
  int ntest;  // incircle evaluations
};

// Grows the cavity of p from the seeds (s1 < 0: one seed) into the group's
// list, S[3 * kRing ..].  Returns the size, or -1 if it exceeds cap or (with
// FILTER) the FP64 filter cannot decide a test: the cavity then goes to the
// cooperative path, which evaluates exactly; this keeps the exact
// evaluations, and the registers and scratch they need, out of the grid
// kernels.  Every value but the list is uniform over the group.
//
// Queue entry: (o, u, v): the edge u -> v of a cavity triangle and the
// triangle o across it, -1 on the hull, or -2 - (4 t + e) for edge e of t
// when it is a subsegment (never crossed).  For each boundary edge: the
// count, the fan orientation (p strictly left of it), and for circumcenters
// an encroached boundary subsegment (all are flagged; a cavity handed over
// has flagged a subset of what the cooperative path flags for it).  The
// split subsegment of a midpoint (skip_k) is not a boundary edge.
template <bool FILTER>
__device__ __forceinline__ int grow_group(const DevMesh &m, const Work &w, int32_t *S, int cap, int s0, int s1,
                                          double2 p, int skip_k, bool is_cc, CavCheck &ck) {
  int32_t *qo = S, *qu = S + kRing, *qv = S + 2 * kRing, *list = S + 3 * kRing;
  const int gl = grp_lane();
  const unsigned below = (1u << gl) - 1u;
  int len = s1 >= 0 && s1 != s0 ? 2 : 1;
  int head = 0, tail = 3 * len;
  ck = CavCheck{0, false, false, 0};
  if (gl < tail) {
    const int t = gl < 3 ? s0 : s1, e = gl < 3 ? gl : gl - 3;
    const int4 tri = m.tv[t];
    const int o = comp(m.tn[t], e);
    qo[gl] = ((tri.w >> e) & 1) ? -2 - (4 * t + e) : (o < 0 ? -1 : o);
    qu[gl] = comp(tri, e);
    qv[gl] = comp(tri, e == 2 ? 0 : e + 1);
  }
  for (int j = 4 * gl; j < kListMax; j += 4 * kGrp)
    *reinterpret_cast<int4 *>(list + j) = make_int4(j == 0 ? s0 : -1, j == 0 && len == 2 ? s1 : -1, -1, -1);
  wave_lds_sync();
  bool stop = false, fan_bad = false, enc = false;  // fan_bad, enc: this lane's
  while (head < tail) {
    // Straight-line code: lanes without an edge repeat the group's last one
    // and an edge without a triangle across reads slot 0 (their results are
    // masked), so a step has no branches but the rare ones.
    const int nrun = min(kGrp, tail - head);
    const bool act = gl < nrun;
    const int qi = (head + min(gl, nrun - 1)) & (kRing - 1);
    const int o = qo[qi], u = qu[qi], v = qv[qi];
    const int oc = max(o, 0);
    const double2 U = m.vxy[u], V = m.vxy[v];
    const int4 to = m.tv[oc], no = m.tn[oc];
    // listed: an internal edge (reached the other way; an edge without a
    // triangle across is none, whatever the list's padding holds)
    bool in = false;
    for (int q = 0; q < len; q += 4) {
      const int4 x = *reinterpret_cast<const int4 *>(list + q);
      in |= (x.x == o) | (x.y == o) | (x.z == o) | (x.w == o);
    }
    in &= o >= 0;
    // far vertex, and its index in the record (the edge is v -> u there)
    const bool f0 = (to.x != u) & (to.x != v), f1 = (to.y != u) & (to.y != v);
    const int fi = f0 ? 0 : (f1 ? 1 : 2);
    const int f = f0 ? to.x : (f1 ? to.y : to.z);
    const double2 F = m.vxy[f];
    // the filters of gdp_exact.h without their branches; the orientation of
    // the edge is one of the circle test's 2x2 minors
    const double fx = F.x - p.x, fy = F.y - p.y, vx = V.x - p.x, vy = V.y - p.y, ux = U.x - p.x, uy = U.y - p.y;
    const double vu1 = vx * uy, vu2 = ux * vy;
    const double uf1 = ux * fy, uf2 = fx * uy;
    const double fv1 = fx * vy, fv2 = vx * fy;
    const double od = vu2 - vu1, op = fabs(vu1) + fabs(vu2), ob = 6.0 * kU * op;
    const double fl = fx * fx + fy * fy, vl = vx * vx + vy * vy, ul = ux * ux + uy * uy;
    const double det = fl * (vu1 - vu2) + vl * (uf1 - uf2) + ul * (fv1 - fv2);
    const double perm = op * fl + (fabs(uf1) + fabs(uf2)) * vl + (fabs(fv1) + fabs(fv2)) * ul;
    const double ib = 12.0 * kU * perm;
    const bool left = (op > kTiny) & (od > ob), right = (op > kTiny) & (-od > ob);
    const bool inside = (perm > kTiny) & (det > ib), outside = (perm > kTiny) & (-det > ib);
    const bool test = act & (o >= 0) & !in;
    bool und = test & !(inside | outside);
    bool acc = test & inside;
    if (!FILTER && und) {
      // (the neighbour's vertices in its own order)
      const double2 A = m.vxy[to.x], B = m.vxy[to.y], C = m.vxy[to.z];
      acc = incircle(A.x, A.y, B.x, B.y, C.x, C.y, p.x, p.y, w.tally) > 0;
      und = false;
    }
    bool bnd = act & !in & !acc;
    if (o <= -2) {
      // a subsegment: the split one is no boundary edge; any other may be
      // encroached by a circumcenter
      const int sid = reinterpret_cast<const int32_t *>(m.ts)[-2 - o];
      if (skip_k >= 0 && sid == skip_k) {
        bnd = false;
      } else if (bnd && is_cc && sid >= 0) {
        int en;
        if (FILTER) {
          en = encroaches_filter(w.enc_mode, U.x, U.y, V.x, V.y, p.x, p.y);
          und |= en == kUndecided;
        } else {
          en = encroached(w, U, V, p) ? 1 : 0;
        }
        if (en == 1) {
          flag_mid(w, sid);
          enc = true;
        }
      }
    }
    const bool o_und = bnd & !(left | right);
    if (FILTER) {
      und |= o_und;
      fan_bad |= bnd & right;
    } else {
      fan_bad |= o_und ? orient_pts(w, U, V, p) <= 0 : (bnd & right);
    }
    ck.ntest += __popc(grp_ballot(test));
    ck.nbnd += __popc(grp_ballot(bnd));
    const unsigned am = grp_ballot(acc);
    int na = __popc(am), r = __popc(am & below);
    stop = (FILTER && grp_ballot(und) != 0) || len + na > cap;
    if (stop) break;
    if (acc) list[len + r] = o;
    wave_lds_sync();
    // two lanes can reach one triangle in the same step: the first one counts
    bool dup = false;
    if (acc)
      for (int k = 0; k < r; k++) dup |= list[len + k] == o;
    if (grp_ballot(dup) != 0) {
      acc = acc && !dup;
      const unsigned am2 = grp_ballot(acc);
      const int na1 = na;
      na = __popc(am2);
      r = __popc(am2 & below);
      wave_lds_sync();
      if (gl < na1) list[len + gl] = -1;
      wave_lds_sync();
      if (acc) list[len + r] = o;
    }
    if (acc) {
      const int e1 = fi, e2 = fi == 0 ? 2 : fi - 1;  // far -> v, u -> far
      const int i1 = (tail + 2 * r) & (kRing - 1), i2 = (i1 + 1) & (kRing - 1);
      const int o1 = max(comp(no, e1), -1), o2 = max(comp(no, e2), -1);
      qo[i1] = ((to.w >> e1) & 1) ? -2 - (4 * o + e1) : o1;
      qu[i1] = f;
      qv[i1] = v;
      qo[i2] = ((to.w >> e2) & 1) ? -2 - (4 * o + e2) : o2;
      qu[i2] = u;
      qv[i2] = f;
    }
    head += nrun;
    tail += 2 * na;
    len += na;
    wave_lds_sync();
  }
  ck.fan_bad = grp_ballot(fan_bad) != 0;
  ck.enc = grp_ballot(enc) != 0;
  return stop ? -1 : len;
}

// Outcome of one group's cavity: alive (cavity left in the group's list),
// dropped (with the counter it feeds) or handed to the cooperative kernel.
struct CavRes {
  int len;        // cavity size when grown (0 otherwise)
  int bnd;        // its boundary edges
  int alive;
  int enc_reject, fan_invalid, unsplittable, mid_cand;
  int ntest;      // incircle evaluations made while growing
  uint64_t key;   // the candidate's (alive)
};

template <bool FILTER>
__device__ __forceinline__ CavRes cavity_one(const DevMesh &m, const Work &w, int32_t *S_lds, int cap, int ci,
                                             int is_cc) {
  CavRes res{0, 0, 0, 0, 0, 0, 0, 0, 0};
  const CandSet &S = is_cc ? w.cc : w.mid;
  const bool lead = grp_lane() == 0;
  int s0 = -1, s1 = -1, skip_k = -1, expect = 2;
  double2 p;
  int st = S.state[ci];
  if (is_cc) {
    // (loaded together; the located triangle is not set unless found)
    s0 = S.loc[ci];
    p = S.p[ci];
    res.key = S.key[ci];
    if ((st & (kStDone | kStSkip | kStBig)) || !(st & kStFound)) return res;
  } else {
    const int k = S.elem[ci];
    if (st & (kStDone | kStSkip | kStBig)) return res;
    res.mid_cand = 1;
    const int a0 = w.sadj[2 * k], a1 = w.sadj[2 * k + 1];  // with the subsegment's record
    const SplitPt r = seg_split(m, k, w.pm, w.split_mode);
    p = make_double2(r.px, r.py);
    res.key = r.key;
    const int2 sk = m.sv[k];
    const double2 A = m.vxy[sk.x], B = m.vxy[sk.y];
    const bool uns = (p.x == A.x && p.y == A.y) || (p.x == B.x && p.y == B.y);
    if (lead) {
      S.key[ci] = r.key;
      S.p[ci] = p;
      if (uns) S.state[ci] = st | kStDone;
    }
    if (uns) {
      res.unsplittable = 1;
      return res;
    }
    s0 = a0 >= 0 ? a0 >> 2 : a1 >> 2;
    s1 = a0 >= 0 && a1 >= 0 ? a1 >> 2 : -1;
    skip_k = k;
    expect = s1 >= 0 ? 2 : 1;
    st |= kStFound;
  }
  CavCheck ck;
  ck = CavCheck{0, false, false, 0};
  // (a subsegment without a triangle on either side has an empty cavity)
  const int len = s0 < 0 ? 0 : grow_group<FILTER>(m, w, S_lds, cap, s0, s1, p, skip_k, is_cc != 0, ck);
  res.ntest = ck.ntest;
  if (len < 0) {
    if (lead) {
      S.state[ci] = st | kStBig | kStFound;
      int q = atomicAdd(&w.cnt->nbig, 1);
      if (q < w.big_cap) w.big[q] = (is_cc ? 0 : (int)0x80000000) | ci;
      else atomicOr(&w.cnt->err, kErrCavity);
    }
    return res;
  }
  res.len = len;
  res.bnd = ck.nbnd;
  const bool rej = is_cc && ck.enc;
  if (rej) res.enc_reject = 1;
  else if (ck.fan_bad || ck.nbnd - len != expect) res.fan_invalid = 1;
  else res.alive = 1;
  if (lead) S.state[ci] = res.alive ? st : (st | kStDone);
  return res;
}

// Pool room for the cavities of a wave (need: the group leaders' sizes, 0 on
// other lanes; all lanes of the wave take part).  Atomics on one address are
// served about 12 ns apart, so a workgroup takes one piece of the pool up
// front (s_pool, chunk_end: LDS, taken by LDS atomics) and a wave that finds
// it empty takes a piece of its own (fb_cur, fb_end), at least `more` long.
__device__ __forceinline__ int pool_take(const Work &w, int need, int *s_pool, int chunk_end, int more, int &fb_cur,
                                         int &fb_end) {
  const int lane = __lane_id();
  int x = need;
  for (int d = kGrp; d < 64; d <<= 1) {
    const int y = __shfl_up(x, d);
    if (lane >= d) x += y;
  }
  const int total = __shfl(x, 64 - kGrp);
  int base = 0;
  if (total > 0) {
    if (chunk_end > 0) {
      if (lane == 0) base = atomicAdd(s_pool, total);
      base = __shfl(base, 0);
    }
    if (base + total > chunk_end) {
      if (total > fb_end - fb_cur) {
        const int take = max(total, more);
        int g = 0;
        if (lane == 0) g = atomicAdd(&w.cnt->pool_used, take);
        fb_cur = __shfl(g, 0);
        fb_end = fb_cur + take;
      }
      base = fb_cur;
      fb_cur += total;
    }
  }
  return base + x - need;
}

// Statistics of a workgroup's cavities, summed in LDS (indexed by StatField)
// and added to its wave's stat line once, after a barrier.
__device__ __forceinline__ void stat_lds_clear(uint32_t *s) {
  for (int f = threadIdx.x; f < kStFields; f += blockDim.x) s[f] = 0;
}
__device__ __forceinline__ void stat_lds_flush(const Work &w, const uint32_t *s) {
  for (int f = threadIdx.x; f < kStFields; f += blockDim.x) {
    const unsigned long long x = s[f];
    if (!x) continue;
    unsigned long long *d = (unsigned long long *)&stat_line(w)->v[f];
    if (f == kStCavMax) atomicMax(d, x);
    else atomicAdd(d, x);
  }
}

// Group cavities of candidates [lo, hi) of one class (hi < 0: to the end of
// the list).  lds: kGrpWords per group; grp: the group's index among those
// that run the loop, ngrp of which take candidates side by side; stat: the
// workgroup's statistics.  The midpoint list is final when this runs for
// midpoints (they are flagged only by the scan, the walk and the
// circumcenter cavities), so its length is read from device memory.  With
// L.blk (grid kernels: every thread of the workgroup runs the loop, which is
// uniform over it) pool space is taken per workgroup.
template <bool FILTER = false>
__device__ __forceinline__ void cavity_part(const DevMesh &m, const Work &w, int is_cc, int32_t *lds, int cap,
                                            uint32_t *stat, int first, int ngrp, int grp, bool blk, int lo = 0,
                                            int hi = -1) {
  __shared__ int s_pool[2];
  const int n = hi >= 0 ? hi : (is_cc ? w.cnt->ncc : w.cnt->nmk);
  const CandSet &S = is_cc ? w.cc : w.mid;
  int32_t *G = lds + grp * kGrpWords;
  const int gl = grp_lane(), g0 = grp_first();
  const int per_blk = blockDim.x / kGrp;
  int chunk_end = 0, fb_cur = 0, fb_end = 0;
  bool have = !blk;
  if (blk && lo + first < n && threadIdx.x == 0) {
    // room for eight triangles per candidate, the usual average, while that
    // leaves a quarter of the pool to the waves' own pieces
    const int iters = (n - lo - first + ngrp - 1) / ngrp;
    const int per = (int)min((int64_t)8, (int64_t)w.pool_cap * 3 / 4 / max(n, 1));
    const int take = iters * per_blk * per;
    const int b = take > 0 ? atomicAdd(&w.cnt->pool_used, take) : 0;
    s_pool[0] = b;
    s_pool[1] = b + take;
  }
  for (int base = lo + first; base < n; base += ngrp) {
    const int ci = base + grp;
    CavRes r{0, 0, 0, 0, 0, 0, 0, 0, 0};
    if (ci < n) r = cavity_one<FILTER>(m, w, G, cap, ci, is_cc);
    if (!have) {
      __syncthreads();
      chunk_end = s_pool[1];
      have = true;
    } else if (!blk) {
      chunk_end = 0;
    }
    const int left = (n - base - 1) / ngrp;  // iterations after this one
    int off = pool_take(w, gl == 0 && r.alive ? r.len : 0, s_pool, chunk_end, min(left, 8) * 64, fb_cur, fb_end);
    off = __shfl(off, g0);
    bool counted = r.len > 0 && !r.alive;  // dropped cavities count in the statistics now
    if (r.alive) {
      if (off + r.len > w.pool_cap) {
        if (gl == 0) atomicOr(&w.cnt->err, kErrPool);  // the round is abandoned and run again
      } else {
        // R8 marks are placed as soon as the cavity is known to be valid:
        // validity depends on this cavity alone, and atomicMax is order free.
        // (The pool keeps the order of growth; the insertion sorts the slots
        // of a winner.)
        for (int j = gl; j < r.len; j += kGrp) {
          const int t = G[3 * kRing + j];
          w.pool[off + j] = t;
          atomicMax((unsigned long long *)&w.mark[t], (unsigned long long)r.key);
        }
        counted = true;
        if (gl == 0) {
          S.off[ci] = off;
          S.len[ci] = r.len;
          S.state[ci] |= kStDone | kStAlive;
        }
      }
    }
    if (gl == 0) {
      if (counted) {
        atomicMax(&stat[kStCavMax], (uint32_t)r.len);
        atomicAdd(&stat[kStCavTri], (uint32_t)r.len);
        if (r.alive) atomicAdd(&stat[is_cc ? kStMarks1 : kStMarks0], (uint32_t)r.len);
      }
      if (r.len) {
        atomicAdd(&stat[is_cc ? kStCavLen1 : kStCavLen0], (uint32_t)r.len);
        atomicAdd(&stat[is_cc ? kStCavBnd1 : kStCavBnd0], (uint32_t)r.bnd);
      }
      if (r.ntest) atomicAdd(&stat[kStInTests], (uint32_t)r.ntest);
      if (r.enc_reject) atomicAdd(&stat[kStEncReject], 1u);
      if (r.fan_invalid) atomicAdd(&stat[kStFanInvalid], 1u);
      if (r.unsplittable) atomicAdd(&stat[kStUnsplittable], 1u);
      if (r.mid_cand) atomicAdd(&stat[kStMidCand], 1u);
    }
  }
}

// One kernel symbol per class (circumcenters: IS_CC = 1), so that profiles
// tell them apart.  cap: a cavity beyond it goes to the cooperative path
// (perf only).
template <int IS_CC>
__device__ __forceinline__ void cavity_grid(const DevMesh &m, const Work &w, int cap, int bx, int nb) {
  __shared__ __attribute__((aligned(16))) int32_t lds[kGrpWords * (kCavBlock / kGrp)];
  __shared__ uint32_t stat[kStFields];
  constexpr int per = kCavBlock / kGrp;
  stat_lds_clear(stat);
  __syncthreads();
  cavity_part<true>(m, w, IS_CC, lds, cap, stat, bx * per, nb * per, (int)threadIdx.x / kGrp, true);
  __syncthreads();
  stat_lds_flush(w, stat);
}
template <int IS_CC>
__global__ __launch_bounds__(kCavBlock, 5) void k_cavity(DevMesh m, Work w, int cap) {
  if (w.st->halt) return;
  cavity_grid<IS_CC>(m, w, cap, (int)blockIdx.x, (int)gridDim.x);
}
template __global__ void k_cavity<0>(DevMesh m, Work w, int cap);
template __global__ void k_cavity<1>(DevMesh m, Work w, int cap);

// Cooperative growth of one large cavity per workgroup (the tuple-parallel
// ExpandList idea of Section 5.3: the frontier of <point, triangle> tuples
// is processed in parallel, new tuples are reserved with atomics).
constexpr int kBigMax = 4096;
constexpr int kHash = 16384;
constexpr int kBigBlock = 256;

__device__ __forceinline__ int hash_insert(int32_t *hs, int v, int *ovf) {
  uint32_t h = ((uint32_t)v * 2654435761u) & (kHash - 1);
  for (int probe = 0; probe < kHash; probe++) {
    int old = atomicCAS(&hs[h], -1, v);
    if (old == -1) return 1;
    if (old == v) return 0;
    h = (h + 1) & (kHash - 1);
  }
  *ovf = 1;
  return 0;
}

struct BigShared {
  int32_t cav[kBigMax];
  int32_t hs[kHash];
  int s_n, s_head, s_ovf, s_nbnd, s_fanbad, s_enc, s_off, s_r;
};

// Ascending sort of a[0..n) by one workgroup: the bitonic network in its
// all-ascending form (each block of size k first compares mirrored pairs,
// then half-cleaners of strides k/4 .. 1; every compare-exchange puts the
// smaller value at the lower index).  Entries beyond n act as +infinity and
// are never touched, so no padding is stored.
__device__ __forceinline__ void block_sort_asc(int32_t *a, int n) {
  int P = 1;
  while (P < n) P <<= 1;
  const int half = P >> 1;
  for (int k = 2; k <= P; k <<= 1) {
    const int hk = k >> 1;
    __syncthreads();
    for (int idx = threadIdx.x; idx < half; idx += blockDim.x) {
      const int blk = idx / hk, o = idx - blk * hk;
      const int i = blk * k + o, l = blk * k + (k - 1 - o);
      if (l < n) {
        const int x = a[i], y = a[l];
        if (x > y) { a[i] = y; a[l] = x; }
      }
    }
    for (int j = k >> 2; j > 0; j >>= 1) {
      __syncthreads();
      for (int idx = threadIdx.x; idx < half; idx += blockDim.x) {
        const int i = (idx / j) * 2 * j + idx % j, l = i + j;
        if (l < n) {
          const int x = a[i], y = a[l];
          if (x > y) { a[i] = y; a[l] = x; }
        }
      }
    }
  }
  __syncthreads();
}

// The rest of a cooperative cavity once its slots are known (cav[0..len),
// any order; LDS or device memory): sort, boundary checks in parallel over
// the cavity triangles, then drop it or take pool space and place its
// marks.  Uniform over the workgroup; the shared scalars are reset here.
__device__ __forceinline__ void coop_finish(const DevMesh &m, const Work &w, BigShared &sh, CandSet S, int ci,
                                            int is_cc, int skip_k, int expect, double2 p, int32_t *cav, int len) {
  const int tid = threadIdx.x;
  if (tid == 0) { sh.s_nbnd = 0; sh.s_fanbad = 0; sh.s_enc = 0; sh.s_off = -1; }
  block_sort_asc(cav, len);
  for (int j = tid; j < len; j += blockDim.x) {
    int t = cav[j];
    int4 tri = m.tv[t];
    int4 nb = m.tn[t];
    int4 ts = tri.w ? m.ts[t] : make_int4(-1, -1, -1, 0);
    for (int e = 0; e < 3; e++) {
      int sid = ((tri.w >> e) & 1) ? comp(ts, e) : -1;
      if (skip_k >= 0 && sid == skip_k) continue;
      int o = comp(nb, e);
      if (sid < 0 && o >= 0 && in_sorted(cav, len, o)) continue;
      atomicAdd(&sh.s_nbnd, 1);
      double2 U = m.vxy[comp(tri, e)], V = m.vxy[comp(tri, (e + 1) % 3)];
      if (is_cc && sid >= 0 && encroached(w, U, V, p)) {
        flag_mid(w, sid);
        sh.s_enc = 1;
      }
      if (orient_pts(w, U, V, p) <= 0) sh.s_fanbad = 1;
    }
  }
  __syncthreads();
  if (tid == 0) {
    atomicAdd((unsigned long long *)&stat_line(w)->v[kStOrTests], (unsigned long long)sh.s_nbnd);
    bool drop = (is_cc && sh.s_enc) || sh.s_fanbad || sh.s_nbnd - len != expect;
    if (drop) {
      atomicAdd((unsigned long long *)&w.cnt->cav_tri_total, (unsigned long long)len);
      atomicMax(&w.cnt->cav_max, len);
      atomicAdd((is_cc && sh.s_enc) ? &w.cnt->n_enc_reject : &w.cnt->n_fan_invalid, 1);
      S.state[ci] |= kStDone;
    } else {
      int off = atomicAdd(&w.cnt->pool_used, len);
      if (off + len > w.pool_cap) atomicOr(&w.cnt->err, kErrPool);
      else {
        sh.s_off = off;
        atomicAdd((unsigned long long *)&w.cnt->cav_tri_total, (unsigned long long)len);
        atomicMax(&w.cnt->cav_max, len);
      }
    }
  }
  __syncthreads();
  int off = sh.s_off;
  if (off >= 0) {
    uint64_t key = S.key[ci];
    for (int j = tid; j < len; j += blockDim.x) {
      w.pool[off + j] = cav[j];
      atomicMax((unsigned long long *)&w.mark[cav[j]], (unsigned long long)key);
    }
    if (tid == 0) {
      atomicAdd((unsigned long long *)&stat_line(w)->v[is_cc ? kStMarks1 : kStMarks0], (unsigned long long)len);
      S.off[ci] = off;
      S.len[ci] = len;
      S.state[ci] |= kStDone | kStAlive;
    }
  }
  __syncthreads();
}

// Candidate of queue entry b and its growth parameters.
struct CoopCand {
  CandSet S;
  int ci, is_cc, skip_k, expect;
  double2 p;
};
__device__ __forceinline__ CoopCand coop_cand(const Work &w, int b) {
  CoopCand c;
  const int ref = w.big[b];
  c.is_cc = (ref & 0x80000000) ? 0 : 1;
  c.ci = ref & 0x7fffffff;
  c.S = c.is_cc ? w.cc : w.mid;
  c.p = c.S.p[c.ci];
  c.skip_k = c.is_cc ? -1 : c.S.elem[c.ci];
  c.expect = c.is_cc ? 2 : ((w.sadj[2 * c.skip_k] >= 0 && w.sadj[2 * c.skip_k + 1] >= 0) ? 2 : 1);
  return c;
}

// Grows queue entry b (uniform over the workgroup) in LDS: the tuple-
// parallel ExpandList of Section 5.3 (Algorithm 3): the frontier of
// <point, triangle> tuples is expanded in parallel and new tuples are
// reserved with an atomic counter.  A cavity beyond the LDS list (kBigMax
// triangles) continues in device memory (huge_one); when the round was
// started without that path, the round is abandoned and run again with it.
__device__ __forceinline__ void big_one(const DevMesh &m, const Work &w, BigShared &sh, int b) {
  int32_t *cav = sh.cav;
  int32_t *hs = sh.hs;
  int tid = threadIdx.x;
  const int ci0 = w.big[b] & 0x7fffffff;
  const CandSet S0 = (w.big[b] & 0x80000000) ? w.mid : w.cc;
  if (!(S0.state[ci0] & kStBig) || (S0.state[ci0] & (kStDone | kStHuge))) return;
  const CoopCand c = coop_cand(w, b);
  for (int i = tid; i < kHash; i += blockDim.x) hs[i] = -1;
  __syncthreads();
  if (tid == 0) {
    sh.s_n = 0; sh.s_head = 0; sh.s_ovf = 0;
    if (c.is_cc) {
      int t = c.S.loc[c.ci];
      hash_insert(hs, t, &sh.s_ovf);
      cav[sh.s_n++] = t;
    } else {
      int a0 = w.sadj[2 * c.skip_k], a1 = w.sadj[2 * c.skip_k + 1];
      if (a0 >= 0 && hash_insert(hs, a0 >> 2, &sh.s_ovf)) cav[sh.s_n++] = a0 >> 2;
      if (a1 >= 0 && hash_insert(hs, a1 >> 2, &sh.s_ovf)) cav[sh.s_n++] = a1 >> 2;
    }
  }
  __syncthreads();
  for (;;) {
    int lo = sh.s_head, hi = sh.s_n < kBigMax ? sh.s_n : kBigMax;
    int ovf = sh.s_ovf;
    __syncthreads();
    if (lo >= hi || ovf) break;
    if (tid == 0) sh.s_head = hi;
    for (int idx = lo + tid; idx < hi; idx += blockDim.x) {
      int t = cav[idx];
      int4 tri = m.tv[t];
      int4 nb = m.tn[t];
      for (int e = 0; e < 3; e++) {
        if ((tri.w >> e) & 1) continue;
        int o = comp(nb, e);
        if (o < 0) continue;
        if (!hash_insert(hs, o, &sh.s_ovf)) continue;
        atomicAdd((unsigned long long *)&stat_line(w)->v[kStInTests], 1ull);
        if (incircle_tri(m, w, m.tv[o], c.p) > 0) {
          int pos = atomicAdd(&sh.s_n, 1);
          if (pos < kBigMax) cav[pos] = o;
          else sh.s_ovf = 1;
        }
      }
    }
    __syncthreads();
  }
  if (sh.s_ovf) {
    if (tid == 0) {
      if (w.huge_ok) {
        c.S.state[c.ci] |= kStHuge;
        atomicAdd(&w.cnt->nhuge, 1);
      } else {
        atomicOr(&w.cnt->err, kErrHuge);
      }
    }
    __syncthreads();
    return;
  }
  coop_finish(m, w, sh, c.S, c.ci, c.is_cc, c.skip_k, c.expect, c.p, cav, sh.s_n);
}

// A cavity beyond the LDS list, grown by one workgroup in device memory
// with no ceiling (the mesh's triangle count bounds it): the frontier and
// the cavity list live in w.hlist (accepted slots from the bottom, slots
// that failed the circle test from the top; every slot enters at most
// once), visited slots are flagged in w.hvis and cleared again at the end.
// Only one workgroup of a mesh runs this at a time (the flags are shared).
__device__ __noinline__ void huge_one(const DevMesh &m, const Work &w, BigShared &sh, int b) {
  const int tid = threadIdx.x;
  const int ci0 = w.big[b] & 0x7fffffff;
  const CandSet S0 = (w.big[b] & 0x80000000) ? w.mid : w.cc;
  if (!(S0.state[ci0] & kStHuge) || (S0.state[ci0] & kStDone)) return;
  const CoopCand c = coop_cand(w, b);
  int32_t *list = w.hlist;
  const int top = w.hcap - 1;
  if (tid == 0) {
    sh.s_n = 0; sh.s_head = 0; sh.s_r = 0;
    if (c.is_cc) {
      int t = c.S.loc[c.ci];
      w.hvis[t] = 1;
      list[sh.s_n++] = t;
    } else {
      int a0 = w.sadj[2 * c.skip_k], a1 = w.sadj[2 * c.skip_k + 1];
      if (a0 >= 0 && atomicExch(&w.hvis[a0 >> 2], 1) == 0) list[sh.s_n++] = a0 >> 2;
      if (a1 >= 0 && atomicExch(&w.hvis[a1 >> 2], 1) == 0) list[sh.s_n++] = a1 >> 2;
    }
  }
  __syncthreads();
  for (;;) {
    int lo = sh.s_head, hi = sh.s_n;
    __syncthreads();
    if (lo >= hi) break;
    if (tid == 0) sh.s_head = hi;
    for (int idx = lo + tid; idx < hi; idx += blockDim.x) {
      int t = list[idx];
      int4 tri = m.tv[t];
      int4 nb = m.tn[t];
      for (int e = 0; e < 3; e++) {
        if ((tri.w >> e) & 1) continue;
        int o = comp(nb, e);
        if (o < 0) continue;
        if (atomicExch(&w.hvis[o], 1) != 0) continue;
        atomicAdd((unsigned long long *)&stat_line(w)->v[kStInTests], 1ull);
        if (incircle_tri(m, w, m.tv[o], c.p) > 0) list[atomicAdd(&sh.s_n, 1)] = o;
        else list[top - atomicAdd(&sh.s_r, 1)] = o;
      }
    }
    __syncthreads();
  }
  const int len = sh.s_n, nrej = sh.s_r;
  __syncthreads();
  // every visited slot is flagged: clear the flags for the next cavity
  for (int j = tid; j < len; j += blockDim.x) w.hvis[list[j]] = 0;
  for (int j = tid; j < nrej; j += blockDim.x) w.hvis[list[top - j]] = 0;
  coop_finish(m, w, sh, c.S, c.ci, c.is_cc, c.skip_k, c.expect, c.p, list, len);
}

// Large cavities of one class (phase 0: circumcenters, 1: midpoints); the
// workgroups stride over the queue.
__global__ __launch_bounds__(kBigBlock) void k_cavity_big(DevMesh m, Work w, int phase) {
  __shared__ BigShared sh;
  if (w.st->halt) return;
  int nbig = min(w.cnt->nbig, w.big_cap);
  for (int b = blockIdx.x; b < nbig; b += gridDim.x) {
    int ref = w.big[b];
    int is_cc = (ref & 0x80000000) ? 0 : 1;
    if (is_cc != (phase == 0 ? 1 : 0)) continue;
    big_one(m, w, sh, b);
    __syncthreads();
  }
}

// Cavities of one class that outgrew the LDS list, one after the other by
// a single workgroup (launched only on meshes that have needed it).
__global__ __launch_bounds__(kHugeBlock) void k_cavity_huge(DevMesh m, Work w, int phase) {
  __shared__ BigShared sh;
  if (w.st->halt || w.cnt->nhuge == 0) return;
  int nbig = min(w.cnt->nbig, w.big_cap);
  for (int b = 0; b < nbig; b++) {
    int ref = w.big[b];
    int is_cc = (ref & 0x80000000) ? 0 : 1;
    if (is_cc != (phase == 0 ? 1 : 0)) continue;
    huge_one(m, w, sh, b);
  }
}

// ---------------------------------------------------------------------------
// R8: priority marks and ownership
// ---------------------------------------------------------------------------
// Loop bodies that load a few records and then use them are written as
// batches: all loads of a batch are issued before any result is needed
// (the stores in between would otherwise keep the compiler from hoisting
// them), which turns a chain of dependent memory latencies into a few.
constexpr int kIlp = 8;

__device__ __forceinline__ bool cand_at(const Work &w, int c, int ncc, CandSet &S, int &ci, int &is_cc) {
  if (c < ncc) { S = w.cc; ci = c; is_cc = 1; return true; }
  S = w.mid; ci = c - ncc; is_cc = 0; return true;
}

// Fresh slots of a winner: two, or one for a midpoint on a hull subsegment.
__device__ __forceinline__ int fresh_of(const Work &w, int is_cc, int e) {
  if (is_cc) return 2;
  return (w.sadj[2 * e] >= 0 && w.sadj[2 * e + 1] >= 0) ? 2 : 1;
}

// Whether candidate c holds every mark of its cavity (lost: it was judged and
// does not).
__device__ __forceinline__ bool own_one(const Work &w, int c, int ncc, int &lost) {
  CandSet S;
  int ci, is_cc;
  cand_at(w, c, ncc, S, ci, is_cc);
  int st = S.state[ci];
  if (!(st & kStAlive)) return false;
  uint64_t key = S.key[ci];
  int off = S.off[ci], len = S.len[ci];
  // independent loads, kIlp slots at a time (the marks are tested after)
  bool own = true;
  for (int j0 = 0; j0 < len && own; j0 += kIlp) {
    int t[kIlp];
    uint64_t mk[kIlp];
#pragma unroll
    for (int i = 0; i < kIlp; i++) t[i] = j0 + i < len ? w.pool[off + j0 + i] : -1;
#pragma unroll
    for (int i = 0; i < kIlp; i++) mk[i] = t[i] >= 0 ? w.mark[t[i]] : key;
#pragma unroll
    for (int i = 0; i < kIlp; i++) own = own && mk[i] == key;
  }
  if (own) {
    S.state[ci] = st | kStW0;
    bit_set(is_cc ? w.w0_t : w.w0_s, S.elem[ci]);
  } else {
    lost++;
  }
  return own;
}

// The owners go to a list, so that the later phases run over them alone (a
// quarter of the candidates of a large round).  A thread of a large round
// judges several candidates before list space is taken, which keeps the
// atomics on the one counter few.
constexpr int kOwnPer = 4;
__device__ __forceinline__ void own_part(const Work &w, const Lanes &L) {
  const int ncc = w.cnt->ncc, n = ncc + w.cnt->nmk;
  const int per = L.blk && n > 65536 ? kOwnPer : 1;
  int n_lost = 0;
  for (int base = L.base0 * per; base < n; base += L.stride * per) {
    unsigned own = 0;
    for (int k = 0; k < per; k++) {
      const int c = base + k * (int)blockDim.x + (int)threadIdx.x;
      if (c < n && own_one(w, c, ncc, n_lost)) own |= 1u << k;
    }
    int off = group_alloc(&w.cnt->nw0, __popc(own), L);
    for (int k = 0; k < per; k++) {
      if (!((own >> k) & 1u)) continue;
      const int c = base + k * (int)blockDim.x + (int)threadIdx.x;
      w.w0_list[off++] = c < ncc ? c : ((int)0x80000000 | (c - ncc));
    }
  }
  stat_add(w, kStLostMark, n_lost);
}

__global__ void k_own(Work w) {
  if (w.st->halt) return;
  own_part(w, grid_lanes());
}

// The insertion phases give each owner (then each winner) a group of kGrp
// lanes, one cavity triangle or fan record per lane: their loads are a few
// dependent levels whatever the cavity's size (one thread per owner walked
// its cavity two triangles at a time: k_dep 33, k_record 45, k_write 87 us
// per round at 50,000 points, for a few thousand winners as for 100,000).
struct GrpLanes {
  int first, stride, grp;  // list entries first + grp, + stride, ...
};
__device__ __forceinline__ GrpLanes grp_lanes(const Lanes &L) {
  return {L.base0 / kGrp, L.stride / kGrp, (int)threadIdx.x / kGrp};
}
__device__ __forceinline__ const CandSet &cand_ref(const Work &w, int ref, int &ci, int &is_cc) {
  is_cc = (ref & 0x80000000) ? 0 : 1;
  ci = ref & 0x7fffffff;
  return is_cc ? w.cc : w.mid;
}

// R9: Delaunay dependency across a shared non-subsegment cavity edge, the
// lanes of a group over the cavity's triangles.  Returns true if the
// candidate is dropped (uniform over the group).
__device__ __forceinline__ bool dep_one(const DevMesh &m, const Work &w, int ref, int &ntest) {
  int ci, is_cc;
  const CandSet &S = cand_ref(w, ref, ci, is_cc);
  const int gl = grp_lane();
  const uint64_t key = S.key[ci];
  const double2 p = S.p[ci];
  const int off = S.off[ci], len = S.len[ci], st = S.state[ci], elem = S.elem[ci];
  bool drop = false;
  for (int j = gl; j < ((len + kGrp - 1) & ~(kGrp - 1)); j += kGrp) {
    bool hit = false;
    if (j < len) {
      const int t = w.pool[off + j];
      const int4 tri = m.tv[t], nb = m.tn[t];
      const int4 ts = tri.w ? m.ts[t] : make_int4(-1, -1, -1, 0);
      uint64_t mo[3];
#pragma unroll
      for (int e = 0; e < 3; e++) {
        // subsegment edges (incl. the split one) and hull edges have no owner across
        const int o = comp(nb, e);
        const bool sub = ((tri.w >> e) & 1) && comp(ts, e) >= 0;
        mo[e] = (!sub && o >= 0) ? w.mark[o] : 0ull;
      }
#pragma unroll
      for (int e = 0; e < 3; e++) {
        // inside this cavity, unclaimed, or the other is the lower key (only
        // the lower key of a dependent pair drops)
        if (mo[e] == key || mo[e] == 0 || !(key < mo[e])) continue;
        const int q_cc = (mo[e] >> 63) ? 0 : 1;
        const int qid = (int)perm32_inv((uint32_t)(mo[e] & 0xffffffffu));
        if (!bit_get(q_cc ? w.w0_t : w.w0_s, qid)) continue;
        const double2 q = q_cc ? w.cc.p[w.cidx_t[qid]] : w.mid.p[w.cidx_s[qid]];
        const double2 U = m.vxy[comp(tri, e)], V = m.vxy[comp(tri, e == 2 ? 0 : e + 1)];
        ntest++;
        hit |= incircle(U.x, U.y, V.x, V.y, p.x, p.y, q.x, q.y, w.tally) > 0;
      }
    }
    drop = grp_ballot(hit) != 0;
    if (drop) break;
  }
  if (!drop && gl == 0) {
    S.state[ci] = st | kStWin;
    bit_set(is_cc ? w.win_t : w.win_s, elem);
    if (!is_cc && fresh_of(w, 0, elem) == 1) bit_set(w.win_h, elem);
  }
  return drop;
}

__device__ __forceinline__ void dep_part(const DevMesh &m, const Work &w, const Lanes &L) {
  const int n = w.cnt->nw0;
  const GrpLanes g = grp_lanes(L);
  int n_drop = 0, ntest = 0;
  for (int i = g.first + g.grp; i < n; i += g.stride)
    if (dep_one(m, w, w.w0_list[i], ntest) && grp_lane() == 0) n_drop++;
  stat_add2(w, kStDepDrop, kStInTests, n_drop, ntest);
}

__global__ void k_dep(DevMesh m, Work w) {
  if (w.st->halt) return;
  dep_part(m, w, grid_lanes());
}

// ---------------------------------------------------------------------------
// Prefix sums (block scan + scan of block sums + add)
// ---------------------------------------------------------------------------
constexpr int kScanBlock = 256;
constexpr int kScanItems = 8;
constexpr int kScanTile = kScanBlock * kScanItems;
static_assert(kScanTile == kScanTileSize, "scan tile size shared with the host and the readers");

// Exclusive scan over a workgroup of up to 1024 threads.
__device__ __forceinline__ int block_excl_scan(int v, int *total) {
  __shared__ int warp_sums[16];
  int lane = __lane_id(), wid = threadIdx.x / 64;
  // inclusive wave scan
  int x = v;
  for (int d = 1; d < 64; d <<= 1) {
    int y = __shfl_up(x, d);
    if (lane >= d) x += y;
  }
  if (lane == 63) warp_sums[wid] = x;
  __syncthreads();
  if (threadIdx.x == 0) {
    int run = 0;
    for (int i = 0; i < (int)(blockDim.x / 64); i++) {
      int s = warp_sums[i];
      warp_sums[i] = run;
      run += s;
    }
    *total = run;
  }
  __syncthreads();
  int r = x - v + warp_sums[wid];
  __syncthreads();
  return r;
}

// Exclusive scans in two launches: per-tile scans (the workgroups stride
// over the tiles of one to three jobs), then one workgroup per job scans the
// tile totals in place.  A reader adds the tile prefix itself:
// value(i) = out[i] + tiles[i / kScanTile].
__device__ void scan_tile(const ScanJob &j, int n, int tile) {
  __shared__ int s_total;
  int base = tile * kScanTile + threadIdx.x * kScanItems;
  int v[kScanItems];
  int sum = 0;
  for (int i = 0; i < kScanItems; i++) {
    int idx = base + i;
    int x = idx < n ? j.in[idx] : 0;
    if (j.mode == 1) x = __popc((uint32_t)x);
    v[i] = x;
    sum += x;
  }
  int excl = block_excl_scan(sum, &s_total);
  for (int i = 0; i < kScanItems; i++) {
    int idx = base + i;
    if (idx < n) j.out[idx] = excl;
    excl += v[i];
  }
  if (threadIdx.x == 0) j.tiles[tile] = s_total;
  __syncthreads();
}

__device__ __forceinline__ void scan_tiles(const ScanJobs &J) {
  int t[3], n[3];
  for (int k = 0; k < 3; k++) {
    n[k] = J.j[k].in ? *J.j[k].n_dev : 0;
    t[k] = (n[k] + kScanTile - 1) / kScanTile;
  }
  for (int tile = blockIdx.x; tile < t[0] + t[1] + t[2]; tile += gridDim.x) {
    if (tile < t[0]) scan_tile(J.j[0], n[0], tile);
    else if (tile < t[0] + t[1]) scan_tile(J.j[1], n[1], tile - t[0]);
    else scan_tile(J.j[2], n[2], tile - t[0] - t[1]);
  }
}

__global__ __launch_bounds__(kScanBlock) void k_scan_tiles(ScanJobs J, const int32_t *halt) {
  if (*halt) return;
  scan_tiles(J);
}

// One workgroup per job.
__device__ __forceinline__ void scan_sums(const ScanJob &j) {
  __shared__ int s_total;
  if (!j.in) return;
  const int ntiles = (*j.n_dev + kScanTile - 1) / kScanTile;
  int carry = 0;
  for (int start = 0; start < ntiles; start += kScanBlock) {
    int idx = start + threadIdx.x;
    int x = idx < ntiles ? j.tiles[idx] : 0;
    int e = block_excl_scan(x, &s_total);
    if (idx < ntiles) j.tiles[idx] = e + carry;
    carry += s_total;
    __syncthreads();
  }
  if (threadIdx.x == 0) *j.total = carry;
}

__global__ __launch_bounds__(kScanBlock) void k_scan_sums(ScanJobs J, const int32_t *halt) {
  if (*halt) return;
  scan_sums(blockIdx.x == 0 ? J.j[0] : (blockIdx.x == 1 ? J.j[1] : J.j[2]));
}

// ---------------------------------------------------------------------------
// R10: insertion
// ---------------------------------------------------------------------------
__device__ __forceinline__ bool owner_wins(const Work &w, uint64_t mo) {
  if (mo == 0) return false;
  int q_cc = (mo >> 63) ? 0 : 1;
  int qid = (int)perm32_inv((uint32_t)(mo & 0xffffffffu));
  return bit_get(q_cc ? w.win_t : w.win_s, qid);
}

// Fan records of a winner: boundary edges in canonical order (cavity slots
// ascending, edge index 0..2; the split subsegment is skipped).  The j-th fan
// triangle takes the j-th cavity slot, then fresh slots.  The lanes of the
// group take one cavity triangle each; a lane's place among the records is
// the boundary edges of the lanes below.  sl: kSortMax LDS words of the
// group; a cavity of at most kSortMax slots is sorted there (rank by
// counting), a larger one is in the pool in ascending order (the cooperative
// paths sort).
constexpr int kSortMax = 64;
static_assert(kListMax <= kSortMax, "cavities of the lane groups are sorted by the insertion");
__device__ __forceinline__ void record_one(const DevMesh &m, const Work &w, int32_t *sl, int ref, int foff, int fresh,
                                           int fresh_base) {
  int ci, is_cc;
  const CandSet &S = cand_ref(w, ref, ci, is_cc);
  const int gl = grp_lane();
  const unsigned below = (1u << gl) - 1u;
  const uint64_t key = S.key[ci];
  const int off = S.off[ci], len = S.len[ci];
  const int skip_k = is_cc ? -1 : S.elem[ci];
  const int b = len + fresh;
  const bool lds = len <= kSortMax;
  if (lds) {
    int x[kSortMax / kGrp];
#pragma unroll
    for (int i = 0; i < kSortMax / kGrp; i++) {
      const int j = i * kGrp + gl;
      x[i] = j < len ? w.pool[off + j] : 0x7fffffff;
      if (i * kGrp < ((len + 3) & ~3)) sl[j] = x[i];
    }
    wave_lds_sync();
    int r[kSortMax / kGrp];
#pragma unroll
    for (int i = 0; i < kSortMax / kGrp; i++) {
      r[i] = 0;
      if (i * kGrp >= len) continue;
      for (int q = 0; q < len; q += 4) {
        const int4 y = *reinterpret_cast<const int4 *>(sl + q);
        r[i] += (y.x < x[i]) + (y.y < x[i]) + (y.z < x[i]) + (y.w < x[i]);
      }
    }
    wave_lds_sync();
#pragma unroll
    for (int i = 0; i < kSortMax / kGrp; i++)
      if (i * kGrp + gl < len) sl[r[i]] = x[i];
    wave_lds_sync();
  }
  int jbase = 0;
  for (int q0 = 0; q0 < len; q0 += kGrp) {
    const int q = q0 + gl;
    const bool v = q < len;
    const int t = v ? (lds ? sl[q] : w.pool[off + q]) : 0;
    const int4 tri = m.tv[t], nb = m.tn[t];
    const int4 ts = tri.w ? m.ts[t] : make_int4(-1, -1, -1, 0);
    uint64_t mk[3];
    int4 to[3];
#pragma unroll
    for (int e = 0; e < 3; e++) {
      const int o = max(comp(nb, e), 0);
      mk[e] = w.mark[o];
      to[e] = m.tv[o];
    }
    bool bnd[3];
    int before = 0, total = 0;
#pragma unroll
    for (int e = 0; e < 3; e++) {
      const int sid = ((tri.w >> e) & 1) ? comp(ts, e) : -1;
      const bool inner = sid < 0 && comp(nb, e) >= 0 && mk[e] == key;
      bnd[e] = v && !inner && !(skip_k >= 0 && sid == skip_k);
      const unsigned bm = grp_ballot(bnd[e]);
      before += __popc(bm & below);
      total += __popc(bm);
    }
    int j = jbase + before;
#pragma unroll
    for (int e = 0; e < 3; e++) {
      if (!bnd[e]) continue;
      const int sid = ((tri.w >> e) & 1) ? comp(ts, e) : -1;
      const int o = comp(nb, e), u = comp(tri, e), vv = comp(tri, e == 2 ? 0 : e + 1);
      const int jn = o < 0 ? -1 : ((to[e].x == vv && to[e].y == u) ? 0 : ((to[e].y == vv && to[e].z == u) ? 1 : 2));
      if (j < b) {  // always, for a cavity that passed the boundary count check
        const int slot = j < len ? (lds ? sl[j] : w.pool[off + j]) : fresh_base + (j - len);
        w.fan[foff + j] = FanRec{slot, u, vv, o, jn, sid};
        w.repl[t * 4 + e] = slot;
      }
      j++;
    }
    jbase += total;
  }
  if (jbase != b && gl == 0) {
    atomicOr(&w.cnt->err, kErrCavity);
    if (atomicCAS(&w.cnt->dbg_set, 0, 1) == 0) {
      w.cnt->dbg[0] = is_cc;
      w.cnt->dbg[1] = S.elem[ci];
      w.cnt->dbg[2] = len;
      w.cnt->dbg[3] = b;
      w.cnt->dbg[4] = jbase;
      w.cnt->dbg[5] = S.state[ci];
    }
  }
}

// Ranks, fan offsets and fan records of the winners.  Winner ranks: midpoints
// by subsegment id, then circumcenters by slot (from the scanned winner
// bitmaps; RANKED: engine_rank has set them).  Fresh slots are given out in
// rank order, two per winner and one per midpoint on the hull, so their
// prefix at rank r is 2 r less the hull midpoints before it.
// The capacity check of the round comes first: every thread evaluates it on
// the same counts; if anything would overflow, the round is abandoned before
// the mesh is written and the host grows the buffers and runs it again.
// A workgroup takes a tile of the list: one thread per entry for the ranks
// and the fan space (one atomic per tile), then one group per entry.  Tiles
// are small while the list is, so that every group of a small round has at
// most a few entries.  lds: kSortMax words per group.
template <bool RANKED>
__device__ __forceinline__ void record_part(const DevMesh &m, const Work &w, int32_t *lds, const Lanes &L) {
  const DevState *st = w.st;
  DevCounters *c = w.cnt;
  const int nwin_mid = c->nwin_mid, nwin = nwin_mid + c->nwin_cc, n_hull = c->nwin_hull, nw0 = c->nw0;
  const int nT = st->nT, fresh_all = 2 * nwin - n_hull;
  // (the winners' cavities are disjoint)
  const int64_t need_fan = (int64_t)min(c->pool_used, nT) + 2 * (int64_t)nwin;
  const bool over = (c->err & (kErrPool | kErrHuge)) || (int64_t)st->nV + nwin > m.capV ||
                    (int64_t)nT + fresh_all > m.capT || (int64_t)st->nS + nwin_mid > m.capS ||
                    need_fan > w.fan_cap || nwin + 1 > w.win_cap;
  if (first_lane(L)) {
    c->nwin = nwin;
    c->fresh_total = fresh_all;
    c->abort = over ? 1 : 0;
  }
  if (over) return;
  const int per = (int)blockDim.x / kGrp, nblk = L.stride / (int)blockDim.x;
  const int tile = min((int)blockDim.x, max(1, (nw0 / nblk + per - 1) / per) * per);
  for (int base = L.base0 / (int)blockDim.x * tile; base < nw0; base += nblk * tile) {
    const int n = min(tile, nw0 - base);
    int b = 0, len = 0, steps = 0, cc = 0;
    const int i = base + (int)threadIdx.x;
    int r = -1, fb = 0;
    if ((int)threadIdx.x < n) {
      int ci;
      const CandSet &S = cand_ref(w, w.w0_list[i], ci, cc);
      const int state = S.state[ci];
      if (state & kStWin) {
        const int e = S.elem[ci];
        len = S.len[ci];
        if (RANKED) {
          r = w.win_rank[i];
          fb = w.win_fresh[i];
        } else if (cc) {
          r = nwin_mid + bit_rank(w.win_t, w.rank_t, w.tiles_t, e);
          fb = 2 * r - n_hull;
        } else {
          r = bit_rank(w.win_s, w.rank_s, w.tiles_s, e);
          fb = 2 * r - bit_rank(w.win_h, w.rank_h, w.tiles_h, e);
        }
        b = len + fresh_of(w, cc, e);
        if (cc) steps = (state >> kStepShift) & 0x7fff;
      }
    }
    const int foff = group_alloc(&c->fan_used, b, L);
    if ((int)threadIdx.x < n) {
      w.win_rank[i] = r;
      w.win_fresh[i] = fb;
      w.fan_off[i] = foff;
      w.fan_len[i] = b;
    }
    // the winners' share of the round's memory work (winners' cavities are
    // disjoint, so a wave's sums of sizes and fan edges stay below 2^32)
    stat_add2(w, kStWinCav, kStWinBnd, len, b);
    stat_add2(w, kStWinCcCav, kStWinCcBnd, cc ? len : 0, cc ? b : 0);
    stat_add(w, kStWinSteps, steps);
    __syncthreads();
    for (int q = (int)threadIdx.x / kGrp; q < n; q += per) {
      const int k = base + q;
      if (w.win_rank[k] < 0) continue;
      int ci, is_cc;
      const int ref = w.w0_list[k];
      const CandSet &S = cand_ref(w, ref, ci, is_cc);
      record_one(m, w, lds + (int)threadIdx.x / kGrp * kSortMax, ref, w.fan_off[k], w.fan_len[k] - S.len[ci],
                 nT + w.win_fresh[k]);
    }
    __syncthreads();
  }
}

__global__ void k_record(DevMesh m, Work w) {
  extern __shared__ __attribute__((aligned(16))) int32_t dyn_lds[];
  if (w.st->halt) return;
  record_part<false>(m, w, dyn_lds, grid_lanes());
}

// Inserts the winner of list entry k, a fan record per lane.  The neighbours
// inside the fan are the records that start where this one ends and end
// where it starts: found among the fan's (u, v) in LDS (lu, lv, ls: kFanMax
// words each), or in memory for a larger fan.
constexpr int kFanMax = 72;
__device__ __forceinline__ void write_one(const DevMesh &m, const Work &w, int32_t *lds, int k, int nV, int nS,
                                          int serial) {
  int32_t *lu = lds, *lv = lds + kFanMax, *ls = lds + 2 * kFanMax;
  const int gl = grp_lane();
  const int r = w.win_rank[k], foff = w.fan_off[k], b = w.fan_len[k];
  int ci, is_cc;
  const CandSet &S = cand_ref(w, w.w0_list[k], ci, is_cc);
  if (r < 0) return;
  const FanRec f0 = w.fan[foff + min(gl, b - 1)];
  const double2 p = S.p[ci];
  const int pid = nV + r;
  int seg = -1, knew = -1, sa = -1, sb = -1;
  if (!is_cc) {
    seg = S.elem[ci];
    knew = nS + r;  // midpoint winners take ranks 0..nwin_mid-1
    const int2 sk = m.sv[seg];
    sa = sk.x;
    sb = sk.y;
  }
  const bool in_lds = b <= kFanMax;
  if (in_lds) {
    const int bp = (b + 3) & ~3;
    for (int j = gl; j < bp; j += kGrp) {
      const FanRec f = j < kGrp ? f0 : w.fan[foff + min(j, b - 1)];
      lu[j] = j < b ? f.u : -2;
      lv[j] = j < b ? f.v : -2;
      ls[j] = f.slot;
    }
    wave_lds_sync();
  }
  for (int j = gl; j < b; j += kGrp) {
    const FanRec f = j < kGrp ? f0 : w.fan[foff + j];
    const int s = f.slot;
    int n0 = -1;
    if (f.o >= 0) {
      const uint64_t mo = w.mark[f.o];
      if (owner_wins(w, mo)) {
        n0 = w.repl[f.o * 4 + f.jn];
      } else {
        n0 = f.o;
        ((int32_t *)m.tn)[f.o * 4 + f.jn] = s;
      }
    }
    int n1 = -1, n2 = -1;
    if (in_lds) {
      int i1 = -1, i2 = -1;
      for (int g = 0; g < b; g += 4) {
        const int4 x = *reinterpret_cast<const int4 *>(lu + g), y = *reinterpret_cast<const int4 *>(lv + g);
        i1 = x.x == f.v ? g : (x.y == f.v ? g + 1 : (x.z == f.v ? g + 2 : (x.w == f.v ? g + 3 : i1)));
        i2 = y.x == f.u ? g : (y.y == f.u ? g + 1 : (y.z == f.u ? g + 2 : (y.w == f.u ? g + 3 : i2)));
      }
      if (i1 >= 0) n1 = ls[i1];
      if (i2 >= 0) n2 = ls[i2];
    } else {
      for (int g = 0; g < b; g++) {
        const FanRec h = w.fan[foff + g];
        if (h.u == f.v) n1 = h.slot;
        if (h.v == f.u) n2 = h.slot;
      }
    }
    int s1 = -1, s2 = -1;
    if (!is_cc) {
      s1 = f.v == sa ? seg : (f.v == sb ? knew : -1);
      s2 = f.u == sa ? seg : (f.u == sb ? knew : -1);
    }
    const int mask = (f.ts >= 0 ? 1 : 0) | (s1 >= 0 ? 2 : 0) | (s2 >= 0 ? 4 : 0);
    m.tv[s] = make_int4(f.u, f.v, pid, mask);
    m.tn[s] = make_int4(n0, n1, n2, 0);
    m.ts[s] = make_int4(f.ts, s1, s2, 0);
    w.tstamp[s] = serial;
  }
  if (gl == 0) {
    m.vxy[pid] = p;
    m.vkind[pid] = is_cc ? 2 : 1;
    if (!is_cc) {
      m.sv[seg] = make_int2(sa, pid);
      m.sv[knew] = make_int2(pid, sb);
      m.spar[knew] = m.spar[seg];
      m.spend[knew] = 0;
      w.sadj[2 * knew] = -1;
      w.sadj[2 * knew + 1] = -1;
      w.mflag[knew] = 0u;
    }
  }
}

constexpr int kWriteWords = 3 * kFanMax;  // LDS of a group in write_part
__device__ __forceinline__ void write_part(const DevMesh &m, const Work &w, int32_t *lds, const Lanes &L) {
  if (w.cnt->abort) return;
  const int n = w.cnt->nw0, nV = w.st->nV, nS = w.st->nS, serial = w.st->serial;
  const GrpLanes g = grp_lanes(L);
  for (int i = g.first + g.grp; i < n; i += g.stride) {
    write_one(m, w, lds + g.grp * kWriteWords, i, nV, nS, serial);
    wave_lds_sync();
  }
}

__global__ void k_write(DevMesh m, Work w) {
  extern __shared__ __attribute__((aligned(16))) int32_t dyn_lds[];
  if (w.st->halt) return;
  write_part(m, w, dyn_lds, grid_lanes());
}

// R11: clear marks and bitmap bits of every candidate; pending flags.  A
// subsegment is split iff its second endpoint is now a new vertex.  After an
// abandoned round nothing was split and the flags are only released.
__device__ __forceinline__ void finish_one(const DevMesh &m, const Work &w, int c, int ncc, int nV, bool aborted) {
  CandSet S;
  int ci, is_cc;
  cand_at(w, c, ncc, S, ci, is_cc);
  int st = S.state[ci];
  if (st & kStAlive) {
    int off = S.off[ci], len = S.len[ci];
    for (int j0 = 0; j0 < len; j0 += kIlp) {
      int t[kIlp];
#pragma unroll
      for (int i = 0; i < kIlp; i++) t[i] = j0 + i < len ? w.pool[off + j0 + i] : -1;
#pragma unroll
      for (int i = 0; i < kIlp; i++)
        if (t[i] >= 0) w.mark[t[i]] = 0ull;
    }
  }
  int e = S.elem[ci];
  uint32_t bit = 1u << (e & 31);
  if (st & kStW0) atomicAnd(&(is_cc ? w.w0_t : w.w0_s)[e >> 5], ~bit);
  if (st & kStWin) {
    atomicAnd(&(is_cc ? w.win_t : w.win_s)[e >> 5], ~bit);
    if (!is_cc) atomicAnd(&w.win_h[e >> 5], ~bit);
  }
  if (!is_cc) {
    // pending := (pending or flagged this round) and not split; an entry the
    // cap skipped is not "flagged" unless R4/R5 flagged it again (own entry)
    if (!aborted) {
      bool split = m.sv[e].y >= nV;
      if (!(st & kStSkip)) m.spend[e] = split ? 0 : 1;
      else if (split) m.spend[e] = 0;
    }
    w.mflag[e] = 0u;
  }
}

// End of a round (run by the last workgroup of k_finish to arrive, or by the
// single-workgroup engine): a
// completed round is recorded in the history, the counts advance, this
// round's lists become the previous ones and the counters are cleared for
// the next round.  An error, an abandoned round or a round without winners
// halts instead (the counters stay for the host to read).
// Folds the stat lines into the round counters and clears them (one
// workgroup; ends with a barrier).
__device__ __forceinline__ void round_fold(const Work &w) {
  __shared__ uint64_t s_fold[kStFields];
  DevCounters *c = w.cnt;
  // fold the stat lines into the counters and clear them (read-and-clear
  // atomics: the lines were written by atomics)
  if (threadIdx.x < kStFields) s_fold[threadIdx.x] = 0;
  __syncthreads();
  constexpr int kGroups = (kStFields + 3) / 4;
  for (int idx = threadIdx.x; idx < kGroups * kStatStripes; idx += blockDim.x) {
    // one stripe, four of its fields (independent read-and-clear atomics),
    // combined in LDS
    const int i = idx / kGroups, f0 = (idx % kGroups) * 4;
    for (int f = f0; f < f0 + 4 && f < kStFields; f++) {
      const uint64_t x = atomicExch((unsigned long long *)&w.stat[i].v[f], 0ull);
      if (!x) continue;
      if (f == kStCavMax) atomicMax((unsigned long long *)&s_fold[f], (unsigned long long)x);
      else atomicAdd((unsigned long long *)&s_fold[f], (unsigned long long)x);
    }
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    c->cav_tri_total += (int64_t)s_fold[kStCavTri];
    c->cav_len[0] += (int64_t)s_fold[kStCavLen0];
    c->cav_len[1] += (int64_t)s_fold[kStCavLen1];
    c->cav_bnd[0] += (int64_t)s_fold[kStCavBnd0];
    c->cav_bnd[1] += (int64_t)s_fold[kStCavBnd1];
    c->n_enc_reject += (int32_t)s_fold[kStEncReject];
    c->n_fan_invalid += (int32_t)s_fold[kStFanInvalid];
    c->n_unsplittable += (int32_t)s_fold[kStUnsplittable];
    c->n_mid_cand += (int32_t)s_fold[kStMidCand];
    c->n_lost_mark += (int32_t)s_fold[kStLostMark];
    c->n_dep_drop += (int32_t)s_fold[kStDepDrop];
    c->n_blocked += (int32_t)s_fold[kStBlocked];
    c->n_coincident += (int32_t)s_fold[kStCoincident];
    c->cav_max = max(c->cav_max, (int32_t)s_fold[kStCavMax]);
    c->n_in_tests += (int64_t)s_fold[kStInTests];
    c->n_or_tests += (int64_t)s_fold[kStOrTests];
    for (int e = 0; e < kExStages; e++) c->n_exact[e] += (int64_t)s_fold[kStExact0 + e];
    c->win_cav += (int64_t)s_fold[kStWinCav];
    c->win_bnd += (int64_t)s_fold[kStWinBnd];
    c->win_steps += (int64_t)s_fold[kStWinSteps];
    c->win_cc_cav += (int64_t)s_fold[kStWinCcCav];
    c->win_cc_bnd += (int64_t)s_fold[kStWinCcBnd];
    c->n_marks[0] += (int64_t)s_fold[kStMarks0];
    c->n_marks[1] += (int64_t)s_fold[kStMarks1];
  }
  __syncthreads();
}

__device__ __forceinline__ void round_end(const Work &w) {
  __shared__ int s_go, s_slot;
  DevState *st = w.st;
  DevCounters *c = w.cnt;
  round_fold(w);
  if (threadIdx.x == 0) {
    s_go = 0;
    s_slot = -1;
    const int err = c->err, nwin = c->nwin;
    if (err & (kErrWalk | kErrInput | kErrCavity)) st->halt = kHaltError;
    else if (c->abort) st->halt = kHaltAbort;
    else if (nwin == 0) st->halt = kHaltStall;
    else {
      s_go = 1;
      const int nh = st->nhist;
      if (nh < w.hist_cap) s_slot = nh;
      st->nhist = nh + 1;
      const int nT = st->nT + c->fresh_total, nS = st->nS + c->nwin_mid;
      st->nV = st->nV + nwin;
      st->nT = nT;
      st->nS = nS;
      st->wT = nT / 32 + 1;
      st->wS = nS / 32 + 1;
      st->rounds = st->rounds + 1;
      st->serial = st->serial + 1;
      st->prev_ncc = c->ncc;
      st->prev_nmk = c->nmk;
      st->prev_fan = c->fan_used;
      st->full = 0;
    }
  }
  __syncthreads();
  if (!s_go) return;
  const int nw = (int)(sizeof(DevCounters) / 4);
  int32_t *src = (int32_t *)c;
  if (s_slot >= 0) {
    int32_t *dst = (int32_t *)&w.hist[s_slot];
    for (int i = threadIdx.x; i < nw; i += blockDim.x) dst[i] = src[i];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nw; i += blockDim.x) src[i] = 0;
}

__device__ __forceinline__ void finish_part(const DevMesh &m, const Work &w, const Lanes &L) {
  const int ncc = w.cnt->ncc, n = ncc + w.cnt->nmk, nV = w.st->nV;
  // an abandoned round, or one that inserts nothing (the refinement stops
  // there), leaves the pending flags as they were
  bool aborted = w.cnt->abort != 0 || w.cnt->nwin == 0;
  for (int base = L.base0; base < n; base += L.stride) {
    int c = base + threadIdx.x;
    if (c < n) finish_one(m, w, c, ncc, nV, aborted);
  }
}

__global__ void k_finish(DevMesh m, Work w) {
  __shared__ int s_last;
  if (w.st->halt) return;
  finish_part(m, w, grid_lanes());
  // every workgroup has read the counts it needs before it arrives here
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    s_last = atomicAdd(&w.st->done_blocks, 1) == (int)gridDim.x - 1;
  }
  __syncthreads();
  if (!s_last) return;
  __threadfence();
  if (threadIdx.x == 0) w.st->done_blocks = 0;
  round_end(w);
}

// ---------------------------------------------------------------------------
// Flip-Flop rounds (Section 4.3): Line 6 claims and the end of the round.
// ---------------------------------------------------------------------------
// Edge of the located triangle a circumcenter lies on, + 1, kept in bits 8-9
// of its state (0: strictly inside).
constexpr int kFfEdgeShift = 8;

// A located circumcenter claims its triangle, or both triangles of the
// interior edge it lies on; one on a subsegment encroaches it and flags it.
__global__ void kf_claim_cc(DevMesh m, Work w) {
  if (w.st->halt) return;
  const Lanes L = grid_lanes();
  const int ncc = w.cnt->ncc;
  int n_rej = 0;
  for (int base = L.base0; base < ncc; base += L.stride) {
    const int c = base + threadIdx.x;
    if (c >= ncc) continue;
    const int st = w.cc.state[c];
    if (!(st & kStFound) || (st & kStDone)) continue;
    const int loc = w.cc.loc[c];
    const int4 tri = m.tv[loc];
    const double2 p = w.cc.p[c];
    const double2 A = m.vxy[tri.x], B = m.vxy[tri.y], C = m.vxy[tri.z];
    const int s0 = orient_pts(w, A, B, p), s1 = orient_pts(w, B, C, p), s2 = orient_pts(w, C, A, p);
    const int e = s0 == 0 ? 0 : (s1 == 0 ? 1 : (s2 == 0 ? 2 : -1));
    int c1 = -1;
    if (e >= 0) {
      if ((tri.w >> e) & 1) {
        flag_mid(w, comp(m.ts[loc], e));
        w.cc.state[c] = st | kStDone;
        n_rej++;
        continue;
      }
      c1 = comp(m.tn[loc], e);
    }
    const uint64_t key = w.cc.key[c];
    w.cc.off[c] = loc;
    w.cc.len[c] = c1;
    w.cc.state[c] = (st & ~(3 << kFfEdgeShift)) | ((e + 1) << kFfEdgeShift);
    atomicMax((unsigned long long *)&w.mark[loc], (unsigned long long)key);
    if (c1 >= 0) atomicMax((unsigned long long *)&w.mark[c1], (unsigned long long)key);
  }
  stat_add(w, kStEncReject, n_rej);
}

// A flagged subsegment's split point claims the triangles on its sides
// (4 * slot + edge of each, -1 none); an unsplittable one is dropped.
__global__ void kf_claim_mid(DevMesh m, Work w) {
  if (w.st->halt) return;
  const Lanes L = grid_lanes();
  const int nmk = w.cnt->nmk;
  int n_cand = 0, n_uns = 0;
  for (int base = L.base0; base < nmk; base += L.stride) {
    const int i = base + threadIdx.x;
    if (i >= nmk) continue;
    const int st = w.mid.state[i];
    if (st & kStSkip) continue;
    const int k = w.mid.elem[i];
    n_cand++;
    const SplitPt sp = seg_split(m, k, w.pm, w.split_mode);
    const int2 s = m.sv[k];
    const double2 A = m.vxy[s.x], B = m.vxy[s.y];
    if ((sp.px == A.x && sp.py == A.y) || (sp.px == B.x && sp.py == B.y)) {
      w.mid.state[i] = st | kStDone;
      n_uns++;
      continue;
    }
    const int c0 = w.sadj[2 * k], c1 = w.sadj[2 * k + 1];
    w.mid.key[i] = sp.key;
    w.mid.p[i] = make_double2(sp.px, sp.py);
    w.mid.off[i] = c0;
    w.mid.len[i] = c1;
    w.mid.state[i] = st | kStFound;
    if (c0 >= 0) atomicMax((unsigned long long *)&w.mark[c0 >> 2], (unsigned long long)sp.key);
    if (c1 >= 0) atomicMax((unsigned long long *)&w.mark[c1 >> 2], (unsigned long long)sp.key);
  }
  stat_add(w, kStMidCand, n_cand);
  stat_add(w, kStUnsplittable, n_uns);
}

// Points that hold every claim go to S (midpoint references have bit 30).
__global__ void kf_own(Work w, FfCount *f, uint64_t *skey, int32_t *sref) {
  if (w.st->halt) return;
  const Lanes L = grid_lanes();
  const int ncc = w.cnt->ncc, n = ncc + w.cnt->nmk;
  int n_lost = 0;
  for (int base = L.base0; base < n; base += L.stride) {
    const int c = base + threadIdx.x;
    if (c >= n) continue;
    const bool is_cc = c < ncc;
    const int ci = is_cc ? c : c - ncc;
    const CandSet &S = is_cc ? w.cc : w.mid;
    const int st = S.state[ci];
    if (!(st & kStFound) || (st & (kStDone | kStSkip))) continue;
    const uint64_t key = S.key[ci];
    int c0 = S.off[ci], c1 = S.len[ci];
    if (!is_cc) {
      c0 = c0 >= 0 ? c0 >> 2 : -1;
      c1 = c1 >= 0 ? c1 >> 2 : -1;
    }
    const bool own = (c0 < 0 || w.mark[c0] == key) && (c1 < 0 || w.mark[c1] == key);
    if (!own) { n_lost++; continue; }
    const int idx = FfDevOps::append(&f->np);
    skey[idx] = ~key;
    sref[idx] = is_cc ? ci : (ci | (1 << 30));
    if (!is_cc) FfDevOps::append(&f->nmid);
  }
  stat_add(w, kStLostMark, n_lost);
}

__global__ void kf_clear_marks(Work w) {
  if (w.st->halt) return;
  const Lanes L = grid_lanes();
  const int ncc = w.cnt->ncc, n = ncc + w.cnt->nmk;
  for (int base = L.base0; base < n; base += L.stride) {
    const int c = base + threadIdx.x;
    if (c >= n) continue;
    const bool is_cc = c < ncc;
    const int ci = is_cc ? c : c - ncc;
    const CandSet &S = is_cc ? w.cc : w.mid;
    const int st = S.state[ci];
    if (!(st & kStFound) || (st & kStSkip)) continue;
    if (is_cc && (st & kStDone)) continue;  // dropped before claiming
    int c0 = S.off[ci], c1 = S.len[ci];
    if (!is_cc) {
      if (st & kStDone) continue;
      c0 = c0 >= 0 ? c0 >> 2 : -1;
      c1 = c1 >= 0 ? c1 >> 2 : -1;
    }
    if (c0 >= 0) w.mark[c0] = 0ull;
    if (c1 >= 0) w.mark[c1] = 0ull;
  }
}

// S by rank (the sorted references): point, class, claims, a midpoint's
// subsegment endpoints; every point starts in the mesh and not redundant.
__global__ void kf_gather(DevMesh m, Work w, FfView V, const int32_t *sref) {
  const int np = V.c->np;
  for (int r = blockIdx.x * blockDim.x + threadIdx.x; r < np; r += gridDim.x * blockDim.x) {
    const int ref = sref[r];
    ff_init_point_one<FfDevOps>(V, r);
    if (ref & (1 << 30)) {
      const int i = ref & ((1 << 30) - 1);
      const int k = w.mid.elem[i];
      V.pt[r] = w.mid.p[i];
      V.pinfo[r] = make_int4(1, k, w.mid.off[i], w.mid.len[i]);
      V.pab[r] = m.sv[k];
    } else {
      const int st = w.cc.state[ref];
      V.pt[r] = w.cc.p[ref];
      V.pinfo[r] = make_int4(0, ((st >> kFfEdgeShift) & 3) - 1, w.cc.off[ref], w.cc.len[ref]);
      V.pab[r] = make_int2(-1, -1);
    }
  }
}

// End of a Flip-Flop round (one workgroup): statistics folded in, the counts
// advanced to the compacted mesh, the round recorded, the counters cleared.
// Every element of the round's candidate lists was consumed by the host-side
// sequence, so the next round collects over the whole mesh again.
__global__ void kf_round_end(Work w, const FfCount *f, int32_t nT_new, int32_t nwin, int32_t nwin_mid) {
  __shared__ int s_slot;
  DevState *st = w.st;
  DevCounters *c = w.cnt;
  round_fold(w);
  if (threadIdx.x == 0) {
    c->n_dep_drop += (int32_t)f->n_dep;
    c->n_enc_reject += (int32_t)f->n_enc;
    c->nwin = nwin;
    c->nwin_mid = nwin_mid;
    c->nwin_cc = nwin - nwin_mid;
    c->fresh_total = nT_new - st->nT;
    c->ff_points = f->np;
    c->ff_iters = f->iters;
    c->ff_flips = f->flips;
    c->ff_passes = f->passes;
    c->ff_removals = f->removals;
    c->ff_rm_passes = f->rm_passes;
    const int nh = st->nhist;
    s_slot = nh < w.hist_cap ? nh : -1;
    st->nhist = nh + 1;
    st->nV = st->nV + nwin;
    st->nT = nT_new;
    st->nS = st->nS + nwin_mid;
    st->wT = nT_new / 32 + 1;
    st->wS = st->nS / 32 + 1;
    st->rounds = st->rounds + 1;
    st->serial = st->serial + 1;
    st->prev_ncc = 0;
    st->prev_nmk = 0;
    st->prev_fan = 0;
    st->full = 1;
  }
  __syncthreads();
  const int nw = (int)(sizeof(DevCounters) / 4);
  int32_t *src = (int32_t *)c;
  if (s_slot >= 0) {
    int32_t *dst = (int32_t *)&w.hist[s_slot];
    for (int i = threadIdx.x; i < nw; i += blockDim.x) dst[i] = src[i];
  }
  __syncthreads();
  for (int i = threadIdx.x; i < nw; i += blockDim.x) src[i] = 0;
}

// ---------------------------------------------------------------------------
// Mesh quality (the bad-area measure of Table 1): every triangle is tested
// with the scan's formula; a bad one adds its doubled area / 2.  Each block
// sums its lanes in a fixed tree order; the partials are summed in index
// order by one thread, so the result depends only on the grid shape.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_quality(DevMesh m, double B2, double L2, unsigned long long *n_part,
                                                 double *a_part) {
  __shared__ unsigned long long s_n[256];
  __shared__ double s_a[256];
  unsigned long long n = 0;
  double a = 0.0;
  for (int t = blockIdx.x * blockDim.x + threadIdx.x; t < m.nT; t += gridDim.x * blockDim.x) {
    SplitPt r = tri_split(m, t, m.tv[t], B2, L2, 0);
    if (r.bad) {
      n++;
      a += r.d * 0.5;
    }
  }
  s_n[threadIdx.x] = n;
  s_a[threadIdx.x] = a;
  __syncthreads();
  for (int h = blockDim.x / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) {
      s_n[threadIdx.x] += s_n[threadIdx.x + h];
      s_a[threadIdx.x] += s_a[threadIdx.x + h];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    n_part[blockIdx.x] = s_n[0];
    a_part[blockIdx.x] = s_a[0];
  }
}

__global__ void k_scatter_copy(const int32_t *src, const CopyEnt *ents, int n) {
  for (int e = blockIdx.x; e < n; e += gridDim.x) {
    const CopyEnt c = ents[e];
    const int32_t *a = src + c.src_off / 4;
    const int64_t words = c.bytes / 4;
    for (int64_t i = threadIdx.x; i < words; i += blockDim.x) c.dst[i] = a[i];
  }
}

// One workgroup.  The areas are added one after the other in the order of the
// workgroups, which is what bounds it: the partials come to LDS side by side,
// and one thread adds them eight loads ahead (512 partials: 9 us; loaded by the
// adding thread one by one, 55 us).
__global__ __launch_bounds__(256) void k_quality_sum(int n_part, const unsigned long long *n_in, const double *a_in,
                                                     unsigned long long *n_out, double *a_out) {
  __shared__ __attribute__((aligned(16))) double s_a[kQualBlocks];
  __shared__ unsigned long long s_n;
  if (threadIdx.x == 0) s_n = 0;
  __syncthreads();
  unsigned long long n = 0;
  double a = 0.0;
  const int m = min(n_part, kQualBlocks);
  for (int i = threadIdx.x; i < m; i += 256) {
    n += n_in[i];
    s_a[i] = a_in[i];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int i = 0;
    for (; i + 8 <= m; i += 8) {
      double x[8];
#pragma unroll
      for (int k = 0; k < 8; k++) x[k] = s_a[i + k];
#pragma unroll
      for (int k = 0; k < 8; k++) a += x[k];
    }
    for (; i < m; i++) a += s_a[i];
  }
  atomicAdd(&s_n, n);
  __syncthreads();
  if (threadIdx.x == 0) {
    *n_out = s_n;
    *a_out = a;
  }
}

// ---------------------------------------------------------------------------
// Single-workgroup engine: whole rounds, every phase of Lines 3-9, inside one
// workgroup, with workgroup barriers between the phases instead of kernel
// launches.  Used for rounds too small to fill the chip (the end of a
// refinement, where launch latency dominates) and, one mesh per workgroup,
// for batches of independent meshes.  The phases are the same functions the
// grid kernels run, so the result is identical.
// ---------------------------------------------------------------------------
// Barrier between two phases.  Every wave of the engine runs on one compute
// unit, so the workgroup-scope release / acquire of the barrier is enough to
// make each phase's writes (stores and atomics) visible to the next phase.
__device__ __forceinline__ void phase_sync() { __syncthreads(); }

// Exclusive scan of *j.n_dev entries by one workgroup: complete prefixes in
// j.out, zero tile prefixes (so that readers that add them are unchanged).
__device__ void engine_scan(const ScanJob &j) {
  __shared__ int s_total;
  const int n = *j.n_dev;
  const int chunk = blockDim.x * kScanItems;
  int carry = 0;
  for (int start = 0; start < n; start += chunk) {
    int base = start + threadIdx.x * kScanItems;
    int v[kScanItems];
    int sum = 0;
    for (int i = 0; i < kScanItems; i++) {
      int idx = base + i;
      int x = idx < n ? j.in[idx] : 0;
      if (j.mode == 1) x = __popc((uint32_t)x);
      v[i] = x;
      sum += x;
    }
    int excl = block_excl_scan(sum, &s_total) + carry;
    for (int i = 0; i < kScanItems; i++) {
      int idx = base + i;
      if (idx < n) j.out[idx] = excl;
      excl += v[i];
    }
    carry += s_total;
    __syncthreads();
  }
  for (int t = threadIdx.x; t <= n / kScanTile; t += blockDim.x) j.tiles[t] = 0;
  if (threadIdx.x == 0) *j.total = carry;
}

// Radix select of the K-th largest key by one workgroup (keys are unique);
// the threshold goes to w.sel[0] (0 when no more than K keys).
__device__ void engine_select(const Work &w, int K, int32_t *h) {
  __shared__ uint64_t s_prefix, s_pmask;
  __shared__ int64_t s_rem;
  const int n = w.cnt->ncc + w.cnt->nmk;
  if (threadIdx.x == 0) {
    s_prefix = 0;
    s_pmask = 0;
    s_rem = K;
  }
  __syncthreads();
  if (n > K) {
    for (int shift = 56; shift >= 0; shift -= 8) {
      for (int i = threadIdx.x; i < 256; i += blockDim.x) h[i] = 0;
      __syncthreads();
      const uint64_t prefix = s_prefix, pmask = s_pmask;
      for (int c = threadIdx.x; c < n; c += blockDim.x) {
        uint64_t k = w.keys[c];
        if ((k & pmask) == prefix) atomicAdd(&h[(k >> shift) & 255u], 1);
      }
      __syncthreads();
      if (threadIdx.x == 0) {
        int64_t cum = 0;
        int d = 255;
        for (; d > 0; d--) {
          if (cum + h[d] >= s_rem) break;
          cum += h[d];
        }
        s_rem -= cum;
        s_prefix |= (uint64_t)d << shift;
        s_pmask |= (uint64_t)0xff << shift;
      }
      __syncthreads();
    }
  }
  if (threadIdx.x == 0) w.sel[0] = s_prefix;
}

// Winner ranks by counting (at most kEngRankMax winners): rank = number of
// winners with a smaller (class, element) key, midpoints first, which is the
// order the bitmap ranks give; the key's lowest bit marks a hull midpoint.
// Returns false if there are more winners.
constexpr int kEngRankMax = 2048;
__device__ bool engine_rank(const Work &w, int32_t *lds) {
  __shared__ int s_nw, s_nmid, s_nhull;
  int32_t *key = lds, *ref = lds + kEngRankMax;
  if (threadIdx.x == 0) {
    s_nw = 0;
    s_nmid = 0;
    s_nhull = 0;
  }
  __syncthreads();
  const int n = w.cnt->nw0;
  for (int i = threadIdx.x; i < n; i += blockDim.x) {
    int ci, is_cc;
    const CandSet &S = cand_ref(w, w.w0_list[i], ci, is_cc);
    if (!(S.state[ci] & kStWin)) continue;
    const int e = S.elem[ci], hull = 2 - fresh_of(w, is_cc, e);
    const int pos = atomicAdd(&s_nw, 1);
    if (!is_cc) atomicAdd(&s_nmid, 1);
    if (hull) atomicAdd(&s_nhull, 1);
    if (pos < kEngRankMax) {
      key[pos] = (int32_t)(((uint32_t)is_cc << 31) | ((uint32_t)e << 1) | (uint32_t)hull);
      ref[pos] = i;
    }
  }
  __syncthreads();
  const int nw = s_nw;
  if (nw > kEngRankMax) return false;
  for (int i = threadIdx.x; i < nw; i += blockDim.x) {
    const uint32_t k = (uint32_t)key[i];
    int r = 0, h = 0;
    for (int j = 0; j < nw; j++) {
      const uint32_t x = (uint32_t)key[j];
      const int lt = x < k;
      r += lt;
      h += lt & (int)(x & 1u) & (int)(~x >> 31);
    }
    w.win_rank[ref[i]] = r;
    w.win_fresh[ref[i]] = 2 * r - h;
  }
  if (threadIdx.x == 0) {
    w.cnt->nwin_mid = s_nmid;
    w.cnt->nwin_cc = nw - s_nmid;
    w.cnt->nwin_hull = s_nhull;
  }
  return true;
}

// The single-workgroup engine's large cavities: growth, bitonic sort and
// checks in LDS, as the cooperative kernel does, by the engine's own
// workgroup.  A cavity beyond the LDS list makes the round abandon itself
// (kErrHuge); the host then runs that mesh's rounds on the grid kernels,
// which finish such cavities in device memory.
__device__ __forceinline__ void engine_big_one(const DevMesh &m, const Work &w, BigShared &sh, int b) {
  int32_t *cav = sh.cav;
  int32_t *hs = sh.hs;
  int &s_n = sh.s_n, &s_head = sh.s_head, &s_ovf = sh.s_ovf, &s_nbnd = sh.s_nbnd, &s_fanbad = sh.s_fanbad,
      &s_enc = sh.s_enc, &s_off = sh.s_off;
  int tid = threadIdx.x;
  int ref = w.big[b];
  int is_cc = (ref & 0x80000000) ? 0 : 1;
  int ci = ref & 0x7fffffff;
  CandSet S = is_cc ? w.cc : w.mid;
  if (!(S.state[ci] & kStBig) || (S.state[ci] & kStDone)) return;
  double2 p = S.p[ci];
  int skip_k = is_cc ? -1 : S.elem[ci];
  for (int i = tid; i < kHash; i += blockDim.x) hs[i] = -1;
  __syncthreads();
  int expect = 2;
  if (tid == 0) {
    s_n = 0; s_head = 0; s_ovf = 0; s_nbnd = 0; s_fanbad = 0; s_enc = 0;
    if (is_cc) {
      int t = S.loc[ci];
      hash_insert(hs, t, &s_ovf);
      cav[s_n++] = t;
    } else {
      int a0 = w.sadj[2 * skip_k], a1 = w.sadj[2 * skip_k + 1];
      if (a0 >= 0 && hash_insert(hs, a0 >> 2, &s_ovf)) cav[s_n++] = a0 >> 2;
      if (a1 >= 0 && hash_insert(hs, a1 >> 2, &s_ovf)) cav[s_n++] = a1 >> 2;
    }
  }
  if (!is_cc) expect = (w.sadj[2 * skip_k] >= 0 && w.sadj[2 * skip_k + 1] >= 0) ? 2 : 1;
  __syncthreads();
  for (;;) {
    int lo = s_head, hi = s_n < kBigMax ? s_n : kBigMax;
    int ovf = s_ovf;
    __syncthreads();
    if (lo >= hi || ovf) break;
    if (tid == 0) s_head = hi;
    for (int idx = lo + tid; idx < hi; idx += blockDim.x) {
      int t = cav[idx];
      int4 tri = m.tv[t];
      int4 nb = m.tn[t];
      for (int e = 0; e < 3; e++) {
        if ((tri.w >> e) & 1) continue;
        int o = comp(nb, e);
        if (o < 0) continue;
        if (!hash_insert(hs, o, &s_ovf)) continue;
        if (incircle_tri(m, w, m.tv[o], p) > 0) {
          int pos = atomicAdd(&s_n, 1);
          if (pos < kBigMax) cav[pos] = o;
          else s_ovf = 1;
        }
      }
    }
    __syncthreads();
  }
  if (s_ovf) {
    if (tid == 0) atomicOr(&w.cnt->err, kErrHuge);
    return;
  }
  int len = s_n;
  int P = 1;
  while (P < len) P <<= 1;
  for (int i = len + tid; i < P; i += blockDim.x) cav[i] = 0x7fffffff;
  for (int size = 2; size <= P; size <<= 1)
    for (int stride = size >> 1; stride > 0; stride >>= 1) {
      __syncthreads();
      for (int i = tid; i < P; i += blockDim.x) {
        int j = i ^ stride;
        if (j > i) {
          bool up = (i & size) == 0;
          int x = cav[i], y = cav[j];
          if ((x > y) == up) { cav[i] = y; cav[j] = x; }
        }
      }
    }
  __syncthreads();
  // boundary checks, in parallel over cavity triangles
  for (int j = tid; j < len; j += blockDim.x) {
    int t = cav[j];
    int4 tri = m.tv[t];
    int4 nb = m.tn[t];
    int4 ts = tri.w ? m.ts[t] : make_int4(-1, -1, -1, 0);
    for (int e = 0; e < 3; e++) {
      int sid = ((tri.w >> e) & 1) ? comp(ts, e) : -1;
      if (skip_k >= 0 && sid == skip_k) continue;
      int o = comp(nb, e);
      if (sid < 0 && o >= 0 && in_sorted(cav, len, o)) continue;
      atomicAdd(&s_nbnd, 1);
      double2 U = m.vxy[comp(tri, e)], V = m.vxy[comp(tri, (e + 1) % 3)];
      if (is_cc && sid >= 0 && encroached(w, U, V, p)) {
        flag_mid(w, sid);
        s_enc = 1;
      }
      if (orient_pts(w, U, V, p) <= 0) s_fanbad = 1;
    }
  }
  __syncthreads();
  if (tid == 0) {
    s_off = -1;
    bool drop = (is_cc && s_enc) || s_fanbad || s_nbnd - len != expect;
    if (drop) {
      atomicAdd((unsigned long long *)&w.cnt->cav_tri_total, (unsigned long long)len);
      atomicMax(&w.cnt->cav_max, len);
      atomicAdd((is_cc && s_enc) ? &w.cnt->n_enc_reject : &w.cnt->n_fan_invalid, 1);
      S.state[ci] |= kStDone;
    } else {
      int off = atomicAdd(&w.cnt->pool_used, len);
      if (off + len > w.pool_cap) atomicOr(&w.cnt->err, kErrPool);
      else {
        s_off = off;
        atomicAdd((unsigned long long *)&w.cnt->cav_tri_total, (unsigned long long)len);
        atomicMax(&w.cnt->cav_max, len);
      }
    }
  }
  __syncthreads();
  int off = s_off;
  if (off >= 0) {
    uint64_t key = S.key[ci];
    for (int j = tid; j < len; j += blockDim.x) {
      w.pool[off + j] = cav[j];
      atomicMax((unsigned long long *)&w.mark[cav[j]], (unsigned long long)key);
    }
    if (tid == 0) {
      S.off[ci] = off;
      S.len[ci] = len;
      S.state[ci] |= kStDone | kStAlive;
    }
  }
}

// Large cavities of one class, one after the other, by the whole workgroup.
__device__ void engine_big(const DevMesh &m, const Work &w, BigShared &sh, int phase) {
  const int nbig = min(w.cnt->nbig, w.big_cap);
  for (int b = 0; b < nbig; b++) {
    int ref = w.big[b];
    int is_cc = (ref & 0x80000000) ? 0 : 1;
    if (is_cc != (phase == 0 ? 1 : 0)) continue;
    engine_big_one(m, w, sh, b);
    __syncthreads();
  }
}

// The engine's group cavities: half the workgroup takes the circumcenters
// while the other half takes the midpoints listed before them, with longer
// lists than the grid kernels' (large cavities are common in small meshes
// with clustered points, and the cooperative path runs them one at a time
// here).
constexpr int kEngCavThreads = kEngBlock / 2;
constexpr int kEngCap = 48;
static_assert(kEngCap <= kListMax, "engine cavity lists");
constexpr int kEngCavWords = kGrpWords * (kEngBlock / kGrp);
constexpr int kEngLdsWords = kEngCavWords > (int)(sizeof(BigShared) / 4) ? kEngCavWords : (int)(sizeof(BigShared) / 4);
static_assert(kApproxMax * kEngBlock <= kEngLdsWords, "prefilter slices fit in the engine's LDS");
static_assert(2 * kEngRankMax <= kEngLdsWords && kWriteWords * (kEngBlock / kGrp) <= kEngLdsWords &&
                  kSortMax * (kEngBlock / kGrp) <= kEngLdsWords,
              "winner keys, cavity sorts and fans fit in the engine's LDS");

// The scans of the winner bitmaps.
__device__ __forceinline__ ScanJobs winner_scans(const Work &w) {
  ScanJobs J;
  J.j[0] = ScanJob{(const int32_t *)w.win_s, w.rank_s, &w.st->wS, w.tiles_s, &w.cnt->nwin_mid, 1};
  J.j[1] = ScanJob{(const int32_t *)w.win_t, w.rank_t, &w.st->wT, w.tiles_t, &w.cnt->nwin_cc, 1};
  J.j[2] = ScanJob{(const int32_t *)w.win_h, w.rank_h, &w.st->wS, w.tiles_h, &w.cnt->nwin_hull, 1};
  return J;
}

// Rounds of one mesh until it halts or round_limit rounds have completed.
__device__ void engine_mesh(const EngDesc &d, int32_t *lds, int round_limit) {
  __shared__ int s_ser, s_full, s_halt, s_mid0;
  __shared__ uint32_t s_stat[kStFields];
  const DevMesh &m = d.m;
  DevState *st = d.w[0].st;
  const Lanes L = block_lanes();
  for (int r = 0; r < round_limit; r++) {
    phase_sync();
    if (threadIdx.x == 0) {
      s_halt = st->halt;
      s_ser = st->serial;
      s_full = st->full;
    }
    __syncthreads();
    if (s_halt) break;
    const Work &w = d.w[s_ser & 1];
    // R1 collection
    if (s_full) {
      scan_part(m, w, d.B2, d.pm, L);
    } else {
      carry_part(w, L);
      dirty_part(m, w, d.B2, d.pm, L);
      phase_sync();
      pending_part(m, w, L);
    }
    phase_sync();
    if (gate_part(w, d.max_rounds)) break;
    phase_sync();
    // R3 candidate cap
    if (d.K > 0) {
      gather_part(m, w, d.pm, L);
      phase_sync();
      engine_select(w, d.K, lds);
      phase_sync();
      apply_part(w, L);
      phase_sync();
    }
    // R4 locate, optional prefilters
    locate_part(m, w, L);
    phase_sync();
    if (d.f1)
      for (int mode = 0; mode < 3; mode++) {
        prefilter_part(m, w, mode, 0, lds, L);
        phase_sync();
      }
    if (d.approx_n > 0)
      for (int mode = 3; mode < 6; mode++) {
        prefilter_part(m, w, mode, d.approx_n, lds, L);
        phase_sync();
      }
    // R5/R6 cavities with their marks: the circumcenters on one half of the
    // workgroup while the midpoints listed so far (collection and walks) run
    // on the other; then the midpoints the circumcenter cavities flagged.
    // (Marks are order free and a midpoint cavity depends on no other.)
    BigShared &sh = *reinterpret_cast<BigShared *>(lds);
    constexpr int kHalf = kEngCavThreads / kGrp;
    const int grp = (int)threadIdx.x / kGrp;
    if (threadIdx.x == 0) s_mid0 = w.cnt->nmk;
    stat_lds_clear(s_stat);
    __syncthreads();
    const int mid0 = s_mid0;
    if (threadIdx.x < kEngCavThreads)
      cavity_part(m, w, 1, lds, kEngCap, s_stat, 0, kHalf, grp, false);
    else
      cavity_part(m, w, 0, lds + kHalf * kGrpWords, kEngCap, s_stat, 0, kHalf, grp - kHalf, false, 0, mid0);
    phase_sync();
    engine_big(m, w, sh, 0);
    phase_sync();
    cavity_part(m, w, 0, lds, kEngCap, s_stat, 0, 2 * kHalf, grp, false, mid0);
    phase_sync();
    stat_lds_flush(w, s_stat);
    phase_sync();
    engine_big(m, w, sh, 1);
    phase_sync();
    // R8 ownership, R9 dependency
    own_part(w, L);
    phase_sync();
    dep_part(m, w, L);
    phase_sync();
    // R10 ranks, fresh slots, capacity check, insertion
    if (engine_rank(w, lds)) {
      phase_sync();
      record_part<true>(m, w, lds, L);
    } else {  // many winners: bitmap ranks as in the grid kernels
      const ScanJobs J = winner_scans(w);
      phase_sync();
      engine_scan(J.j[0]);
      engine_scan(J.j[1]);
      engine_scan(J.j[2]);
      phase_sync();
      record_part<false>(m, w, lds, L);
    }
    phase_sync();
    write_part(m, w, lds, L);
    phase_sync();
    finish_part(m, w, L);
    phase_sync();
    round_end(w);
  }
}

// Each workgroup takes meshes from a queue (head counts the taken ones) and
// runs each for at most round_limit rounds.
__global__ __launch_bounds__(kEngBlock) void k_engine(const EngDesc *descs, int n_mesh, int32_t *head,
                                                      int round_limit) {
  __shared__ __attribute__((aligned(16))) int32_t lds[kEngLdsWords];
  __shared__ int s_i;
  for (;;) {
    __syncthreads();
    if (threadIdx.x == 0) s_i = atomicAdd(head, 1);
    __syncthreads();
    const int i = s_i;
    if (i >= n_mesh) return;
    engine_mesh(descs[i], lds, round_limit);
  }
}

// ---------------------------------------------------------------------------
// Round-boundary batching: the round's phases for a set of meshes, one
// launch each.  The bodies are the single-mesh phases.  A workgroup of a
// phase over elements finds its mesh in a table (map) and its place among
// that mesh's workgroups in the mesh's descriptor, so that meshes of
// different sizes share the chip by their work; the others are launched with
// gridDim.y = meshes.  Each workgroup copies its mesh's descriptor (mesh
// arrays and the round's workspace, chosen by the mesh's own serial) into
// registers first.
// ---------------------------------------------------------------------------
#define GANG_MESH_OF(y_)                                    \
  const GangDesc &g_ = G[y_];                               \
  const int par_ = __builtin_amdgcn_readfirstlane(g_.e.w[0].st->serial & 1); \
  const DevMesh m = g_.e.m;                                 \
  const Work w = g_.e.w[par_];
#define GANG_MESH GANG_MESH_OF(blockIdx.y)
#define GANG_SHARE(kind)                                    \
  GANG_MESH_OF(__builtin_amdgcn_readfirstlane(map[blockIdx.x]))                            \
  const int bx_ = (int)blockIdx.x - g_.b0[kind], nb_ = g_.nb[kind];
#define GANG_LANES (Lanes{bx_ * (int)blockDim.x, nb_ * (int)blockDim.x, 1})

__global__ void kg_collect(const GangDesc *G, const int32_t *map) {
  GANG_SHARE(kGangElem)
  if (w.st->halt) return;
  if (w.st->full) {
    scan_part(m, w, g_.e.B2, g_.e.pm, GANG_LANES);
  } else {
    carry_part(w, GANG_LANES);
    dirty_part(m, w, g_.e.B2, g_.e.pm, GANG_LANES);
  }
}

__global__ void kg_pending(const GangDesc *G, const int32_t *map) {
  GANG_SHARE(kGangElem)
  if (w.st->halt || w.st->full) return;
  pending_part(m, w, GANG_LANES);
}

__global__ void kg_gate(const GangDesc *G) {
  GANG_MESH
  (void)m;
  (void)gate_part(w, g_.e.max_rounds);
}

__global__ void kg_gather_keys(const GangDesc *G, const int32_t *map) {
  GANG_SHARE(kGangElem)
  if (w.st->halt || g_.e.K <= 0) return;
  gather_part(m, w, g_.e.pm, GANG_LANES);
}

__global__ void kg_radix_hist(const GangDesc *G, const int32_t *map, int shift) {
  __shared__ int h[256];
  GANG_SHARE(kGangElem)
  (void)m;
  if (w.st->halt || g_.e.K <= 0) return;
  const int n = w.cnt->ncc + w.cnt->nmk;
  const uint64_t prefix = w.sel[0], pmask = w.sel[1];
  for (int i = threadIdx.x; i < 256; i += blockDim.x) h[i] = 0;
  __syncthreads();
  for (int c = bx_ * blockDim.x + threadIdx.x; c < n; c += nb_ * blockDim.x) {
    uint64_t k = w.keys[c];
    if ((k & pmask) == prefix) atomicAdd(&h[(k >> shift) & 255u], 1);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 256; i += blockDim.x)
    if (h[i]) atomicAdd(&w.rhist[i], h[i]);
}

__global__ void kg_radix_pick(const GangDesc *G, int shift) {
  GANG_MESH
  (void)m;
  if (w.st->halt || g_.e.K <= 0) return;
  radix_pick_part(w, shift, g_.e.K);
}

__global__ void kg_apply_cap(const GangDesc *G, const int32_t *map) {
  GANG_SHARE(kGangElem)
  (void)m;
  if (w.st->halt || g_.e.K <= 0) return;
  apply_part(w, GANG_LANES);
}

__global__ void kg_locate(const GangDesc *G, const int32_t *map) {
  GANG_SHARE(kGangElem)
  if (w.st->halt) return;
  locate_part(m, w, GANG_LANES);
}

__global__ __launch_bounds__(kPreBlock) void kg_prefilter(const GangDesc *G, const int32_t *map, int mode) {
  __shared__ int32_t lds[kApproxMax * kPreBlock];
  GANG_SHARE(kGangElem)
  if (w.st->halt) return;
  if (mode < 3 ? !g_.e.f1 : g_.e.approx_n <= 0) return;
  prefilter_part(m, w, mode, mode < 3 ? 0 : g_.e.approx_n, lds, GANG_LANES);
}

template <int IS_CC>
__global__ __launch_bounds__(kCavBlock, 5) void kg_cavity(const GangDesc *G, const int32_t *map) {
  GANG_SHARE(kGangGroup)
  if (w.st->halt) return;
  cavity_grid<IS_CC>(m, w, kCap, bx_, nb_);
}
template __global__ void kg_cavity<0>(const GangDesc *G, const int32_t *map);
template __global__ void kg_cavity<1>(const GangDesc *G, const int32_t *map);

// The large cavities of all n meshes, shared out one by one over the
// workgroups: a mesh's queue length is known on the device only, and the
// meshes differ (most have none, one can have thousands).  Every workgroup
// sums the queues of kBigBlock meshes at a time and finds its entries by the
// sums.  A fixed 256 / n workgroups for each mesh instead left a round of 64
// or 256 meshes waiting for one of them.
__global__ __launch_bounds__(kBigBlock) void kg_cavity_big(const GangDesc *G, int n, int phase) {
  __shared__ BigShared sh;
  __shared__ int s_first[kBigBlock], s_total;
  for (int base = 0; base < n; base += kBigBlock) {
    const int q = base + (int)threadIdx.x;
    int len = 0;
    if (q < n) {
      const Work &w = G[q].e.w[0];  // (the counters are the same for both parities)
      if (!w.st->halt) len = min(w.cnt->nbig, w.big_cap);
    }
    const int first = block_excl_scan(len, &s_total);
    s_first[threadIdx.x] = first;
    __syncthreads();
    const int total = s_total;
    for (int i = blockIdx.x; i < total; i += gridDim.x) {
      int lo = 0, hi = kBigBlock - 1;  // the last mesh whose entries start at or before i
      while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s_first[mid] <= i) lo = mid;
        else hi = mid - 1;
      }
      const int e = i - s_first[lo];
      GANG_MESH_OF(__builtin_amdgcn_readfirstlane(base + lo))
      const int is_cc = (w.big[e] & 0x80000000) ? 0 : 1;
      if (is_cc == (phase == 0 ? 1 : 0)) big_one(m, w, sh, e);
      __syncthreads();
    }
    __syncthreads();
  }
}

__global__ __launch_bounds__(kHugeBlock) void kg_cavity_huge(const GangDesc *G, int phase) {
  __shared__ BigShared sh;
  GANG_MESH
  if (w.st->halt || w.cnt->nhuge == 0) return;
  int nbig = min(w.cnt->nbig, w.big_cap);
  for (int b = 0; b < nbig; b++) {
    int ref = w.big[b];
    int is_cc = (ref & 0x80000000) ? 0 : 1;
    if (is_cc != (phase == 0 ? 1 : 0)) continue;
    huge_one(m, w, sh, b);
  }
}

__global__ void kg_own(const GangDesc *G, const int32_t *map) {
  GANG_SHARE(kGangElem)
  (void)m;
  if (w.st->halt) return;
  own_part(w, GANG_LANES);
}

__global__ void kg_dep(const GangDesc *G, const int32_t *map) {
  GANG_SHARE(kGangGroup)
  if (w.st->halt) return;
  dep_part(m, w, GANG_LANES);
}

__global__ __launch_bounds__(kScanBlock) void kg_scan_tiles(const GangDesc *G) {
  const GangDesc &g = G[blockIdx.y];
  if (g.e.w[0].st->halt) return;
  scan_tiles(winner_scans(g.e.w[0]));
}

// Launched with gridDim.x = 3.
__global__ __launch_bounds__(kScanBlock) void kg_scan_sums(const GangDesc *G) {
  const GangDesc &g = G[blockIdx.y];
  if (g.e.w[0].st->halt) return;
  const ScanJobs J = winner_scans(g.e.w[0]);
  scan_sums(blockIdx.x == 0 ? J.j[0] : (blockIdx.x == 1 ? J.j[1] : J.j[2]));
}

__global__ void kg_record(const GangDesc *G, const int32_t *map) {
  extern __shared__ __attribute__((aligned(16))) int32_t dyn_lds[];
  GANG_SHARE(kGangGroup)
  if (w.st->halt) return;
  record_part<false>(m, w, dyn_lds, GANG_LANES);
}

__global__ void kg_write(const GangDesc *G, const int32_t *map) {
  extern __shared__ __attribute__((aligned(16))) int32_t dyn_lds[];
  GANG_SHARE(kGangGroup)
  if (w.st->halt) return;
  write_part(m, w, dyn_lds, GANG_LANES);
}

__global__ void kg_finish(const GangDesc *G, const int32_t *map) {
  __shared__ int s_last;
  GANG_SHARE(kGangFinish)
  if (w.st->halt) return;
  finish_part(m, w, GANG_LANES);
  __syncthreads();
  if (threadIdx.x == 0) {
    __threadfence();
    s_last = atomicAdd(&w.st->done_blocks, 1) == nb_ - 1;
  }
  __syncthreads();
  if (!s_last) return;
  __threadfence();
  if (threadIdx.x == 0) w.st->done_blocks = 0;
  round_end(w);
}

// One workgroup per mesh; the history is handed over, so the mesh's next
// group starts an empty one.
__global__ void kg_status(const GangDesc *G, int rounds, int32_t *out, int stride_words) {
  const GangDesc &g = G[blockIdx.y];
  const Work &w = g.e.w[0];
  int32_t *o = out + (size_t)blockIdx.y * stride_words;
  const int ns = (int)(sizeof(DevState) / 4), nc = (int)(sizeof(DevCounters) / 4);
  const int32_t *st = (const int32_t *)w.st, *cn = (const int32_t *)w.cnt, *hi = (const int32_t *)w.hist;
  for (int i = threadIdx.x; i < ns; i += blockDim.x) o[i] = st[i];
  for (int i = threadIdx.x; i < nc; i += blockDim.x) o[ns + i] = cn[i];
  for (int i = threadIdx.x; i < rounds * nc; i += blockDim.x) o[ns + nc + i] = hi[i];
  __syncthreads();
  if (threadIdx.x == 0) w.st->nhist = 0;
}
#undef GANG_LANES
#undef GANG_SHARE
#undef GANG_MESH
#undef GANG_MESH_OF

// ---------------------------------------------------------------------------
// Measurement: 64-bit atomicMax at random slots of a table in device memory,
// the access pattern of the priority marks (random slot, one read-modify-
// write each).  Slot and value of operation i come from a fixed mix of i.
// ---------------------------------------------------------------------------
__global__ void k_atomic_max_bench(uint64_t *table, uint64_t n_slots, int64_t n_ops, uint64_t seed) {
  const int64_t stride = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n_ops; i += stride) {
    uint64_t h = (uint64_t)i * 0x9e3779b97f4a7c15ull + seed;
    h ^= h >> 31;
    h *= 0xbf58476d1ce4e5b9ull;
    h ^= h >> 29;
    atomicMax((unsigned long long *)&table[h % n_slots], (unsigned long long)(h | 1ull));
  }
}

// ---------------------------------------------------------------------------
// Test entry: the predicates above, one thread per query.
// ---------------------------------------------------------------------------
__global__ void k_predicates(int kind, int n, const double *pts, int32_t *out, uint64_t *tally) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int w = kind == 1 ? 8 : 6;
  const double *q = pts + (size_t)i * w;
  int r = 0;
  if (kind == 0) r = orient2d(q[0], q[1], q[2], q[3], q[4], q[5], tally);
  else if (kind == 1) r = incircle(q[0], q[1], q[2], q[3], q[4], q[5], q[6], q[7], tally);
  else if (kind == 2) r = indiametral(q[0], q[1], q[2], q[3], q[4], q[5], tally);
  else r = encroaches(1, q[0], q[1], q[2], q[3], q[4], q[5], tally) ? 1 : 0;
  out[i] = r;
}

}  // namespace gdp
