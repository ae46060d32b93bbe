// gdp_ff.hip -- the Flip-Flop insertion of Line 8 (Section 4.3) as kernels:
// grid-stride loops over the elements, each element one step of
// gdp_ff_core.h with device atomics.  The host sequence that drives them
// (one round: splits, flip passes, detection, removal passes, final ids,
// compaction) is ff_loop / ff_line8 in gdp_api.hip.
#include "gdp_kernels.h"

namespace gdp {

using DO = FfDevOps;
static_assert(kFfScanTile == kScanTileSize, "the ranks are scanned with the refinement's tile");

#define FF_LOOP(i, n) \
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < (n); i += gridDim.x * blockDim.x)

__global__ void kf_split(FfView V, int split_stamp, int wst, int tst) {
  const int np = V.c->np;
  FF_LOOP(r, np) ff_split_one<DO>(V, r, split_stamp, wst, tst);
}

__global__ void kf_split_fix(FfView V, int split_stamp) {
  const int np = V.c->np;
  FF_LOOP(r, np) ff_split_fix_one<DO>(V, r, split_stamp);
}

// Control words moved by one thread: op 0 empties worklist count `arg` and
// both candidate counts, op 2 starts a detection, op 4 the compaction lists.
__global__ void kf_ctl(FfCount *c, int op, int arg) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  switch (op) {
    case 0:
      c->n_list[arg] = 0;
      c->n_cnd[0] = 0;
      c->n_cnd[1] = 0;
      break;
    case 2:
      c->n_red = 0;
      c->n_hole = 0;
      c->star_used = 0;
      c->iters++;
      break;
    default:
      c->n_hole = 0;
      c->n_mover = 0;
      break;
  }
}

// A flip pass is these two launches: the list lengths and candidate counts
// are entries of FfCount chosen by the host (two lists and two candidate
// counts alternate), so no launch is needed between passes.
__global__ void kf_flip_check(FfView V, int in_stamp, uint64_t pass) {
  const int n = *V.n_in;
  if (blockIdx.x == 0 && threadIdx.x == 0) ff_check_begin<DO>(V);
  FF_LOOP(i, n) ff_flip_check_one<DO>(V, i, in_stamp, pass);
}

__global__ void kf_flip_apply(FfView V, int wst, int tst) {
  const int nc = *V.n_cand;
  if (blockIdx.x == 0 && threadIdx.x == 0) ff_apply_begin<DO>(V);
  FF_LOOP(i, min(nc, V.cand_cap)) ff_flip_apply_one<DO>(V, i, wst, tst);
  if (nc > V.cand_cap) {
    const int n_in = *V.n_in;
    FF_LOOP(i, n_in) ff_flip_requeue_one<DO>(V, i, wst);
  }
}

__global__ void kf_vtri(FfView V) {
  const int n = V.c->n_touched, np = V.c->np;
  FF_LOOP(i, n) ff_vtri_one<DO>(V, i, np);
}

__global__ void kf_detect(FfView V) {
  const int np = V.c->np;
  FF_LOOP(r, np) ff_detect_one<DO>(V, r);
}

// Flip passes over a short worklist inside one workgroup, two barriers instead
// of two launches each, until it is empty, longer than kFfTailMax or has taken
// kFfTailPasses passes: the passes used are left in c->tail_passes (their
// stamps and numbers follow stamp and pass one by one), the rest of the list in
// list0 / list1 by their parity.  Bound by latency: a pass is two chains of
// three dependent loads and two of atomics, 6.3 us, against 10 us for the two
// launches of an empty grid pass (26 us on average).  Lists of up to 1,024 or
// 4,096 entries here instead of 2,048: 106, 108 ms a refinement of 30,011
// points against 104.
__global__ __launch_bounds__(kFfTailBlk) void kf_flip_tail(FfView V, int32_t *list0, int32_t *list1, int cur0,
                                                           int in_stamp, int stamp, uint64_t pass, int tst) {
  __shared__ int32_t s_n[2], s_cand;
  const int n0 = V.c->n_list[cur0];
  if (threadIdx.x == 0) V.c->tail_passes = 0;
  if (n0 == 0 || n0 > kFfTailMax) return;
  if (threadIdx.x == 0) s_n[0] = n0;
  FfView T = V;
  T.n_cand = &s_cand;
  int cur = 0, used = 0;
  for (; used < kFfTailPasses; used++) {
    __syncthreads();
    const int n = s_n[cur];
    if (n == 0 || n > kFfTailMax) break;
    __syncthreads();
    if (threadIdx.x == 0) {
      s_n[cur ^ 1] = 0;
      s_cand = 0;
    }
    __syncthreads();
    T.list_in = cur ? list1 : list0;
    T.list_out = cur ? list0 : list1;
    T.n_in = &s_n[cur];
    T.n_out = &s_n[cur ^ 1];
    pass++;
    for (int i = threadIdx.x; i < n; i += kFfTailBlk) ff_flip_check_one<DO>(T, i, in_stamp, pass);
    __syncthreads();
    const int nc = s_cand;
    in_stamp = ++stamp;
    for (int i = threadIdx.x; i < min(nc, T.cand_cap); i += kFfTailBlk) ff_flip_apply_one<DO>(T, i, in_stamp, tst);
    if (nc > T.cand_cap)
      for (int i = threadIdx.x; i < n; i += kFfTailBlk) ff_flip_requeue_one<DO>(T, i, in_stamp);
    cur ^= 1;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    V.c->n_list[cur0 ^ (used & 1)] = s_n[cur];
    V.c->n_list[cur0 ^ (used & 1) ^ 1] = 0;
    V.c->n_cnd[0] = 0;
    V.c->n_cnd[1] = 0;
    V.c->tail_passes = used;
    V.c->passes += used;
  }
}

// ---------------------------------------------------------------------------
// Removal passes, kRmGrp lanes to a redundant point; a pass is two launches.
// The points left are entries of a list (two alternate).  kf_rm_mark walks a
// point's star once, keeps it (k triangles, their k or k + 1 link vertices; the
// flip candidates' memory: all stars together have at most three entries per
// triangle and one more per point, and it holds four per slot), and puts the
// point's stamp on its link.  kf_rm_apply compares the stamps of the kept
// link, so it reads no triangle that another point's removal writes, and
// removes the points that own theirs.  Bound by latency: the walk, then three
// dependent loads and the steps of the clipping.  Over the passes of a
// refinement of 30,011 points (up to 9,600 points left of 14,500) a pass takes
// 11 + 26 us; one thread per point and three launches over all of S, with the
// polygon in memory and its edges matched by search, took 27 + 27 + 213 us.
// Links above kRmGrp left to one thread: 112 us instead of 26.
// ---------------------------------------------------------------------------
constexpr int kRmGrp = 16;
constexpr int kRmWave = 64;  // link vertices that a whole wave takes
constexpr int kRmBlk = 256;
constexpr int kRmPer = kRmBlk / kRmGrp;

// Space from a counter for the groups of a workgroup (n: this group's, the
// same in all its lanes): one atomic per workgroup.
__device__ __forceinline__ int rm_take(int32_t *counter, int n) {
  __shared__ int s_part[kRmPer], s_base;
  const int g = threadIdx.x / kRmGrp;
  if (threadIdx.x % kRmGrp == 0) s_part[g] = n;
  __syncthreads();
  if (threadIdx.x == 0) {
    int acc = 0;
    for (int i = 0; i < kRmPer; i++) {
      const int t = s_part[i];
      s_part[i] = acc;
      acc += t;
    }
    s_base = acc ? atomicAdd(counter, acc) : 0;
  }
  __syncthreads();
  const int at = s_base + s_part[g];
  __syncthreads();
  return at;
}

// Duties of one thread: the removals' pool and the list of the points left
// start empty, the pass is counted.
__global__ __launch_bounds__(kRmBlk) void kf_rm_mark(FfView V, const int32_t *list, const int32_t *n_list,
                                                     int32_t *n_next, uint64_t pbase) {
  __shared__ int s_star[kRmPer][kRmWave], s_ring[kRmPer][kRmWave + 1];
  const int n = *n_list, gl = threadIdx.x % kRmGrp, g = threadIdx.x / kRmGrp;
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    V.c->pool_used = 0;
    V.c->pool_short = 0;
    *n_next = 0;
    if (n > 0) V.c->rm_passes++;
  }
  int32_t *stars = (int32_t *)V.fc0, *rings = (int32_t *)V.fc1;
  for (int base = blockIdx.x * kRmPer; base < n; base += gridDim.x * kRmPer) {
    const int i = base + g, r = i < n ? list[i] : -1;
    const int p = V.nV + r;
    int k = 0, open = 0, start = -1;
    if (r >= 0) {
      // every lane of the group walks: the loads are the same
      start = V.vtri[r];
      int t = start;
      for (;;) {
        const int4 tri = V.tv[t], nb = V.tn[t];
        const int q = ff_vidx(tri, p);
        if (q < 0 || k > kFfWalkCap) { k = 0; break; }
        if (k < kRmWave && gl == 0) {
          s_star[g][k] = t;
          s_ring[g][k] = ffc(tri, q == 2 ? 0 : q + 1);
          s_ring[g][k + 1] = ffc(tri, q == 0 ? 2 : q - 1);
        }
        k++;
        t = ffc(nb, q == 0 ? 2 : q - 1);  // across (previous vertex, p): counter-clockwise
        if (t == start) break;
        if (t >= 0) continue;
        if (open) break;
        // on the hull: to the other end of the star and again
        open = 1;
        k = 0;
        for (int steps = 0;; steps++) {
          const int4 tr = V.tv[start], tb = V.tn[start];
          const int x = ff_vidx(tr, p);
          if (x < 0 || steps > kFfWalkCap) { start = -1; break; }
          const int prev = ffc(tb, x);
          if (prev < 0) break;
          start = prev;
        }
        if (start < 0) break;
        t = start;
      }
      if (k == 0 && gl == 0) DO::err(&V.c->err, 8);
    }
    const int off = rm_take(&V.c->star_used, k ? k + 1 : 0);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    if (r < 0) continue;
    if (k == 0 || (int64_t)off + k + 1 > 4 * (int64_t)V.cand_cap) {
      if (gl == 0) {
        V.moved[i] = -1;
        DO::err(&V.c->err, 21);
      }
      continue;
    }
    const uint64_t prio = pbase | (uint64_t)(r + 1);
    if (gl == 0) {
      V.moved[i] = off;
      stars[off] = 2 * k + open;
      DO::max64(&V.vmark[p], prio);
    }
    if (k <= kRmWave) {
      for (int q = gl; q < k; q += kRmGrp) {
        stars[off + 1 + q] = s_star[g][q];
        rings[off + q] = s_ring[g][q];
        DO::max64(&V.vmark[s_ring[g][q]], prio);
      }
      if (open && gl == 0) {
        rings[off + k] = s_ring[g][k];
        DO::max64(&V.vmark[s_ring[g][k]], prio);
      }
    } else if (gl == 0) {
      int t = start;
      for (int x = 0; x < k; x++) {
        const int4 tri = V.tv[t];
        const int q = ff_vidx(tri, p);
        stars[off + 1 + x] = t;
        rings[off + x] = ffc(tri, (q + 1) % 3);
        DO::max64(&V.vmark[ffc(tri, (q + 1) % 3)], prio);
        if (open && x == k - 1) {
          rings[off + k] = ffc(tri, (q + 2) % 3);
          DO::max64(&V.vmark[ffc(tri, (q + 2) % 3)], prio);
        }
        t = ffc(V.tn[t], (q + 2) % 3);
      }
    }
  }
}

// A point's polygon(s) are filled by clipping ears: each lane holds a corner
// and every step clips the ears that are ears at the same time (no two of them
// neighbours; the smaller lane goes first), so a link of eight vertices takes
// two or three steps.  The corner test is ff_clip's.  Codes of an edge: >= 0
// the outer triangle, -1 none, kRmClose - side the closing edge of a midpoint's
// side, kRmTri - q the emitted triangle q.
constexpr int kRmClose = -2;  // .. -3
constexpr int kRmTri = -10;

// G: the lanes of a group, kRmGrp or kRmWave.
template <int G>
struct RmShared {
  int ev[3 * G], en[3 * G], es[3 * G];
  int clos[2];
};

template <int G>
__device__ __forceinline__ uint64_t rm_ballot(bool x, int g0) {
  return G == 64 ? __ballot(x) : (__ballot(x) >> g0) & ((1ull << (G & 63)) - 1);
}

// One edge of emitted triangle t: its code and subsegment, and the other
// side's where that is an emitted triangle or closes a side.
template <int G>
__device__ __forceinline__ void rm_edge(RmShared<G> &S, int t, int h, int code, int sub, int side) {
  S.en[3 * t + h] = code;
  S.es[3 * t + h] = sub;
  if (code <= kRmTri) S.en[3 * (kRmTri - code) + 2] = kRmTri - t;  // its edge 2 was the polygon's
  if (code == kRmClose - side) S.clos[side] = t;
}

// Lane gl < m holds corner gl: vertex pv at B, the edge to the next corner
// (code info, subsegment sd).  Returns the number of triangles emitted in all,
// -1 if no ear was found.
template <int G>
__device__ int rm_clip(RmShared<G> &S, double2 P, int m, int pv, double2 B, int info, int sd, int ne, int side) {
  const int gl = threadIdx.x % G, g0 = __lane_id() - gl;
  bool alive = gl < m;
  int nx = gl + 1 >= m ? 0 : gl + 1, pr = gl == 0 ? m - 1 : gl - 1;
  int left = m;
  bool general = false;
  if (m < 3) return -1;
  while (left > 3) {
    const double2 A = make_double2(__shfl(B.x, g0 + pr), __shfl(B.y, g0 + pr));
    const double2 C = make_double2(__shfl(B.x, g0 + nx), __shfl(B.y, g0 + nx));
    bool ear = alive && orient2d(A.x, A.y, B.x, B.y, C.x, C.y) > 0;
    if (!general) {
      ear = ear && orient2d(A.x, A.y, C.x, C.y, P.x, P.y) > 0;
    } else {
      const uint64_t live = rm_ballot<G>(alive, g0);
      for (int q = 0; q < m; q++) {
        const double2 Q = make_double2(__shfl(B.x, g0 + q), __shfl(B.y, g0 + q));
        if (!ear || !((live >> q) & 1) || q == gl || q == pr || q == nx) continue;
        if (orient2d(A.x, A.y, B.x, B.y, Q.x, Q.y) >= 0 && orient2d(B.x, B.y, C.x, C.y, Q.x, Q.y) >= 0 &&
            orient2d(C.x, C.y, A.x, A.y, Q.x, Q.y) >= 0)
          ear = false;
      }
    }
    const uint64_t ears = rm_ballot<G>(ear, g0);
    if (!ears) {
      if (general) return -1;
      general = true;
      continue;
    }
    const bool first = ear && !(((ears >> pr) & 1) && pr < gl) && !(((ears >> nx) & 1) && nx < gl);
    uint64_t sel = rm_ballot<G>(first, g0);
    if (general || left == 4) sel &= 0ull - sel;  // (five corners or more keep three)
    const int ci = __shfl(info, g0 + pr), cs = __shfl(sd, g0 + pr), va = __shfl(pv, g0 + pr), vc = __shfl(pv, g0 + nx);
    if ((sel >> gl) & 1) {
      const int t = ne + __popcll(sel & ((1ull << gl) - 1));
      S.ev[3 * t] = va;
      S.ev[3 * t + 1] = pv;
      S.ev[3 * t + 2] = vc;
      S.en[3 * t + 2] = -1;  // set by the triangle that takes the new edge
      S.es[3 * t + 2] = -1;
      rm_edge(S, t, 0, ci, cs, side);
      rm_edge(S, t, 1, info, sd, side);
      alive = false;
    }
    const int nnx = __shfl(nx, g0 + nx), npr = __shfl(pr, g0 + pr);
    const bool clip_n = (sel >> nx) & 1, clip_p = (sel >> pr) & 1;
    if (alive && clip_n) {
      info = kRmTri - (ne + __popcll(sel & ((1ull << nx) - 1)));
      sd = -1;
      nx = nnx;
    }
    if (alive && clip_p) pr = npr;
    left -= __popcll(sel);
    ne += __popcll(sel);
    general = false;
  }
  const int ci = __shfl(info, g0 + pr), cs = __shfl(sd, g0 + pr), va = __shfl(pv, g0 + pr);
  const int ni = __shfl(info, g0 + nx), ns = __shfl(sd, g0 + nx), vc = __shfl(pv, g0 + nx);
  if (alive && (rm_ballot<G>(alive, g0) & ((1ull << gl) - 1)) == 0) {
    S.ev[3 * ne] = va;
    S.ev[3 * ne + 1] = pv;
    S.ev[3 * ne + 2] = vc;
    rm_edge(S, ne, 0, ci, cs, side);
    rm_edge(S, ne, 1, info, sd, side);
    rm_edge(S, ne, 2, ni, ns, side);
  }
  return ne + 1;
}

// Removes point r, whose star (k triangles from stars[0], at most G link
// vertices) it owns.  All lanes of the group.
template <int G>
__device__ void rm_remove(const FfView &V, RmShared<G> &S, int r, int k, int open, const int32_t *stars, int wst, int tst) {
  const int gl = threadIdx.x % G, g0 = __lane_id() - gl, p = V.nV + r;
  const int4 info4 = V.pinfo[r];
  const double2 P = V.vxy[p];
  int slot = -1, ring = -1, last = -1, onb = -1, osd = -1;
  if (gl < k) {
    slot = stars[gl];
    const int4 tri = V.tv[slot], nb = V.tn[slot], z = V.ts[slot];
    const int q = ff_vidx(tri, p), q1 = q == 2 ? 0 : q + 1;
    ring = ffc(tri, q1);
    last = ffc(tri, q == 0 ? 2 : q - 1);
    onb = ffc(nb, q1);
    osd = ff_sid(tri, z, q1);
  }
  const int endv = __shfl(last, g0 + k - 1);
  if (open && gl == k) ring = endv;
  const double2 R = ring >= 0 ? V.vxy[ring] : P;
  int ne = 0, sl_side = -1, sl_x = -1, sl_u = -1, sl_v = -1;
  if (gl < 2) S.clos[gl] = -1;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  if (info4.x == 0) {
    ne = rm_clip(S, P, k, ring, R, onb, osd, 0, 0);
  } else {
    // the polygons of a midpoint (ff_rm_apply_one): the chain closed by the
    // restored subsegment, on both sides unless it is on the hull; a side that
    // is the single edge of the subsegment has nothing to fill
    const int2 ab = V.pab[r];
    const int sides = open ? 1 : 2;
    int from = 0, to = k;
    if (!open) {
      const uint64_t ma = rm_ballot<G>(gl < k && ring == ab.x, g0), mb = rm_ballot<G>(gl < k && ring == ab.y, g0);
      if (!ma || !mb) {
        if (gl == 0) DO::err(&V.c->err, 10);
        return;
      }
      from = __ffsll((unsigned long long)ma) - 1;
      to = __ffsll((unsigned long long)mb) - 1;
    }
    for (int side = 0; side < sides && ne >= 0; side++) {
      const int m = open ? k + 1 : (to - from + k) % k + 1;
      if (m == 2) {
        if (sl_side >= 0) {
          if (gl == 0) DO::err(&V.c->err, 11);
          return;
        }
        sl_side = side;
        sl_x = __shfl(onb, g0 + from);
        sl_u = __shfl(ring, g0 + from);
        sl_v = __shfl(ring, g0 + to);
      } else {
        int src = from + gl;
        if (!open && src >= k) src -= k;
        src = g0 + (gl < m ? src : 0);
        const int pv = __shfl(ring, src);
        const double2 B = make_double2(__shfl(R.x, src), __shfl(R.y, src));
        int info = __shfl(onb, src), sd = __shfl(osd, src);
        if (gl == m - 1) {
          info = open ? -1 : kRmClose - side;
          sd = info4.y;
        }
        ne = rm_clip(S, P, m, pv, B, info, sd, ne, side);
      }
      const int x = from;
      from = to;
      to = x;
    }
  }
  if (ne < 0 || ne > k) {
    if (gl == 0) DO::err(&V.c->err, 12);
    return;
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  // the first ne star slots take the triangles; the rest are freed
  const int np = V.c->np;
  int v[3], nn[3], ss[3], code[3];
#pragma unroll
  for (int h = 0; h < 3; h++) {
    const int at = 3 * min(gl, max(ne - 1, 0)) + h;
    v[h] = S.ev[at];
    code[h] = S.en[at];
    ss[h] = S.es[at];
    int from = -1;  // the emitted triangle across the edge
    if (gl < ne && code[h] <= kRmTri) from = kRmTri - code[h];
    const bool close = gl < ne && (code[h] == kRmClose || code[h] == kRmClose - 1);
    if (close && sl_side < 0) from = S.clos[code[h] == kRmClose ? 1 : 0];
    const int s = __shfl(slot, g0 + max(from, 0));
    nn[h] = from >= 0 ? s : (close ? sl_x : code[h]);
    if (close && nn[h] < 0) DO::err(&V.c->err, 13);
  }
  if (gl < ne) {
    ff_store(V, slot, v[0], v[1], v[2], nn[0], nn[1], nn[2], ss[0], ss[1], ss[2]);
#pragma unroll
    for (int h = 0; h < 3; h++) {
      if (code[h] >= 0) {
        const int j = ff_eidx(V.tv[code[h]], v[h == 2 ? 0 : h + 1], v[h]);
        if (j < 0) DO::err(&V.c->err, 14);
        else ff_set(V, V.tn, code[h], j, slot);
      }
      if (v[h] >= V.nV && v[h] != p && v[h] < V.nV + np) V.vtri[v[h] - V.nV] = slot;
    }
    ff_wrote<DO>(V, slot, wst, tst);
  } else if (gl < k) {
    V.tv[slot] = make_int4(-1, -1, -1, 0);
    V.tn[slot] = make_int4(-1, -1, -1, 0);
    V.dead[DO::append(&V.c->n_dead)] = slot;
  }
  const int partner = sl_side >= 0 && !open ? __shfl(slot, g0 + max(S.clos[sl_side ^ 1], 0)) : -1;
  if (gl == 0) {
    if (sl_side >= 0) {
      const int4 tx = sl_x >= 0 ? V.tv[sl_x] : make_int4(-1, -1, -1, 0);
      const int jx = sl_x >= 0 ? ff_eidx(tx, sl_v, sl_u) : -1;
      if (jx < 0 || (!open && S.clos[sl_side ^ 1] < 0)) {
        DO::err(&V.c->err, 18);
        return;
      }
      ff_set(V, V.tn, sl_x, jx, partner);
      ff_set(V, V.ts, sl_x, jx, info4.y);
      V.tv[sl_x] = make_int4(tx.x, tx.y, tx.z, tx.w | (1 << jx));
      ff_wrote<DO>(V, sl_x, wst, tst);
    }
    V.alive[r] = 0;
    V.red[r] = 0;
    DO::inc64(&V.c->removals);
  }
}

// (star_used is emptied here: the next pass's mark takes from it)
__global__ __launch_bounds__(kRmBlk) void kf_rm_apply(FfView V, const int32_t *list, const int32_t *n_list,
                                                      int32_t *next, int32_t *n_next, uint64_t pbase, int wst, int tst) {
  // a wave's groups and the whole wave use the same memory, one after the other
  union RmMem {
    RmShared<kRmGrp> grp[64 / kRmGrp];
    RmShared<kRmWave> wave;
  };
  __shared__ RmMem s_rm[kRmBlk / 64];
  RmMem &mem = s_rm[threadIdx.x / 64];
  const int n = *n_list, gl = threadIdx.x % kRmGrp, g = threadIdx.x / kRmGrp, g0 = __lane_id() - gl;
  if (blockIdx.x == 0 && threadIdx.x == 0) V.c->star_used = 0;
  const int32_t *stars = (const int32_t *)V.fc0, *rings = (const int32_t *)V.fc1;
  for (int base = blockIdx.x * kRmPer; base < n; base += gridDim.x * kRmPer) {
    const int i = base + g, r = i < n ? list[i] : -1;
    const int off = r >= 0 ? V.moved[i] : -1;
    int k = 0, open = 0;
    bool own = off >= 0;
    if (own) {
      const uint64_t prio = pbase | (uint64_t)(r + 1);
      k = stars[off] >> 1;
      open = stars[off] & 1;
      bool mine = V.vmark[V.nV + r] == prio;
      for (int q = gl; q < k + open; q += kRmGrp) mine = mine && V.vmark[rings[off + q]] == prio;
      own = rm_ballot<kRmGrp>(mine, g0) == (1ull << kRmGrp) - 1;
    }
    bool left = r >= 0 && !own;
    // the links too large for a group: the whole wave, one after the other, or
    // one thread, which may find no room
    for (uint64_t big = __ballot(own && k + open > kRmGrp && gl == 0); big; big &= big - 1) {
      const int l = __ffsll((unsigned long long)big) - 1;
      const int lr = __shfl(r, l), lk = __shfl(k, l), lopen = __shfl(open, l), loff = __shfl(off, l);
      if (lk + lopen <= kRmWave) {
        rm_remove<kRmWave>(V, mem.wave, lr, lk, lopen, stars + loff + 1, wst, tst);
      } else {
        int ok = 1;
        if (__lane_id() == l) {
          V.red[lr] |= 4;
          ff_rm_apply_one<DO>(V, lr, wst, tst);
          ok = V.red[lr] == 0;
        }
        if (__shfl(ok, l) == 0 && g0 == l) left = true;
      }
      if (g0 == l) own = false;
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    const int at = rm_take(n_next, left ? 1 : 0);
    if (left && gl == 0) next[at] = r;
    if (own) rm_remove<kRmGrp>(V, mem.grp[g & (64 / kRmGrp - 1)], r, k, open, stars + off + 1, wst, tst);
  }
}

// The number of kept midpoints (the midpoints are ranks 0..nmid-1), once
// the ranks are scanned (one thread).
__global__ void kf_nwin_mid(FfView V) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  const int np = V.c->np, nmid = V.c->nmid;
  V.c->nwin_mid = nmid < np ? ff_newid(V, nmid) : V.c->nwin;
}

__global__ void kf_final_point(FfView V) {
  const int np = V.c->np;
  FF_LOOP(r, np) ff_final_point_one<DO>(V, r);
}

__global__ void kf_final_tri(FfView V) {
  const int n = V.c->n_touched;
  FF_LOOP(i, n) ff_final_tri_one<DO>(V, i);
}

__global__ void kf_final_mid(FfView V) {
  FF_LOOP(i, V.nmk) ff_final_mid_one<DO>(V, i);
}

__global__ void kf_final_flag(FfView V) {
  const int nmid = V.c->nmid;
  FF_LOOP(k, V.nS) ff_final_flag_one<DO>(V, k, nmid);
}

__global__ void kf_final_flag_clear(FfView V) {
  const int nmid = V.c->nmid;
  FF_LOOP(r, nmid) ff_final_flag_clear_one<DO>(V, r);
}

__global__ void kf_compact_list(FfView V, int n_alloc, int n_live) {
  const int nd = V.c->n_dead;
  FF_LOOP(i, nd) ff_compact_hole_one<DO>(V, i, n_live);
  FF_LOOP(j, n_alloc - n_live) ff_compact_mover_one<DO>(V, n_live + j);
}

__global__ void kf_compact_move(FfView V) {
  const int n = min(V.c->n_hole, V.c->n_mover);
  FF_LOOP(i, n) ff_compact_move_one<DO>(V, i);
}

__global__ void kf_compact_fix(FfView V, int n_live) {
  const int n = min(V.c->n_hole, V.c->n_mover);
  FF_LOOP(i, n) ff_compact_fix_one<DO>(V, i, n_live);
}

__global__ void kf_rotate(FfView V, int n) {
  FF_LOOP(s, n) ff_rotate_one<DO>(V, s);
}

__global__ void kf_all_slots(FfView V, int n, int wst) {
  FF_LOOP(s, n) {
    V.wstamp[s] = wst;
    V.list_out[s] = s;
  }
  if (blockIdx.x == 0 && threadIdx.x == 0) *V.n_out = n;
}

#undef FF_LOOP

}  // namespace gdp
