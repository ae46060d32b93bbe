// ff_lanes.cpp -- the removal kernels of the Flip-Flop insertion, as they
// stand in gdp_ff.hip, run on the host lane by lane (TEST INFRASTRUCTURE).
//
// A workgroup is kRmBlk coroutines, one for each lane, that run one after the
// other up to their next collective operation (a shuffle, a ballot, a fence, a
// barrier).  The collective is carried out when every lane of its scope has
// come to it: the workgroup for a barrier, else the lanes of the function's
// group (its template parameter G) or the wave.  Where the lanes of a group
// wait at different places (a ballot under a condition), the ballot is carried
// out for those lanes alone that came to it, as the hardware does.  Stores take
// effect at once, so a lane that reads what another one writes without a
// collective in between reads it in the worst order or finds nothing.  (Two
// turns of a kernel's loop over its list are kept in order by the lanes of a
// wave running together, which this does not do: a grid has to have a group for
// every entry.)
#include <ucontext.h>

#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include <hip/hip_runtime.h>

namespace emu {
constexpr int kLanes = 256;
enum Op { kRun, kDone, kBarrier, kFence, kShfl, kBallot };
struct Lane {
  ucontext_t at;
  std::vector<char> stack;
  Op op = kDone;
  int scope = 64;         // lanes of the collective
  const char *where = nullptr;
  int line = 0, src = 0;
  uint64_t in = 0, out = 0;
};
struct Dim {
  unsigned x = 0;
};
inline Lane lanes[kLanes];
inline ucontext_t main_ctx;
inline int cur = 0;
inline Dim tid, bid, bdim{kLanes}, gdim;
inline void (*body)(void *) = nullptr;
inline void *arg = nullptr;
inline const char *stuck = nullptr;

inline void entry() {
  body(arg);
  lanes[cur].op = kDone;
  swapcontext(&lanes[cur].at, &main_ctx);
}
inline int scope_of(const char *fn) {
  static std::map<const char *, int> known;
  int &s = known[fn];
  if (!s) s = strstr(fn, "G = 16") ? 16 : 64;
  return s;
}
inline uint64_t wait(Op op, uint64_t in, int src, const char *fn, int line) {
  Lane &l = lanes[cur];
  l.op = op;
  l.scope = op == kBarrier ? kLanes : scope_of(fn);
  l.where = fn;
  l.line = line;
  l.in = in;
  l.src = src;
  swapcontext(&l.at, &main_ctx);
  return l.out;
}
template <class T>
T shfl(T x, int src, const char *fn, int line) {
  static_assert(sizeof(T) <= 8, "a shuffle moves up to 8 bytes");
  uint64_t b = 0;
  memcpy(&b, &x, sizeof x);
  b = wait(kShfl, b, src, fn, line);
  memcpy(&x, &b, sizeof x);
  return x;
}
inline uint64_t ballot(bool x, const char *fn, int line) { return wait(kBallot, x, 0, fn, line); }

// Carries out the collective of lanes[lo .. hi) for the lanes that wait at the
// same place as lane `first`.
inline void carry_out(int lo, int hi, int first) {
  const Lane &f = lanes[first];
  const Op op = f.op;
  const char *where = f.where;
  const int line = f.line, wave = first & ~63;
  auto in = [&](int i) { return lanes[i].op == op && lanes[i].where == where && lanes[i].line == line; };
  uint64_t bits = 0;
  std::vector<int> who;
  for (int i = lo; i < hi; i++)
    if (in(i)) {
      who.push_back(i);
      if (op == kBallot && lanes[i].in) bits |= 1ull << (i - wave);
    }
  for (int i : who) {
    if (op == kBallot) lanes[i].out = bits;
    if (op == kShfl) lanes[i].out = lanes[wave + (lanes[i].src & 63)].in;
  }
  for (int i : who) lanes[i].op = kRun;
}

// Runs fn for a grid of workgroups; false if a workgroup got stuck.
inline bool launch(int grid, void (*fn)(void *), void *a) {
  body = fn;
  arg = a;
  gdim.x = (unsigned)grid;
  for (int b = 0; b < grid; b++) {
    bid.x = (unsigned)b;
    for (int i = 0; i < kLanes; i++) {
      Lane &l = lanes[i];
      l.stack.resize(128 << 10);
      getcontext(&l.at);
      l.at.uc_stack.ss_sp = l.stack.data();
      l.at.uc_stack.ss_size = l.stack.size();
      l.at.uc_link = &main_ctx;
      makecontext(&l.at, entry, 0);
      l.op = kRun;
    }
    for (;;) {
      int done = 0;
      for (int i = 0; i < kLanes; i++) {
        if (lanes[i].op == kDone) done++;
        if (lanes[i].op != kRun) continue;
        cur = i;
        tid.x = (unsigned)i;
        swapcontext(&main_ctx, &lanes[i].at);
        if (lanes[i].op == kDone) done++;
      }
      if (done == kLanes) break;
      bool moved = false;
      for (int scope : {16, 64, kLanes})
        for (int lo = 0; lo < kLanes; lo += scope) {
          bool all = true;
          for (int i = lo; i < lo + scope; i++)
            all = all && lanes[i].op > kDone && lanes[i].scope == scope && lanes[i].op == lanes[lo].op &&
                  lanes[i].where == lanes[lo].where && lanes[i].line == lanes[lo].line;
          if (all) {
            carry_out(lo, lo + scope, lo);
            moved = true;
          }
        }
      for (int scope : {16, 64})
        for (int lo = 0; lo < kLanes && !moved; lo += scope)
          for (int i = lo; i < lo + scope && !moved; i++)
            if (lanes[i].op == kBallot && lanes[i].scope == scope) {
              carry_out(lo, lo + scope, i);
              moved = true;
            }
      if (!moved) {
        stuck = "lanes wait at different collectives";
        return false;
      }
    }
  }
  return true;
}
}  // namespace emu

// The device's names for the kernels' text.
#undef __shared__
#define __shared__ static
#undef __launch_bounds__
#define __launch_bounds__(...)
#define threadIdx emu::tid
#define blockIdx emu::bid
#define blockDim emu::bdim
#define gridDim emu::gdim
#define __shfl(x, s) emu::shfl((x), (s), __PRETTY_FUNCTION__, __LINE__)
#define __ballot(x) emu::ballot((x) != 0, __PRETTY_FUNCTION__, __LINE__)
#define __syncthreads() (void)emu::wait(emu::kBarrier, 0, 0, __PRETTY_FUNCTION__, __LINE__)
#define __builtin_amdgcn_fence(...) (void)emu::wait(emu::kFence, 0, 0, __PRETTY_FUNCTION__, __LINE__)
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __lane_id() (emu::cur & 63)
#define __ffsll(x) __builtin_ffsll((long long)(x))
#define __popcll(x) __builtin_popcountll(x)
template <class T>
inline T atomicAdd(T *p, T v) { const T o = *p; *p = o + v; return o; }
template <class T>
inline T atomicMax(T *p, T v) { const T o = *p; *p = std::max(o, v); return o; }
template <class T>
inline T atomicExch(T *p, T v) { const T o = *p; *p = v; return o; }
template <class T>
inline T atomicOr(T *p, T v) { const T o = *p; *p = o | v; return o; }
template <class T>
inline T atomicCAS(T *p, T c, T v) { const T o = *p; if (o == c) *p = v; return o; }
using std::min;
using std::max;

#include "gdp_ff_core.h"
#define FfDevOps FfHostOps
#include "gdp_ff.hip"

using namespace gdp;

// Points taken in by the passes so far: link of a group's, a wave's, more.
extern "C" int64_t ffemu_links[3];
int64_t ffemu_links[3];

// One removal pass over the list, as ff_line8 launches it: both kernels, with a
// grid of the given workgroups.  Returns 0, or 1 if the lanes got stuck.
extern "C" int ffemu_removal_pass(const FfView *V, const int32_t *list, const int32_t *n_list, int32_t *next,
                                  int32_t *n_next, uint64_t pbase, int wst, int tst, int grid) {
  struct Args {
    const FfView &V;
    const int32_t *list, *n_list;
    int32_t *next, *n_next;
    uint64_t pbase;
    int wst, tst;
  } a{*V, list, n_list, next, n_next, pbase, wst, tst};
  static_assert(kRmBlk == emu::kLanes && kRmGrp == 16, "the kernels' groups and workgroup");
  if (!emu::launch(grid, [](void *p) {
        Args &x = *(Args *)p;
        kf_rm_mark(x.V, x.list, x.n_list, x.n_next, x.pbase);
      }, &a))
    return 1;
  for (int i = 0; i < *n_list && !V->c->err; i++) {
    const int s = ((const int32_t *)V->fc0)[V->moved[i]], link = (s >> 1) + (s & 1);
    ffemu_links[link <= kRmGrp ? 0 : (link <= kRmWave ? 1 : 2)]++;
  }
  return emu::launch(grid, [](void *p) {
    Args &x = *(Args *)p;
    kf_rm_apply(x.V, x.list, x.n_list, x.next, x.n_next, x.pbase, x.wst, x.tst);
  }, &a) ? 0 : 1;
}
