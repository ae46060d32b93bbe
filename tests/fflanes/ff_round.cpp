// ff_round.cpp -- the sequential host run of a Flip-Flop round
// (tests/ffemu/ff_emu.cpp) with its removal passes replaced by the removal
// kernels' own text, lane by lane (ff_lanes.cpp; TEST INFRASTRUCTURE).
#include <algorithm>
#include <cstring>
#include <vector>

#include "gdp_ff_core.h"

using namespace gdp;

extern "C" int ffemu_removal_pass(const FfView *V, const int32_t *list, const int32_t *n_list, int32_t *next,
                                  int32_t *n_next, uint64_t pbase, int wst, int tst, int grid);

namespace {
// A pass of the sequential run marks, decides and applies point after point;
// here the points that still have to go are listed while they are marked, and
// the kernels take the whole list with the last point that is applied.
struct Pass {
  std::vector<int32_t> list, next;
  uint64_t pbase = 0;
  int applied = 0;
} g_pass;
template <class O>
void lanes_mark_one(const FfView &V, int r, uint64_t pbase) {
  g_pass.pbase = pbase;
  if (V.alive[r] && V.red[r]) g_pass.list.push_back(r);
}
template <class O>
void lanes_decide_one(const FfView &, int, uint64_t) {}
template <class O>
void lanes_apply_one(const FfView &V, int, int wst, int tst) {
  if (++g_pass.applied < V.c->np) return;
  const int32_t n = (int32_t)g_pass.list.size();
  int32_t left = 0;
  g_pass.next.resize(n + 1);
  V.c->star_used = 0;
  if (n > 0 && ffemu_removal_pass(&V, g_pass.list.data(), &n, g_pass.next.data(), &left, g_pass.pbase, wst, tst,
                                  (n + 15) / 16))
    FfHostOps::err(&V.c->err, 203);
  V.c->n_left = left;
  g_pass = Pass();
}
}  // namespace

#define ff_rm_mark_one lanes_mark_one
#define ff_rm_decide_one lanes_decide_one
#define ff_rm_apply_one lanes_apply_one
#include "../ffemu/ff_emu.cpp"
