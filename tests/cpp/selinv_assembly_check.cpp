// Host check of the reads of a front's assembly (k_assemble in selinv.hip):
// for every child that has_update names, the kernel reads entries (a, b),
// 0 <= a, b < F - k, of the matrix that starts at off + k F + k with column
// stride F, and (0, 0) of it wherever a row or column of the parent has no
// counterpart.  All of them have to lie inside the child's own block; no child
// with an update matrix may be left out.
#include <cstdio>
#include <cstdlib>
#include <string>
#include <vector>

#include "../../paper_2607_05818_amd/csrc/selinv_plan.h"

using namespace reff;

static void chk(bool c, const char* what, const char* stack) {
  if (!c) {
    fprintf(stderr, "FAIL %s: %s\n", stack, what);
    exit(1);
  }
}

// An nt x nx x ny stack of unit conductances, TSVs at every third column.
static SelinvPlan plan_of(int nt, int nx, int ny, const std::vector<int32_t>& pads) {
  std::vector<double> gx((size_t)nt * ny * (nx - 1), 1.0), gy((size_t)nt * (ny - 1) * nx, 1.0);
  std::vector<int32_t> txy;
  if (nt > 1)
    for (int v = 0; v < nx * ny; v += 3) txy.push_back(v % nx), txy.push_back(v / nx);
  std::vector<double> tg(txy.size() / 2 * (size_t)(nt - 1), 1.0);
  SelinvPlan P;
  std::string err;
  if (!build_selinv_plan(nt, nx, ny, gx.data(), gy.data(), (int32_t)(txy.size() / 2), txy.data(),
                         tg.data(), (int32_t)(pads.size() / 2), pads.data(), 16, P, err)) {
    fprintf(stderr, "FAIL plan: %s\n", err.c_str());
    exit(1);
  }
  return P;
}

// Returns how many fronts below a parent have no update rows.
static int check(const SelinvPlan& P, const char* name) {
  int empty = 0;
  for (const SnFront& g : P.fronts) {
    if (g.parent < 0) {
      chk(!has_update(g), "a root has no parent to add to", name);
      continue;
    }
    chk(g.rank == 0 || g.rank == 1, "rank", name);
    if (g.F == g.k) ++empty;
    if (!has_update(g)) {
      chk(g.F == g.k, "every update matrix is added", name);
      continue;
    }
    const int64_t first = g.off + (int64_t)g.k * g.F + g.k, q = g.F - g.k;
    const int64_t last = first + (q > 0 ? (q - 1) * g.F + q - 1 : 0), end = g.off + (int64_t)g.F * g.F;
    chk(first < end && last < end, "reads inside the child's block", name);
    chk(end <= P.arena, "block inside the arena", name);
  }
  printf("%s: %zu fronts, %d without update rows\n", name, P.fronts.size(), empty);
  return empty;
}

int main() {
  std::vector<int32_t> wall;  // the root's wall of a 31-wide tier
  for (int y = 0; y < 16; ++y) wall.push_back(15), wall.push_back(y);
  const SelinvPlan a = plan_of(1, 67, 1, {50, 0}), b = plan_of(1, 31, 16, wall),
                   c = plan_of(3, 20, 17, {3, 4, 11, 2}), d = plan_of(1, 40, 1, {20, 0, 10, 0, 31, 0});
  chk(check(a, "67 x 1, one pad") > 0, "has an empty update set", "67 x 1, one pad");
  chk(check(b, "31 x 16, wall of pads") > 0, "has an empty update set", "31 x 16, wall of pads");
  chk(check(d, "40 x 1, pads on walls") > 0, "has an empty update set", "40 x 1, pads on walls");
  check(c, "3 x 20 x 17");
  std::vector<int64_t> base;
  chk(check(merge_selinv_plans({c, a, b, d}, base), "forest") > 0, "has an empty update set", "forest");
  printf("all ok\n");
  return 0;
}
