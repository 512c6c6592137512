// Host check of the strip heights (strips.h): the strips of a launch group,
// counted here tier by tier, against the cap on their number.
#include <cstdio>
#include <cstdlib>

#include "../../paper_2607_05818_amd/csrc/strips.h"

using namespace reff;

struct Plan {
  int64_t cbase, n, plane;
  int32_t nx;
};

static Plan plan(int64_t cbase, int64_t nt, int64_t nx, int64_t ny) {
  return Plan{cbase, nt * nx * ny, nx * ny, (int32_t)nx};
}

static int64_t strips_of(const std::vector<Plan>& g, int64_t rows) {
  int64_t n = 0;
  for (const Plan& p : g) {
    const int64_t ny = p.plane / p.nx, segs = strip_segments(ny, rows), h = (ny + segs - 1) / segs;
    n += p.n / p.plane * ((p.nx + STRIP_WIDTH - 1) / STRIP_WIDTH) * ((ny + h - 1) / h);
  }
  return n;
}

static int bad = 0;

// At most `cap` strips; heights lo .. hi, of which `rows` may be more than a tier
// has.
static void check(const char* name, const std::vector<Plan>& g, int64_t cap, int64_t lo, int64_t hi) {
  for (int fp32 = 0; fp32 < 2; ++fp32) {
    const int64_t rows = target_rows(g, fp32 != 0, DEFAULT_STRIPS), n = strips_of(g, rows);
    const bool ok = n <= cap && rows >= lo && rows <= hi;
    printf("%s, %s: %lld rows, %lld strips%s\n", name, fp32 ? "float32" : "float64", (long long)rows,
           (long long)n, ok ? "" : "  FAIL");
    bad |= !ok;
  }
}

int main() {
  // narrow tiers: 64 rows of them would make 484375, 60544, 31250, 28124, 18400,
  // 46870 and 24000 strips
  check("1 x 31e6", {plan(0, 1, 1, 31000000)}, 31000000 / 2048, 65, 31000000);
  check("4 x 8 x 968750", {plan(0, 4, 8, 968750)}, 31000000 / 2048, 65, 968750);
  check("2 x 1 x 1e6", {plan(0, 2, 1, 1000000)}, 2048, 65, 1000000);
  check("2 x 33 x 450000", {plan(0, 2, 33, 450000)}, 29700000 / 2048, 65, 450000);
  check("200 blocks of 33 x 3000", std::vector<Plan>(200, plan(0, 1, 33, 3000)), 16384, 65, 3000);
  check("10 blocks of 1 x 300000", std::vector<Plan>(10, plan(0, 1, 1, 300000)), 10240, 65, 600);
  std::vector<Plan> g;
  for (int i = 0; i < 3000; ++i) g.push_back(plan(i, 2, 16, 300 + i % 7));
  check("3000 plans of 2 x 16 x 300", g, 16384, 65, 1000);
  // a tier's columns one strip each at the least
  g.clear();
  for (int i = 0; i < 20000; ++i) g.push_back(plan(i, 1, 20, 20));
  check("20000 plans of 20 x 20", g, 20000, 20, 256);
  // heights the cap does not touch
  check("4 x 512 x 512", {plan(0, 4, 512, 512)}, 1024, 32, 64);
  g.assign(8, plan(0, 4, 512, 512));
  check("8 blocks of 4 x 512 x 512", g, 4096, 64, 64);
  check("8 x 2048 x 2048", {plan(0, 8, 2048, 2048)}, 16384, 64, 64);
  check("8 x 1000 x 1000", {plan(0, 8, 1000, 1000)}, 4096, 60, 64);
  check("82 x 56", {plan(0, 1, 82, 56)}, 168, 1, 1);
  // a tuning database has the layout of a call without one among its candidates
  bool found = false;
  for (int t : STRIP_TARGETS) {
    const std::vector<Plan> one{plan(0, 2, 158, 195)};
    found |= target_rows(one, true, t) == strip_rows(one, 512, 5) &&
             target_rows(one, false, t) == strip_rows(one, 256, 7);
  }
  if (!found) printf("the default heights are no candidate  FAIL\n");
  bad |= !found;
  printf(bad ? "FAILED\n" : "all ok\n");
  return bad;
}
