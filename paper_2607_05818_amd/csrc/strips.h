// Heights of the strips that the stencil kernels march over (Strip in
// reff_internal.h).  Plain C++ (no HIP types): a plan is anything with the
// members n, plane, nx and cbase of a solve block (PlanDesc).
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <map>
#include <vector>

namespace reff {

constexpr int64_t STRIP_WIDTH = 32;    // columns of a strip
constexpr int64_t STRIP_COLUMNS = 64;  // right-hand sides per node

// Most strips of 64 rows of a launch group of n nodes in `blocks` solve blocks:
// as many as full-width ones would be, or 1024 per block (2048 to 16384 in all, so
// that a block that runs on alone still spreads); groups above it take taller
// ones.  Each float32 strip keeps its partial Grams (131 KB, written and summed in
// every iteration) whatever it holds: 64 rows of a full-width strip are 2048
// nodes with 6.3 MB of vectors, of a tier one node wide 64 nodes with 0.2 MB, so a
// group of 31M nodes of one-wide tiers would keep 63 GB of partials beside its
// 96 GB of vectors.
inline int64_t max_strips(int64_t n, int64_t blocks) {
  const int64_t few = std::min<int64_t>(16384, std::max<int64_t>(2048, 1024 * blocks));
  return std::max(few, n / (64 * STRIP_WIDTH));
}

// Most rows of one strip for the three-step Chebyshev pass, which addresses
// a strip's rows through unsigned 32-bit byte offsets from a base three rows
// before it: (rows + 8) x nx x 64 words stay below 2^31 bytes.  0 when even
// one row does not fit (the pass is then not used).
inline int64_t max_strip_rows(int64_t nx, size_t word) {
  return std::max<int64_t>(0, (int64_t(1) << 31) / (nx * STRIP_COLUMNS * (int64_t)word) - 8);
}

// y segments of a tier of ny rows for strips of about H rows; from 64 on a tier
// is cut only into segments of H rows or more.
inline int64_t strip_segments(int64_t ny, int64_t H) {
  return H >= 64 ? std::max<int64_t>(1, ny / H) : (ny + H - 1) / H;
}

// Rows per strip of a group: a launch takes as many rounds as its strips fill
// the chip's workgroup slots (`slots`: one per CU in float64, two in float32),
// and a round the rows of a mean strip and `extra` more (halo rows, prologue), so
// the height with the fewest row times in all is taken, the taller one on a tie
// (less halo traffic), up to 64 rows so that a block that runs on alone still
// spreads.  Where those are more than max_strips, the height with the
// fewest row times from the first that keeps it to twice that one.  The
// stacks of a batch converge at different times: there the rounds of half the
// strips count as well.  Against about 1024 strips per launch whatever their rounds:
// float64: 8-row strips in four rounds at one block of 4 x 256 x 256 and 6-row
// strips in five at four blocks of 3 x 128 x 128 took 194 and 166 us a pass, one
// round of 32 and 26 rows 153 and 127 us; stacks of 4000 to 12000 nodes take
// one row per strip (12 columns on 82 x 56 nodes 4.7 ms, 5.8 with eight rows at
// least).  float32: a batch of 24 plans of 30 to 233 nodes a side 2.4 rounds of
// 64 rows, 97.9 ms, now 94.3; 91 samples of 2 x 158 x 195 8.5 -> 7.7 ms; 4 x 512 x
// 512 keeps two rounds of 64.  When the blocks of a batch leave is not known here,
// and half the strips a guess: 14 drawn batches of 2 to 22 plans took from 3 %
// more to 12 % less time, 3 % less on average; of the heights from 16 to 60 the
// best was up to 5 % better than the one taken.  Narrow tiers, 64 samples mixed: 4 x 8 x 200000 in
// 12,500 strips of 64 rows 1236 ms, in 1024 to 2048 taller ones 1208; 1 x 1 x 1.1M
// 4048 and 3998 ms, and 2.2 GB less.
template <typename Plan>
int64_t strip_rows(const std::vector<Plan>& plans, int64_t slots, double extra) {
  bool batch = false;
  std::map<int64_t, int64_t> tiers;  // rows of a tier -> 32-wide columns of that many rows
  int64_t rows = 0, nodes = 0;
  for (const Plan& p : plans) {
    const int64_t ny = p.plane / p.nx, across = p.n / p.plane * ((p.nx + STRIP_WIDTH - 1) / STRIP_WIDTH);
    batch = batch || p.cbase != plans[0].cbase;
    tiers[ny] += across;
    rows += across * ny;
    nodes += p.n;
  }
  auto count = [&](int64_t H) {
    int64_t n = 0;
    for (const auto& t : tiers) n += t.second * strip_segments(t.first, H);
    return n;
  };
  int64_t best = 64;
  double cost = INFINITY;
  auto consider = [&](int64_t H) {
    const int64_t n = count(H);
    const int64_t rounds = (n + slots - 1) / slots + (batch ? (n / 2 + slots - 1) / slots : 0);
    const double c = (double)rounds * ((double)rows / (double)n + extra);
    if (c <= cost) cost = c, best = H;
  };
  const int64_t most = max_strips(nodes, (int64_t)plans.size());
  if (count(64) <= most) {
    for (int64_t H = 1; H <= 64; ++H) consider(H);
    return best;
  }
  int64_t H = 64;
  const int64_t tallest = tiers.rbegin()->first;
  while (count(H) > most && H < tallest) H += (H + 63) / 64;
  for (const int64_t end = 2 * H; H <= end; H += (H + 63) / 64) consider(H);
  return best;
}

// Strips per launch that a tuning database can name; DEFAULT_STRIPS stands for
// the heights of strip_rows, the layout without a database, so that a tuned call
// has it among its candidates.
constexpr int DEFAULT_STRIPS = 1024;
constexpr int STRIP_TARGETS[] = {256, 512, DEFAULT_STRIPS, 2048};

// Rows per strip of a group for a target of strips, 0: as many segments as make
// about that many.
template <typename Plan>
int64_t target_rows(const std::vector<Plan>& plans, bool fp32, int target) {
  if (target != DEFAULT_STRIPS) return 0;
  return fp32 ? strip_rows(plans, 512, 5) : strip_rows(plans, 256, 7);
}

}  // namespace reff
