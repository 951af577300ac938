// Host-only checker of the routes that the planner gives the forwards, built by the CPU
// test suite with g++ under AddressSanitizer and UndefinedBehaviorSanitizer: the route
// follows from sizes and flags, never from the blocks or (down to the least scratch that
// a route needs) from the budget.  Prints "route_check OK" and returns 0 when every check
// holds.
#include <cstdio>
#include <random>

#include "plan.h"

using namespace ccl;

static int g_fail = 0;
#define CHECK(cond)                                                                     \
  do {                                                                                  \
    if (!(cond)) {                                                                      \
      std::fprintf(stderr, "FAILED %s:%d: %s (o=%d v=%d P=%d flags=%u)\n", __FILE__,    \
                   __LINE__, #cond, o, v, P, opts.flags);                               \
      ++g_fail;                                                                         \
    }                                                                                   \
  } while (0)

static int route(const Plan& p) {  // -1: laid out past the plan's scratch
  FoldPlan f;
  StackedPlan q;
  if (plan_fold(p, &f)) return f.bytes <= p.bytes ? 1 : -1;
  if (plan_stacked_i8(p, &q)) return q.bytes <= p.bytes ? 1 : -1;
  return 0;
}

static void forward_routes(std::mt19937_64& rng, int precision, int plans) {
  int folded = 0, direct = 0, less = 0;
  for (int it = 0; it < plans; ++it) {
    cc_ladder_opts opts{};
    if (precision == CC_LADDER_SPLIT_INT8) opts.split_slices = it % 3 ? 0 : 4;
    const int o = 1 + static_cast<int>(rng() % 76), v = 40 + static_cast<int>(rng() % 260);
    const int P = 1 + static_cast<int>(rng() % (4 * (o + v)));
    const unsigned sets[] = {0, CC_LADDER_PAIR_SYMMETRIC, CC_LADDER_EXCHANGE,
                             CC_LADDER_PAIR_SYMMETRIC | CC_LADDER_EXCHANGE,
                             CC_LADDER_PAIR_SYMMETRIC | CC_LADDER_CHECK_SYMMETRY};
    opts.flags = sets[rng() % 5];
    Plan whole, p;
    CHECK(make_plan(o, v, P, precision, 0, 0, &opts, &whole) == CC_LADDER_OK);
    const int r = route(whole);
    r ? ++folded : ++direct;
    // any block, without a limit
    for (int k = 0; k < 4; ++k) {
      opts.a_block = k == 0 ? 1 : 1 + static_cast<int>(rng() % v);
      CHECK(make_plan(o, v, P, precision, 0, 0, &opts, &p) == CC_LADDER_OK);
      CHECK(route(p) == r);
    }
    opts.a_block = 1;
    CHECK(make_plan(o, v, P, precision, 0, 0, &opts, &p) == CC_LADDER_OK);
    const size_t least = p.bytes;
    opts.a_block = 0;
    // any budget from the least on; below it every plan is the direct route's
    for (int k = 0; k < 6; ++k) {
      const size_t span = whole.bytes > least ? whole.bytes - least : 0;
      const size_t budget = k == 0 ? least : least + (span ? rng() % span : 0);
      CHECK(make_plan(o, v, P, precision, 0, budget, &opts, &p) == CC_LADDER_OK);
      CHECK(p.bytes <= budget && route(p) == r);
      const size_t under = k == 0 ? least - 1 : 1 + rng() % (least - 1);
      const int rc = make_plan(o, v, P, precision, 0, under, &opts, &p);
      CHECK(rc == CC_LADDER_OK || rc == CC_LADDER_ENOMEM);
      if (!rc) {
        CHECK(p.bytes <= under && route(p) == 0);
        ++less;
      }
    }
  }
  cc_ladder_opts opts{};
  const int o = 0, v = 0, P = 0;
  CHECK(folded > plans / 5 && direct > plans / 5 && less > plans / 5);
}

// Products whose kernel was measured against the alternatives.
static void measured_picks() {
  cc_ladder_opts opts{};
  const int o = 0, v = 0, P = 0;
  // float32 rows of 4096: 0.62 ms on the register-direct kernel, 0.40 on 64 x 64 tiles
  CHECK(pick_tiles(kTilesKC, 1681, 2624, 4096, 1681, 2624, 8, 4, false, true).side == 0);
  // float64 X terms with odd rows, K in ranges on the register-direct kernel: 15 ms, 9.3 in
  // one piece (o=44 v=229); 0.04 ms for 0.21 (o=8 v=101)
  CHECK(!split_pays(pick_part_tiles(1936, 1936, 52441, 2, 1639, 8, false), 1936, 1936, 52441, 2, 3278, 8));
  CHECK(split_pays(pick_part_tiles(64, 64, 10201, 9, 71, 8, false), 64, 64, 10201, 9, 638, 8));
  // odd float64 rows: 1.84 ms on 64 x 128 tiles, 2.61 on the register-direct kernel; 10.0,
  // 12.6 on 128 x 256; 2.0 on 128 x 256, 3.2 on the register-direct kernel; and with row-contiguous
  // columns 0.24 ms on the register-direct kernel, 0.30 on 128 x 256
  const TilePick kc1 = pick_tiles(kTilesKCDword, 3249, 3249, 4489, 3249, 3249, 281, 8, true, true);
  const TilePick kc2 = pick_tiles(kTilesKCDword, 4900, 4900, 12321, 4900, 4900, 771, 8, true, true);
  const TilePick kc3 = pick_tiles(kTilesKCDword, 2704, 2704, 7569, 2704, 2704, 474, 8, true, true);
  const TilePick kr = pick_tiles(kTilesKRDword, 900, 7569, 900, 900, 7569, 57, 8, true, true);
  CHECK(kc1.side == 0 && kc1.bm == 64 && kc1.bn == 128);
  CHECK(kc2.side == 0 && kc2.bm == 64 && kc2.bn == 128);
  CHECK(kc3.side == 0);
  CHECK(kr.side > 0);
  // a float32 build of one 128 x 256 tile over 5625: 24 us on the register-direct kernel, 320
  CHECK(pick_tiles(kTilesKR, 49, 49, 5625, 49, 49, 11, 4, false, false).side > 0);
}

// Routes whose times lie apart (direct against folded or stacked, measured).
static void measured_routes() {
  const struct { int o, v, P, precision; unsigned flags; int folded; } sizes[] = {
      {40, 360, 1200, 0, 0, 1}, {20, 72, 276, 0, 0, 1}, {9, 71, 263, 0, 0, 1},  // 1.84, 1.82, 1.3 x
      {46, 64, 20, 0, 0, 1}, {46, 72, 30, 0, CC_LADDER_PAIR_SYMMETRIC, 1},      // 1.15, 1.4 x
      {9, 71, 60, 0, 0, 0}, {8, 64, 200, 0, 0, 0}, {60, 64, 372, 0, 0, 0},      // 0.93, 0.95, 0.8 x
      {12, 100, 300, 0, CC_LADDER_PAIR_SYMMETRIC, 0},                           // 0.83 x
      {40, 360, 1200, 3, 0, 1}, {30, 65, 285, 3, 0, 1},                         // 1.18, 1.43 x
      {60, 64, 372, 3, 0, 0}, {40, 96, 24, 3, 0, 0}};                           // 0.74, 0.95 x
  for (const auto& x : sizes) {
    const int o = x.o, v = x.v, P = x.P;
    cc_ladder_opts opts{};
    opts.flags = x.flags;
    Plan p;
    CHECK(make_plan(o, v, P, x.precision, 0, size_t(128) << 30, &opts, &p) == CC_LADDER_OK);
    CHECK(route(p) == x.folded);
  }
}

int main() {
  std::mt19937_64 rng(4321);
  measured_routes();
  measured_picks();
  forward_routes(rng, CC_LADDER_FP64, 1500);
  forward_routes(rng, CC_LADDER_SPLIT_INT8, 1000);
  if (g_fail) {
    std::fprintf(stderr, "route_check: %d failures\n", g_fail);
    return 1;
  }
  std::printf("route_check OK\n");
  return 0;
}
