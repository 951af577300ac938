// Host-only checker of the scratch layouts that lie inside another plan's bytes (folded
// forward and adjoint, stacked split-int8 forward) and of the planner's kernel choices,
// built by the CPU test suite with g++ under AddressSanitizer and
// UndefinedBehaviorSanitizer.  Buffers that live in the same stage must lie inside the plan
// and apart, partial sums must fit the buffer they reuse, and every pick must name a tile
// that the launcher has a kernel for.  Prints "layout_check OK" and returns 0 when every
// check holds.
#include <cstdio>
#include <random>
#include <vector>

#include "plan.h"
#include "split.hpp"

using namespace ccl;

static int g_fail = 0;
#define CHECK(cond)                                                                     \
  do {                                                                                  \
    if (!(cond)) {                                                                      \
      if (++g_fail < 20) std::fprintf(stderr, "FAILED line %d: %s\n", __LINE__, #cond); \
    }                                                                                   \
  } while (0)

struct Range {
  size_t off, bytes;
};

// Inside [0, total), on 256-byte boundaries, no two overlapping.
static bool apart(const std::vector<Range>& r, size_t total) {
  for (size_t i = 0; i < r.size(); ++i) {
    if (r[i].off % 256 || r[i].off + r[i].bytes > total) return false;
    for (size_t j = 0; j < i; ++j)
      if (r[i].bytes && r[j].bytes && r[i].off < r[j].off + r[j].bytes &&
          r[j].off < r[i].off + r[i].bytes)
        return false;
  }
  return true;
}

// The most pairs a <= b and a < b of one of nb blocks, and its most virtuals.
static void widest(int v, int nb, size_t* np, size_t* nm, size_t* na) {
  *np = *nm = *na = 0;
  for (int k = 0; k < nb; ++k) {
    const int a0 = pair_block_start(v, nb, k), a1 = pair_block_start(v, nb, k + 1);
    const size_t p = pair_prefix(a1, v) - pair_prefix(a0, v), n = a1 - a0;
    *np = p > *np ? p : *np;
    *nm = p - n > *nm ? p - n : *nm;
    *na = n > *na ? n : *na;
  }
}

static int g_fold = 0, g_adjoint = 0, g_stacked = 0, g_split = 0;

static void check_fold(const Plan& p) {
  FoldPlan f;
  if (!plan_fold(p, &f)) return;
  ++g_fold;
  const size_t v2 = (size_t)p.v * p.v;
  size_t np, nm, na;
  widest(p.v, f.nb, &np, &nm, &na);
  CHECK(f.bytes <= p.bytes);
  CHECK(f.ldp % 2 == 0 && f.ldm % 2 == 0 && f.ldp >= (long long)(v2 + p.v) / 2);
  CHECK(apart({{f.off_Tp, f.rows_p * f.ldp * 8}, {f.off_Tm, f.rows_m * f.ldm * 8}, {f.off_V, np * v2 * 8},
               {f.off_Vp, np * f.ldp * 8}, {f.off_Vm, nm * f.ldm * 8},
               {f.off_tiles, ((na * p.v + 127) / 128 + 1) * 4}}, p.bytes));
  const long long kp = (v2 + p.v) / 2, km = kp - p.v;
  const PairPick pick = pick_pair_products({f.rows_p, kp, f.rows_m, km},
                                           {f.rows_p, (long long)np, f.rows_m, (long long)nm}, kp, 8, 1,
                                           v2 / (f.rows_p + f.rows_m));
  CHECK(pick.splits * (f.rows_p * np + f.rows_m * nm) <= np * v2);
  g_split += pick.splits > 1;
}

static void check_adjoint(const Plan& p) {
  FoldAdjoint a;
  if (!plan_fold_adjoint(p, &a)) return;
  ++g_adjoint;
  const FoldPlan& f = a.f;
  const size_t v2 = (size_t)p.v * p.v, kp = (v2 + p.v) / 2, km = kp - p.v;
  std::vector<Range> rows = {{f.off_Tp, f.rows_p * f.ldp * 8}, {f.off_Tm, f.rows_m * f.ldm * 8},
                             {a.off_Mp, f.rows_p * f.ldp * 8}, {a.off_Mm, f.rows_m * f.ldm * 8}};
  std::vector<Range> dt = rows, dl = rows;
  if (p.gsym) {
    CHECK(p.ldg == f.ldp);
    dt.push_back({a.off_Lp, p.P * f.ldp * 8ul});
    dt.push_back({a.off_G, f.ldp * f.ldp * 8ul});
  }
  dt.push_back({f.off_V, kp * v2 * 8});
  dt.push_back({f.off_Vp, kp * f.ldp * 8});
  dt.push_back({f.off_Vm, km * f.ldm * 8});
  const size_t tile_rows = p.gsym ? f.ldp : v2;
  dt.push_back({f.off_tiles, ((tile_rows + 127) / 128 + 1) * 4});
  dl.push_back({a.off_Wp, kp * f.ldp * 8});
  dl.push_back({a.off_Wm, km * f.ldm * 8});
  dl.push_back({a.off_S, v2 * a.lds * 8});
  if (a.copy_L) dl.push_back({a.off_L, p.P * a.lds * 8ul});
  CHECK(f.nb == 1 && a.lds >= (long long)v2 && a.bytes <= p.bytes);
  CHECK(!a.copy_L || a.lds % 2 == 0);
  CHECK(apart(dt, p.bytes) && apart(dl, p.bytes));
}

static void check_stacked(const Plan& p) {
  StackedPlan q;
  if (!plan_stacked_i8(p, &q)) return;
  ++g_stacked;
  const size_t v2 = (size_t)p.v * p.v, o2 = (size_t)p.o * p.o, s = p.slices;
  size_t np, nm, na;
  widest(p.v, q.nb, &np, &nm, &na);
  const SliceDims dL = slice_dims(v2, p.P), dt = slice_dims(2 * o2, v2), dV = slice_dims(np, v2);
  auto digits = [&](const SliceDims& d) { return s * d.rows_pad * d.k_pad; };
  auto exps = [](const SliceDims& d) { return (size_t)d.rows_pad * i8_chunks(d.k_pad) * 4; };
  CHECK(q.npk == (long long)np);
  CHECK(apart({{q.off_L, digits(dL)}, {q.off_Lexp, exps(dL)}, {q.off_t, digits(dt)}, {q.off_texp, exps(dt)},
               {q.off_V, (np > o2 ? np : o2) * v2 * 8}, {q.off_Vs, digits(dV)}, {q.off_Vexp, exps(dV)},
               {q.off_tiles, ((na * p.v + 127) / 128 + 1) * 4}}, p.bytes));
}

static void layouts(std::mt19937_64& rng) {
  const unsigned P = CC_LADDER_PAIR_SYMMETRIC, X = CC_LADDER_EXCHANGE, S = CC_LADDER_SYMMETRIC_VECTORS,
                 C = CC_LADDER_CHECK_SYMMETRY;
  const unsigned sets[] = {0, P, X, P | X, P | S, P | S | X, P | C, P | S | C};
  for (int it = 0; it < 6000; ++it) {
    const int o = 1 + rng() % 60, v = 1 + rng() % 260, np = 1 + rng() % 2000;
    const int precision = it % 3 == 2 ? CC_LADDER_SPLIT_INT8 : CC_LADDER_FP64, backward = it % 3 == 1;
    cc_ladder_opts opts{};
    opts.flags = sets[rng() % 8];
    opts.a_block = rng() % 3 ? 0 : 1 + rng() % v;
    if (precision == CC_LADDER_SPLIT_INT8) opts.split_slices = rng() % 2 ? 0 : 4;
    const size_t budget = rng() % 2 ? 0 : size_t(1) << (18 + rng() % 18);
    Plan p;
    if (make_plan(o, v, np, precision, backward, budget, &opts, &p)) continue;
    if (backward)
      check_adjoint(p);
    else if (precision == CC_LADDER_FP64)
      check_fold(p);
    else
      check_stacked(p);
  }
  CHECK(g_fold > 200 && g_adjoint > 500 && g_stacked > 100 && g_split > 50);
}

// The launcher's tiles: 160 x 256 of the K-contiguous kernel in float64, 128 x 256 with a
// 64-row rest, 64 x 128 and 64 x 64 (with dword loads only in float32), 128 x 128 of the
// register-staged kernel; at most 16 waves of the register-direct kernel.
static void picks(std::mt19937_64& rng) {
  const TileClass all[] = {kTilesKC, kTilesKR, kTilesKCDword, kTilesKRDword, kTilesStaged};
  for (int it = 0; it < 200000; ++it) {
    auto size = [&](int bits) { return 1 + (long long)(rng() % (1ull << (1 + rng() % bits))); };
    const long long M = size(14), N = size(18), K = size(18);
    const int es = rng() % 2 ? 8 : 4, bk = 128 / es;
    const TileClass cls = all[rng() % 5];
    const bool tall = es == 8, split = rng() % 2;
    const long long nk = (K + bk - 1) / bk, units = es == 4 ? (nk + 15) / 16 : nk;
    const TilePick p = pick_tiles(cls, M, N, K, M, N, units, es, tall, split);
    if (p.side) {
      CHECK((p.side == 1 || p.side == 2) && p.wk >= 1 && p.side * p.side * p.wk <= 16);
      CHECK((p.wk & (p.wk - 1)) == 0);
    } else if (cls == kTilesKC) {
      CHECK((p.bm == 160 && p.bn == 256 && es == 8) || (p.bm == 128 && p.bn == 256) ||
            (p.bm == 64 && (p.bn == 128 || p.bn == 64)));
      CHECK(p.main_rows == M || (split && p.bm == 128 && p.main_rows > 0 && M - p.main_rows <= 64));
    } else if (cls == kTilesKCDword) {
      CHECK((p.bm == 128 && p.bn == 256) || (p.bm == 64 && p.bn == 128) ||
            (es == 4 && p.bm == 64 && p.bn == 64) || (es == 8 && p.bm == 128 && p.bn == 128));
      CHECK(p.main_rows == M);
    } else if (cls == kTilesStaged) {
      CHECK(p.bm == 128 && p.bn == 128);
    } else {
      CHECK((p.bm == 128 && p.bn == 256) ||
            (es == 8 && p.bm == 64 && (p.bn == 128 || (p.bn == 64 && cls == kTilesKR))) ||
            (es == 8 && cls == kTilesKRDword && p.bm == 128 && p.bn == 128));
    }
    const int splits = 1 + rng() % 16;
    const bool direct = rng() % 2;
    const TilePick q = pick_part_tiles(M, N, K, splits, units, es, direct);
    CHECK(q.side ? q.side * q.side * q.wk <= 16 && q.bm == 32 * q.side && q.bn == q.bm
                 : direct && ((q.bm == 128 && q.bn == 256) || (q.bm == 64 && (q.bn == 128 || q.bn == 64))));
    const PairExtents e{M, N, M - 1, N - 1};
    const PairPick r = pick_pair_products(e, e, K, es, es == 4 ? 16 : 1, rng() % 20);
    CHECK(r.splits >= 0 && r.splits <= kPairSplits);
    auto tile = [&](int bm, int bn) {
      return (bn == 256 && (bm == 128 || (bm == 160 && es == 8))) || (bm == 64 && (bn == 128 || bn == 64));
    };
    CHECK(!r.splits || (tile(r.bm, r.bn) && tile(r.bm2, r.bn2)));
    CHECK(r.apart || (r.bm == r.bm2 && r.bn == r.bn2));
  }
}

int main() {
  std::mt19937_64 rng(99);
  layouts(rng);
  picks(rng);
  if (g_fail) {
    std::fprintf(stderr, "layout_check: %d failures\n", g_fail);
    return 1;
  }
  std::printf("layout_check OK\n");
  return 0;
}
