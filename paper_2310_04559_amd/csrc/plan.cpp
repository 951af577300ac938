// Host-only planner: buffer layout and block-size selection.
#include "plan.h"

#include "split.hpp"

#include <cmath>
#include <cstdint>

namespace ccl {

namespace {

constexpr size_t kAlign = 256;

size_t round_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// Appends a buffer of `bytes` at the end of the layout and returns its offset.
size_t take(size_t* cursor, size_t bytes) {
  size_t off = *cursor;
  *cursor = round_up(off + bytes);
  return off;
}

}  // namespace

int check_dims(int o, int v, int P) {
  if (o <= 0 || v <= 0 || P <= 0) return CC_LADDER_EINVAL;
  // o^2 and v^2 are GEMM extents held in 32-bit ints.
  if (o > 46340 || v > 46340 || P > (1 << 24)) return CC_LADDER_EINVAL;
  // element counts of the arrays (o^2 v^2, P v^2, P o v) stay far inside size_t
  // byte counts: at most 2^52 elements each
  const unsigned long long o2 = static_cast<unsigned long long>(o) * o;
  const unsigned long long v2 = static_cast<unsigned long long>(v) * v;
  constexpr unsigned long long kMaxElems = 1ull << 52;
  if (o2 * v2 > kMaxElems || static_cast<unsigned long long>(P) * v2 > kMaxElems ||
      static_cast<unsigned long long>(P) * o * v > kMaxElems)
    return CC_LADDER_EINVAL;
  return CC_LADDER_OK;
}

int check_precision_opts(int precision, const cc_ladder_opts* opts) {
  if (precision != CC_LADDER_FP64 && precision != CC_LADDER_FP32 &&
      precision != CC_LADDER_SPLIT_BF16 && precision != CC_LADDER_SPLIT_INT8)
    return CC_LADDER_EINVAL;
  if (!opts) return CC_LADDER_OK;
  if (opts->a_block < 0 || opts->split_depth < 0 || opts->split_depth > 2) return CC_LADDER_EINVAL;
  if ((opts->flags & ~(CC_LADDER_PAIR_SYMMETRIC | CC_LADDER_EXCHANGE | CC_LADDER_CHECK_SYMMETRY |
                       CC_LADDER_PLUS_MINUS | CC_LADDER_SYMMETRIC_VECTORS)) != 0 ||
      opts->reserved != 0)
    return CC_LADDER_EINVAL;
  // the symmetric/antisymmetric combinations and the whole pair-pair integral
  // serve the pair-symmetric paths
  if ((opts->flags & (CC_LADDER_PLUS_MINUS | CC_LADDER_SYMMETRIC_VECTORS)) &&
      !(opts->flags & CC_LADDER_PAIR_SYMMETRIC))
    return CC_LADDER_EINVAL;
  if (opts->split_slices != 0) {
    const int lo = precision == CC_LADDER_SPLIT_INT8 ? 4 : 2;
    const int hi = precision == CC_LADDER_SPLIT_INT8 ? 5 : 4;
    if (opts->split_slices < lo || opts->split_slices > hi) return CC_LADDER_EINVAL;
  }
  if (opts->k_chunk < 0 || opts->k_chunk % 64 != 0) return CC_LADDER_EINVAL;
  if (opts->workspace && (reinterpret_cast<uintptr_t>(opts->workspace) % kAlign) != 0)
    return CC_LADDER_EINVAL;
  return CC_LADDER_OK;
}

bool overlaps(const void* a, size_t abytes, const void* b, size_t bbytes) {
  if (!abytes || !bbytes) return false;
  const uintptr_t x = reinterpret_cast<uintptr_t>(a), y = reinterpret_cast<uintptr_t>(b);
  return x < y + bbytes && y < x + abytes;
}

int check_residual_args(int o, int v, int P, const double* L, const double* t, const double* R,
                        int precision, const cc_ladder_opts* opts, Operand ops[3]) {
  int rc = check_dims(o, v, P);
  if (rc) return rc;
  rc = check_precision_opts(precision, opts);
  if (rc) return rc;
  if (!L || !t || !R) return CC_LADDER_EINVAL;
  const size_t nt = static_cast<size_t>(o) * o * v * v * sizeof(double);
  const size_t nL = static_cast<size_t>(P) * v * v * sizeof(double);
  ops[0] = {L, nL};
  ops[1] = {t, nt};
  ops[2] = {R, nt};
  if (overlaps(R, nt, t, nt) || overlaps(R, nt, L, nL)) return CC_LADDER_EINVAL;
  return CC_LADDER_OK;
}

int check_backward_args(int o, int v, int P, const double* L, const double* t, const double* lam,
                        const double* dL, const double* dt, int precision,
                        const cc_ladder_opts* opts, Operand ops[5]) {
  int rc = check_dims(o, v, P);
  if (rc) return rc;
  rc = check_precision_opts(precision, opts);
  if (rc) return rc;
  if (!L || !t || !lam || !dL || !dt) return CC_LADDER_EINVAL;
  const size_t nt = static_cast<size_t>(o) * o * v * v * sizeof(double);
  const size_t nL = static_cast<size_t>(P) * v * v * sizeof(double);
  ops[0] = {L, nL};
  ops[1] = {t, nt};
  ops[2] = {lam, nt};
  ops[3] = {dL, nL};
  ops[4] = {dt, nt};
  if (overlaps(dt, nt, t, nt) || overlaps(dt, nt, lam, nt) || overlaps(dt, nt, L, nL) ||
      overlaps(dL, nL, L, nL) || overlaps(dL, nL, t, nt) || overlaps(dL, nL, lam, nt) ||
      overlaps(dL, nL, dt, nt))
    return CC_LADDER_EINVAL;
  return CC_LADDER_OK;
}

int check_workspace(const cc_ladder_opts* opts, size_t plan_bytes, const Operand* ops, int n) {
  if (!opts || !opts->workspace) return CC_LADDER_OK;
  for (int i = 0; i < n; ++i)
    if (overlaps(opts->workspace, plan_bytes, ops[i].p, ops[i].bytes)) return CC_LADDER_EINVAL;
  return CC_LADDER_OK;
}

int pair_block_start(int v, int nb, int k) {
  if (k <= 0) return 0;
  if (k >= nb) return v;
  const long long target = (long long)k * ((long long)v * (v + 1) / 2);
  // smallest a with pair_prefix(a) * nb >= target: the root of the quadratic, then exactly
  const double b = 2.0 * v + 1.0, d = b * b - 8.0 * static_cast<double>(target) / nb;
  int a = static_cast<int>((b - std::sqrt(d > 0.0 ? d : 0.0)) * 0.5);
  a = a < 0 ? 0 : (a > v ? v : a);
  while (a < v && pair_prefix(a, v) * nb < target) ++a;
  while (a > 0 && pair_prefix(a - 1, v) * nb >= target) --a;
  return a;
}

void block_range(const Plan& pl, int blk, int* a0, int* na) {
  if (pl.balanced) {
    *a0 = pair_block_start(pl.v, pl.nblocks, blk);
    *na = pair_block_start(pl.v, pl.nblocks, blk + 1) - *a0;
    return;
  }
  *a0 = blk * pl.n_a;
  *na = (pl.v - *a0) < pl.n_a ? (pl.v - *a0) : pl.n_a;
}

namespace {
RouteRule route_rule(int o, int v, int P, int precision, int backward, int slices, unsigned flags,
                     bool least);
}  // namespace

int layout_plan(int o, int v, int P, int precision, int backward, int n_a,
                int slices, int depth, int k_chunk, unsigned flags, Plan* plan, int nb,
                bool padded, const RouteRule* rule) {
  const int pairsym = (flags & CC_LADDER_PAIR_SYMMETRIC) ? 1 : 0;
  Plan p;
  // packed forward in pair-balanced blocks: the widest block sizes the tile
  // table, the block with the most pairs (a <= b, and a < b) the buffers
  size_t npk_max = 0, nstrict_max = 0;
  if (nb > 0 && pairsym && !backward) {
    if (nb > v) return CC_LADDER_EINVAL;
    p.balanced = 1;
    n_a = 0;
    for (int k = 0; k < nb; ++k) {
      const int a0 = pair_block_start(v, nb, k), a1 = pair_block_start(v, nb, k + 1);
      const size_t np = static_cast<size_t>(pair_prefix(a1, v) - pair_prefix(a0, v));
      n_a = (a1 - a0) > n_a ? (a1 - a0) : n_a;
      npk_max = np > npk_max ? np : npk_max;
      const size_t ns = np - static_cast<size_t>(a1 - a0);
      nstrict_max = ns > nstrict_max ? ns : nstrict_max;
    }
  }
  if (n_a < 1 || n_a > v) return CC_LADDER_EINVAL;
  p.o = o; p.v = v; p.P = P;
  p.precision = precision;
  p.backward = backward ? 1 : 0;
  p.n_a = n_a;
  p.nblocks = p.balanced ? nb : (v + n_a - 1) / n_a;
  const size_t v2 = static_cast<size_t>(v) * v;
  const size_t o2 = static_cast<size_t>(o) * o;
  p.pairsym = (pairsym && !backward) ? 1 : 0;
  p.pairsym_adj = (pairsym && backward) ? 1 : 0;
  // entries of one integral block: n_a*v rows (a,b); packed rows a <= b when the
  // amplitudes are pair-symmetric (with equal virtual counts the first block
  // holds the most).  The adjoint's W block always has n_a*v rows.
  const size_t npk = p.balanced ? npk_max : static_cast<size_t>(pair_prefix(n_a, v));
  p.npk = p.pairsym ? static_cast<long long>(npk) : 0;
  const size_t npk_ld = (npk + 3) / 4 * 4;  // row stride of the adjoint's gathered lam
  const size_t rows = (p.pairsym || p.pairsym_adj) ? npk : static_cast<size_t>(n_a) * v;
  const size_t ldk = padded && precision == CC_LADDER_FP32 && !pairsym ? (v2 + 3) / 4 * 4 : v2;
  p.ldk = static_cast<long long>(ldk);
  const size_t blk = rows * ldk;
  const size_t blk_w = static_cast<size_t>(n_a) * v * ldk;
  size_t cur = 0;
  p.exchange = (flags & CC_LADDER_EXCHANGE) ? 1 : 0;
  p.pm = (p.pairsym && (flags & CC_LADDER_PLUS_MINUS)) ? 1 : 0;
  // symmetric vectors: the whole pair-pair integral G [ldg][ldg] and the packed
  // vectors [P][ldg] (side v(v+1)/2 rounded to 4, pads zero) replace the packed
  // build in the FP64 and FP32 pair-symmetric paths and in the split
  // pair-symmetric forwards (there G is float64, built from digits of the packed
  // vectors)
  const size_t es_g = precision == CC_LADDER_FP32 ? sizeof(float) : sizeof(double);
  p.gsym = ((flags & CC_LADDER_SYMMETRIC_VECTORS) &&
            (((p.pairsym || p.pairsym_adj) &&
              (precision == CC_LADDER_FP64 || precision == CC_LADDER_FP32)) ||
             (p.pairsym && !p.backward &&
              (precision == CC_LADDER_SPLIT_INT8 || precision == CC_LADDER_SPLIT_BF16)))) ? 1 : 0;
  if (p.gsym) p.ldg = static_cast<long long>((static_cast<size_t>(v) * (v + 1) / 2 + 3) / 4 * 4);
  if (p.exchange) {
    // the float32 form swaps while converting into its own operand copy; the
    // combinations t+- of swapped amplitudes are t+ and -t-, made without a copy
    if (precision != CC_LADDER_FP32 && !p.pm) p.off_tx = take(&cur, o2 * v2 * sizeof(double));
    if (p.backward) p.off_dtx = take(&cur, o2 * v2 * sizeof(double));
  }
  if (p.pm) {
    if (precision == CC_LADDER_SPLIT_BF16 || precision == CC_LADDER_SPLIT_INT8)
      return CC_LADDER_EUNSUPPORTED;
    // operand rows over the pairs c <= d (t+, V+) and c < d (t-, V-), strides
    // rounded to 16-byte multiples of either element size
    const size_t es = precision == CC_LADDER_FP64 ? sizeof(double) : sizeof(float);
    const size_t kp = static_cast<size_t>(v) * (v + 1) / 2, km = static_cast<size_t>(v) * (v - 1) / 2;
    p.ldp = static_cast<long long>((kp + 3) / 4 * 4);
    p.ldm = static_cast<long long>((km + 3) / 4 * 4);
    const size_t mp = static_cast<size_t>(o) * (o + 1) / 2, mm = static_cast<size_t>(o) * (o - 1) / 2;
    // packed rows of the largest block: a <= b, and a < b
    const size_t np = npk, nm = p.balanced ? nstrict_max : npk - static_cast<size_t>(n_a);
    p.off_Tp = take(&cur, mp * p.ldp * es);
    p.off_Tm = take(&cur, mm * p.ldm * es);
    p.off_Vp = take(&cur, np * p.ldp * es);
    p.off_Vm = take(&cur, nm * p.ldm * es);
    if (precision == CC_LADDER_FP32) p.k_chunk = k_chunk ? k_chunk : 512;
    if (p.gsym) {
      // no packed block: V+- are gathered from G
      p.off_Lp = take(&cur, static_cast<size_t>(P) * p.ldg * es);
      p.off_G = take(&cur, static_cast<size_t>(p.ldg) * p.ldg * es);
    } else {
      if (precision == CC_LADDER_FP32)
        p.off_L = take(&cur, static_cast<size_t>(P) * v2 * sizeof(float));
      p.off_V = take(&cur, blk * es);
    }
  } else {
  switch (precision) {
    case CC_LADDER_FP64:
      p.off_V = take(&cur, blk * sizeof(double));
      if (p.backward) p.off_W = take(&cur, blk_w * sizeof(double));
      if (p.pairsym_adj) p.off_lamP = take(&cur, o2 * npk_ld * sizeof(double));
      break;
    case CC_LADDER_FP32:
      p.k_chunk = k_chunk ? k_chunk : 512;
      // the forward over G needs no float32 copy of L (the adjoint's dL does)
      if (!p.gsym || p.backward) p.off_L = take(&cur, static_cast<size_t>(P) * ldk * sizeof(float));
      p.off_t = take(&cur, o2 * ldk * sizeof(float));
      if (p.backward) p.off_lam = take(&cur, o2 * ldk * sizeof(float));
      p.off_V = take(&cur, blk * sizeof(float));
      if (p.backward) p.off_W = take(&cur, blk_w * sizeof(float));
      if (p.pairsym_adj) p.off_lamP = take(&cur, o2 * npk_ld * sizeof(float));
      break;
    case CC_LADDER_SPLIT_BF16: {
      if (p.backward) return CC_LADDER_EUNSUPPORTED;
      p.slices = slices ? slices : 4;
      // automatic depth: the 4-slice form keeps the triangle's next anti-diagonal
      p.split_depth = depth ? depth : (p.slices == 4 ? 2 : 1);
      const size_t s = static_cast<size_t>(p.slices);
      // digits of L's columns (a,c), or of the packed vectors' columns {a,c}
      const SliceDims dL = slice_dims(p.gsym ? p.ldg : static_cast<long long>(v2), P);
      const SliceDims dt = slice_dims(static_cast<long long>(o2), static_cast<int>(v2));
      const SliceDims dV = slice_dims(static_cast<long long>(rows), static_cast<int>(v2));
      p.off_L = take(&cur, s * dL.rows_pad * dL.k_pad * 2);
      p.off_Lexp = take(&cur, static_cast<size_t>(dL.rows_pad) * sizeof(int));
      p.off_t = take(&cur, s * dt.rows_pad * dt.k_pad * 2);
      p.off_texp = take(&cur, static_cast<size_t>(dt.rows_pad) * exp_chunks(dt.k_pad, p.slices) * sizeof(int));
      p.off_V = take(&cur, blk * sizeof(double));
      p.off_Vs = take(&cur, s * dV.rows_pad * dV.k_pad * 2);
      p.off_Vexp = take(&cur, static_cast<size_t>(dV.rows_pad) * exp_chunks(dV.k_pad, p.slices) * sizeof(int));
      break;
    }
    case CC_LADDER_SPLIT_INT8: {
      if (p.backward) return CC_LADDER_EUNSUPPORTED;
      p.slices = slices ? slices : 5;
      p.split_depth = depth ? depth : 1;
      // the kernels hold S + depth - 1 int32 sums per output: 5 at most
      if (p.slices + p.split_depth - 1 > 5) return CC_LADDER_EUNSUPPORTED;
      const size_t s = static_cast<size_t>(p.slices);  // one byte per digit
      // digits of the vectors' columns (a,c), or with symmetric vectors of the
      // packed vectors' columns {a,c}, a <= c
      const SliceDims dL = slice_dims(p.gsym ? p.ldg : static_cast<long long>(v2), P);
      const SliceDims dt = slice_dims(static_cast<long long>(o2), static_cast<int>(v2));
      const SliceDims dV = slice_dims(static_cast<long long>(rows), static_cast<int>(v2));
      p.off_L = take(&cur, s * dL.rows_pad * dL.k_pad);
      p.off_Lexp = take(&cur, static_cast<size_t>(dL.rows_pad) * i8_chunks(dL.k_pad) * sizeof(int));
      p.off_t = take(&cur, s * dt.rows_pad * dt.k_pad);
      p.off_texp = take(&cur, static_cast<size_t>(dt.rows_pad) * i8_chunks(dt.k_pad) * sizeof(int));
      p.off_V = take(&cur, blk * sizeof(double));
      p.off_Vs = take(&cur, s * dV.rows_pad * dV.k_pad);
      p.off_Vexp = take(&cur, static_cast<size_t>(dV.rows_pad) * i8_chunks(dV.k_pad) * sizeof(int));
      break;
    }
    default:
      return CC_LADDER_EINVAL;
  }
  }
  if (p.pairsym_adj) {
    // the adjoint's dt accumulates B[(ij)][(cd)] over packed rows; dt += B + mirror(B)
    p.off_B = take(&cur, o2 * v2 * sizeof(double));
  }
  if (p.gsym && !p.pm) {
    p.off_Lp = take(&cur, static_cast<size_t>(P) * p.ldg * es_g);
    p.off_G = take(&cur, static_cast<size_t>(p.ldg) * p.ldg * es_g);
  }
  if ((p.pairsym || p.pairsym_adj) && (flags & CC_LADDER_CHECK_SYMMETRY)) {
    // two maxima of the pair-symmetry check (bit patterns of non-negative doubles)
    p.check_sym = 1;
    p.off_check = take(&cur, 2 * sizeof(unsigned long long));
  }
  if (p.pairsym || p.pairsym_adj) {
    // tile-row offsets of the packed build's compact grid (128-row tiles; 64 rows
    // in the split form), or of the upper-triangle grid of the pair-pair integral
    const size_t bm = precision == CC_LADDER_SPLIT_BF16 ? 64 : 128;
    const size_t rows_m = p.gsym ? static_cast<size_t>(p.ldg) : static_cast<size_t>(n_a) * v;
    const size_t tiles_m = (rows_m + bm - 1) / bm;
    p.off_tiles = take(&cur, (tiles_m + 1) * sizeof(int));
  }
  if (!p.gsym) {
    const RouteRule by_size =
        rule ? *rule : route_rule(o, v, P, precision, backward, p.slices, flags, true);
    if (by_size.blocks) {
      (precision == CC_LADDER_FP64 ? p.fold : p.stacked) = by_size.blocks;
      const size_t need = by_size.bytes + (p.check_sym ? kAlign : 0);
      cur = need > cur ? need : cur;
    }
  }
  p.bytes = cur;
  *plan = p;
  return CC_LADDER_OK;
}

namespace {

// Largest block of first indices (1..n_max) whose layout fits `budget`
// (0 = unlimited), then equalised: the same block count with the smallest
// block that achieves it.  `fixed` > 0 takes that block size as given.
template <class Layout>
int search_block(int n_max, size_t budget, int fixed, Layout layout, Plan* plan) {
  int rc;
  if (fixed > 0) {
    rc = layout(fixed < n_max ? fixed : n_max, plan);
    if (rc) return rc;
    return (budget && plan->bytes > budget) ? CC_LADDER_ENOMEM : CC_LADDER_OK;
  }
  // the footprint grows monotonically with the block size
  Plan best;
  rc = layout(n_max, plan);
  if (rc || !budget || plan->bytes <= budget) return rc;
  rc = layout(1, &best);
  if (rc) return rc;
  if (budget && best.bytes > budget) return CC_LADDER_ENOMEM;
  int lo = 1, hi = n_max;
  while (lo < hi) {
    const int mid = lo + (hi - lo + 1) / 2;
    Plan trial;
    rc = layout(mid, &trial);
    if (rc) return rc;
    if (!budget || trial.bytes <= budget) {
      lo = mid;
      best = trial;
    } else {
      hi = mid - 1;
    }
  }
  const int nb = (n_max + best.n_a - 1) / best.n_a;
  const int n_eq = (n_max + nb - 1) / nb;
  if (n_eq != best.n_a) {
    rc = layout(n_eq, &best);
    if (rc) return rc;
  }
  *plan = best;
  return CC_LADDER_OK;
}

}  // namespace

namespace {

int make_plan_flags(int o, int v, int P, int precision, int backward, size_t budget,
                    const cc_ladder_opts* opts, unsigned flags, const RouteRule& rule, Plan* plan) {
  const int slices = opts ? opts->split_slices : 0;
  const int depth = opts ? opts->split_depth : 0;
  const int k_chunk = opts ? opts->k_chunk : 0;
  const int fixed = opts ? opts->a_block : 0;
  if ((flags & CC_LADDER_PAIR_SYMMETRIC) && !backward && fixed == 0) {
    // packed forward: blocks of about equal pair counts (equal virtual counts
    // would leave the last blocks, whose virtuals pair with few others, a
    // small fraction of the first one's work); the fewest blocks that fit
    auto fits = [&](int nb, Plan* p) {
      const int rc = layout_plan(o, v, P, precision, backward, 0, slices, depth, k_chunk, flags, p,
                                 nb, false, &rule);
      if (rc) return rc;
      return (budget && p->bytes > budget) ? CC_LADDER_ENOMEM : CC_LADDER_OK;
    };
    int rc = fits(1, plan);
    if (rc != CC_LADDER_ENOMEM) return rc;
    Plan best;
    rc = fits(v, &best);
    if (rc) return rc;
    int lo = 1, hi = v;
    while (lo < hi) {
      const int mid = lo + (hi - lo) / 2;
      Plan trial;
      rc = fits(mid, &trial);
      if (rc == CC_LADDER_OK) {
        hi = mid;
        best = trial;
      } else if (rc == CC_LADDER_ENOMEM) {
        lo = mid + 1;
      } else {
        return rc;
      }
    }
    if (best.nblocks != lo) {
      rc = fits(lo, &best);
      if (rc) return rc;
    }
    *plan = best;
    return CC_LADDER_OK;
  }
  const int rc = search_block(v, budget, fixed, [&](int n_a, Plan* p) {
    return layout_plan(o, v, P, precision, backward, n_a, slices, depth, k_chunk, flags, p, 0,
                       false, &rule);
  }, plan);
  if (rc || precision != CC_LADDER_FP32 || v % 2 == 0) return rc;
  // odd v: padded rows where the same blocks still fit (a plan sized without the
  // pads keeps its blocks and its rows)
  Plan pad;
  if (layout_plan(o, v, P, precision, backward, plan->n_a, slices, depth, k_chunk, flags, &pad, 0,
                  true) == CC_LADDER_OK &&
      (!budget || pad.bytes <= budget))
    *plan = pad;
  return rc;
}

}  // namespace

int make_plan(int o, int v, int P, int precision, int backward, size_t budget,
              const cc_ladder_opts* opts, Plan* plan) {
  int rc = check_dims(o, v, P);
  if (rc) return rc;
  rc = check_precision_opts(precision, opts);
  if (rc) return rc;
  const unsigned flags = opts ? opts->flags : 0u;
  const int slices = opts && opts->split_slices ? opts->split_slices : 5;  // (of split-int8)
  RouteRule rule = route_rule(o, v, P, precision, backward, slices, flags, false);
  if (rule.blocks) {
    // the least scratch of the route counts only where the whole does not fit
    rc = make_plan_flags(o, v, P, precision, backward, 0, opts, flags, rule, plan);
    const bool whole = plan->nblocks == 1 && (!budget || plan->bytes <= budget);
    if (rc || whole) return rc;
    rule = route_rule(o, v, P, precision, backward, slices, flags, true);
  }
  rc = make_plan_flags(o, v, P, precision, backward, budget, opts, flags, rule, plan);
  // the whole pair-pair integral does not fit: the packed blocks instead
  const unsigned packed = flags & ~CC_LADDER_SYMMETRIC_VECTORS;
  if (rc == CC_LADDER_ENOMEM && packed != flags)
    rc = make_plan_flags(o, v, P, precision, backward, budget, opts, packed, rule, plan);
  // nor do the folded route's fewest buffers: the direct one
  if (rc == CC_LADDER_ENOMEM && rule.blocks)
    rc = make_plan_flags(o, v, P, precision, backward, budget, opts, packed, RouteRule{}, plan);
  return rc;
}

int choose_kc_tiling(long long M, long long N, bool tall, bool split, long long* main_rows) {
  constexpr long long kCUs = 256;  // compute units of one MI355X
  constexpr long long kTN = 256;   // the K-contiguous kernel's tile width
  const long long tn = (N + kTN - 1) / kTN;
  // one workgroup per CU at a time: a launch lasts about (rounds of its grid
  // over the CUs) x (one tile's time, proportional to its height)
  auto span = [&](long long rows, long long bm) {
    const long long tiles = (rows + bm - 1) / bm * tn;
    return (tiles + kCUs - 1) / kCUs * bm;
  };
  const long long rem = M % 128;
  long long best = span(M, 128);
  int choice = 128;
  if (tall && span(M, 160) < best) {
    best = span(M, 160);
    choice = 160;
  }
  if (split && M > 128 && rem > 0 && rem <= 64 && span(M - rem, 128) + span(rem, 64) < best) {
    best = span(M - rem, 128) + span(rem, 64);
    choice = 64;
  }
  *main_rows = choice == 64 ? M - rem : M;
  return choice;
}

int choose_k_splits(long long M, long long N, long long K, int bk) {
  constexpr long long kCUs = 256;           // compute units of one MI355X
  constexpr long long kTM = 128, kTN = 256;  // the K-contiguous kernel's tile
  const long long tiles = ((M + kTM - 1) / kTM) * ((N + kTN - 1) / kTN);
  const long long nk = (K + bk - 1) / bk;
  if (tiles <= 0 || tiles >= kCUs) return 1;
  int best = 1;
  double best_cost = 1.0;  // waves per unit of work without a split
  for (int s = 2; s <= 16; ++s) {
    if (nk / s < 64) break;
    const double cost = static_cast<double>((tiles * s + kCUs - 1) / kCUs) / s;
    if (cost < best_cost * 0.999) {
      best = s;
      best_cost = cost;
    }
  }
  return best;
}

namespace {

// Time of a launch per unit of K, in multiply-adds of one compute unit: rounds of
// the grid over the 256 compute units times the tile, over the share of the matrix
// cores' rate that the tile reaches.  The shares are float64 measurements on
// products that fill whole rounds: 128 x 256 (and 160) 0.88 (o=40 v=360 P=1200
// contraction), 64 x 128 0.82 (225 x 16290 x 16290: 2.05 ms against 2.17 on 64 x 256),
// 64 x 64 0.78 (400 x 16290 x 16290: 3.66 ms).  The smaller tiles win where the larger ones would leave part of a
// round idle: 169 x 4753 x 4753 0.19 ms on 64 x 64 against 1.17 on 128 x 256,
// 800 x 4950 x 4950 0.63 on 64 x 128 against 1.23.
double tile_cost(long long M, long long N, int bm, int bn, double rate) {
  const long long tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
  return static_cast<double>((tiles + 255) / 256) * bm * bn / rate;
}

// Tiles of a launch; of an upper one those with columns n >= their first row m.
long long tiles_run(long long M, long long N, long long bm, long long bn, bool upper) {
  const long long tm = (M + bm - 1) / bm, tn = (N + bn - 1) / bn;
  return upper ? tm * tn - tm * (tm - 1) * bm / (2 * bn) : tm * tn;
}

// The register-staged kernel: float64 workgroups run two to a compute unit and reach
// 0.80 (0.84 over a long K), an odd one alone 0.70 over a long K (1936 x 1936 x 22201, one
// round: 3.6 ms) but 0.50 over a short one, which is filling and stores (2556 x 2556 x 263
// above the diagonal, 210 tiles: 61 us, on the register-direct kernel 54; o=10 v=64 P=230 +-
// forward 224 -> 206 us, adjoint 524 -> 497).
double staged_cost(long long M, long long N, long long K, int es, bool upper) {
  const long long rounds = (tiles_run(M, N, 128, 128, upper) + 255) / 256;
  const long long alone = es == 8 ? rounds % 2 : 0;
  const bool deep = es == 8 && K >= 1024;
  return 128.0 * 128.0 * (static_cast<double>(rounds - alone) / (deep ? 0.84 : 0.80) +
                          static_cast<double>(alone) / (deep ? 0.70 : 0.50));
}

// The register-direct kernel reaches 0.62 of the rate while its operands stay in
// the 256 MB last-level cache (400 x 4950 x 4950: 0.40 ms on 32 x 32, 0.49 on 64 x
// 64 direct-to-LDS tiles) and 0.42 beyond (400 x 16290 x 16290: 6.7 ms against 3.7), or
// where float32 rows lie whole multiples of 16 KB apart, on the same memory channels
// (1681 x 2624 x 4096: 0.62 ms against 0.40 on 64 x 64 tiles).  Float64 rows off 16-byte
// boundaries: K-contiguous and both sides over 1024 0.55, from 128 MB on 0.50 (3249 x 3249 x
// 4489: 2.61 ms, 1.84 on 64 x 128 tiles), with row-contiguous columns 0.70.
enum { kRowsAligned, kRowsOddKC, kRowsOddKR };
double wave_rate(long long M, long long N, long long K, int es, int rows, bool channels) {
  const double bytes = (static_cast<double>(M) + static_cast<double>(N)) * K * es;
  if (bytes > 256e6 || channels) return 0.42;
  if (rows == kRowsOddKC && M > 1024 && N > 1024) return bytes > 128e6 ? 0.50 : 0.55;
  return rows == kRowsOddKR ? 0.70 : 0.62;
}

// A compute unit needs eight waves to cover the latency of their loads.
double wave_cost(long long M, long long N, double rate, int side, int wk, bool upper) {
  const long long t = 32 * side;
  const long long tiles = tiles_run(M, N, t, t, upper);
  const long long rounds = (tiles + 255) / 256;
  const long long waves = rounds * side * side * wk;
  const double busy = waves >= 8 ? 1.0 : static_cast<double>(waves) / 8;
  return static_cast<double>(rounds) * t * t / (rate * busy);
}

// Waves along K: each with at least two pieces, at most eight per compute unit.
int waves_along_k(long long M, long long N, long long units, int side) {
  const long long t = 32 * side;
  const long long rounds = (((M + t - 1) / t) * ((N + t - 1) / t) + 255) / 256;
  int wk = 1;
  while (2 * wk * side * side <= 16 && units >= 4LL * wk && rounds * wk * side * side < 8) wk *= 2;
  return wk;
}

TilePick pick_launch(TileClass cls, long long M, long long N, long long K, long long units, int es,
                     bool tall, bool split, bool upper = false) {
  TilePick p;
  double best = 0.0;
  auto take = [&](int bm, int bn, long long main_rows, double cost) {
    if (p.bm && cost >= best) return;
    best = cost;
    p.bm = bm;
    p.bn = bn;
    p.main_rows = main_rows;
  };
  // Dword loads, float64 (o = 38 to 76, v = 51 to 229, K from 2600 on): X on 128 x 256 tiles
  // 0.88 to 0.92, on 64 x 128 0.84 to 0.87 (4900 x 4900 x 12321: 12.6 ms in 3.05 rounds, 10.0 in
  // 11.7, the register-staged kernel 10.1), the hole-hole ladder 0.86 to 0.89, 0.82 to 0.84 and
  // there 0.81 to 0.94 (3600 x 7569 x 3600: 3.86, 3.54 and 3.30 ms), less over a shorter K
  // (900: 0.71, 0.73; the register-direct kernel 0.70 to 0.78); 64 x 64 tiles were slower
  // than the register-direct kernel (400 x 2016 x 3969 0.314 against 0.309 ms).
  const bool dword = (cls == kTilesKCDword || cls == kTilesKRDword) && es == 8;
  const bool kr = cls == kTilesKRDword, shallow = dword && kr && K < 2048;
  const double big = shallow ? 0.76 : dword && !kr ? 0.90 : 0.88;
  const double mid = shallow ? 0.74 : dword ? (kr ? 0.82 : 0.85) : es == 4 ? 0.77 : 0.82;
  const double small = es == 4 ? 0.70 : 0.78;
  if (cls == kTilesKCDword) {
    take(128, 256, M, tile_cost(M, N, 128, 256, big));
    // (a single round of them 0.66 to 0.78)
    const bool one = dword && ((M + 63) / 64) * ((N + 127) / 128) <= 256;
    take(64, 128, M, tile_cost(M, N, 64, 128, one ? 0.75 : mid));
    if (!dword) take(64, 64, M, tile_cost(M, N, 64, 64, small));
    if (dword) take(128, 128, M, staged_cost(M, N, K, es, false));
  } else if (cls == kTilesKC) {
    long long main_rows = M;
    const int bm = choose_kc_tiling(M, N, tall, split, &main_rows);
    const double cost = bm == 64 ? tile_cost(main_rows, N, 128, 256, 0.88) +
                                       tile_cost(M - main_rows, N, 64, 256, 0.88)
                                 : tile_cost(M, N, bm, 256, 0.88);
    take(bm == 64 ? 128 : bm, 256, main_rows, cost);
    // (float32 has twice the rate for the same bytes: 576 x 41209 x 41209 16.8 ms on 64
    // x 128)
    take(64, 128, M, tile_cost(M, N, 64, 128, mid));
    take(64, 64, M, tile_cost(M, N, 64, 64, small));
  } else if (cls == kTilesKR || cls == kTilesKRDword) {
    take(128, 256, M, tile_cost(M, N, 128, 256, big));
    if (tall) {
      take(64, 128, M, tile_cost(M, N, 64, 128, mid));
      if (!dword) take(64, 64, M, tile_cost(M, N, 64, 64, small));
      if (dword) take(128, 128, M, staged_cost(M, N, K, es, false));
    }
  } else {
    take(128, 128, M, staged_cost(M, N, K, es, upper));
  }
  const double rate = wave_rate(M, N, K, es, !dword ? kRowsAligned : kr ? kRowsOddKR : kRowsOddKC,
                                cls == kTilesKC && es == 4 && K % 4096 == 0);
  for (int side = 2; side >= 1; --side) {
    const int wk = waves_along_k(M, N, units, side);
    const double cost = wave_cost(M, N, rate, side, wk, upper);
    if (cost < best) {
      best = cost;
      p.side = side;
      p.wk = wk;
    }
  }
  p.cost = best;
  return p;
}

}  // namespace

TilePick pick_tiles(TileClass cls, long long M, long long N, long long K, long long mt,
                    long long nt, long long units, int es, bool tall, bool split,
                    bool upper) {
  const TilePick whole = pick_launch(cls, mt, nt, K, units, es, tall, split, upper);
  if (whole.side && whole.wk > 1) return whole;
  // one wave along K or a big tile: the same order of the sums, so the launch's own
  // extents decide
  return pick_launch(cls, M, N, K, 1, es, tall, split, upper);
}

TilePick pick_part_tiles(long long M, long long N, long long K, int splits, long long units, int es,
                         bool direct) {
  TilePick p;
  p.main_rows = M;
  double best = 0.0;
  auto rounds = [&](long long bm, long long bn) {
    return static_cast<double>((((M + bm - 1) / bm) * ((N + bn - 1) / bn) * splits + 255) / 256);
  };
  auto take = [&](int bm, int bn, double rate) {
    const double cost = rounds(bm, bn) * bm * bn / rate;
    if (p.bm && cost >= best) return;
    best = cost;
    p.bm = bm;
    p.bn = bn;
  };
  if (direct) {
    take(128, 256, 0.88);
    // (shares on short ranges of K; 1600 x 1600 over 14 ranges of 9257: 18.6 ms on
    // 128 x 256, 19.8 on 64 x 128)
    take(64, 128, 0.78);
    take(64, 64, 0.76);
  }
  const double rate = wave_rate(M, N, K, es, !direct && es == 8 ? kRowsOddKC : kRowsAligned, false);
  for (int side = 2; side >= 1; --side) {
    const int t = 32 * side;
    const double r = rounds(t, t);
    int wk = 1;
    while (2 * wk * side * side <= 16 && units >= 4LL * wk && r * wk * side * side < 8) wk *= 2;
    const double busy = r * wk * side * side >= 8 ? 1.0 : r * wk * side * side / 8;
    const double cost = r * t * t / (rate * busy);
    if (p.bm && cost >= best) continue;
    best = cost;
    p.bm = p.bn = t;
    p.side = side;
    p.wk = wk;
  }
  p.cost = best;
  return p;
}

bool split_pays(const TilePick& part, long long M, long long N, long long K, int splits,
                long long units, int es) {
  const TilePick whole = pick_launch(kTilesKCDword, M, N, K, units, es, es == 8, true);
  // a partial is written and read (16 bytes at 4 TB/s)
  const double sums = 16.0 * splits * M * N * 0.14e12 / 4e12 * (es == 4 ? 2.0 : 1.0);
  // (about equal: the ranges, whose workgroups are spread over more compute units, o=6 v=99
  // float32 X 81 against 97 us)
  return part.cost * K / splits + sums < 1.1 * whole.cost * K;
}

PairPick pick_pair_products(const PairExtents& whole, const PairExtents& block, long long kp, int es,
                            int chunk, long long max_splits) {
  PairPick pick;
  const int bk = 128 / es;
  const long long nk = (kp + bk - 1) / bk;
  if (whole.mp <= 0 || whole.np <= 0 || nk <= 0 || max_splits < 1) return pick;
  auto steps_of = [&](int s) {
    const long long n = (nk + s - 1) / s;
    return (n + chunk - 1) / chunk * chunk;
  };
  // multiply-adds of one compute unit, as tile_cost; a partial is written and read
  // (16 bytes at 4 TB/s)
  const double kPartial = 16.0 * 0.14e12 / 4e12 * (es == 4 ? 2.0 : 1.0);
  const struct { int bm, bn; double rate; } tiles[] = {
      {160, 256, 0.86}, {128, 256, 0.86}, {64, 128, 0.82}, {64, 64, 0.78}};
  struct Counts { long long p[4], m[4]; double values; };  // tiles of either product
  auto count = [&](const PairExtents& e) {
    Counts c{{}, {}, static_cast<double>(e.mp) * e.np + static_cast<double>(e.mm) * e.nm};
    for (int i = 0; i < 4; ++i) {
      c.p[i] = ((e.mp + tiles[i].bm - 1) / tiles[i].bm) * ((e.np + tiles[i].bn - 1) / tiles[i].bn);
      c.m[i] = ((e.mm + tiles[i].bm - 1) / tiles[i].bm) * ((e.nm + tiles[i].bn - 1) / tiles[i].bn);
    }
    return c;
  };
  auto best_tile = [&](const Counts& c, int s, PairPick* p) {
    double best = 0.0;
    const double steps = static_cast<double>(steps_of(s)) * bk;
    auto time = [&](long long n, int i) {
      return static_cast<double>((n * s + 255) / 256) * tiles[i].bm * tiles[i].bn * steps / tiles[i].rate;
    };
    for (int i = es == 4 ? 1 : 0; i < 4; ++i) {
      const auto& t = tiles[i];
      const double cost = time(c.p[i] + c.m[i], i);
      if (best == 0.0 || cost < best) {
        best = cost;
        p->bm = p->bm2 = t.bm;
        p->bn = p->bn2 = t.bn;
        p->apart = false;
      }
    }
    // Two launches on tiles of different heights where the rows of both products then
    // end on whole rounds and a round is long: o=40 v=360, rows 820 and 780 in 7 rounds of
    // 128 and 5 of 160, 220 -> 211 ms; o=60 v=360 492 -> 465.  Shorter ones leave more idle
    // between the launches (o=36 v=160 7.0 -> 7.3 ms).
    if (es == 8 && kp >= 32768)
      for (int i = 0; i < 2; ++i) {
        const int j = 1 - i;
        const double cost = time(c.p[i], i) + time(c.m[j], j);
        if (cost >= 0.975 * best) continue;
        best = cost;
        p->bm = tiles[i].bm;
        p->bm2 = tiles[j].bm;
        p->bn = p->bn2 = tiles[i].bn;
        p->apart = true;
      }
    return best + c.values * s * kPartial;
  };
  const Counts all = count(whole);
  double best = 0.0;
  for (int s = 1; s <= kPairSplits && s <= max_splits; ++s) {
    if (s > 1 && (steps_of(s) < 8 || (nk + steps_of(s) - 1) / steps_of(s) != s)) continue;
    PairPick p;
    const double cost = best_tile(all, s, &p);
    if (pick.splits == 0 || cost < 0.99 * best) {
      best = cost;
      pick.splits = s;
    }
  }
  pick.cost = best_tile(count(block), pick.splits, &pick);
  return pick;
}

namespace {

// Layout for nb pair-balanced blocks; bytes is 0 when nb exceeds v.
FoldPlan layout_fold(const Plan& pl, int nb) {
  FoldPlan f;
  const int v = pl.v;
  if (nb < 1 || nb > v) return f;
  const size_t v2 = static_cast<size_t>(v) * v;
  f.nb = nb;
  f.ldp = static_cast<long long>((static_cast<size_t>(v) * (v + 1) / 2 + 3) / 4 * 4);
  f.ldm = static_cast<long long>((static_cast<size_t>(v) * (v - 1) / 2 + 3) / 4 * 4);
  const bool pairs = pl.pairsym || pl.pairsym_adj;
  f.rows_p = pairs ? (long long)pl.o * (pl.o + 1) / 2 : (long long)pl.o * pl.o;
  f.rows_m = pairs ? (long long)pl.o * (pl.o - 1) / 2 : (long long)pl.o * pl.o;
  size_t np = 0, nm = 0, na_max = 0;
  for (int k = 0; k < nb; ++k) {
    const int a0 = pair_block_start(v, nb, k), a1 = pair_block_start(v, nb, k + 1);
    const size_t n = static_cast<size_t>(pair_prefix(a1, v) - pair_prefix(a0, v));
    const size_t na = static_cast<size_t>(a1 - a0);
    np = n > np ? n : np;
    nm = n - na > nm ? n - na : nm;
    na_max = na > na_max ? na : na_max;
  }
  size_t cur = 0;
  f.off_Tp = take(&cur, f.rows_p * f.ldp * sizeof(double));
  f.off_Tm = take(&cur, f.rows_m * f.ldm * sizeof(double));
  f.off_V = take(&cur, np * v2 * sizeof(double));
  f.off_Vp = take(&cur, np * f.ldp * sizeof(double));
  f.off_Vm = take(&cur, nm * f.ldm * sizeof(double));
  // tile rows of the packed build, or of the pair-pair integral's upper triangle
  const size_t rows_m = pl.gsym ? static_cast<size_t>(f.ldp) : na_max * v;
  f.off_tiles = take(&cur, ((rows_m + 127) / 128 + 1) * sizeof(int));
  f.bytes = cur;
  return f;
}

}  // namespace

bool plan_fold(const Plan& pl, FoldPlan* f) {
  if (!pl.fold) return false;
  const size_t room = pl.bytes - (pl.check_sym ? kAlign : 0);  // the same choice with the check
  // The fewest blocks that fit (the footprint shrinks, but for the odd pair, as their count
  // grows; most plans hold few), at most the least scratch's, which do.
  int lo = 1, hi = 1;
  while (hi < pl.fold && layout_fold(pl, hi).bytes > room) {
    lo = hi + 1;
    hi = 2 * hi < pl.fold ? 2 * hi : pl.fold;
  }
  while (lo < hi) {
    const int mid = lo + (hi - lo) / 2;
    if (layout_fold(pl, mid).bytes <= room) hi = mid; else lo = mid + 1;
  }
  *f = layout_fold(pl, hi);
  return true;
}

namespace {

// Times of the two float64 forwards in so many equal blocks, in multiply-adds of one
// compute unit (0.14e12 a second): builds and contractions as they are tiled, or the bytes
// of the integral where these take longer (memory passes at 4 TB/s), launches at 5 us.  On
// 440 sizes (o = 1 to 75, v = 48 to 180, P = v / 4 and 3 (o + v), either flag, whole scratch
// and a fifth) the ratio of the two is within 17% rms of the measured one, which runs from
// 0.3 (o=2 v=65 pair-symmetric: combining costs more than the small contraction saves) to
// 1.9 (o=20 v=72); the wrong choice costs 0.8% on average.  Where 2 o^2 > v^2 the scratch
// holds no partial sums and the folded contraction scatters its results, in more blocks
// for the larger t+-: o=60 v=64 direct 2.28 ms, folded 2.83; o=46 v=64 1.71 and 1.48.
constexpr double kLaunch = 5e-6 * 0.14e12, kByte = 0.14e12 / 4e12;

double build_cost(long long rows, long long cols, int P, long long values) {
  const double build = pick_launch(kTilesStaged, rows, cols, P, (P + 15) / 16, sizeof(double), true,
                                   false).cost * P;
  const double write = 8.0 * values * kByte;
  return build > write ? build : write;
}

double direct_forward_cost(int o, int v, int P, bool pairs, bool exchange, int blocks) {
  const long long v2 = (long long)v * v, o2 = (long long)o * o, n = pairs ? (v2 + v) / 2 : v2;
  const long long nb = (n + blocks - 1) / blocks;
  const double contract = pick_launch(v % 2 ? kTilesKCDword : kTilesKC, o2, nb, v2, (v2 + 15) / 16,
                                      sizeof(double), true, true).cost * v2;
  // (the exchange partner's swapped copy of t; t+- need none)
  return blocks * (build_cost((v2 + blocks - 1) / blocks, pairs ? v2 / 2 : v2, P, nb * v2) +
                   contract + (pairs ? 3 : 2) * kLaunch) +
         (exchange ? kLaunch + 16.0 * o2 * v2 * kByte : 0.0);
}

double folded_forward_cost(int o, int v, int P, bool pairs, int blocks) {
  const long long v2 = (long long)v * v, o2 = (long long)o * o, kp = (v2 + v) / 2, km = kp - v;
  const long long rp = pairs ? (o2 + o) / 2 : o2, rm = pairs ? rp - o : o2;
  const long long np = (kp + blocks - 1) / blocks, nm = (km + blocks - 1) / blocks;
  double cost = build_cost((v2 + blocks - 1) / blocks, v2 / 2, P, np * v2) +
                16.0 * np * v2 * kByte + 3 * kLaunch;
  const PairPick pick = pick_pair_products(PairExtents{rp, kp, rm, km}, PairExtents{rp, np, rm, nm},
                                           kp, sizeof(double), 1, v2 / (rp + rm));
  if (pick.splits)
    cost += pick.cost + 32.0 * rp * np * kByte + 2 * kLaunch;
  else
    cost += pick_launch(kTilesKC, rp, np, kp, (kp + 15) / 16, sizeof(double), true, true).cost * kp +
            pick_launch(kTilesKC, rm, nm, km, (km + 15) / 16, sizeof(double), true, true).cost * km +
            128.0 * rp * np * kByte + 2 * kLaunch;
  return blocks * cost + 16.0 * rp * v2 * kByte + kLaunch;
}

// The same of the split-int8 forward.  Against the direct route the stacked one has half the
// build and half the re-cut integral rows, and twice the re-cut t: over o = 2 to 75, v =
// 64 to 150 it took 0.61 to 0.99 of the direct route's time for v >= 3 o (o=20 v=64 P=16
// 1.05) and up to 1.47 below (o=60 v=64 1.13 -> 1.52 ms, o=40 v=96 P=24 2.11 -> 2.21), but where
// its contraction takes fewer rounds of the compute units (o=30 v=65: one for two, 685 -> 488 us).
RouteRule stacked_rule(int o, int v, int P, int slices, unsigned flags, bool least);

// `least` false: bytes is what the direct route's whole scratch holds, not the least.
RouteRule route_rule(int o, int v, int P, int precision, int backward, int slices, unsigned flags,
                     bool least) {
  RouteRule r;
  if (precision == CC_LADDER_SPLIT_INT8 && !backward) return stacked_rule(o, v, P, slices, flags, least);
  // Below 64 virtuals the extra launches take what the products save.
  if (precision != CC_LADDER_FP64 || backward || (flags & CC_LADDER_PLUS_MINUS) || v < 64) return r;
  const bool pairs = (flags & CC_LADDER_PAIR_SYMMETRIC) != 0, swap = (flags & CC_LADDER_EXCHANGE) != 0;
  Plan pl;
  pl.o = o;
  pl.v = v;
  pl.P = P;
  pl.pairsym = pairs ? 1 : 0;
  const size_t v2 = static_cast<size_t>(v) * v;
  const size_t row = v2 * sizeof(double), rows = pairs ? (v2 + v) / 2 : v2;
  int nb = 1;
  while (nb <= 32 && nb < v && layout_fold(pl, nb).bytes > rows * row) ++nb;
  // The faster route in the direct one's whole scratch, and down to the scratch where the
  // direct one's blocks would be the faster ones (it needs no t+-).
  for (int blocks = 1; nb <= v; nb = nb == v ? v + 1 : nb + nb / 2 + 1 < v ? nb + nb / 2 + 1 : v) {
    const size_t bytes = layout_fold(pl, nb).bytes;
    if (bytes > rows * row) break;
    if (r.blocks) {  // rows of a direct block in the scratch of one folded block less
      size_t held = (nb > 1 ? layout_fold(pl, nb - 1).bytes : bytes) / row;
      if (!pairs) held = held / v * v;
      blocks = held ? static_cast<int>((rows + held - 1) / held) : v;
      if (blocks < 1) blocks = 1;
    }
    // (a tenth more on the way down: the rounds of either grid jump by as much)
    const double folded = folded_forward_cost(o, v, P, pairs, nb);
    if (folded >= (r.blocks ? 1.1 : 1.0) * direct_forward_cost(o, v, P, pairs, swap, blocks)) break;
    r.blocks = nb;
    r.bytes = bytes;
    if (!least) break;
  }
  return r;
}

}  // namespace

namespace {

StackedPlan layout_stacked_i8(const Plan& pl, int nb) {
  StackedPlan q;
  const int v = pl.v;
  if (nb < 1 || nb > v) return q;
  const size_t v2 = static_cast<size_t>(v) * v, o2 = static_cast<size_t>(pl.o) * pl.o;
  size_t np = 0, na_max = 0;
  for (int k = 0; k < nb; ++k) {
    const int a0 = pair_block_start(v, nb, k), a1 = pair_block_start(v, nb, k + 1);
    const size_t n = static_cast<size_t>(pair_prefix(a1, v) - pair_prefix(a0, v));
    np = n > np ? n : np;
    na_max = static_cast<size_t>(a1 - a0) > na_max ? static_cast<size_t>(a1 - a0) : na_max;
  }
  q.nb = nb;
  q.npk = static_cast<long long>(np);
  const size_t s = static_cast<size_t>(pl.slices);
  const SliceDims dL = slice_dims(static_cast<long long>(v2), pl.P);
  const SliceDims dt = slice_dims(static_cast<long long>(2 * o2), static_cast<int>(v2));
  const SliceDims dV = slice_dims(q.npk, static_cast<int>(v2));
  size_t cur = 0;
  q.off_L = take(&cur, s * dL.rows_pad * dL.k_pad);
  q.off_Lexp = take(&cur, static_cast<size_t>(dL.rows_pad) * i8_chunks(dL.k_pad) * sizeof(int));
  q.off_t = take(&cur, s * dt.rows_pad * dt.k_pad);
  q.off_texp = take(&cur, static_cast<size_t>(dt.rows_pad) * i8_chunks(dt.k_pad) * sizeof(int));
  q.off_V = take(&cur, (np > o2 ? np : o2) * v2 * sizeof(double));
  q.off_Vs = take(&cur, s * dV.rows_pad * dV.k_pad);
  q.off_Vexp = take(&cur, static_cast<size_t>(dV.rows_pad) * i8_chunks(dV.k_pad) * sizeof(int));
  q.off_tiles = take(&cur, ((na_max * v + 127) / 128 + 1) * sizeof(int));
  q.bytes = cur;
  return q;
}

RouteRule stacked_rule(int o, int v, int P, int slices, unsigned flags, bool least) {
  RouteRule r;
  if ((flags & CC_LADDER_PAIR_SYMMETRIC) || v < 64) return r;
  const long long o2 = (long long)o * o, v2 = (long long)v * v;
  auto rounds = [](long long M, long long N) { return ((M + 127) / 128 * ((N + 127) / 128) + 255) / 256; };
  if (v < 3 * o && 4 * rounds(2 * o2, (v2 + v) / 2) > 3 * rounds(o2, v2)) return r;
  Plan pl, one;  // the direct route's whole range and one virtual
  const RouteRule none;
  if (layout_plan(o, v, P, CC_LADDER_SPLIT_INT8, 0, v, slices, 0, 0, flags, &pl, 0, false, &none) ||
      layout_plan(o, v, P, CC_LADDER_SPLIT_INT8, 0, 1, slices, 0, 0, flags, &one, 0, false, &none))
    return r;
  const double per = static_cast<double>(pl.bytes - one.bytes) / (v - 1);
  // as long as it needs at most twice the blocks that the direct route would have in the
  // same scratch
  for (int nb = 1; nb <= v; nb = nb == v ? v + 1 : nb + nb / 2 + 1 < v ? nb + nb / 2 + 1 : v) {
    const size_t bytes = layout_stacked_i8(pl, nb).bytes;
    if (bytes > pl.bytes) continue;
    if (r.blocks) {
      const double held = 1.0 + (static_cast<double>(bytes) - static_cast<double>(one.bytes)) / per;
      if (held >= 1.0 && nb > 2 * ((v + static_cast<int>(held) - 1) / static_cast<int>(held))) break;
    }
    r.blocks = nb;
    r.bytes = bytes;
    if (!least) break;
  }
  return r;
}

}  // namespace

bool plan_stacked_i8(const Plan& pl, StackedPlan* q) {
  if (!pl.stacked) return false;
  int nb = 1;
  while (nb < pl.stacked && layout_stacked_i8(pl, nb).bytes > pl.bytes) ++nb;
  // One persistent workgroup per compute unit walks a contraction's 128 x 128 tiles: a
  // block or two more may leave fewer rounds (o=30 v=128 in a third of the whole scratch: 3
  // blocks of 2 rounds, or 4 of one)
  auto rounds = [&](int n) {
    const long long tm = (2LL * pl.o * pl.o + 127) / 128;
    double sum = 0.05 * n;
    for (int k = 0; k < n; ++k) {
      const int a0 = pair_block_start(pl.v, n, k), a1 = pair_block_start(pl.v, n, k + 1);
      const long long np = pair_prefix(a1, pl.v) - pair_prefix(a0, pl.v);
      sum += static_cast<double>((tm * ((np + 127) / 128) + 255) / 256);
    }
    return sum;
  };
  *q = layout_stacked_i8(pl, nb);
  double best = rounds(nb);
  for (int n = nb + 1; n <= nb + 3 && n <= pl.stacked; ++n) {
    const StackedPlan more = layout_stacked_i8(pl, n);
    if (more.bytes > pl.bytes || rounds(n) >= best) continue;
    best = rounds(n);
    *q = more;
  }
  return true;
}

bool plan_fold_adjoint(const Plan& pl, FoldAdjoint* a) {
  // From 64 virtuals on, as the forward: below, the extra launches take what the
  // products save; from 16 for pair-symmetric t and lam, whose direct route has as many
  // launches and K-banded products (o=6 v=33 P=120: 567 -> 93 us).  W is
  // formed whole, so a plan of several blocks keeps the direct route; in a plan of one
  // block dt's stage is the smaller one (1 v^4 values against W+- and S, 1.5 v^4; with
  // symmetric vectors G beside it, which the plan holds too).
  if (pl.op != kOpLadder || pl.precision != CC_LADDER_FP64 || !pl.backward || pl.n_a != pl.v ||
      pl.v < (pl.pairsym_adj ? 16 : 64))
    return false;
  const size_t room = pl.bytes - (pl.check_sym ? kAlign : 0);
  const int v = pl.v;
  const size_t v2 = static_cast<size_t>(v) * v;
  const size_t kp = static_cast<size_t>(v) * (v + 1) / 2;
  // (odd v: with S and a copy of L on padded rows where they fit)
  for (int pad = v % 2; pad >= 0; --pad) {
    FoldAdjoint p;
    p.f = layout_fold(pl, 1);  // t+- first, then the integrals
    p.lds = static_cast<long long>(v2) + pad;
    p.copy_L = pad != 0;
    const size_t ldp = p.f.ldp, ldm = p.f.ldm;
    // lam+- after t+-; dt's stage (the integrals) and W+-, S share what follows
    size_t cur = p.f.off_V;
    p.off_Mp = take(&cur, p.f.rows_p * ldp * sizeof(double));
    p.off_Mm = take(&cur, p.f.rows_m * ldm * sizeof(double));
    if (pl.gsym) {
      p.off_Lp = take(&cur, static_cast<size_t>(pl.P) * ldp * sizeof(double));
      p.off_G = take(&cur, ldp * ldp * sizeof(double));
    }
    const size_t shift = cur - p.f.off_V;
    p.f.off_V += shift;
    p.f.off_Vp += shift;
    p.f.off_Vm += shift;
    p.f.off_tiles += shift;
    p.f.bytes += shift;
    // (W+- and S follow lam+-, in the place of the vectors and G as well)
    cur = p.off_Mm + (p.f.rows_m * ldm * sizeof(double) + kAlign - 1) / kAlign * kAlign;
    p.off_Wp = take(&cur, kp * ldp * sizeof(double));
    p.off_Wm = take(&cur, (kp - v) * ldm * sizeof(double));
    p.off_S = take(&cur, v2 * p.lds * sizeof(double));
    if (p.copy_L) p.off_L = take(&cur, static_cast<size_t>(pl.P) * p.lds * sizeof(double));
    p.bytes = cur > p.f.bytes ? cur : p.f.bytes;
    if (p.bytes <= room) {
      *a = p;
      return true;
    }
  }
  return false;
}

int layout_intermediate(int which, int o, int v, int P, int precision, int n_p, int k_chunk,
                        Plan* plan) {
  const int n_first = which == CC_INTERMEDIATE_IJBK ? v : o;
  if (n_p < 1 || n_p > n_first) return CC_LADDER_EINVAL;
  Plan p;
  p.o = o; p.v = v; p.P = P;
  p.precision = precision;
  p.op = which == CC_INTERMEDIATE_IJKL ? kOpIjkl : which == CC_INTERMEDIATE_IJBK ? kOpIjbk : kOpHole;
  p.n_a = n_p;
  p.nblocks = (n_first + n_p - 1) / n_p;
  const size_t v2 = static_cast<size_t>(v) * v;
  const size_t o2 = static_cast<size_t>(o) * o;
  const size_t ov = static_cast<size_t>(o) * v;
  // integral block: [n_p][o][v][v] for the intermediates, (ik|jl) as [n_p][o][o][o]
  // for the hole-hole ladder
  const size_t blk = p.op == kOpHole ? static_cast<size_t>(n_p) * o * o2
                                     : static_cast<size_t>(n_p) * o * v2;
  size_t cur = 0;
  switch (precision) {
    case CC_LADDER_FP64:
      // (bd|kc) is built with its last two indices in (d, c) order and met by
      // the amplitudes with c, d swapped
      if (p.op == kOpIjbk) p.off_tx = take(&cur, o2 * v2 * sizeof(double));
      p.off_V = take(&cur, blk * sizeof(double));
      break;
    case CC_LADDER_FP32:
      p.k_chunk = k_chunk ? k_chunk : 512;
      // L_ov (L_oo for the hole-hole ladder)
      p.off_L = take(&cur, static_cast<size_t>(P) * (p.op == kOpHole ? o2 : ov) * sizeof(float));
      if (p.op == kOpIjbk) p.off_L2 = take(&cur, static_cast<size_t>(P) * v2 * sizeof(float));
      p.off_t = take(&cur, o2 * v2 * sizeof(float));
      p.off_V = take(&cur, blk * sizeof(float));
      break;
    case CC_LADDER_SPLIT_BF16:
    case CC_LADDER_SPLIT_INT8:
      return CC_LADDER_EUNSUPPORTED;
    default:
      return CC_LADDER_EINVAL;
  }
  if (p.op != kOpHole) {
    // split K from the whole output's tile count, so every block sums in the
    // same order whatever n_p is
    p.k_splits = choose_k_splits(static_cast<long long>(o2), static_cast<long long>(n_first) * o,
                                 static_cast<long long>(v2), precision == CC_LADDER_FP64 ? 16 : 32);
    if (p.k_splits > 1)
      p.off_part = take(&cur, static_cast<size_t>(p.k_splits) * o2 * n_p * o * sizeof(double));
  }
  p.bytes = cur;
  *plan = p;
  return CC_LADDER_OK;
}

int make_plan_intermediate(int which, int o, int v, int P, int precision, size_t budget,
                           const cc_ladder_opts* opts, Plan* plan) {
  if (which != CC_INTERMEDIATE_IJKL && which != CC_INTERMEDIATE_IJBK && which != CC_HOLE_LADDER)
    return CC_LADDER_EINVAL;
  int rc = check_dims(o, v, P);
  if (rc) return rc;
  rc = check_precision_opts(precision, opts);
  if (rc) return rc;
  // the packed and exchange variants belong to the ladder term only
  if (opts && opts->flags) return CC_LADDER_EUNSUPPORTED;
  const int k_chunk = opts ? opts->k_chunk : 0;
  const int n_first = which == CC_INTERMEDIATE_IJBK ? v : o;
  return search_block(n_first, budget, opts ? opts->a_block : 0, [&](int n_p, Plan* p) {
    return layout_intermediate(which, o, v, P, precision, n_p, k_chunk, p);
  }, plan);
}

}  // namespace ccl
