// Register-direct GEMM for products whose 128 x 256 tile grid leaves compute
// units idle (gfx950): small C, or a C of few rows, with any layout and any
// element-aligned operand.
//
//   C[m][n] (+)= sum_k A(m,k) B(k,n)     (layouts and epilogues of gemm.hpp)
//
// Each wave owns a 32 x 32 sub-tile (2 x 2 blocks of 16 x 16) and loads its MFMA
// operands from global memory straight into registers, one K-step ahead; a
// workgroup is WM x WN sub-tiles times WK waves along K (WK = waves / (WM * WN),
// at most 16 waves).  What bounds the small products is the serial K loop of a
// few workgroups and the latency of every step, not bandwidth: one float64 MFMA
// occupies its SIMD for 64 cycles, so a wave's step (16 k, 16 MFMAs) takes 1024
// cycles against 8 KB of operands (32 rows and 32 columns), 8 bytes a cycle and wave;
// with the eight waves that hide the latency that is what the vector cache of a
// compute unit delivers, and why full grids reach 0.62 of the matrix rate here and
// 0.78 to 0.88 on the LDS-staged tiles.  The K-steps are dealt to the WK waves in turn (step s to wave s mod
// WK; for float32 whole drain chunks, so that every float32 partial sum is the
// one of the larger kernels), and the waves' sums are added in LDS as a fixed
// binary tree.
//
// Measured on MI355X, float64, against the kernels it replaces there: contractions
// of 25 x 400 x 400 102 -> 10 us and 36 x 2556 x 2556 628 -> 37 us (128 x 256
// tiles), 400 x 4950 x 4950 1223 -> 398 us; builds of v = 20, P = 75 19 -> 6 us and
// v = 71, P = 263 277 -> 239 us (128 x 128 tiles).
//
// Row-contiguous operands: lane r of a block pair holds rows 2r and 2r + 1 of the
// 32 (block i's row r is sub-tile row 2r + i), one 2-element load per k.  Rows
// past M (columns past N) are clamped onto valid ones and never stored; the
// last, ragged K-step loads element by element with zero fill.
#pragma once

#include "gemm.hpp"

namespace ccl {

constexpr int kWTile = 32;      // sub-tile side of one wave
constexpr int kWMaxWaves = 16;  // waves per workgroup

// LDS bytes of a workgroup of wmn sub-tiles times wk waves along K (at most 64 KB).
inline unsigned wave_lds_bytes(int wmn, int wk) {
  return static_cast<unsigned>(wk / 2 * wmn) * 16u * 64u * sizeof(double);
}

// One operand of a wave: 32 rows (A) or columns (B) from `row0`.
template <class Tr, int LAY>
struct WaveOp {
  using T = typename Tr::T;
  static constexpr int CH = Tr::CH;
  static constexpr int STEP = 8 * CH;  // k per step: two k-groups of 4 * CH
  typedef T Vec __attribute__((ext_vector_type(LAY == KC ? CH : 2), aligned(sizeof(T))));
  // values of one step: KC [group][block] chunks of CH k; RC [group][k in chunk] row pairs
  static constexpr int NV = LAY == KC ? 4 : 2 * CH;

  const T* p;      // this lane's first value at k = 0
  const T* p1;     // KC: second block
  long long ld;
  bool last;       // RC: the pair's load starts one row early (odd edge)
  int slot;

  __device__ __forceinline__ void init(const T* base, long long ld_, int row0, int nrows, int lane) {
    ld = ld_;
    slot = lane >> 4;
    const int r = lane & 15;
    last = false;
    if (LAY == KC) {
      int a = row0 + r, b = row0 + 16 + r;
      a = a < nrows ? a : nrows - 1;
      b = b < nrows ? b : nrows - 1;
      p = base + (long long)a * ld + CH * slot;
      p1 = base + (long long)b * ld + CH * slot;
    } else {
      int a = row0 + 2 * r;
      last = a == nrows - 1;
      a = a < nrows - 1 ? a : nrows - 2;  // nrows >= 2 (checked by the host)
      p = base + (long long)(CH * slot) * ld + a;
      p1 = p;
    }
  }

  // full step at k0 (k0 + STEP <= K)
  __device__ __forceinline__ void load(Vec (&v)[NV], int k0) const {
    if (LAY == KC) {
#pragma unroll
      for (int gi = 0; gi < 2; ++gi) {
        v[2 * gi] = *reinterpret_cast<const Vec*>(p + k0 + 4 * CH * gi);
        v[2 * gi + 1] = *reinterpret_cast<const Vec*>(p1 + k0 + 4 * CH * gi);
      }
    } else {
#pragma unroll
      for (int gi = 0; gi < 2; ++gi)
#pragma unroll
        for (int e = 0; e < CH; ++e)
          v[gi * CH + e] = *reinterpret_cast<const Vec*>(p + (long long)(k0 + 4 * CH * gi + e) * ld);
    }
  }

  // the last step when K is not a multiple of STEP: zeros at k >= K
  __device__ __forceinline__ void load_tail(Vec (&v)[NV], int k0, int K) const {
#pragma unroll
    for (int gi = 0; gi < 2; ++gi) {
      const int kb = k0 + 4 * CH * gi;  // slot offset is in p
#pragma unroll
      for (int e = 0; e < CH; ++e) {
        const bool ok = kb + CH * slot + e < K;
        if (LAY == KC) {
          v[2 * gi][e] = ok ? p[kb + e] : T(0);
          v[2 * gi + 1][e] = ok ? p1[kb + e] : T(0);
        } else {
          Vec z = {T(0), T(0)};
          if (ok) z = *reinterpret_cast<const Vec*>(p + (long long)(kb + e) * ld);
          v[gi * CH + e] = z;
        }
      }
    }
  }

  // MFMA operand of block i, MFMA step e of group gi
  __device__ __forceinline__ T get(const Vec (&v)[NV], int gi, int e, int i) const {
    if (LAY == KC) return v[2 * gi + i][e];
    const Vec x = v[gi * CH + e];
    return i == 0 ? (last ? x[1] : x[0]) : x[1];
  }

  // sub-tile row of block i's row r
  __device__ static __forceinline__ int pos(int i, int r) {
    return LAY == KC ? 16 * i + r : 2 * r + i;
  }
};

template <class Tr, int LA, int LB, int EPI, int WM, int WN>
__global__ __launch_bounds__(64 * kWMaxWaves) void gemm_wave_kernel(GemmArgs<typename Tr::T> g) {
  using T = typename Tr::T;
  using Acc = typename Tr::Acc;
  using OA = WaveOp<Tr, LA>;
  using OB = WaveOp<Tr, LB>;
  constexpr int CH = Tr::CH;
  constexpr int STEP = OA::STEP;
  constexpr int BM = kWTile * WM, BN = kWTile * WN;
  // the sums that half of the waves along K hand over: 16 doubles per lane and
  // wave (wave_lds_bytes; none when WK is 1)
  extern __shared__ double wave_red[];
  double(*red)[16][64] = reinterpret_cast<double(*)[16][64]>(wave_red);

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int WK = static_cast<int>(blockDim.x >> 6) / (WM * WN);
  const int wk = wave / (WM * WN), wt = wave % (WM * WN);
  int tm, tn;
  const int nk_all = (g.K + STEP - 1) / STEP;
  int ks0 = 0, nk = nk_all;  // K-steps of this workgroup
  if (EPI == EPI_PART) {
    // grid = tiles x splits, as in the K-contiguous direct kernel
    const int ntiles = g.tiles_m * g.tiles_n;
    const int id = xcd_linear(blockIdx.x, gridDim.x);
    const int split = id / ntiles;
    tile_from_linear(id - split * ntiles, ntiles, g.tiles_m, g.group_m, tm, tn);
    ks0 = split * g.split_steps;
    nk = ks0 + g.split_steps < nk_all ? ks0 + g.split_steps : nk_all;
    g.C = static_cast<double*>(g.C) + split * g.part_stride;
  } else if (EPI == EPI_PACK || EPI == EPI_SYM) {
    // tiles below the diagonal end at once: dealt to the XCDs in turn, so that each has
    // as many of the others
    tile_from_linear(blockIdx.x, gridDim.x, g.tiles_m, g.group_m, tm, tn);
  } else if (g.kband) {
    tile_of_banded(g.kband, blockIdx.x, gridDim.x, g.tiles_m, g.group_m, tm, tn);
    k_band(g, tn * BN, STEP, ks0, nk);
  } else {
    tile_of(blockIdx.x, gridDim.x, g.tiles_m, g.group_m, tm, tn);
  }
  const int m0 = tm * BM, n0 = tn * BN;
  if (EPI == EPI_PACK || EPI == EPI_SYM) {
    // every column's b below every row's a: nothing of this tile is kept
    const int nlast = ((n0 + BN < g.N) ? n0 + BN : g.N) - 1;
    if (nlast / g.v < m0 / g.v) return;
  }
  const int wm0 = m0 + (wt / WN) * kWTile, wn0 = n0 + (wt % WN) * kWTile;

  OA a;
  OB b;
  a.init(g.A, g.lda, wm0, g.M, lane);
  b.init(g.B, g.ldb, wn0, g.N, lane);

  Acc acc[2][2];
  f64x4 sum[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      acc[i][j] = Acc{0, 0, 0, 0};
      sum[i][j] = f64x4{0, 0, 0, 0};
    }
  auto compute = [&](const typename OA::Vec (&va)[OA::NV], const typename OB::Vec (&vb)[OB::NV]) {
#pragma unroll
    for (int gi = 0; gi < 2; ++gi)
#pragma unroll
      for (int e = 0; e < CH; ++e) {
        T fa[2], fb[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) fa[i] = a.get(va, gi, e, i);
#pragma unroll
        for (int j = 0; j < 2; ++j) fb[j] = b.get(vb, gi, e, j);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = Tr::mfma(fa[i], fb[j], acc[i][j]);
      }
  };
  typename OA::Vec a0[OA::NV], a1[OA::NV];
  typename OB::Vec b0[OB::NV], b1[OB::NV];
  // steps loaded without tests: all but a ragged last one of the whole product
  const int nfull = nk < g.K / STEP ? nk : g.K / STEP;

  // Steps s, s + stride, ... < s1 of this wave, all full: loads one step ahead.
  auto run = [&](int s, int s1, int stride) {
    if (s >= s1) return;
    a.load(a0, s * STEP);
    b.load(b0, s * STEP);
    for (; s + stride < s1; s += 2 * stride) {
      a.load(a1, (s + stride) * STEP);
      b.load(b1, (s + stride) * STEP);
      compute(a0, b0);
      const int s2 = s + 2 * stride < s1 ? s + 2 * stride : s + stride;  // in range either way
      a.load(a0, s2 * STEP);
      b.load(b0, s2 * STEP);
      compute(a1, b1);
    }
    if (s < s1) compute(a0, b0);
  };
  auto tail = [&]() {
    const int kt = g.K / STEP * STEP;
    a.load_tail(a0, kt, g.K);
    b.load_tail(b0, kt, g.K);
    compute(a0, b0);
  };
  if (!Tr::kDrain) {
    run(ks0 + wk, nfull, WK);
    if (nk > nfull && (nfull - ks0) % WK == wk) tail();
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) sum[i][j][r] = static_cast<double>(acc[i][j][r]);
  } else {
    // chunks of drain_steps K-steps: float32 within a chunk, float64 across
    for (int c = ks0 + wk * g.drain_steps; c < nk; c += WK * g.drain_steps) {
      const int e = c + g.drain_steps < nk ? c + g.drain_steps : nk;
      run(c, e < nfull ? e : nfull, 1);
      if (e > nfull) tail();
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            sum[i][j][r] += static_cast<double>(acc[i][j][r]);
            acc[i][j][r] = 0;
          }
    }
  }

  // tree over the waves along K: the upper half hands its sums to the lower half
  for (int n = WK; n > 1;) {
    const int h = (n + 1) >> 1;
    if (wk >= h && wk < n) {
      double(*dst)[64] = red[(wk - h) * (WM * WN) + wt];
#pragma unroll
      for (int q = 0; q < 16; ++q) dst[q][lane] = sum[q >> 3][(q >> 2) & 1][q & 3];
    }
    __syncthreads();
    if (wk + h < n) {
      const double(*src)[64] = red[wk * (WM * WN) + wt];
#pragma unroll
      for (int q = 0; q < 16; ++q) sum[q >> 3][(q >> 2) & 1][q & 3] += src[q][lane];
    }
    __syncthreads();
    n = h;
  }
  if (wk != 0) return;

#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int n = wn0 + OB::pos(j, lane & 15);
    if (n >= g.N) continue;
    const EpiCol ec = epi_col<T, EPI>(g, n);
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = wm0 + OA::pos(i, Tr::row_of(lane, r));
        if (m >= g.M) continue;
        epi_store<T, EPI>(g, m, n, ec, sum[i][j][r]);
      }
  }
}

}  // namespace ccl
