// Amplitude-contraction GEMM with direct global->LDS operand loads (gfx950).
//
//   C[m][n] (+)= sum_k A[m*lda + k] B[n*ldb + k]   (both operands KC; EPI_ACC, EPI_PAIR,
//                                                   EPI_PM, EPI_FOLD, or EPI_PART: one
//                                                   K-range per workgroup)
//
// 512 threads = 8 wave64s in a 2 x 4 grid over a BM x 256 tile (BM = 128; the
// K-contiguous kernel also 64 and, for float64, 160); each wave owns (BM/2) x 64 =
// BM/32 x 4 MFMA blocks (v_mfma_f64_16x16x4_f64 or v_mfma_f32_16x16x4_f32).
// Every K-step is 128 bytes of each operand row.  Operand slabs of 8 rows go
// from global memory into LDS with global_load_lds_dwordx4 (lane l of a wave
// writes 16 bytes at the wave's LDS base + 16*l): lane l takes row l/8 and
// physical 16-byte slot l%8, which holds the logical k-chunk
// (l%8) ^ ((row/2) % 8).  Fragment reads undo the XOR, so the 16 rows read by
// 16 lanes of one ds_read_b128 land on 16 distinct 4-bank groups.  Three K-steps
// are in flight in a ring of LDS stages; one barrier per K-step.  Rows past M
// or N are clamped onto valid rows (their outputs are never stored); a ragged
// last K-step is loaded through registers with zero fill.
#pragma once

#include "gemm.hpp"

namespace ccl {

constexpr int kDBM = 128, kDBN = 256;
constexpr int kDThreads = 512;
constexpr int kDStages = 3;
constexpr int kDRow = 128;  // bytes of one operand row per K-step

typedef __attribute__((address_space(3))) void lds_void;

__device__ __forceinline__ void d_wait_vm(int n) {
  switch (n) {
#define CCL_DVM(N) \
  case N:          \
    __builtin_amdgcn_s_waitcnt(((N)&15) | (7 << 4) | (15 << 8) | (((N) >> 4) << 14)); \
    break;
    CCL_DVM(0) CCL_DVM(2) CCL_DVM(3) CCL_DVM(5) CCL_DVM(6) CCL_DVM(7) CCL_DVM(8) CCL_DVM(12)
    CCL_DVM(24)
#undef CCL_DVM
    default:
      __builtin_amdgcn_s_waitcnt(7 << 4 | 15 << 8);
  }
}

// BM = 128 (4 x 4 blocks per wave); for float64 without drains also 160 (5 x 4
// blocks per wave, 156 KB of LDS), whose tiles divide o^2 = 1600 exactly and pad
// 900 and 3600 less; and 64 (2 x 4 blocks per wave) for the remainder rows of a
// product whose last 128-row tile row would be at most half full.
// BN = 256; with BM = 64 also 128 and 64 (two workgroups per compute unit), for
// products whose 256-wide tiles leave compute units idle: one 128 x 256 tile takes
// its compute unit 4 us per 16 k (two waves per SIMD, 64 float64 MFMAs of 64 cycles
// each), so a short grid is bound by that serial loop.  169 x 4753 x 4753 float64:
// 1.17 ms on 128 x 256 tiles (38 workgroups), 0.19 ms on 64 x 64 (225); 800 x 4950 x
// 4950: 1.23 -> 0.63 ms on 64 x 128.
template <int BM, int BN>
constexpr int kc_groups() { return BM == 64 && BN < 256 ? 2 : 1; }  // per compute unit

// Dword load q (of four) of a 1 KB slab (8 rows of 128 bytes) of a K-contiguous operand,
// to the image that one 16-byte load per lane leaves: it brings rows 2q and 2q + 1.
// `tile` is the tile's first row at this step, `row` the slab's first row in the tile and
// `last` the last one that exists (rows past it repeat it; never stored).  Row addresses
// are uniform; a lane keeps the swizzled offset `at` and its second row's `hi`.
__device__ __forceinline__ void d_slab_dword(const char* tile, int row, int last, int ld_bytes,
                                             int q, unsigned at, unsigned hi,
                                             unsigned char* slab) {
  const int r = row + 2 * q;
  const char* base = tile + static_cast<unsigned>((r < last ? r : last) * ld_bytes);
  __builtin_amdgcn_global_load_lds((const void*)(base + (at + (r < last ? hi : 0u))),
                                   (lds_void*)(slab + 256 * q), 4, 0, 0);
}

// float64 steps issue the dword loads between their products: 24 in a row hold a wave's
// MFMAs up behind the address unit (o=75 v=225 X 57.3 -> 52.2 ms, Y 171 -> 155).  float32
// ones, whose drained sums fill the registers, keep them together (o=40 v=211 packed
// forward 54.2 ms, 67.2 with the spread loop's spills).
template <class T, bool DW>
constexpr bool d_spread() { return DW && sizeof(T) == 8; }

// The swizzled byte offset of a lane in load q of a slab of the wave's parity.
__device__ __forceinline__ unsigned d_dword_at(int lane, int wave, int q) {
  return ((((lane & 31) >> 2) ^ ((4 * (wave & 1) + q) & 7)) << 4) + ((lane & 3) << 2);
}

// Dword load q of a 1 KB piece of a row-contiguous operand (k rows of ROW bytes): 256
// bytes of one k row; a lane keeps the clamped column offset `at` of that quarter.
template <int ROW>
__device__ __forceinline__ void d_piece_dword(const char* step, int piece, int ld_bytes, int q,
                                              unsigned at, unsigned char* dst) {
  const char* base = step + static_cast<unsigned>((piece * 1024 + 256 * q) / ROW * ld_bytes);
  __builtin_amdgcn_global_load_lds((const void*)(base + at), (lds_void*)(dst + 256 * q), 4, 0, 0);
}

// The column offset of a lane in load q of the wave's pieces (pieces wave + 8j: 8 KB
// apart, so at the same place of a row).
template <class T, int ROW>
__device__ __forceinline__ unsigned d_dword_col(int lane, int wave, int q, int first, int count) {
  const int at = (wave * 1024 + 256 * q) % ROW + 4 * lane;
  int c = at / static_cast<int>(sizeof(T));
  c = first + c < count ? c : count - 1 - first;
  return static_cast<unsigned>(c * static_cast<int>(sizeof(T)) + at % static_cast<int>(sizeof(T)));
}

// The workgroup `bid` of `nwg` of one product.
// DW: operand rows that are not on 16-byte boundaries (odd lengths), loaded as dwords:
// four instructions of 256 bytes (two rows) in the place of one of 1 KB, to the same
// LDS image.  Against the register-staged kernel that such rows took before: o=75 v=225
// float64 X 57.5 -> 52.2 ms, Y 165 -> 155; o=41 v=201 float32 occupied terms 29.4 -> 24.7.
template <class Tr, int EPI, int BM, int BN, bool DW>
__device__ __forceinline__ void kc_direct_body(GemmArgs<typename Tr::T> g, const int bid,
                                               const int nwg) {
  static_assert(EPI == EPI_ACC || EPI == EPI_PAIR || EPI == EPI_PART || EPI == EPI_PM ||
                    EPI == EPI_FOLD,
                "K-contiguous epilogues");
  static_assert(BM == kDBM || BM == 64 || (BM == 160 && !Tr::kDrain), "tile heights");
  using T = typename Tr::T;
  using Acc = typename Tr::Acc;
  using Chunk = typename Tr::Chunk;
  constexpr int CH = Tr::CH;                 // elements per 16 bytes
  constexpr int BK = kDRow / sizeof(T);      // K per step (16 float64 / 32 float32)
  constexpr int MI = BM / 32;                // row blocks per wave (2 wave rows)
  constexpr int NJ = BN / 64;                // column blocks per wave (4 wave columns)
  constexpr int A_BYTES = BM * kDRow;        // 8, 16 or 20 KB
  constexpr int B_BYTES = BN * kDRow;        // 8, 16 or 32 KB
  constexpr int STAGE = A_BYTES + B_BYTES;
  constexpr int A_SLABS = BM / 8, JA = (A_SLABS + 7) / 8;  // 8-row slabs of A; per wave at most JA
  static_assert(kDStages * STAGE <= 160 * 1024, "LDS");
  __shared__ __attribute__((aligned(1024))) unsigned char lds[kDStages * STAGE];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave >> 2) * (BM / 2);
  const int wn = (wave & 3) * (16 * NJ);
  // slabs this wave loads per stage: A slabs wave + 8j < A_SLABS, and NJ of B
  // (a compile-time count when the A slabs split evenly over the 8 waves)
  constexpr bool A_EVEN = A_SLABS % 8 == 0;
  static_assert(A_EVEN || !DW, "dword loads");
  const int LOADS = (A_EVEN ? A_SLABS / 8 + NJ : (A_SLABS - wave + 7) / 8 + NJ) * (DW ? 4 : 1);
  int tm, tn;
  const int nk_all = (g.K + BK - 1) / BK;
  int ks0 = 0, ks1 = nk_all;  // K-steps of this workgroup
  if (EPI == EPI_PART) {
    // grid = tiles x splits; the split is the outer index of the linear id
    const int ntiles = g.tiles_m * g.tiles_n;
    const int id = xcd_linear(bid, nwg);
    const int split = id / ntiles;
    tile_from_linear(id - split * ntiles, ntiles, g.tiles_m, g.group_m, tm, tn);
    ks0 = split * g.split_steps;
    ks1 = ks0 + g.split_steps < nk_all ? ks0 + g.split_steps : nk_all;
    g.C = static_cast<double*>(g.C) + split * g.part_stride;
  } else if (g.kband) {
    tile_of_banded(g.kband, bid, nwg, g.tiles_m, g.group_m, tm, tn);
  } else {
    tile_of(bid, nwg, g.tiles_m, g.group_m, tm, tn);
  }
  const int m0 = tm * BM, n0 = tn * BN;
  if (EPI != EPI_PART && g.kband) k_band(g, n0, BK, ks0, ks1);

  // Slabs: A rows 8*(wave + 8*j), j < JA; B rows 8*(wave + 8*j), j < NJ.  The
  // swizzle of a lane depends on the slab's parity only (slab origin 8*s rows).
  const int lrow = lane >> 3;
  const int sw_even = ((lane & 7) ^ ((lane >> 4) & 7)) * CH;        // slab index even
  const int sw_odd = ((lane & 7) ^ ((4 + (lane >> 4)) & 7)) * CH;   // slab index odd
  const int my_sw = (wave & 1) ? sw_odd : sw_even;  // slabs wave + 8j share the wave's parity
  const T* pa[JA];
  const T* pb[NJ];
  auto row_a = [&](int j) {
    const int row = m0 + 8 * (wave + 8 * j) + lrow;
    return g.A + (long long)(row < g.M ? row : g.M - 1) * g.lda + my_sw;
  };
  auto row_b = [&](int j) {
    const int row = n0 + 8 * (wave + 8 * j) + lrow;
    return g.B + (long long)(row < g.N ? row : g.N - 1) * g.ldb + my_sw;
  };
  unsigned cq[4];
  const unsigned hi_a = (lane >> 5) * static_cast<unsigned>(g.lda * sizeof(T));
  const unsigned hi_b = (lane >> 5) * static_cast<unsigned>(g.ldb * sizeof(T));
  const char* base_a = reinterpret_cast<const char*>(g.A + (long long)m0 * g.lda);
  const char* base_b = reinterpret_cast<const char*>(g.B + (long long)n0 * g.ldb);
  if constexpr (DW) {
#pragma unroll
    for (int q = 0; q < 4; ++q) cq[q] = d_dword_at(lane, wave, q);
  } else {
#pragma unroll
    for (int j = 0; j < JA; ++j) pa[j] = row_a(j);
#pragma unroll
    for (int j = 0; j < NJ; ++j) pb[j] = row_b(j);
  }
  constexpr bool kSpread = d_spread<T, DW>();
  auto issue_dw = [&](int kt, int q) {
    unsigned char* st = lds + (kt % kDStages) * STAGE;
    const int ko = kt * BK;
    const long long kb = (long long)ko * static_cast<int>(sizeof(T));
#pragma unroll
    for (int j = 0; j < JA; ++j)
      d_slab_dword(base_a + kb, 8 * (wave + 8 * j), g.M - 1 - m0,
                    static_cast<int>(g.lda * sizeof(T)), q, cq[q], hi_a,
                    st + 8 * (wave + 8 * j) * kDRow);
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      d_slab_dword(base_b + kb, 8 * (wave + 8 * j), g.N - 1 - n0,
                    static_cast<int>(g.ldb * sizeof(T)), q, cq[q], hi_b,
                    st + A_BYTES + 8 * (wave + 8 * j) * kDRow);
  };
  auto issue = [&](int kt) {
    unsigned char* st = lds + (kt % kDStages) * STAGE;
    const int ko = kt * BK;
    if constexpr (DW) {
#pragma unroll
      for (int q = 0; q < 4; ++q) issue_dw(kt, q);
      return;
    }
#pragma unroll
    for (int j = 0; j < JA; ++j)
      if (A_EVEN || wave + 8 * j < A_SLABS)
        __builtin_amdgcn_global_load_lds((const void*)(pa[j] + ko),
                                         (lds_void*)(st + 8 * (wave + 8 * j) * kDRow), 16, 0, 0);
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      __builtin_amdgcn_global_load_lds((const void*)(pb[j] + ko),
                                       (lds_void*)(st + A_BYTES + 8 * (wave + 8 * j) * kDRow), 16,
                                       0, 0);
  };
  // Ragged last K-step: same LDS image, loaded through registers with zero fill.
  auto issue_tail = [&](int kt) {
    unsigned char* st = lds + (kt % kDStages) * STAGE;
    const int k0 = kt * BK;
    auto one = [&](const T* p, unsigned char* dst) {
      const int kk = k0 + my_sw;  // this lane's first k (p already points my_sw past the row)
      Chunk c;
#pragma unroll
      for (int e = 0; e < CH; ++e) c[e] = (kk + e < g.K) ? p[k0 + e] : T(0);
      *reinterpret_cast<Chunk*>(dst + 16 * lane) = c;
    };
#pragma unroll
    for (int j = 0; j < JA; ++j)
      if (A_EVEN || wave + 8 * j < A_SLABS) one(DW ? row_a(j) : pa[j], st + 8 * (wave + 8 * j) * kDRow);
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      one(DW ? row_b(j) : pb[j], st + A_BYTES + 8 * (wave + 8 * j) * kDRow);
    __builtin_amdgcn_s_waitcnt(0xF | (7 << 4) | (3 << 14));  // lgkmcnt(0): the LDS writes landed
  };

  Acc acc[MI][NJ];
  f64x4 acc64[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      acc[i][j] = Acc{0, 0, 0, 0};
      acc64[i][j] = f64x4{0, 0, 0, 0};
    }

  // fragment: row (lane & 15) of a 16-row block (block origins are multiples
  // of 16, so the row's swizzle is ((lane & 15) >> 1)), logical chunk 4*gi + lane/16
  const int frow = (lane & 15) * kDRow;
  const int fsw = (lane & 15) >> 1;
  const int nk = ks1;        // one past this workgroup's last K-step
  const int nkf = g.K / BK;  // full K-steps; a ragged last one goes through registers
  auto stage_in = [&](int kt) {
    if (kt < nkf)
      issue(kt);
    else
      issue_tail(kt);
  };
  if (ks0 < nk) stage_in(ks0);
  if (ks0 + 1 < nk) stage_in(ks0 + 1);
  for (int k0 = ks0; k0 < nk;) {
    const int kend = (Tr::kDrain && k0 + g.drain_steps < nk) ? k0 + g.drain_steps : nk;
    for (int kt = k0; kt < kend; ++kt) {
      // step kt's direct loads have landed once only step kt+1's remain in flight
      // (a ragged step kt+1 goes through registers and is already complete, and
      // past this workgroup's range nothing more was issued)
      d_wait_vm(kt + 1 < nkf && kt + 1 < nk ? LOADS : 0);
      __builtin_amdgcn_s_barrier();
      const bool dw_next = kSpread && kt + 2 < nk && kt + 2 < nkf;
      if (kt + 2 < nk && !dw_next) stage_in(kt + 2);
      const unsigned char* st = lds + (kt % kDStages) * STAGE;
#pragma unroll
      for (int gi = 0; gi < 2; ++gi) {
        const int chunk = ((4 * gi + (lane >> 4)) ^ fsw) * 16;
        Chunk fa[MI], fb[NJ];
#pragma unroll
        for (int i = 0; i < MI; ++i)
          fa[i] = *reinterpret_cast<const Chunk*>(st + (wm + 16 * i) * kDRow + frow + chunk);
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          fb[j] = *reinterpret_cast<const Chunk*>(st + A_BYTES + (wn + 16 * j) * kDRow + frow + chunk);
#pragma unroll
        for (int e = 0; e < CH; ++e) {
          if (dw_next && e % (CH / 2) == 0) issue_dw(kt + 2, 2 * gi + e / (CH / 2));
#pragma unroll
          for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[i][j] = Tr::mfma(fa[i][e], fb[j][e], acc[i][j]);
        }
      }
    }
    if (Tr::kDrain) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            acc64[i][j][r] += static_cast<double>(acc[i][j][r]);
            acc[i][j][r] = 0;
          }
    }
    k0 = kend;
  }

  const int col = lane & 15;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int n = n0 + wn + 16 * j + col;
    if (n >= g.N) continue;
    const EpiCol ec = epi_col<T, EPI>(g, n);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + wm + 16 * i + Tr::row_of(lane, r);
        if (m >= g.M) continue;
        const double val = Tr::kDrain ? acc64[i][j][r] : static_cast<double>(acc[i][j][r]);
        epi_store<T, EPI>(g, m, n, ec, val);
      }
  }
}

template <class Tr, int EPI, int BM = kDBM, int BN = kDBN, bool DW = false>
__global__ __launch_bounds__(kDThreads, (2 * kc_groups<BM, BN>())) void gemm_kc_direct_kernel(
    GemmArgs<typename Tr::T> g) {
  kc_direct_body<Tr, EPI, BM, BN, DW>(g, blockIdx.x, gridDim.x);
}

// Two products in one launch, workgroups [0, n1) of the first: what the last rounds of
// one leave idle, the other fills.
template <class Tr, int BM, int BN>
__global__ __launch_bounds__(kDThreads, (2 * kc_groups<BM, BN>())) void gemm_kc_two_kernel(
    GemmArgs<typename Tr::T> g, GemmArgs<typename Tr::T> h, int n1) {
  const bool second = static_cast<int>(blockIdx.x) >= n1;
  kc_direct_body<Tr, EPI_PART, BM, BN, false>(second ? h : g, second ? blockIdx.x - n1 : blockIdx.x,
                                       second ? gridDim.x - n1 : n1);
}

}  // namespace ccl

namespace ccl {

// Integral-build GEMM with both operands row-contiguous (RC) and direct
// global->LDS loads (gfx950):
//
//   C = perm( sum_k A[k*lda + m] B[k*ldb + n] )          (EPI_PERM store in the operand type)
//
// Float32 only (float64 builds are faster on the register-staged kernel).
// Same 128 x 256 tile, 8 waves and 3-stage LDS ring as the K-contiguous kernel.
// A stage holds BK rows of k: 128 contiguous m of A and 256 contiguous n of B per
// row, filled 1 KB per wave instruction (lane l writes 16 bytes at +16*l).  An
// MFMA operand needs one value per lane from one k row, so the rows of the 4 x 4
// blocks of a wave are interleaved: block i's row r is wave row 4r + i, making the
// values a lane needs for all four blocks one 16-byte LDS read, the 16 lanes of a k
// row reading 256 contiguous bytes (no bank conflicts, no swizzle).
// Columns are interleaved the same way, which also makes the values a lane stores
// for the four column blocks adjacent in the output: the permuted epilogue writes
// them with 16-byte stores where they do not wrap around a row (dword-aligned: any v;
// o=20 v=130 P=500 float32 forward 4.54 -> 3.84 ms, o=24 v=203 P=777 31.6 -> 28.7 ms
// against element stores where v is no multiple of the chunk).  Needs 16-byte
// aligned operand rows of whole 16-byte chunks (M and N, or readable pads: m_load,
// n_load); rows past M or N are clamped onto the last chunk (never stored); a
// ragged last K-step is loaded through registers with zero fill.
//
// KMAP deals the k of a step to the MFMA slots: 0 four adjacent rows per MFMA; 1 as
// the register-staged kernel does (slot j of MFMA e in a group of 4*CH takes
// CH*j + e), so that operands padded for this kernel keep the sums they had there.
//
// SYM (EPI_PERM, M = N, A = B): the integral (ac|bd) = (bd|ac) of a block that holds
// all virtuals.  Only the tiles that meet n >= m run, on a compact grid, and each
// value is stored at (m, n) and (n, m): half the multiply-adds for the same bytes.
// A lane's 4 x 4 group of adjacent rows and columns makes both stores 16-byte
// vectors.  o=40 v=360 P=1200 float32 forward: 728 -> 573 ms.  (An instantiation of its
// own: as a branch it cost every other build of this kernel 8 to 10 us a tile.)

// Row (column) of the tile that row r of a wave's block i stands for, in this kernel and
// for the columns of the mixed one below: 4r + i (float32) or 32*(i/2) + 2r + (i%2)
// (float64).
template <class Tr>
__device__ __forceinline__ int rc_pos(int i, int r) {
  if constexpr (Tr::CH == 4)
    return 4 * r + i;
  else
    return 32 * (i >> 1) + 2 * r + (i & 1);
}

// Compact grid of the 128 x 256 tiles that meet the diagonal or lie above it:
// tile row t holds tiles_n - t/2 of them, the rows before it
// t*tiles_n - floor((t-1)^2 / 4).
__host__ __device__ inline long long sym_tiles_before(long long t, long long tiles_n) {
  return t * tiles_n - (t - 1) * (t - 1) / 4;
}

__device__ inline void sym_tile(long long id, int tiles_m, int tiles_n, int& tm, int& tn) {
  const double tnd = tiles_n;
  int t = static_cast<int>(2.0 * (tnd - sqrt(tnd * tnd - static_cast<double>(id))));
  t = t < 0 ? 0 : (t >= tiles_m ? tiles_m - 1 : t);
  while (t + 1 < tiles_m && sym_tiles_before(t + 1, tiles_n) <= id) ++t;
  while (t > 0 && sym_tiles_before(t, tiles_n) > id) --t;
  tm = t;
  tn = t / 2 + static_cast<int>(id - sym_tiles_before(t, tiles_n));
}

template <class Tr, int EPI, int KMAP = 0, bool DW = false, bool SYM = false>
__global__ __launch_bounds__(kDThreads, 1) void gemm_rc_direct_kernel(GemmArgs<typename Tr::T> g) {
  static_assert(EPI == EPI_PERM || EPI == EPI_PACK || EPI == EPI_UNPACK || EPI == EPI_SYM,
                "integral-block stores");
  static_assert(Tr::CH == 4 && Tr::kDrain && (!SYM || EPI == EPI_PERM), "float32");
  using T = typename Tr::T;
  using Acc = typename Tr::Acc;
  using Chunk = typename Tr::Chunk;
  constexpr int CH = Tr::CH;
  constexpr int BK = kDRow / sizeof(T);          // 32 k rows per stage
  constexpr int ROWA = kDBM * sizeof(T);         // bytes of one k row of A (128 m)
  constexpr int ROWB = kDBN * sizeof(T);         // bytes of one k row of B (256 n)
  constexpr int A_BYTES = BK * ROWA;             // 16 KB
  constexpr int B_BYTES = BK * ROWB;             // 32 KB
  constexpr int STAGE = A_BYTES + B_BYTES;
  constexpr int AI = A_BYTES / 1024 / 8;         // 1 KB wave instructions per wave: A (2)
  constexpr int BI = B_BYTES / 1024 / 8;         // B (4)
  constexpr int LOADS = (AI + BI) * (DW ? 4 : 1);
  constexpr int CPRA = kDBM / CH;                // 16-byte chunks per A row
  constexpr int CPRB = kDBN / CH;                // per B row
  __shared__ __attribute__((aligned(1024))) unsigned char lds[kDStages * STAGE];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave >> 2) * 64;
  const int wn = (wave & 3) * 64;
  int tm, tn;
  if (EPI == EPI_PACK || EPI == EPI_SYM) {
    // compact grid over the tiles on or above the a = b diagonal
    // (each XCD a contiguous run of them, which shares row panels: o=40 v=360 float64
    // forward 768 -> 764 ms)
    const int id = xcd_linear(blockIdx.x, gridDim.x);
    int lo = 0, hi = g.tiles_m - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (g.row_tiles[mid] <= id) lo = mid; else hi = mid - 1;
    }
    tm = lo;
    tn = pack_first_tile(tm, kDBM, kDBN, g.v) + (id - g.row_tiles[tm]);
  } else if (SYM) {
    sym_tile(xcd_linear(blockIdx.x, gridDim.x), g.tiles_m, g.tiles_n, tm, tn);
  } else {
    tile_of(blockIdx.x, gridDim.x, g.tiles_m, g.group_m, tm, tn);
  }
  const int m0 = tm * kDBM, n0 = tn * kDBN;

  // Wave instruction q of a stage covers bytes [q KB, q KB + 1 KB) of the A (or B)
  // slab: flattened chunk q*64 + lane -> (k row, chunk).  This lane's k row and
  // source pointer at k = 0 for each of its instructions.
  const int ml = g.m_load ? g.m_load : g.M, nl = g.n_load ? g.n_load : g.N;
  const T* pa[AI];
  const T* pb[BI];
  int ra[AI], rb[BI];
#pragma unroll
  for (int j = 0; j < AI; ++j) ra[j] = ((wave + 8 * j) * 64 + lane) / CPRA;
#pragma unroll
  for (int j = 0; j < BI; ++j) rb[j] = ((wave + 8 * j) * 64 + lane) / CPRB;
  // DW: dword loads of rows that are not on 16-byte boundaries, each value's row or
  // column clamped by itself
  unsigned at_a[4], at_b[4];
  if constexpr (DW) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      at_a[q] = d_dword_col<T, ROWA>(lane, wave, q, m0, g.M);
      at_b[q] = d_dword_col<T, ROWB>(lane, wave, q, n0, g.N);
    }
  } else {
#pragma unroll
    for (int j = 0; j < AI; ++j) {
      int m = m0 + (((wave + 8 * j) * 64 + lane) % CPRA) * CH;
      m = m < ml ? m : ml - CH;
      pa[j] = g.A + (long long)ra[j] * g.lda + m;
    }
#pragma unroll
    for (int j = 0; j < BI; ++j) {
      int n = n0 + (((wave + 8 * j) * 64 + lane) % CPRB) * CH;
      n = n < nl ? n : nl - CH;
      pb[j] = g.B + (long long)rb[j] * g.ldb + n;
    }
  }
  auto issue_dw = [&](int kt, int q) {
    unsigned char* st = lds + (kt % kDStages) * STAGE;
    const long long ka = (long long)kt * BK * g.lda, kb = (long long)kt * BK * g.ldb;
    const char* sa = reinterpret_cast<const char*>(g.A + m0 + ka);
    const char* sb = reinterpret_cast<const char*>(g.B + n0 + kb);
#pragma unroll
    for (int j = 0; j < AI; ++j)
      d_piece_dword<ROWA>(sa, wave + 8 * j, static_cast<int>(g.lda * sizeof(T)), q, at_a[q],
                           st + (wave + 8 * j) * 1024);
#pragma unroll
    for (int j = 0; j < BI; ++j)
      d_piece_dword<ROWB>(sb, wave + 8 * j, static_cast<int>(g.ldb * sizeof(T)), q, at_b[q],
                           st + A_BYTES + (wave + 8 * j) * 1024);
  };
  auto issue = [&](int kt) {
    unsigned char* st = lds + (kt % kDStages) * STAGE;
    const long long ka = (long long)kt * BK * g.lda, kb = (long long)kt * BK * g.ldb;
    if constexpr (DW) {
#pragma unroll
      for (int q = 0; q < 4; ++q) issue_dw(kt, q);
      return;
    }
#pragma unroll
    for (int j = 0; j < AI; ++j)
      __builtin_amdgcn_global_load_lds((const void*)(pa[j] + ka),
                                       (lds_void*)(st + (wave + 8 * j) * 1024), 16, 0, 0);
#pragma unroll
    for (int j = 0; j < BI; ++j)
      __builtin_amdgcn_global_load_lds((const void*)(pb[j] + kb),
                                       (lds_void*)(st + A_BYTES + (wave + 8 * j) * 1024), 16, 0, 0);
  };
  // Ragged last K-step: the same LDS image through registers, k rows >= K zero.
  auto issue_tail = [&](int kt) {
    unsigned char* st = lds + (kt % kDStages) * STAGE;
    const int k0 = kt * BK;
    const long long ka = (long long)k0 * g.lda, kb = (long long)k0 * g.ldb;
    if constexpr (DW) {
      auto one = [&](const T* row, int first, int count, bool in) {
        Chunk c;
#pragma unroll
        for (int e = 0; e < CH; ++e) c[e] = in ? row[first + e < count ? first + e : count - 1] : T(0);
        return c;
      };
#pragma unroll
      for (int j = 0; j < AI; ++j)
        *reinterpret_cast<Chunk*>(st + (wave + 8 * j) * 1024 + 16 * lane) =
            one(g.A + (long long)ra[j] * g.lda + ka,
                m0 + (((wave + 8 * j) * 64 + lane) % CPRA) * CH, g.M, k0 + ra[j] < g.K);
#pragma unroll
      for (int j = 0; j < BI; ++j)
        *reinterpret_cast<Chunk*>(st + A_BYTES + (wave + 8 * j) * 1024 + 16 * lane) =
            one(g.B + (long long)rb[j] * g.ldb + kb,
                n0 + (((wave + 8 * j) * 64 + lane) % CPRB) * CH, g.N, k0 + rb[j] < g.K);
      __builtin_amdgcn_s_waitcnt(0xF | (7 << 4) | (3 << 14));  // lgkmcnt(0)
      return;
    }
#pragma unroll
    for (int j = 0; j < AI; ++j) {
      Chunk c = {};
      if (k0 + ra[j] < g.K) c = *reinterpret_cast<const Chunk*>(pa[j] + ka);
      *reinterpret_cast<Chunk*>(st + (wave + 8 * j) * 1024 + 16 * lane) = c;
    }
#pragma unroll
    for (int j = 0; j < BI; ++j) {
      Chunk c = {};
      if (k0 + rb[j] < g.K) c = *reinterpret_cast<const Chunk*>(pb[j] + kb);
      *reinterpret_cast<Chunk*>(st + A_BYTES + (wave + 8 * j) * 1024 + 16 * lane) = c;
    }
    __builtin_amdgcn_s_waitcnt(0xF | (7 << 4) | (3 << 14));  // lgkmcnt(0): the LDS writes landed
  };

  Acc acc[4][4];
  f64x4 acc64[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      acc[i][j] = Acc{0, 0, 0, 0};
      acc64[i][j] = f64x4{0, 0, 0, 0};
    }

  // fragment reads: k row (lane / 16) of each 4-deep MFMA step, wave row/column
  // pos(., lane % 16) of the four blocks
  const int kr = lane >> 4;
  const int r16 = lane & 15;
  const int offa = (wm + 4 * r16) * (int)sizeof(T);
  const int offb = (wn + 4 * r16) * (int)sizeof(T);
  const int nk = (g.K + BK - 1) / BK;
  const int nkf = g.K / BK;
  auto stage_in = [&](int kt) {
    if (kt < nkf)
      issue(kt);
    else
      issue_tail(kt);
  };
  stage_in(0);
  if (nk > 1) stage_in(1);
  for (int k0 = 0; k0 < nk;) {
    const int kend = k0 + g.drain_steps < nk ? k0 + g.drain_steps : nk;
    for (int kt = k0; kt < kend; ++kt) {
      d_wait_vm(kt + 1 < nkf ? LOADS : 0);
      __builtin_amdgcn_s_barrier();
      if (kt + 2 < nk) stage_in(kt + 2);
      const unsigned char* st = lds + (kt % kDStages) * STAGE;
#pragma unroll
      for (int kk = 0; kk < BK / 4; ++kk) {
        const int krow = KMAP ? 4 * CH * (kk / CH) + CH * kr + kk % CH : 4 * kk + kr;
        const unsigned char* ra_ = st + krow * ROWA + offa;
        const unsigned char* rb_ = st + A_BYTES + krow * ROWB + offb;
        const Chunk fa = *reinterpret_cast<const Chunk*>(ra_);
        const Chunk fb = *reinterpret_cast<const Chunk*>(rb_);
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 4; ++j) acc[i][j] = Tr::mfma(fa[i], fb[j], acc[i][j]);
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          acc64[i][j][r] += static_cast<double>(acc[i][j][r]);
          acc[i][j][r] = 0;
        }
    k0 = kend;
  }

  // epilogue: a lane's four column blocks are 4 adjacent n.
  // EPI_PERM: m = (a, x), n = (y, d) -> C[(a*(N/v) + y)*ldv + x*v + d];
  // EPI_PACK: m = (a - a0, c), n = (b - a0, d), kept for b >= a, at packed row
  // pair(a, b) - pair(a0, a0): C[row*v^2 + c*v + d];
  // EPI_UNPACK: m = pair(a, b) - pair(a0, a0) (m < m_keep), n = (c, d) ->
  // C[(a - a0)*v^3 + c*v^2 + b*v + d].
  const long long v = g.v;
  // vector stores need dword alignment only, so rows of any length take them
  typedef T ChunkU __attribute__((ext_vector_type(CH), aligned(sizeof(T))));
  T* C = static_cast<T*>(g.C);
  const int nb = n0 + wn + 4 * r16;  // first column
  if (nb >= g.N) return;
  const int yb = nb / g.v, db = nb - yb * g.v;
  auto value = [&](int i, int e, int r) { return static_cast<T>(acc64[i][e][r]); };
  if constexpr (SYM) {
    // 4 adjacent rows m and columns n: the group on or above the diagonal, and its
    // mirror with rows and columns exchanged
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int mb = m0 + wm + 4 * Tr::row_of(lane, r);
      if (mb >= g.M) continue;
      const int ab = mb / g.v, xb = mb - ab * g.v;
      if (mb + CH - 1 <= nb && nb + CH <= g.N && db + CH <= g.v && xb + CH <= g.v) {
        // wholly on or above the diagonal, and in one row of (c, d) either way
        T* up = C + ab * g.lda_v + yb * g.ldv + (long long)xb * v + db;
        T* down = C + yb * g.lda_v + ab * g.ldv + (long long)db * v + xb;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
          ChunkU x, y;
#pragma unroll
          for (int e = 0; e < CH; ++e) {
            x[e] = value(i, e, r);
            y[e] = value(e, i, r);
          }
          *reinterpret_cast<ChunkU*>(up + i * v) = x;
          *reinterpret_cast<ChunkU*>(down + i * v) = y;
        }
      } else {
        // element by element, the indices (a, x) and (y, d) carried along
        int a = ab, x = xb;
#pragma unroll
        for (int i = 0; i < CH; ++i) {
          int y = yb, d = db;
#pragma unroll
          for (int e = 0; e < CH; ++e) {
            const int m = mb + i, n = nb + e;
            if (m < g.M && n < g.N && m <= n) {
              C[a * g.lda_v + y * g.ldv + (long long)x * v + d] = value(i, e, r);
              C[y * g.lda_v + a * g.ldv + (long long)d * v + x] = value(i, e, r);
            }
            if (++d == g.v) { d = 0; ++y; }
          }
          if (++x == g.v) { x = 0; ++a; }
        }
      }
    }
    return;
  }
  auto dst_of = [&](int m, int y, int d) -> long long {  // -1: not stored
    if (EPI == EPI_UNPACK) {
      if (m >= g.m_keep) return -1;
      const long long q = pair_prefix_d(g.a0, v) + m;
      const int a = pair_row(q, g.v);
      const int b = a + static_cast<int>(q - pair_prefix_d(a, v));
      return (long long)(a - g.a0) * v * v * v + (long long)y * v * v + (long long)b * v + d;
    }
    const int a = m / g.v, x = m - a * g.v;
    if (EPI == EPI_PERM) return a * g.lda_v + y * g.ldv + (long long)x * v + d;
    if (y < a) return -1;
    const long long row = pair_prefix_d(g.a0 + a, v) - pair_prefix_d(g.a0, v) + (y - a);
    return row * v * v + (long long)x * v + d;
  };
  const bool one_row = nb + CH <= g.N && db + CH <= g.v;  // the 4 columns share y
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int m = m0 + wm + 4 * Tr::row_of(lane, r) + i;
      if (m >= g.M) continue;
      if constexpr (EPI == EPI_SYM) {
        // the 4 columns, and their mirrors down one column m
        Chunk val;
#pragma unroll
        for (int e = 0; e < CH; ++e) val[e] = value(i, e, r);
        if (g.ldc % CH == 0) {
          *reinterpret_cast<Chunk*>(C + (long long)m * g.ldc + nb) = val;
        } else {
#pragma unroll
          for (int e = 0; e < CH; ++e) C[(long long)m * g.ldc + nb + e] = val[e];
        }
#pragma unroll
        for (int e = 0; e < CH; ++e) C[(long long)(nb + e) * g.ldc + m] = val[e];
      } else if (one_row) {
        const long long o0 = dst_of(m, yb, db);
        if (o0 >= 0) {
          ChunkU x;
#pragma unroll
          for (int e = 0; e < CH; ++e) x[e] = value(i, e, r);
          *reinterpret_cast<ChunkU*>(C + o0) = x;
        }
      } else {
#pragma unroll
        for (int e = 0; e < CH; ++e) {
          if (nb + e >= g.N) continue;
          const int y = (nb + e) / g.v;
          const long long oe = dst_of(m, y, nb + e - y * g.v);
          if (oe >= 0) C[oe] = value(i, e, r);
        }
      }
    }
}

}  // namespace ccl

namespace ccl {

// Mixed-layout GEMM with direct global->LDS loads (gfx950): A K-contiguous, B
// row-contiguous, float64 accumulation into C:
//
//   C[m*ldc + n] += sum_k A[m*lda + k] B[k*ldb + n]        (EPI_ACC, EPI_FOLD or EPI_PM)
//
// (the adjoint's dt and second dL term, the hole-hole ladder's contraction).
// BM x BN tiles: 128 x 256 (2 x 4 waves of 64 x 64); float64 also 64 x 128 (2 x 4
// waves of 32 x 32) and 64 x 64 (4 x 2 waves of 16 x 32), two workgroups per compute
// unit, where the larger tiles would leave compute units idle (pick_tiles).  A is
// staged like the K-contiguous kernel (8-row slabs of 128-byte rows, XOR-swizzled
// chunks), B like the row-contiguous kernel (BK rows of 256 contiguous n, columns
// of a wave's four blocks interleaved).  In MFMA step e of k-group gi, slot j of
// both operands carries k = gi*4*CH + CH*j + e: A's lane reads its CH consecutive
// k once per group, B's lane reads that k row's four (float32) or two-plus-two
// (float64) interleaved columns once per step.  Needs 16-byte aligned rows and whole
// 16-byte chunks of columns (N, or N and readable pads: n_load); rows past M are
// clamped, columns past N clamped onto the last chunk (never stored), a ragged
// last K-step goes through registers with zero fill.
template <class Tr, int EPI = EPI_ACC, int BM = kDBM, int BN = kDBN, bool DW = false>
__global__ __launch_bounds__(kDThreads, (2 * kc_groups<BM, BN>())) void gemm_kr_direct_kernel(
    GemmArgs<typename Tr::T> g) {
  static_assert(EPI == EPI_ACC || EPI == EPI_FOLD || EPI == EPI_PM, "float64 accumulation");
  static_assert((BM == kDBM && BN == kDBN) || (BM == 64 && BN <= 128 && Tr::CH == 2),
                "tiles; the interleave of two column blocks is float64's");
  using T = typename Tr::T;
  using Acc = typename Tr::Acc;
  using Chunk = typename Tr::Chunk;
  constexpr int CH = Tr::CH;
  constexpr int BK = kDRow / sizeof(T);          // 16 float64 / 32 float32
  constexpr int ROWB = BN * sizeof(T);           // bytes of one k row of B
  constexpr int A_BYTES = BM * kDRow;
  constexpr int B_BYTES = BK * ROWB;
  constexpr int STAGE = A_BYTES + B_BYTES;
  constexpr int AL = BM / 8 / 8;                 // A: 8-row slabs per wave
  constexpr int BI = B_BYTES / 1024 / 8;         // B: 1 KB instructions per wave
  constexpr int LOADS = (AL + BI) * (DW ? 4 : 1);
  constexpr int CPRB = BN / CH;                  // 16-byte chunks per B row
  constexpr int WC = BN == 64 ? 2 : 4;           // wave columns
  constexpr int MI = BM / (16 * (8 / WC)), NJ = BN / (16 * WC);  // blocks per wave
  __shared__ __attribute__((aligned(1024))) unsigned char lds[kDStages * STAGE];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave / WC) * (16 * MI);
  const int wn = (wave % WC) * (16 * NJ);
  int tm, tn;
  if (g.kband)
    tile_of_banded(g.kband, blockIdx.x, gridDim.x, g.tiles_m, g.group_m, tm, tn);
  else
    tile_of(blockIdx.x, gridDim.x, g.tiles_m, g.group_m, tm, tn);
  const int m0 = tm * BM, n0 = tn * BN;
  int ks0, ks1;  // this tile's K-steps
  k_band(g, n0, BK, ks0, ks1);

  // A: slabs of 8 rows, lane -> row lane/8, physical chunk lane%8 holding
  // logical chunk (lane%8) ^ ((row/2)%8)
  const int lrow = lane >> 3;
  const int sw_even = ((lane & 7) ^ ((lane >> 4) & 7)) * CH;
  const int sw_odd = ((lane & 7) ^ ((4 + (lane >> 4)) & 7)) * CH;
  const int my_sw = (wave & 1) ? sw_odd : sw_even;
  const T* pa[AL];
  auto row_a = [&](int j) {
    const int row = m0 + 8 * (wave + 8 * j) + lrow;
    return g.A + (long long)(row < g.M ? row : g.M - 1) * g.lda + my_sw;
  };
  // B: wave instruction q covers the 1 KB [q KB, q KB + 1 KB) of the stage's B slab
  const int nl = g.n_load ? g.n_load : g.N;
  const T* pb[BI];
  int rb[BI];
#pragma unroll
  for (int j = 0; j < BI; ++j) rb[j] = ((wave + 8 * j) * 64 + lane) / CPRB;
  // DW: dword loads of rows that are not on 16-byte boundaries, each value's column
  // clamped by itself
  unsigned cq[4], at_b[4];
  const unsigned hi_a = (lane >> 5) * static_cast<unsigned>(g.lda * sizeof(T));
  const char* base_a = reinterpret_cast<const char*>(g.A + (long long)m0 * g.lda);
  if constexpr (DW) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      cq[q] = d_dword_at(lane, wave, q);
      at_b[q] = d_dword_col<T, ROWB>(lane, wave, q, n0, g.N);
    }
  } else {
#pragma unroll
    for (int j = 0; j < AL; ++j) pa[j] = row_a(j);
#pragma unroll
    for (int j = 0; j < BI; ++j) {
      int n = n0 + (((wave + 8 * j) * 64 + lane) % CPRB) * CH;
      n = n < nl ? n : nl - CH;
      pb[j] = g.B + (long long)rb[j] * g.ldb + n;
    }
  }
  constexpr bool kSpread = d_spread<T, DW>();
  auto issue_dw = [&](int kt, int q) {
    unsigned char* st = lds + (kt % kDStages) * STAGE;
    const int ko = kt * BK;
    const long long kb = (long long)ko * g.ldb;
    const char* sb = reinterpret_cast<const char*>(g.B + n0 + kb);
#pragma unroll
    for (int j = 0; j < AL; ++j)
      d_slab_dword(base_a + (long long)ko * static_cast<int>(sizeof(T)), 8 * (wave + 8 * j),
                    g.M - 1 - m0, static_cast<int>(g.lda * sizeof(T)), q, cq[q], hi_a,
                    st + 8 * (wave + 8 * j) * kDRow);
#pragma unroll
    for (int j = 0; j < BI; ++j)
      d_piece_dword<ROWB>(sb, wave + 8 * j, static_cast<int>(g.ldb * sizeof(T)), q, at_b[q],
                           st + A_BYTES + (wave + 8 * j) * 1024);
  };
  auto issue = [&](int kt) {
    unsigned char* st = lds + (kt % kDStages) * STAGE;
    const int ko = kt * BK;
    const long long kb = (long long)ko * g.ldb;
    if constexpr (DW) {
#pragma unroll
      for (int q = 0; q < 4; ++q) issue_dw(kt, q);
      return;
    }
#pragma unroll
    for (int j = 0; j < AL; ++j)
      __builtin_amdgcn_global_load_lds((const void*)(pa[j] + ko),
                                       (lds_void*)(st + 8 * (wave + 8 * j) * kDRow), 16, 0, 0);
#pragma unroll
    for (int j = 0; j < BI; ++j)
      __builtin_amdgcn_global_load_lds((const void*)(pb[j] + kb),
                                       (lds_void*)(st + A_BYTES + (wave + 8 * j) * 1024), 16, 0, 0);
  };
  auto issue_tail = [&](int kt) {
    unsigned char* st = lds + (kt % kDStages) * STAGE;
    const int k0 = kt * BK;
#pragma unroll
    for (int j = 0; j < AL; ++j) {
      const int kk = k0 + my_sw;  // this lane's first k
      Chunk c;
#pragma unroll
      for (int e = 0; e < CH; ++e) c[e] = (kk + e < g.K) ? (DW ? row_a(j) : pa[j])[k0 + e] : T(0);
      *reinterpret_cast<Chunk*>(st + 8 * (wave + 8 * j) * kDRow + 16 * lane) = c;
    }
    const long long kb = (long long)k0 * g.ldb;
#pragma unroll
    for (int j = 0; j < BI; ++j) {
      Chunk c = {};
      if (DW) {
        const int nc = n0 + (((wave + 8 * j) * 64 + lane) % CPRB) * CH;
        const T* row = g.B + kb + (long long)rb[j] * g.ldb;
#pragma unroll
        for (int e = 0; e < CH; ++e)
          c[e] = k0 + rb[j] < g.K ? row[nc + e < g.N ? nc + e : g.N - 1] : T(0);
      } else if (k0 + rb[j] < g.K) {
        c = *reinterpret_cast<const Chunk*>(pb[j] + kb);
      }
      *reinterpret_cast<Chunk*>(st + A_BYTES + (wave + 8 * j) * 1024 + 16 * lane) = c;
    }
    __builtin_amdgcn_s_waitcnt(0xF | (7 << 4) | (3 << 14));  // lgkmcnt(0): the LDS writes landed
  };

  Acc acc[MI][NJ];
  f64x4 acc64[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      acc[i][j] = Acc{0, 0, 0, 0};
      acc64[i][j] = f64x4{0, 0, 0, 0};
    }

  const int frow = (lane & 15) * kDRow;
  const int fsw = (lane & 15) >> 1;
  const int slot = lane >> 4;
  const int r16 = lane & 15;
  const int offb = (wn + (CH == 4 ? 4 * r16 : 2 * r16)) * (int)sizeof(T);
  const int nk = ks1;
  const int nkf = g.K / BK;
  auto stage_in = [&](int kt) {
    if (kt < nkf)
      issue(kt);
    else
      issue_tail(kt);
  };
  stage_in(ks0);
  if (ks0 + 1 < nk) stage_in(ks0 + 1);
  for (int k0 = ks0; k0 < nk;) {
    const int kend = (Tr::kDrain && k0 + g.drain_steps < nk) ? k0 + g.drain_steps : nk;
    for (int kt = k0; kt < kend; ++kt) {
      // step kt's direct loads have landed once only step kt+1's remain in flight
      d_wait_vm(kt + 1 < nkf && kt + 1 < nk ? LOADS : 0);
      __builtin_amdgcn_s_barrier();
      const bool dw_next = kSpread && kt + 2 < nk && kt + 2 < nkf;
      if (kt + 2 < nk && !dw_next) stage_in(kt + 2);
      const unsigned char* st = lds + (kt % kDStages) * STAGE;
#pragma unroll
      for (int gi = 0; gi < 2; ++gi) {
        const int chunk = ((4 * gi + slot) ^ fsw) * 16;
        Chunk fa[MI];
#pragma unroll
        for (int i = 0; i < MI; ++i)
          fa[i] = *reinterpret_cast<const Chunk*>(st + (wm + 16 * i) * kDRow + frow + chunk);
#pragma unroll
        for (int e = 0; e < CH; ++e) {
          if (dw_next && e % (CH / 2) == 0) issue_dw(kt + 2, 2 * gi + e / (CH / 2));
          // k row gi*4*CH + CH*slot + e of B, this lane's interleaved columns
          const unsigned char* rb_ = st + A_BYTES + (4 * CH * gi + CH * slot + e) * ROWB + offb;
          T fb[NJ];
#pragma unroll
          for (int h = 0; h < NJ / CH; ++h) {
            const Chunk b = *reinterpret_cast<const Chunk*>(rb_ + h * 32 * sizeof(T));
#pragma unroll
            for (int q = 0; q < CH; ++q) fb[CH * h + q] = b[q];
          }
#pragma unroll
          for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NJ; ++j) acc[i][j] = Tr::mfma(fa[i][e], fb[j], acc[i][j]);
        }
      }
    }
    if (Tr::kDrain) {
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            acc64[i][j][r] += static_cast<double>(acc[i][j][r]);
            acc[i][j][r] = 0;
          }
    }
    k0 = kend;
  }

#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int n = n0 + wn + rc_pos<Tr>(j, r16);
    if (n >= g.N) continue;
    const EpiCol ec = epi_col<T, EPI>(g, n);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int m = m0 + wm + 16 * i + Tr::row_of(lane, r);
        if (m >= g.M) continue;
        epi_store<T, EPI>(g, m, n, ec,
                          Tr::kDrain ? acc64[i][j][r] : static_cast<double>(acc[i][j][r]));
      }
  }
}

}  // namespace ccl
