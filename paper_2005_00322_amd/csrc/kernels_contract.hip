// Dense per-axis contraction on MFMA with the leapfrog update fused into the epilogue (FP32 / FP64).
//
// One call applies an axis operator A (M x K, constants folded in) along one axis of a field X and
// updates the field Y on the other grid in place:  Y = beta * Y + alpha * scale .* (A X).
// This is one half of Eq. (dtt_pstd_solution) for one axis: the forward transform, k-space multiply
// with the sine<->cosine switch and inverse transform collapsed into one matrix, then the
// finite-difference time update.
//
// Two layouts:
//   strided     the contracted axis is not the last one.  X is viewed as [batch][K][C] and Y as
//               [batch][M][C] (C = product of the trailing extents, unit stride):
//               Y[b][m][c] += sum_k A[m][k] X[b][k][c].  The columns (b, c) of all batches are one range, so a tile may
//               span several batches and only the last one is partly empty (C = 129: 1 tile in 25800 / 64 against every third).
//   contiguous  the contracted axis is the last one.  X is [R][K], Y is [R][M]:
//               Y[r][m] += sum_k X[r][k] A[m][k]
// The tile product is tile_core.h's; the columns of its output run along the unit stride of Y in both layouts.
// us per launch before (64 x 64 tiles, 16-deep slices, both operands through LDS, one tile range per batch) and now, axes
// x / y / z: 256^3 FP32 159 / 154 / 196 -> 105 / 105 / 97 (82-89 TFLOP/s of the 150 a large FP32 product reaches here);
// 161 x 200 x 129 FP32 44 / 71 / 36 -> 30 / 38 / 20; 161 x 200 x 129 FP64 63 / 99 / 53 -> 38 / 50 / 27.  Counters at the latter size in
// FP32 with a map: matrix cores 26-38% busy, vector ALU 20-26%, 1.5-1.8 TB/s.  A launch of one axis has about 1250 blocks, four per
// CU and a fifth of a second round.
#include <algorithm>

#include "tile_core.h"

namespace pstd {
namespace {

// FP32 sums of one chunk, 16 k
template <typename T, int MT> using ContractTile = Tile<T, MT, 1>;

template <typename T>
struct KArgs {
  const T* op;          // operator fragments
  int M, K, Kp;
  const T* X;
  T* Y;
  int64_t inner, lines;       // strided: C and batch * C columns; contiguous: rows (inner unused)
  int64_t x_bstride, y_bstride;
  double alpha, beta;
  const T* scale;
  int mtiles;
};

// PLAIN: beta = 1 and no map (the velocity update).
template <typename T, bool ROWS, int MT, bool PLAIN>
__device__ __forceinline__ void contract_tile(const KArgs<T>& a, int tile, T* lds) {
  typedef ContractTile<T, MT> TL;
  const int m0 = (tile % a.mtiles) * TL::E;
  const int64_t l0 = static_cast<int64_t>(tile / a.mtiles) * TL::E;
  constexpr uint32_t ES = sizeof(T);
  const int lane = threadIdx.x & 63;
  typename TL::template Field<ROWS> X;
  X.K = a.K;
  // the first line's batch (strided).  A lane's offsets from there fit 32 bits through the limits on an axis, 4097 nodes along a
  // dense one and 8193 (FP64: 4097) along any: a middle axis has batches of at most 4097 x 8193 values, and a tile's lines
  // span at most two of them or 128 x 4097 values; the first axis is one batch, with rows at most 8193^2 values apart, and a
  // lane's first row is 12 from its wave's at most (FP64: 3 of 4097^2): 3.2 GB.
  const int64_t b0 = ROWS ? 0 : l0 / a.inner, c0 = ROWS ? 0 : l0 - b0 * a.inner;
  auto line_off = [&](int64_t l, int64_t bstride) {   // elements from line l0 to line l0 + l (clamped)
    const int64_t c = c0 + min(l, a.lines - 1 - l0), b = c / a.inner;
    return b * bstride + (c - b * a.inner) - c0;
  };
  if constexpr (ROWS) {
    X.x = a.X + l0 * a.K;
    X.ld = a.K;
    X.set_rows(static_cast<int>(min(a.lines - l0, static_cast<int64_t>(TL::E))));
  } else {
    X.x = a.X + b0 * a.x_bstride + c0;
    X.ld = a.inner;
    X.off[0] = ES * static_cast<uint32_t>(line_off(X.line(0), a.x_bstride));
  }
  // Outputs: value (row, column) of the tile, columns along the unit stride.  A lane's column gives a 32-bit offset, its
  // rows are row_step apart from a wave-uniform start.
  const int64_t row_step = ROWS ? a.M : a.inner;
  const int64_t first = (ROWS ? l0 : m0) + TL::row0();
  const int64_t ybase = first * row_step + (ROWS ? m0 + TL::template op0<ROWS>() : b0 * a.y_bstride + c0);
  const int lr = Mma<T>::lane_row(lane);
  const int rows_left = static_cast<int>(min((ROWS ? a.lines : a.M) - first, static_cast<int64_t>(16 * MT))) - lr;
  uint32_t coff[MT];
#pragma unroll
  for (int j = 0; j < MT; ++j) {
    const int cl = 16 * j + (lane & 15);
    bool ok;
    int64_t o;
    if constexpr (ROWS) {
      ok = m0 + TL::template op0<ROWS>() + cl < a.M;
      o = cl;
    } else {
      ok = l0 + TL::template line0<ROWS>() + cl < a.lines;
      o = line_off(TL::template line0<ROWS>() + cl, a.y_bstride);
    }
    coff[j] = ok ? ES * static_cast<uint32_t>(o + lr * row_step) : ~0u;
  }
  T yv[MT][MT][4];
  double acc[MT][MT][4] = {};
  auto valid = [&](int i, int j, int r) { return coff[j] != ~0u && 16 * i + Mma<T>::reg_row(r) < rows_left; };
  auto at = [&](int i, int r) { return ybase + (16 * i + Mma<T>::reg_row(r)) * row_step; };
  TL::template contract<ROWS>(a.op + static_cast<int64_t>(m0) * a.Kp, 16 * static_cast<int64_t>(a.Kp), X, lds,
                               m0 + TL::template op0<ROWS>() >= a.M || l0 + TL::template line0<ROWS>() >= a.lines, acc, [&] {
    if (!PLAIN && a.beta == 0.0) return;
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < MT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (valid(i, j, r)) yv[i][j][r] = ld_at(a.Y + at(i, r), coff[j]);
  });
  // fused update epilogue: the product, the map factor and the update are formed in FP64 and rounded once
  T sv[MT][MT][4];
  if (!PLAIN && a.scale) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < MT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (valid(i, j, r)) sv[i][j][r] = ld_at(a.scale + at(i, r), coff[j]);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < MT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][j][r] *= static_cast<double>(sv[i][j][r]);
  }
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < MT; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (!valid(i, j, r)) continue;
        const double y0 = static_cast<double>(yv[i][j][r]);
        const double old = PLAIN ? y0 : (a.beta != 0.0 ? a.beta * y0 : 0.0);
        T* y = reinterpret_cast<T*>(reinterpret_cast<char*>(a.Y + at(i, r)) + coff[j]);
        *y = static_cast<T>(fma(a.alpha, acc[i][j][r], old));
      }
}

template <typename T, bool ROWS, int MT>
__global__ __launch_bounds__(256, MT == 2 ? 4 : 6) void contract_kernel(KArgs<T> a) {
  __shared__ __attribute__((aligned(16))) T lds[ContractTile<T, MT>::lds_values];
  contract_tile<T, ROWS, MT, false>(a, xcd_tile(blockIdx.x, gridDim.x), lds);
}

// Up to three contractions (beta = 1, no map) with outputs of their own in one grid (the velocity terms of a step: all read p), so that
// the partly filled last round of blocks comes once instead of once per axis.  tiles[i]: tiles of contraction i; every
// XCD takes its run of each contraction's tiles in turn (xcd_tile; the counts are rounded up to whole rounds of the
// XCDs by blocks that end at once).  161 x 200 x 129 FP32: a step of 184 us with one launch per axis takes 178 (with FP32 sums
// of 32 k; 190 with 16).  Three waves per SIMD for 64-wide tiles: with four the two forms of the tile in one kernel leave no
// register free (192).
template <typename T>
struct MultiArgs {
  KArgs<T> a[3];
  int tiles[3], rows[3], count;
};

template <typename T, int MT>
__global__ __launch_bounds__(256, MT == 2 ? 3 : 6) void contract_multi_kernel(MultiArgs<T> m) {
  __shared__ __attribute__((aligned(16))) T lds[ContractTile<T, MT>::lds_values];
  int b = blockIdx.x;
  for (int i = 0; i < m.count; ++i) {
    const int n = (m.tiles[i] + 7) & ~7;
    if (b >= n) {
      b -= n;
      continue;
    }
    const int tile = xcd_tile(b, n);
    if (tile >= m.tiles[i]) return;
    if (m.rows[i]) contract_tile<T, true, MT, true>(m.a[i], tile, lds);
    else contract_tile<T, false, MT, true>(m.a[i], tile, lds);
    return;
  }
}

template <typename T>
bool make_args(const ContractArgs& c, KArgs<T>* a) {
  if (!c.frag || c.batch < 1 || c.ncols < 1 || c.M < 1 || c.K < 1) return false;
  a->op = static_cast<const T*>(c.frag);
  a->M = c.M;
  a->K = c.K;
  a->Kp = c.lda;
  a->X = static_cast<const T*>(c.X);
  a->Y = static_cast<T*>(c.Y);
  a->inner = c.ncols;
  a->lines = c.ncols * c.batch;
  a->x_bstride = c.x_bstride;
  a->y_bstride = c.y_bstride;
  a->alpha = c.alpha_d;
  a->beta = c.beta_d;
  a->scale = static_cast<const T*>(c.scale);
  return true;
}

template <typename T>
int64_t tiles_of(const KArgs<T>& a, int edge) {
  return ((a.M + edge - 1) / edge) * ((a.lines + edge - 1) / edge);
}

// 64 x 64 tiles from about 400 of them on (1.5 per CU), 32 x 32 before that: four times the blocks, twice the operand
// traffic for a product.  us at 32 / 64, middle axis: 314 tiles (100^3) FP32 9.8 / 12.4, FP64 11.9 / 13.8; 400 (128 x 100^2)
// 11.6 / 12.2 and 14.5 / 13.9; 512 (128^3) 13.6 / 13.3 and 18.0 / 16.2: the sides cross at about 390 tiles in FP64 and 470 in FP32.
constexpr int64_t kBigTiles = 400;

template <typename T>
hipError_t launch_t(const ContractArgs& c, bool contiguous, hipStream_t s) {
  static_assert(kRowPad % 64 == 0 && kColPad % 32 == 0, "operator padding must cover whole tiles and slices");
  KArgs<T> a;
  if (!make_args(c, &a)) return hipErrorInvalidValue;
  const bool big = tiles_of(a, 64) >= kBigTiles;
  const int edge = big ? 64 : 32;
  a.mtiles = (c.M + edge - 1) / edge;
  const int64_t n = tiles_of(a, edge);
  if (n > 0x7fffffff) return hipErrorInvalidConfiguration;
  const dim3 grid(static_cast<unsigned>(n)), blk(256);
  if (big) {
    if (contiguous) hipLaunchKernelGGL((contract_kernel<T, true, 2>), grid, blk, 0, s, a);
    else hipLaunchKernelGGL((contract_kernel<T, false, 2>), grid, blk, 0, s, a);
  } else {
    if (contiguous) hipLaunchKernelGGL((contract_kernel<T, true, 1>), grid, blk, 0, s, a);
    else hipLaunchKernelGGL((contract_kernel<T, false, 1>), grid, blk, 0, s, a);
  }
  return hipGetLastError();
}

template <typename T>
hipError_t launch_multi_t(const ContractArgs* c, const bool* contiguous, int count, hipStream_t s) {
  MultiArgs<T> m{};
  if (count < 1 || count > 3) return hipErrorInvalidValue;
  int order[3] = {0, 1, 2};
  std::sort(order, order + count, [&](int x, int y) { return c[x].K > c[y].K; });   // the longest products first
  int64_t t64 = 0;
  for (int i = 0; i < count; ++i) {
    const ContractArgs& ci = c[order[i]];
    if (!make_args(ci, &m.a[i]) || ci.beta_d != 1.0 || ci.scale) return hipErrorInvalidValue;
    m.rows[i] = contiguous[order[i]];
    t64 += tiles_of(m.a[i], 64);
  }
  m.count = count;
  const bool big = t64 >= kBigTiles;
  const int edge = big ? 64 : 32;
  int64_t n = 0;
  for (int i = 0; i < count; ++i) {
    m.a[i].mtiles = (m.a[i].M + edge - 1) / edge;
    const int64_t t = tiles_of(m.a[i], edge);
    if (t > 0x7ffffff0) return hipErrorInvalidConfiguration;
    m.tiles[i] = static_cast<int>(t);
    n += round_up(t, 8);
  }
  if (n > 0x7fffffff) return hipErrorInvalidConfiguration;
  const dim3 grid(static_cast<unsigned>(n)), blk(256);
  if (big) hipLaunchKernelGGL((contract_multi_kernel<T, 2>), grid, blk, 0, s, m);
  else hipLaunchKernelGGL((contract_multi_kernel<T, 1>), grid, blk, 0, s, m);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_contract_fp32(const ContractArgs& c, bool contiguous, hipStream_t s) {
  return launch_t<float>(c, contiguous, s);
}

hipError_t launch_contract_fp64(const ContractArgs& c, bool contiguous, hipStream_t s) {
  return launch_t<double>(c, contiguous, s);
}

hipError_t launch_contract_multi(bool dbl, const ContractArgs* c, const bool* contiguous, int count, hipStream_t s) {
  return dbl ? launch_multi_t<double>(c, contiguous, count, s) : launch_multi_t<float>(c, contiguous, count, s);
}

}  // namespace pstd
