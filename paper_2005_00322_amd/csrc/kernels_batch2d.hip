// Batched 2D solver: many independent 2D boxes of different sizes stepped together.
//
// Every solve advances with Eq. (dtt_pstd_solution) in its 2D form (§4.3).  A step is two launches: the velocity
// tiles of every solve, then the pressure tiles of every solve (each p tile takes both axes' terms); the steps replay from
// captured HIP graphs, 1.6 us between launches.  Output tiles are 32 x 32 or 64 x 64, chosen per batch by the
// autotuner.  Each XCD (blocks of index b run on XCD b mod 8) has a run of the tiles, solve after solve and of equal
// cost, so a solve's operator rows and field strips meet in one L2; within a run the tiles come longest
// contraction first or in order.  (One persistent launch for all steps, with tile tickets per XCD and a grid
// barrier after each phase, spent 170 us per phase on them.)  us per step, that launch with its own tile product and
// now, tiles 64: two solves of 304 x 304 231 -> 36 (tiles 32: 288 -> 22), 32 of them 384 -> 119, 256 uneven ones of
// 96 .. 512 a side 1623 -> 923 (72 TFLOP/s).
//
// Operators are unscaled (dx = 1) FP32 matrices shared by all solves with the same (n, boundary pair);
// each solve's constants -dt/(rho0 dx) and -dt rho0 c0^2/dx are applied in the FP64 epilogue.  The tile product is
// tile_core.h's (a pressure tile runs it once per axis into the same accumulators); three (64-wide tiles) or more blocks per CU keep
// the matrix cores busy while others stage, load or wait.
#include <algorithm>

#include "tile_core.h"

namespace pstd {

namespace {

constexpr int NT = 256;

// FP32 sums of 16 k in 32-wide tiles and of 32 k in 64-wide ones
template <int MT> using BatchTile = Tile<float, MT, MT>;

// PH 0: a velocity tile (T.kind 0 or 1), PH 1: a pressure tile (T.kind 2).
template <int MT, int PH>
__device__ __forceinline__ void run_task(const BatchSolve& S, const BatchTask& T, float* lds) {
  typedef BatchTile<MT> TL;
  const int lane = threadIdx.x & 63;
  const int nx = S.nx, ny = S.ny, i0 = T.i0, j0 = T.j0;
  float* const Y = PH == 1 ? S.p : T.kind == 0 ? S.ux : S.uy;
  const int rows = PH == 0 && T.kind == 0 ? nx - 1 : nx, cols = PH == 0 && T.kind == 1 ? ny - 1 : ny;
  const bool idle = i0 + TL::row0() >= rows || j0 + TL::col0() >= cols;
  // this lane's outputs: rows from r0 + lane_row on, one column per block j (offset in bytes, ~0 outside)
  const int r0 = i0 + TL::row0(), lr = Mma<float>::lane_row(lane), rows_left = rows - r0 - lr;
  uint32_t coff[MT];
#pragma unroll
  for (int j = 0; j < MT; ++j) {
    const int c = j0 + TL::col0() + 16 * j + (lane & 15);
    coff[j] = c < cols ? 4u * static_cast<uint32_t>(lr * cols + c) : ~0u;
  }
  auto valid = [&](int i, int j, int r) { return coff[j] != ~0u && 16 * i + Mma<float>::reg_row(r) < rows_left; };
  auto at = [&](int i, int r) { return (r0 + 16 * i + Mma<float>::reg_row(r)) * cols; };
  float yv[MT][MT][4], cv[MT][MT][4];
  const float* const c2 = PH == 1 ? S.c2 : nullptr;   // pressure tiles of a heterogeneous solve take c0(x)^2 pointwise
  auto load_old = [&] {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < MT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (valid(i, j, r)) yv[i][j][r] = ld_at(Y + at(i, r), coff[j]);
  };
  double acc[MT][MT][4] = {};
  // column contraction: operator rows i0 .. along x, field columns j0 ..; row contraction: field rows i0 .., operator j0 ..
  auto columns = [&](const float* op, int ld_op, const float* X, int K, auto&& before_last) {
    typename TL::template Field<false> f;
    f.x = X + j0;
    f.ld = ny;
    f.K = K;
    f.off[0] = 4u * static_cast<uint32_t>(min(f.line(0), ny - 1 - j0));
    TL::template contract<false>(op + static_cast<int64_t>(i0) * ld_op, 16 * static_cast<int64_t>(ld_op), f, lds, idle, acc,
                                 before_last);
  };
  auto lines = [&](const float* op, int ld_op, const float* X, int K, auto&& before_last) {
    typename TL::template Field<true> f;
    f.x = X + static_cast<int64_t>(i0) * K;
    f.ld = K;
    f.K = K;
    f.set_rows(nx - i0);
    TL::template contract<true>(op + static_cast<int64_t>(j0) * ld_op, 16 * static_cast<int64_t>(ld_op), f, lds, idle, acc,
                                before_last);
  };
  if constexpr (PH == 1) {
    // p[i][j] += sD * (sum_k Dx[i][k] u_x[k][j] + sum_k u_y[i][k] Dy[j][k])
    columns(S.fDx, S.lddx, S.ux, nx - 1, [] {});
    lines(S.fDy, S.lddy, S.uy, ny - 1, load_old);
  } else if (T.kind == 0) {
    // u_x[i][j] += sG * sum_k Gx[i][k] p[k][j]
    columns(S.fGx, S.ldgx, S.p, nx, load_old);
  } else {
    // u_y[i][j] += sG * sum_k p[i][k] Gy[j][k]
    lines(S.fGy, S.ldgy, S.p, ny, load_old);
  }
  if (idle) return;
  if (c2) {
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < MT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (valid(i, j, r)) cv[i][j][r] = ld_at(c2 + at(i, r), coff[j]);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < MT; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[i][j][r] *= static_cast<double>(cv[i][j][r]);
  }
  const double scale = PH == 1 ? S.sD : S.sG;
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < MT; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (valid(i, j, r))
          *reinterpret_cast<float*>(reinterpret_cast<char*>(Y + at(i, r)) + coff[j]) =
              static_cast<float>(fma(scale, acc[i][j][r], static_cast<double>(yv[i][j][r])));
}

// One phase: slot b takes tile b / 8 of the run of XCD b % 8; a block has one slot, or with a limit on the blocks (LIMIT, `slots` in
// all) every gridDim.x-th.  64-wide tiles at three blocks per CU: a fourth costs 38 spilled registers (256 uneven solves
// 1028 against 923 us per step).
template <int TILE, int PH, bool LIMIT>
__global__ __launch_bounds__(NT, TILE == 64 ? 3 : 6) void batch2d_kernel(const BatchSolve* __restrict__ solves,
                                                        const BatchTask* __restrict__ tasks, BatchRuns runs, int slots) {
  __shared__ __attribute__((aligned(16))) float lds[BatchTile<TILE / 32>::lds_values];
  for (int b = blockIdx.x; b < (LIMIT ? slots : static_cast<int>(gridDim.x)); b += gridDim.x) {
    const int q = b % kBatchQueues, t = runs.beg[q] + b / kBatchQueues;
    if (t < runs.beg[q + 1]) {
      const BatchTask T = tasks[t];
      run_task<TILE / 32, PH>(solves[T.solve], T, lds);
    }
    if (!LIMIT) break;
  }
}

// What of a solve changes between steps: the caller's states and maps.
struct BatchState {
  float *p, *ux, *uy;
  const float* c2;
  double sD;
};
constexpr int kMaxStates = 96;   // 40 bytes each, within a launch's 4 KB of arguments
struct StateArgs {
  BatchState s[kMaxStates];
};

__global__ __launch_bounds__(128) void batch_states_kernel(StateArgs a, int count, BatchSolve* table) {
  const int i = threadIdx.x;
  if (i >= count) return;
  table[i].p = a.s[i].p;
  table[i].ux = a.s[i].ux;
  table[i].uy = a.s[i].uy;
  table[i].c2 = a.s[i].c2;
  table[i].sD = a.s[i].sD;
}

template <int TILE, int PH>
void launch_t(const BatchSolve* solves, const BatchTask* tasks, const BatchRuns& runs, int slots, int blocks, hipStream_t s) {
  if (blocks > 0 && blocks < slots)
    hipLaunchKernelGGL((batch2d_kernel<TILE, PH, true>), dim3(blocks), dim3(NT), 0, s, solves, tasks, runs, slots);
  else
    hipLaunchKernelGGL((batch2d_kernel<TILE, PH, false>), dim3(slots), dim3(NT), 0, s, solves, tasks, runs, slots);
}

}  // namespace

hipError_t launch_batch_states(const BatchSolve* solves, int count, BatchSolve* table, hipStream_t s) {
  for (int i = 0; i < count; i += kMaxStates) {
    StateArgs a{};
    const int n = std::min(count - i, kMaxStates);
    for (int k = 0; k < n; ++k) a.s[k] = BatchState{solves[i + k].p, solves[i + k].ux, solves[i + k].uy, solves[i + k].c2, solves[i + k].sD};
    hipLaunchKernelGGL(batch_states_kernel, dim3(1), dim3(128), 0, s, a, n, table + i);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_batch2d(int phase, const BatchSolve* solves, const BatchTask* tasks, const BatchRuns& runs, int tile,
                          int blocks, hipStream_t s) {
  int most = 0;
  for (int q = 0; q < kBatchQueues; ++q) most = std::max(most, runs.beg[q + 1] - runs.beg[q]);
  if (most < 1 || most > 0x7fffffff / kBatchQueues / 2 || (tile != 32 && tile != 64)) return hipErrorInvalidValue;
  const int slots = most * kBatchQueues;
  if (tile == 64 && phase == 0) launch_t<64, 0>(solves, tasks, runs, slots, blocks, s);
  else if (tile == 64) launch_t<64, 1>(solves, tasks, runs, slots, blocks, s);
  else if (phase == 0) launch_t<32, 0>(solves, tasks, runs, slots, blocks, s);
  else launch_t<32, 1>(solves, tasks, runs, slots, blocks, s);
  return hipGetLastError();
}

}  // namespace pstd
