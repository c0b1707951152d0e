// The tile product shared by the contraction and the batched kernels: a square tile of C = P Q^T by four waves,
// one operand an axis operator in fragment order, the other a field.  FP32 and FP64.
//
// What bounds it is MFMA issue, as long as nothing else stalls a wave, so the loop holds little else:
//   - the operator comes straight into the MFMA registers, one 16-byte (FP64: 32-byte) run per lane and 16 x 16
//     block, from L2 / L1 (fragment order, DevOperator::frag); no LDS, no address arithmetic;
//   - the field goes through LDS as [line][k] with a row stride of 128 + 16 bytes, which spreads the 16-byte fragment reads and
//     writes and the single values of a contiguous field over the banks (counters: conflicts are a third of the LDS cycles of a
//     contraction, which are 5-8% of its time);
//   - loads past the end of a line or of the field are clamped to its last value (the outputs of such lines are not
//     stored, and the k past a line's end are cleared on their way to LDS: the operator is zero there, but a
//     non-finite value times zero would not be);
//   - one barrier per slice of 128 bytes of k: slice s + 1 is written while slice s is multiplied, the loads of
//     s + 2 are in flight.
// FP32 products are summed on the MFMA for one chunk (16 k), and FL chunks (1 or 2) are added to FP64 registers at a time:
// a long FP32 sum of the cancelling terms of a spectral derivative loses more than the rounding of operator and
// state together.  The FP64 adds of FL = 1 take issue slots of other waves' MFMAs (161 x 200 x 129: 180 us per step with
// FL = 2, 190 with FL = 1; held back one chunk, to issue among its own wave's MFMAs, they cost 16 more registers and no less time).
//
// MFMA v_mfma_{f32,f64}_16x16x4: lane l supplies P[l%16][l/16] and Q[l%16][l/16] and receives C[4*(l/16)+r][l%16]
// (f32) or C[4*r+l/16][l%16] (f64) in register r (measured on gfx950).  A lane holds the k 4 e + l / 16, e < 4, of a
// 16-wide chunk as one vector and feeds component e to the e-th of four MFMAs, which so contracts the consecutive k
// 4 e .. 4 e + 3: neighbouring entries of a derivative operator alternate in sign, and sums over every fourth one (a lane
// holding four consecutive k) would cancel only later, at a larger rounding error.  LDS lines hold each chunk in that
// order: position p has k = chunk_k(p).
#pragma once

#include <type_traits>

#include "common.h"

namespace pstd {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <typename T> struct Mma;
template <> struct Mma<float> {
  typedef f32x4 v4;
  static __device__ __forceinline__ v4 mma(float a, float b, v4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
  }
  // row of register r in lane l: lane_row(l) + reg_row(r)
  static __device__ __forceinline__ int lane_row(int lane) { return 4 * (lane >> 4); }
  static constexpr __device__ __forceinline__ int reg_row(int r) { return r; }
  static __device__ __forceinline__ int row(int lane, int r) { return lane_row(lane) + reg_row(r); }
};
template <> struct Mma<double> {
  typedef f64x4 v4;
  static __device__ __forceinline__ v4 mma(double a, double b, v4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
  }
  static __device__ __forceinline__ int lane_row(int lane) { return lane >> 4; }
  static constexpr __device__ __forceinline__ int reg_row(int r) { return 4 * r; }
  static __device__ __forceinline__ int row(int lane, int r) { return lane_row(lane) + reg_row(r); }
};

// One value at a wave-uniform address plus a 32-bit byte offset of the lane: the address arithmetic of a loop then runs
// on the scalar unit, not on the vector one that the products' flushes need.
template <typename T>
__device__ __forceinline__ T ld_at(const T* base, uint32_t off) {
  return *reinterpret_cast<const T*>(reinterpret_cast<const char*>(base) + off);
}
// k of position p (0 .. 15) of a chunk in fragment order, and the other way round
constexpr __host__ __device__ __forceinline__ int chunk_k(int p) { return ((p & 3) << 2) | (p >> 2); }
__device__ __forceinline__ int wave_index() { return __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); }

// Block b of n runs on XCD b % 8: the tile (in the order of the grid) that gives each XCD a run of consecutive
// ones, whose operator rows and field lines then meet in one L2.
__device__ __forceinline__ int xcd_tile(int b, int n) {
  const int x = b & 7, q = n >> 3, r = n & 7;
  return x * q + min(x, r) + (b >> 3);
}

// A tile of edge 32 MT: four waves of (16 MT) x (16 MT) outputs, MT x MT MFMA blocks each.  FL: chunks of an FP32 sum.
template <typename T, int MT, int FL>
struct Tile {
  static_assert(FL == 1 || FL == 2, "chunks of an FP32 sum");
  typedef typename Mma<T>::v4 v4;
  static constexpr int E = 32 * MT, NT = 256;
  static constexpr int BK = 128 / static_cast<int>(sizeof(T)), V = 16 / static_cast<int>(sizeof(T));
  static constexpr int LD = BK + V, CH = BK / 16;     // LDS row stride, chunks of a slice
  static constexpr int NX = E * BK / NT;             // field values a thread stages per slice
  static constexpr int NU = NX / V;                   // and 16-byte units of them
  static constexpr size_t lds_values = 2 * E * LD;    // two slices

  // first row and column of this wave's quadrant of the output tile, and where they lie on the operator and the field: ROWS,
  // the field's lines are the rows and the operator's rows the columns; otherwise the other way round
  static __device__ __forceinline__ int row0() { return (wave_index() & 1) * 16 * MT; }
  static __device__ __forceinline__ int col0() { return (wave_index() >> 1) * 16 * MT; }
  template <bool ROWS> static __device__ __forceinline__ int op0() { return ROWS ? col0() : row0(); }
  template <bool ROWS> static __device__ __forceinline__ int line0() { return ROWS ? row0() : col0(); }

  // The field operand: lines 0 .. E - 1 of the tile, of which `lines` exist.  ROWS: line l is the row at x + l * ld, k
  // contiguous; otherwise value (l, k) lies at x + off + k * ld with off this thread's line offset in bytes.  A thread
  // stages NX values of a slice: ROWS, one k of NX lines; otherwise NU units of V k of one line (E = 64: the k of a unit are
  // the same for the whole wave).
  template <bool ROWS>
  struct Field {
    const T* x;      // wave-uniform
    int64_t ld;
    int K;
    uint32_t off[ROWS ? NX : 1];
    static __device__ __forceinline__ int line(int i) {
      return ROWS ? static_cast<int>(threadIdx.x) / BK + i * (NT / BK) : static_cast<int>(threadIdx.x) % E;
    }
    // ROWS: the lines past `lines` read the last one
    __device__ __forceinline__ void set_rows(int lines) {
#pragma unroll
      for (int i = 0; i < NX; ++i)
        off[i] = static_cast<uint32_t>(sizeof(T)) * static_cast<uint32_t>(min(line(i), lines - 1)) * static_cast<uint32_t>(ld);
    }
    // the k this thread stages of a slice (ROWS), or k of value e of its unit i, and the LDS position of that unit
    static __device__ __forceinline__ int row_k() { return static_cast<int>(threadIdx.x) % BK; }
    static __device__ __forceinline__ int unit_pos(int i) {
      const int g = E == 64 ? wave_index() : static_cast<int>(threadIdx.x) / E;
      return V * (g + i * (NT / E));
    }
    static __device__ __forceinline__ int unit_k(int i, int e) {
      const int p = unit_pos(i) + e;
      return (p & ~15) + chunk_k(p & 15);
    }
    __device__ __forceinline__ void load(int s, T (&v)[NX]) const {
      if constexpr (ROWS) {
        const uint32_t k = static_cast<uint32_t>(sizeof(T)) * static_cast<uint32_t>(max(min(row_k(), K - 1 - s * BK), 0));
        const T* p = x + min(s * BK, K - 1);
#pragma unroll
        for (int i = 0; i < NX; ++i) v[i] = ld_at(p, off[i] + k);
      } else {
#pragma unroll
        for (int i = 0; i < NU; ++i)
#pragma unroll
          for (int e = 0; e < V; ++e) v[i * V + e] = ld_at(x + min(s * BK + unit_k(i, e), K - 1) * ld, off[0]);
      }
    }
    // MASK: the slice may hold k past the line's end
    template <bool MASK>
    __device__ __forceinline__ void store(int s, T* lds, const T (&v)[NX]) const {
      typedef T vec __attribute__((ext_vector_type(V)));
      if constexpr (ROWS) {
        const bool in = !MASK || s * BK + row_k() < K;
        const int p = (row_k() & ~15) + chunk_k(row_k() & 15);
#pragma unroll
        for (int i = 0; i < NX; ++i) lds[line(i) * LD + p] = in ? v[i] : T(0);
      } else {
#pragma unroll
        for (int i = 0; i < NU; ++i) {
          vec w;
#pragma unroll
          for (int e = 0; e < V; ++e) w[e] = !MASK || s * BK + unit_k(i, e) < K ? v[i * V + e] : T(0);
          *reinterpret_cast<vec*>(lds + line(0) * LD + unit_pos(i)) = w;
        }
      }
    }
  };

  // acc += this wave's blocks of P Q^T over K (nothing where idle: a wave whose outputs all lie outside only stages).  ROWS: P the field's lines, Q the operator's rows; otherwise P the operator
  // and Q the field.  op: fragments of the operator rows the tile needs, a row block of 16 every op_block values.
  // before_last() runs before the products of the last slice (loads for the epilogue: nothing else is in flight then).
  template <bool ROWS, typename F>
  static __device__ __forceinline__ void contract(const T* op, int64_t op_block, const Field<ROWS>& X, T* lds, bool idle,
                                                  double (&acc)[MT][MT][4], F&& before_last) {
    const int lane = threadIdx.x & 63;
    const int nsl = (X.K + BK - 1) / BK, nch = (X.K + 15) / 16;
    const T* a0 = op + op0<ROWS>() / 16 * op_block;
    const uint32_t al = static_cast<uint32_t>(4 * sizeof(T)) * static_cast<uint32_t>(lane);
    const T* xs = lds + (line0<ROWS>() + (lane & 15)) * LD + 4 * (lane >> 4);   // this lane's fragment in buffer 0
    v4 A[CH][MT];
    T xr[NX];
    auto load_op = [&](int c, int ch) {
#pragma unroll
      for (int m = 0; m < MT; ++m)
        A[c][m] = *reinterpret_cast<const v4*>(
            reinterpret_cast<const char*>(a0 + m * op_block + static_cast<int64_t>(min(ch, nch - 1)) * 256) + al);
    };
    {
      T x0[NX];
      X.load(0, x0);
#pragma unroll
      for (int c = 0; c < CH; ++c) load_op(c, c);
      X.load(1, xr);
      lds_barrier();   // the buffers' previous user is done
      X.template store<true>(0, lds, x0);
      lds_barrier();
    }
    constexpr bool kEach = sizeof(T) == 4 && FL == 1;   // every chunk's sum goes to the accumulators by itself
    auto add = [&](const v4 (&c)[MT][MT]) {
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[i][j][r] += static_cast<double>(c[i][j][r]);
    };
    auto slice = [&](int s, auto last) {
      constexpr bool kLast = decltype(last)::value;
      const int buf = (s & 1) * (E * LD);
      if constexpr (kLast) {
        before_last();
      } else {
        if (s + 2 < nsl) X.template store<false>(s + 1, lds + (E * LD - buf), xr);
        else X.template store<true>(s + 1, lds + (E * LD - buf), xr);
        X.load(s + 2, xr);
      }
      v4 part[MT][MT];   // the slice's sum (FP64: the accumulators themselves; kEach: unused)
#pragma unroll
      for (int c = 0; c < CH; ++c) {
        if (kLast && s * CH + c >= nch) break;
        v4 x[MT], c4[MT][MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) x[m] = *reinterpret_cast<const v4*>(xs + buf + 16 * m * LD + 16 * c);
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) c4[i][j][r] = sizeof(T) == 8 ? static_cast<T>(acc[i][j][r]) : T(0);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < MT; ++j)
              c4[i][j] = ROWS ? Mma<T>::mma(x[i][e], A[c][j][e], c4[i][j]) : Mma<T>::mma(A[c][i][e], x[j][e], c4[i][j]);
        if constexpr (!kLast) load_op(c, (s + 1) * CH + c);
        if constexpr (kEach) {
          add(c4);
        } else {
#pragma unroll
          for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int j = 0; j < MT; ++j)
#pragma unroll
              for (int r = 0; r < 4; ++r) part[i][j][r] = c == 0 ? c4[i][j][r] : part[i][j][r] + c4[i][j][r];
        }
      }
      if constexpr (sizeof(T) == 8) {
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
          for (int j = 0; j < MT; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[i][j][r] = static_cast<double>(part[i][j][r]);
      } else if constexpr (!kEach) {
        add(part);
      }
      if constexpr (!kLast) lds_barrier();
    };
    if (idle) {   // a loop of its own: a test inside the products' loop costs every wave its schedule
      for (int s = 0; s + 1 < nsl; ++s) {
        X.template store<true>(s + 1, lds + (1 - (s & 1)) * (E * LD), xr);
        X.load(s + 2, xr);
        lds_barrier();
      }
      return;
    }
    for (int s = 0; s + 1 < nsl; ++s) slice(s, std::false_type{});
    slice(nsl - 1, std::true_type{});
  }
};

}  // namespace pstd
