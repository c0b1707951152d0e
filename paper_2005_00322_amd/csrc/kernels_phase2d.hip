// Two fused phase kernels per step for 2D plans (FP32 and FP64).
//
// Eq. (dtt_pstd_solution) in its 2D form (§4.3) splits into a velocity phase and a pressure phase:
//   velocity  u_x += G~x p   and   u_y += p G~y^T           (one launch)
//   pressure  p += c2 .* (D~x u_x + u_y D~y^T)               (one launch)
// Each block owns one square output tile of the phase: in the velocity phase the u_x and the u_y tile at
// the same (i, j) position, in the pressure phase one p tile with both axes' terms.  Both phases are thus
// two contractions of the same shape,
//   contraction 0:  out0[i][j] = sum_k A0[i][k] X0[k][j]   (operator rows, columns of a field)
//   contraction 1:  out1[i][j] = sum_k X1[i][k] A1[j][k]   (rows of a field, operator rows)
// and the eight waves of a block split them as (contraction, quarter of the k chunks of 16).
//
// A box of a few hundred nodes a side is bound by latency, not by bandwidth or MFMA rate.  As the waves of a block
// split k and each computes the whole tile, no operand element is used by two waves, so nothing is shared before
// the partial tiles meet in LDS:
//   operators  are kept in fragment order (DevOperator::frag): the 16 rows x 16 k that one wave feeds to four MFMAs are
//              one run of 64 lanes x 4 values, loaded straight into the MFMA registers;
//   X0         16 lanes read 16 neighbouring columns of a row, straight into the registers;
//   X1         rows are read with neighbouring lanes along k (one value a lane: rows of odd length start at any
//              value, and 16-byte loads off their alignment cost more than they save) and turned into fragments
//              through a strip of LDS that belongs to the wave (no block barrier).
// Loaded as fragments, each quad of lanes would touch four rows, four cache lines for 64 bytes.
// Loads run NR rounds of RC chunks ahead; the kernel boundary between the phases is the grid-wide dependency of the
// scheme, and graph replay keeps the launch gaps short.
//
// Tile edge 16 MT.  A block reads 2 x 16 MT operand rows for (16 MT)^2 outputs, so at MT = 1 the operands'
// path into the CU (64 bytes per clock) is exactly as busy as the matrix cores and at MT = 2 half as busy, but MT = 2
// has a quarter of the blocks: the rule is at tile_edge().
//
// A lane's four values of a 16-wide chunk feed four MFMAs, k order and layouts as in tile_core.h.  FP32 sums are of 4 (MT = 1) or
// 8 k and are added in FP64 (50 steps of 16 boxes of 256 x 256: 1.99 ms, with sums of 32 k 1.81), the waves' shares and the
// contractions too, and the update is rounded once.
#include <algorithm>

#include "tile_core.h"

namespace pstd {
namespace {

typedef double f64x2 __attribute__((ext_vector_type(2)));
typedef __amdgpu_buffer_rsrc_t rsrc_t;

constexpr int NT = 512;                 // eight waves
constexpr uint32_t kOOB = 0x80000000u;  // buffer offset past every range: the load returns zero

// mx, my: staggered points along x and y, n - 1 between two walls and n on a periodic axis
template <typename T>
struct Phase2DArgs {
  const T* Gx; int ldgx, mgx;   // mx x nx operator in fragment order, ldgx columns, mgx rows (zero padded)
  const T* Gy; int ldgy, mgy;   // my x ny
  const T* Dx; int lddx, mdx;   // nx x mx
  const T* Dy; int lddy, mdy;   // ny x my
  T* p;                         // nx x ny
  T* ux;                        // mx x ny
  T* uy;                        // nx x my
  const T* c2;                  // nx x ny or null
  int nx, ny, mx, my;
  double sv, sp;                // velocity / pressure factors on the contractions (1 for folded operators)
  bool fresh;                   // velocity phase: the fields' old values do not count (and are dropped)
};

__device__ __forceinline__ rsrc_t make_rsrc(const void* ptr, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(ptr), 0, static_cast<int>(bytes), 0x00020000);
}
__device__ __forceinline__ void ld1(float& v, rsrc_t r, uint32_t o) {
  v = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, o, 0, 0));
}
__device__ __forceinline__ void ld1(double& v, rsrc_t r, uint32_t o) {
  v = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, o, 0, 0));
}
__device__ __forceinline__ void ld4(f32x4& v, rsrc_t r, uint32_t o) {
  v = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(r, o, 0, 0));
}
__device__ __forceinline__ void ld4(f64x4& v, rsrc_t r, uint32_t o) {
  const f64x2 a = __builtin_bit_cast(f64x2, __builtin_amdgcn_raw_buffer_load_b128(r, o, 0, 0));
  const f64x2 b = __builtin_bit_cast(f64x2, __builtin_amdgcn_raw_buffer_load_b128(r, o + 16, 0, 0));
  v = f64x4{a[0], a[1], b[0], b[1]};
}

// 0, or the bit that takes a byte offset (below 2^31) out of every range.  Arithmetic on purpose: a uniform condition
// written as a choice between two offsets becomes a branch with the load on either side and a wait in each.
__device__ __forceinline__ uint32_t oob_unless(bool in) { return (static_cast<uint32_t>(in) - 1u) & kOOB; }

__host__ __device__ __forceinline__ int pad64(int k) { return (k + 63) & ~63; }

// Tile shapes: RC chunks of 16 k per round.  NR: rounds in flight (a second one spills at four waves per SIMD).
template <typename T, int MT, int RC>
struct Shape {
  static constexpr int NR = 1;
  static constexpr int RL = 16 * RC;                           // lanes along a row
  static constexpr int RI = 16 * MT * RL / 64;                 // loads of a round (64 / RL rows each)
  static constexpr int V = 16 / static_cast<int>(sizeof(T));   // values of a 16-byte LDS read
  static constexpr int LD = 16 * RC + V;                       // LDS row stride: those reads without bank conflicts
  static constexpr size_t strip = sizeof(T) * 16 * MT * LD;    // LDS of one wave's rows
};

// This wave's share of one contraction: acc[a][b] (the MT x MT sub-tiles) += sum over its chunks of P Q^T.
// C = 0: P the operator rows i0 .., Q the columns j0 .. of the field X (row stride ldx);
// C = 1: P the rows i0 .. of X, Q the operator rows j0 ...  K: contracted length, h: the wave's quarter of it.
// The operator is zero for k >= K, up to pad64(K); X's rows k >= K lie past its end and read as zero, and the
// elements of a row past K would be the next row's, so they are not read (a NaN there would not vanish).
template <typename T, int MT, int RC, int C>
__device__ __forceinline__ void contract_share(rsrc_t rA, int lda, rsrc_t rX, int ldx, int i0, int j0, int K, int h,
                                               T* strip, double (&acc)[MT][MT][4]) {
  typedef typename Mma<T>::v4 v4;
  typedef T vec __attribute__((ext_vector_type(16 / sizeof(T))));
  typedef Shape<T, MT, RC> S;
  constexpr int NR = S::NR, V = S::V, RL = S::RL, RI = S::RI, LD = S::LD;
  constexpr uint32_t ES = sizeof(T);
  constexpr bool kFlush = sizeof(T) == 4;
  const int lane = threadIdx.x & 63, lr = lane & 15, lk = 4 * (lane >> 4);   // lk: the lane's place in a chunk
  const int nit = pad64(K) / 64;            // chunks of a wave
  const int c0 = h * nit;                   // its first
  v4 A[NR][RC][MT], X0[C == 0 ? NR : 1][RC][MT];
  T X1[C == 1 ? NR : 1][RI];
  const int r0 = (C == 0 ? i0 : j0) >> 4, nc = lda >> 4;
  // in the order of use, kept by the scheduler barriers: the first products start while later chunks are on their way
  auto load = [&](int slot, int rd) {
    if constexpr (C == 1) {
      const int k = 16 * (c0 + rd * RC) + lane % RL;
      const uint32_t past = oob_unless(k < min(16 * (c0 + nit), K));
#pragma unroll
      for (int i = 0; i < RI; ++i) {
        const int r = i0 + i * (64 / RL) + lane / RL;
        ld1(X1[slot][i], rX, past | ES * static_cast<uint32_t>(r * ldx + k));
      }
    }
#pragma unroll
    for (int q = 0; q < RC; ++q) {
      const int it = rd * RC + q, ch = c0 + it;
      const uint32_t past = oob_unless(it < nit);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int a = 0; a < MT; ++a) {
        ld4(A[slot][q][a], rA, past | ES * static_cast<uint32_t>(((r0 + a) * nc + ch) * 256 + 4 * lane));
        if constexpr (C == 0) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            T v;
            ld1(v, rX, past | ES * static_cast<uint32_t>((16 * ch + 4 * e + (lane >> 4)) * ldx + j0 + 16 * a + lr));
            X0[slot][q][a][e] = v;
          }
        }
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  v4 c[MT][MT];
  const v4 zero = {0, 0, 0, 0};
#pragma unroll
  for (int a = 0; a < MT; ++a)
#pragma unroll
    for (int b = 0; b < MT; ++b) c[a][b] = zero;
#pragma unroll
  for (int s = 0; s < NR; ++s) load(s, s);
  const int nrd = (nit + RC - 1) / RC;
  for (int rd = 0; rd < nrd; rd += NR) {
#pragma unroll
    for (int s = 0; s < NR; ++s) {
      if (rd + s >= nrd) break;
      if constexpr (C == 1) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");   // the last round's reads come first
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int i = 0; i < RI; ++i)
          strip[(i * (64 / RL) + lane / RL) * LD + (lane % RL & ~15) + chunk_k(lane & 15)] = X1[s][i];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local");
        __builtin_amdgcn_wave_barrier();
      }
#pragma unroll
      for (int q = 0; q < RC; ++q) {
        if ((rd + s) * RC + q >= nit) break;
        v4 X[MT];
#pragma unroll
        for (int a = 0; a < MT; ++a) {
          if constexpr (C == 0) {
            X[a] = X0[s][q][a];
          } else {
#pragma unroll
            for (int e = 0; e < 4; e += V) {
              const vec v = *reinterpret_cast<const vec*>(strip + (16 * a + lr) * LD + 16 * q + lk + e);
#pragma unroll
              for (int f = 0; f < V; ++f) X[a][e + f] = v[f];
            }
          }
        }
        if constexpr (MT == 1) {
          // one tile: four independent products, so none waits for the one before it
          v4 m[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) m[e] = C == 0 ? Mma<T>::mma(A[s][q][0][e], X[0][e], zero)
                                                    : Mma<T>::mma(X[0][e], A[s][q][0][e], zero);
#pragma unroll
          for (int r = 0; r < 4; ++r)
            acc[0][0][r] += (static_cast<double>(m[0][r]) + static_cast<double>(m[1][r])) +
                            (static_cast<double>(m[2][r]) + static_cast<double>(m[3][r]));
        } else {
#pragma unroll
          for (int a = 0; a < MT; ++a)
#pragma unroll
            for (int b = 0; b < MT; ++b) {
              auto mm = [&](int e, v4 c0) {
                return C == 0 ? Mma<T>::mma(A[s][q][a][e], X[b][e], c0) : Mma<T>::mma(X[a][e], A[s][q][b][e], c0);
              };
              if constexpr (kFlush) {
                const v4 h0 = mm(1, mm(0, zero)), h1 = mm(3, mm(2, zero));
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[a][b][r] += static_cast<double>(h0[r]) + static_cast<double>(h1[r]);
              } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) c[a][b] = mm(e, c[a][b]);
              }
            }
        }
      }
      if (rd + s + NR < nrd) load(s, rd + s + NR);
    }
  }
  if constexpr (MT > 1 && !kFlush) {
#pragma unroll
    for (int a = 0; a < MT; ++a)
#pragma unroll
      for (int b = 0; b < MT; ++b)
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[a][b][r] += static_cast<double>(c[a][b][r]);
  }
}

// PH 0: velocity phase, PH 1: pressure phase.  tile: index of the block's tile.
template <typename T, int MT, int RC, int PH>
__device__ __forceinline__ void phase2d_body(const Phase2DArgs<T>& a, int tile) {
  constexpr int E = 16 * MT, G = MT * MT * 4;   // tile edge, register groups of a tile (64 values each)
  constexpr uint32_t ES = sizeof(T);
  // the partial tiles of the eight waves; before that the row strips of waves 4 .. 7
  constexpr size_t kRed = sizeof(double) * 8 * G * 64, kStrips = 4 * Shape<T, MT, RC>::strip;
  __shared__ __attribute__((aligned(16))) unsigned char lds[kRed > kStrips ? kRed : kStrips];
  double (*red)[G][64] = reinterpret_cast<double (*)[G][64]>(lds);
  const int nx = a.nx, ny = a.ny, mx = a.mx, my = a.my;
  const int tiles_y = (ny + E - 1) / E;
  const int i0 = (tile / tiles_y) * E, j0 = (tile % tiles_y) * E;
  // the wave index through readfirstlane keeps per-wave buffer descriptors in scalar registers
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);

  // this wave's share of the epilogue: velocity, groups (wave % 4) + 4 g of u_x (wave < 4) or u_y; pressure,
  // groups wave + 8 g of p (for a 16 x 16 tile waves 0 .. 3 have one each).  Old values and c2 are loaded first.
  constexpr int NG = PH == 0 ? G / 4 : (G + 7) / 8;
  const bool ux = wave < 4;
  T* const Y = PH == 1 ? a.p : (ux ? a.ux : a.uy);
  const int rows = PH == 1 ? nx : (ux ? mx : nx), cols = PH == 1 ? ny : (ux ? ny : my);
  const int g0 = PH == 0 ? (wave & 3) : wave, gs = PH == 0 ? 4 : 8;
  const rsrc_t rY = make_rsrc(Y, ES * static_cast<uint32_t>(rows * cols));
  const rsrc_t rC = make_rsrc(a.c2, PH == 1 && a.c2 ? ES * static_cast<uint32_t>(nx * ny) : 0u);   // no map: zeros
  T old[NG], cf[NG];
  int off[NG];   // element offset, -1 outside the field or past the tile's groups
#pragma unroll
  for (int g = 0; g < NG; ++g) {
    const int grp = g0 + gs * g, sub = grp >> 2;
    const int oi = i0 + 16 * (sub / MT) + Mma<T>::row(lane, grp & 3), oj = j0 + 16 * (sub % MT) + (lane & 15);
    off[g] = (grp < G && oi < rows && oj < cols) ? oi * cols + oj : -1;
    const uint32_t o = oob_unless(off[g] >= 0) | ES * static_cast<uint32_t>(off[g]);
    ld1(old[g], rY, o);
    if (PH == 1) ld1(cf[g], rC, o);
  }

  double acc[MT][MT][4] = {};
  if (ux) {
    const T* A = PH == 0 ? a.Gx : a.Dx;
    const int lda = PH == 0 ? a.ldgx : a.lddx, ma = PH == 0 ? a.mgx : a.mdx, K = PH == 0 ? nx : mx;
    contract_share<T, MT, RC, 0>(make_rsrc(A, ES * static_cast<uint32_t>(ma * lda)), lda,
                                    make_rsrc(PH == 0 ? a.p : a.ux, ES * static_cast<uint32_t>(K * ny)), ny, i0, j0, K,
                                    wave, nullptr, acc);
  } else {
    const T* A = PH == 0 ? a.Gy : a.Dy;
    const int lda = PH == 0 ? a.ldgy : a.lddy, ma = PH == 0 ? a.mgy : a.mdy, K = PH == 0 ? ny : my;
    contract_share<T, MT, RC, 1>(make_rsrc(A, ES * static_cast<uint32_t>(ma * lda)), lda,
                                    make_rsrc(PH == 0 ? a.p : a.uy, ES * static_cast<uint32_t>(nx * K)), K, i0, j0, K,
                                    wave - 4, reinterpret_cast<T*>(lds + (wave - 4) * Shape<T, MT, RC>::strip), acc);
  }
  lds_barrier();   // the strips are read
#pragma unroll
  for (int x = 0; x < MT; ++x)
#pragma unroll
    for (int y = 0; y < MT; ++y)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[wave][(x * MT + y) * 4 + r][lane] = acc[x][y][r];
  lds_barrier();

#pragma unroll
  for (int g = 0; g < NG; ++g) {
    const int grp = g0 + gs * g;
    if (off[g] < 0) continue;
    auto part = [&](int w) { return red[w][grp][lane]; };
    const int w0 = PH == 0 && !ux ? 4 : 0;
    double v = (part(w0) + part(w0 + 1)) + (part(w0 + 2) + part(w0 + 3));
    if (PH == 1) v += (part(4) + part(5)) + (part(6) + part(7));
    v *= PH == 0 ? a.sv : a.sp;
    if (PH == 1 && a.c2) v *= static_cast<double>(cf[g]);
    if (PH == 0 && a.fresh) old[g] = T(0);
    Y[off[g]] = static_cast<T>(static_cast<double>(old[g]) + v);
  }
}

template <typename T, int MT, int RC, int PH>
__global__ __launch_bounds__(NT, 4) void phase2d_kernel(Phase2DArgs<T> a) {
  phase2d_body<T, MT, RC, PH>(a, xcd_tile(blockIdx.x, gridDim.x));
}

// One phase of many solves of one shape: tiles solve after solve, the solve's unscaled operators and factors
// from the batch's solve table.  start (velocity phase): u^{-1/2} = -1/2 sG (G p), whatever u holds.
template <int MT, int RC, int PH>
__global__ __launch_bounds__(NT, 4) void phase2d_batch_kernel(const BatchSolve* __restrict__ solves, int tiles,
                                                              bool start) {
  const int t = xcd_tile(blockIdx.x, gridDim.x);
  const BatchSolve& S = solves[t / tiles];
  const Phase2DArgs<float> a{S.fGx, S.ldgx, S.mgx, S.fGy, S.ldgy, S.mgy, S.fDx, S.lddx, S.mdx, S.fDy, S.lddy, S.mdy,
                             S.p, S.ux, S.uy, S.c2, S.nx, S.ny, S.nx - 1, S.ny - 1, start ? -0.5 * S.sG : S.sG, S.sD, start};
  phase2d_body<float, MT, RC, PH>(a, t % tiles);
}

int tiles_of(int nx, int ny, int edge) { return ((nx + edge - 1) / edge) * ((ny + edge - 1) / edge); }

// Tile edge for `count` boxes of nx x ny nodes: 16 while its tiles are at most two per CU (each tile is then little more
// than one round trip to memory), 32 beyond.  us per phase at 16 / 32, FP32 and FP64: 256 x 256 (256 tiles)
// 3.9 / 6.8 and 4.6 / 7.7; 320 x 320 (400) 6.5 / 8.1 and 7.6 / 9.0; 360 x 360 (529) 9.6 / 9.0 and 10.8 / 10.1; 512 x 300 (608)
// 9.8 / 9.2 and 11.4 / 10.3; 512 x 512 (1024) 14.0 / 11.0 and 18.4 / 14.4.
int tile_edge(int nx, int ny, int count) { return static_cast<int64_t>(tiles_of(nx, ny, 16)) * count > 512 ? 32 : 16; }

// Chunks per round: 256 / MT bytes of a row, or half of that where it covers a wave's whole share (chunks past the share
// are still loads, if empty ones: 123 x 123 FP32 3.57 us per phase with four chunks for its two, 3.26 with two).
template <typename T, int MT>
constexpr int round_chunks() { return (sizeof(T) == 4 ? 4 : 2) / MT; }
template <typename T, int MT>
bool half_round(int nx, int ny) { return MT == 1 && pad64(std::max(nx, ny)) / 64 <= round_chunks<T, MT>() / 2; }

template <typename T>
hipError_t launch_one(int which, const Phase2DArgs<T>& a, hipStream_t s) {
  const int edge = tile_edge(a.nx, a.ny, 1);
  const dim3 grid(tiles_of(a.nx, a.ny, edge)), blk(NT);
#define PSTD_PHASE(MT, RC)                                                                      \
  if (which == 0) hipLaunchKernelGGL((phase2d_kernel<T, MT, RC, 0>), grid, blk, 0, s, a);       \
  else hipLaunchKernelGGL((phase2d_kernel<T, MT, RC, 1>), grid, blk, 0, s, a);
  constexpr int RC1 = round_chunks<T, 1>(), RC2 = round_chunks<T, 2>();
  if (edge == 32) { PSTD_PHASE(2, RC2) }
  else if (half_round<T, 1>(a.nx, a.ny)) { PSTD_PHASE(1, RC1 / 2) }
  else { PSTD_PHASE(1, RC1) }
#undef PSTD_PHASE
  return hipGetLastError();
}

template <typename T>
Phase2DArgs<T> make_args(const DevOperator& Gx, const DevOperator& Gy, const DevOperator& Dx, const DevOperator& Dy,
                         void* p, void* ux, void* uy, const void* c2, int nx, int ny) {
  return Phase2DArgs<T>{static_cast<const T*>(Gx.frag), Gx.Kp, Gx.Mp, static_cast<const T*>(Gy.frag), Gy.Kp, Gy.Mp,
                        static_cast<const T*>(Dx.frag), Dx.Kp, Dx.Mp, static_cast<const T*>(Dy.frag), Dy.Kp, Dy.Mp,
                        static_cast<T*>(p), static_cast<T*>(ux), static_cast<T*>(uy), static_cast<const T*>(c2), nx, ny,
                        Gx.M, Gy.M, 1.0, 1.0, false};
}

// Every k < pad64(K) has its chunk of the zero-padded fragments, and rows past the allocation read as zero.  The staggered extent of an axis (the
// rows of G, the columns of D) is n - 1 between walls or n on a periodic axis.
bool operators_fit(const DevOperator& Gx, const DevOperator& Gy, const DevOperator& Dx, const DevOperator& Dy,
                   int nx, int ny) {
  const int mx = Gx.M, my = Gy.M;
  return Gx.frag && Gy.frag && Dx.frag && Dy.frag && Gx.K == nx && Gy.K == ny && Dx.M == nx && Dy.M == ny && Dx.K == mx && Dy.K == my &&
         (mx == nx - 1 || mx == nx) && (my == ny - 1 || my == ny) && Gx.Kp >= pad64(nx) && Gy.Kp >= pad64(ny) &&
         Dx.Kp >= pad64(mx) && Dy.Kp >= pad64(my) && Gx.Kp % 16 == 0 && Gy.Kp % 16 == 0 && Dx.Kp % 16 == 0 &&
         Dy.Kp % 16 == 0;
}

}  // namespace

bool phase2d_supported(int nx, int ny) { return nx >= 3 && ny >= 3 && nx <= 512 && ny <= 512; }

hipError_t launch_phase2d_one(bool dbl, int which, const DevOperator& Gx, const DevOperator& Gy, const DevOperator& Dx,
                              const DevOperator& Dy, void* p, void* ux, void* uy, const void* c2, int nx, int ny,
                              hipStream_t s) {
  if (!phase2d_supported(nx, ny) || !operators_fit(Gx, Gy, Dx, Dy, nx, ny)) return hipErrorInvalidValue;
  return dbl ? launch_one(which, make_args<double>(Gx, Gy, Dx, Dy, p, ux, uy, c2, nx, ny), s)
             : launch_one(which, make_args<float>(Gx, Gy, Dx, Dy, p, ux, uy, c2, nx, ny), s);
}

hipError_t launch_phase2d(bool dbl, const DevOperator& Gx, const DevOperator& Gy, const DevOperator& Dx,
                          const DevOperator& Dy, void* p, void* ux, void* uy, const void* c2, int nx, int ny,
                          int64_t steps, hipStream_t s) {
  for (int64_t t = 0; t < steps; ++t)
    for (int which = 0; which < 2; ++which) {
      const hipError_t e = launch_phase2d_one(dbl, which, Gx, Gy, Dx, Dy, p, ux, uy, c2, nx, ny, s);
      if (e != hipSuccess) return e;
    }
  return hipSuccess;
}

// One phase of `count` solves of one shape from the batch's device solve table (unscaled operators; the
// factors sG, sD and the c0^2 maps of the table apply in the epilogue).  The caller checks that the
// operators' padded rows cover pad64(K) columns (batch2d_phase_fits).
hipError_t launch_phase2d_batch(int which, const BatchSolve* solves, int count, int nx, int ny, bool start,
                                hipStream_t s) {
  if (!phase2d_supported(nx, ny) || count < 1 || count > 65535 || (start && which != 0)) return hipErrorInvalidValue;
  const int edge = tile_edge(nx, ny, count), tiles = tiles_of(nx, ny, edge);
  const dim3 grid(static_cast<unsigned>(tiles) * static_cast<unsigned>(count)), blk(NT);
#define PSTD_PHASE(MT, RC)                                                                                          \
  if (which == 0) hipLaunchKernelGGL((phase2d_batch_kernel<MT, RC, 0>), grid, blk, 0, s, solves, tiles, start);     \
  else hipLaunchKernelGGL((phase2d_batch_kernel<MT, RC, 1>), grid, blk, 0, s, solves, tiles, start);
  if (edge == 32) { PSTD_PHASE(2, 2) }
  else if (half_round<float, 1>(nx, ny)) { PSTD_PHASE(1, 2) }
  else { PSTD_PHASE(1, 4) }
#undef PSTD_PHASE
  return hipGetLastError();
}

namespace {

// Zeroes the Dirichlet wall nodes of every solve's p (block y: solve).
__global__ __launch_bounds__(256) void batch_walls_kernel(const BatchSolve* __restrict__ solves) {
  const BatchSolve& S = solves[blockIdx.y];
  const int nx = S.nx, ny = S.ny, i = blockIdx.x * 256 + threadIdx.x;
  if (i < ny) {
    if (S.walls & 1) S.p[i] = 0.f;
    if (S.walls & 2) S.p[static_cast<int64_t>(nx - 1) * ny + i] = 0.f;
  }
  if (i < nx) {
    if (S.walls & 4) S.p[static_cast<int64_t>(i) * ny] = 0.f;
    if (S.walls & 8) S.p[static_cast<int64_t>(i) * ny + ny - 1] = 0.f;
  }
}

}  // namespace

hipError_t launch_batch_walls(const BatchSolve* solves, int count, int nx, int ny, hipStream_t s) {
  if (count < 1 || count > 65535) return hipErrorInvalidValue;
  hipLaunchKernelGGL(batch_walls_kernel, dim3((std::max(nx, ny) + 255) / 256, count), dim3(256), 0, s, solves);
  return hipGetLastError();
}

bool batch2d_phase_fits(int ldgx, int ldgy, int lddx, int lddy, int nx, int ny) {
  return ldgx >= pad64(nx) && ldgy >= pad64(ny) && lddx >= pad64(nx - 1) && lddy >= pad64(ny - 1) && ldgx % 16 == 0 &&
         ldgy % 16 == 0 && lddx % 16 == 0 && lddy % 16 == 0;
}

}  // namespace pstd
