// Split-bfloat16 per-axis contraction with the operator in MFMA fragment order (FP32 state).
//
// Y = beta*Y + alpha*scale.*(A X) along one axis, the product formed as A_hi X_hi + A_hi X_lo + A_lo X_hi with bfloat16
// operands and FP32 accumulation: A = A_hi + A_lo is split on the host, X = X_hi + X_lo while a slice of it is staged into
// LDS.  The dropped A_lo X_lo term is below 2^-16 of the product.
//
// A launch has to move the field once and the output twice through HBM; the matrix cores need about 40% of that time, and what
// costs more is a poor overlap of the two (one block of eight waves per CU, K loop and update one after the other, the
// operator through LDS: 184-195 us a launch at 384^3, 75-84 at 260^3, 13-15 at 128^3, 16-18 for a 256 x 256 plane).  Here
// (173-190, 50-51, 6.8-7.8 and 8-10):
//   - the four waves of a block split the operator's rows, so no two of them need the same operator fragment: it
//     comes straight from L2 into the MFMA registers (16 bytes per lane, runs of 1 KB, one chunk of 16 k ahead) and
//     nothing of it passes through LDS or the vector ALU;
//   - a block takes all rows (up to 384) of 64 field lines, so the field is read once and its 8 KB of hi and lo parts per
//     slice of 32 k are all that LDS holds (two slices); three blocks fit a CU, and some load, stage or update
//     while another multiplies;
//   - addresses advance on the scalar unit (buffer accesses: the lane's offset stays, the k or row step is the scalar
//     offset, and an out-of-range offset drops the access, so no load or store sits behind a branch).
//
// MFMA v_mfma_f32_32x32x16_bf16: lane l supplies P[l%32][8*(l/32) .. +7] and Q[l%32][8*(l/32) .. +7] and receives
// C[8*(r/4) + 4*(l/32) + r%4][l%32] in register r.  Output columns follow the lane, so the operand whose rows are unit-stride
// in Y is Q: strided layout P = operator rows, Q = field lines; contiguous layout P = field lines, Q = operator rows.
#include <algorithm>

#include "tile_core.h"

namespace pstd {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// LDS row stride in bf16: 80 bytes.  16-byte accesses of a strided field are free of conflicts; the stores of contiguous rows
// are not (a quarter of the LDS cycles, 1.5% of the time).
constexpr int NT = 256, BK = 32, LD = BK + 8;
constexpr int JL = 2, LINES = kSplitLines;         // field lines of a block
static_assert(LINES == 32 * JL && NT == 64 * kSplitWaves, "block shape");
constexpr int PART = LINES * LD;                   // hi or lo part of a slice

typedef __amdgpu_buffer_rsrc_t rsrc_t;
constexpr uint32_t kOOB = 0x80000000u;   // byte offset past every field (all below 2 GiB)

__device__ __forceinline__ rsrc_t make_rsrc(const void* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, static_cast<int>(bytes), 0x00020000);
}
__device__ __forceinline__ float ld_f32(rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, soff, 0));
}

struct FArgs {
  const __bf16* op;        // fragments: [32 rows][16 k][hi, lo][lane][8]
  int M, K, nch;           // nch: chunks of 16 k in the padded operator
  const float* X;
  float* Y;
  int64_t inner, lines, x_bstride, y_bstride;
  float alpha, beta;
  const float* scale;
  int mtiles, rb;          // operator row tiles and row blocks (of 32 rows)
};

// FMODE: 0 strided lines; 1 contiguous rows, lanes along k; 2 contiguous rows, 16-byte loads (aligned, K a multiple of 4).
template <int FMODE>
struct Stage {
  rsrc_t x;                // the whole field
  uint32_t ld;             // strided: bytes from k to k + 1
  int K;
  uint32_t off[FMODE == 1 ? 8 : 1];   // byte offsets of this thread's lines
  float v[8];

  __device__ __forceinline__ void load(int s) {
    const int k0 = s * BK;
    if constexpr (FMODE == 0) {
      const int g = k0 + 8 * wave_index();
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = ld_f32(x, off[0], static_cast<uint32_t>(min(g + j, K - 1)) * ld);
    } else if constexpr (FMODE == 1) {
      const uint32_t k = 4u * static_cast<uint32_t>(max(min(static_cast<int>(threadIdx.x) % 32, K - 1 - k0), 0));
#pragma unroll
      for (int j = 0; j < 8; ++j) v[j] = ld_f32(x, off[j] + k, 4u * static_cast<uint32_t>(min(k0, K - 1)));
    } else {
      // groups of 8 k; a half past the row's end repeats the row's last four values (cleared in store)
      const int g = 8 * (static_cast<int>(threadIdx.x) % 4);
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const uint32_t k = 4u * static_cast<uint32_t>(min(k0 + g + 4 * h, K - 4));
        const f32x4 w = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(x, off[0] + k, 0, 0));
#pragma unroll
        for (int j = 0; j < 4; ++j) v[4 * h + j] = w[j];
      }
    }
  }

  // split into bf16 hi and lo, to LDS [line][k] (hi part, then lo); MASK: the slice may hold k past the lines' end
  template <bool MASK>
  __device__ __forceinline__ void store(int s, __bf16* lds) {
    const int t = threadIdx.x, k0 = s * BK;
    if constexpr (FMODE == 1) {
      // lanes 2m and 2m+1 hold neighbouring k of one line: both form the pair, the even lane stores its hi parts, the odd
      // lane its lo parts, each as one dword
      const int k = t % 32;
      const bool in = !MASK || k0 + k < K, odd = (k & 1) != 0;
      __bf16* dst = lds + (odd ? PART : 0) + (k & ~1);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float a = in ? v[j] : 0.f;
        const float b = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, a), 0xB1, 0xF, 0xF, false));
        const float e = odd ? b : a, o = odd ? a : b;
        const __bf16 he = static_cast<__bf16>(e), ho = static_cast<__bf16>(o);
        const __bf16 pe = odd ? static_cast<__bf16>(e - static_cast<float>(he)) : he;
        const __bf16 po = odd ? static_cast<__bf16>(o - static_cast<float>(ho)) : ho;
        *reinterpret_cast<uint32_t*>(dst + (t / 32 + 8 * j) * LD) =
            static_cast<uint32_t>(__builtin_bit_cast(uint16_t, pe)) | (static_cast<uint32_t>(__builtin_bit_cast(uint16_t, po)) << 16);
      }
    } else {
      const int line = FMODE == 0 ? t % LINES : t / 4, g = 8 * (FMODE == 0 ? wave_index() : t % 4);
      bf16x8 h, l;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float a = !MASK || k0 + g + j < K ? v[j] : 0.f;
        h[j] = static_cast<__bf16>(a);
        l[j] = static_cast<__bf16>(a - static_cast<float>(h[j]));
      }
      *reinterpret_cast<bf16x8*>(lds + line * LD + g) = h;
      *reinterpret_cast<bf16x8*>(lds + PART + line * LD + g) = l;
    }
  }
};

// The whole contraction of a wave with NW row blocks (row blocks wave, wave + 4, .. of the tile).
template <int FMODE, int NW>
__device__ __forceinline__ void run_wave(const FArgs& a, Stage<FMODE>& X, __bf16* lds, int rb0, int64_t l0) {
  constexpr bool CONTIG = FMODE != 0;
  constexpr int NB = NW > 0 ? NW : 1;
  const int lane = threadIdx.x & 63, wave = wave_index();
  const int nsl = (a.K + BK - 1) / BK, nck = (a.K + 15) / 16;
  f32x16 acc[NB][JL];
#pragma unroll
  for (int i = 0; i < NB; ++i)
#pragma unroll
    for (int j = 0; j < JL; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
  bf16x8 A[2][NB][2];
  const uint32_t al = 16u * static_cast<uint32_t>(lane);
  auto load_op = [&](int set, int ch) {
    if constexpr (NW > 0) {
#pragma unroll
      for (int i = 0; i < NW; ++i) {
        const __bf16* p = a.op + (static_cast<int64_t>(rb0 + wave + 4 * i) * a.nch + min(ch, nck - 1)) * 1024;
#pragma unroll
        for (int n = 0; n < 2; ++n) {
          const int q = CONTIG ? n : 1 - n;   // in the order of their first use (the other order: 4-13% slower)
          A[set][i][q] = *reinterpret_cast<const bf16x8*>(reinterpret_cast<const char*>(p + 512 * q) + al);
        }
      }
    }
  };
  load_op(0, 0);
  const __bf16* xs = lds + (lane & 31) * LD + 8 * (lane >> 5);
  for (int s = 0; s < nsl; ++s) {
    const int buf = (s & 1) * 2 * PART;
    if (s + 2 < nsl) {
      X.template store<false>(s + 1, lds + (2 * PART - buf));
      X.load(s + 2);
    } else if (s + 1 < nsl) {
      X.template store<true>(s + 1, lds + (2 * PART - buf));
    }
    if constexpr (NW > 0) {
#pragma unroll
      for (int c = 0; c < 2; ++c) {
        load_op(1 - c, 2 * s + c + 1);
        bf16x8 x[JL][2];
#pragma unroll
        for (int j = 0; j < JL; ++j)
#pragma unroll
          for (int q = 0; q < 2; ++q) x[j][q] = *reinterpret_cast<const bf16x8*>(xs + buf + q * PART + 32 * j * LD + 16 * c);
        // lo hi, hi lo, hi hi (of the ports P and Q): the products of one kind together, so none waits for the one before it
#pragma unroll
        for (int p = 0; p < 3; ++p)
#pragma unroll
          for (int i = 0; i < NW; ++i)
#pragma unroll
            for (int j = 0; j < JL; ++j) {
              const bf16x8 o = A[c][i][p == (CONTIG ? 1 : 0)], f = x[j][p == (CONTIG ? 0 : 1)];
              acc[i][j] = CONTIG ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(f, o, acc[i][j], 0, 0, 0)
                                 : __builtin_amdgcn_mfma_f32_32x32x16_bf16(o, f, acc[i][j], 0, 0, 0);
            }
      }
    }
    lds_barrier();
  }
  if constexpr (NW > 0) {
    // Update: value (row, column) of a block, columns (lanes) along the unit stride of Y, rows row_step apart.
    const int lr = 4 * (lane >> 5), lc = lane & 31;
    const uint32_t bytes = static_cast<uint32_t>(4 * a.lines * a.M);
    const rsrc_t rY = make_rsrc(a.Y, bytes), rS = make_rsrc(a.scale, a.scale ? bytes : 0u);
    const uint32_t row_step = 4u * static_cast<uint32_t>(CONTIG ? a.M : a.inner);
    auto rr = [](int r) { return 8 * (r >> 2) + (r & 3); };
    uint32_t off[NB][JL];   // this lane's byte offset of register 0, kOOB where its column is outside
    int rows[NB][JL];       // rows from there to the field's or the operator's end
#pragma unroll
    for (int i = 0; i < NW; ++i)
#pragma unroll
      for (int j = 0; j < JL; ++j) {
        const int m = 32 * (rb0 + wave + 4 * i);
        const int64_t l = l0 + 32 * j;
        if constexpr (CONTIG) {
          off[i][j] = m + lc < a.M ? 4u * static_cast<uint32_t>((l + lr) * a.M + m + lc) : kOOB;
          rows[i][j] = static_cast<int>(min(max(a.lines - l, int64_t(0)), static_cast<int64_t>(32))) - lr;
        } else {
          const int64_t c = l + lc, b = c / a.inner;
          off[i][j] = c < a.lines ? 4u * static_cast<uint32_t>(b * a.y_bstride + (c - b * a.inner) + (m + lr) * a.inner) : kOOB;
          rows[i][j] = min(a.M - m, 32) - lr;
        }
      }
    auto at = [&](int i, int j, int r) { return rr(r) < rows[i][j] ? off[i][j] : kOOB; };
    // a row step past a small field's end would wrap the range check; no lane's value lies there
    auto step = [&](int r) { return min(rr(r) * row_step, bytes); };
    constexpr bool kAhead = CONTIG || NW < 3;   // strided with 96 accumulators: 161 registers without, 182 with
    float y[2][16] = {}, sc[16];
    auto load_y = [&](int set, int i, int j) {
      if (a.beta == 0.f) return;   // (the same for the whole grid)
#pragma unroll
      for (int r = 0; r < 16; ++r) y[set][r] = ld_f32(rY, at(i, j, r), step(r));
    };
    // the old values of the next block are on their way while this one is updated
    if constexpr (kAhead) load_y(0, 0, 0);
#pragma unroll
    for (int n = 0; n < NW * JL; ++n) {
      const int i = n / JL, j = n % JL;
      if constexpr (!kAhead) load_y(n & 1, i, j);
      else if (n + 1 < NW * JL) load_y((n + 1) & 1, (n + 1) / JL, (n + 1) % JL);
      if (a.scale) {
#pragma unroll
        for (int r = 0; r < 16; ++r) sc[r] = ld_f32(rS, at(i, j, r), step(r));
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][j][r] *= sc[r];
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float v = a.beta != 0.f ? a.beta * y[n & 1][r] + a.alpha * acc[i][j][r] : a.alpha * acc[i][j][r];
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), rY, at(i, j, r), step(r), 0);
      }
    }
  }
}

// NB: row blocks of the waves that have most; the others have one fewer (SplitTiles; a branch per wave, not per product).
template <int FMODE, int NB>
__global__ __launch_bounds__(NT, 3) void split_kernel(FArgs a) {
  __shared__ __attribute__((aligned(16))) __bf16 lds[4 * PART];
  const int tile = xcd_tile(blockIdx.x, gridDim.x);
  const int mt = tile % a.mtiles, rb0 = split_first(a.rb, a.mtiles, mt);
  const int64_t l0 = static_cast<int64_t>(tile / a.mtiles) * LINES;
  Stage<FMODE> X;
  X.K = a.K;
  X.x = make_rsrc(a.X, static_cast<uint32_t>(4 * a.lines * a.K));
  auto row_off = [&](int l) { return 4u * static_cast<uint32_t>(min(l0 + l, a.lines - 1) * a.K); };
  if constexpr (FMODE == 0) {
    const int64_t l = min(l0 + static_cast<int64_t>(threadIdx.x % LINES), a.lines - 1), b = l / a.inner;
    X.ld = 4u * static_cast<uint32_t>(a.inner);
    X.off[0] = 4u * static_cast<uint32_t>(b * a.x_bstride + (l - b * a.inner));
  } else if constexpr (FMODE == 1) {
#pragma unroll
    for (int j = 0; j < 8; ++j) X.off[j] = row_off(static_cast<int>(threadIdx.x) / 32 + 8 * j);
  } else {
    X.off[0] = row_off(static_cast<int>(threadIdx.x) / 4);
  }
  X.load(0);
  X.template store<true>(0, lds);
  X.load(1);
  lds_barrier();
  if (split_wave_blocks(split_first(a.rb, a.mtiles, mt + 1) - rb0, wave_index()) == NB) run_wave<FMODE, NB>(a, X, lds, rb0, l0);
  else run_wave<FMODE, NB - 1>(a, X, lds, rb0, l0);
}

template <int FMODE>
hipError_t launch_f(const FArgs& a, int per_wave, unsigned blocks, hipStream_t s) {
  const dim3 grid(blocks), blk(NT);
  switch (per_wave) {
    case 1: hipLaunchKernelGGL((split_kernel<FMODE, 1>), grid, blk, 0, s, a); break;
    case 2: hipLaunchKernelGGL((split_kernel<FMODE, 2>), grid, blk, 0, s, a); break;
    case 3: hipLaunchKernelGGL((split_kernel<FMODE, 3>), grid, blk, 0, s, a); break;
    default: return hipErrorInvalidConfiguration;
  }
  return hipGetLastError();
}

}  // namespace

// All rows in one tile up to 384 (three row blocks per wave: 96 accumulators), so that the field is read once; shorter
// row tiles where that leaves CUs without a block (256 x 256 plane: 10.5 us with all rows, 8.1 with 128;
// 700 x 1000: 41 and 30; with 500 x 40 x 500, 313 blocks of all rows, 39.8 and 42.7).
SplitTiles split_tiles(int M, int64_t lines) {
  SplitTiles t;
  t.rb = (M + 31) / 32;
  t.line_tiles = (lines + kSplitLines - 1) / kSplitLines;
  int most = 3 * kSplitWaves;
  while (most > kSplitWaves && t.line_tiles * ((t.rb + most - 1) / most) < 256) most -= kSplitWaves;
  t.tiles = (t.rb + most - 1) / most;
  t.per_wave = ((t.rb + t.tiles - 1) / t.tiles + kSplitWaves - 1) / kSplitWaves;
  return t;
}

hipError_t launch_contract_split(const ContractArgs& c, bool contiguous, hipStream_t s) {
  if (!c.frag || c.batch < 1 || c.ncols < 1 || c.M < 1 || c.K < 1) return hipErrorInvalidValue;
  static_assert(kRowPad % 32 == 0 && kColPad % BK == 0, "operator padding must cover whole fragments");
  FArgs a;
  a.op = static_cast<const __bf16*>(c.frag);
  a.M = c.M;
  a.K = c.K;
  a.nch = c.lda / 16;
  a.X = static_cast<const float*>(c.X);
  a.Y = static_cast<float*>(c.Y);
  a.inner = c.ncols;
  a.lines = contiguous ? c.ncols : c.ncols * c.batch;
  a.x_bstride = c.x_bstride;
  a.y_bstride = c.y_bstride;
  a.alpha = c.alpha;
  a.beta = c.beta;
  a.scale = static_cast<const float*>(c.scale);
  const SplitTiles t = split_tiles(c.M, a.lines);
  a.rb = t.rb;
  a.mtiles = t.tiles;
  const int64_t blocks = t.line_tiles * t.tiles;
  // 32-bit byte offsets from a block's first line: a whole field stays below 2 GiB (checked at plan creation)
  const int64_t xb = 4 * a.lines * c.K, yb = 4 * a.lines * c.M;
  if (blocks > 0x7fffffff || xb >= (int64_t(1) << 31) || yb >= (int64_t(1) << 31)) return hipErrorInvalidValue;
  const unsigned n = static_cast<unsigned>(blocks);
  if (!contiguous) return launch_f<0>(a, t.per_wave, n, s);
  return c.K % 4 == 0 && (reinterpret_cast<uintptr_t>(c.X) & 15) == 0 ? launch_f<2>(a, t.per_wave, n, s)
                                                                              : launch_f<1>(a, t.per_wave, n, s);
}

}  // namespace pstd
