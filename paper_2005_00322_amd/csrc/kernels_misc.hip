// Single-workgroup 1D stepper, wall handling, the reflection-coefficient combination and checks.
#include <algorithm>

#include "common.h"

namespace pstd {
namespace {

// Whole 1D time loop in one workgroup: p and u live in LDS for all steps, the operators (stored
// transposed, K x M with row stride ldt, so that consecutive lanes read consecutive rows' entries)
// stream from L2.  Each step is Eq. (dtt_pstd_solution): u += G~ p, then p += D~ u (scaled pointwise by
// c0(x)^2 when a sound-speed map is given).  Threads split every dot product 4 ways; the sums and the
// update are formed in FP64 for both state types and rounded once into the state.  One CU reads its
// operators at well under the L2 rate (n = 1000, FP32: 509 us per step), so this is only the fallback of
// step1d_multi_kernel below, and for calls without a workspace.
template <typename T>
__device__ void step1d_one_block(const T* __restrict__ GT, int ldg, const T* __restrict__ DT, int ldd, T* __restrict__ p,
                                 T* __restrict__ u, int n, int64_t steps, const T* __restrict__ scale) {
  extern __shared__ unsigned char smem_raw[];
  T* sp = reinterpret_cast<T*>(smem_raw);
  T* su = sp + n;
  // 4 partial sums per row, 8-byte aligned after the two state vectors
  double* part = reinterpret_cast<double*>(smem_raw + ((2 * n * sizeof(T) + 7) & ~static_cast<size_t>(7)));
  const int tid = threadIdx.x;
  const int nt = blockDim.x;
  for (int i = tid; i < n; i += nt) sp[i] = p[i];
  for (int i = tid; i < n - 1; i += nt) su[i] = u[i];
  const int nm = n - 1;
  for (int64_t s = 0; s < steps; ++s) {
    __syncthreads();
    // u_i += sum_k G~[i][k] p_k, k split in 4 interleaved quarters
    for (int e = tid; e < 4 * nm; e += nt) {
      const int i = e % nm, q = e / nm;
      double acc = 0;
      for (int k = q; k < n; k += 4) acc += static_cast<double>(GT[static_cast<int64_t>(k) * ldg + i]) * sp[k];
      part[q * n + i] = acc;
    }
    __syncthreads();
    for (int i = tid; i < nm; i += nt)
      su[i] = static_cast<T>(su[i] + ((part[i] + part[n + i]) + (part[2 * n + i] + part[3 * n + i])));
    __syncthreads();
    // p_i += c(x_i) * sum_k D~[i][k] u_k
    for (int e = tid; e < 4 * n; e += nt) {
      const int i = e % n, q = e / n;
      double acc = 0;
      for (int k = q; k < nm; k += 4) acc += static_cast<double>(DT[static_cast<int64_t>(k) * ldd + i]) * su[k];
      part[q * n + i] = acc;
    }
    __syncthreads();
    for (int i = tid; i < n; i += nt) {
      double d = (part[i] + part[n + i]) + (part[2 * n + i] + part[3 * n + i]);
      if (scale) d *= static_cast<double>(scale[i]);
      sp[i] = static_cast<T>(sp[i] + d);
    }
  }
  __syncthreads();
  for (int i = tid; i < n; i += nt) p[i] = sp[i];
  for (int i = tid; i < n - 1; i += nt) u[i] = su[i];
}

// ---- 1D lines above 128 nodes: the time loop over many workgroups --------------------------------------
// Workgroup w owns rows 16 w .. 16 w + 15 of both operators, held in registers (as double) for all steps:
// half a wave per row, lane l of the half holding columns l + 32 k.  Per half step a workgroup gathers the
// other field into LDS, forms its 16 dot products (FP64), updates its values and publishes them.  n^2 FP64
// products are spread over n / 16 CUs (0.2 us of them at n = 1000), so what bounds a half step is the exchange between
// CUs: a value travels as one 64-bit word holding the float and the half step's number (FP64: two words with half
// the bits each), so readers poll the values themselves and no barrier, fence or second round trip is needed.
// A buffer per field is enough: a workgroup publishes step t + 1 of a field only after it has read all of
// the other field, each value of which was published after its owner had read all of step t.  That holds a reader's
// values only if it owns a word of the other field itself, so u has n words too, the last of them a zero: with n - 1 the last
// workgroup of n = 16 m + 1 nodes owns row n - 1 of p alone, and nobody waits for it before p moves on.
// n = 1000, FP32 with a map, 50 steps: 25.5 ms in one workgroup, 0.265 ms here (2.5 us per half step).
//
// The workgroups have to be resident together.  A wait is bounded: a workgroup that gives up sets
// head->abort and ends, and so do the others in turn.  Results go to a copy; the commit kernel that follows
// either moves them into the state or, after an abort, runs all the steps in one workgroup from the state,
// which is still untouched.  head->epoch numbers the half steps of successive launches (kept on the device, so
// a captured launch can be replayed).
struct LineHead {
  unsigned epoch, abort;
};
constexpr int kLineThreads = 32 * kLineRows;

template <typename T>
__device__ __forceinline__ void line_publish(unsigned long long* x, int n, int i, T v, unsigned tag) {
  const unsigned long long t = static_cast<unsigned long long>(tag) << 32;
  if constexpr (sizeof(T) == 4) {
    __hip_atomic_store(x + i, t | __builtin_bit_cast(unsigned, v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  } else {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    __hip_atomic_store(x + i, t | (b & 0xffffffffull), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(x + n + i, t | (b >> 32), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// Values x[tid], x[tid + 512], .. below count into LDS once they carry `tag`; false if the wait ran out.
template <typename T, int PER>
__device__ __forceinline__ bool line_gather(const unsigned long long* x, int n, int count, unsigned tag, double* lds,
                                            unsigned spins) {
  const int tid = threadIdx.x;
  unsigned long long a[PER], b[PER];
  for (unsigned k = 0;; ++k) {
    bool all = true;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int i = tid + q * kLineThreads;
      if (i < count) {
        a[q] = __hip_atomic_load(x + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if constexpr (sizeof(T) == 8) b[q] = __hip_atomic_load(x + n + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      if (tid + q * kLineThreads >= count) continue;
      all = all && static_cast<unsigned>(a[q] >> 32) == tag;
      if constexpr (sizeof(T) == 8) all = all && static_cast<unsigned>(b[q] >> 32) == tag;
    }
    if (all) break;
    if (k >= spins) return false;
  }
#pragma unroll
  for (int q = 0; q < PER; ++q) {
    const int i = tid + q * kLineThreads;
    if (i >= count) continue;
    if constexpr (sizeof(T) == 4)
      lds[i] = static_cast<double>(__builtin_bit_cast(float, static_cast<unsigned>(a[q])));
    else
      lds[i] = __builtin_bit_cast(double, (b[q] << 32) | (a[q] & 0xffffffffull));
  }
  return true;
}

// x plus the value of the lane a DPP control selects (both halves of the double move together)
template <int CTRL>
__device__ __forceinline__ double dpp_add(double x) {
  const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
  const unsigned lo = __builtin_amdgcn_update_dpp(0, static_cast<int>(b), CTRL, 0xf, 0xf, true);
  const unsigned hi = __builtin_amdgcn_update_dpp(0, static_cast<int>(b >> 32), CTRL, 0xf, 0xf, true);
  return x + __builtin_bit_cast(double, (static_cast<unsigned long long>(hi) << 32) | lo);
}

// Sum over the 32 lanes of a half wave, in all of them, in a fixed order: quad_perm [1,0,3,2] and [2,3,0,1],
// then row_half_mirror and row_mirror (every lane of a quad, then of eight, holds the same sum), then the
// neighbouring row of 16.
__device__ __forceinline__ double half_wave_sum(double x) {
  x = dpp_add<0xB1>(x);
  x = dpp_add<0x4E>(x);
  x = dpp_add<0x141>(x);
  x = dpp_add<0x140>(x);
  return x + __shfl_xor(x, 16);
}

// KPL columns per lane: n <= 32 KPL.
template <typename T, int KPL>
__global__ __launch_bounds__(kLineThreads) void step1d_multi_kernel(const T* __restrict__ G, int ldg,
                                                                    const T* __restrict__ D, int ldd,
                                                                    const T* __restrict__ p, const T* __restrict__ u,
                                                                    int n, int64_t steps, const T* __restrict__ scale,
                                                                    LineHead* head, unsigned long long* xp,
                                                                    unsigned long long* xu, T* __restrict__ p_out,
                                                                    T* __restrict__ u_out, unsigned spins) {
  constexpr int PER = (32 * KPL + kLineThreads - 1) / kLineThreads;
  __shared__ double sp[32 * KPL], su[32 * KPL];
  __shared__ int gave_up[2];   // one per gather of a step, so a wave's next gather cannot change what others read
  const int tid = threadIdx.x, l = tid & 31, nm = n - 1;
  const int i = blockIdx.x * kLineRows + (tid >> 5);   // this half wave's row
  double g[KPL], d[KPL];
#pragma unroll
  for (int k = 0; k < KPL; ++k) {
    const int c = l + 32 * k;
    g[k] = (i < nm && c < n) ? static_cast<double>(G[static_cast<int64_t>(i) * ldg + c]) : 0.0;
    d[k] = (i < n && c < nm) ? static_cast<double>(D[static_cast<int64_t>(i) * ldd + c]) : 0.0;
  }
  const double sc = (scale && i < n) ? static_cast<double>(scale[i]) : 1.0;
  T pi = i < n ? p[i] : T(0), ui = i < nm ? u[i] : T(0);
  for (int e = tid; e < 32 * KPL; e += kLineThreads) {
    sp[e] = e < n ? static_cast<double>(p[e]) : 0.0;
    su[e] = 0.0;
  }
  if (tid < 2) gave_up[tid] = 0;
  bool stop = false;
  unsigned tag = head->epoch;
  __syncthreads();
  auto dot = [&](const double (&a)[KPL], const double* x) {
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < KPL; ++k) acc[k & 3] = fma(a[k], x[l + 32 * k], acc[k & 3]);
    return half_wave_sum((acc[0] + acc[1]) + (acc[2] + acc[3]));
  };
  for (int64_t s = 0; s < steps; ++s) {
    if (s) {
      if (!line_gather<T, PER>(xp, n, n, tag, sp, spins)) gave_up[0] = 1;
      __syncthreads();
      if ((stop = gave_up[0] != 0)) break;
    }
    ui = static_cast<T>(static_cast<double>(ui) + dot(g, sp));
    ++tag;
    if (l == 0 && i < line_u_words(n)) line_publish<T>(xu, n, i, i < nm ? ui : T(0), tag);
    if (!line_gather<T, PER>(xu, n, line_u_words(n), tag, su, spins)) gave_up[1] = 1;
    __syncthreads();
    if ((stop = gave_up[1] != 0)) break;
    pi = static_cast<T>(static_cast<double>(pi) + dot(d, su) * sc);
    ++tag;
    if (l == 0 && i < n) line_publish<T>(xp, n, i, pi, tag);
  }
  if (stop) {
    if (tid == 0) __hip_atomic_store(&head->abort, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return;
  }
  if (l == 0 && i < n) p_out[i] = pi;
  if (l == 0 && i < nm) u_out[i] = ui;
}

// One workgroup, after step1d_multi_kernel: its results into the state, or all the steps here if it gave up.
template <typename T>
__global__ __launch_bounds__(1024) void step1d_commit_kernel(const T* __restrict__ GT, int ldg, const T* __restrict__ DT,
                                                             int ldd, T* __restrict__ p, T* __restrict__ u, int n,
                                                             int64_t steps, const T* __restrict__ scale, LineHead* head,
                                                             const T* __restrict__ p_out, const T* __restrict__ u_out) {
  const unsigned abort = head->abort, epoch = head->epoch;
  __syncthreads();
  if (threadIdx.x == 0) {
    head->epoch = epoch + static_cast<unsigned>(2 * steps);
    head->abort = 0;
  }
  if (abort) {
    step1d_one_block<T>(GT, ldg, DT, ldd, p, u, n, steps, scale);
    return;
  }
  for (int i = threadIdx.x; i < n; i += blockDim.x) p[i] = p_out[i];
  for (int i = threadIdx.x; i < n - 1; i += blockDim.x) u[i] = u_out[i];
}

// All steps in one workgroup, without a workspace.
template <typename T>
__global__ __launch_bounds__(1024) void step1d_one_kernel(const T* __restrict__ GT, int ldg, const T* __restrict__ DT, int ldd,
                                                          T* __restrict__ p, T* __restrict__ u, int n, int64_t steps,
                                                          const T* __restrict__ scale) {
  step1d_one_block<T>(GT, ldg, DT, ldd, p, u, n, steps, scale);
}

// A single step of a line of at most kOnceNodes nodes in one workgroup: half wave w takes rows w, w + 32, .., the sums in the
// order of step1d_multi_kernel's (so a call of one step and one of many give the same bits).  A call of one step is bound by
// its launches and one round trip for the operators; the two launches of the general path cost more than they spread.
constexpr int kOnceNodes = 160, kOnceRows = kOnceNodes / 32;

template <typename T>
__global__ __launch_bounds__(1024) void step1d_once_kernel(const T* __restrict__ G, int ldg, const T* __restrict__ D, int ldd,
                                                           T* __restrict__ p, T* __restrict__ u, int n,
                                                           const T* __restrict__ scale) {
  __shared__ double sp[kOnceNodes], su[kOnceNodes];
  const int tid = threadIdx.x, l = tid & 31, w = tid >> 5, nm = n - 1;
  T g[kOnceRows][kOnceRows], d[kOnceRows][kOnceRows];   // [row][column l + 32 k]
#pragma unroll
  for (int r = 0; r < kOnceRows; ++r)
#pragma unroll
    for (int k = 0; k < kOnceRows; ++k) {
      const int i = w + 32 * r, c = l + 32 * k;
      g[r][k] = (i < nm && c < n) ? G[static_cast<int64_t>(i) * ldg + c] : T(0);
      d[r][k] = (i < n && c < nm) ? D[static_cast<int64_t>(i) * ldd + c] : T(0);
    }
  if (tid < kOnceNodes) {
    sp[tid] = tid < n ? static_cast<double>(p[tid]) : 0.0;
    su[tid] = 0.0;
  }
  auto dot = [&](const T (&a)[kOnceRows], const double* x) {
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k = 0; k < kOnceRows; ++k) acc[k & 3] = fma(static_cast<double>(a[k]), x[l + 32 * k], acc[k & 3]);
    return half_wave_sum((acc[0] + acc[1]) + (acc[2] + acc[3]));
  };
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kOnceRows; ++r) {
    const int i = w + 32 * r;
    const double s = dot(g[r], sp);
    if (l == 0 && i < nm) {
      const T v = static_cast<T>(static_cast<double>(u[i]) + s);
      u[i] = v;
      su[i] = static_cast<double>(v);
    }
  }
  __syncthreads();
#pragma unroll
  for (int r = 0; r < kOnceRows; ++r) {
    const int i = w + 32 * r;
    const double s = dot(d[r], su);
    if (l == 0 && i < n) p[i] = static_cast<T>(sp[i] + s * (scale ? static_cast<double>(scale[i]) : 1.0));
  }
}

// The whole time loop of a line of n <= 128 nodes in one workgroup, both operators in registers for all steps:
// thread t owns row t / 8 of each operator and its 16 entries in columns t % 8 + 8 j, so a step reads no
// global memory and the eight addresses that a wave reads from the state in LDS lie in different banks.  A row's
// eight partial dot products are added across its eight lanes (DPP, a fixed order).  Per step: u += G~ p, a
// barrier, p += D~ u (times c0(x)^2 with a map), a barrier.  Sums and updates in FP64, rounded once into the
// state; operators and state are held as double for both state types, so a float is converted once.  Latency is
// all there is: LDS read, 16 FMAs in four chains, three DPP adds, LDS write, barrier.  n = 128, FP64, 20 steps:
// 62.6 us with 16 consecutive columns per lane (eight-way bank conflicts) and shuffles, 27.5 us like this.
template <typename T>
__global__ __launch_bounds__(1024) void step1d_reg_kernel(const T* __restrict__ G, int ldg, const T* __restrict__ D,
                                                          int ldd, T* __restrict__ p, T* __restrict__ u, int n,
                                                          int64_t steps, const T* __restrict__ scale) {
  __shared__ double sp[128], su[128];
  const int tid = threadIdx.x, i = tid >> 3, q = tid & 7;
  const int nm = n - 1;
  double g[16], d[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) {
    const int k = q + 8 * j;
    g[j] = (i < nm && k < n) ? static_cast<double>(G[static_cast<int64_t>(i) * ldg + k]) : 0.0;
    d[j] = (i < n && k < nm) ? static_cast<double>(D[static_cast<int64_t>(i) * ldd + k]) : 0.0;
  }
  const double sc = (scale && i < n) ? static_cast<double>(scale[i]) : 1.0;
  T pi = i < n ? p[i] : T(0), ui = i < nm ? u[i] : T(0);   // the row's own values, in all its lanes
  if (q == 0) sp[i] = static_cast<double>(pi);
  auto dot = [&](const double (&a)[16], const double* x) {
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[j & 3] = fma(a[j], x[q + 8 * j], acc[j & 3]);
    double v = (acc[0] + acc[1]) + (acc[2] + acc[3]);
    v = dpp_add<0xB1>(v);      // quad_perm [1,0,3,2]
    v = dpp_add<0x4E>(v);      // quad_perm [2,3,0,1]
    return dpp_add<0x141>(v);  // row_half_mirror
  };
  lds_barrier();
  for (int64_t s = 0; s < steps; ++s) {
    ui = static_cast<T>(static_cast<double>(ui) + dot(g, sp));
    if (q == 0) su[i] = static_cast<double>(ui);
    lds_barrier();
    pi = static_cast<T>(static_cast<double>(pi) + dot(d, su) * sc);
    if (q == 0) sp[i] = static_cast<double>(pi);
    lds_barrier();
  }
  if (q == 0 && i < n) p[i] = pi;
  if (q == 0 && i < nm) u[i] = ui;
}

// cols = rows^T by tiles of 64 x 64 (a long line's operators, once per plan: 1365 nodes in FP64 take the host 8 ms, bound by the
// strided side).
template <typename T>
__global__ __launch_bounds__(256) void transpose_kernel(const T* __restrict__ rows, int Mp, int Kp, T* __restrict__ cols) {
  __shared__ T tile[64][65];
  const int i0 = blockIdx.y * 64, k0 = blockIdx.x * 64, l = threadIdx.x & 63, w = threadIdx.x >> 6;
  for (int r = w; r < 64; r += 4) tile[r][l] = rows[static_cast<int64_t>(i0 + r) * Kp + k0 + l];
  __syncthreads();
  for (int r = w; r < 64; r += 4) cols[static_cast<int64_t>(k0 + r) * Mp + i0 + l] = tile[l][r];
}

template <typename T>
__global__ void zero_dirichlet_kernel(T* p, int ndim, int64_t n0, int64_t n1, int64_t n2, int lo0, int hi0, int lo1,
                                      int hi1, int lo2, int hi2) {
  const int64_t total = n0 * n1 * n2;
  for (int64_t idx = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; idx < total;
       idx += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const int64_t i2 = idx % n2;
    const int64_t i1 = (idx / n2) % n1;
    const int64_t i0 = idx / (n1 * n2);
    bool wall = (lo0 && i0 == 0) || (hi0 && i0 == n0 - 1);
    if (ndim > 1) wall = wall || (lo1 && i1 == 0) || (hi1 && i1 == n1 - 1);
    if (ndim > 2) wall = wall || (lo2 && i2 == 0) || (hi2 && i2 == n2 - 1);
    if (wall) p[idx] = T(0);
  }
}

template <typename T>
__global__ void fill_zero_kernel(T* x, int64_t count) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < count;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x)
    x[i] = T(0);
}

template <typename T>
__global__ void square_kernel(const float* in, T* out, int64_t count) {
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < count;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const T v = static_cast<T>(in[i]);
    out[i] = v * v;
  }
}

constexpr int kMaxFields = 64;
struct CombineArgs {
  const float* f[kMaxFields];
  float w[kMaxFields];
  int nf;
};

// out = sum_i w_i f_i (§5), 4 elements per lane with a scalar tail.
__global__ __launch_bounds__(256) void combine_kernel(CombineArgs a, float* out, int64_t count) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  const int64_t nvec = count / 4;
  bool aligned = (reinterpret_cast<uintptr_t>(out) & 15) == 0;
  for (int i = 0; i < a.nf; ++i) aligned = aligned && ((reinterpret_cast<uintptr_t>(a.f[i]) & 15) == 0);
  const int64_t start = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  if (aligned) {
    for (int64_t v = start; v < nvec; v += stride) {
      float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
      for (int i = 0; i < a.nf; ++i) {
        const float4 x = reinterpret_cast<const float4*>(a.f[i])[v];
        acc.x += a.w[i] * x.x;
        acc.y += a.w[i] * x.y;
        acc.z += a.w[i] * x.z;
        acc.w += a.w[i] * x.w;
      }
      reinterpret_cast<float4*>(out)[v] = acc;
    }
    for (int64_t e = 4 * nvec + start; e < count; e += stride) {
      float acc = 0.f;
      for (int i = 0; i < a.nf; ++i) acc += a.w[i] * a.f[i][e];
      out[e] = acc;
    }
  } else {
    for (int64_t e = start; e < count; e += stride) {
      float acc = 0.f;
      for (int i = 0; i < a.nf; ++i) acc += a.w[i] * a.f[i][e];
      out[e] = acc;
    }
  }
}

// out = wn pn + wd pd of many pairs of fields in one launch (block y: pair); one launch per pair took 4.4 us each.
constexpr int kMaxPairs = 80;   // 40 bytes each, within a launch's 4 KB of arguments
struct PairArgs {
  CombinePair p[kMaxPairs];
};

__global__ __launch_bounds__(256) void combine_pairs_kernel(PairArgs a) {
  const CombinePair& c = a.p[blockIdx.y];
  const int64_t stride = static_cast<int64_t>(gridDim.x) * 256, start = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const bool aligned =
      ((reinterpret_cast<uintptr_t>(c.out) | reinterpret_cast<uintptr_t>(c.n) | reinterpret_cast<uintptr_t>(c.d)) & 15) == 0;
  const int64_t nvec = aligned ? c.count / 4 : 0;
  // the products are added in the order of combine_kernel's fields (Neumann first), from zero
  for (int64_t v = start; v < nvec; v += stride) {
    const float4 n = reinterpret_cast<const float4*>(c.n)[v], d = reinterpret_cast<const float4*>(c.d)[v];
    float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
    o.x += c.wn * n.x; o.y += c.wn * n.y; o.z += c.wn * n.z; o.w += c.wn * n.w;
    o.x += c.wd * d.x; o.y += c.wd * d.y; o.z += c.wd * d.z; o.w += c.wd * d.w;
    reinterpret_cast<float4*>(c.out)[v] = o;
  }
  for (int64_t e = 4 * nvec + start; e < c.count; e += stride) {
    float o = 0.f;
    o += c.wn * c.n[e];
    o += c.wd * c.d[e];
    c.out[e] = o;
  }
}

template <typename T>
__global__ void nonfinite_kernel(const T* x, int64_t count, int* flag) {
  bool bad = false;
  for (int64_t i = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x; i < count;
       i += static_cast<int64_t>(gridDim.x) * blockDim.x) {
    const T v = x[i];
    bad = bad || !(v - v == T(0));
  }
  if (bad) atomicOr(flag, 1);
}

unsigned blocks_for(int64_t count, int threads) {
  int64_t b = (count + threads - 1) / threads;
  if (b < 1) b = 1;
  if (b > 8192) b = 8192;
  return static_cast<unsigned>(b);
}

}  // namespace

namespace {

// Layout of a plan's line workspace: the head (256 bytes), the exchanged words of p and of u (two per value in
// FP64), the result copies.
size_t line_words(int prec, int n) { return static_cast<size_t>(prec == PSTD_FP64 ? 2 : 1) * n; }

template <typename T>
hipError_t launch_step1d_t(int prec, const DevOperator& Go, const DevOperator& Do, T* p, T* u, int n, int64_t steps,
                           const T* scale, void* work, unsigned spins, hipStream_t s) {
  const T *G = static_cast<const T*>(Go.rows), *D = static_cast<const T*>(Do.rows);
  if (!G || !D || (n > 128 && (!Go.cols || !Do.cols))) return hipErrorInvalidValue;
  if (n <= 128) {
    hipLaunchKernelGGL(step1d_reg_kernel<T>, dim3(1), dim3(1024), 0, s, G, Go.Kp, D, Do.Kp, p, u, n, steps, scale);
    return hipGetLastError();
  }
  // one step, us a call with this kernel / with the two launches below: 130 nodes 8.8 / 11.5 (FP32), 7.9 / 12.1 (FP64), 160
  // nodes 9.5 / 11.8, 8.9 / 11.2; beyond, the rows of a sixth pass would not fit the registers
  if (steps == 1 && n <= kOnceNodes) {
    hipLaunchKernelGGL(step1d_once_kernel<T>, dim3(1), dim3(1024), 0, s, G, Go.Kp, D, Do.Kp, p, u, n, scale);
    return hipGetLastError();
  }
  const size_t shmem = ((sizeof(T) * 2 * static_cast<size_t>(n) + 7) & ~static_cast<size_t>(7)) + 8 * static_cast<size_t>(4) * n;
  if (shmem > 64 * 1024 || n > kLineMaxNodes) return hipErrorInvalidConfiguration;
  if (!work) {
    hipLaunchKernelGGL(step1d_one_kernel<T>, dim3(1), dim3(1024), shmem, s, static_cast<const T*>(Go.cols), Go.Mp,
                       static_cast<const T*>(Do.cols), Do.Mp, p, u, n, steps, scale);
    return hipGetLastError();
  }
  LineHead* head = static_cast<LineHead*>(work);
  unsigned long long* xp = reinterpret_cast<unsigned long long*>(static_cast<unsigned char*>(work) + 256);
  unsigned long long* xu = xp + line_words(prec, n);
  T* po = reinterpret_cast<T*>(xu + line_words(prec, n));
  T* uo = po + n;
  const dim3 grid(line_workgroups(n)), blk(kLineThreads);
#define PSTD_LINE(KPL)                                                                                                \
  hipLaunchKernelGGL((step1d_multi_kernel<T, KPL>), grid, blk, 0, s, G, Go.Kp, D, Do.Kp, p, u, n, steps, scale, head, \
                     xp, xu, po, uo, spins)
  if (n <= 32 * 8) PSTD_LINE(8);
  else if (n <= 32 * 16) PSTD_LINE(16);
  else if (n <= 32 * 24) PSTD_LINE(24);
  else if (n <= 32 * 32) PSTD_LINE(32);
  else PSTD_LINE(43);
#undef PSTD_LINE
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(step1d_commit_kernel<T>, dim3(1), dim3(1024), shmem, s, static_cast<const T*>(Go.cols), Go.Mp,
                     static_cast<const T*>(Do.cols), Do.Mp, p, u, n, steps, scale, head, po, uo);
  return hipGetLastError();
}

}  // namespace

size_t step1d_work_bytes(int prec, int n) {
  if (n <= 128) return 0;
  return round_up(256 + 2 * line_words(prec, n) * 8 + 2 * static_cast<size_t>(prec == PSTD_FP64 ? 8 : 4) * n, 256);
}

hipError_t launch_step1d(int prec, const DevOperator& G, const DevOperator& D, void* p, void* u, int n,
                         int64_t steps, const void* scale, void* work, unsigned spins, hipStream_t s) {
  if (prec == PSTD_FP64)
    return launch_step1d_t<double>(prec, G, D, static_cast<double*>(p), static_cast<double*>(u), n, steps,
                                   static_cast<const double*>(scale), work, spins, s);
  return launch_step1d_t<float>(prec, G, D, static_cast<float*>(p), static_cast<float*>(u), n, steps,
                                static_cast<const float*>(scale), work, spins, s);
}

hipError_t launch_transpose(bool dbl, const void* rows, int Mp, int Kp, void* cols, hipStream_t s) {
  if (Mp < 64 || Kp < 64 || Mp % 64 || Kp % 64) return hipErrorInvalidValue;
  const dim3 grid(Kp / 64, Mp / 64), blk(256);
  if (dbl)
    hipLaunchKernelGGL(transpose_kernel<double>, grid, blk, 0, s, static_cast<const double*>(rows), Mp, Kp, static_cast<double*>(cols));
  else
    hipLaunchKernelGGL(transpose_kernel<float>, grid, blk, 0, s, static_cast<const float*>(rows), Mp, Kp, static_cast<float*>(cols));
  return hipGetLastError();
}

hipError_t launch_zero_dirichlet(int prec, void* p, int ndim, const int64_t* n, const int* lo, const int* hi,
                                 hipStream_t s) {
  const int64_t total = n[0] * n[1] * n[2];
  const unsigned nb = blocks_for(total, 256);
  if (prec == PSTD_FP64)
    hipLaunchKernelGGL(zero_dirichlet_kernel<double>, dim3(nb), dim3(256), 0, s, static_cast<double*>(p), ndim, n[0],
                       n[1], n[2], lo[0], hi[0], lo[1], hi[1], lo[2], hi[2]);
  else
    hipLaunchKernelGGL(zero_dirichlet_kernel<float>, dim3(nb), dim3(256), 0, s, static_cast<float*>(p), ndim, n[0],
                       n[1], n[2], lo[0], hi[0], lo[1], hi[1], lo[2], hi[2]);
  return hipGetLastError();
}

hipError_t launch_fill_zero(int prec, void* x, int64_t count, hipStream_t s) {
  const unsigned nb = blocks_for(count, 256);
  if (prec == PSTD_FP64)
    hipLaunchKernelGGL(fill_zero_kernel<double>, dim3(nb), dim3(256), 0, s, static_cast<double*>(x), count);
  else
    hipLaunchKernelGGL(fill_zero_kernel<float>, dim3(nb), dim3(256), 0, s, static_cast<float*>(x), count);
  return hipGetLastError();
}

hipError_t launch_square(int prec, const float* in, void* out, int64_t count, hipStream_t s) {
  if (prec == PSTD_FP64)
    hipLaunchKernelGGL(square_kernel<double>, dim3(blocks_for(count, 256)), dim3(256), 0, s, in,
                       static_cast<double*>(out), count);
  else
    hipLaunchKernelGGL(square_kernel<float>, dim3(blocks_for(count, 256)), dim3(256), 0, s, in,
                       static_cast<float*>(out), count);
  return hipGetLastError();
}

hipError_t launch_combine(const float* const* f, const float* w, int nf, float* out, int64_t count, hipStream_t s) {
  if (nf < 1 || nf > kMaxFields) return hipErrorInvalidValue;
  CombineArgs a;
  for (int i = 0; i < nf; ++i) {
    a.f[i] = f[i];
    a.w[i] = w[i];
  }
  a.nf = nf;
  hipLaunchKernelGGL(combine_kernel, dim3(blocks_for((count + 3) / 4, 256)), dim3(256), 0, s, a, out, count);
  return hipGetLastError();
}

hipError_t launch_combine_pairs(const CombinePair* pairs, int count, hipStream_t s) {
  for (int i = 0; i < count; i += kMaxPairs) {
    PairArgs a;
    const int n = std::min(count - i, kMaxPairs);
    int64_t most = 0;
    for (int k = 0; k < n; ++k) {
      a.p[k] = pairs[i + k];
      most = std::max(most, pairs[i + k].count);
    }
    for (int k = n; k < kMaxPairs; ++k) a.p[k] = CombinePair{};
    hipLaunchKernelGGL(combine_pairs_kernel, dim3(std::min(blocks_for((most + 3) / 4, 256), 64u), n), dim3(256), 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_nonfinite(int prec, const void* x, int64_t count, int* flag, hipStream_t s) {
  const unsigned nb = blocks_for(count, 256);
  if (prec == PSTD_FP64)
    hipLaunchKernelGGL(nonfinite_kernel<double>, dim3(nb), dim3(256), 0, s, static_cast<const double*>(x), count, flag);
  else
    hipLaunchKernelGGL(nonfinite_kernel<float>, dim3(nb), dim3(256), 0, s, static_cast<const float*>(x), count, flag);
  return hipGetLastError();
}

}  // namespace pstd
