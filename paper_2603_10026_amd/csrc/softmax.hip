// Safe softmax over the last axis: the max -> sum-exp cascade (paper
// Section 2.2; Appendix A.2, first two reductions) fused at wavefront level.
//
// Kernel 1 (rows that fit in registers): one 64-lane wavefront owns one row.
// The row is read once with 128-bit loads and stays in registers; the row max
// and the row sum are reduced lane-locally, then across the wavefront with
// DPP; the normalised row is written once with 128-bit stores.  HBM traffic is
// the algorithmic minimum (one read + one write).
//
// Rows that start at any element or hold no whole number of vectors take the same kernels with
// unaligned vectors (below); rows of less than one vector take a lane each.
//
// Kernel 2 (rows too long for the registers of a workgroup): one workgroup streams a row, every
// lane carrying the level-1 incremental state (m, l) (Appendix A.2,
// incremental form), corrected once per 128-bit vector; lane states are merged
// with the level-k fused expression (Section 3.2 Eq. (11)) across the wavefront
// and then across wavefronts through LDS; a second sweep over the row writes
// the result.
#include <type_traits>

#include "rf_device.h"
#include "rf_launch.h"

namespace rf {

constexpr int kSoftmaxWavesPerWg = 4;

namespace {

// Rows that start anywhere (natural element alignment) and hold any number n >= V of elements,
// in 16-byte vectors all the same: vector idx covers elements idx V .. idx V + V - 1, and the one
// that would reach past the end is moved back to the last V elements, where it repeats up to V - 1
// elements of its neighbour.  A repeated element does not change a maximum and is stored twice
// with the same value; only the sum has to leave it out.  Vectors past the end sit in the same
// place and contribute nothing.  (A wavefront's 1 KB then touches nine 128-byte lines instead of
// eight.)  256 rows of 50001 fp32 values take 22 us where element-wise accesses and two sweeps took
// 112; 4096 rows of 4095 bf16 values 13.0 where they took 26.5.

template <typename T>
__device__ __forceinline__ u32x4 ragged_load(const T* row, int idx, int n) {
  constexpr int V = Elem<T>::kPerVec;
  return __builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(row + min(idx * V, n - V)));
}
template <typename T>
__device__ __forceinline__ void ragged_store(T* row, int idx, int n, const u32x4& v) {
  constexpr int V = Elem<T>::kPerVec;
  __builtin_nontemporal_store(v, reinterpret_cast<u32x4_any*>(row + min(idx * V, n - V)));
}
// What the exponents are formed with, exp2(e log2 e + this).  A maximum whose product with log2 e leaves
// fp32 (rows of nothing but the type's lowest value) is subtracted from the values first.
template <int N, int V>
__device__ __forceinline__ float exponent_base(float (&e)[N][V], float m) {
  if (fabsf(m) >= 2e38f) {
#pragma unroll
    for (int c = 0; c < N; ++c)
#pragma unroll
      for (int i = 0; i < V; ++i) e[c][i] -= m;
    return 0.f;
  }
  return -m * kLog2e;
}
// Exponentials of a vector, in place; returns s + their sum.
template <int V>
__device__ __forceinline__ float exp_sum(float s, float* e, float mb) {
#pragma unroll
  for (int i = 0; i < V; ++i) {
    e[i] = fast_exp2(fmaf(e[i], kLog2e, mb));
    s += e[i];
  }
  return s;
}
// whole: wave-uniform, no lane's vector reaches past the end
template <int V>
__device__ __forceinline__ float ragged_exp_sum(float s, float* e, float mb, int idx, int n, bool whole) {
  if (whole) return exp_sum<V>(s, e, mb);
  const int first = idx * V - min(idx * V, n - V);  // elements below it are the neighbour's (V or more: none is ours)
#pragma unroll
  for (int i = 0; i < V; ++i) {
    e[i] = fast_exp2(fmaf(e[i], kLog2e, mb));
    s += i >= first ? e[i] : 0.f;
  }
  return s;
}

}  // namespace

// One wavefront per row; NCH 128-bit chunks per lane; n % kPerVec == 0.
// LANE_LEVEL = false (the shipped path): the two reductions are fused at wavefront level,
// the row max is known before the sum starts, nothing is ever corrected.
// LANE_LEVEL = true (fusion-level study only, Section 5.3): every lane runs the level-1
// incremental form over its own elements, one correction per element, and the 64 lane
// states are merged with the level-k fused expression.
// Wavefronts per SIMD the register allocator has to leave room for, by the number of fp32 values
// a lane holds: without the bound the scheduler spends registers on instruction-level
// parallelism this HBM-bound kernel has no use for, and occupancy (bytes in flight) drops.
constexpr int softmax_waves_per_simd(int floats_per_lane) {
  return floats_per_lane <= 32 ? 8 : floats_per_lane <= 64 ? 4 : 2;
}

template <typename T, int NCH, bool RAGGED, bool LANE_LEVEL = false>
__global__ __launch_bounds__(kSoftmaxWavesPerWg * kWave,
                             softmax_waves_per_simd(NCH * Elem<T>::kPerVec) * 4 / kSoftmaxWavesPerWg)
void softmax_row_in_regs_kernel(
    const T* __restrict__ x, T* __restrict__ y, int64_t rows, int n, int64_t x_pitch,
    int64_t y_pitch) {
  constexpr int V = Elem<T>::kPerVec;
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t row = (int64_t)blockIdx.x * kSoftmaxWavesPerWg + (threadIdx.x >> 6);
  if (row >= rows) return;
  const u32x4* xr = reinterpret_cast<const u32x4*>(x + row * x_pitch);
  u32x4* yr = reinterpret_cast<u32x4*>(y + row * y_pitch);
  const int nvec = RAGGED ? (n + V - 1) / V : n / V;

  // Straight-line code: vectors past the end of the row are loaded from the last valid
  // vector and replaced by -inf (the identity of the max stage; exp gives 0 for the sum
  // stage), so no stage below needs a branch.  Only the stores are predicated.
  // The row lives in registers as fp32 from here on: e[][] holds x, then exp(x - m).
  constexpr uint32_t kNegInf = std::is_same<T, float>::value ? 0xFF800000u : 0xFF80FF80u;
  // Full vectors sit at one lane address plus a constant; the vector that holds the end of the
  // row (and any vector past it) is read at a clamped address of its own.
  const u32x4* xl = xr + lane;
  const u32x4* xt = xr + min((nvec - 1) / kWave * kWave + lane, nvec - 1);
  float e[NCH][V];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int idx = c * kWave + lane;
    if constexpr (RAGGED) {
      Elem<T>::unpack(ragged_load(x + row * x_pitch, idx, n), e[c]);
      continue;
    }
    const bool full = (c + 1) * kWave <= nvec;  // wave-uniform
    u32x4 r = __builtin_nontemporal_load(full ? xl + c * kWave : xt);
    const bool ok = idx < nvec;
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = ok ? r[j] : kNegInf;
    Elem<T>::unpack(r, e[c]);
  }
  float m = -INFINITY;
  float l = 0.f;
  if constexpr (LANE_LEVEL) {
    // per-lane incremental state, then the merge; exponentials are taken again afterwards
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      if (c * kWave + lane < nvec) {
#pragma unroll
        for (int i = 0; i < V; ++i) {
          const float mn = fmaxf(m, e[c][i]);
          l = l * fast_exp2((m - mn) * kLog2e) + fast_exp2((e[c][i] - mn) * kLog2e);
          m = mn;
        }
      }
    }
    const float mw = wave_max(m);
    l = wave_sum((m == -INFINITY) ? 0.f : l * fast_exp2((m - mw) * kLog2e));
    m = mw;
    const float mb = -m * kLog2e;
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
      for (int i = 0; i < V; ++i) e[c][i] = fast_exp2(fmaf(e[c][i], kLog2e, mb));
  } else {
    // cascade stage 1: row max
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
      for (int i = 0; i < V; ++i) m = fmaxf(m, e[c][i]);
    m = wave_max(m);
    // cascade stage 2: sum of exp(x - m), exponentials kept for the epilogue
    const float mb = exponent_base(e, m);
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      if constexpr (RAGGED) l = ragged_exp_sum<V>(l, e[c], mb, c * kWave + lane, n, (c + 1) * kWave * V <= n);
      else l = exp_sum<V>(l, e[c], mb);
      __builtin_amdgcn_sched_barrier(0);  // one vector at a time: no extra live temporaries
    }
    l = wave_sum(l);
  }
  const float inv = 1.0f / l;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int idx = c * kWave + lane;
    if (idx < nvec) {
      float f[V];
#pragma unroll
      for (int i = 0; i < V; ++i) f[i] = e[c][i] * inv;
      if constexpr (RAGGED) ragged_store(y + row * y_pitch, idx, n, Elem<T>::pack(f));
      else __builtin_nontemporal_store(Elem<T>::pack(f), yr + idx);
    }
  }
}

// Short rows (at most LPR vectors of 16 bytes): 64 / LPR rows per wavefront, one vector per
// lane, the two reductions over the LPR lanes of a row by butterfly shuffles.  A wavefront per
// row would leave most lanes (and most of every 128-byte line fetched) idle.
template <typename T, int LPR, bool RAGGED>
__global__ __launch_bounds__(kSoftmaxWavesPerWg * kWave) void softmax_short_rows_kernel(
    const T* __restrict__ x, T* __restrict__ y, int64_t rows, int n, int64_t x_pitch,
    int64_t y_pitch) {
  constexpr int V = Elem<T>::kPerVec;
  constexpr int RPW = kWave / LPR;  // rows per wavefront
  constexpr uint32_t kNegInf = std::is_same<T, float>::value ? 0xFF800000u : 0xFF80FF80u;
  const int lane = threadIdx.x & (kWave - 1);
  const int sub = lane % LPR;       // vector index inside the row
  const int64_t row = ((int64_t)blockIdx.x * kSoftmaxWavesPerWg + (threadIdx.x >> 6)) * RPW + lane / LPR;
  const int nvec = RAGGED ? (n + V - 1) / V : n / V;
  const bool ok = row < rows && sub < nvec;
  u32x4 r;
  if constexpr (RAGGED) {
    r = ragged_load(x + (row < rows ? row : 0) * x_pitch, sub, n);
  } else {
    // lanes without a vector read a valid address (their own row's first vector, or row 0's)
    const u32x4* src = reinterpret_cast<const u32x4*>(x + (row < rows ? row : 0) * x_pitch) + (sub < nvec ? sub : 0);
    r = __builtin_nontemporal_load(src);
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = ok ? r[j] : kNegInf;
  }
  float e[V];
  Elem<T>::unpack(r, e);
  float m = e[0];
#pragma unroll
  for (int i = 1; i < V; ++i) m = fmaxf(m, e[i]);
#pragma unroll
  for (int off = LPR / 2; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off, kWave));
#pragma unroll
  for (int i = 0; i < V; ++i) e[i] -= m;  // (as exponent_base: here cheaper than a branch)
  float l = RAGGED ? ragged_exp_sum<V>(0.f, e, 0.f, sub, n, false) : exp_sum<V>(0.f, e, 0.f);
#pragma unroll
  for (int off = LPR / 2; off > 0; off >>= 1) l += __shfl_xor(l, off, kWave);
  const float inv = 1.0f / l;
#pragma unroll
  for (int i = 0; i < V; ++i) e[i] *= inv;
  if (ok) {
    if constexpr (RAGGED) ragged_store(y + row * y_pitch, sub, n, Elem<T>::pack(e));
    else __builtin_nontemporal_store(Elem<T>::pack(e), reinterpret_cast<u32x4*>(y + row * y_pitch) + sub);
  }
}

// Rows of less than one vector: a lane each, a wavefront per workgroup (pitched rows are a cache line
// each: spread over the chip).  With a workgroup per row 100000 rows of 5 bf16 values took 52 us, 2.8 here.
template <typename T>
__global__ __launch_bounds__(kWave) void softmax_tiny_rows_kernel(
    const T* __restrict__ x, T* __restrict__ y, int64_t rows, int n, int64_t x_pitch, int64_t y_pitch) {
  constexpr int N = Elem<T>::kPerVec - 1;
  const int64_t row = (int64_t)blockIdx.x * kWave + threadIdx.x;
  if (row >= rows) return;
  const T* xr = x + row * x_pitch;
  float e[N], m = -INFINITY, l = 0.f;
#pragma unroll
  for (int i = 0; i < N; ++i) {
    e[i] = i < n ? Elem<T>::load(xr + i) : -INFINITY;
    m = fmaxf(m, e[i]);
  }
#pragma unroll
  for (int i = 0; i < N; ++i) {
    e[i] = i < n ? fast_exp2((e[i] - m) * kLog2e) : 0.f;
    l += e[i];
  }
  const float inv = 1.0f / l;
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (i < n) Elem<T>::store(y + row * y_pitch + i, e[i] * inv);
}

// Long rows that still fit the registers of one workgroup (up to WAVES * 64 lanes * 64 values):
// one workgroup per row, the row read once and kept as fp32; the two reductions go through
// the wavefronts' DPP reductions and one LDS exchange each.
template <typename T, int NCH, int WAVES, bool RAGGED>
__global__ __launch_bounds__(WAVES * kWave) void softmax_row_in_regs_wg_kernel(
    const T* __restrict__ x, T* __restrict__ y, int64_t rows, int n, int64_t x_pitch,
    int64_t y_pitch) {
  constexpr int V = Elem<T>::kPerVec;
  constexpr int TH = WAVES * kWave;
  constexpr uint32_t kNegInf = std::is_same<T, float>::value ? 0xFF800000u : 0xFF80FF80u;
  __shared__ float s_max[WAVES], s_sum[WAVES];
  const int tid = threadIdx.x;
  const int64_t row = blockIdx.x;
  const u32x4* xr = reinterpret_cast<const u32x4*>(x + row * x_pitch);
  u32x4* yr = reinterpret_cast<u32x4*>(y + row * y_pitch);
  const int nvec = RAGGED ? (n + V - 1) / V : n / V;
  float e[NCH][V];
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int idx = c * TH + tid;
    if constexpr (RAGGED) {
      Elem<T>::unpack(ragged_load(x + row * x_pitch, idx, n), e[c]);
      continue;
    }
    u32x4 r = __builtin_nontemporal_load(xr + min(idx, nvec - 1));
    const bool ok = idx < nvec;
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = ok ? r[j] : kNegInf;
    Elem<T>::unpack(r, e[c]);
  }
  // cascade stage 1: row max
  float m = -INFINITY;
#pragma unroll
  for (int c = 0; c < NCH; ++c)
#pragma unroll
    for (int i = 0; i < V; ++i) m = fmaxf(m, e[c][i]);
  m = wave_max(m);
  if ((tid & (kWave - 1)) == 0) s_max[tid >> 6] = m;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < WAVES; ++w) m = fmaxf(m, s_max[w]);
  // cascade stage 2: sum of exp(x - m), exponentials kept for the epilogue
  const float mb = exponent_base(e, m);
  float l = 0.f;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    if constexpr (RAGGED) l = ragged_exp_sum<V>(l, e[c], mb, c * TH + tid, n, (c + 1) * TH * V <= n);
    else l = exp_sum<V>(l, e[c], mb);
  }
  l = wave_sum(l);
  if ((tid & (kWave - 1)) == 0) s_sum[tid >> 6] = l;
  __syncthreads();
  l = 0.f;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) l += s_sum[w];   // same order in every lane
  const float inv = 1.0f / l;
#pragma unroll
  for (int c = 0; c < NCH; ++c) {
    const int idx = c * TH + tid;
    if (idx < nvec) {
      float f[V];
#pragma unroll
      for (int i = 0; i < V; ++i) f[i] = e[c][i] * inv;
      if constexpr (RAGGED) ragged_store(y + row * y_pitch, idx, n, Elem<T>::pack(f));
      else __builtin_nontemporal_store(Elem<T>::pack(f), yr + idx);
    }
  }
}

// One workgroup per row, any n; two sweeps over the row (the second one is served by the
// L2 for rows of a few hundred KB).  Both sweeps use 128-bit accesses, at any alignment, and the
// incremental state is corrected once per vector; what is left of the row after the last whole
// vector is taken element by element.
constexpr int kStreamThreads = 256;
template <typename T>
__global__ __launch_bounds__(kStreamThreads) void softmax_row_streaming_kernel(
    const T* __restrict__ x, T* __restrict__ y, int64_t rows, int64_t n, int64_t x_pitch,
    int64_t y_pitch) {
  constexpr int V = Elem<T>::kPerVec;
  __shared__ float sm[kStreamThreads / kWave];
  __shared__ float sl[kStreamThreads / kWave];
  const int64_t row = blockIdx.x;
  if (row >= rows) return;
  const T* xr = x + row * x_pitch;
  T* yr = y + row * y_pitch;
  const int64_t nvec = n / V;   // full vectors; the rest is handled element-wise
  // Level-1 incremental state per lane.  The reference starts at kLowRef in place of -inf: against it
  // masked values (-inf or the type's lowest) give 0, as they have to once a larger one arrives, and no
  // exponent is formed from two infinities.
  constexpr float kLowRef = -2e38f;
  float m = kLowRef, l = 0.f;
  {
    const u32x4_any* xv = reinterpret_cast<const u32x4_any*>(xr);
    for (int64_t j = threadIdx.x; j < nvec; j += kStreamThreads) {
      float f[V];
      Elem<T>::unpack(xv[j], f);
      float vm = f[0];
#pragma unroll
      for (int i = 1; i < V; ++i) vm = fmaxf(vm, f[i]);
      const float mn = fmaxf(m, vm);
      const float mb = -mn * kLog2e;
      float sum = 0.f;
#pragma unroll
      for (int i = 0; i < V; ++i) sum += fast_exp2(fmaf(f[i], kLog2e, mb));
      l = l * fast_exp2((m - mn) * kLog2e) + sum;
      m = mn;
    }
  }
  for (int64_t j = nvec * V + threadIdx.x; j < n; j += kStreamThreads) {
    const float v = Elem<T>::load(xr + j);
    const float mn = fmaxf(m, v);
    l = l * fast_exp2((m - mn) * kLog2e) + fast_exp2((v - mn) * kLog2e);
    m = mn;
  }
  // merge lane states across the wavefront, then across wavefronts: l_c * exp(m_c - m)
  const int wave = threadIdx.x >> 6;
  auto all_max = [&](float v) {
    v = wave_max(v);
    if ((threadIdx.x & 63) == 0) sm[wave] = v;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kStreamThreads / kWave; ++w) v = fmaxf(v, sm[w]);
    return v;
  };
  auto all_sum = [&](float v) {
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) sl[wave] = v;
    __syncthreads();
    v = sl[0];
#pragma unroll
    for (int w = 1; w < kStreamThreads / kWave; ++w) v += sl[w];
    return v;
  };
  const float mg = all_max(m);
  if (!(mg > kLowRef && mg < -kLowRef)) {  // uniform
    // Nothing but masked values, or a maximum whose product with log2 e leaves fp32: one element at a
    // time, differences first.
    float mx = -INFINITY, t = 0.f;
    for (int64_t j = threadIdx.x; j < n; j += kStreamThreads) mx = fmaxf(mx, Elem<T>::load(xr + j));
    __syncthreads();  // the maxima of the first sweep have been read
    mx = all_max(mx);
    for (int64_t j = threadIdx.x; j < n; j += kStreamThreads) t += fast_exp2((Elem<T>::load(xr + j) - mx) * kLog2e);
    const float inv = 1.0f / all_sum(t);
    for (int64_t j = threadIdx.x; j < n; j += kStreamThreads)
      Elem<T>::store(yr + j, fast_exp2((Elem<T>::load(xr + j) - mx) * kLog2e) * inv);
    return;
  }
  const float inv = 1.0f / all_sum(l * fast_exp2((m - mg) * kLog2e));
  const float mb = -mg * kLog2e;
  {
    const u32x4_any* xv = reinterpret_cast<const u32x4_any*>(xr);
    u32x4_any* yv = reinterpret_cast<u32x4_any*>(yr);
    for (int64_t j = threadIdx.x; j < nvec; j += kStreamThreads) {
      float f[V];
      Elem<T>::unpack(xv[j], f);
#pragma unroll
      for (int i = 0; i < V; ++i) f[i] = fast_exp2(fmaf(f[i], kLog2e, mb)) * inv;
      __builtin_nontemporal_store(Elem<T>::pack(f), yv + j);
    }
  }
  for (int64_t j = nvec * V + threadIdx.x; j < n; j += kStreamThreads) {
    const float v = Elem<T>::load(xr + j);
    Elem<T>::store(yr + j, fast_exp2(fmaf(v, kLog2e, mb)) * inv);
  }
}

// RAGGED: rows that do not start on 16 bytes or do not hold a whole number of vectors.
template <typename T, bool RAGGED>
static hipError_t launch_softmax_t(const T* x, T* y, int64_t rows, int64_t n, int64_t x_pitch,
                                   int64_t y_pitch, hipStream_t s) {
  constexpr int V = Elem<T>::kPerVec;
  const int64_t per_chunk = (int64_t)V * kWave;
  if (n < V) {
    hipLaunchKernelGGL((softmax_tiny_rows_kernel<T>), dim3((unsigned)((rows + kWave - 1) / kWave)), dim3(kWave), 0, s, x, y,
                       rows, (int)n, x_pitch, y_pitch);
  } else if (n <= 32 * V) {
    // short rows: 2, 4, 8 or 16 rows per wavefront
    const int nvec = (int)((n + V - 1) / V);
    const int lpr = nvec <= 4 ? 4 : nvec <= 8 ? 8 : nvec <= 16 ? 16 : 32;
    const int64_t rows_per_wg = (int64_t)kSoftmaxWavesPerWg * (kWave / lpr);
    const unsigned grid = (unsigned)((rows + rows_per_wg - 1) / rows_per_wg);
    const dim3 block(kSoftmaxWavesPerWg * kWave);
#define RF_SOFTMAX_SHORT(L)                                                               \
  hipLaunchKernelGGL((softmax_short_rows_kernel<T, L, RAGGED>), dim3(grid), block, 0, s, x, y, rows, \
                     (int)n, x_pitch, y_pitch)
    if (lpr == 4) RF_SOFTMAX_SHORT(4);
    else if (lpr == 8) RF_SOFTMAX_SHORT(8);
    else if (lpr == 16) RF_SOFTMAX_SHORT(16);
    else RF_SOFTMAX_SHORT(32);
#undef RF_SOFTMAX_SHORT
  } else if (n <= (64 / V) * per_chunk) {
    // one wavefront per row, at most 64 values per lane
    const int nch = (int)((n + per_chunk - 1) / per_chunk);
    const unsigned grid = (unsigned)((rows + kSoftmaxWavesPerWg - 1) / kSoftmaxWavesPerWg);
    const dim3 block(kSoftmaxWavesPerWg * kWave);
#define RF_SOFTMAX_CASE(N)                                                              \
  hipLaunchKernelGGL((softmax_row_in_regs_kernel<T, N, RAGGED>), dim3(grid), block, 0, s, x, y, \
                     rows, (int)n, x_pitch, y_pitch)
    // (six and twelve between the powers of two: 4000 rows of 2560 bf16 values 9.2 -> 8.5 us)
    if (nch <= 1) RF_SOFTMAX_CASE(1);
    else if (nch <= 2) RF_SOFTMAX_CASE(2);
    else if (nch <= 3) RF_SOFTMAX_CASE(3);
    else if (nch <= 4) RF_SOFTMAX_CASE(4);
    else if (nch <= 6) RF_SOFTMAX_CASE(6);
    else if (nch <= 8) RF_SOFTMAX_CASE(8);
    else if (nch <= 12) RF_SOFTMAX_CASE(12);
    else RF_SOFTMAX_CASE(16);
#undef RF_SOFTMAX_CASE
  } else if (n <= 16 * 64 * (int64_t)kWave) {
    // 2 / 4 / 8 / 16 wavefronts of at most 64 values per lane (rows of 8K, 16K, 32K, 64K values);
    // rows of up to three quarters of that hold 48 values per lane, so that at most a third of
    // the lanes' vectors lie past the end (1000 rows of 20001 bf16 values: 20.1 -> 18.5 us; a
    // wavefront count fitted to the row instead leaves the SIMDs unevenly filled: 23.8 us).
    constexpr int NCHW = 64 / V;
    const int64_t per_wave = (int64_t)NCHW * V * kWave;   // 4096 values
    const int w = n <= 2 * per_wave ? 2 : n <= 4 * per_wave ? 4 : n <= 8 * per_wave ? 8 : 16;
    const bool few = 4 * n <= 3 * w * per_wave;
#define RF_SOFTMAX_WG(W)                                                                           \
  if (w == W && few)                                                                               \
    hipLaunchKernelGGL((softmax_row_in_regs_wg_kernel<T, NCHW * 3 / 4, W, RAGGED>), dim3((unsigned)rows), \
                       dim3(W * kWave), 0, s, x, y, rows, (int)n, x_pitch, y_pitch);               \
  else if (w == W)                                                                                 \
    hipLaunchKernelGGL((softmax_row_in_regs_wg_kernel<T, NCHW, W, RAGGED>), dim3((unsigned)rows),  \
                       dim3(W * kWave), 0, s, x, y, rows, (int)n, x_pitch, y_pitch);
    RF_SOFTMAX_WG(2) RF_SOFTMAX_WG(4) RF_SOFTMAX_WG(8) RF_SOFTMAX_WG(16)
#undef RF_SOFTMAX_WG
  } else {  // longer rows
    hipLaunchKernelGGL((softmax_row_streaming_kernel<T>), dim3((unsigned)rows),
                       dim3(kStreamThreads), 0, s, x, y, rows, n, x_pitch, y_pitch);
  }
  return hipGetLastError();
}

// ---- fusion-level study (Section 5.3): the unfused chain as three kernels ----
// One wavefront per row, 128-bit loads; m and l pass through memory between the kernels.
// PASS 0: m = max x;  PASS 1: l = sum exp(x - m);  PASS 2: y = exp(x - m) / l.
template <typename T, int PASS>
__global__ __launch_bounds__(kSoftmaxWavesPerWg * kWave) void softmax_unfused_pass_kernel(
    const T* __restrict__ x, T* __restrict__ y, float* __restrict__ m_buf, float* __restrict__ l_buf,
    int64_t rows, int n, int64_t x_pitch, int64_t y_pitch) {
  constexpr int V = Elem<T>::kPerVec;
  const int lane = threadIdx.x & (kWave - 1);
  const int64_t row = (int64_t)blockIdx.x * kSoftmaxWavesPerWg + (threadIdx.x >> 6);
  if (row >= rows) return;
  const u32x4* xr = reinterpret_cast<const u32x4*>(x + row * x_pitch);
  u32x4* yr = reinterpret_cast<u32x4*>(y + row * y_pitch);
  const int nvec = n / V;
  float acc = PASS == 0 ? -INFINITY : 0.f;
  const float mb = PASS == 0 ? 0.f : -m_buf[row] * kLog2e;
  const float inv = PASS == 2 ? 1.0f / l_buf[row] : 0.f;
  for (int idx = lane; idx < nvec; idx += kWave) {
    float f[V];
    Elem<T>::unpack(xr[idx], f);
    if constexpr (PASS == 0) {
#pragma unroll
      for (int i = 0; i < V; ++i) acc = fmaxf(acc, f[i]);
    } else if constexpr (PASS == 1) {
#pragma unroll
      for (int i = 0; i < V; ++i) acc += fast_exp2(fmaf(f[i], kLog2e, mb));
    } else {
#pragma unroll
      for (int i = 0; i < V; ++i) f[i] = fast_exp2(fmaf(f[i], kLog2e, mb)) * inv;
      yr[idx] = Elem<T>::pack(f);
    }
  }
  if constexpr (PASS == 0) { acc = wave_max(acc); if (lane == 0) m_buf[row] = acc; }
  if constexpr (PASS == 1) { acc = wave_sum(acc); if (lane == 0) l_buf[row] = acc; }
}

// ---- fusion-level study: fused across workgroups (the paper's inter-block level) ----
// A row is cut into kInterBlockSegs segments, one wavefront (of different workgroups) each.
// Kernel 1 reads its segment once and stores the segment's fused state (m_s, l_s); kernel 2
// merges the row's states with the level-k expression (Eq. (11)), reads its segment again and
// writes y.  Two reads of x and a round trip of the states through memory: the cost the paper
// attributes to this level.  m_buf, l_buf: rows * kInterBlockSegs floats each.
constexpr int kInterBlockSegs = 4;
template <typename T, int PASS>
__global__ __launch_bounds__(kSoftmaxWavesPerWg * kWave) void softmax_interblock_kernel(
    const T* __restrict__ x, T* __restrict__ y, float* __restrict__ m_buf, float* __restrict__ l_buf,
    int64_t rows, int n, int64_t x_pitch, int64_t y_pitch) {
  constexpr int V = Elem<T>::kPerVec;
  const int lane = threadIdx.x & (kWave - 1);
  // consecutive wavefronts of a workgroup take different rows: the segments of one row run in
  // different workgroups
  const int64_t unit = (int64_t)blockIdx.x * kSoftmaxWavesPerWg + (threadIdx.x >> 6);
  const int seg = (int)(unit / rows);
  const int64_t row = unit % rows;
  if (seg >= kInterBlockSegs) return;
  const int nvec = n / V;
  const int per_seg = (nvec + kInterBlockSegs - 1) / kInterBlockSegs;
  const int v0 = seg * per_seg, v1 = min(nvec, v0 + per_seg);
  const u32x4* xr = reinterpret_cast<const u32x4*>(x + row * x_pitch);
  if constexpr (PASS == 0) {
    // the segment's state, level-1 incremental form per lane, lanes merged with Eq. (11)
    float m = -INFINITY, l = 0.f;
    for (int idx = v0 + lane; idx < v1; idx += kWave) {
      float f[V];
      Elem<T>::unpack(xr[idx], f);
      float vm = f[0];
#pragma unroll
      for (int i = 1; i < V; ++i) vm = fmaxf(vm, f[i]);
      const float m_new = fmaxf(m, vm);
      float part = 0.f;
#pragma unroll
      for (int i = 0; i < V; ++i) part += fast_exp2((f[i] - m_new) * kLog2e);
      l = l * ((m == -INFINITY) ? 0.f : fast_exp2((m - m_new) * kLog2e)) + part;
      m = m_new;
    }
    const float mw = wave_max(m);
    const float lw = wave_sum((m == -INFINITY) ? 0.f : l * fast_exp2((m - mw) * kLog2e));
    if (lane == 0) { m_buf[row * kInterBlockSegs + seg] = mw; l_buf[row * kInterBlockSegs + seg] = lw; }
  } else {
    float ms[kInterBlockSegs], ls[kInterBlockSegs];
    float m = -INFINITY;
#pragma unroll
    for (int c = 0; c < kInterBlockSegs; ++c) {
      ms[c] = m_buf[row * kInterBlockSegs + c];
      ls[c] = l_buf[row * kInterBlockSegs + c];
      m = fmaxf(m, ms[c]);
    }
    float l = 0.f;
#pragma unroll
    for (int c = 0; c < kInterBlockSegs; ++c) l += (ms[c] == -INFINITY) ? 0.f : ls[c] * fast_exp2((ms[c] - m) * kLog2e);
    const float inv = 1.0f / l, mb = -m * kLog2e;
    u32x4* yr = reinterpret_cast<u32x4*>(y + row * y_pitch);
    for (int idx = v0 + lane; idx < v1; idx += kWave) {
      float f[V];
      Elem<T>::unpack(xr[idx], f);
#pragma unroll
      for (int i = 0; i < V; ++i) f[i] = fast_exp2(fmaf(f[i], kLog2e, mb)) * inv;
      yr[idx] = Elem<T>::pack(f);
    }
  }
}

// level 0: unfused (three kernels, needs ml_buf = 2 * rows floats); 1: fused per lane;
// 2: fused per wavefront (the shipped kernel for rows of up to 4096 values); 3: fused per workgroup (the streaming kernel);
// 4: fused across workgroups (two kernels, needs ml_buf = 8 * rows floats).
// bf16 only, n a multiple of 8 and at most 8192, 16-byte aligned rows.
hipError_t launch_softmax_level(const void* x, void* y, int64_t rows, int64_t n, int64_t x_pitch,
                                int64_t y_pitch, int level, float* ml_buf, hipStream_t s) {
  typedef bf16_t T;
  const T* xp = (const T*)x;
  T* yp = (T*)y;
  const int64_t per_chunk = (int64_t)Elem<T>::kPerVec * kWave;
  if (n % Elem<T>::kPerVec != 0 || n > 16 * per_chunk || level < 0 || level > 4) return hipErrorInvalidValue;
  const unsigned grid = (unsigned)((rows + kSoftmaxWavesPerWg - 1) / kSoftmaxWavesPerWg);
  const dim3 block(kSoftmaxWavesPerWg * kWave);
  if (level == 0) {
    if (ml_buf == nullptr) return hipErrorInvalidValue;
    hipLaunchKernelGGL((softmax_unfused_pass_kernel<T, 0>), dim3(grid), block, 0, s, xp, yp, ml_buf, ml_buf + rows, rows, (int)n, x_pitch, y_pitch);
    hipLaunchKernelGGL((softmax_unfused_pass_kernel<T, 1>), dim3(grid), block, 0, s, xp, yp, ml_buf, ml_buf + rows, rows, (int)n, x_pitch, y_pitch);
    hipLaunchKernelGGL((softmax_unfused_pass_kernel<T, 2>), dim3(grid), block, 0, s, xp, yp, ml_buf, ml_buf + rows, rows, (int)n, x_pitch, y_pitch);
  } else if (level == 1 || level == 2) {
    const int nch = (int)((n + per_chunk - 1) / per_chunk);
#define RF_SOFTMAX_LEVEL_CASE(N)                                                                    \
  if (level == 1)                                                                                   \
    hipLaunchKernelGGL((softmax_row_in_regs_kernel<T, N, false, true>), dim3(grid), block, 0, s, xp, yp,   \
                       rows, (int)n, x_pitch, y_pitch);                                             \
  else                                                                                              \
    hipLaunchKernelGGL((softmax_row_in_regs_kernel<T, N, false, false>), dim3(grid), block, 0, s, xp, yp,  \
                       rows, (int)n, x_pitch, y_pitch)
    if (nch <= 1) { RF_SOFTMAX_LEVEL_CASE(1); }
    else if (nch <= 2) { RF_SOFTMAX_LEVEL_CASE(2); }
    else if (nch <= 4) { RF_SOFTMAX_LEVEL_CASE(4); }
    else if (nch <= 8) { RF_SOFTMAX_LEVEL_CASE(8); }
    else { RF_SOFTMAX_LEVEL_CASE(16); }
#undef RF_SOFTMAX_LEVEL_CASE
  } else if (level == 3) {
    hipLaunchKernelGGL((softmax_row_streaming_kernel<T>), dim3((unsigned)rows), dim3(kStreamThreads), 0, s,
                       xp, yp, rows, n, x_pitch, y_pitch);
  } else {
    if (ml_buf == nullptr) return hipErrorInvalidValue;
    const int64_t units = rows * kInterBlockSegs;
    const int64_t g4 = (units + kSoftmaxWavesPerWg - 1) / kSoftmaxWavesPerWg;
    if (g4 > INT32_MAX) return hipErrorInvalidValue;
    float* lb = ml_buf + rows * kInterBlockSegs;
    hipLaunchKernelGGL((softmax_interblock_kernel<T, 0>), dim3((unsigned)g4), block, 0, s, xp, yp, ml_buf, lb, rows, (int)n, x_pitch, y_pitch);
    hipLaunchKernelGGL((softmax_interblock_kernel<T, 1>), dim3((unsigned)g4), block, 0, s, xp, yp, ml_buf, lb, rows, (int)n, x_pitch, y_pitch);
  }
  return hipGetLastError();
}

hipError_t launch_softmax(const void* x, void* y, bool is_bf16, int64_t rows, int64_t n,
                          int64_t x_pitch, int64_t y_pitch, bool vec_ok, hipStream_t s) {
  const int64_t v = is_bf16 ? Elem<bf16_t>::kPerVec : Elem<float>::kPerVec;
  const bool ragged = !vec_ok || n % v != 0;
#define RF_SOFTMAX(T, R) launch_softmax_t<T, R>((const T*)x, (T*)y, rows, n, x_pitch, y_pitch, s)
  if (is_bf16) return ragged ? RF_SOFTMAX(bf16_t, true) : RF_SOFTMAX(bf16_t, false);
  return ragged ? RF_SOFTMAX(float, true) : RF_SOFTMAX(float, false);
#undef RF_SOFTMAX
}

}  // namespace rf
