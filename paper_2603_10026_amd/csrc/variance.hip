// Mean and population variance over the last axis: the cascade
//   m = (1/L) sum_l x[l];   var = (1/L) sum_l (x[l] - m)^2
// (paper Appendix, evaluation on non-ML workloads) in single-pass form.
//
// The second map (x - m)^2 is not G(x) (x) H(m) for one pair of operators;
// expanding the square gives decomposable terms, and carrying them as
// (count, mean, M2 = sum (x - mean)^2) gives a running state whose merge is
//   n = n_a + n_b;  d = mean_b - mean_a;  mean = mean_a + d n_b / n;
//   M2 = M2_a + M2_b + d^2 n_a n_b / n
// (the level-k fused expression of Section 3.2 for this cascade; the cross term
// of the expanded square vanishes).  It is associative and commutative, so the
// same operator merges vectors, lanes, wavefronts.
//
// Short rows take a wavefront or less each (variance_rows_kernel), those of less than one vector a lane.  For longer ones,
// one workgroup (4 wavefronts, or 16 when rows are few and long) streams one row once.  Every lane turns each
// 128-bit vector into an exact state (two passes over 4 or 8 registers), merges
// the eight vectors of a chunk pairwise (equal counts: no division), and folds
// the result into its running state (what is left of a row after the full chunks
// goes through chunks of 4, 2 and 1 vectors per lane); lanes merge through DPP / shuffles,
// wavefronts through LDS.  HBM traffic is one read of x.  Rows may start at any element: all
// loads are 16-byte vectors at whatever alignment that gives.
#include <math.h>

#include <type_traits>

#include "rf_device.h"
#include "rf_launch.h"

namespace rf {

namespace {

struct VarState {
  float n, mean, m2;
};

__device__ __forceinline__ VarState var_merge(const VarState& a, const VarState& b) {
  VarState r;
  r.n = a.n + b.n;
  const float inv = r.n > 0.f ? fast_rcp(r.n) : 0.f;  // empty + empty stays empty
  const float d = b.mean - a.mean;
  const float wb = b.n * inv;
  r.mean = fmaf(d, wb, a.mean);
  r.m2 = a.m2 + b.m2 + d * d * a.n * wb;
  return r;
}
// both sides hold the same, non-zero count
__device__ __forceinline__ VarState var_merge_equal(const VarState& a, const VarState& b) {
  VarState r;
  const float d = b.mean - a.mean;
  r.n = a.n + a.n;
  r.mean = fmaf(d, 0.5f, a.mean);
  r.m2 = a.m2 + b.m2 + d * d * (0.5f * a.n);
  return r;
}
// Exact state of the first `cnt` of V values held in registers.  (Here and below the values are scaled by
// 1 / V, a power of two, before they are added up: the same bits, and no sum past the end of fp32.)
template <int V>
__device__ __forceinline__ VarState var_of_vector(const float* f, int cnt) {
  VarState r;
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < V; ++i) s = (i < cnt) ? fmaf(f[i], 1.0f / V, s) : s;
  r.n = (float)cnt;
  r.mean = cnt > 0 ? s * ((float)V / (float)cnt) : 0.f;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < V; ++i) {
    const float d = f[i] - r.mean;
    q += (i < cnt) ? d * d : 0.f;
  }
  r.m2 = q;
  return r;
}
template <int V>
__device__ __forceinline__ VarState var_of_full_vector(const float* f) {
  VarState r;
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < V; ++i) s = fmaf(f[i], 1.0f / V, s);
  r.n = (float)V;
  r.mean = s;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < V; ++i) {
    const float d = f[i] - r.mean;
    q = fmaf(d, d, q);
  }
  r.m2 = q;
  return r;
}

__device__ __forceinline__ VarState var_shfl_xor(const VarState& a, int mask) {
  VarState b;
  b.n = __shfl_xor(a.n, mask, 64);
  b.mean = __shfl_xor(a.mean, mask, 64);
  b.m2 = __shfl_xor(a.m2, mask, 64);
  return b;
}

constexpr int kVarRowsThreads = 256;
constexpr int kVarUnroll = 8;  // 128-bit loads in flight per lane in a full chunk

}  // namespace

// Rows of one to 512 vectors: LPR lanes hold a row in registers, NCH
// vectors each, and take the two stages one after the other, each over registers and reduced by
// shuffles over the lanes of the row.  The workgroup-per-row kernel below spends such a row's time
// on its barrier and its state merges and leaves lanes idle: 16384 rows of 1000 bf16 values
// 20.5 us there, 7.4 here; 32768 rows of 64 fp32 values 30.2 and 3.0.
// Rows may start at any element: vector idx covers elements idx V .., and the one that would
// reach past the end is moved back to the last V elements, where it repeats elements of its
// neighbour, which both sums leave out.
template <typename T, int NCH, int LPR>
__global__ __launch_bounds__(kVarRowsThreads) void variance_rows_kernel(
    const T* __restrict__ x, float* __restrict__ mean_out, float* __restrict__ var_out, int64_t rows, int n,
    int64_t x_pitch) {
  constexpr int V = Elem<T>::kPerVec;
  const int lane = threadIdx.x & (kWave - 1);
  const int sub = lane % LPR;
  const int64_t row = ((int64_t)blockIdx.x * (kVarRowsThreads / kWave) + (threadIdx.x >> 6)) * (kWave / LPR) + lane / LPR;
  const T* xr = x + min(row, rows - 1) * x_pitch;
  float f[NCH][V];
#pragma unroll
  for (int c = 0; c < NCH; ++c)
    Elem<T>::unpack(__builtin_nontemporal_load(reinterpret_cast<const u32x4_any*>(xr + min((c * LPR + sub) * V, n - V))), f[c]);
  auto lanes_sum = [](float v) {
#pragma unroll
    for (int off = LPR / 2; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
  };
  // sum over the row of g(element); chunks that no vector leaves are summed without masks
  auto row_sum = [&](auto g) {
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      float part = 0.f;
      if ((c + 1) * LPR * V <= n) {  // uniform
#pragma unroll
        for (int i = 0; i < V; ++i) part += g(f[c][i]);
      } else {
        const int e0 = (c * LPR + sub) * V;
        const int first = e0 - min(e0, n - V);  // elements below it are the neighbour's (V or more: none is ours)
#pragma unroll
        for (int i = 0; i < V; ++i) part += i >= first ? g(f[c][i]) : 0.f;
      }
      s += part;
    }
    return lanes_sum(s);
  };
  const float inv_n = 1.0f / (float)n;
  float mean = row_sum([](float v) { return v; }) * inv_n;
  // (a sum past the end of fp32 is not a mean past it: the terms are divided first then.  All lanes of
  // a row agree.)
  if (!(fabsf(mean) < INFINITY)) mean = row_sum([inv_n](float v) { return v * inv_n; });
  const float m2 = row_sum([mean](float v) { return (v - mean) * (v - mean); });
  if (sub == 0 && row < rows) {
    mean_out[row] = mean;
    var_out[row] = m2 * inv_n;
  }
}

// Rows of less than one vector: a lane each.  (A workgroup per row, 100000 rows of 5 bf16 values: 107 us,
// 2.6 here.)
template <typename T>
__global__ __launch_bounds__(kWave) void variance_tiny_rows_kernel(
    const T* __restrict__ x, float* __restrict__ mean_out, float* __restrict__ var_out, int64_t rows, int n,
    int64_t x_pitch) {
  constexpr int V = Elem<T>::kPerVec;
  const int64_t row = (int64_t)blockIdx.x * kWave + threadIdx.x;
  if (row >= rows) return;
  const T* xr = x + row * x_pitch;
  float f[V];
#pragma unroll
  for (int i = 0; i < V; ++i) f[i] = i < n ? Elem<T>::load(xr + i) : 0.f;
  const VarState st = var_of_vector<V>(f, n);
  mean_out[row] = st.mean;
  var_out[row] = st.m2 / (float)n;
}

// Longer rows.  kVarWaves wavefronts share a row: 4 when there are enough rows to fill the GPU, 16
// when there are few (each row then needs more loads in flight to be read at speed).
template <typename T, int kVarWaves>
__global__ __launch_bounds__(kVarWaves * kWave) void variance_kernel(const T* __restrict__ x,
                                                                     float* __restrict__ mean_out,
                                                                     float* __restrict__ var_out,
                                                                     int64_t n, int64_t x_pitch) {
  constexpr int kVarThreads = kVarWaves * kWave;
  constexpr int V = Elem<T>::kPerVec;
  __shared__ float s_n[kVarWaves], s_mean[kVarWaves], s_m2[kVarWaves];
  const int tid = threadIdx.x;
  const int64_t row = blockIdx.x;
  const T* xr = x + row * x_pitch;

  VarState st{0.f, 0.f, 0.f};
  {
    const u32x4_any* xv = reinterpret_cast<const u32x4_any*>(xr);
    const int64_t nvec = n / V;  // full vectors
    int64_t base = 0;
    // a chunk: every lane owns U full vectors, all U loads in flight together
    auto chunk = [&](auto utag) {
      constexpr int U = decltype(utag)::value;
      u32x4 raw[U];
#pragma unroll
      for (int u = 0; u < U; ++u) raw[u] = __builtin_nontemporal_load(xv + base + u * kVarThreads + tid);
      VarState c[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        float f[V];
        Elem<T>::unpack(raw[u], f);
        c[u] = var_of_full_vector<V>(f);
      }
      // pairwise tree over the equal-count states
#pragma unroll
      for (int w = 1; w < U; w <<= 1) {
#pragma unroll
        for (int u = 0; u < U; u += 2 * w) c[u] = var_merge_equal(c[u], c[u + w]);
      }
      st = var_merge(st, c[0]);
      base += (int64_t)U * kVarThreads;
    };
    while (base + (int64_t)kVarUnroll * kVarThreads <= nvec) chunk(std::integral_constant<int, kVarUnroll>{});
    if (base + 4 * (int64_t)kVarThreads <= nvec) chunk(std::integral_constant<int, 4>{});
    if (base + 2 * (int64_t)kVarThreads <= nvec) chunk(std::integral_constant<int, 2>{});
    if (base + (int64_t)kVarThreads <= nvec) chunk(std::integral_constant<int, 1>{});
    // fewer than one vector per lane left, then the ragged tail (fewer than V elements)
    if (base + tid < nvec) {
      float f[V];
      Elem<T>::unpack(__builtin_nontemporal_load(xv + base + tid), f);
      st = var_merge(st, var_of_full_vector<V>(f));
    }
    const int64_t tail0 = nvec * V;
    if (tid == 0 && tail0 < n) {
      float f[V];
#pragma unroll
      for (int i = 0; i < V; ++i) f[i] = (tail0 + i < n) ? Elem<T>::load(xr + tail0 + i) : 0.f;
      st = var_merge(st, var_of_vector<V>(f, (int)(n - tail0)));
    }
  }

  // merge the 64 lane states, then the wavefront states
#pragma unroll
  for (int mask = 1; mask < 64; mask <<= 1) st = var_merge(st, var_shfl_xor(st, mask));
  const int wave = tid >> 6;
  if ((tid & 63) == 0) { s_n[wave] = st.n; s_mean[wave] = st.mean; s_m2[wave] = st.m2; }
  __syncthreads();
  if (tid == 0) {
    VarState r{s_n[0], s_mean[0], s_m2[0]};
#pragma unroll
    for (int w = 1; w < kVarWaves; ++w) r = var_merge(r, VarState{s_n[w], s_mean[w], s_m2[w]});
    mean_out[row] = r.mean;
    var_out[row] = r.m2 / (float)n;
  }
}

template <typename T>
static hipError_t launch_variance_t(const T* x, float* mean, float* var, int64_t rows, int64_t n,
                                    int64_t x_pitch, hipStream_t s) {
  constexpr int V = Elem<T>::kPerVec;
  if (n < V) {
    hipLaunchKernelGGL((variance_tiny_rows_kernel<T>), dim3((unsigned)((rows + kWave - 1) / kWave)), dim3(kWave), 0, s, x, mean, var, rows, (int)n, x_pitch);
    return hipGetLastError();
  }
  const int64_t nvec64 = (n + V - 1) / V;
  // A wavefront per row up to 6 vectors a lane (1.0 to 5 times the workgroup's speed for 16 to
  // 16384 rows), up to 8 where there are rows to fill the GPU (2 times at 16384 rows of 4095 bf16
  // values, 0.96 at 256); with more, too few wavefronts fit the registers (16384 x 4095 fp32: 0.96).
  if (nvec64 <= (rows >= 1024 ? 8 : 6) * kWave) {
    const int nvec = (int)nvec64;
    const int lpr = nvec <= 4 ? 4 : nvec <= 8 ? 8 : nvec <= 16 ? 16 : nvec <= 32 ? 32 : 64;
    const int nch = (nvec + lpr - 1) / lpr;  // 1 for less than 64 lanes
    const int64_t rows_per_wg = (kVarRowsThreads / kWave) * (kWave / lpr);
    const dim3 grid((unsigned)((rows + rows_per_wg - 1) / rows_per_wg)), block(kVarRowsThreads);
#define RF_VAR_ROWS(NCH, LPR)                                                                        \
  hipLaunchKernelGGL((variance_rows_kernel<T, NCH, LPR>), grid, block, 0, s, x, mean, var, rows, (int)n, x_pitch)
    if (lpr == 4) RF_VAR_ROWS(1, 4);
    else if (lpr == 8) RF_VAR_ROWS(1, 8);
    else if (lpr == 16) RF_VAR_ROWS(1, 16);
    else if (lpr == 32) RF_VAR_ROWS(1, 32);
    else if (nch <= 1) RF_VAR_ROWS(1, 64);
    else if (nch <= 2) RF_VAR_ROWS(2, 64);
    else if (nch <= 3) RF_VAR_ROWS(3, 64);
    else if (nch <= 4) RF_VAR_ROWS(4, 64);
    else if (nch <= 6) RF_VAR_ROWS(6, 64);
    else RF_VAR_ROWS(8, 64);
#undef RF_VAR_ROWS
    return hipGetLastError();
  }
  // Few long rows: 16 wavefronts per row instead of 4.  Measured per call under graph replay:
  // 128 rows of 32768 go from 8.5 to 6.0 us, one such row from 4.2 to 3.8; rows of 8192 are
  // faster with 4 wavefronts (2.7 against 3.2 us), and so are 512 rows or more of any length.
  const bool wide = rows <= 256 && n >= 16384;
  const dim3 grid((unsigned)rows), block((wide ? 16 : 4) * kWave);
  if (wide) hipLaunchKernelGGL((variance_kernel<T, 16>), grid, block, 0, s, x, mean, var, n, x_pitch);
  else hipLaunchKernelGGL((variance_kernel<T, 4>), grid, block, 0, s, x, mean, var, n, x_pitch);
  return hipGetLastError();
}

hipError_t launch_variance(const void* x, bool is_bf16, float* mean, float* var, int64_t rows,
                           int64_t n, int64_t x_pitch, hipStream_t s) {
  if (rows > INT32_MAX) return hipErrorInvalidValue;
  return is_bf16 ? launch_variance_t((const bf16_t*)x, mean, var, rows, n, x_pitch, s)
                 : launch_variance_t((const float*)x, mean, var, rows, n, x_pitch, s);
}

}  // namespace rf
