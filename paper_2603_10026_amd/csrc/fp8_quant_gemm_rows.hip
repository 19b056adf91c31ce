// FP8 per-token quantisation + GEMM for few tokens (a decode batch): the cascade of
// fp8_quant_gemm.hip, cut for launches whose time is the trip of w from memory.
//
//   m_i = max_k |a[i,k]|;   c[i,n] = sum_k q(MAX a[i,k] / m_i) w[n,k],   MAX = 448
//
// A 128 x 256 tile of the large kernel leaves all but N / 256 compute units idle here.  This one
// cuts the output into 16 MT tokens x 16 NT channels and gives every workgroup the whole
// contraction axis, its 128-k tiles dealt to 8 wavefronts in runs:
//
//   C^T = W A_q^T      A = W rows, B = quantised tokens (16x16x128 FP8 MFMA, fp32 accumulate)
//
// w goes from memory into the A operand as it lies there (a lane's 32 bytes of its row), and a
// wavefront quantises the token values of its tiles straight into the B operand: no wavefront
// needs another one's values, so nothing but maxima and sums goes through LDS.
//   1. A wavefront requests all token values of its run (they stay in registers) and its first
//      weight tiles, takes max |a| of its tiles and tells the others the maximum of the run.
//   2. A tile is quantised with the prefix maximum that includes it, the same codes the large
//      kernel forms; the sums are rescaled where the maximum moved.  A wavefront's sums are in
//      units of its own last maximum; they are added up in units of the token's (as in the large
//      kernel, only the result has to be in range).
#include <math.h>

#include "rf_device.h"
#include "rf_launch.h"

namespace rf {

namespace {
constexpr int kFWaves = 8;
constexpr int kFThreads = kFWaves * kWave;
constexpr int kFRedTiles = 4;  // 16 x 16 output tiles that go through the reduction buffer at once
typedef __attribute__((__vector_size__(4 * sizeof(int)))) int i32x4;

__device__ __forceinline__ int quant4(uint32_t p0, uint32_t p1, float s) {
  int t = 0;
  t = __builtin_amdgcn_cvt_pk_fp8_f32(bf16_lo(p0) * s, bf16_hi(p0) * s, t, false);
  t = __builtin_amdgcn_cvt_pk_fp8_f32(bf16_lo(p1) * s, bf16_hi(p1) * s, t, true);
  return t;
}
}  // namespace

// TPW: tiles a wavefront can hold (K <= 1024 TPW); PW: weight tiles in flight
template <int MT, int NT, int TPW, int PW>
__global__ __launch_bounds__(kFThreads, 2) void fp8_quant_gemm_rows_kernel(
    const bf16_t* __restrict__ a, const unsigned char* __restrict__ w, bf16_t* __restrict__ c, int M,
    int K, int N, int64_t lda, int64_t ldw, int64_t ldc, int n_mtiles) {
  constexpr float kE4M3Max = 448.0f;
  constexpr int kTiles = NT * MT;
  constexpr int kG = kTiles < kFRedTiles ? kTiles : kFRedTiles;
  static_assert(kTiles % kG == 0 && TPW % PW == 0, "whole groups of tiles");
  __shared__ float s_max[kFWaves][16 * MT], s_all[16 * MT];
  __shared__ f32x4 s_red[kFWaves * kG * kWave];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15;
  const int g4 = lane >> 4;

  // Workgroups are dealt round-robin to the 8 XCDs, each with its own L2: the token tiles that
  // read the same channels of w go to one XCD, one after the other.
  const int j = blockIdx.x >> 3;
  const int mt = __builtin_amdgcn_readfirstlane(j % n_mtiles);
  const int nt = __builtin_amdgcn_readfirstlane(j / n_mtiles * 8 + (blockIdx.x & 7));
  const int m0 = mt * 16 * MT, n0 = nt * 16 * NT;
  if (n0 >= N) return;
  const int nk = K / 128;
  const int run = (nk + kFWaves - 1) / kFWaves;  // <= TPW
  const int t0 = wave * run;
  const int mine = max(0, min(run, nk - t0));

  // Slot (g4, byte j) of a 128-k MFMA stands for k = 16 g4 + j (j < 16) or 64 + 16 g4 + j - 16 on
  // both operands: a load of w then covers 64 contiguous bytes of each of its 16 rows.
  // Rows past the end repeat the last one; their results are not stored.
  uint32_t w_lane[NT], a_lane[MT];
#pragma unroll
  for (int n = 0; n < NT; ++n)
    w_lane[n] = (uint32_t)((int64_t)min(n0 + 16 * n + i16, N - 1) * ldw + 16 * g4);
#pragma unroll
  for (int t = 0; t < MT; ++t)
    a_lane[t] = (uint32_t)(((int64_t)min(16 * t + i16, M - 1 - m0) * lda + 16 * g4) * 2);
  const char* abase = reinterpret_cast<const char*>(a + (int64_t)m0 * lda);
  const char* wbase = reinterpret_cast<const char*>(w);
  // (surplus requests re-read the last tile of the run, of the matrix for an empty run)
  auto tile = [&](int i) { return min(t0 + min(i, max(mine - 1, 0)), nk - 1); };

  u32x4 xr[TPW][MT][4], wr[PW][NT][2];
  auto load_w = [&](int p, int i) {
    const char* wt = wbase + (int64_t)tile(i) * 128;
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      wr[p][n][0] = *reinterpret_cast<const u32x4*>(wt + w_lane[n]);
      wr[p][n][1] = *reinterpret_cast<const u32x4*>(wt + w_lane[n] + 64);
    }
  };
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    const char* at = abase + (int64_t)tile(i) * 256;
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
      for (int h = 0; h < 4; ++h)
        xr[i][t][h] = *reinterpret_cast<const u32x4*>(at + a_lane[t] + 128 * (h >> 1) + 16 * (h & 1));
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int p = 0; p < PW; ++p) load_w(p, p);
  __builtin_amdgcn_sched_barrier(0);

  // ---- maxima ----
  // For non-negative values the bf16 bit patterns order like unsigned integers: the maximum is
  // taken on packed 16-bit integers with the sign bits cleared.
  float am[TPW][MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < TPW; ++i) {
      typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
      u16x2 v = __builtin_bit_cast(u16x2, xr[i][t][0][0] & 0x7fff7fffu);
#pragma unroll
      for (int h = 0; h < 4; ++h)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          v = __builtin_elementwise_max(v, __builtin_bit_cast(u16x2, xr[i][t][h][e] & 0x7fff7fffu));
      float x = __uint_as_float((uint32_t)(v[0] > v[1] ? v[0] : v[1]) << 16);
      x = i < mine ? x : 0.f;
      x = fmaxf(x, __shfl_xor(x, 16, 64));
      x = fmaxf(x, __shfl_xor(x, 32, 64));
      m = fmaxf(m, x);
      am[i][t] = m;  // prefix maximum inside the run
    }
    if (g4 == 0) s_max[wave][16 * t + i16] = m;
  }
  __syncthreads();

  // ---- products ----
  f32x4 acc[NT][MT];  // acc[n][t][r] = C[token 16 t + i16][channel 16 n + 4 g4 + r], in units of m_run[t]
  float before[MT], all[MT], m_run[MT], qscale[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    before[t] = 0.f;
    all[t] = 0.f;
#pragma unroll
    for (int wv = 0; wv < kFWaves; ++wv) {
      const float o = s_max[wv][16 * t + i16];
      before[t] = wv < wave ? fmaxf(before[t], o) : before[t];
      all[t] = fmaxf(all[t], o);
    }
    if (wave == 0 && g4 == 0) s_all[16 * t + i16] = all[t];
    m_run[t] = 0.f;
    qscale[t] = 0.f;
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[n][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
#pragma unroll
  for (int i = 0; i < TPW; ++i) {
    if (i < mine) {
      i32x8 b[MT];
#pragma unroll
      for (int t = 0; t < MT; ++t) {
        const float m_new = fmaxf(before[t], am[i][t]);
        if (__builtin_amdgcn_ballot_w64(m_new != m_run[t]) != 0) {  // uniform
          qscale[t] = m_new > 0.f ? kE4M3Max / m_new : 0.f;  // IEEE division: it decides the FP8 codes
          const float corr = (m_new == m_run[t]) ? 1.0f : m_run[t] * fast_rcp(m_new);
          m_run[t] = m_new;
          if (i > 0) {
#pragma unroll
            for (int n = 0; n < NT; ++n) acc[n][t] *= corr;
          }
        }
#pragma unroll
        for (int h = 0; h < 4; ++h) {
          b[t][2 * h] = quant4(xr[i][t][h][0], xr[i][t][h][1], qscale[t]);
          b[t][2 * h + 1] = quant4(xr[i][t][h][2], xr[i][t][h][3], qscale[t]);
        }
      }
#pragma unroll
      for (int n = 0; n < NT; ++n) {
        const i32x8 av = __builtin_shufflevector(__builtin_bit_cast(i32x4, wr[i % PW][n][0]),
                                                 __builtin_bit_cast(i32x4, wr[i % PW][n][1]), 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
        for (int t = 0; t < MT; ++t)
          acc[n][t] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(av, b[t], acc[n][t], 0, 0, 0, 0x7f7f7f7f, 0,
                                                                        0x7f7f7f7f);
      }
      if (i + PW < TPW) {
        load_w(i % PW, i + PW);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }

  // ---- add the wavefronts' sums ----
  float unit[MT];  // this wavefront's maximum in units of the token's
#pragma unroll
  for (int t = 0; t < MT; ++t) unit[t] = (m_run[t] == all[t]) ? 1.0f : m_run[t] * fast_rcp(all[t]);
#pragma unroll
  for (int q0 = 0; q0 < kTiles; q0 += kG) {
    if (q0 > 0) __syncthreads();  // the previous group's sums have been read
#pragma unroll
    for (int q = 0; q < kG; ++q) {
      const int t = (q0 + q) % MT, n = (q0 + q) / MT;
      s_red[(wave * kG + q) * kWave + lane] = acc[n][t] * unit[t];
    }
    __syncthreads();
    for (int idx = tid; idx < kG * kWave; idx += kFThreads) {
      const int q = idx >> 6, l = idx & 63;
      f32x4 v = s_red[q * kWave + l];
#pragma unroll
      for (int wv = 1; wv < kFWaves; ++wv) v += s_red[(wv * kG + q) * kWave + l];
      const int t = (q0 + q) % MT, n = (q0 + q) / MT;
      v *= s_all[16 * t + (l & 15)] * (1.0f / kE4M3Max);
      const int m = m0 + 16 * t + (l & 15);
      const int col = n0 + 16 * n + 4 * (l >> 4);
      if (m < M && col < N) {  // (N is a multiple of 8: four channels are all in or all out)
        u32x2 o;
        o[0] = pack_bf16(v[0], v[1]);
        o[1] = pack_bf16(v[2], v[3]);
        *reinterpret_cast<u32x2*>(c + (int64_t)m * ldc + col) = o;
      }
    }
  }
}

namespace {
struct FShape { int mt, nt; };
constexpr FShape kFShapes[] = {{1, 1}, {2, 1}, {4, 1}, {1, 2}, {2, 2}, {4, 2}, {1, 4}, {2, 4}, {4, 4}};
// Tiles per wavefront that the registers hold; times the token tiles at most 8 (128 registers).
inline int tiles_held(int K) { return K <= 2048 ? 2 : K <= 4096 ? 4 : 8; }
// Expected us.  A workgroup takes its tile shape's time, most of it the trips to memory and the
// quantisation of its tokens; more workgroups than the 32 compute units of an XCD take turns (the
// channel tiles are dealt to the 8 XCDs, so some get a row of workgroups more: 168 x 512 x 1272 as
// 1 x 4, 33 workgroups on half of them, took 11.7 us instead of 7).  Within 10 % of the
// measured times of all shapes for 512 to 8192 k, 512 to 8192 channels and 1 to 512 tokens, e.g.
// 9.5 us for 16 x 4096 x 4096 as 1 x 1, 18.3 for 128 x 4096 x 4096 as 2 x 4, 23.9 for
// 128 x 8192 x 2048 as 1 x 4.
inline double rows_us(const FShape& r, int M, int K, int N) {
  const double k = K <= 2048 ? fmax(K / 1024.0, 1.5) : tiles_held(K);  // (all held tiles are fetched)
  const double one = 1.2 + 2.6 * r.mt + 0.7 * r.nt + (k - 1) * (1.0 + 0.4 * r.mt + 0.2 * r.nt);
  const int n_nt = (N + 16 * r.nt - 1) / (16 * r.nt);
  const double wg_xcd = (double)((M + 16 * r.mt - 1) / (16 * r.mt)) * ((n_nt + 7) / 8);
  return 2.0 + (one - 2.0) * ceil(wg_xcd / 32);
}
FShape best_shape(int M, int K, int N) {
  FShape best = kFShapes[0];
  for (const FShape& r : kFShapes)
    if (r.mt * tiles_held(K) <= 8 && rows_us(r, M, K, N) < rows_us(best, M, K, N)) best = r;
  return best;
}
}  // namespace

// The large kernel takes 6 us and 9 for every 1024 k as long as its tiles leave compute units idle
// (35 to 48 us at 4096 k, 65 to 86 at 8192), whatever the token count.  Both sides at the line:
// 256 x 4096 x 4096: 34.3 us here, 46.9 there; 384: 49.5 and 48.5.  64 x 8192 x 8192: 46 and 77;
// 100: 89 and 83.  1672 x 256 x 40: 13.8 and 7.7 (a handful of channel tiles leaves XCDs idle).
bool fp8_quant_gemm_rows_wins(int M, int K, int N, const void* c, int64_t ldc) {
  // (8-byte stores of c)
  if (K > 8192 || N % 8 != 0 || reinterpret_cast<uintptr_t>(c) % 8 != 0 || (M > 1 && ldc % 4 != 0)) return false;
  return 1.05 * rows_us(best_shape(M, K, N), M, K, N) < 6.0 + 9.0 * (K / 1024.0);
}

double fp8_quant_gemm_rows_us(int M, int K, int N) { return rows_us(best_shape(M, K, N), M, K, N); }

int fp8_quant_gemm_rows_tile(int M, int K, int N) {
  const FShape r = best_shape(M, K, N);
  return 16 * r.mt * 1000 + 16 * r.nt;
}

hipError_t launch_fp8_quant_gemm_rows(const void* a, const void* w, void* c, int M, int K, int N,
                                      int64_t lda, int64_t ldw, int64_t ldc, hipStream_t s) {
  const int tpw = tiles_held(K);
  const FShape best = best_shape(M, K, N);
  const int n_mt = (M + 16 * best.mt - 1) / (16 * best.mt);
  const int n_nt = (N + 16 * best.nt - 1) / (16 * best.nt);
  const int64_t grid = (int64_t)((n_nt + 7) / 8 * 8) * n_mt;
  if (grid > INT32_MAX) return hipErrorInvalidValue;
#define RF_F8ROWS(MT, NT, TPW, PW)                                                                           \
  if (best.mt == MT && best.nt == NT && tpw == TPW)                                                          \
    hipLaunchKernelGGL((fp8_quant_gemm_rows_kernel<MT, NT, TPW, PW>), dim3((unsigned)grid), dim3(kFThreads), 0, s, \
                       (const bf16_t*)a, (const unsigned char*)w, (bf16_t*)c, M, K, N, lda, ldw, ldc, n_mt);
  RF_F8ROWS(1, 1, 2, 2) RF_F8ROWS(2, 1, 2, 2) RF_F8ROWS(4, 1, 2, 2)
  RF_F8ROWS(1, 2, 2, 2) RF_F8ROWS(2, 2, 2, 2) RF_F8ROWS(4, 2, 2, 2)
  RF_F8ROWS(1, 4, 2, 2) RF_F8ROWS(2, 4, 2, 2) RF_F8ROWS(4, 4, 2, 1)
  RF_F8ROWS(1, 1, 4, 4) RF_F8ROWS(2, 1, 4, 4) RF_F8ROWS(1, 2, 4, 4) RF_F8ROWS(2, 2, 4, 2)
  RF_F8ROWS(1, 4, 4, 2) RF_F8ROWS(2, 4, 4, 1)
  RF_F8ROWS(1, 1, 8, 8) RF_F8ROWS(1, 2, 8, 4) RF_F8ROWS(1, 4, 8, 2)
#undef RF_F8ROWS
  return hipGetLastError();
}

}  // namespace rf
