// RMSNorm + linear in two launches, for callers that hand over a workspace:
//   1. rms_rows_kernel: x g rounded to bf16, as the single-launch kernels round it, and
//      H(ss) = (sum x^2 / K + eps)^(-1/2) of every row, one read of x;
//   2. bf16_gemm_kernel: y[i,n] = H_i sum_k xg[i,k] w[k,n].
// The single-launch kernels form x g beside the matrix pipe once for every 128 or 512 columns, in tiles of 128 x 512
// that leave compute units idle below some 4000 rows, or with every operand straight into registers.
//
// The contraction.  Y^T = W^T X^T with 32x32x16 bf16 MFMAs (A = columns, B = rows: an accumulator lane holds one
// row, one scale).  A workgroup of 4 wavefronts owns a tile of 32 TM WM rows x 32 TN WN columns; a stage is 32 KH k of
// the rows (k innermost) and of w (columns innermost), fetched by direct-to-LDS loads into a ring of NS stages; rows
// leave LDS as they lie, w by transpose reads.  In phase t a wavefront multiplies stage t, whose operands it already
// holds in registers, requests those of stage t+1 behind its first MFMAs, and requests stage t+NS into the slot that
// stage t left: no wavefront waits for LDS data behind the one barrier of a phase.
//
// What bounds it: the matrix pipe (1.2 PFLOP/s at 4096^3, where the first launch takes back what this gains) and, with
// fewer tiles than compute units, the lines a unit has in flight.  us a call, one launch / two: 2048 x 4096 x 4096
// 90.7 / 69.3, 1024 x 4096 x 4096 62.2 / 41.4, 600 x 2048 x 4096 34.0 / 21.9, 2727 x 1152 x 1360 30.3 / 20.0,
// 4000 x 512 x 1024 17.0 / 12.7, 2596 x 1216 x 6736 74.9 / 64.5.
#include <math.h>

#include <type_traits>

#include "rf_device.h"
#include "rf_launch.h"

namespace rf {

namespace {
constexpr int kGThreads = 256;
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
}  // namespace

// WPR wavefronts per row, VPT vectors of 8 values per lane (VPT = 0: rows of any length).
template <int VPT, int WPR>
__global__ __launch_bounds__(kGThreads) void rms_rows_kernel(const bf16_t* __restrict__ x, const bf16_t* __restrict__ g,
                                                             bf16_t* __restrict__ xg, float* __restrict__ row_scale,
                                                             int M, int K, int64_t ldx, float inv_k, float eps) {
  constexpr int kRows = 4 / WPR;
  __shared__ float s_sum[4];
  const int wave = threadIdx.x >> 6;
  const int row = blockIdx.x * kRows + (WPR == 1 ? wave : 0);
  const int vec = WPR == 1 ? (threadIdx.x & 63) : threadIdx.x;
  const int step = 64 * WPR;
  const int nv = K / 8;
  if (WPR == 1 && row >= M) return;
  const u32x4* src = reinterpret_cast<const u32x4*>(x + (int64_t)row * ldx);
  const u32x4* gv = reinterpret_cast<const u32x4*>(g);
  u32x4* dst = reinterpret_cast<u32x4*>(xg + (int64_t)row * K);
  float ss = 0.f;
  auto one = [&](int i, const u32x4& v, const u32x4& w) {
    u32x4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float a = bf16_lo(v[j]), b = bf16_hi(v[j]);
      ss = fmaf(a, a, ss);
      ss = fmaf(b, b, ss);
      o[j] = pack_bf16(a * bf16_lo(w[j]), b * bf16_hi(w[j]));
    }
    dst[i] = o;
  };
  if constexpr (VPT > 0) {
    u32x4 v[VPT], w[VPT];
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      v[i] = src[min(vec + i * step, nv - 1)];
      w[i] = gv[min(vec + i * step, nv - 1)];
    }
#pragma unroll
    for (int i = 0; i < VPT; ++i)
      if (vec + i * step < nv) one(vec + i * step, v[i], w[i]);
  } else {
    for (int i = vec; i < nv; i += step) one(i, src[i], gv[i]);
  }
  ss = wave_sum(ss);
  if constexpr (WPR == 4) {
    if ((threadIdx.x & 63) == 0) s_sum[wave] = ss;
    __syncthreads();
    ss = (s_sum[0] + s_sum[1]) + (s_sum[2] + s_sum[3]);
  }
  if (vec == 0) row_scale[row] = 1.0f / sqrtf(ss * inv_k + eps);
}

namespace {
template <int TM, int TN, int WM, int WN, int KH, int NS>
struct GTile {
  static_assert(WM * WN == 4, "4 wavefronts");
  static constexpr int kM = 32 * TM * WM, kN = 32 * TN * WN;
  static constexpr int kK = 32 * KH, kRowB = 64 * KH;
  static constexpr int kXB = kM * kRowB, kWB = kK * kN * 2, kStageB = kXB + kWB;
  static constexpr int kLoadsA = kXB / 4096, kLoadsW = kWB / 4096, kLoads = kLoadsA + kLoadsW;
  static_assert(kXB % 4096 == 0 && kWB % 4096 == 0, "whole loads");
  static constexpr int kOutB = 4 * 32 * (64 * TN + 16);
  static constexpr int kLdsB = NS * kStageB > kOutB ? NS * kStageB : kOutB;
};
}  // namespace

template <int TM, int TN, int WM, int WN, int KH, int NS, int OCC>
__global__ __launch_bounds__(kGThreads, OCC) void bf16_gemm_kernel(
    const bf16_t* __restrict__ xg, const float* __restrict__ row_scale, const bf16_t* __restrict__ w,
    bf16_t* __restrict__ c, int M, int K, int N, int64_t ldw, int64_t ldc, int n_mtiles, int n_ntiles) {
  using T = GTile<TM, TN, WM, WN, KH, NS>;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[T::kLdsB];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i32 = lane & 31, hh = lane >> 5;
  const int wm = wave % WM, wn = wave / WM;

  // Workgroups are dealt round-robin to the 8 XCDs, each with its own L2: an XCD takes a run of
  // tiles, four row tiles wide, whose operands it reads once.
  int mt, nt;
  {
    const int total = n_mtiles * n_ntiles;
    const int q = total >> 3, r = total & 7;
    const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
    const int t = x * q + min(x, r) + j;
    constexpr int kG = 4;
    const int per = kG * n_ntiles;
    const int g = t / per, rem = t - g * per;
    const int gm = min(kG, n_mtiles - g * kG);
    mt = g * kG + rem % gm;
    nt = rem / gm;
  }
  mt = __builtin_amdgcn_readfirstlane(mt);
  nt = __builtin_amdgcn_readfirstlane(nt);
  const int m0 = mt * T::kM, n0 = nt * T::kN;
  const int n_stages = K / T::kK;
  constexpr int kLanesRow = T::kRowB / 16, kRowsL = 64 / kLanesRow;
  constexpr int kLanesW = T::kN / 8, kRowsW = 64 / kLanesW;
  static_assert(kLanesW <= 64, "a row of w per load at least");
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;
  // 16-byte slots of a row are XOR-swizzled with the row, so that the reads below meet every bank evenly: one row per
  // lane of x g, four rows at a time of w
  auto swz = [](int row) { return KH == 2 ? (row >> 1) & 7 : (row >> 2) & 3; };
  auto swz_w = [](int krow) { return T::kN >= 128 ? (krow & 3) << 2 : ((krow >> 1) & 1) << 2; };
  uint32_t a_off[T::kLoadsA], w_off[T::kLoadsW];
#pragma unroll
  for (int e = 0; e < T::kLoadsA; ++e) {
    const int row = (4 * e + wave) * kRowsL + lane / kLanesRow;  // (the workspace holds whole tiles of rows)
    a_off[e] = (uint32_t)(row * K * 2 + (((lane % kLanesRow) ^ swz(row)) << 4));
  }
#pragma unroll
  for (int e = 0; e < T::kLoadsW; ++e) {
    const int krow = (4 * e + wave) * kRowsW + lane / kLanesW;
    const int piece = (lane % kLanesW) ^ swz_w(krow);  // columns past the end repeat the last ones
    w_off[e] = (uint32_t)(krow * (uint32_t)(ldw * 2) + min(n0 + 8 * piece, N - 8) * 2);
  }
  const char* abase = reinterpret_cast<const char*>(xg + (int64_t)m0 * K);
  const char* wbase = reinterpret_cast<const char*>(w);
  auto request = [&](int e, int t, uint32_t slot_off) {  // load e of stage t (past the end the last one once more)
    const bool tok = e < T::kLoadsA;
    const int tt = min(t, n_stages - 1);
    const char* base = tok ? abase + (int64_t)tt * T::kRowB : wbase + (int64_t)tt * (T::kK * 2) * ldw;
    const uint32_t dst = lds_base + slot_off + (tok ? (4 * e + wave) * 1024 : T::kXB + (4 * (e - T::kLoadsA) + wave) * 1024);
    const uint32_t off = tok ? a_off[tok ? e : 0] : w_off[tok ? 0 : e - T::kLoadsA];
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(dst), "v"(off), "s"(base)
                 : "memory", "m0");
  };

  // Row operand: lane (i32, hh) reads 16 bytes, k 16 s + 8 hh .., of row i32 of a block.  Column operand by transpose
  // reads: lane = 32 hh + 16 g2 + 4 j + a reads 8 bytes of k-row 16 s + 8 hh + 4 w2 + j at column 16 g2 + 4 a of a block
  constexpr int S2 = 2 * KH;  // 16-k steps of a stage
  uint32_t frag_t[S2], frag_w[S2][2];
#pragma unroll
  for (int s = 0; s < S2; ++s) {
    frag_t[s] = (wm * TM * 32 + i32) * T::kRowB + (((2 * s + hh) ^ swz(i32)) << 4);
    const int i16 = lane & 15, g2 = (lane >> 4) & 1, j = i16 >> 2, a = i16 & 3;
#pragma unroll
    for (int w2 = 0; w2 < 2; ++w2) {
      const int krow = 16 * s + 8 * hh + 4 * w2 + j;
      const int piece = wn * TN * 4 + 2 * g2 + (a >> 1);  // + 4 n
      frag_w[s][w2] = T::kXB + krow * (2 * T::kN) + 8 * (a & 1) + (piece << 4);
    }
  }
  const int w_swz = swz_w(8 * hh + ((lane & 15) >> 2)) << 4;  // (the row mod 4 of all of this lane's reads)
  auto read_t = [&](int s, int i, uint32_t slot_off) {
    return __builtin_bit_cast(bf16x8, *reinterpret_cast<const u32x4*>(lds + slot_off + frag_t[s] + i * 32 * T::kRowB));
  };
  auto read_w = [&](int s, int i, uint32_t slot_off) {
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(lds + slot_off + ((frag_w[s][0] + 64 * i) ^ w_swz)));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(lds + slot_off + ((frag_w[s][1] + 64 * i) ^ w_swz)));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  f32x16 acc[TN][TM];
#pragma unroll
  for (int n = 0; n < TN; ++n)
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[n][m][r] = 0.f;
  bf16x8 ft[2][S2][TM], fw[2][S2][TN];
#define RF_FENCE __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int t = 0; t < NS; ++t)
#pragma unroll
    for (int e = 0; e < T::kLoads; ++e) request(e, t, t * T::kStageB);
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 1) * T::kLoads) : "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int s = 0; s < S2; ++s) {
#pragma unroll
    for (int i = 0; i < TM; ++i) ft[0][s][i] = read_t(s, i, 0);
#pragma unroll
    for (int i = 0; i < TN; ++i) fw[0][s][i] = read_w(s, i, 0);
  }
  constexpr int kMfmas = S2 * TM * TN, kReads = S2 * (TM + TN);
  constexpr int kRate = (2 * kReads + kMfmas - 1) / kMfmas;  // operands behind an MFMA: all in the first half
  uint32_t slot = 0;
  auto phase = [&](auto cur_c, int t) __attribute__((always_inline)) {
    constexpr int cur = decltype(cur_c)::value, nxt = cur ^ 1;
    const uint32_t next = slot == (NS - 1) * T::kStageB ? 0 : slot + T::kStageB;
#pragma unroll
    for (int s = 0; s < S2; ++s) {
#pragma unroll
      for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(ft[cur][s][i]));
#pragma unroll
      for (int i = 0; i < TN; ++i) asm volatile("" : "+v"(fw[cur][s][i]));
    }
    // stage t+1 has landed, for every wavefront; stage t's slot has been read by all of them
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * T::kLoads) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    RF_FENCE
#pragma unroll
    for (int q = 0; q < kMfmas; ++q) {
      const int s = q / (TM * TN), n = q / TM % TN, m = q % TM;
      acc[n][m] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[cur][s][n], ft[cur][s][m], acc[n][m], 0, 0, 0);
#pragma unroll
      for (int f = min(kReads, q * kRate); f < min(kReads, (q + 1) * kRate); ++f) {
        const int fk = f / (TM + TN), i = f % (TM + TN);
        if (i < TM) ft[nxt][fk][i < TM ? i : 0] = read_t(fk, i, next);
        else fw[nxt][fk][i < TM ? 0 : i - TM] = read_w(fk, i - TM, next);
      }
#pragma unroll
      for (int e = q * T::kLoads / kMfmas; e < (q + 1) * T::kLoads / kMfmas; ++e) request(e, t + NS, slot);
      RF_FENCE
    }
    slot = next;
  };
  int t = 0;
  for (; t + 1 < n_stages; t += 2) {
    phase(std::integral_constant<int, 0>{}, t);
    phase(std::integral_constant<int, 1>{}, t + 1);
  }
  if (t < n_stages) phase(std::integral_constant<int, 0>{}, t);
#undef RF_FENCE
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the surplus requests have landed
  __syncthreads();

  // An accumulator lane holds one row and runs of four columns: a block of 32 rows goes through LDS and leaves
  // in 16-byte pieces, 64 TN contiguous bytes of a row.
  constexpr int kPitch = 64 * TN + 16;
  unsigned char* stage = lds + wave * (32 * kPitch);
#pragma unroll
  for (int m = 0; m < TM; ++m) {
    const int tok0 = m0 + (wm * TM + m) * 32;
    const float f = tok0 + i32 < M ? row_scale[tok0 + i32] : 0.f;
#pragma unroll
    for (int n = 0; n < TN; ++n)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        u32x2 o;
        o[0] = pack_bf16(acc[n][m][4 * r] * f, acc[n][m][4 * r + 1] * f);
        o[1] = pack_bf16(acc[n][m][4 * r + 2] * f, acc[n][m][4 * r + 3] * f);
        *reinterpret_cast<u32x2*>(stage + i32 * kPitch + 64 * n + 16 * r + 8 * hh) = o;
      }
    constexpr int kSlots = 4 * TN, kRows = 64 / kSlots;  // 16-byte pieces of a row, rows per store
    static_assert(64 % kSlots == 0, "whole rows per store");
#pragma unroll
    for (int i = 0; i < 32 / kRows; ++i) {
      const int row = i * kRows + lane / kSlots, piece = lane % kSlots;
      const u32x4 o = *reinterpret_cast<const u32x4*>(stage + row * kPitch + 16 * piece);
      const int tok = tok0 + row, ch = n0 + wn * TN * 32 + 8 * piece;
      if (tok < M && ch < N)  // (N is a multiple of 8)
        __builtin_nontemporal_store(o, reinterpret_cast<u32x4*>(c + (int64_t)tok * ldc + ch));
    }
  }
}

namespace {
// The tiles: row and column blocks of 32 per wavefront; wavefronts along rows and columns; pieces of 32 k per stage;
// stages; workgroups a compute unit is to hold.  With them the expected us of a launch: `launch` + turns over the
// 256 compute units x (`turn` + (`step` + `full` x the share of the units in use) per 64 k): the chip's clock falls with
// its load.  Fitted to graph replays of every tile on 146 products of 60 to 4500 rows (most within 8 %); the
// tile chosen by them takes 0.4 % more than the best one, 11 % at worst.
struct NShape { int m, n; double launch, turn, step, full; };
#define RF_NTILES(X)                                                                                             \
  X(0, (4, 4, 2, 2, 1, 4, 1), 0.0, 9.8, 0.917, 0.582) X(1, (2, 4, 2, 2, 2, 3, 1), 1.4, 5.3, 0.573, 0.304)        \
  X(2, (2, 2, 2, 2, 2, 4, 1), 1.3, 4.0, 0.345, 0.155) X(3, (1, 2, 2, 2, 2, 3, 2), 2.8, 0.75, 0.302, 0.046)       \
  X(4, (1, 1, 2, 2, 2, 4, 2), 2.5, 0.67, 0.207, 0.027)
#define RF_NSHAPE_OF(TM, TN, WM, WN, KH, NS, OCC) 32 * TM * WM, 32 * TN * WN
#define RF_NSHAPE(I, P, L, T, S, F) {RF_NSHAPE_OF P, L, T, S, F},
constexpr NShape kNShapes[] = {RF_NTILES(RF_NSHAPE)};
constexpr int kPadRows = 256;  // the workspace holds whole tiles of rows

double tile_us(const NShape& g, int M, int K, int N) {
  const double tiles = ceil((double)M / g.m) * ceil((double)N / g.n), turns = ceil(tiles / 256);
  return g.launch + turns * (g.turn + (g.step + g.full * tiles / (256 * turns)) * (K / 64));
}
int best_tile(int M, int K, int N) {
  int best = 0;
  double best_us = tile_us(kNShapes[0], M, K, N);
  for (int i = 1; i < (int)(sizeof(kNShapes) / sizeof(kNShapes[0])); ++i) {
    const double us = tile_us(kNShapes[i], M, K, N);
    if (us < best_us) best = i, best_us = us;
  }
  return best;
}
// Rows beyond what kNormWorkspaceMax holds go slab by slab through the same workspace.
int slab_rows(int M, int K) {
  const int64_t fit = kNormWorkspaceMax / (2 * (int64_t)K + 4) / kPadRows * kPadRows;
  return (int)(fit < M ? fit : M);
}
int64_t padded(int rows) { return ((int64_t)rows + kPadRows - 1) / kPadRows * kPadRows; }
}  // namespace

// Both launches against the single one.  The first takes 2.7 us for the smallest and 11.6 for 4096 x 4096, and a
// second launch adds some 3.5 us to a call that is waited for (none to calls in a row).  Of the 146 products above
// this takes 59, 1.44 times faster in a row; 4096^3 (123.7, 126.9 in one launch), 323 x 3200 x 4208 (24.9, 26.9) and
// 300 x 1024 x 1024 (8.9, 5.7) stay.
bool rmsnorm_gemm_two_pass_wins(int M, int K, int N, double single_us) {
  if (K >= (1 << 22) || slab_rows(M, K) < (M < 2048 ? M : 2048)) return false;  // 32-bit offsets inside a tile
  const double first = 1.9 + 4.0 * M * (double)K / 6.5e6;
  if (first + 3.1 + 3.5 >= 0.92 * single_us) return false;  // (no tile takes less: the smallest calls end here, their host time counts)
  return first + tile_us(kNShapes[best_tile(M, K, N)], M, K, N) + 3.5 < 0.92 * single_us;
}

size_t rmsnorm_gemm_two_pass_bytes(int M, int K) {
  const int slab = slab_rows(M, K);
  return (size_t)(padded(slab) * K * 2 + 4 * (((int64_t)slab + 3) / 4 * 4));
}

int rmsnorm_gemm_two_pass_tile(int M, int K, int N) {
  const NShape g = kNShapes[best_tile(M, K, N)];
  return g.m * 1000 + g.n;
}

hipError_t launch_rmsnorm_gemm_two_pass(const void* x, const void* g, const void* w, void* y, int M, int K, int N,
                                        int64_t ldx, int64_t ldw, int64_t ldy, float eps, void* workspace,
                                        hipStream_t s) {
  const int slab = slab_rows(M, K);
  bf16_t* xg = (bf16_t*)workspace;
  float* row_scale = (float*)(xg + padded(slab) * K);
  const int nv = K / 8;
  for (int64_t r0 = 0; r0 < M; r0 += slab) {
    const int rows = (int)(M - r0 < slab ? M - r0 : slab);
    const int tile = best_tile(rows, K, N);
    const NShape sh = kNShapes[tile];
    const int n_mt = (rows + sh.m - 1) / sh.m, n_nt = (N + sh.n - 1) / sh.n;
    // a grid of 2^32 threads or more is not launched whole
    if ((int64_t)n_mt * n_nt >= ((int64_t)1 << 32) / kGThreads) return hipErrorInvalidValue;
#define RF_ROWS_OF(VPT, WPR)                                                                                      \
  hipLaunchKernelGGL((rms_rows_kernel<VPT, WPR>), dim3((unsigned)((rows + 4 / WPR - 1) / (4 / WPR))),             \
                     dim3(kGThreads), 0, s, (const bf16_t*)x + r0 * ldx, (const bf16_t*)g, xg, row_scale, rows, K, ldx, \
                     1.0f / (float)K, eps)
    if (nv <= 64) RF_ROWS_OF(1, 1);
    else if (nv <= 128) RF_ROWS_OF(2, 1);
    else if (nv <= 256) RF_ROWS_OF(1, 4);
    else if (nv <= 512) RF_ROWS_OF(2, 4);
    else if (nv <= 1024) RF_ROWS_OF(4, 4);
    else RF_ROWS_OF(0, 4);
#undef RF_ROWS_OF
    bf16_t* ys = (bf16_t*)y + r0 * ldy;
#define RF_NGEMM_OF(TM, TN, WM, WN, KH, NS, OCC) bf16_gemm_kernel<TM, TN, WM, WN, KH, NS, OCC>
#define RF_NGEMM(I, P, L, T, S, F)                                                                                \
  if (tile == I)                                                                                                  \
    hipLaunchKernelGGL((RF_NGEMM_OF P), dim3((unsigned)(n_mt * n_nt)), dim3(kGThreads), 0, s, xg, row_scale,      \
                       (const bf16_t*)w, ys, rows, K, N, ldw, ldy, n_mt, n_nt);
    RF_NTILES(RF_NGEMM)
#undef RF_NGEMM
    if (hipError_t e = hipGetLastError()) return e;
  }
  return hipSuccess;
}

}  // namespace rf
