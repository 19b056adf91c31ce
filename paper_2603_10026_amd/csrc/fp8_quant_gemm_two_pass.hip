// FP8 per-token quantisation + GEMM in two launches, for callers that hand over a workspace:
//   1. fp8_quant_rows_kernel: for every tile of 128 k the maximum m' of the token up to the tile's end
//      and the codes q(MAX a / m') of the tile, MAX = 448, one read of a;
//   2. fp8_gemm_kernel: the incremental sum over the tiles, acc = acc * (m'_old / m'_new) + code . w,
//      c = acc * m / MAX.
// The single-launch kernels form the same codes once for every 256 or 512 channels beside the matrix
// pipe; here the contraction reads them, half the token bytes, and all that is left beside its matrix
// instructions is the rescaling.  Where one wavefront sums the whole axis (WK = 1) the result is that of
// the 128-token single-launch tiles to the bit.
//
// The contraction.  C^T = W A_q^T with v_mfma_f32_32x32x64_f8f6f4 (A = channels, B = tokens: an
// accumulator lane holds one token, one scale).  A workgroup of 4 or 8 wavefronts owns a tile of
// 32 TM WM tokens x 32 TN WN channels; tokens and channels both lie with k innermost, so a stage
// is KH x 64 bytes of every row and the tokens' maxima, fetched by direct-to-LDS loads into a ring of
// NS stages and read as the operands lie.  In phase t a wavefront multiplies stage t, whose operands
// it already holds in registers, requests those of stage t+1 behind its first MFMAs, and requests stage
// t+NS into the slot that stage t left: no wavefront waits for LDS data behind the one barrier of a
// phase, and a tile has NS - 1 phases to arrive.
//
// What bounds it.  Large products: the matrix pipe beside LDS (a 256 x 256 tile over 8 wavefronts reads
// 96 KB of operands and writes 32 KB of tiles per 64 k) and the sums' rescaling, which most tiles of 32
// tokens need for one of them.  4096 x 8192 x 3584: 17.6 us of quantisation (5.7 TB/s) + 113 us of contraction
// (2.1 PFLOP/s), 130 in all where the single launch takes 176 on the same card; 4096 x 3584 x 8192: 152 -> 125.
// Smaller ones: the lines a compute unit has in flight (50 to 70 GB/s each), so tiles are
// made as small as fills the chip, and below 64 x 64 the wavefronts take parts of the axis (WK)
// rather than of the tile: 1348 x 3456 x 2336 48 -> 26 us, 141 x 3456 x 7200 43 -> 17,
// 36 x 12800 x 2008 121 -> 20.
#include <math.h>

#include <type_traits>

#include "rf_device.h"
#include "rf_launch.h"

namespace rf {

namespace {
constexpr float kE4M3Max = 448.0f;
constexpr int kGThreads = 256;
typedef __attribute__((__vector_size__(4 * sizeof(int)))) int i32x4;

__device__ __forceinline__ int codes4(uint32_t p0, uint32_t p1, float s) {
  int t = 0;
  t = __builtin_amdgcn_cvt_pk_fp8_f32(bf16_lo(p0) * s, bf16_hi(p0) * s, t, false);
  t = __builtin_amdgcn_cvt_pk_fp8_f32(bf16_lo(p1) * s, bf16_hi(p1) * s, t, true);
  return t;
}
typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
// For non-negative values the bf16 bit patterns order like unsigned integers: maxima are taken on
// packed 16-bit integers with the sign bits cleared.
__device__ __forceinline__ u16x2 absmax8(u16x2 m, const u32x4& r) {
#pragma unroll
  for (int j = 0; j < 4; ++j) m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, r[j] & 0x7fff7fffu));
  return m;
}
}  // namespace

// Codes and prefix maxima of a row.  16 lanes (a DPP row) hold a tile of 128 k; WPR wavefronts per row, VPT vectors of
// 8 values per lane held in registers.  Rows of any length (VPT = 0) go chunk by chunk, 16 tiles at a time: a tile is
// quantised with the maximum up to its own end, so nothing is read twice.
template <int VPT, int WPR>
__global__ __launch_bounds__(kGThreads) void fp8_quant_rows_kernel(const bf16_t* __restrict__ a,
                                                                   unsigned char* __restrict__ codes,
                                                                   float* __restrict__ maxima, int M, int K,
                                                                   int64_t lda, int pitch, int run) {
  constexpr int kTiles = VPT > 0 ? 4 * WPR * VPT : 32;  // (VPT = 0: two chunks of 16, in turn)
  static_assert(VPT == 0 ? WPR == 4 : kTiles <= 64, "a lane per tile in the scan");
  __shared__ float s_max[WPR == 4 ? kTiles : 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int row = blockIdx.x * 4 + wave;
  if constexpr (WPR == 4) {
    // runs of rows on one XCD (workgroups are dealt to the 8 in turn): their maxima share lines
    const int j = blockIdx.x >> 3;
    row = (j / run * 8 + (blockIdx.x & 7)) * run + j % run;
  }
  if (row >= M) return;
  const int vec = WPR == 1 ? lane : threadIdx.x;  // this lane's first vector of the row
  const int in_step = vec >> 4;                   // and its tile
  constexpr int kStep = 64 * WPR, kStepTiles = 4 * WPR;
  const int nv = K / 8, nk = K / 128;
  const u32x4* src = reinterpret_cast<const u32x4*>(a + (int64_t)row * lda);
  u32x2* dst = reinterpret_cast<u32x2*>(codes + (int64_t)row * K);
  float* out = maxima + row;
  auto put = [&](int i, const u32x4& v, float m) {
    const float s = m > 0.f ? kE4M3Max / m : 0.f;  // IEEE division: it decides the codes
    u32x2 o;
    o[0] = (uint32_t)codes4(v[0], v[1], s);
    o[1] = (uint32_t)codes4(v[2], v[3], s);
    dst[i] = o;
    if ((lane & 15) == 0) out[(int64_t)(i >> 4) * pitch] = m;
  };
  auto tile_max = [](const u32x4& v) {
    const u16x2 m = absmax8(u16x2{0, 0}, v);
    return row16_max(__uint_as_float((uint32_t)(m[0] > m[1] ? m[0] : m[1]) << 16));
  };
  if constexpr (VPT > 0) {
    u32x4 x[VPT];
    float mine[VPT];  // maximum of this lane's tile
#pragma unroll
    for (int i = 0; i < VPT; ++i) x[i] = src[min(vec + i * kStep, nv - 1)];
#pragma unroll
    for (int i = 0; i < VPT; ++i) mine[i] = tile_max(x[i]);
    // prefix maxima, a tile per lane (tiles past the end come after all others)
    float upto;
    if constexpr (WPR == 4) {
#pragma unroll
      for (int i = 0; i < VPT; ++i)
        if ((lane & 15) == 0) s_max[i * kStepTiles + in_step] = mine[i];
      __syncthreads();
      upto = s_max[lane % kTiles];
    } else {
      upto = __shfl(mine[0], (lane & 3) * 16, 64);
#pragma unroll
      for (int i = 1; i < VPT; ++i) {
        const float o = __shfl(mine[i], (lane & 3) * 16, 64);
        upto = (lane >> 2) == i ? o : upto;
      }
    }
#pragma unroll
    for (int d = 1; d < kTiles; d *= 2) {
      const float o = __shfl_up(upto, d, 64);
      upto = lane >= d ? fmaxf(upto, o) : upto;
    }
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const float m = __shfl(upto, i * kStepTiles + in_step, 64);
      if (vec + i * kStep < nv) put(vec + i * kStep, x[i], m);
    }
  } else {
    float before = 0.f;
    u32x4 x = src[min(vec, nv - 1)];
    for (int i = vec, turn = 0; i < nv + vec; i += kStep, turn ^= 1) {
      const u32x4 following = src[min(i + kStep, nv - 1)];
      const float mine = tile_max(x);
      if ((lane & 15) == 0) s_max[16 * turn + in_step] = mine;
      __syncthreads();  // (a wavefront is at most one chunk ahead: two buffers do)
      float upto = s_max[16 * turn + (lane & 15)];
#pragma unroll
      for (int d = 1; d < 16; d *= 2) {
        const float o = __shfl_up(upto, d, 16);
        upto = (lane & 15) >= d ? fmaxf(upto, o) : upto;
      }
      const float m = fmaxf(before, __shfl(upto, in_step, 16));
      before = fmaxf(before, __shfl(upto, 15, 16));
      if (i < nv) put(i, x, m);
      x = following;
    }
  }
}

namespace {
template <int TM, int TN, int WM, int WN, int WK, int KH, int NS>
struct GTile {
  static constexpr int kWaves = WM * WN * WK, kThreads = kWaves * kWave;
  static_assert(kWaves == 4 || (kWaves == 8 && WK == 1), "4 or 8 wavefronts");
  static constexpr int kM = 32 * TM * WM, kN = 32 * TN * WN;
  static constexpr int kRowB = 64 * KH;                  // bytes of a row in a stage
  static constexpr int kGroupB = (kM + kN) * kRowB;      // what one of the WK parts of a stage holds
  static constexpr int kMaxAt = WK * kGroupB, kStageB = kMaxAt + WK * kM * 4;  // the tokens' maxima behind the operands
  // direct-to-LDS loads per wavefront and stage, one of them for maxima (64 each: wavefronts share them where they are fewer)
  static constexpr int kLoadsA = WK * kM * kRowB / (1024 * kWaves), kLoadsW = WK * kN * kRowB / (1024 * kWaves);
  static constexpr int kLoads = kLoadsA + kLoadsW + 1;
  static constexpr int kMaxLoads = WK * kM / 64;
  static_assert(kMaxLoads >= 1 && kMaxLoads <= 4 && WK * kM % 64 == 0 && (kM % 64 == 0 || kM == 32), "a load of maxima each");
  static_assert(WK * kM * kRowB % (1024 * kWaves) == 0 && WK * kN * kRowB % (1024 * kWaves) == 0, "whole loads");
  // output staging: 32 tokens per wavefront (padded rows); with WK > 1 the sums of all wavefronts before that
  static constexpr int kOutB = WK > 1 ? 4 * TM * TN * 4096 + 4 * 32 * 80 : kWaves * 32 * (64 * TN + 16);
  static constexpr int kLdsB = NS * kStageB > kOutB ? NS * kStageB : kOutB;
};
}  // namespace

template <int TM, int TN, int WM, int WN, int WK, int KH, int NS, int OCC>
__global__ __launch_bounds__(WM * WN * WK * kWave, OCC) void fp8_gemm_kernel(
    const unsigned char* __restrict__ codes, const float* __restrict__ maxima, const unsigned char* __restrict__ w,
    bf16_t* __restrict__ c, int M, int K, int N, int64_t ldw, int64_t ldc, int pitch, int n_mtiles, int n_ntiles) {
  using T = GTile<TM, TN, WM, WN, WK, KH, NS>;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[T::kLdsB];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i32 = lane & 31, hh = lane >> 5;
  const int wm = wave % WM, wn = wave / WM % WN, wk = wave / (WM * WN);

  // Workgroups are dealt round-robin to the 8 XCDs, each with its own L2: an XCD takes a run of
  // tiles, four token tiles wide, whose rows it reads once.
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
  const int n_pieces = K / T::kRowB;  // (K is a multiple of 128)
  const int n_stages = (n_pieces + WK - 1) / WK;

  // ---- requests: a load covers 1 KB = kRowsL rows of a stage, the wavefronts take them in turn ----
  constexpr int kLanesRow = T::kRowB / 16;  // lanes per row (4 or 8)
  constexpr int kRowsL = 64 / kLanesRow;
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;
  // 16-byte slots of a row are XOR-swizzled with the row, so that the fragment reads (one row per
  // lane) meet every bank evenly
  auto swz = [](int row) { return KH == 2 ? (row >> 1) & 7 : (row >> 2) & 3; };
  const int lrow = lane / kLanesRow, lslot = lane % kLanesRow;
  constexpr int kLA = T::kM / kRowsL, kLW = T::kN / kRowsL;  // loads of a group
  uint32_t a_off[T::kLoadsA], w_off[T::kLoadsW];  // from the tile's first row; + piece * kRowB
#pragma unroll
  for (int e = 0; e < T::kLoadsA; ++e) {
    const int row = (T::kWaves * e + wave) % kLA * kRowsL + lrow;  // (the workspace holds whole tiles of rows)
    a_off[e] = (uint32_t)(row * K + ((lslot ^ swz(row)) << 4));
  }
#pragma unroll
  for (int e = 0; e < T::kLoadsW; ++e) {
    const int row = (T::kWaves * e + wave) % kLW * kRowsL + lrow;  // channels past the end repeat the last one
    w_off[e] = (uint32_t)(min(row, N - 1 - n0) * (int)ldw + ((lslot ^ swz(row)) << 4));
  }
  const unsigned char* abase = codes + (int64_t)m0 * K;
  const unsigned char* wbase = w + (int64_t)n0 * ldw;
  const int max_at = wave % T::kMaxLoads * 64 + lane;  // this lane's maximum in a stage: [part of the axis][token]
  const int max_grp = max_at / T::kM;
  const uint32_t max_off = (uint32_t)min(m0 + max_at % T::kM, M - 1) * 4;  // (tokens past the end repeat the last one)
  // load e of stage t (past the end of the axis the last piece once more, which nothing multiplies)
  auto request = [&](int e, int t, uint32_t slot_off) {
    if (e == T::kLoads - 1) {
      const int tile = min(t * WK + max_grp, n_pieces - 1) / (2 / KH);
      const uint32_t dst = lds_base + slot_off + T::kMaxAt + wave % T::kMaxLoads * 256;
      const uint32_t off = max_off + (uint32_t)tile * (uint32_t)pitch * 4;
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
                   :
                   : "s"(dst), "v"(off), "s"(maxima)
                   : "memory", "m0");
      return;
    }
    const bool tok = e < T::kLoadsA;
    const int idx = T::kWaves * (tok ? e : e - T::kLoadsA) + wave;
    const int per = tok ? kLA : kLW;
    const int grp = idx / per;
    const unsigned char* base = (tok ? abase : wbase) + (int64_t)min(t * WK + grp, n_pieces - 1) * T::kRowB;
    const uint32_t dst = lds_base + slot_off + grp * T::kGroupB + (tok ? 0 : T::kM * T::kRowB) + idx % per * 1024;
    const uint32_t off = tok ? a_off[tok ? e : 0] : w_off[tok ? 0 : e - T::kLoadsA];
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :
                 : "s"(dst), "v"(off), "s"(base)
                 : "memory", "m0");
  };

  // ---- fragments: 32 bytes per lane, row i32 of a block, bytes 32 hh .. 32 hh + 31 of its 64 ----
  uint32_t frag_t[KH][2], frag_w[KH][2];  // byte address in slot 0
#pragma unroll
  for (int kh = 0; kh < KH; ++kh)
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const uint32_t in_row = i32 * T::kRowB + (((4 * kh + 2 * hh + h) ^ swz(i32)) << 4);
      frag_t[kh][h] = wk * T::kGroupB + wm * TM * 32 * T::kRowB + in_row;
      frag_w[kh][h] = wk * T::kGroupB + (T::kM + wn * TN * 32) * T::kRowB + in_row;
    }
  auto read_t = [&](int kh, int i, uint32_t slot_off) {
    const i32x4 lo = *reinterpret_cast<const i32x4*>(lds + slot_off + frag_t[kh][0] + i * 32 * T::kRowB);
    const i32x4 hi = *reinterpret_cast<const i32x4*>(lds + slot_off + frag_t[kh][1] + i * 32 * T::kRowB);
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };
  auto read_w = [&](int kh, int i, uint32_t slot_off) {
    const i32x4 lo = *reinterpret_cast<const i32x4*>(lds + slot_off + frag_w[kh][0] + i * 32 * T::kRowB);
    const i32x4 hi = *reinterpret_cast<const i32x4*>(lds + slot_off + frag_w[kh][1] + i * 32 * T::kRowB);
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  };

  f32x16 acc[TN][TM];  // C^T: rows = channels, columns = tokens
#pragma unroll
  for (int n = 0; n < TN; ++n)
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[n][m][r] = 0.f;
  i32x8 ft[2][KH][TM], fw[2][KH][TN];  // operands of the stage being multiplied and of the next
  float mx[2][TM];                     // and the maxima of this lane's tokens up to there
  float m_run[TM];                     // the sums are in units of these
#pragma unroll
  for (int m = 0; m < TM; ++m) m_run[m] = 0.f;
  auto read_max = [&](int m, uint32_t slot_off) {
    return *reinterpret_cast<const float*>(lds + slot_off + T::kMaxAt + (wk * T::kM + (wm * TM + m) * 32 + i32) * 4);
  };

#define RF_FENCE __builtin_amdgcn_sched_barrier(0);
  // Stages 0 .. NS-1 are requested (surplus ones re-read the last), the operands of stage 0 read.
#pragma unroll
  for (int t = 0; t < NS; ++t)
#pragma unroll
    for (int e = 0; e < T::kLoads; ++e) request(e, t, t * T::kStageB);
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 1) * T::kLoads) : "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
#pragma unroll
  for (int kh = 0; kh < KH; ++kh) {
#pragma unroll
    for (int i = 0; i < TM; ++i) ft[0][kh][i] = read_t(kh, i, 0);
#pragma unroll
    for (int i = 0; i < TN; ++i) fw[0][kh][i] = read_w(kh, i, 0);
  }
#pragma unroll
  for (int m = 0; m < TM; ++m) mx[0][m] = read_max(m, 0);
  // Brings the sums of token block m to the units of a stage, where one of its tokens has a new maximum (uniform).
  auto rescale = [&](auto cur_c, int m) __attribute__((always_inline)) {
    const float m_new = mx[decltype(cur_c)::value][m];
    if (__builtin_amdgcn_ballot_w64(!(m_new == m_run[m])) != 0) {
      const float corr = m_new == m_run[m] ? 1.0f : m_run[m] * fast_rcp(m_new);
      m_run[m] = m_new;
#pragma unroll
      for (int n = 0; n < TN; ++n)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[n][m][r] *= corr;
    }
  };

  // Phase t: see the head of the file.  `cur`: which set of operand registers stage t is in.
  constexpr int kMfmas = KH * TM * TN, kReads = KH * (TM + TN);
  constexpr int kRate = (2 * kReads + kMfmas - 1) / kMfmas;  // operands behind an MFMA: all in the first half
  uint32_t slot = 0;  // byte offset of stage t's ring slot
  auto phase = [&](auto cur_c, int t) __attribute__((always_inline)) {
    constexpr int cur = decltype(cur_c)::value, nxt = cur ^ 1;
    const uint32_t next = slot == (NS - 1) * T::kStageB ? 0 : slot + T::kStageB;
    // stage t+1 has landed, for every wavefront; stage t's slot has been read by all of them
#pragma unroll
    for (int kh = 0; kh < KH; ++kh) {
#pragma unroll
      for (int i = 0; i < TM; ++i) asm volatile("" : "+v"(ft[cur][kh][i]));
#pragma unroll
      for (int i = 0; i < TN; ++i) asm volatile("" : "+v"(fw[cur][kh][i]));
    }
#pragma unroll
    for (int i = 0; i < TM; ++i)
      if (KH == 2 || cur == 0) asm volatile("" : "+v"(mx[cur][i]));
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * T::kLoads) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    RF_FENCE
#pragma unroll
    for (int q = 0; q < kMfmas; ++q) {
      const int kh = q / (TM * TN), m = q / TN % TM, n = q % TN;
      // a block's rescaling runs behind the MFMAs of the one before (stages of 64 k: every other one starts a tile)
      if (kh == 0 && n == 0 && (KH == 2 || cur == 0)) rescale(cur_c, m);
      acc[n][m] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fw[cur][kh][n], ft[cur][kh][m], acc[n][m], 0, 0, 0, 0, 0, 0);
#pragma unroll
      for (int f = min(kReads, q * kRate); f < min(kReads, (q + 1) * kRate); ++f) {
        const int fk = f / (TM + TN), i = f % (TM + TN);
        if (i < TM) ft[nxt][fk][i < TM ? i : 0] = read_t(fk, i, next);
        else fw[nxt][fk][i < TM ? 0 : i - TM] = read_w(fk, i - TM, next);
      }
      if (q < TM && (KH == 2 || nxt == 0)) mx[nxt][q < TM ? q : 0] = read_max(q, next);
#pragma unroll
      for (int e = q * T::kLoads / kMfmas; e < (q + 1) * T::kLoads / kMfmas; ++e) request(e, t + NS, slot);
      RF_FENCE
    }
    slot = next;
  };
  int t = 0;
  if constexpr (WK == 1) {
    for (; t + 1 < n_stages; t += 2) {
      phase(std::integral_constant<int, 0>{}, t);
      phase(std::integral_constant<int, 1>{}, t + 1);
    }
    if (t < n_stages) phase(std::integral_constant<int, 0>{}, t);
  } else {
    // in the last stage a run of wavefronts may be past the end of the axis
    auto last = [&](auto cur_c) {
      constexpr int cur = decltype(cur_c)::value;
      if ((n_stages - 1) * WK + wk < n_pieces) {
#pragma unroll
        for (int m = 0; m < TM; ++m) rescale(cur_c, m);
#pragma unroll
        for (int q = 0; q < kMfmas; ++q) {
          const int kh = q / (TM * TN), m = q / TN % TM, n = q % TN;
          acc[n][m] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fw[cur][kh][n], ft[cur][kh][m], acc[n][m], 0, 0, 0, 0, 0, 0);
        }
      }
    };
    for (; t + 2 < n_stages; t += 2) {
      phase(std::integral_constant<int, 0>{}, t);
      phase(std::integral_constant<int, 1>{}, t + 1);
    }
    if (t + 1 < n_stages) {
      phase(std::integral_constant<int, 0>{}, t);
      last(std::integral_constant<int, 1>{});
    } else {
      last(std::integral_constant<int, 0>{});
    }
  }
#undef RF_FENCE
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the surplus requests have landed
  __syncthreads();

  // ---- c = acc * m / MAX ----
  // An accumulator lane holds one token and runs of four channels: a block of 32 tokens goes
  // through LDS and leaves in 16-byte pieces, 64 TN contiguous bytes of a row.
  if constexpr (WK > 1) {
    // the sums over parts of the axis meet in LDS, a 32 x 32 block per wavefront in turn
    f32x4* red = reinterpret_cast<f32x4*>(lds);
    const float* m_all = maxima + (int64_t)(K / 128 - 1) * pitch;  // the tokens' own maxima
    float unit[TM];                                                // this wavefront's in units of those
#pragma unroll
    for (int m = 0; m < TM; ++m) {
      const float all = m_all[min(m0 + (wm * TM + m) * 32 + i32, M - 1)];
      unit[m] = m_run[m] == all ? 1.0f : m_run[m] * fast_rcp(all);
    }
#pragma unroll
    for (int b = 0; b < TM * TN; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        f32x4 v;
#pragma unroll
        for (int x = 0; x < 4; ++x) v[x] = acc[b / TM][b % TM][4 * r + x] * unit[b % TM];
        red[((wave * TM * TN + b) * 4 + r) * 64 + lane] = v;
      }
    __syncthreads();
    unsigned char* stage = lds + 4 * TM * TN * 4096 + wave * (32 * 80);
    for (int b = wk; b < TM * TN; b += WK) {
      const int n = b / TM, m = b % TM;
      const int tok0 = m0 + (wm * TM + m) * 32;
      const float f = m_all[min(tok0 + i32, M - 1)] * (1.0f / kE4M3Max);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        f32x4 v = red[(((wave % (WM * WN)) * TM * TN + b) * 4 + r) * 64 + lane];
#pragma unroll
        for (int k = 1; k < WK; ++k) v += red[(((wave % (WM * WN) + k * WM * WN) * TM * TN + b) * 4 + r) * 64 + lane];
        u32x2 o;
        o[0] = pack_bf16(v[0] * f, v[1] * f);
        o[1] = pack_bf16(v[2] * f, v[3] * f);
        *reinterpret_cast<u32x2*>(stage + i32 * 80 + 16 * r + 8 * hh) = o;
      }
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        const int row = i * 16 + lane / 4, piece = lane & 3;
        const u32x4 o = *reinterpret_cast<const u32x4*>(stage + row * 80 + 16 * piece);
        const int tok = tok0 + row, ch = n0 + (wn * TN + n) * 32 + 8 * piece;
        if (tok < M && ch < N) *reinterpret_cast<u32x4*>(c + (int64_t)tok * ldc + ch) = o;
      }
    }
    return;
  }
  constexpr int kPitch = 64 * TN + 16;
  unsigned char* stage = lds + wave * (32 * kPitch);
#pragma unroll
  for (int m = 0; m < TM; ++m) {
    const int tok0 = m0 + (wm * TM + m) * 32;
    const float f = m_run[m] * (1.0f / kE4M3Max);
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
// The tiles: token and channel blocks of 32 per wavefront; wavefronts along tokens, channels and the axis;
// 64-byte pieces of a row per stage; stages; wavefronts a SIMD is to hold.  (Two: the sums then stay in registers that
// the vector ALU reaches; the 512-register form would move each of them over and back to rescale it.)  With them the
// expected us of a launch: `launch` + rounds over the 256 compute units x (`round` + (`piece` + `full` x the share of
// the units in use) per 128 k), where a second workgroup of a compute unit takes `second` of the first one's time,
// + the stores of c.  Fitted to graph replays of every tile on 330 products of 1 to 4096 tokens, 32 to 8192 channels
// and 512 to 8192 k (within 12 % for nine in ten); the tile chosen by them takes 0.4 % more than the best one, 9 %
// at worst.
struct GShape { int m, n; double launch, round, piece, full, second; };
#define RF_GTILES(X)                                                                                                   \
  X(0, (4, 2, 2, 4, 1, 1, 4, 2), 0.0, 4.93, 1.133, 0.529, 1.0) X(1, (2, 2, 2, 2, 1, 2, 2, 2), 1.88, 0.78, 0.67, 0.188, 0.054) \
  X(2, (1, 2, 2, 2, 1, 2, 3, 2), 2.65, 0.27, 0.326, 0.099, 0.435) X(3, (1, 1, 2, 2, 1, 2, 4, 2), 2.04, 0.62, 0.226, 0.077, 0.375) \
  X(4, (1, 1, 1, 2, 2, 2, 4, 1), 1.4, 1.67, 0.17, 0.029, 1.0) X(5, (1, 1, 1, 1, 4, 2, 4, 1), 1.37, 1.94, 0.104, 0.018, 1.0)
#define RF_SHAPE_OF(TM, TN, WM, WN, WK, KH, NS, OCC) 32 * TM * WM, 32 * TN * WN
#define RF_THREADS_OF(TM, TN, WM, WN, WK, KH, NS, OCC) WM * WN * WK * kWave
#define RF_SHAPE(I, P, L, R, S, F, W) {RF_SHAPE_OF P, L, R, S, F, W},
constexpr GShape kGShapes[] = {RF_GTILES(RF_SHAPE)};
constexpr int kPadRows = 256;  // the codes hold whole tiles of rows
constexpr int kMaxThreads = 512;  // of a workgroup

double tile_us(const GShape& g, int M, int K, int N) {
  const double tiles = ceil((double)M / g.m) * ceil((double)N / g.n);
  const double rounds = ceil(tiles / 256), seconds = floor(rounds / 2);
  return g.launch + (rounds - seconds * (1.0 - g.second)) * (g.round + (g.piece + g.full * tiles / (256 * rounds)) * (K / 128)) +
         M * (double)N / 1.5e6;
}
int best_tile(int M, int K, int N) {
  int best = 0;
  double best_us = tile_us(kGShapes[0], M, K, N);
  for (int i = 1; i < (int)(sizeof(kGShapes) / sizeof(kGShapes[0])); ++i) {
    const double us = tile_us(kGShapes[i], M, K, N);
    if (us < best_us) best = i, best_us = us;
  }
  return best;
}
int64_t padded(int rows) { return ((int64_t)rows + kPadRows - 1) / kPadRows * kPadRows; }
// Bytes of a row: its codes and a maximum for every 128 of them.
int64_t row_bytes(int64_t K) { return K + K / 32; }
// Tokens beyond what kFp8WorkspaceMax holds go slab by slab through the same workspace.
int slab_rows(int M, int K) {
  const int64_t fit = kFp8WorkspaceMax / row_bytes(K) / kPadRows * kPadRows;
  return (int)(fit < M ? fit : M);
}
}  // namespace

// Both launches against the single one.  The quantisation reads a and writes the codes (2.7 us for the smallest,
// 17.7 for 4096 x 8192).  A second launch adds some 3.5 us to a call that is waited for (none to calls in a row);
// 0.9 for the fits' errors.  Of the 330 products above this takes 122, 1.86 times faster in a row, the least 1.25.  (Below 8 tokens
// the single launch's figure is too high at a long axis: 2 x 5248 x 2408 takes 11.0 there and 10.9 here.)
bool fp8_quant_gemm_two_pass_wins(int M, int K, int N, double single_us) {
  if (K >= (1 << 23) || slab_rows(M, K) < (M < 2048 ? M : 2048)) return false;  // 32-bit offsets inside a tile
  if (M < 8) return false;
  const double most = 0.9 * single_us - 3.5 - 2.6 - 0.46e-6 * M * (double)K;
  if (most <= 3.4) return false;  // (no tile takes less: the smallest calls end here, their host time counts)
  return tile_us(kGShapes[best_tile(M, K, N)], M, K, N) < most;
}

size_t fp8_quant_gemm_two_pass_bytes(int M, int K) { return (size_t)(padded(slab_rows(M, K)) * row_bytes(K)); }

int fp8_quant_gemm_two_pass_tile(int M, int K, int N) {
  const GShape g = kGShapes[best_tile(M, K, N)];
  return g.m * 1000 + g.n;
}

namespace {
void launch_quant(const bf16_t* a, unsigned char* codes, float* maxima, int M, int K, int64_t lda, int pitch, hipStream_t s) {
  const int nv = K / 8;
  const int run = M >= 2048 ? 32 : 1;
#define RF_QUANT(VPT, WPR)                                                                                        \
  hipLaunchKernelGGL((fp8_quant_rows_kernel<VPT, WPR>),                                                          \
                     dim3((unsigned)(WPR == 1 ? (M + 3) / 4 : (M + 8 * run - 1) / (8 * run) * (8 * run))),        \
                     dim3(kGThreads), 0, s, a, codes, maxima, M, K, lda, pitch, run)
  if (nv <= 64) RF_QUANT(1, 1);
  else if (nv <= 128) RF_QUANT(2, 1);
  else if (nv <= 256) RF_QUANT(1, 4);
  else if (nv <= 512) RF_QUANT(2, 4);
  else if (nv <= 1024) RF_QUANT(4, 4);
  else RF_QUANT(0, 4);
#undef RF_QUANT
}
}  // namespace

hipError_t launch_fp8_quant_gemm_two_pass(const void* a, const void* w, void* c, int M, int K, int N, int64_t lda,
                                          int64_t ldw, int64_t ldc, void* workspace, hipStream_t s) {
  const int slab = slab_rows(M, K);
  unsigned char* codes = (unsigned char*)workspace;
  const int pitch = (int)padded(slab);
  float* maxima = (float*)(codes + (int64_t)pitch * K);  // [tile of 128 k][row]
  for (int64_t r0 = 0; r0 < M; r0 += slab) {
    const int rows = (int)(M - r0 < slab ? M - r0 : slab);
    const int tile = best_tile(rows, K, N);
    const GShape g = kGShapes[tile];
    const int n_mt = (rows + g.m - 1) / g.m, n_nt = (N + g.n - 1) / g.n;
    // a grid of 2^32 threads or more is not launched whole
    if ((int64_t)n_mt * n_nt >= ((int64_t)1 << 32) / kMaxThreads) return hipErrorInvalidValue;
    launch_quant((const bf16_t*)a + r0 * lda, codes, maxima, rows, K, lda, pitch, s);
    bf16_t* cs = (bf16_t*)c + r0 * ldc;
#define RF_GEMM_OF(TM, TN, WM, WN, WK, KH, NS, OCC) fp8_gemm_kernel<TM, TN, WM, WN, WK, KH, NS, OCC>
#define RF_GEMM(I, P, L, R, S, F, W)                                                                                   \
  if (tile == I)                                                                                                  \
    hipLaunchKernelGGL((RF_GEMM_OF P), dim3((unsigned)(n_mt * n_nt)), dim3(RF_THREADS_OF P), 0, s, codes, maxima, \
                       (const unsigned char*)w, cs, rows, K, N, ldw, ldc, pitch, n_mt, n_nt);
    RF_GTILES(RF_GEMM)
#undef RF_GEMM
    if (hipError_t e = hipGetLastError()) return e;
  }
  return hipSuccess;
}

}  // namespace rf
