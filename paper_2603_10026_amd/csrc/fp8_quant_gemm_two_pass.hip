// FP8 per-token quantisation + GEMM in two launches, for callers that hand over a workspace:
//   1. fp8_quant_rows_kernel: m_i = max_k |a[i,k]| and the codes q(MAX a[i,k] / m_i), MAX = 448,
//      one read of a;
//   2. fp8_gemm_kernel: c[i,n] = (m_i / MAX) sum_k code[i,k] w[n,k].
// The single-launch kernels quantise a token tile once for every 256 or 512 channels beside the
// matrix pipe and rescale their sums whenever a running maximum moves; here the contraction is
// nothing but matrix instructions and their operands, and half the token bytes.
//
// The contraction.  C^T = W A_q^T with v_mfma_f32_32x32x64_f8f6f4 (A = channels, B = tokens: an
// accumulator lane holds one token, one scale).  A workgroup of 4 wavefronts owns a tile of
// 32 TM WM tokens x 32 TN WN channels; tokens and channels both lie with k innermost, so a stage
// is KH x 64 bytes of every row, fetched by direct-to-LDS loads into a ring of NS stages and read
// as the operands lie.  In phase t a wavefront multiplies stage t, whose operands it already
// holds in registers, requests those of stage t+1 behind its first MFMAs, and requests stage t+NS
// into the slot that stage t left: no wavefront waits for LDS data behind the one barrier of a
// phase, and a tile has NS - 1 phases to arrive.
//
// What bounds it.  Large products: the matrix pipe beside LDS (a 256 x 256 tile over 4 wavefronts
// reads 64 KB of operands and writes 32 KB of tiles per 64 k, 768 of the 1024 clocks that its
// matrix instructions take).  4096 x 8192 x 3584: 15.8 us of quantisation (6.3 TB/s) + 92.5 us of
// contraction (2.6 PFLOP/s), where the single launch takes 142 to 160; 4096 x 3584 x 8192: 148 ->
// 109.  Smaller ones: the lines a compute unit has in flight (50 to 70 GB/s each), so tiles are
// made as small as fills the chip, and below 64 x 64 the wavefronts take parts of the axis (WK)
// rather than of the tile: 1348 x 3456 x 2336 46 -> 21 us, 141 x 3456 x 7200 42.6 -> 13.4,
// 64 x 8192 x 8192 46 -> 15.8, 64 x 4096 x 4096 13.5 -> 8.5.
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

// WPR wavefronts per row, VPT vectors of 8 values per lane held in registers (VPT = 0: a row of
// any length is read twice, the second time from the cache).
template <int VPT, int WPR>
__global__ __launch_bounds__(kGThreads) void fp8_quant_rows_kernel(const bf16_t* __restrict__ a,
                                                                   unsigned char* __restrict__ codes,
                                                                   float* __restrict__ row_max, int M, int K,
                                                                   int64_t lda) {
  constexpr int kRows = 4 / WPR;
  __shared__ float s_max[4];
  const int wave = threadIdx.x >> 6;
  const int row = blockIdx.x * kRows + (WPR == 1 ? wave : 0);
  const int vec = WPR == 1 ? (threadIdx.x & 63) : threadIdx.x;  // this lane's first vector of the row
  const int step = 64 * WPR;
  const int nv = K / 8;
  if (WPR == 1 && row >= M) return;
  const u32x4* src = reinterpret_cast<const u32x4*>(a + (int64_t)row * lda);
  u32x2* dst = reinterpret_cast<u32x2*>(codes + (int64_t)row * K);
  constexpr int kHeld = VPT > 0 ? VPT : 1;
  u32x4 x[kHeld];
  u16x2 mx = {0, 0};
  if constexpr (VPT > 0) {
#pragma unroll
    for (int i = 0; i < VPT; ++i) x[i] = src[min(vec + i * step, nv - 1)];
#pragma unroll
    for (int i = 0; i < VPT; ++i) mx = absmax8(mx, x[i]);
  } else {
    for (int i = vec; i < nv; i += step) mx = absmax8(mx, src[i]);
  }
  float m = __uint_as_float((uint32_t)(mx[0] > mx[1] ? mx[0] : mx[1]) << 16);
  m = wave_max(m);
  if constexpr (WPR == 4) {
    if ((threadIdx.x & 63) == 0) s_max[wave] = m;
    __syncthreads();
    m = fmaxf(fmaxf(s_max[0], s_max[1]), fmaxf(s_max[2], s_max[3]));
  }
  if (vec == 0) row_max[row] = m;
  const float s = m > 0.f ? kE4M3Max / m : 0.f;  // IEEE division: it decides the codes
  auto put = [&](int i, const u32x4& v) {
    u32x2 o;
    o[0] = (uint32_t)codes4(v[0], v[1], s);
    o[1] = (uint32_t)codes4(v[2], v[3], s);
    dst[i] = o;
  };
  if constexpr (VPT > 0) {
#pragma unroll
    for (int i = 0; i < VPT; ++i)
      if (vec + i * step < nv) put(vec + i * step, x[i]);
  } else {
    for (int i = vec; i < nv; i += step) put(i, src[i]);
  }
}

template <int TM, int TN, int WM, int WN, int WK, int KH, int NS>
struct GTile {
  static_assert(WM * WN * WK == 4, "4 wavefronts");
  static constexpr int kM = 32 * TM * WM, kN = 32 * TN * WN;
  static constexpr int kRowB = 64 * KH;                  // bytes of a row in a stage
  static constexpr int kGroupB = (kM + kN) * kRowB;      // what one of the WK parts of a stage holds
  static constexpr int kStageB = WK * kGroupB;
  // direct-to-LDS loads per wavefront and stage
  static constexpr int kLoadsA = WK * kM * kRowB / 4096, kLoadsW = WK * kN * kRowB / 4096, kLoads = kLoadsA + kLoadsW;
  static_assert(WK * kM * kRowB % 4096 == 0 && WK * kN * kRowB % 4096 == 0, "whole loads");
  // output staging: 32 tokens per wavefront (padded rows); with WK > 1 the sums of all wavefronts before that
  static constexpr int kOutB = WK > 1 ? 4 * TM * TN * 4096 + 4 * 32 * 80 : 4 * 32 * (64 * TN + 16);
  static constexpr int kLdsB = NS * kStageB > kOutB ? NS * kStageB : kOutB;
};

template <int TM, int TN, int WM, int WN, int WK, int KH, int NS, int OCC>
__global__ __launch_bounds__(kGThreads, OCC) void fp8_gemm_kernel(
    const unsigned char* __restrict__ codes, const float* __restrict__ row_max, const unsigned char* __restrict__ w,
    bf16_t* __restrict__ c, int M, int K, int N, int64_t ldw, int64_t ldc, int n_mtiles, int n_ntiles) {
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
    const int row = (4 * e + wave) % kLA * kRowsL + lrow;  // (the workspace holds whole tiles of rows)
    a_off[e] = (uint32_t)(row * K + ((lslot ^ swz(row)) << 4));
  }
#pragma unroll
  for (int e = 0; e < T::kLoadsW; ++e) {
    const int row = (4 * e + wave) % kLW * kRowsL + lrow;  // channels past the end repeat the last one
    w_off[e] = (uint32_t)(min(row, N - 1 - n0) * (int)ldw + ((lslot ^ swz(row)) << 4));
  }
  const unsigned char* abase = codes + (int64_t)m0 * K;
  const unsigned char* wbase = w + (int64_t)n0 * ldw;
  // load e of stage t (past the end of the axis the last piece once more, which nothing multiplies)
  auto request = [&](int e, int t, uint32_t slot_off) {
    const bool tok = e < T::kLoadsA;
    const int idx = 4 * (tok ? e : e - T::kLoadsA) + wave;
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

  // Phase t: see the head of the file.  `cur`: which set of operand registers stage t is in.
  constexpr int kMfmas = KH * TM * TN, kReads = KH * (TM + TN);
  constexpr int kRate = (2 * kReads + kMfmas - 1) / kMfmas;  // operands behind an MFMA: all in the first half
  uint32_t slot = 0;  // byte offset of stage t's ring slot
  auto phase = [&](auto cur_c, int t) {
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
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * T::kLoads) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    RF_FENCE
#pragma unroll
    for (int q = 0; q < kMfmas; ++q) {
      const int kh = q / (TM * TN), n = q / TM % TN, m = q % TM;
      acc[n][m] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(fw[cur][kh][n], ft[cur][kh][m], acc[n][m], 0, 0, 0, 0, 0, 0);
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
        for (int q = 0; q < kMfmas; ++q) {
          const int kh = q / (TM * TN), n = q / TM % TN, m = q % TM;
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
#pragma unroll
    for (int b = 0; b < TM * TN; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        f32x4 v;
#pragma unroll
        for (int x = 0; x < 4; ++x) v[x] = acc[b / TM][b % TM][4 * r + x];
        red[((wave * TM * TN + b) * 4 + r) * 64 + lane] = v;
      }
    __syncthreads();
    unsigned char* stage = lds + 4 * TM * TN * 4096 + wave * (32 * 80);
    for (int b = wk; b < TM * TN; b += WK) {
      const int n = b / TM, m = b % TM;
      const int tok0 = m0 + (wm * TM + m) * 32;
      const float f = tok0 + i32 < M ? row_max[tok0 + i32] * (1.0f / kE4M3Max) : 0.f;
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
    const float f = tok0 + i32 < M ? row_max[tok0 + i32] * (1.0f / kE4M3Max) : 0.f;
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
// 64-byte pieces of a row per stage; stages; workgroups a compute unit is to hold.  With them the expected us of
// a launch: `launch` + rounds over the 256 compute units x (`round` + `piece` per 128 k).  Fitted to graph
// replays of every tile on 260 products of 1 to 4096 tokens, 16 to 8192 channels and 512 to 8192 k (within 10 %
// for nine in ten); the tile chosen by them takes 0.3 % more than the best one, 13 % at worst.
struct GShape { int m, n; double launch, round, piece; };
#define RF_GTILES(X)                                                                               \
  X(0, (4, 4, 2, 2, 1, 1, 4, 1), 0.0, 6.3, 1.095) X(1, (2, 4, 2, 2, 1, 2, 3, 1), 0.0, 5.4, 0.553)  \
  X(2, (2, 2, 2, 2, 1, 2, 4, 1), 0.0, 4.3, 0.338) X(3, (1, 2, 2, 2, 1, 2, 3, 2), 1.4, 1.7, 0.271)  \
  X(4, (1, 1, 2, 2, 1, 2, 4, 2), 1.9, 1.0, 0.173) X(5, (1, 1, 1, 2, 2, 2, 4, 1), 1.1, 2.0, 0.125)  \
  X(6, (1, 1, 1, 1, 4, 2, 4, 1), 1.2, 2.1, 0.084)
#define RF_SHAPE_OF(TM, TN, WM, WN, WK, KH, NS, OCC) 32 * TM * WM, 32 * TN * WN
#define RF_SHAPE(I, P, L, R, S) {RF_SHAPE_OF P, L, R, S},
constexpr GShape kGShapes[] = {RF_GTILES(RF_SHAPE)};
constexpr int kPadRows = 256;  // the codes hold whole tiles of rows

double tile_us(const GShape& g, int M, int K, int N) {
  const double tiles = ceil((double)M / g.m) * ceil((double)N / g.n);
  return g.launch + ceil(tiles / 256) * (g.round + g.piece * (K / 128));
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
int64_t slab_bytes(int64_t rows, int64_t K) { return (rows + kPadRows - 1) / kPadRows * kPadRows * K + 4 * ((rows + 3) / 4 * 4); }
// Tokens beyond what kFp8WorkspaceMax holds go slab by slab through the same workspace.
int slab_rows(int M, int K) {
  const int64_t fit = kFp8WorkspaceMax / ((int64_t)K + 4) / kPadRows * kPadRows;
  return (int)(fit < M ? fit : M);
}
}  // namespace

// Both launches against the single one.  The quantisation reads a and writes the codes (2.2 us for the smallest,
// 15.9 for 4096 x 8192).  A second launch adds some 3.5 us to a call that is waited for (none to calls in a row):
// 12 x 2432 x 5664 takes 7.1 us here and 9.0 there in a row, but 26.4 and 21.7 alone, and stays there;
// 64 x 4096 x 4096 takes 8.5 and 13.5 in a row and the same alone.
bool fp8_quant_gemm_two_pass_wins(int M, int K, int N, double single_us) {
  if (K >= (1 << 23) || slab_rows(M, K) < (M < 2048 ? M : 2048)) return false;  // 32-bit offsets inside a tile
  const double quant = 1.9 + 3.0 * M * (double)K / 7.2e6;
  if (quant + 2.9 + 3.5 >= 0.95 * single_us) return false;  // (no tile takes less: the smallest calls end here, their host time counts)
  return quant + tile_us(kGShapes[best_tile(M, K, N)], M, K, N) + 3.5 < 0.95 * single_us;
}

size_t fp8_quant_gemm_two_pass_bytes(int M, int K) { return (size_t)slab_bytes(slab_rows(M, K), K); }

int fp8_quant_gemm_two_pass_tile(int M, int K, int N) {
  const GShape g = kGShapes[best_tile(M, K, N)];
  return g.m * 1000 + g.n;
}

namespace {
void launch_quant(const bf16_t* a, unsigned char* codes, float* row_max, int M, int K, int64_t lda, hipStream_t s) {
  const int nv = K / 8;
#define RF_QUANT(VPT, WPR)                                                                                        \
  hipLaunchKernelGGL((fp8_quant_rows_kernel<VPT, WPR>), dim3((unsigned)((M + 4 / WPR - 1) / (4 / WPR))),          \
                     dim3(kGThreads), 0, s, a, codes, row_max, M, K, lda)
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
  float* row_max = (float*)(codes + (int64_t)(slab + kPadRows - 1) / kPadRows * kPadRows * K);
  for (int r0 = 0; r0 < M; r0 += slab) {
    const int rows = M - r0 < slab ? M - r0 : slab;
    const int tile = best_tile(rows, K, N);
    const GShape g = kGShapes[tile];
    const int n_mt = (rows + g.m - 1) / g.m, n_nt = (N + g.n - 1) / g.n;
    // a grid of 2^32 threads or more is not launched whole
    if ((int64_t)n_mt * n_nt >= ((int64_t)1 << 32) / kGThreads) return hipErrorInvalidValue;
    launch_quant((const bf16_t*)a + r0 * lda, codes, row_max, rows, K, lda, s);
    bf16_t* cs = (bf16_t*)c + r0 * ldc;
#define RF_GEMM_OF(TM, TN, WM, WN, WK, KH, NS, OCC) fp8_gemm_kernel<TM, TN, WM, WN, WK, KH, NS, OCC>
#define RF_GEMM(I, P, L, R, S)                                                                                    \
  if (tile == I)                                                                                                  \
    hipLaunchKernelGGL((RF_GEMM_OF P), dim3((unsigned)(n_mt * n_nt)), dim3(kGThreads), 0, s, codes, row_max,      \
                       (const unsigned char*)w, cs, rows, K, N, ldw, ldc, n_mt, n_nt);
    RF_GTILES(RF_GEMM)
#undef RF_GEMM
    if (hipError_t e = hipGetLastError()) return e;
  }
  return hipSuccess;
}

}  // namespace rf
