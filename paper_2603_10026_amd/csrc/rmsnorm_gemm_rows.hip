// RMSNorm + linear for few rows (the tokens of a decode step): the "sum + sum" cascade of
// rmsnorm_gemm.hip, cut for launches whose time is the trip of w from memory.
//
// A 128 x 512 tile of the large kernel leaves all but N / 512 compute units idle here.  This
// kernel cuts the output into 16 MT x 16 C tiles (C columns of w per lane) and gives every
// workgroup the whole contraction axis, split over its 4 wavefronts by interleaved 64-k steps:
// no LDS, no barrier and no shared state until the wavefronts' sums are added at the end.
//
//   Y^T = W^T X^T      A = W^T, B = X^T (16x16x32 bf16 MFMA)
//
// A lane loads C neighbouring columns of 8 rows of w, which after pairing rows in registers is
// the A operand of C MFMAs; the row of x times g, rounded to bf16 as in the large kernel, is the B
// operand.  (The roundings a row meets do not depend on the kernel its batch selects: what is left
// between the two is the order of fp32 sums.)  ss is the diagonal of X X^T, taken by the matrix
// pipe from the x that is in registers already.
//
// (This kernel serves tiles of 64 rows or 128 columns, and of the smaller ones those that `straight` below names;
// the others go through LDS.)
// What bounds it: the 128-byte lines a compute unit can have on their way.  A read of w alone in
// this pattern takes 15.9 us when w comes from HBM (4096 x 4096, C = 2, 128 workgroups), 17.7 us with
// whole lines and half the workgroups (C = 4), and cache-policy bits change nothing; the last 50 GB/s
// per compute unit are its 32 KB of L1 lines in flight over the memory latency.  Two steps in
// flight and 4 wavefronts are therefore faster than 8 wavefronts with more (which evict each
// other's lines): 48 x 4096 x 4096, repeated on the same w (33 MB: it stays in the memory-side cache),
// takes 13.8 us a call here, and 86.4 in 128 x 512 tiles.  A few hundred rows are bound by the same lines in
// either kernel, and 64 x 128 tiles move fewest of them per compute unit in use: 1024 x 8192 x 2048
// takes 57 to 62 us, by the card, against 171.
#include <math.h>

#include "rf_device.h"
#include "rf_launch.h"

namespace rf {

namespace {
constexpr int kRWaves = 4;
constexpr int kRThreads = kRWaves * kWave;
}  // namespace

// P: steps of 32 k in flight per wavefront.  (Two workgroups per compute unit in the bounds: with
// more registers to give away the compiler keeps the sums in accumulation registers and copies
// them around every step, 48 x 4096 x 4096 16.5 us.)
template <int MT, int C, int P>
__global__ __launch_bounds__(kRThreads, 2) void rmsnorm_gemm_rows_kernel(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ g, const bf16_t* __restrict__ w,
    bf16_t* __restrict__ y, int M, int K, int N, int64_t ldx, int64_t ldw, int64_t ldy,
    float inv_k, float eps, int n_mtiles) {
  constexpr int CD = C / 2;  // 32-bit words of w per lane and k-row
  // Requests are waited for in order.  Two row tiles against a narrow tile of w have as much work in
  // x g as in pairing w and start it first (48 x 4096 x 4096: 14.5 us, 15.2 the other way round);
  // the other shapes want w first (32 x 8192 x 1024 in one row tile: 15.6 and 20.3).
  constexpr bool kXFirst = MT == 2 && C == 2;
  __shared__ f32x4 s_acc[kRWaves][C * MT][kWave];
  __shared__ float s_ss[kRWaves][16 * MT];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15;
  const int g4 = lane >> 4;

  // Workgroups are dealt round-robin to the 8 XCDs, each with its own L2.  The row tiles of a
  // column tile, and the column tiles that share the 128-byte lines of w, go to one XCD; these
  // groups are dealt round-robin, so that every XCD reads all over a row of w.
  constexpr int GC = C >= 4 ? 1 : 4 / C;  // column tiles per 128-byte line
  const int unit = GC * n_mtiles;
  const int j = blockIdx.x >> 3;
  const int mt = __builtin_amdgcn_readfirstlane(j % unit % n_mtiles);
  const int nt = __builtin_amdgcn_readfirstlane((j / unit * 8 + (blockIdx.x & 7)) * GC + j % unit / n_mtiles);
  const int m0 = mt * 16 * MT, n0 = nt * 16 * C;
  if (n0 >= N) return;

  const int mine = 2 * ((K / 64 - wave + kRWaves - 1) / kRWaves);  // 32-k steps of this wavefront, in pairs

  // Buffer loads: a scalar byte offset per (step, row) and one loop-invariant lane offset, so the
  // loop has no vector address arithmetic.  Columns past N re-read the last ones and are not stored.
  const auto wrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(w), 0, 0xffffffffu, 0x00020000);
  const auto xrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(x + (int64_t)m0 * ldx), 0, 0xffffffffu, 0x00020000);
  const auto grs = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(g), 0, 0xffffffffu, 0x00020000);
  const uint32_t ldw2 = (uint32_t)ldw * 2;
  const uint32_t w_lane = 8 * g4 * ldw2 + min(n0 + C * i16, N - C) * 2;
  uint32_t x_lane[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t)
    x_lane[t] = (uint32_t)(min(m0 + 16 * t + i16, M - 1) - m0) * (uint32_t)(ldx * 2) + 16 * g4;

  uint32_t wr[P][8][CD];
  u32x4 xr[P][MT], gr[P];
  auto load = [&](int p, int i) {
    const int ii = min(i, mine - 1);
    const uint32_t k0 = (wave + kRWaves * (ii >> 1)) * 64 + (ii & 1) * 32;
    const uint32_t wo = k0 * ldw2;
    auto load_x = [&] {
#pragma unroll
      for (int t = 0; t < MT; ++t) xr[p][t] = __builtin_amdgcn_raw_buffer_load_b128(xrs, x_lane[t], k0 * 2, 0);
      gr[p] = __builtin_amdgcn_raw_buffer_load_b128(grs, 16 * g4, k0 * 2, 0);
    };
    if constexpr (kXFirst) load_x();
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if constexpr (CD == 4) {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(wrs, w_lane, wo + e * ldw2, 0);
#pragma unroll
        for (int d = 0; d < CD; ++d) wr[p][e][d] = v[d];
      } else if constexpr (CD == 1) {
        wr[p][e][0] = __builtin_amdgcn_raw_buffer_load_b32(wrs, w_lane, wo + e * ldw2, 0);
      } else {
        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(wrs, w_lane, wo + e * ldw2, 0);
#pragma unroll
        for (int d = 0; d < CD; ++d) wr[p][e][d] = v[d];
      }
    }
    if constexpr (!kXFirst) load_x();
  };

  f32x4 acc[C][MT], sq[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    sq[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < C; ++c) acc[c][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  auto step = [&](int p) {
    u32x4 af[C];
#pragma unroll
    for (int e2 = 0; e2 < 4; ++e2)
#pragma unroll
      for (int d = 0; d < CD; ++d) {
        af[2 * d][e2] = pair_lo(wr[p][2 * e2][d], wr[p][2 * e2 + 1][d]);
        af[2 * d + 1][e2] = pair_hi(wr[p][2 * e2][d], wr[p][2 * e2 + 1][d]);
      }
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const bf16x8 raw = __builtin_bit_cast(bf16x8, xr[p][t]);
      u32x4 xg;
#pragma unroll
      for (int e2 = 0; e2 < 4; ++e2)
        xg[e2] = pack_bf16(bf16_lo(xr[p][t][e2]) * bf16_lo(gr[p][e2]), bf16_hi(xr[p][t][e2]) * bf16_hi(gr[p][e2]));
      const bf16x8 b = __builtin_bit_cast(bf16x8, xg);
#pragma unroll
      for (int c = 0; c < C; ++c)
        acc[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, af[c]), b, acc[c][t], 0, 0, 0);
      sq[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(raw, raw, sq[t], 0, 0, 0);
    }
  };

  if (mine > 0) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
      load(p, p);
      __builtin_amdgcn_sched_barrier(0);
    }
    int i = 0;
    for (; i + P <= mine; i += P) {
#pragma unroll
      for (int p = 0; p < P; ++p) {
        step(p);
        load(p, i + P + p);
        __builtin_amdgcn_sched_barrier(0);  // (keeps the requests in the order they are waited for)
      }
    }
#pragma unroll
    for (int p = 0; p < P; ++p)
      if (i + p < mine) step(p);
  }

  // ---- add the wavefronts' sums ----
  // acc[c][t] of lane (i16, g4), element r: row m0 + 16 t + i16, column n0 + C (4 g4 + r) + c
#pragma unroll
  for (int c = 0; c < C; ++c)
#pragma unroll
    for (int t = 0; t < MT; ++t) s_acc[wave][c * MT + t][lane] = acc[c][t];
  if ((i16 >> 2) == g4) {  // this lane holds the diagonal element of row i16
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const f32x4 s = sq[t];
      const int r = i16 & 3;
      s_ss[wave][16 * t + i16] = r == 0 ? s[0] : r == 1 ? s[1] : r == 2 ? s[2] : s[3];
    }
  }
  __syncthreads();
  for (int idx = tid; idx < MT * kWave; idx += kRThreads) {
    const int t = idx >> 6, l = idx & 63;
    float ss = 0.f;
#pragma unroll
    for (int wv = 0; wv < kRWaves; ++wv) ss += s_ss[wv][16 * t + (l & 15)];
    const float rs = 1.0f / sqrtf(ss * inv_k + eps);
    const int m = m0 + 16 * t + (l & 15);
    const int n = n0 + 4 * C * (l >> 4);
    float out[4][C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
      f32x4 v = s_acc[0][c * MT + t][l];
#pragma unroll
      for (int wv = 1; wv < kRWaves; ++wv) v += s_acc[wv][c * MT + t][l];
#pragma unroll
      for (int r = 0; r < 4; ++r) out[r][c] = v[r] * rs;
    }
    if (m < M) {
#pragma unroll
      for (int h = 0; h < C / 2; ++h) {  // 8 columns at a time (N is a multiple of 8)
        u32x4 o;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int q = 8 * h + 2 * j;
          o[j] = pack_bf16(out[q / C][q % C], out[(q + 1) / C][(q + 1) % C]);
        }
        if (n + 8 * h < N) *reinterpret_cast<u32x4*>(y + (int64_t)m * ldy + n + 8 * h) = o;
      }
    }
  }
}

namespace {
constexpr int kLWaves = 8;
constexpr int kLThreads = kLWaves * kWave;
constexpr int kGChunk = 4096;  // k whose g is held in LDS
}  // namespace

// The smaller tiles through LDS: 8 wavefronts deal the 64-k pieces of the axis among themselves, each with a stage
// of its own that direct-to-LDS loads fill (a row of x is 128 bytes of it, a row of w 32 C), so there is still no
// barrier in the loop but where the next 4096 values of g are fetched.  x and w leave LDS in operand layout, w by
// transpose reads: no pairing of rows in registers, and the loads hold no registers.  A piece is requested as soon as
// the one before is in registers; rings of 2 or 4 stages with 4 wavefronts are no faster or slower (48 x 4096 x 4096
// 13.2 and 14.1 us, 13.0 here; 16 x 4096 x 4096 in 16 x 32 tiles 11.8 and 12.4, 11.5 here): what counts is that
// many wavefronts have requests under way, not how many each has.  us a call, registers / LDS: 48 x 4096 x 4096
// 15.2 / 13.0, 16 x 4096 x 4096 14.2 / 11.5, 154 x 4416 x 1024 14.5 / 10.4, 23 x 2432 x 1008 7.2 / 5.7, 5 x 1920 x 832
// 6.3 / 5.1 (140 products, 1.11 x on average).
template <int MT, int C>
__global__ __launch_bounds__(kLThreads, 2) void rmsnorm_gemm_rows_lds_kernel(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ g, const bf16_t* __restrict__ w,
    bf16_t* __restrict__ y, int M, int K, int N, int64_t ldx, int64_t ldw, int64_t ldy,
    float inv_k, float eps, int n_mtiles) {
  constexpr int kXB = 2048 * MT, kWB = 2048 * C, kStageB = kXB + kWB;  // 64 k: [row][k], [k][column]
  constexpr int kXL = 2 * MT, kWL = 2 * C, kL = kXL + kWL;             // direct-to-LDS loads of a stage
  constexpr int kRedB = C * MT * 1024;                                 // a wavefront's sums
  __shared__ __attribute__((aligned(1024))) unsigned char lds[kLWaves * (kStageB > kRedB ? kStageB : kRedB)];
  __shared__ __attribute__((aligned(16))) bf16_t s_g[kGChunk];
  __shared__ float s_ss[kLWaves][16 * MT];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15, g4 = lane >> 4;

  constexpr int GC = C >= 4 ? 1 : 4 / C;  // column tiles per 128-byte line
  const int unit = GC * n_mtiles;
  const int j = blockIdx.x >> 3;
  const int mt = __builtin_amdgcn_readfirstlane(j % unit % n_mtiles);
  const int nt = __builtin_amdgcn_readfirstlane((j / unit * 8 + (blockIdx.x & 7)) * GC + j % unit / n_mtiles);
  const int m0 = mt * 16 * MT, n0 = nt * 16 * C;
  if (n0 >= N) return;
  const uint32_t stage = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds + wave * kStageB);
  const unsigned char* st = lds + wave * kStageB;
  // 16-byte slots of a row are XOR-swizzled with the row where the operand reads would meet the same banks
  auto fx = [](int row) { return (row >> 1) & 7; };
  auto fw = [](int krow) { return C == 4 ? 2 * ((krow >> 1) & 1) : 0; };
  uint32_t x_off[kXL], w_off[kWL];
#pragma unroll
  for (int e = 0; e < kXL; ++e) {
    const int row = 8 * e + (lane >> 3);
    x_off[e] = (uint32_t)(min(row, M - 1 - m0) * (uint32_t)(ldx * 2) + (((lane & 7) ^ fx(row)) << 4));
  }
  constexpr int SL = 2 * C;  // 16-byte slots per k-row
#pragma unroll
  for (int e = 0; e < kWL; ++e) {
    const int krow = (64 / SL) * e + lane / SL;
    const int piece = (lane % SL) ^ fw(krow);
    w_off[e] = (uint32_t)(krow * (uint32_t)(ldw * 2) + min(n0 + 8 * piece, N - 8) * 2);
  }
  const char* xb = reinterpret_cast<const char*>(x + (int64_t)m0 * ldx);
  const char* wb = reinterpret_cast<const char*>(w);
  auto request = [&](int first, int i) {  // this wavefront's piece i of those from `first` on
    const int p = first + wave + kLWaves * i;
    const char* xp = xb + (int64_t)p * 128;
    const char* wp = wb + (int64_t)p * 128 * ldw;
#pragma unroll
    for (int e = 0; e < kL; ++e) {
      const bool is_w = e < kWL;
      const uint32_t dst = stage + (is_w ? kXB + e * 1024 : (e - kWL) * 1024);
      const uint32_t off = is_w ? w_off[is_w ? e : 0] : x_off[is_w ? 0 : e - kWL];
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                   :
                   : "s"(dst), "v"(off), "s"(is_w ? wp : xp)
                   : "memory", "m0");
    }
  };
  f32x4 acc[C][MT], sq[MT];
#pragma unroll
  for (int t = 0; t < MT; ++t) {
    sq[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int c = 0; c < C; ++c) acc[c][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4* lds_s16x4;
  uint32_t x_at[2], w_at[2][2][C];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    x_at[kk] = i16 * 128 + (((4 * kk + g4) ^ fx(i16)) << 4);  // (+ 2048 t: the swizzle repeats after 16 rows)
#pragma unroll
    for (int w2 = 0; w2 < 2; ++w2)
#pragma unroll
      for (int c = 0; c < C; ++c) {
        const int krow = 32 * kk + 8 * g4 + 4 * w2 + (i16 >> 2), a = i16 & 3;
        w_at[kk][w2][c] = kXB + krow * 32 * C + (((2 * c + (a >> 1)) ^ fw(krow)) << 4) + 8 * (a & 1);
      }
  }
  for (int kc = 0; kc < K; kc += kGChunk) {
    const int pieces = min(K - kc, kGChunk) / 64;
    const int mine = (pieces - wave + kLWaves - 1) / kLWaves;
    if (mine > 0) request(kc / 64, 0);
    if (kc > 0) __syncthreads();  // (everyone is done with the g before)
    for (int k = tid * 8; k < 64 * pieces; k += kLThreads * 8)
      *reinterpret_cast<u32x4*>(s_g + k) = *reinterpret_cast<const u32x4*>(g + kc + k);
    __syncthreads();
    for (int i = 0; i < mine; ++i) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this piece has landed
      u32x4 xf[2][MT], gf[2];
      s16x4 wf[2][C][2];
      const int k0 = (wave + kLWaves * i) * 64;
#pragma unroll
      for (int kk = 0; kk < 2; ++kk) {
        gf[kk] = *reinterpret_cast<const u32x4*>(s_g + k0 + 32 * kk + 8 * g4);
#pragma unroll
        for (int t = 0; t < MT; ++t) xf[kk][t] = *reinterpret_cast<const u32x4*>(st + x_at[kk] + 2048 * t);
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
          for (int w2 = 0; w2 < 2; ++w2) wf[kk][c][w2] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(st + w_at[kk][w2][c]));
      }
      // the stage is in registers: the next piece takes it
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      if (i + 1 < mine) request(kc / 64, i + 1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int t = 0; t < MT; ++t) {
          const bf16x8 raw = __builtin_bit_cast(bf16x8, xf[kk][t]);
          u32x4 xg;
#pragma unroll
          for (int e2 = 0; e2 < 4; ++e2)
            xg[e2] = pack_bf16(bf16_lo(xf[kk][t][e2]) * bf16_lo(gf[kk][e2]), bf16_hi(xf[kk][t][e2]) * bf16_hi(gf[kk][e2]));
          const bf16x8 b = __builtin_bit_cast(bf16x8, xg);
#pragma unroll
          for (int c = 0; c < C; ++c) {
            const auto a = __builtin_shufflevector(wf[kk][c][0], wf[kk][c][1], 0, 1, 2, 3, 4, 5, 6, 7);
            acc[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), b, acc[c][t], 0, 0, 0);
          }
          sq[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(raw, raw, sq[t], 0, 0, 0);
        }
    }
  }

  // ---- add the wavefronts' sums ----
  // acc[c][t] of lane (i16, g4), element r: row m0 + 16 t + i16, column n0 + 16 c + 4 g4 + r
  __syncthreads();
  f32x4* s_acc = reinterpret_cast<f32x4*>(lds);
#pragma unroll
  for (int c = 0; c < C; ++c)
#pragma unroll
    for (int t = 0; t < MT; ++t) s_acc[(wave * C * MT + c * MT + t) * 64 + lane] = acc[c][t];
  if ((i16 >> 2) == g4) {  // this lane holds the diagonal element of row i16
#pragma unroll
    for (int t = 0; t < MT; ++t) {
      const f32x4 s = sq[t];
      const int r = i16 & 3;
      s_ss[wave][16 * t + i16] = r == 0 ? s[0] : r == 1 ? s[1] : r == 2 ? s[2] : s[3];
    }
  }
  __syncthreads();
  for (int idx = tid; idx < C * MT * 64; idx += kLThreads) {
    const int ct = idx >> 6, l = idx & 63, c = ct / MT, t = ct % MT;
    float ss = 0.f;
    f32x4 v = s_acc[idx];
#pragma unroll
    for (int wv = 1; wv < kLWaves; ++wv) v += s_acc[wv * C * MT * 64 + idx];
#pragma unroll
    for (int wv = 0; wv < kLWaves; ++wv) ss += s_ss[wv][16 * t + (l & 15)];
    const float rs = 1.0f / sqrtf(ss * inv_k + eps);
    const int m = m0 + 16 * t + (l & 15), n = n0 + 16 * c + 4 * (l >> 4);
    if (m < M && n < N) {  // (N is a multiple of 8)
      u32x2 o;
      o[0] = pack_bf16(v[0] * rs, v[1] * rs);
      o[1] = pack_bf16(v[2] * rs, v[3] * rs);
      *reinterpret_cast<u32x2*>(y + (int64_t)m * ldy + n) = o;
    }
  }
}

namespace {
// Tile shapes and what a workgroup of each takes: us for the launch and the sums, us per 1024 k.
// The latter is its lines' way through the compute unit, 46 GB/s of w and x at C <= 4 and 62-67 at
// C = 8, where a lane's load of w is 16 bytes: bigger tiles win as soon as there are enough of them.
struct RowsShape { int mt, c; double us, us_per_k; };
constexpr RowsShape kRowsShapes[] = {{1, 2, 2.9, 2.6}, {2, 2, 3.2, 3.0}, {1, 4, 3.3, 3.05}, {2, 4, 3.7, 4.05},
                                     {4, 4, 4.6, 5.5}, {2, 8, 4.4, 4.6}, {4, 8, 6.0, 6.3}};
// Columns of whole 128-byte lines: two tiles at C = 2, else one.
inline int group_cols(int c) { return c > 4 ? 16 * c : 64; }
// More workgroups than the 32 compute units of an XCD take turns (the column groups are dealt to the
// 8 XCDs, so some may get one more).  Within 10 % of the measured times of all shapes
// for 512 to 8192 k, 512 to 8192 columns and 1 to 2048 rows.
inline double rows_us(const RowsShape& r, int M, int K, int N) {
  const int group = group_cols(r.c), n_groups = (N + group - 1) / group;
  const double wg_xcd = (double)((M + 16 * r.mt - 1) / (16 * r.mt)) * ((n_groups + 7) / 8) * (group / (16 * r.c));
  return 2.0 + (r.us + r.us_per_k * (K / 1024.0) - 2.0) * ceil(wg_xcd / 32);
}
const RowsShape& best_shape(int M, int K, int N) {
  const RowsShape* best = kRowsShapes;
  for (const RowsShape& r : kRowsShapes)
    if (rows_us(r, M, K, N) < rows_us(*best, M, K, N)) best = &r;
  return *best;
}
// Which of the tiles that have both kernels take operands straight into registers.  LDS serves every tile whose w comes
// out of an L2 (several row tiles, which share it: 0.87 to 0.98 of the time in 365 of 365 products), and rows of w that all
// start on the same memory channels (a pitch of whole 256 bytes, which piles up the 4 or 8 rows that a register load
// of w touches: 0.88, 1.02 at most).  What is left is one row tile whose w comes from memory once.  There straight is the
// shorter way, by up to 10 %, where a short axis leaves the LDS kernel's 8 wavefronts without a piece of 64 k each, where many
// workgroups have requests enough under way, and with a handful of rows, whose LDS stages are mostly padding, already
// where few of them do, the fewer the longer the axis.  us straight / LDS, three sets of operands in turn: 48 x 4096 x
// 4096 15.3 / 13.6, 16 x 4096 x 4096 14.7 / 12.6, 37 x 2880 x 616 9.0 / 8.4; 19 x 1408 x 4784 7.55 / 7.9, 18 x 1024 x 6648 7.1 / 7.6,
// 3 x 2304 x 872 6.9 / 7.4, 2 x 768 x 4792 5.0 / 5.3, 1 x 448 x 8776 5.65 / 6.1.  Of 2100 products of 1 to 400 rows, two thirds
// of them drawn after the lines were placed, one is slower than straight by more than 2 % (1 x 7296 x 120, 2.8); the
// others gain 1.08 on average, 1.10 if every one took its better kernel.
bool straight(const RowsShape& r, int M, int K, int N, int64_t ldw) {
  if (r.mt == 2 && r.c == 4) return false;
  if (K <= 256) return true;
  if (M > 16 * r.mt || ldw % 128 == 0) return false;
  const int wg = (N + 16 * r.c - 1) / (16 * r.c);
  return wg > 128 || (M <= 5 && wg > (K <= 2048 ? 40 : K <= 4096 ? 20 : 16));
}
}  // namespace

// The 128 x 512 tiles take 5 us and 20.5 for every 1024 k up to 64 of them, 29 at 256, whatever the
// row count.  Both sides at the line (us here / there): 1024 x 4096 x 4096 68 / 89, 1500 rows 101 / 90;
// 768 x 8192 x 8192 171 / 174, 1024 rows 225 / 172; 2048 x 8192 x 2048 117 / 170.
// (the buffer loads take 32-bit byte offsets inside w; rows of y are stored 16 bytes at a time)
static double large_us(int M, int K, int N) {
  const double wg = (double)((M + 127) / 128) * ((N + 511) / 512);
  return 5.0 + (K / 1024.0) * (20.5 + 8.5 * fmin(fmax((wg - 64) / 192, 0.0), 1.0)) * ceil(wg / 256);
}
bool rmsnorm_gemm_rows_wins(int M, int K, int N, int64_t ldw, const void* y, int64_t ldy) {
  if ((int64_t)K * ldw * 2 >= ((int64_t)1 << 32) || (ldy & 7) != 0 || (reinterpret_cast<uintptr_t>(y) & 15) != 0) return false;
  return 1.15 * rows_us(best_shape(M, K, N), M, K, N) < large_us(M, K, N);
}
// Expected us of the call in one launch.  (Tiles of up to 32 x 64 take 0.9 times what the rule's figures say.)
double rmsnorm_gemm_us(int M, int K, int N) {
  const RowsShape& r = best_shape(M, K, N);
  if (!rmsnorm_gemm_rows_wins(M, K, N, N, nullptr, N)) return large_us(M, K, N);
  return (r.mt <= 2 && r.c <= 4 ? 0.9 : 1.0) * rows_us(r, M, K, N);
}

bool rmsnorm_gemm_rows_straight(int M, int K, int N, int64_t ldw) { return straight(best_shape(M, K, N), M, K, N, ldw); }

int rmsnorm_gemm_rows_tile(int M, int K, int N) {
  const RowsShape& r = best_shape(M, K, N);
  return 16 * r.mt * 1000 + 16 * r.c;
}

hipError_t launch_rmsnorm_gemm_rows(const void* x, const void* g, const void* w, void* y, int M,
                                    int K, int N, int64_t ldx, int64_t ldw, int64_t ldy, float eps,
                                    hipStream_t s) {
  const RowsShape& best = best_shape(M, K, N);
  const int n_mt = (M + 16 * best.mt - 1) / (16 * best.mt);
  const int group = group_cols(best.c);
  const int64_t groups = ((int64_t)N + group - 1) / group;
  const int64_t grid = (groups + 7) / 8 * 8 * (group / (16 * best.c)) * n_mt;
  if (grid > INT32_MAX) return hipErrorInvalidValue;
#define RF_ROWS(MT, C, P)                                                                            \
  if (best.mt == MT && best.c == C)                                                                  \
    hipLaunchKernelGGL((rmsnorm_gemm_rows_kernel<MT, C, P>), dim3((unsigned)grid), dim3(kRThreads), 0, s, \
                       (const bf16_t*)x, (const bf16_t*)g, (const bf16_t*)w, (bf16_t*)y, M, K, N, ldx, ldw, \
                       ldy, 1.0f / (float)K, eps, n_mt);
#define RF_ROWS_LDS(MT, C)                                                                                 \
  if (best.mt == MT && best.c == C)                                                                        \
    hipLaunchKernelGGL((rmsnorm_gemm_rows_lds_kernel<MT, C>), dim3((unsigned)grid), dim3(kLThreads), 0, s, \
                       (const bf16_t*)x, (const bf16_t*)g, (const bf16_t*)w, (bf16_t*)y, M, K, N, ldx, ldw, \
                       ldy, 1.0f / (float)K, eps, n_mt);
  if (straight(best, M, K, N, ldw)) {
    RF_ROWS(1, 2, 4) RF_ROWS(2, 2, 2) RF_ROWS(1, 4, 2)
  } else {
    RF_ROWS_LDS(1, 2) RF_ROWS_LDS(2, 2) RF_ROWS_LDS(1, 4) RF_ROWS_LDS(2, 4)
  }
  RF_ROWS(4, 4, 2) RF_ROWS(2, 8, 2) RF_ROWS(4, 8, 2)
#undef RF_ROWS_LDS
#undef RF_ROWS
  return hipGetLastError();
}

}  // namespace rf
