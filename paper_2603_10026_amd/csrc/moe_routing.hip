// MoE routing: scores GEMM -> softmax -> top-k (paper Appendix A.2, "MoE
// routing"), as a multi-segment cascade (Section 4.3):
//   p[e] = sum_c x[c] w[c,e];  m = max_e p[e];  t = sum_e exp(p[e]-m);
//   s = TopK_e p[e];  output exp(s-m)/t with the experts' indices.
// TopK acts on the raw scores (softmax keeps their order); equal scores are
// ordered by expert index, lowest first.
//
// The router GEMM is skinny (a few thousand tokens x 32..128 experts) and its
// cost is reading x once, so the contraction axis is split over workgroups:
//
// Kernel 1 (scores): workgroup (row block of 4096 / E tokens, k slice).  x and w tiles
//   of 128 k go HBM -> LDS with direct-to-LDS 128-bit loads three tiles ahead of their
//   use (four LDS stages), one barrier per tile.  32x32x16 bf16 MFMAs: X fragments come from 128-bit
//   LDS reads, W fragments from 64-bit transpose reads.  A wavefront owns 32 tokens x 32 experts; the fp32
//   partial scores of the slice are written to the caller's workspace.
// Kernel 2 (cascade): a wavefront per token adds the slices' partial scores in slice
//   order, then runs the cascade over its lanes; with many tokens 16 lanes each, up to 8 experts
//   a lane.
#include <math.h>

#include <atomic>

#include "rf_device.h"
#include "rf_launch.h"

namespace rf {

// Scratch memory of the entry point that must not allocate: fp32 partial scores of one call.
// A file-scope device array: every GPU the library runs on holds its own copy, at its own
// address, until the process ends.  In host code this name is only a handle for
// hipGetSymbolAddress; kernels are always handed the address that call returned.
static __device__ __align__(256) unsigned char scratch[kMoeStaticScratchBytes];

namespace {

constexpr int kMoeThreads = 256;
constexpr int kMoeRows = 64;    // tokens per workgroup
constexpr int kMoeKB = 128;     // k per LDS tile
constexpr int kMoeXTileB = kMoeRows * kMoeKB * 2;  // 16 KB, [row][k], 256-byte rows

typedef __attribute__((address_space(3))) void lds_void_m;
typedef __attribute__((address_space(1))) const void global_cvoid_m;

// 16-byte slot swizzles (slot = piece ^ f(row))
__device__ __forceinline__ int fXm(int row) { return row & 15; }
template <int PPR>
__device__ __forceinline__ int fWm(int krow) { return ((krow & 3) << 2) & (PPR - 1); }
constexpr int kMoeFusedWaves = 8;

// Maximum / sum over all 64 lanes, every lane gets the result; vector-ALU lane swaps only.
__device__ __forceinline__ float wave_max_valu(float v) {
  v = row16_max(v);
  auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
  s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(s[0]), __uint_as_float(s[1]));
}
__device__ __forceinline__ float wave_sum_valu(float v) {
  v = row16_sum(v);
  auto s = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(s[0]) + __uint_as_float(s[1]);
  s = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(s[0]) + __uint_as_float(s[1]);
}

}  // namespace

// The cascade of one token, a wavefront per token: p[i] of a lane is the score of expert EPL lane + i
// (-inf past the last expert).  Here for any scores: a round of the TopK is one maximum over the lanes
// (vector-ALU swaps), after which the scalar unit finds the lowest expert that holds it in the
// comparison masks.
template <int EPL>
__device__ __forceinline__ void moe_cascade_token_any(float (&p)[EPL], int E, int lane, int row, int topk,
                                                      float* __restrict__ prob, int32_t* __restrict__ idx,
                                                      int64_t ldp, int64_t ldi) {
  // stage 1: max;  stage 2: sum of exponentials
  float m = p[0];
#pragma unroll
  for (int i = 1; i < EPL; ++i) m = fmaxf(m, p[i]);
  m = wave_max_valu(m);
  float t = 0.f;
#pragma unroll
  for (int i = 0; i < EPL; ++i) t += EPL * lane + i < E ? fast_exp2((p[i] - m) * kLog2e) : 0.f;
  t = wave_sum_valu(t);
  const float inv_t = 1.0f / t;
  // stage 3: TopK.  Each round takes the largest remaining score of the token (ties: the lowest
  // expert index).
  float my_prob = 0.f;
  int my_idx = 0;
  for (int j = 0; j < topk; ++j) {
    float bv = p[0];
#pragma unroll
    for (int i = 1; i < EPL; ++i) bv = fmaxf(bv, p[i]);
    bv = wave_max_valu(bv);
    int bi = E;  // no candidate
    if (__builtin_amdgcn_readfirstlane(__float_as_uint(bv)) != 0xff800000u) {
#pragma unroll
      for (int i = EPL - 1; i >= 0; --i) {
        const uint64_t mask = __builtin_amdgcn_ballot_w64(p[i] == bv);
        if (mask != 0) bi = min(bi, EPL * __builtin_ctzll(mask) + i);
      }
    }
    bv = bi == E ? -INFINITY : bv;
#pragma unroll
    for (int i = 0; i < EPL; ++i) p[i] = bi == EPL * lane + i ? -INFINITY : p[i];
    if (lane == j) {
      my_prob = fast_exp2((bv - m) * kLog2e) * inv_t;
      my_idx = bi;
    }
  }
  if (lane < topk) {
    prob[(int64_t)row * ldp + lane] = my_prob;
    idx[(int64_t)row * ldi + lane] = my_idx;
  }
}

// The same where no score is NaN or -inf and no two of the best are equal, which is nearly always.
// The chain of the TopK rounds is what this costs, so a round is nothing but the maximum: scores become
// integers of the same order (maxima fold into the lane exchange), an expert that holds the maximum
// keeps the round's number as its place and drops out, and at the end every expert with a place
// stores its own result.  2048 x 1024 x 128 experts, top 8, in one launch 9.1 -> 7.4 us, 16 x 896 x 128 8.5 -> 6.9.
template <int EPL>
__device__ __forceinline__ void moe_cascade_token(float (&p)[EPL], int E, int lane, int row, int topk,
                                                  float* __restrict__ prob, int32_t* __restrict__ idx,
                                                  int64_t ldp, int64_t ldi) {
  const bool live = EPL * lane < E;
  bool odd = false;
#pragma unroll
  for (int i = 0; i < EPL; ++i) odd = odd || (live && !(p[i] > -INFINITY));
  if (__builtin_amdgcn_ballot_w64(odd) != 0) {
    moe_cascade_token_any<EPL>(p, E, lane, row, topk, prob, idx, ldp, ldi);
    return;
  }
  constexpr int kOut = INT32_MIN;  // below every score
  int key[EPL], place[EPL];
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    const int b = (int)__float_as_uint(p[i] + 0.f);  // (-0 is 0)
    key[i] = live ? b ^ ((b >> 31) & 0x7fffffff) : kOut;
    place[i] = topk;
  }
  auto wave_max_key = [](int v) {
    v = max(v, dpp_i32<kDppQuadXor1>(v));
    v = max(v, dpp_i32<kDppQuadXor2>(v));
    v = max(v, dpp_i32<kDppRowHalfMirror>(v));
    v = max(v, dpp_i32<kDppRowMirror>(v));
    auto s = __builtin_amdgcn_permlane16_swap((uint32_t)v, (uint32_t)v, false, false);
    v = max((int)s[0], (int)s[1]);
    s = __builtin_amdgcn_permlane32_swap((uint32_t)v, (uint32_t)v, false, false);
    return max((int)s[0], (int)s[1]);
  };
  float m = 0.f;
  for (int j = 0; j < topk; ++j) {
    int best = key[0];
#pragma unroll
    for (int i = 1; i < EPL; ++i) best = max(best, key[i]);
    best = wave_max_key(best);
    if (j == 0) m = __uint_as_float((uint32_t)(best ^ ((best >> 31) & 0x7fffffff)));
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      const bool hit = key[i] == best;
      place[i] = hit ? j : place[i];
      key[i] = hit ? kOut : key[i];
    }
  }
  int placed = 0;
#pragma unroll
  for (int i = 0; i < EPL; ++i) placed += __builtin_popcountll(__builtin_amdgcn_ballot_w64(place[i] < topk));
  if (placed != topk) {  // equal scores among the best
    moe_cascade_token_any<EPL>(p, E, lane, row, topk, prob, idx, ldp, ldi);
    return;
  }
  float e[EPL], t = 0.f;
#pragma unroll
  for (int i = 0; i < EPL; ++i) {
    e[i] = fast_exp2((p[i] - m) * kLog2e);
    t += live ? e[i] : 0.f;
  }
  const float inv_t = 1.0f / wave_sum_valu(t);
#pragma unroll
  for (int i = 0; i < EPL; ++i)
    if (place[i] < topk) {
      prob[(int64_t)row * ldp + place[i]] = e[i] * inv_t;
      idx[(int64_t)row * ldi + place[i]] = EPL * lane + i;
    }
}

// The same on 16 lanes, lane q with experts q EPL ..: four tokens per wavefront.  A TopK round is a longer
// chain (a compare per expert held, then an exchange of (score, index) pairs), but four tokens share it:
// the better one as soon as there are tokens enough to fill the chip.
template <int EPL>
__device__ __forceinline__ void moe_cascade_token16(const float (&p)[EPL], int q, int row, bool live, int topk,
                                                    float* __restrict__ prob, int32_t* __restrict__ idx,
                                                    int64_t ldp, int64_t ldi) {
  constexpr int E = 16 * EPL;
  // stage 1: max;  stage 2: sum of exponentials
  float m = p[0];
#pragma unroll
  for (int i = 1; i < EPL; ++i) m = fmaxf(m, p[i]);
  m = row16_max(m);
  float t = 0.f;
#pragma unroll
  for (int i = 0; i < EPL; ++i) t += fast_exp2((p[i] - m) * kLog2e);
  const float inv_t = 1.0f / row16_sum(t);
  // stage 3: TopK.  Each round takes the largest remaining score of the token (ties: the
  // lowest expert index): lane-local best, then a 16-lane merge of (score, index) pairs.
  uint32_t taken = 0;
  float my_prob = 0.f;
  int my_idx = 0;
  for (int j = 0; j < topk; ++j) {
    float bv = -INFINITY;
    int bi = E;  // no candidate
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      const bool ok = !((taken >> i) & 1u) && (p[i] > bv);  // strict: keeps the lowest index
      bv = ok ? p[i] : bv;
      bi = ok ? q * EPL + i : bi;
    }
#define RF_MERGE_TOP(CTRL)                                         \
  {                                                                \
    const float ov = dpp_f32<CTRL>(bv);                            \
    const int oi = dpp_i32<CTRL>(bi);                              \
    const bool take = (ov > bv) || (ov == bv && oi < bi);          \
    bv = take ? ov : bv;                                           \
    bi = take ? oi : bi;                                           \
  }
    RF_MERGE_TOP(kDppQuadXor1) RF_MERGE_TOP(kDppQuadXor2) RF_MERGE_TOP(kDppRowHalfMirror) RF_MERGE_TOP(kDppRowMirror)
#undef RF_MERGE_TOP
    if (bi / EPL == q && bi < E) taken |= 1u << (bi % EPL);
    if ((j & 15) == q) {
      my_prob = fast_exp2((bv - m) * kLog2e) * inv_t;
      my_idx = bi;
    }
  }
  if (live && q < topk) {
    prob[(int64_t)row * ldp + q] = my_prob;
    idx[(int64_t)row * ldi + q] = my_idx;
  }
}

// Single-segment strategy (Section 4.3): 16 tokens and the whole contraction axis per workgroup,
// the scores never leave the chip and the workgroup runs the cascade on them itself.  Chosen where
// the contraction axis is short enough that splitting it only buys a second launch.
//
// What bounds it is latency: the wavefronts split the 32-k steps among themselves and take x and w
// straight from memory into the operands, w as whole rows whose pairs are joined in registers, with
// no LDS and no barrier before their sums are added.  2048 x 1024 x 128 experts 9.2 us, 22.3 with x
// and w through LDS in tiles of 128 k and 64 tokens; 16 x 896 x 128 8.8 and 21.2.
template <int E>
__global__ __launch_bounds__(kMoeFusedWaves * kWave, 2) void moe_fused_kernel(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ w, int S, int n_steps, int64_t ldx,
    int64_t ldw, int topk, float* __restrict__ prob, int32_t* __restrict__ idx, int64_t ldp,
    int64_t ldi) {
  constexpr int NW = kMoeFusedWaves;
  constexpr int P = 4;         // steps in flight per wavefront
  constexpr int C = E / 16;    // experts per lane of a row of w
  constexpr int CD = C / 2;    // 32-bit words of it
  constexpr int kPitch = E + 4;
  __shared__ __attribute__((aligned(16))) float s_p[NW][16][kPitch];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int i16 = lane & 15;
  const int g4 = lane >> 4;
  const int row0 = blockIdx.x * 16;
  // this wavefront's run of 32-k steps
  const int a0 = n_steps * wave / NW;
  const int mine = n_steps * (wave + 1) / NW - a0;

  // Slot (g4, e) of a 32-k step stands for k = 8 g4 + e on both operands.  (Rows past the end
  // repeat the last token; their scores are not stored.)
  const uint32_t x_lane = (uint32_t)(((int64_t)min(row0 + i16, S - 1) * ldx + 8 * g4) * 2);
  const uint32_t ldw2 = (uint32_t)ldw * 2;
  const uint32_t w_lane = 8 * g4 * ldw2 + 2 * C * i16;
  uint32_t wr[P][8][CD];
  u32x4 xr[P];
  auto load = [&](int p, int i) {
    const int n = a0 + min(i, mine - 1);
    const char* xt = reinterpret_cast<const char*>(x) + (int64_t)n * 64;
    const char* wt = reinterpret_cast<const char*>(w) + (int64_t)n * 32 * ldw * 2;
    xr[p] = *reinterpret_cast<const u32x4*>(xt + x_lane);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const char* src = wt + (int64_t)e * ldw * 2 + w_lane;
      if constexpr (CD == 4) {
        const u32x4 v = *reinterpret_cast<const u32x4*>(src);
#pragma unroll
        for (int d = 0; d < CD; ++d) wr[p][e][d] = v[d];
      } else if constexpr (CD == 2) {
        const u32x2 v = *reinterpret_cast<const u32x2*>(src);
#pragma unroll
        for (int d = 0; d < CD; ++d) wr[p][e][d] = v[d];
      } else {
        wr[p][e][0] = *reinterpret_cast<const uint32_t*>(src);
      }
    }
  };
  f32x4 acc[C];  // acc[c][r]: P[token i16][expert C (4 g4 + r) + c]
#pragma unroll
  for (int c = 0; c < C; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto step = [&](int p) {
    const bf16x8 bx = __builtin_bit_cast(bf16x8, xr[p]);
#pragma unroll
    for (int d = 0; d < CD; ++d) {
      u32x4 lo, hi;
#pragma unroll
      for (int e2 = 0; e2 < 4; ++e2) {
        lo[e2] = pair_lo(wr[p][2 * e2][d], wr[p][2 * e2 + 1][d]);
        hi[e2] = pair_hi(wr[p][2 * e2][d], wr[p][2 * e2 + 1][d]);
      }
      acc[2 * d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, lo), bx, acc[2 * d], 0, 0, 0);
      acc[2 * d + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, hi), bx, acc[2 * d + 1], 0, 0, 0);
    }
  };
  if (mine > 0) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
      load(p, p);
      __builtin_amdgcn_sched_barrier(0);
    }
    int i = 0;
    for (; i + P < mine; i += P) {
#pragma unroll
      for (int p = 0; p < P; ++p) {
        step(p);
        load(p, i + P + p);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int p = 0; p < P; ++p)
      if (i + p < mine) step(p);
  }

  // ---- add the wavefronts' sums, in a fixed order ----
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    float* dst = &s_p[wave][i16][C * (4 * g4 + r)];
    if constexpr (C >= 4) {
#pragma unroll
      for (int c = 0; c < C; c += 4)
        *reinterpret_cast<f32x4*>(dst + c) = f32x4{acc[c][r], acc[c + 1][r], acc[c + 2][r], acc[c + 3][r]};
    } else {
#pragma unroll
      for (int c = 0; c < C; ++c) dst[c] = acc[c][r];
    }
  }
  __syncthreads();
  constexpr int EPL = E > 64 ? E / 64 : 1;
  for (int tok = wave; tok < 16 && row0 + tok < S; tok += NW) {
    float p[EPL];
#pragma unroll
    for (int i = 0; i < EPL; ++i) {
      const int e = EPL * lane + i;
      p[i] = -INFINITY;
      if (e < E) {
        p[i] = s_p[0][tok][e];
#pragma unroll
        for (int u = 1; u < NW; ++u) p[i] += s_p[u][tok][e];
      }
    }
    moe_cascade_token<EPL>(p, E, lane, row0 + tok, topk, prob, idx, ldp, ldi);
  }
}

// Multi-segment strategy: part[ks][row][e] = sum over the k slice of x[row,k] w[k,e].  A workgroup takes
// 4096 / E tokens, a wavefront 32 of them and 32 experts: nothing is added up between wavefronts, and
// with 32 tokens of 128 experts half as many slices fill the chip as with 64, so half the partial
// scores pass through memory.  What bounds it is that one trip: launch, the first tile's latency, x at
// the rate of memory, the partial scores.  Both launches, 64 tokens a workgroup with the tiles' steps dealt to
// the wavefronts / this: 2048 x 4096 x 128, top 8, 17.4 / 13.3 us, 512 x 4096 x 128 15.4 / 9.5,
// 3000 x 8192 x 128 31.5 / 26.2, 2048 x 8192 x 64 14.2 / 13.5; 32 experts 4096 x 4096 12.4 / 11.9.
template <int E>
struct MoeTile {
  static constexpr int kWaveE = E / 32, kWaveT = 4 / kWaveE;  // wavefronts along experts and tokens
  static constexpr int kTokens = 32 * kWaveT;
  static constexpr int kXB = kTokens * kMoeKB * 2, kWB = kMoeKB * E * 2;  // [token][k] and [k][expert]
  static constexpr int kStageB = kXB + kWB;
  static constexpr int kStages = 4;
  static_assert(kStages == 4, "three tiles in flight: the waits below");
};

// NA sums for a tile's eight steps of 16 k in turn, added up pairwise at the end, with 8 after every `fold_tiles` tiles too:
// no chain is longer than those of four wavefronts that share a tile's steps over a third of the axis.  One chain over a
// slice is 0.3 us faster and its error against 64 bits larger, 2048 x 4096 x 128 3.7e-7 (here 2.0e-7), 6000 x 8192 x 128
// 16e-7 (2.2e-7).  Adding up costs some 0.3 us each time, so slices of up to 8 tiles make do with 4 sums, but for three or
// fewer of more than 4 tiles, which leave little else to add up; up to 24 tiles are folded in even parts of up to 8, longer
// ones every 16.  (4 sums up to 8 tiles and a fold every 16: 4000 x 1920 x 128 2.0e-7, here 1.7e-7, 12.0 -> 12.3 us;
// 5000 x 2304 x 128 2.1e-7, here 1.7e-7, 17.6 -> 17.8.)  LDS is handed over by the launch: with its size known the
// compiler would keep the sums in registers that the vector ALU does not reach.
template <int E, int NA>
__global__ __launch_bounds__(kMoeThreads, 2) void moe_scores_kernel(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ w, float* __restrict__ part, int S,
    int n_kblocks, int64_t ldx, int64_t ldw, int fold_tiles) {
  using T = MoeTile<E>;
  constexpr int PPR = E / 8;                // 16-byte pieces of a row of w
  constexpr int kXLoads = T::kXB / 4096, kWLoads = T::kWB / 4096;  // direct-to-LDS loads per wavefront and tile
  constexpr int kLoads = kXLoads + kWLoads, NS = T::kStages;
  extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i32 = lane & 31, hh = lane >> 5;
  const int wt = wave % T::kWaveT, we = wave / T::kWaveT;
  const int row0 = blockIdx.x * T::kTokens;
  const int KS = gridDim.y, ks = blockIdx.y;
  const int b0 = (int)((int64_t)n_kblocks * ks / KS);  // this slice's tiles: b0 .. b0 + nb - 1
  const int nb = (int)((int64_t)n_kblocks * (ks + 1) / KS) - b0;
  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;

  uint32_t x_off[kXLoads], w_off[kWLoads];
#pragma unroll
  for (int e = 0; e < kXLoads; ++e) {
    const int row = 4 * (kXLoads * wave + e) + (lane >> 4);
    const int piece = (lane & 15) ^ fXm(row);
    x_off[e] = (uint32_t)(((int64_t)min(row0 + row, S - 1) * ldx + 8 * piece) * 2);
  }
#pragma unroll
  for (int e = 0; e < kWLoads; ++e) {
    const int p = 64 * (kWLoads * wave + e) + lane;
    const int krow = p / PPR;
    const int piece = (p % PPR) ^ fWm<PPR>(krow);
    w_off[e] = (uint32_t)(((int64_t)krow * ldw + 8 * piece) * 2);
  }
  // Where a wavefront loads the rows of x that it multiplies (one column of experts), those past the end are left out with
  // all that is done on them.  us: 1 x 1152 x 32 4.79 -> 4.69, 32 x 4096 x 32 5.99 -> 5.72.
  const bool idle = T::kWaveE == 1 && row0 + 32 * wave >= S;
  auto request = [&](int blk, int stage) {  // tile b0 + blk
    const int b = b0 + blk;
    const char* xt = reinterpret_cast<const char*>(x) + (int64_t)b * kMoeKB * 2;
    const char* wt_ = reinterpret_cast<const char*>(w) + (int64_t)b * kMoeKB * ldw * 2;
#pragma unroll
    for (int e = 0; e < kLoads; ++e) {
      const bool tok = e < kXLoads;
      if (tok && idle) continue;
      const uint32_t dst = lds_base + stage * T::kStageB +
                           (tok ? (kXLoads * wave + e) * 1024 : T::kXB + (kWLoads * wave + e - kXLoads) * 1024);
      const uint32_t off = tok ? x_off[tok ? e : 0] : w_off[tok ? 0 : e - kXLoads];
      asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                   :
                   : "s"(dst), "v"(off), "s"(tok ? xt : wt_)
                   : "memory", "m0");
    }
  };

  // ---- fragments ----
  // A operand (tokens): lane (i32, hh) reads row 32 wt + i32, slot 2 kk + hh.
  // B operand (experts) by transpose reads: lane = 32 hh + 16 g2 + 4 j + a reads 8 bytes of k-row
  // 16 kk + 8 hh + 4 w2 + j at expert 32 we + 16 g2 + 4 a
  const int xrow = 32 * wt + i32;
  uint32_t x_at[8], w_at[2];
#pragma unroll
  for (int kk = 0; kk < 8; ++kk) x_at[kk] = xrow * 256 + (((2 * kk + hh) ^ fXm(xrow)) << 4);
  {
    const int i16 = lane & 15, g2 = (lane >> 4) & 1;
    const int j = i16 >> 2, c = i16 & 3;
    const int piece = (32 * we + 16 * g2 + 4 * c) >> 3;
#pragma unroll
    for (int w2 = 0; w2 < 2; ++w2) {
      const int krow = 8 * hh + 4 * w2 + j;  // (+ 16 kk: the swizzle looks at the row mod 4)
      w_at[w2] = T::kXB + krow * (E * 2) + ((piece ^ fWm<PPR>(krow)) << 4) + 8 * (c & 1);
    }
  }
  typedef short s16x4 __attribute__((ext_vector_type(4)));
  typedef __attribute__((address_space(3))) s16x4* lds_s16x4;

  f32x16 acc[NA], sum;  // rows = tokens, columns = experts
  auto clear = [&](f32x16& v) {
#pragma unroll
    for (int r = 0; r < 16; ++r) v[r] = 0.f;
  };
#pragma unroll
  for (int c = 0; c < NA; ++c) clear(acc[c]);
  clear(sum);
  auto fold = [&]() {
#pragma unroll
    for (int h = NA / 2; h >= 1; h /= 2)
#pragma unroll
      for (int c = 0; c < h; ++c) acc[c] += acc[c + h];
    if constexpr (NA == 8) sum += acc[0];
    else sum = acc[0];  // (once, at the end)
  };

  // NS - 1 tiles are in flight; the one that follows them goes to the stage that the tile before this one left.
#pragma unroll
  for (int t = 0; t < NS - 1; ++t)
    if (t < nb) request(t, t);
  int stage = 0, left = fold_tiles;
  for (int blk = 0; blk < nb; ++blk) {
    // this tile has landed (loads retire in order: the younger tiles' may be in flight), and the reads of the
    // tile before are back; then both hold for every wavefront
    if (blk + 2 < nb && !idle) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(2 * kLoads) : "memory");
    else if (blk + 2 < nb) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(2 * kWLoads) : "memory");
    else if (blk + 1 < nb && !idle) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(kLoads) : "memory");
    else if (blk + 1 < nb) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(kWLoads) : "memory");
    else asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    if (blk + NS - 1 < nb) request(blk + NS - 1, stage == 0 ? NS - 1 : stage - 1);
    const uint32_t at = stage * T::kStageB;
    stage = stage == NS - 1 ? 0 : stage + 1;
    if (idle) continue;
    u32x4 bx[8];
    s16x4 bw[8][2];
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      bx[kk] = *reinterpret_cast<const u32x4*>(lds + at + x_at[kk]);
#pragma unroll
      for (int w2 = 0; w2 < 2; ++w2)
        bw[kk][w2] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(lds + at + w_at[w2] + kk * 16 * (E * 2)));
    }
#pragma unroll
    for (int kk = 0; kk < 8; ++kk) {
      const auto b = __builtin_shufflevector(bw[kk][0], bw[kk][1], 0, 1, 2, 3, 4, 5, 6, 7);
      acc[kk % NA] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, bx[kk]), __builtin_bit_cast(bf16x8, b),
                                                        acc[kk % NA], 0, 0, 0);
    }
    if (NA == 8 && --left == 0 && blk + 1 < nb) {
      left = fold_tiles;
      fold();
#pragma unroll
      for (int c = 0; c < NA; ++c) clear(acc[c]);
    }
  }
  if (idle) return;
  fold();

  // A register is one token's 32 experts over 32 lanes: 128 contiguous bytes.
  float* dst = part + ((int64_t)ks * S + row0 + 32 * wt) * E + 32 * we + i32;
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const int t = 8 * (r >> 2) + 4 * hh + (r & 3);
    if (row0 + 32 * wt + t < S) dst[(int64_t)t * E] = sum[r];
  }
}

// Single-segment strategy for many tokens: 64 of them and the whole contraction axis per workgroup; the
// scores never leave the chip, the workgroup runs the cascade on them.  NT = E / 32.
template <int NT>
__global__ __launch_bounds__(kMoeThreads) void moe_fused64_kernel(
    const bf16_t* __restrict__ x, const bf16_t* __restrict__ w, int S, int n_kblocks, int64_t ldx,
    int64_t ldw, int topk, float* __restrict__ prob, int32_t* __restrict__ idx, int64_t ldp,
    int64_t ldi) {
  constexpr int E = 32 * NT;
  constexpr int PPR = E / 8;               // 16-byte pieces per W row
  constexpr int kWTileB = kMoeKB * E * 2;  // [k][e]
  constexpr int kStageB = kMoeXTileB + kWTileB;
  constexpr int kWLoads = kWTileB / 1024 / 4;  // direct-to-LDS loads per wavefront per tile
  constexpr int kAccB = 2 * NT * 16 * 64 * 4;  // one wavefront's accumulators
  constexpr int kStages = 3;
  constexpr int kLdsB = (kStages * kStageB > 4 * kAccB) ? kStages * kStageB : 4 * kAccB;
  constexpr int kLoadsPerTile = 4 + kWLoads;  // per wavefront
  __shared__ __attribute__((aligned(1024))) unsigned char lds[kLdsB];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int i32 = lane & 31;
  const int hh = lane >> 5;
  const int row0 = blockIdx.x * kMoeRows;
  const int b0 = 0, b1 = n_kblocks;

  const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds;

  // ---- direct-to-LDS roles ----
  // X: 4 loads per wavefront per tile; load e covers rows 16 wave + 4e .. +3, lane -> (row, slot)
  uint32_t xsrc_off[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int row = 16 * wave + 4 * e + (lane >> 4);
    const int piece = (lane & 15) ^ fXm(row);
    xsrc_off[e] = (uint32_t)(((int64_t)min(row0 + row, S - 1) * ldx + 8 * piece) * 2);
  }
  // W: pieces numbered row-major over the tile; load e of wavefront `wave` covers pieces
  // 64 (kWLoads wave + e) .. +63
  uint32_t wsrc_off[kWLoads];
#pragma unroll
  for (int e = 0; e < kWLoads; ++e) {
    const int p = 64 * (kWLoads * wave + e) + lane;
    const int krow = p / PPR;
    const int piece = (p % PPR) ^ fWm<PPR>(krow);
    wsrc_off[e] = (uint32_t)(((int64_t)krow * ldw + 8 * piece) * 2);
  }
  auto issue_tile = [&](int blk, int stage) {
    const char* xt = reinterpret_cast<const char*>(x) + (int64_t)blk * kMoeKB * 2;
    const char* wt = reinterpret_cast<const char*>(w) + (int64_t)blk * kMoeKB * ldw * 2;
    unsigned char* xdst = lds + stage * kStageB + wave * 4096;
    unsigned char* wdst = lds + stage * kStageB + kMoeXTileB + wave * (kWLoads * 1024);
#pragma unroll
    for (int e = 0; e < 4; ++e)
      __builtin_amdgcn_global_load_lds((global_cvoid_m*)(xt + xsrc_off[e]),
                                       (lds_void_m*)(xdst + e * 1024), 16, 0, 0);
#pragma unroll
    for (int e = 0; e < kWLoads; ++e)
      __builtin_amdgcn_global_load_lds((global_cvoid_m*)(wt + wsrc_off[e]),
                                       (lds_void_m*)(wdst + e * 1024), 16, 0, 0);
  };

  // ---- fragment read addresses (stage 0, this wavefront's two contraction steps) ----
  // B operand (X): lane (i32, hh) of token tile mi reads row 32mi + i32, slot 2kk + hh
  uint32_t xaddr[2][2];  // [step][mi]
#pragma unroll
  for (int st = 0; st < 2; ++st)
#pragma unroll
    for (int mi = 0; mi < 2; ++mi) {
      const int row = 32 * mi + i32;
      const int kk = 2 * wave + st;
      xaddr[st][mi] = lds_base + row * 256 + (((2 * kk + hh) ^ fXm(row)) << 4);
    }
  // A operand (W^T) by transpose reads: lane = 32hh + 16g2 + 4j + a reads 8 bytes of k-row
  // 16kk + 8hh + 4w2 + j at expert column 32ni + 16g2 + 4a
  uint32_t waddr[2][NT][2];  // [step][ni][w2]
  {
    const int i16 = lane & 15, g2 = (lane >> 4) & 1;
    const int j = i16 >> 2, a = i16 & 3;
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int ni = 0; ni < NT; ++ni)
#pragma unroll
        for (int w2 = 0; w2 < 2; ++w2) {
          const int krow = 16 * (2 * wave + st) + 8 * hh + 4 * w2 + j;
          const int piece = (32 * ni + 16 * g2 + 4 * a) >> 3;
          waddr[st][ni][w2] = lds_base + kMoeXTileB + krow * (E * 2) +
                              ((piece ^ fWm<PPR>(krow)) << 4) + 8 * (a & 1);
        }
  }

  f32x16 acc[NT][2];  // [ni][mi]: P^T tile (rows = experts, columns = tokens)
#pragma unroll
  for (int a = 0; a < NT; ++a)
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][c][r] = 0.f;

  if (b0 < b1) issue_tile(b0, 0);
  if (b0 + 1 < b1) issue_tile(b0 + 1, 1);
  if (b0 + 2 < b1) issue_tile(b0 + 2, 2);
  int stage = 0;
  for (int blk = b0; blk < b1; ++blk) {
    // This wavefront's loads of the tile have landed (loads retire in order; only the
    // next tile's, at first the next two tiles', may still be in flight); then everyone's have,
    // and everyone is done reading the stage that the tile after next goes to.
    if (blk == b0 && blk + 2 < b1)
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(2 * kLoadsPerTile) : "memory");
    else if (blk + 1 < b1)
      asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" : : "n"(kLoadsPerTile) : "memory");
    else
      asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    if (blk > b0 && blk + 2 < b1) issue_tile(blk + 2, stage == 0 ? 2 : stage - 1);
    const uint32_t soff = stage * kStageB;
    stage = stage == 2 ? 0 : stage + 1;
    // Fragment reads are raw instructions with a hand-placed wait: through the compiler's
    // intrinsics every LDS read would first wait for the direct-to-LDS loads of the next
    // tile, just issued.
    u32x2 af[2][NT][2];
    u32x4 bfr[2][2];
#pragma unroll
    for (int st = 0; st < 2; ++st) {
      const uint32_t xa0 = xaddr[st][0] + soff, xa1 = xaddr[st][1] + soff;
#pragma unroll
      for (int ni = 0; ni < NT; ++ni)
#pragma unroll
        for (int w2 = 0; w2 < 2; ++w2) {
          const uint32_t wa = waddr[st][ni][w2] + soff;
          asm volatile("ds_read_b64_tr_b16 %0, %1" : "=v"(af[st][ni][w2]) : "v"(wa));
        }
      asm volatile("ds_read_b128 %0, %1" : "=v"(bfr[st][0]) : "v"(xa0));
      asm volatile("ds_read_b128 %0, %1" : "=v"(bfr[st][1]) : "v"(xa1));
    }
    // all reads of this step are back (the fragment registers are tied to the wait)
#pragma unroll
    for (int st = 0; st < 2; ++st) {
#pragma unroll
      for (int ni = 0; ni < NT; ++ni)
        asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(af[st][ni][0]), "+v"(af[st][ni][1]));
      asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(bfr[st][0]), "+v"(bfr[st][1]));
    }
#pragma unroll
    for (int st = 0; st < 2; ++st)
#pragma unroll
      for (int ni = 0; ni < NT; ++ni) {
        u32x4 a;
        a[0] = af[st][ni][0][0]; a[1] = af[st][ni][0][1];
        a[2] = af[st][ni][1][0]; a[3] = af[st][ni][1][1];
#pragma unroll
        for (int mi = 0; mi < 2; ++mi)
          acc[ni][mi] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              __builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, bfr[st][mi]), acc[ni][mi],
              0, 0, 0);
      }
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __syncthreads();  // every wavefront has left the loop: LDS is free

  // ---- sum the four wavefronts' accumulators (fixed order 0, 1, 2, 3) ----
  // Every wavefront parks its accumulators in LDS as 128-bit chunks [chunk][lane]; chunk
  // c = (ni * 2 + mi) * 4 + r4 holds P[token 32 mi + i32][experts 32 ni + 8 r4 + 4 hh .. +3].
  // Wavefront v then sums chunks [v CPW, (v+1) CPW) over the four copies and stores them.
  constexpr int kChunks = 2 * NT * 4;
  constexpr int CPW = kChunks / 4;
  f32x4* red = reinterpret_cast<f32x4*>(lds);
  {
    f32x4* dst = red + wave * (kChunks * 64) + lane;
#pragma unroll
    for (int ni = 0; ni < NT; ++ni)
#pragma unroll
      for (int mi = 0; mi < 2; ++mi)
#pragma unroll
        for (int r4 = 0; r4 < 4; ++r4) {
          f32x4 v;
#pragma unroll
          for (int j = 0; j < 4; ++j) v[j] = acc[ni][mi][4 * r4 + j];
          dst[((ni * 2 + mi) * 4 + r4) * 64] = v;
        }
  }
  __syncthreads();
  // sums in the same fixed order, kept in registers until every wavefront has read the four
  // copies, then laid out [token][expert] at the start of LDS
  f32x4 sum[CPW];
#pragma unroll
  for (int cc = 0; cc < CPW; ++cc) {
    const int c = wave * CPW + cc;
    sum[cc] = red[c * 64 + lane];
#pragma unroll
    for (int r = 1; r < 4; ++r) sum[cc] += red[r * (kChunks * 64) + c * 64 + lane];
  }
  __syncthreads();
  float* sc = reinterpret_cast<float*>(lds);  // [kMoeRows][E + 4] (padded rows)
#pragma unroll
  for (int cc = 0; cc < CPW; ++cc) {
    const int c = wave * CPW + cc;
    const int ni = c >> 3, mi = (c >> 2) & 1, r4 = c & 3;
    *reinterpret_cast<f32x4*>(sc + (32 * mi + i32) * (E + 4) + 32 * ni + 8 * r4 + 4 * hh) = sum[cc];
  }
  __syncthreads();
  // the cascade: 16 lanes per token, 16 tokens per pass
  constexpr int EPL = E / 16;
  const int q = tid & 15;
#pragma unroll 1
  for (int pass = 0; pass < kMoeRows / 16; ++pass) {
    const int tl = 16 * pass + (tid >> 4);
    const int row = row0 + tl;
    float p[EPL];
#pragma unroll
    for (int i = 0; i < EPL; i += 2) {
      const float2 v2 = *reinterpret_cast<const float2*>(sc + tl * (E + 4) + q * EPL + i);
      p[i] = v2.x;
      p[i + 1] = v2.y;
    }
    moe_cascade_token16<EPL>(p, q, row, row < S, topk, prob, idx, ldp, ldi);
  }
}

constexpr int kCascadeThreads = 256;  // 4 tokens per workgroup

// U slices are requested at a time.  (A remainder loop would wait for each: 512 x 4096 x 128 experts took 11.9 us
// with 15 slices in batches of 16, 8.6 with 16.)
template <int E, int U>
__global__ __launch_bounds__(kCascadeThreads) void moe_cascade_kernel(
    const float* __restrict__ part, int KS, int S, int topk, float* __restrict__ prob,
    int32_t* __restrict__ idx, int64_t ldp, int64_t ldi) {
  constexpr int EPL = E > 64 ? E / 64 : 1;
  typedef __attribute__((__vector_size__(EPL * sizeof(float)))) float vec_t;
  const int lane = threadIdx.x & 63;
  const int row = __builtin_amdgcn_readfirstlane(blockIdx.x * (kCascadeThreads / kWave) + (threadIdx.x >> 6));
  if (row >= S) return;
  // scores: slices added in slice order
  float p[EPL];
#pragma unroll
  for (int i = 0; i < EPL; ++i) p[i] = 0.f;
  const int at = E < 64 ? min(lane, E - 1) : lane;
  for (int s0 = 0; s0 < KS; s0 += U) {
    vec_t v[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      v[u] = reinterpret_cast<const vec_t*>(part + ((int64_t)min(s0 + u, KS - 1) * S + row) * E)[at];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < EPL; ++i) p[i] += s0 + u < KS ? v[u][i] : 0.f;
  }
  if (E < 64 && lane >= E) p[0] = -INFINITY;
  moe_cascade_token<EPL>(p, E, lane, row, topk, prob, idx, ldp, ldi);
}

// Many tokens: 16 lanes each.
constexpr int kCascade16Threads = 64;  // one wavefront = 4 tokens per workgroup
template <int EPL, int U>
__global__ __launch_bounds__(kCascade16Threads) void moe_cascade16_kernel(
    const float* __restrict__ part, int KS, int S, int topk, float* __restrict__ prob,
    int32_t* __restrict__ idx, int64_t ldp, int64_t ldi) {
  constexpr int E = 16 * EPL;
  const int tid = threadIdx.x;
  const int q = tid & 15;
  const int row = blockIdx.x * (kCascade16Threads / 16) + (tid >> 4);
  const bool live = row < S;
  const int rrow = live ? row : S - 1;  // dead groups repeat the last token, store nothing

  // scores: slices added in slice order, U of them requested at a time
  float p[EPL];
#pragma unroll
  for (int i = 0; i < EPL; ++i) p[i] = 0.f;
  for (int s0 = 0; s0 < KS; s0 += U) {
    float2 v[U][EPL / 2];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float* src = part + ((int64_t)min(s0 + u, KS - 1) * S + rrow) * E + q * EPL;
#pragma unroll
      for (int i = 0; i < EPL / 2; ++i) v[u][i] = reinterpret_cast<const float2*>(src)[i];
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int i = 0; i < EPL / 2; ++i) {
        p[2 * i] += s0 + u < KS ? v[u][i].x : 0.f;
        p[2 * i + 1] += s0 + u < KS ? v[u][i].y : 0.f;
      }
  }
  moe_cascade_token16<EPL>(p, q, row, live, topk, prob, idx, ldp, ldi);
}

// Device address of `scratch` on the current device, resolved once per device (with that
// device current) and kept.  Returns nullptr if the runtime cannot resolve the symbol.
static float* moe_static_scratch() {
  constexpr int kMaxDevices = 64;
  static std::atomic<void*> cache[kMaxDevices];
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
  void* ptr = cache[dev].load(std::memory_order_acquire);
  if (ptr == nullptr) {
    if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || ptr == nullptr) return nullptr;
    cache[dev].store(ptr, std::memory_order_release);  // (two threads racing here store the same address)
  }
  return static_cast<float*>(ptr);
}

hipError_t launch_moe_routing_static(const void* x, const void* w, int S, int hd, int E, int topk,
                                     int64_t ldx, int64_t ldw, float* prob, int32_t* idx,
                                     int64_t ldp, int64_t ldi, hipStream_t s) {
  if ((size_t)moe_workspace_slices(S, hd) * (size_t)S * (size_t)E * sizeof(float) > kMoeStaticScratchBytes)
    return hipErrorInvalidValue;  // (the C-ABI layer has already refused this size)
  float* part = moe_static_scratch();
  if (part == nullptr) return hipErrorInvalidSymbol;
  // Nothing in the scratch array has to start at zero: the scores kernel writes every partial
  // score the cascade kernel reads, and what an earlier, larger call left behind is never read.
  return launch_moe_routing(x, w, S, hd, E, topk, ldx, ldw, prob, idx, ldp, ldi, part, s);
}

// Contraction axes of at most this length are not split: one launch, scores stay on chip.
// Every workgroup streams all of w, at the 60 GB/s a compute unit's loads reach: 9.2 us at 1024
// for 2048 tokens and 128 experts, 8.8 at 896 for 16 tokens, growing with hd; the two launches take
// 13.7 and 7.9 us at 2048.
constexpr int kMoeSingleSegmentMaxHd = 1024;

// What a workspace holds: a slice for each round of 256 workgroups of 64 tokens.  The size a caller asks for, and what is
// refused as too small or too large, hang on this alone: how the kernels cut the axis inside it is free to change.
// (Rows of scores come to 16384 and less than S more, so a workspace for S tokens serves most smaller batches too.)
int moe_workspace_slices(int S, int hd) {
  if (hd <= kMoeSingleSegmentMaxHd) return 1;  // (one slice is still what the workspace query promises room for)
  const int64_t n_rb = ((int64_t)S + kMoeRows - 1) / kMoeRows;
  return (int)fmin(fmin((double)((256 + n_rb - 1) / n_rb), 64), hd / kMoeKB);
}

// How the axis is cut: a workgroup (one per compute unit) costs 1.2 us and 0.3 us for each of its tiles of 128 k
// (0.7 with 128 tokens of 32 experts), a slice 0.05 us and 0.29 us for each MB of partial scores.  Fitted to 90 problems of
// 1 to 6000 tokens and 1152 to 8192 k with every cut from 1 to 64; the one it takes is 0.8 % from the best on
// average, 6 % at most.  2048 x 4096 x 128: 4 slices 11.9 us, 2 14.9; 512 x 4096 x 128: 8 slices 7.9, 16 8.8;
// 2869 x 7552 x 128: 2 slices 21.2, 3, which the compute units take in two turns, 27.2.
int moe_num_slices(int S, int hd, int E) {
  const int64_t n_rb = ((int64_t)S * E + 4095) / 4096;
  const int n_kblocks = hd / kMoeKB, most = moe_workspace_slices(S, hd);
  int best = 1;
  double best_us = 0;
  for (int ks = 1; ks <= most; ++ks) {
    const double tiles = (n_kblocks + ks - 1) / ks;
    const double us = ceil((double)n_rb * ks / 256) * (1.25 + (E == 32 ? 0.74 : E == 64 ? 0.31 : 0.33) * tiles) + 0.053 * ks +
                      0.286 * 4e-6 * S * E * ks;
    if (ks == 1 || us < best_us) {
      best = ks;
      best_us = us;
    }
  }
  return best;
}

// Many tokens on a short axis: 64 of them per workgroup instead of 16, for a quarter of the trips of w.  Until the
// 16-token kernel's workgroups exceed one per compute unit it is up to twice as fast; beyond, both take
// turns, and which one wins depends on the cascade's share.  us a turn, fitted per number of experts; us 64 /
// 16 tokens: 12000 x 256 x 128 experts, top 1, 8.5 / 15.5, top 16, 29.7 / 33.6; 8000 x 1024 x 64, top 8, 18.2 / 12.3;
// 4096 x 256 x 128, top 1, 8.4 / 6.5.  (Also where the grid of the 16-token kernel would pass 2^32 threads.)
static bool moe_fused64_wins(int S, int hd, int E, int topk) {
  const int64_t wg16 = ((int64_t)S + 15) / 16, wg64 = ((int64_t)S + kMoeRows - 1) / kMoeRows;
  if (wg16 > UINT32_MAX / (kMoeFusedWaves * kWave)) return true;
  if (wg16 <= 256) return false;
  struct Cost { double launch, turn, axis, round; };
  constexpr Cost c16[] = {{4.1, 0.65, 0.5, 0.26}, {4.0, 1.33, 1.06, 0.26}, {2.0, 3.12, 1.6, 0.41}};
  constexpr Cost c64[] = {{1.2, 3.78, 3.62, 1.0}, {1.65, 4.05, 4.31, 1.13}, {1.6, 5.11, 6.71, 1.38}};
  const int e = E / 64;  // 32, 64, 128 experts: 0, 1, 2
  const double us16 = c16[e].launch + (double)((wg16 + 255) / 256) * (c16[e].turn + (hd > 128 ? c16[e].axis : 0) + c16[e].round * (topk - 1));
  const int64_t turn = E == 32 ? 512 : 256;  // (two workgroups of 32 experts share a compute unit)
  const double us64 = c64[e].launch + (double)((wg64 + turn - 1) / turn) * (c64[e].turn + c64[e].axis * hd / 1024 + c64[e].round * (topk - 1));
  return us64 < us16;
}

// The cascade's wavefront per token pays off until there are some 32 of them per compute unit: both calls' us with 16 lanes /
// a wavefront a token: 2457 x 7552 x 64, top 6, 15.2 / 13.8; 6126 x 2816 x 64, top 8, 14.6 / 13.4; 8101 x 1920 x 128,
// top 1, 15.3 / 15.3; 10983 x 2176 x 32, top 1, 13.8 / 14.7.
static bool moe_cascade16_wins(int S) { return S > 8192; }

hipError_t launch_moe_routing(const void* x, const void* w, int S, int hd, int E, int topk,
                              int64_t ldx, int64_t ldw, float* prob, int32_t* idx, int64_t ldp,
                              int64_t ldi, float* part, hipStream_t s) {
  const int n_kblocks = hd / kMoeKB;
  const int KS = moe_num_slices(S, hd, E);
  // 32-bit lane offsets inside x and inside one 128-row tile of w
  if ((int64_t)S * ldx * 2 >= ((int64_t)1 << 32) || (int64_t)kMoeKB * ldw * 2 >= ((int64_t)1 << 32))
    return hipErrorInvalidValue;
  const bf16_t* xb = (const bf16_t*)x;
  const bf16_t* wb = (const bf16_t*)w;
  if (hd <= kMoeSingleSegmentMaxHd && moe_fused64_wins(S, hd, E, topk)) {
#define RF_MOE_FUSED64(NT)                                                                                        \
  hipLaunchKernelGGL((moe_fused64_kernel<NT>), dim3((unsigned)((S + kMoeRows - 1) / kMoeRows)), dim3(kMoeThreads), 0, s, xb, \
                     wb, S, n_kblocks, ldx, ldw, topk, prob, idx, ldp, ldi)
    switch (E) {
      case 32: RF_MOE_FUSED64(1); break;
      case 64: RF_MOE_FUSED64(2); break;
      case 128: RF_MOE_FUSED64(4); break;
      default: return hipErrorInvalidValue;
    }
#undef RF_MOE_FUSED64
    return hipGetLastError();
  }
  if (hd <= kMoeSingleSegmentMaxHd) {
    // single-segment strategy: scores GEMM and cascade in one kernel
#define RF_MOE_FUSED(EE)                                                                                   \
  hipLaunchKernelGGL((moe_fused_kernel<EE>), dim3((unsigned)((S + 15) / 16)), dim3(kMoeFusedWaves * kWave), 0, s, xb, \
                     wb, S, hd / 32, ldx, ldw, topk, prob, idx, ldp, ldi)
    switch (E) {
      case 32: RF_MOE_FUSED(32); break;
      case 64: RF_MOE_FUSED(64); break;
      case 128: RF_MOE_FUSED(128); break;
      default: return hipErrorInvalidValue;
    }
#undef RF_MOE_FUSED
    return hipGetLastError();
  }
  // (see moe_scores_kernel)
  const int tiles = (n_kblocks + KS - 1) / KS, parts = (tiles + 7) / 8, fold_tiles = tiles <= 24 ? (tiles + parts - 1) / parts : 16;
  const bool long_slices = tiles > (KS <= 3 ? 4 : 8);
#define RF_MOE_SCORES_NA(EE, NA)                                                                                  \
  hipLaunchKernelGGL((moe_scores_kernel<EE, NA>), dim3((unsigned)((S + MoeTile<EE>::kTokens - 1) / MoeTile<EE>::kTokens), (unsigned)KS), \
                     dim3(kMoeThreads), MoeTile<EE>::kStages * MoeTile<EE>::kStageB, s, xb, wb, part, S, n_kblocks, ldx, ldw, fold_tiles)
#define RF_MOE_SCORES(EE)                    \
  if (long_slices) RF_MOE_SCORES_NA(EE, 8); \
  else RF_MOE_SCORES_NA(EE, 4)
  switch (E) {
    case 32: RF_MOE_SCORES(32); break;
    case 64: RF_MOE_SCORES(64); break;
    case 128: RF_MOE_SCORES(128); break;
    default: return hipErrorInvalidValue;
  }
#undef RF_MOE_SCORES_NA
#undef RF_MOE_SCORES
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (moe_cascade16_wins(S)) {
    const dim3 grid16((unsigned)((S + kCascade16Threads / 16 - 1) / (kCascade16Threads / 16)));
#define RF_MOE_CASCADE16(EPL, U) \
  hipLaunchKernelGGL((moe_cascade16_kernel<EPL, U>), grid16, dim3(kCascade16Threads), 0, s, part, KS, S, topk, prob, idx, ldp, ldi)
#define RF_MOE_CASCADE16_U(EPL)           \
  if (KS == 1) RF_MOE_CASCADE16(EPL, 1);  \
  else if (KS == 2) RF_MOE_CASCADE16(EPL, 2); \
  else RF_MOE_CASCADE16(EPL, 4)
    if (E == 32) { RF_MOE_CASCADE16_U(2); }
    else if (E == 64) { RF_MOE_CASCADE16_U(4); }
    else { RF_MOE_CASCADE16_U(8); }
#undef RF_MOE_CASCADE16_U
#undef RF_MOE_CASCADE16
    return hipGetLastError();
  }
  constexpr int kTokens = kCascadeThreads / kWave;
  const dim3 grid2((unsigned)((S + kTokens - 1) / kTokens)), block2(kCascadeThreads);
#define RF_MOE_CASCADE(EE, U) \
  hipLaunchKernelGGL((moe_cascade_kernel<EE, U>), grid2, block2, 0, s, part, KS, S, topk, prob, idx, ldp, ldi)
#define RF_MOE_CASCADE_U(EE)              \
  if (KS <= 4) RF_MOE_CASCADE(EE, 4);     \
  else if (KS <= 8) RF_MOE_CASCADE(EE, 8); \
  else RF_MOE_CASCADE(EE, 16)
  switch (E) {
    case 32: RF_MOE_CASCADE_U(32); break;
    case 64: RF_MOE_CASCADE_U(64); break;
    case 128: RF_MOE_CASCADE_U(128); break;
    default: return hipErrorInvalidValue;
  }
#undef RF_MOE_CASCADE_U
#undef RF_MOE_CASCADE
  return hipGetLastError();
}

}  // namespace rf
