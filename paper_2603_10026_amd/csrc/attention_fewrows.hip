// bf16 attention for launches with few query tiles: a decode step, a few draft tokens, one short
// or single-head prompt.  The same cascade as attention_bf16.hip / attention_splitk.hip
// (max -> sum-exp -> weighted sum, unnormalised accumulators), cut for latency.
//
// The tiled kernel gives 128 query rows of one head to a workgroup that walks the keys one tile
// after the other: with a handful of such workgroups the launch takes Lk / 64 dependent steps on
// an idle chip.  Here a workgroup owns 16 query rows (the Hq/Hkv heads that share a KV head times
// Lq, packed) and its NW wavefronts deal the 32-key tiles of the range among themselves; their
// states are merged through LDS with the level-k expression at the end.
//
//   S^T = K Q^T, O^T += V^T P^T      16x16x32 bf16 MFMAs, fp32 accumulate
//
// K comes straight from memory in operand layout (a lane's 16 bytes of its key row) and V as
// whole rows that are transposed in registers, so a wavefront meets no LDS, no barrier and no
// other wavefront before the merge, and a tile's K and V are all on their way at once.  The
// registers of K are refilled as soon as the scores are formed, those of V after the second
// product.
//
// DIRECT: the whole key range, O = acc / l in bf16.  Otherwise one chunk of the key axis, its
// state (m, l, acc) in fp32.
#include <math.h>

#include "rf_device.h"
#include "rf_launch.h"

namespace rf {

namespace {
constexpr int kFewKeys = 32;  // keys per wavefront step
// Wavefronts per SIMD the registers leave room for: one direct workgroup is usually alone on its
// compute unit, chunks come several to a unit and are over after a step or two.
constexpr int few_min_waves(bool direct) { return direct ? 2 : 4; }
// Wavefronts per workgroup.  4, 8 and 16 take the same time where a workgroup is alone on its
// compute unit (70.7, 71.8, 75.0 us for one row tile of 8000 keys: the cache lines the unit has
// in flight set the pace, 58 GB/s), and 4 leave the smallest merge.
constexpr int kDirectWaves = 4, kSplitWaves = 4;
}  // namespace

template <int D, int NW, bool DIRECT>
__global__ __launch_bounds__(NW * kWave, few_min_waves(DIRECT)) void attention_fewrows_kernel(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ k, const bf16_t* __restrict__ v,
    Strides4 sq, Strides4 sk, Strides4 sv, bf16_t* __restrict__ o, Strides4 so,
    float* __restrict__ part_m, float* __restrict__ part_l, float* __restrict__ part_acc, int Hq,
    int Hkv, int Lq, int Lk, int S, int chunk, float scale_log2e, int causal, int n_rtiles) {
  constexpr int KS = D / 32;    // contraction steps of S^T
  constexpr int DPL = D / 16;   // head-dim values per lane of a V row
  constexpr int VW = DPL / 2;
  constexpr int kPitch = D + 4;
  // K of the next tile is requested ahead of the softmax where there are registers for it
  constexpr bool kEarlyK = D == 64 || few_min_waves(DIRECT) == 2;
  __shared__ __attribute__((aligned(16))) float s_acc[NW * 16 * kPitch];
  __shared__ float s_m[NW * 16], s_l[NW * 16];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int i16 = lane & 15;
  const int g = lane >> 4;

  // Workgroups are dealt round-robin to the 8 XCDs, each with its own L2: the row tiles of one
  // chunk of keys go to one XCD.
  int wg = blockIdx.x;
  if ((gridDim.x & 7) == 0) wg = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const int unit = __builtin_amdgcn_readfirstlane(wg / n_rtiles);
  int rt = wg % n_rtiles;
  if (causal) {
    // Late rows see the most keys.  The 32 compute units of an XCD take workgroups one after the
    // other, so those 32 apart share one: blocks of 32 heavy tiles, heaviest first, and of 32 light
    // ones, lightest first, take turns, and what is left of a head (all of a short one) runs
    // upwards in even heads and downwards in odd ones.
    const int full = n_rtiles & ~63;
    if (rt < full) {
      const int i = (rt >> 6) * 32 + (rt & 31);
      rt = (rt & 32) ? i : n_rtiles - 1 - i;
    } else {
      const int i = rt - full;
      rt = full / 2 + ((unit & 1) ? n_rtiles - full - 1 - i : i);
    }
  }
  rt = __builtin_amdgcn_readfirstlane(rt);
  const int c = __builtin_amdgcn_readfirstlane(unit % S);
  const int hk = __builtin_amdgcn_readfirstlane(unit / S % Hkv);
  const int b = __builtin_amdgcn_readfirstlane(unit / S / Hkv);
  const int grp = Hq / Hkv;
  const int R = grp * Lq;  // query rows sharing this KV head
  const int r0 = rt * 16;
  const int shift = Lk - Lq;

  const int lo = min(Lk, c * chunk);
  int hi = min(Lk, lo + chunk);
  if (causal) {  // the last key any row of the tile sees
    const int r1 = min(R, r0 + 16) - 1;
    const int iq_max = __builtin_amdgcn_readfirstlane((r0 / Lq == r1 / Lq) ? r1 % Lq : Lq - 1);
    hi = max(lo, min(hi, iq_max + shift + 1));
  }

  // this lane's query row (column of the transposed score tile)
  const int r = r0 + i16;
  const bool row_ok = r < R;
  const int h = hk * grp + (row_ok ? r / Lq : 0);
  const int iq = row_ok ? r % Lq : 0;
  const int my_last = row_ok ? (causal ? min(hi - 1, iq + shift) : hi - 1) : -1;

  const bf16_t* kb = k + (int64_t)b * sk.b + (int64_t)hk * sk.h;
  const bf16_t* vb = v + (int64_t)b * sv.b + (int64_t)hk * sv.h;
  // Buffer loads whose range ends with the last key's row: what a ragged last tile asks for past
  // it comes back as zeros (and is masked).  All offsets are 32-bit (checked by the launcher).
  const uint32_t sk2 = (uint32_t)sk.l * 2, sv2 = (uint32_t)sv.l * 2;
  const auto krs = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(kb), 0, (uint32_t)(Lk - 1) * sk2 + 2 * D, 0x00020000);
  const auto vrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(vb), 0, (uint32_t)(Lk - 1) * sv2 + 2 * D, 0x00020000);
  const uint32_t k_lane = i16 * sk2 + 16 * g;
  const uint32_t v_lane = 4 * g * sv2 + 2 * DPL * i16;

  // kf[half][kk]: K[key 16 half + i16][32 kk + 8 g ..];  vf[e]: V[key 4 g + e (e < 4), 16 + 4 g +
  // e - 4][DPL i16 ..], the contraction slots (g, e) of the second product
  u32x4 kf[2][KS];
  uint32_t vf[8][VW];
  // (opaque copies of the lane offsets: the offsets of the single rows are then formed here and
  // not carried through the loop in registers)
  auto load_k = [&](int key0) {
    uint32_t kl = k_lane;
    asm volatile("" : "+v"(kl));
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      const uint32_t off = kl + (uint32_t)(key0 + 16 * hf) * sk2;
#pragma unroll
      for (int kk = 0; kk < KS; ++kk) kf[hf][kk] = __builtin_amdgcn_raw_buffer_load_b128(krs, off + 64 * kk, 0, 0);
    }
  };
  auto load_v = [&](int key0) {
    uint32_t vl = v_lane;
    asm volatile("" : "+v"(vl));
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const uint32_t off = vl + (uint32_t)(key0 + ((e < 4) ? e : 12 + e)) * sv2;
      if constexpr (VW == 4) {
        const u32x4 t = __builtin_amdgcn_raw_buffer_load_b128(vrs, off, 0, 0);
#pragma unroll
        for (int i = 0; i < VW; ++i) vf[e][i] = t[i];
      } else {
        const u32x2 t = __builtin_amdgcn_raw_buffer_load_b64(vrs, off, 0, 0);
#pragma unroll
        for (int i = 0; i < VW; ++i) vf[e][i] = t[i];
      }
    }
  };

  int key0 = lo + wave * kFewKeys;
  load_k(key0 < hi ? key0 : Lk);

  // Q^T fragments: contraction slot (g, e) of step kk stands for d = 32 kk + 8 g + e
  u32x4 qf[KS];
  {
    const bf16_t* qp = q + (int64_t)b * sq.b + (int64_t)h * sq.h + (int64_t)iq * sq.l + 8 * g;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) qf[kk] = *reinterpret_cast<const u32x4*>(qp + 32 * kk);
  }
  load_v(key0 < hi ? key0 : Lk);

  float m2 = -INFINITY, l = 0.f;
  f32x4 acc[DPL];  // acc[t][rr] = O[row i16][d = DPL (4 g + rr) + t]
#pragma unroll
  for (int t = 0; t < DPL; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (; key0 < hi; key0 += NW * kFewKeys) {
    // (the last turn asks for keys past the end: nothing is fetched, and there is no branch around
    // the loads that would keep two copies of the registers)
    const int next = key0 + NW * kFewKeys < hi ? key0 + NW * kFewKeys : Lk;
    f32x4 s[2];
#pragma unroll
    for (int hf = 0; hf < 2; ++hf) {
      s[hf] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < KS; ++kk)
        s[hf] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[hf][kk]),
                                                        __builtin_bit_cast(bf16x8, qf[kk]), s[hf], 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (kEarlyK) load_k(next);
    __builtin_amdgcn_sched_barrier(0);
    // ---- stage 1: running max ----
    float sc[8];
    float tmax = -INFINITY;
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int key = key0 + 4 * g + ((e < 4) ? e : 12 + e);
      sc[e] = (key <= my_last) ? s[e >> 2][e & 3] * scale_log2e : -INFINITY;
      tmax = fmaxf(tmax, sc[e]);
    }
    tmax = fmaxf(tmax, __shfl_xor(tmax, 16, 64));
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
    const float m_new = fmaxf(m2, tmax);
    const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
    const float corr = fast_exp2(m2 - m_use);
    m2 = m_new;
    // ---- stage 2: running sum of exponentials ----
    // (a whole row's sum runs over the rounded probabilities, the values the second product sees, as in
    // the tiled kernel: their error cancels in O = acc / l.  A chunk's l is the sum itself.)
    float psum = 0.f;
    u32x4 pb;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float p0 = fast_exp2(sc[2 * e] - m_use), p1 = fast_exp2(sc[2 * e + 1] - m_use);
      pb[e] = pack_bf16(p0, p1);
      if constexpr (DIRECT) {
        typedef __attribute__((__vector_size__(2 * sizeof(__bf16)))) __bf16 bf16x2;
        psum = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, (uint32_t)pb[e]),
                                               __builtin_bit_cast(bf16x2, 0x3f803f80u), psum, false);
      } else {
        psum += p0;
        psum += p1;
      }
    }
    l = l * corr + psum;
    // ---- stage 3: acc = acc * corr + V^T P^T (16-bit transpose of V in registers) ----
#pragma unroll
    for (int tp = 0; tp < VW; ++tp) {
      u32x4 lo4, hi4;
#pragma unroll
      for (int ep = 0; ep < 4; ++ep) {
        lo4[ep] = pair_lo(vf[2 * ep][tp], vf[2 * ep + 1][tp]);
        hi4[ep] = pair_hi(vf[2 * ep][tp], vf[2 * ep + 1][tp]);
      }
      acc[2 * tp] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
          __builtin_bit_cast(bf16x8, lo4), __builtin_bit_cast(bf16x8, pb), acc[2 * tp] * corr, 0, 0, 0);
      acc[2 * tp + 1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
          __builtin_bit_cast(bf16x8, hi4), __builtin_bit_cast(bf16x8, pb), acc[2 * tp + 1] * corr, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (!kEarlyK) load_k(next);
    load_v(next);
    __builtin_amdgcn_sched_barrier(0);
  }

  // ---- merge the wavefront states (level-k fused expression) ----
  l += __shfl_xor(l, 16, 64);
  l += __shfl_xor(l, 32, 64);
  if (g == 0) { s_m[wave * 16 + i16] = m2; s_l[wave * 16 + i16] = l; }
#pragma unroll
  for (int rr = 0; rr < 4; ++rr) {
    float* dst = s_acc + (wave * 16 + i16) * kPitch + DPL * (4 * g + rr);
#pragma unroll
    for (int t = 0; t < DPL; t += 4)
      *reinterpret_cast<f32x4*>(dst + t) = f32x4{acc[t][rr], acc[t + 1][rr], acc[t + 2][rr], acc[t + 3][rr]};
  }
  __syncthreads();
  const int rows_here = min(16, R - r0);
  for (int idx = threadIdx.x; idx < rows_here * (D / 4); idx += NW * kWave) {
    const int rr = idx / (D / 4);
    const int c4 = idx % (D / 4);
    float mg = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) mg = fmaxf(mg, s_m[w * 16 + rr]);
    const float mg_use = (mg == -INFINITY) ? 0.f : mg;
    float lg = 0.f;
    f32x4 og = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float wgt = fast_exp2(s_m[w * 16 + rr] - mg_use);  // 0 for an empty state
      lg += s_l[w * 16 + rr] * wgt;
      og += *reinterpret_cast<const f32x4*>(s_acc + (w * 16 + rr) * kPitch + 4 * c4) * wgt;
    }
    const int rq = r0 + rr;
    const int hh = hk * grp + rq / Lq;
    const int ii = rq % Lq;
    if constexpr (DIRECT) {
      const float inv = lg > 0.f ? 1.0f / lg : 0.f;
      u32x2 w2;
      w2[0] = pack_bf16(og[0] * inv, og[1] * inv);
      w2[1] = pack_bf16(og[2] * inv, og[3] * inv);
      *reinterpret_cast<u32x2*>(o + (int64_t)b * so.b + (int64_t)hh * so.h + (int64_t)ii * so.l + 4 * c4) = w2;
    } else {
      const int64_t prow = (((int64_t)b * Hq + hh) * Lq + ii) * S + c;
      *reinterpret_cast<f32x4*>(part_acc + prow * D + 4 * c4) = og;
      if (c4 == 0) {
        part_m[prow] = mg * 0.6931471805599453f;  // back to natural-log units
        part_l[prow] = lg;
      }
    }
  }
}

static int64_t row_tiles(const AttnShape& a) { return ((int64_t)(a.Hq / a.Hkv) * a.Lq + 15) / 16; }

// 32-bit byte offsets inside one head of k and of v, with room for a step past the end
static bool offsets_fit(const AttnShape& a, const Strides4& sk, const Strides4& sv, int nw) {
  const int64_t rows = (int64_t)a.Lk + (nw + 1) * kFewKeys;
  auto ok = [&](int64_t l) { return l >= 0 && l < ((int64_t)1 << 30) && (rows * l + a.d) * 2 < ((int64_t)1 << 32); };
  return a.Lk >= 1 && ok(sk.l) && ok(sv.l);
}

// A grid holds less than 2^32 threads.  (Several row tiles per head make more workgroups here than in the
// kernels that take over where they do not fit.)
constexpr int64_t max_workgroups(int nw) { return UINT32_MAX / (nw * kWave); }

// Expected us, for the comparison with the tiled kernel (fitted together with its figures: see there).  A
// workgroup walks the keys in steps of 128.
double attention_fewrows_us(const AttnShape& a, const Strides4& sk, const Strides4& sv) {
  const int64_t wgs = row_tiles(a) * a.B * a.Hkv;
  if (!offsets_fit(a, sk, sv, kDirectWaves) || wgs > max_workgroups(kDirectWaves)) return INFINITY;
  constexpr AttnCost d128 = {3.5, 1.21, 0.24, 1.21}, d64 = {3.5, 0.73, 0.15, 0.71};
  return (a.d == 128 ? d128 : d64).us(a.Lk / 128.0 + 0.5, (double)wgs, tile_keys(a, 16) / 128 + 0.5);
}

hipError_t launch_attention_fewrows(const void* q, const void* k, const void* v, void* o, Strides4 sq,
                                    Strides4 sk, Strides4 sv, Strides4 so, const AttnShape& a, hipStream_t s) {
  const int64_t n_rt = row_tiles(a);
  const int64_t grid = n_rt * a.B * a.Hkv;
  if (grid > max_workgroups(kDirectWaves)) return hipErrorInvalidValue;
#define RF_FEW(DD)                                                                                              \
  hipLaunchKernelGGL((attention_fewrows_kernel<DD, kDirectWaves, true>), dim3((unsigned)grid),                  \
                     dim3(kDirectWaves * kWave), 0, s, (const bf16_t*)q, (const bf16_t*)k, (const bf16_t*)v, sq, sk, \
                     sv, (bf16_t*)o, so, nullptr, nullptr, nullptr, a.Hq, a.Hkv, a.Lq, a.Lk, 1, a.Lk,            \
                     a.scale * kLog2e, a.causal, (int)n_rt)
  if (a.d == 128) RF_FEW(128);
  else if (a.d == 64) RF_FEW(64);
  else return hipErrorInvalidValue;
#undef RF_FEW
  return hipGetLastError();
}

// While K and V are small and a chunk is a few tiles, the time is latency and this kernel's shorter
// chain wins (us, here against the streaming kernel): 8.0 / 9.5 for 714 chunks of 63 keys, 15.5 / 18.0
// for 1024 of 64 with 32 rows each (two row tiles in parallel here, one after the other there).
// Beyond, K and V stream from memory and the other kernel's whole-row, non-temporal loads win: at
// 109 MB the two take the same time on new inputs and this one is 2 us ahead on repeated ones, at 221 MB
// it is 17 us behind on new inputs (they do not stay in the 256 MB memory-side cache until they are
// asked for) and 2 on repeated ones, at 2 GB 377 against 324.
// With one row tile per KV head the two kernels' workgroups do the same work, and the other one streams a
// long chunk better (K two steps ahead): launches of one round keep chunks up to about 200 keys here,
// many rounds up to about 400 (11 workgroups with chunks of 2493 keys: 32.7 us here, 21.9 there; 36 of
// 636, 11.6 and 8.6; 1024 of 94, the rule's figures fitted to 369 calls like these, 11.2 and 12.7).
bool attention_fewrows_splitk_wins(const AttnShape& a, const Strides4& sk, const Strides4& sv, int num_splits) {
  if (!offsets_fit(a, sk, sv, kSplitWaves) || (double)a.B * a.Hkv * a.Lk * a.d * 4 > 128e6) return false;
  if ((double)row_tiles(a) * a.B * a.Hkv * num_splits > (double)max_workgroups(kSplitWaves)) return false;
  if (row_tiles(a) > 1) return true;
  constexpr AttnCost here = {3.6, 0, 0.65, 1.54}, there = {3.1, 0, 1.59, 1.33};
  const double wgs = (double)a.B * a.Hkv * num_splits, steps = ceil((double)a.Lk / num_splits) / 128;
  return here.us(0, wgs, steps) < 0.93 * there.us(0, wgs, steps);
}

hipError_t launch_attention_fewrows_splitk(const void* q, const void* k, const void* v, Strides4 sq, Strides4 sk,
                                           Strides4 sv, int num_splits, float* part_m, float* part_l,
                                           float* part_acc, const AttnShape& a, hipStream_t s) {
  const int64_t n_rt = row_tiles(a);
  const int64_t grid = n_rt * a.B * a.Hkv * num_splits;
  if (grid > max_workgroups(kSplitWaves) || a.d != 128) return hipErrorInvalidValue;
  const int chunk = (a.Lk + num_splits - 1) / num_splits;
  hipLaunchKernelGGL((attention_fewrows_kernel<128, kSplitWaves, false>), dim3((unsigned)grid),
                     dim3(kSplitWaves * kWave), 0, s, (const bf16_t*)q, (const bf16_t*)k, (const bf16_t*)v, sq, sk, sv,
                     (bf16_t*)nullptr, Strides4{0, 0, 0}, part_m, part_l, part_acc, a.Hq, a.Hkv, a.Lq, a.Lk,
                     num_splits, chunk, a.scale * kLog2e, a.causal, (int)n_rt);
  return hipGetLastError();
}

}  // namespace rf
