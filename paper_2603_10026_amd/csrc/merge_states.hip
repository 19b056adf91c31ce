// Merge of partial (m, l, acc) states: the level-k fused expression of the
// attention cascade (paper Section 3.2 Eq. (11); Appendix A.2 level-k form)
//   m = max_c m_c;  l = sum_c l_c exp(m_c - m);  O = sum_c acc_c exp(m_c - m) / l
// One workgroup per output row.  Thread (sg, c) accumulates a float4 column c
// of acc over the chunks s = sg, sg + G, ...; the G partial sums are added
// through LDS.  Every partial-state byte is read once, with 128-bit loads.
#include "rf_device.h"
#include "rf_launch.h"

namespace rf {

constexpr int kMergeThreads = 256;

constexpr int kPre = 8;  // acc loads a thread can issue before it knows the weights

// PRE 2: at most 64 chunks and kPre per thread.  PRE 1: at most kPre per thread (narrow heads with more
// chunks): acc is requested at once as well, the weights are formed as for any number.  PRE 0: any number.
template <bool OUT_BF16, int PRE>
__global__ __launch_bounds__(kMergeThreads) void merge_states_kernel(
    const float* __restrict__ part_m, const float* __restrict__ part_l,
    const float* __restrict__ part_acc, void* __restrict__ o, int Hq, int Lq, int S, int d,
    int ncol_p2, Strides4 so) {
  __shared__ float s_red[kMergeThreads / kWave];
  __shared__ float s_red2[kMergeThreads / kWave];
  __shared__ f32x4 s_part[kMergeThreads];

  // (32-bit index arithmetic: a 64-bit division costs some hundred instructions)
  const uint32_t row32 = blockIdx.x;
  const int i = (int)(row32 % (uint32_t)Lq);
  const int h = (int)(row32 / (uint32_t)Lq % (uint32_t)Hq);
  const int b = (int)(row32 / (uint32_t)Lq / (uint32_t)Hq);
  const int64_t row = row32;
  const float* pm = part_m + row * S;
  const float* pl = part_l + row * S;
  const float* pa = part_acc + row * (int64_t)S * d;
  const int tid = threadIdx.x;

  float m, l, wgt = 0.f;
  f32x4 pre[kPre];
  float mc = -INFINITY, lc = 0.f;
  if constexpr (PRE == 2) {
    const int lane = tid & 63;
    mc = lane < S ? pm[lane] : -INFINITY;
    lc = lane < S ? pl[lane] : 0.f;
  }
  if constexpr (PRE > 0) {
    const int G0 = kMergeThreads / ncol_p2;
    const int c0 = tid % ncol_p2, sg0 = tid / ncol_p2;
#pragma unroll
    for (int i = 0; i < kPre; ++i) {
      const int s = sg0 + i * G0;
      pre[i] = (s < S && c0 < d / 4) ? __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(pa + (int64_t)s * d + 4 * c0))
                                     : f32x4{0.f, 0.f, 0.f, 0.f};
    }
  }
  if constexpr (PRE == 2) {
    // Everything is on its way at once, so the whole kernel pays one memory latency, and every
    // wavefront forms m, l and the chunks' weights by itself, a chunk per lane: no barrier and no
    // second trip for them.
    m = wave_max(mc);
    const float m_use = (m == -INFINITY) ? 0.f : m;
    wgt = (mc == -INFINITY) ? -1.f : fast_exp2((mc - m_use) * kLog2e);  // -1: an empty chunk
    l = wave_sum((mc == -INFINITY) ? 0.f : lc * wgt);
  } else {
    // m = max over chunks
    m = -INFINITY;
    for (int s = tid; s < S; s += kMergeThreads) m = fmaxf(m, pm[s]);
    m = wave_max(m);
    if ((tid & 63) == 0) s_red[tid >> 6] = m;
    __syncthreads();
    m = fmaxf(fmaxf(s_red[0], s_red[1]), fmaxf(s_red[2], s_red[3]));
    const float m_use = (m == -INFINITY) ? 0.f : m;
    // l = sum over chunks of l_c exp(m_c - m)
    l = 0.f;
    for (int s = tid; s < S; s += kMergeThreads) {
      const float mc = pm[s];
      if (mc != -INFINITY) l += pl[s] * fast_exp2((mc - m_use) * kLog2e);
    }
    l = wave_sum(l);
    if ((tid & 63) == 0) s_red2[tid >> 6] = l;
    __syncthreads();
    l = (s_red2[0] + s_red2[1]) + (s_red2[2] + s_red2[3]);
  }
  const float m_use = (m == -INFINITY) ? 0.f : m;
  const float inv = l > 0.f ? 1.0f / l : 0.f;

  // O = sum over chunks of acc_c exp(m_c - m) / l
  const int ncol = d / 4;
  const int G = kMergeThreads / ncol_p2;  // chunk groups
  const int c = tid % ncol_p2;
  const int sg = tid / ncol_p2;
  f32x4 sum = f32x4{0.f, 0.f, 0.f, 0.f};
  if constexpr (PRE > 0) {
    // (the kPre loads of this thread were issued at kernel entry)
#pragma unroll
    for (int i = 0; i < kPre; ++i) {
      const int s = sg + i * G;
      if constexpr (PRE == 2) {
        const float w = __shfl(wgt, s & 63, 64);  // (all lanes: the weight of chunk s is in lane s)
        if (s < S && !(w < 0.f)) sum += pre[i] * w;
      } else if (s < S && c < ncol) {
        const float ms = pm[s];
        if (ms != -INFINITY) sum += pre[i] * fast_exp2((ms - m_use) * kLog2e);
      }
    }
  } else if (c < ncol) {
    for (int s = sg; s < S; s += G) {
      const float mc = pm[s];
      if (mc == -INFINITY) continue;
      const float w = fast_exp2((mc - m_use) * kLog2e);
      const f32x4 a = __builtin_nontemporal_load(reinterpret_cast<const f32x4*>(pa + (int64_t)s * d + 4 * c));
      sum += a * w;
    }
  }
  s_part[tid] = sum;
  __syncthreads();
  if (sg == 0 && c < ncol) {
    for (int gq = 1; gq < G; ++gq) sum += s_part[gq * ncol_p2 + c];
    sum *= inv;
    const int64_t off = (int64_t)b * so.b + (int64_t)h * so.h + (int64_t)i * so.l + 4 * c;
    if (OUT_BF16) {
      u32x2 r;
      r[0] = pack_bf16(sum[0], sum[1]);
      r[1] = pack_bf16(sum[2], sum[3]);
      *reinterpret_cast<u32x2*>(reinterpret_cast<bf16_t*>(o) + off) = r;
    } else {
      *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(o) + off) = sum;
    }
  }
}

hipError_t launch_merge_states(const float* part_m, const float* part_l, const float* part_acc,
                               void* o, bool o_is_bf16, int B, int Hq, int Lq, int S, int d,
                               Strides4 so, hipStream_t s) {
  const int64_t rows = (int64_t)B * Hq * Lq;
  if (rows > INT32_MAX) return hipErrorInvalidValue;
  const int ncol = d / 4;
  int p2 = 1;
  while (p2 < ncol) p2 <<= 1;
  if (p2 > kMergeThreads) return hipErrorInvalidValue;
  // (us, PRE 1 against 0: 1024 rows of 128 chunks, d = 64, 6.5 and 10.0; of 200 chunks, d = 32, 7.0 and 10.0)
  const int pre = S > kPre * (kMergeThreads / p2) ? 0 : S > kWave ? 1 : 2;
#define RF_MERGE_LAUNCH(B16, PRE)                                                                  \
  hipLaunchKernelGGL((merge_states_kernel<B16, PRE>), dim3((unsigned)rows), dim3(kMergeThreads), 0, \
                     s, part_m, part_l, part_acc, o, Hq, Lq, S, d, p2, so)
#define RF_MERGE(B16) \
  if (pre == 2) RF_MERGE_LAUNCH(B16, 2); else if (pre == 1) RF_MERGE_LAUNCH(B16, 1); else RF_MERGE_LAUNCH(B16, 0)
  if (o_is_bf16) { RF_MERGE(true); } else { RF_MERGE(false); }
#undef RF_MERGE
#undef RF_MERGE_LAUNCH
  return hipGetLastError();
}

}  // namespace rf
