// fp32 attention for launches with few query tiles (one short head, a few queries against a long
// context): the cascade of attention_f32.hip (max -> sum-exp -> weighted sum, all in fp32) in
// tiles of 4 query rows.
//
// At 16 rows per workgroup such a launch occupies a handful of compute units, and their fp32
// matrix pipes (or the chain of memory trips) set its time: 128 x 512 x 64 on 8 workgroups is
// 3.4 us of matrix work alone.  v_mfma_f32_4x4x1 does the same work per cycle on 16 independent
// 4 x 4 blocks, so 4 rows lose nothing: 4 times the workgroups, a quarter of the work in each.
//
//   S = Q K^T     A = Q, one head-dim index at a time, broadcast to all 16 blocks; B = K^T, block b
//                 = keys 4 b .. 4 b + 3: lane l ends up with the scores of key l for the 4 rows
//   O = P V       A = P of 4 keys (one from each quarter of the tile), broadcast within the
//                 quarter's 4 blocks; B = V, quarter G = lanes 16 G ..: a lane holds 4 (8)
//                 head-dim values per key, summed over its quarter's keys
//
// A wavefront takes tiles of 64 keys.  K goes through a wavefront-private LDS tile (whole rows in,
// one row per lane out), V straight into registers; all of a tile is requested at once.  The NW
// wavefronts' states are merged through LDS at the end.  Rows are packed: the Hq / Hkv heads that
// share a KV head times Lq.
#include <utility>

#include "rf_device.h"
#include "rf_launch.h"

namespace rf {

namespace {
constexpr int kF4Waves = 8;
constexpr int kF4Keys = 64;    // keys per wavefront step
constexpr int kF4Pitch = 272;  // bytes per staged K row of 64 floats: 16 lanes' rows start in 16 different slots

template <typename F, int... I>
__device__ __forceinline__ void static_for_(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_(f, std::make_integer_sequence<int, N>{});
}
}  // namespace

template <int D>
__global__ __launch_bounds__(kF4Waves * kWave, 2) void attention_f32_few_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    float* __restrict__ o, Strides4 sq, Strides4 sk, Strides4 sv, Strides4 so, int Hq, int Hkv,
    int Lq, int Lk, float scale_log2e, int causal, int n_rtiles) {
  constexpr int NW = kF4Waves;
  constexpr int DH = D / 64;  // 64-float pieces of a row
  __shared__ __attribute__((aligned(16))) unsigned char smem[NW * kF4Keys * kF4Pitch];
  __shared__ float s_m[NW][4], s_l[NW][4];
  static_assert(NW * 16 * D * 4 <= NW * kF4Keys * kF4Pitch, "the merge buffer fits the staging space");

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c16 = lane & 15;
  const int g = lane >> 4;

  // (workgroups are dealt round-robin to the 8 XCDs: the row tiles of a head go to one)
  int wg = blockIdx.x;
  if ((gridDim.x & 7) == 0) wg = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const int rt = __builtin_amdgcn_readfirstlane(wg % n_rtiles);
  const int unit = __builtin_amdgcn_readfirstlane(wg / n_rtiles);
  const int hk = __builtin_amdgcn_readfirstlane(unit % Hkv);
  const int b = __builtin_amdgcn_readfirstlane(unit / Hkv);
  const int grp = Hq / Hkv;
  const int R = grp * Lq;
  const int r0 = rt * 4;
  const int shift = Lk - Lq;

  // last visible key of each row (rows past the end repeat the last one and are not stored)
  int last[4], hi = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int r = min(r0 + i, R - 1);
    last[i] = __builtin_amdgcn_readfirstlane(causal ? min(Lk - 1, r % Lq + shift) : Lk - 1);
    hi = max(hi, last[i] + 1);
  }

  const float* kb = k + (int64_t)b * sk.b + (int64_t)hk * sk.h;
  const float* vb = v + (int64_t)b * sv.b + (int64_t)hk * sv.h;
  // Buffer loads whose range ends with the last key's row: what a ragged last tile asks for past
  // it comes back as zeros (and is masked).  All offsets are 32-bit (checked by the launcher).
  const uint32_t sk4 = (uint32_t)sk.l * 4, sv4 = (uint32_t)sv.l * 4;
  const auto krs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(kb), 0, (uint32_t)(Lk - 1) * sk4 + 4 * D, 0x00020000);
  const auto vrs = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(vb), 0, (uint32_t)(Lk - 1) * sv4 + 4 * D, 0x00020000);

  // One 64-float piece h of a tile's K or V each: kr[n] = K[key 4 n + g][64 h + 4 c16 ..],
  // vr[n] = V[key 16 g + n][64 h + 4 c16 ..].  At D = 128 kr holds the second piece of V once the
  // second piece of K has gone to LDS.
  u32x4 kr[16], vr[16];
  auto load_k = [&](u32x4 (&reg)[16], int key0, int h) {
    uint32_t off = (uint32_t)(key0 + g) * sk4 + 16 * c16 + 256 * h;
#pragma unroll
    for (int n = 0; n < 16; ++n) {
      reg[n] = __builtin_amdgcn_raw_buffer_load_b128(krs, off, 0, 0);
      off += 4 * sk4;
    }
  };
  auto load_v = [&](u32x4 (&reg)[16], int key0, int h) {
    uint32_t off = (uint32_t)(key0 + 16 * g) * sv4 + 16 * c16 + 256 * h;
#pragma unroll
    for (int n = 0; n < 16; ++n) {
      reg[n] = __builtin_amdgcn_raw_buffer_load_b128(vrs, off, 0, 0);
      off += sv4;
    }
  };

  int key0 = wave * kF4Keys;
  // Q, A operand: qa[m] of lane (block bb, row i) = Q[row i][16 m + bb]
  float qa[4 * DH];
  {
    const int r = min(r0 + (lane & 3), R - 1);
    const float* qp = q + (int64_t)b * sq.b + (int64_t)(hk * grp + r / Lq) * sq.h + (int64_t)(r % Lq) * sq.l + (lane >> 2);
#pragma unroll
    for (int m = 0; m < 4 * DH; ++m) qa[m] = qp[16 * m];
  }
  __builtin_amdgcn_sched_barrier(0);
  load_k(kr, key0 < hi ? key0 : Lk, 0);
  __builtin_amdgcn_sched_barrier(0);
  load_v(vr, key0 < hi ? key0 : Lk, 0);
  __builtin_amdgcn_sched_barrier(0);

  unsigned char* ktile = smem + wave * (kF4Keys * kF4Pitch);
  float m2[4], l[4];
  f32x4 acc[4 * DH];  // acc[4 h + e][i] = O[row i][64 h + 4 c16 + e], keys of quarter g
#pragma unroll
  for (int i = 0; i < 4; ++i) { m2[i] = -INFINITY; l[i] = 0.f; }
#pragma unroll
  for (int e = 0; e < 4 * DH; ++e) acc[e] = f32x4{0.f, 0.f, 0.f, 0.f};

  for (; key0 < hi; key0 += NW * kF4Keys) {
    // (the last turn asks for keys past the end: nothing is fetched, and there is no branch)
    const int next = key0 + NW * kF4Keys < hi ? key0 + NW * kF4Keys : Lk;
    f32x4 s4[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) s4[m] = f32x4{0.f, 0.f, 0.f, 0.f};
    static_for<DH>([&](auto h_) {
      constexpr int h = decltype(h_)::value;
#pragma unroll
      for (int n = 0; n < 16; ++n)
        *reinterpret_cast<u32x4*>(ktile + (4 * n + g) * kF4Pitch + 16 * c16) = kr[n];
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
      if constexpr (h + 1 < DH) load_k(kr, key0, h + 1);
      else if constexpr (DH == 2) load_v(kr, key0, 1);
      else load_k(kr, next, 0);
      __builtin_amdgcn_sched_barrier(0);
      static_for<16>([&](auto c_) {  // head-dim indices 64 h + 4 c .. + 3
        constexpr int c = decltype(c_)::value;
        const f32x4 kv = *reinterpret_cast<const f32x4*>(ktile + lane * kF4Pitch + 16 * c);
        constexpr int m = c >> 2;
        s4[m] = __builtin_amdgcn_mfma_f32_4x4x1f32(qa[4 * h + m], kv[0], s4[m], 4, 4 * (c & 3) + 0, 0);
        s4[m] = __builtin_amdgcn_mfma_f32_4x4x1f32(qa[4 * h + m], kv[1], s4[m], 4, 4 * (c & 3) + 1, 0);
        s4[m] = __builtin_amdgcn_mfma_f32_4x4x1f32(qa[4 * h + m], kv[2], s4[m], 4, 4 * (c & 3) + 2, 0);
        s4[m] = __builtin_amdgcn_mfma_f32_4x4x1f32(qa[4 * h + m], kv[3], s4[m], 4, 4 * (c & 3) + 3, 0);
      });
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
    });
    const f32x4 s = (s4[0] + s4[1]) + (s4[2] + s4[3]);
    // s[i] = score(row i, key key0 + lane); stages 1 and 2: running max, running sum
    float p[4], corr[4], tmax[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      p[i] = (key0 + lane <= last[i]) ? s[i] * scale_log2e : -INFINITY;
      tmax[i] = wave_max(p[i]);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float m_new = fmaxf(m2[i], tmax[i]);
      const float m_use = (m_new == -INFINITY) ? 0.f : m_new;  // identity repair
      corr[i] = fast_exp2(m2[i] - m_use);
      m2[i] = m_new;
      p[i] = fast_exp2(p[i] - m_use);
      l[i] = l[i] * corr[i] + p[i];
    }
    // stage 3: 4 x 4 transpose inside every block of 4 lanes (register i, lane j <-> register j,
    // lane i) makes the probabilities the A operand
    float pt[4];
    static_for<4>([&](auto j_) {
      constexpr int j = decltype(j_)::value;
      constexpr int kBcast = j * 0x55;  // quad_perm [j, j, j, j]
      const float a0 = dpp_f32<kBcast>(p[0]), a1 = dpp_f32<kBcast>(p[1]);
      const float a2 = dpp_f32<kBcast>(p[2]), a3 = dpp_f32<kBcast>(p[3]);
      const float lo = (lane & 1) ? a1 : a0, up = (lane & 1) ? a3 : a2;
      pt[j] = (lane & 2) ? up : lo;
    });
#pragma unroll
    for (int e = 0; e < 4 * DH; ++e)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[e][i] *= corr[i];
    static_for<DH>([&](auto h_) {
      constexpr int h = decltype(h_)::value;
      static_for<16>([&](auto n_) {
        constexpr int n = decltype(n_)::value;
        const u32x4 vv = h == 0 ? vr[n] : kr[n];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc[4 * h + e] = __builtin_amdgcn_mfma_f32_4x4x1f32(pt[n & 3], __uint_as_float(vv[e]), acc[4 * h + e], 2, n >> 2, 0);
      });
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (h == 0) load_v(vr, next, 0);
      else load_k(kr, next, 0);
      __builtin_amdgcn_sched_barrier(0);
    });
  }

  // ---- merge the wavefront states (level-k fused expression) ----
#pragma unroll
  for (int i = 0; i < 4; ++i) l[i] = wave_sum(l[i]);
  if (lane == 0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) { s_m[wave][i] = m2[i]; s_l[wave][i] = l[i]; }
  }
  __syncthreads();  // K staging is dead from here on
  float* s_acc = reinterpret_cast<float*>(smem);  // [wave][quarter][row][D]
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int h = 0; h < DH; ++h)
      *reinterpret_cast<f32x4*>(s_acc + ((wave * 4 + g) * 4 + i) * D + 64 * h + 4 * c16) =
          f32x4{acc[4 * h][i], acc[4 * h + 1][i], acc[4 * h + 2][i], acc[4 * h + 3][i]};
  __syncthreads();
  if (threadIdx.x < 4 * D) {
    const int i = threadIdx.x / D, d = threadIdx.x % D;
    float mg = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) mg = fmaxf(mg, s_m[w][i]);
    const float mg_use = (mg == -INFINITY) ? 0.f : mg;
    float lg = 0.f, og = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float wgt = fast_exp2(s_m[w][i] - mg_use);  // 0 for an empty state
      lg += s_l[w][i] * wgt;
      const float* a = s_acc + (w * 16 + i) * D + d;
      og += ((a[0] + a[4 * D]) + (a[8 * D] + a[12 * D])) * wgt;
    }
    const int r = r0 + i;
    if (r < R) {
      const float inv = lg > 0.f ? 1.0f / lg : 0.f;
      o[(int64_t)b * so.b + (int64_t)(hk * grp + r / Lq) * so.h + (int64_t)(r % Lq) * so.l + d] = og * inv;
    }
  }
}

static int64_t f32_few_tiles(const AttnShape& a) { return ((int64_t)(a.Hq / a.Hkv) * a.Lq + 3) / 4; }

// Up to a workgroup per compute unit, and keys for most of the wavefronts.  us here / in tiles of
// 16 rows: 128 x 512 x 64 8.0 / 10.7, 7 queries of 6 heads over 1699 keys 13.9 / 23.8, 1024 x 2048 x
// 128 29.2 / 66.1 (256 workgroups); beyond one round the 16-row tiles' reuse of K and V wins
// (16 heads of 128 x 512 x 64, 512 workgroups here: 15.5 / 11.3), and so do they on a key tile or
// two (36 keys: 6.3 / 5.4).
bool attention_f32_few_wins(const AttnShape& a, const Strides4& sk, const Strides4& sv) {
  // 32-bit byte offsets inside one head of k and of v, with room for a step past the end
  const int64_t rows = (int64_t)a.Lk + (kF4Waves + 1) * kF4Keys;
  auto ok = [&](int64_t l) { return l >= 0 && l < ((int64_t)1 << 29) && (rows * l + a.d) * 4 < ((int64_t)1 << 32); };
  return a.Lk > 2 * kF4Keys && ok(sk.l) && ok(sv.l) && f32_few_tiles(a) * a.B * a.Hkv <= 256;
}

hipError_t launch_attention_f32_few(const float* q, const float* k, const float* v, float* o, Strides4 sq,
                                    Strides4 sk, Strides4 sv, Strides4 so, const AttnShape& a, hipStream_t s) {
  const int64_t n_rt = f32_few_tiles(a);
  const int64_t grid = n_rt * a.B * a.Hkv;
  if (grid > INT32_MAX || (a.d != 64 && a.d != 128)) return hipErrorInvalidValue;
#define RF_F32_FEW(DD)                                                                                        \
  hipLaunchKernelGGL((attention_f32_few_kernel<DD>), dim3((unsigned)grid), dim3(kF4Waves * kWave), 0, s, q, k, v, \
                     o, sq, sk, sv, so, a.Hq, a.Hkv, a.Lq, a.Lk, a.scale * kLog2e, a.causal, (int)n_rt)
  if (a.d == 64) RF_F32_FEW(64);
  else RF_F32_FEW(128);
#undef RF_F32_FEW
  return hipGetLastError();
}

}  // namespace rf
