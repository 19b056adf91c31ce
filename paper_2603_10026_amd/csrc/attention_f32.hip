// fp32 fused attention, single-segment strategy (paper Section 4.3; Appendix
// A.2 incremental forms), full-precision fp32 MFMA (16x16x4).
//
// One workgroup owns 16 query rows of one (batch, head).  Its NW wavefronts
// split the key axis by interleaved 16-key tiles; each wavefront streams its
// tiles carrying the running state (m, l, acc) of the max -> sum-exp ->
// weighted-sum cascade and rescales it as each tile arrives.  The NW states
// are then merged through LDS with the level-k fused expression (Section 3.2
// Eq. (11)); acc is divided by l once, in that merge.
//
// The score tile is computed transposed, S^T = K Q^T, so that the MFMA
// accumulator layout (lane = query column, registers = key rows) is already
// the B-operand layout of the second product O^T = V^T P^T: the probabilities
// never leave their registers.
#include <type_traits>

#include "rf_device.h"
#include "rf_launch.h"

namespace rf {

// QT: tiles of 16 query rows per workgroup; a wavefront multiplies every K/V fragment it has
// fetched by all of them.
template <int D, int NW, int QT>
__global__ __launch_bounds__(NW * kWave) void attention_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
    float* __restrict__ o, Strides4 sq, Strides4 sk, Strides4 sv, Strides4 so, int Hq, int Hkv,
    int Lq, int Lk, float scale_log2e, int causal, int n_qtiles) {
  constexpr int DJ = D / 16;  // 16-wide slices of the head dim
  __shared__ float s_m[NW][16 * QT];
  __shared__ float s_l[NW][16 * QT];
  __shared__ float s_acc[NW][16 * QT][D + 4];

  // (every argument is named here so that the compiler fetches the whole argument block with its
  // first scalar loads and waits for it once: fetched where first used, the block came in three
  // round trips, each behind the wait for the previous one)
  // (n_qtiles passes through the statement: the index arithmetic below depends on it and so
  // cannot be scheduled ahead of it)
  asm volatile("" : "+s"(n_qtiles) : "s"(q), "s"(k), "s"(v), "s"(o), "s"(sq.b), "s"(sq.h), "s"(sq.l), "s"(sk.b),
               "s"(sk.h), "s"(sk.l), "s"(sv.b), "s"(sv.h), "s"(sv.l), "s"(so.b), "s"(so.h), "s"(so.l),
               "s"(Hq), "s"(Hkv), "s"(Lq), "s"(Lk), "s"(scale_log2e), "s"(causal));
  // Groups of whole tiles and the one with a ragged tile in a body each.  A choice per tile joins the registers
  // of its two sides, and where the compiler copies there it waits for a tile's loads before the next one's
  // are issued; in one line it also keeps fewer of them (77 registers, 176 before): 9216 workgroups x 872 keys
  // 543 -> 368 us, 23 heads of 395 x 3967 161 -> 145.  The other instances have no such copies and lose up
  // to 10 % on short key axes (128 heads of 100 x 300, d = 128, 41.5 -> 46.2).
  constexpr bool kTwoBodies = D == 64 && NW == 8 && QT == 1;
  const int lane = threadIdx.x & 63;
  const int wave = kTwoBodies ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : threadIdx.x >> 6;
  const int i16 = lane & 15;  // query column / key row / head-dim row inside a tile
  const int g = lane >> 4;    // lane group 0..3

  // (integer division runs on the vector unit even for wave-uniform operands: the results are
  // handed back to the scalar unit, so that the base pointers below are scalar)
  // Workgroups are dealt round-robin to the 8 XCDs, each with its own L2.  Numbered so that XCD x
  // takes a run of consecutive (head, query tile) pairs, the query tiles of one head read its K
  // and V through one L2 instead of eight (batched fp32 launch, 512 heads of 128 x 512 x 64:
  // 1.09 GB fetched from the fabric before, against 0.15 GB of inputs).
  int wg = blockIdx.x;
  if ((gridDim.x & 7) == 0) wg = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);
  const int qt = __builtin_amdgcn_readfirstlane(wg % n_qtiles);
  const int bh = __builtin_amdgcn_readfirstlane(wg / n_qtiles);
  const int h = __builtin_amdgcn_readfirstlane(bh % Hq);
  const int b = __builtin_amdgcn_readfirstlane(bh / Hq);
  const int hk = __builtin_amdgcn_readfirstlane(h / (Hq / Hkv));
  const int q0 = qt * 16 * QT;

  const float* qb = q + (int64_t)b * sq.b + (int64_t)h * sq.h;
  const float* kb = k + (int64_t)b * sk.b + (int64_t)hk * sk.h;
  const float* vb = v + (int64_t)b * sv.b + (int64_t)hk * sv.h;
  // At the sizes this kernel serves, the run time is a chain of memory latencies.  All kernel
  // arguments are therefore fetched in one go (the K/V base pointers are formed here, ahead of
  // the first load, instead of behind the wait for Q), and Q is read without branches, so
  // that its loads are only waited for at the first product, with the first K/V group already
  // on its way.
  asm volatile("" : : "s"(kb), "s"(vb));

  // Q^T fragments.  Contraction slot (g, e) of step j stands for head-dim index
  // 16j + 4g + e on both operands.
  f32x4 qf[QT][DJ];
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    // (rows past the end repeat the last query: their results are computed and never stored)
    const int qi = min(q0 + 16 * t + i16, Lq - 1);
#pragma unroll
    for (int j = 0; j < DJ; ++j)
      qf[t][j] = *reinterpret_cast<const f32x4*>(qb + (int64_t)qi * sq.l + 16 * j + 4 * g);
  }

  // last visible key of this lane's query, and of the whole query tile
  const int shift = Lk - Lq;
  int my_last[QT];
#pragma unroll
  for (int t = 0; t < QT; ++t) my_last[t] = causal ? min(Lk - 1, q0 + 16 * t + i16 + shift) : Lk - 1;
  const int tile_last = causal ? min(Lk - 1, min(Lq - 1, q0 + 16 * QT - 1) + shift) : Lk - 1;
  const int n_ktiles = tile_last >= 0 ? tile_last / 16 + 1 : 0;

  float m2[QT];  // running max, in log2 units (score * scale * log2 e)
  float l[QT];   // running sum, this lane's keys only
  // Row i of the t-th O^T tile stands for head-dim index DJ * i + t (not 16 t + i): the DJ
  // A-operand values a lane needs for one key are then DJ consecutive floats of the V row,
  // fetched with 128-bit loads, and one load instruction reads whole 64 DJ-byte row pieces.
  f32x4 acc[QT][DJ];  // acc[.][t][r] = O^T[head-dim DJ * (4g + r) + t][query i16]
#pragma unroll
  for (int qq = 0; qq < QT; ++qq) {
    m2[qq] = -INFINITY;
    l[qq] = 0.f;
#pragma unroll
    for (int t = 0; t < DJ; ++t) acc[qq][t] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // A wavefront's tiles are taken TG at a time: all K and V fragments of the group are
  // requested before the first product, so memory latency is paid once per group, not twice
  // per tile (at the small sizes this kernel serves, that latency is most of the run time).
  constexpr int TG = ((D == 64 && NW <= 8) ? 4 : 2) / QT;
  const bool small_pitch = sk.l < (1 << 26) && sv.l < (1 << 26);  // 32-bit byte offsets inside a 16-key tile
  const uint32_t k_lane = (uint32_t)(((int64_t)i16 * sk.l + 4 * g) * 4);
  const uint32_t v_lane = (uint32_t)(((int64_t)(4 * g) * sv.l + DJ * i16) * 4);
  enum { kWhole, kRagged, kEither };  // what the group's tiles are known to be
  auto group = [&](int kt0, auto kind_tag) {
    constexpr int kKind = decltype(kind_tag)::value;
    f32x4 kf[TG][DJ];
    f32x4 vf[TG][4][DJ / 4];  // vf[.][u][c][e] = V[key of step u][DJ * i16 + 4c + e]
#pragma unroll
    for (int jj = 0; jj < TG; ++jj) {
      const int key0 = min(kt0 + NW * jj, n_ktiles - 1) * 16;  // (a surplus slot re-reads the last tile)
      if (kKind == kWhole || (kKind == kEither && key0 + 16 <= Lk && small_pitch)) {
        // whole tile: a wavefront-uniform base (scalar unit) plus loop-invariant 32-bit lane
        // offsets, no per-lane 64-bit address arithmetic (which is most of this kernel's set-up)
        const char* kbase = reinterpret_cast<const char*>(kb) + (int64_t)key0 * sk.l * 4;
#pragma unroll
        for (int j = 0; j < DJ; ++j)
          kf[jj][j] = *reinterpret_cast<const f32x4*>(kbase + k_lane + 64 * j);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          // contraction slot g of step u stands for key key0 + 4g + u
          const char* vbase = reinterpret_cast<const char*>(vb) + (int64_t)(key0 + u) * sv.l * 4;
#pragma unroll
          for (int c = 0; c < DJ / 4; ++c)
            vf[jj][u][c] = *reinterpret_cast<const f32x4*>(vbase + v_lane + 16 * c);
        }
      } else {
        const float* kp = kb + (int64_t)min(key0 + i16, Lk - 1) * sk.l + 4 * g;
#pragma unroll
        for (int j = 0; j < DJ; ++j) kf[jj][j] = *reinterpret_cast<const f32x4*>(kp + 16 * j);
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const float* vp = vb + (int64_t)min(key0 + 4 * g + u, Lk - 1) * sv.l + DJ * i16;
#pragma unroll
          for (int c = 0; c < DJ / 4; ++c) vf[jj][u][c] = *reinterpret_cast<const f32x4*>(vp + 4 * c);
        }
      }
    }
#pragma unroll
    for (int jj = 0; jj < TG; ++jj) {
      const int kt = kt0 + NW * jj;
      if (kt >= n_ktiles) break;  // uniform per wavefront
      const int key0 = kt * 16;
#pragma unroll
      for (int qq = 0; qq < QT; ++qq) {
        // ---- S^T tile = K_tile Q^T (fp32 MFMA), as two independent accumulation chains ----
        f32x4 s = f32x4{0.f, 0.f, 0.f, 0.f}, s_b = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < DJ; j += 2) {
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            s = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[jj][j][e], qf[qq][j][e], s, 0, 0, 0);
            s_b = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[jj][j + 1][e], qf[qq][j + 1][e], s_b, 0, 0, 0);
          }
        }
        s += s_b;
        // s[r] = score(key key0 + 4g + r, query i16); mask, then stage 1: running max
        float tmax = -INFINITY;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int key = key0 + 4 * g + r;
          s[r] = (key <= my_last[qq]) ? s[r] * scale_log2e : -INFINITY;
          tmax = fmaxf(tmax, s[r]);
        }
        tmax = fmaxf(tmax, __shfl_xor(tmax, 16, 64));
        tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
        const float m_new = fmaxf(m2[qq], tmax);
        const float m_use = (m_new == -INFINITY) ? 0.f : m_new;  // identity repair
        const float corr = fast_exp2(m2[qq] - m_use);            // 0 when m2 == -inf
        m2[qq] = m_new;
        // stage 2: running sum of exponentials
        float p[4];
        float psum = 0.f;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          p[r] = fast_exp2(s[r] - m_use);
          psum += p[r];
        }
        l[qq] = l[qq] * corr + psum;
        // stage 3: rescale acc, then acc += V^T P^T
#pragma unroll
        for (int t = 0; t < DJ; ++t) {
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[qq][t][r] *= corr;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
#pragma unroll
          for (int t = 0; t < DJ; ++t)
            acc[qq][t] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[jj][u][t / 4][t % 4], p[u], acc[qq][t], 0, 0, 0);
        }
      }
    }
  };
  int kt0 = wave;
  if constexpr (kTwoBodies) {
    const int n_whole = small_pitch ? Lk / 16 : 0;
    for (; kt0 < n_ktiles && min(kt0 + NW * (TG - 1), n_ktiles - 1) < n_whole; kt0 += NW * TG)
      group(kt0, std::integral_constant<int, kWhole>{});
    for (; kt0 < n_ktiles; kt0 += NW * TG) group(kt0, std::integral_constant<int, kRagged>{});
  } else {
    for (; kt0 < n_ktiles; kt0 += NW * TG) group(kt0, std::integral_constant<int, kEither>{});
  }

  // ---- merge the NW wavefront states (level-k fused expression) ----
#pragma unroll
  for (int qq = 0; qq < QT; ++qq) {
    l[qq] += __shfl_xor(l[qq], 16, 64);
    l[qq] += __shfl_xor(l[qq], 32, 64);
    if (g == 0) { s_m[wave][16 * qq + i16] = m2[qq]; s_l[wave][16 * qq + i16] = l[qq]; }
#pragma unroll
    for (int t = 0; t < DJ; ++t) {
#pragma unroll
      for (int r = 0; r < 4; ++r) s_acc[wave][16 * qq + i16][DJ * (4 * g + r) + t] = acc[qq][t][r];
    }
  }
  __syncthreads();
  for (int idx = threadIdx.x; idx < 16 * QT * (D / 4); idx += NW * kWave) {
    const int qi = idx / (D / 4);
    const int c4 = idx % (D / 4);
    float mg = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) mg = fmaxf(mg, s_m[w][qi]);
    float lg = 0.f;
    f32x4 og = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float mw = s_m[w][qi];
      const float wgt = (mw == -INFINITY) ? 0.f : fast_exp2(mw - mg);
      lg += s_l[w][qi] * wgt;
      const f32x4 a = *reinterpret_cast<const f32x4*>(&s_acc[w][qi][4 * c4]);
      og += a * wgt;
    }
    const float inv = lg > 0.f ? 1.0f / lg : 0.f;
    if (q0 + qi < Lq) {
      float* op = o + (int64_t)b * so.b + (int64_t)h * so.h + (int64_t)(q0 + qi) * so.l + 4 * c4;
      *reinterpret_cast<f32x4*>(op) = og * inv;
    }
  }
}

// One or two tiles of 16 rows per workgroup.  A compute unit holds one workgroup at a time, and
// one with two tiles takes 1.4 times as long (K and V cross the L2 once for both): two tiles where they
// save enough turns.  Under a mask the turns of single tiles differ in length and fill each other's gaps,
// so that the keys a tile sees on average count, not the turns alone.  Figures fitted to 570 random
// calls; us with one / two tiles, d = 64: 512 heads of 128 x 512 148 / 111, 32 heads x 32 rows x 600
// 23.3 / 18.3, 288 workgroups of one tile x 1520 keys, causal, 39.7 / 35.1; 256 workgroups x 512 keys
// 10.2 / 15.0, 8 heads of 944 x 409, causal, 11.4 / 13.8.  d = 128: two tiles take 8 wavefronts, 512
// workgroups x 1000 keys 61.9 / 50.3, 8 heads of 1017 x 516, causal, 22.2 / 29.7; on short key axes one
// tile and 4 wavefronts, two workgroups to a compute unit, do better (512 x 256 keys 18.5 / 19.3), and 8
// wavefronts where there is a unit for each workgroup (160 x 1546 keys 52.1 with 4, 45.2 with 8).
AttnF32Route attention_f32_route(const AttnShape& a, const Strides4& sk, const Strides4& sv) {
  if (attention_f32_few_wins(a, sk, sv)) return AttnF32Route::kFewRows;
  const int64_t wg16 = (int64_t)((a.Lq + 15) / 16) * a.B * a.Hq, wg32 = (int64_t)((a.Lq + 31) / 32) * a.B * a.Hq;
  const int d128 = a.d == 128;
  const bool long_axis = !d128 || a.Lk >= 512;
  constexpr AttnCost kOne[] = {{2.0, 0, 1.64, 1.83}, {2.6, 4.4, 0, 3.4}}, kTwo[] = {{2.0, 2.67, 1.75, 2.58}, {2.0, 5.5, 1.67, 5.48}};
  auto us_of = [&](const AttnCost& c, int rows, int64_t wgs) {
    return c.us(a.Lk / 128.0 + 0.5, (double)wgs, tile_keys(a, rows) / 128 + 0.5);
  };
  if (long_axis && wg16 > 256 && us_of(kTwo[d128], 32, wg32) < 0.9 * us_of(kOne[d128], 16, wg16)) return AttnF32Route::kTwoTiles;
  // few workgroups and many keys: 16 wavefronts share the key axis of a query tile
  if (!d128) return wg16 < 256 && a.Lk > 128 ? AttnF32Route::kWaves16 : AttnF32Route::kWaves8;
  return long_axis && wg16 <= 256 ? AttnF32Route::kWaves8 : AttnF32Route::kWaves4;
}

hipError_t launch_attention_f32(const float* q, const float* k, const float* v, float* o,
                                Strides4 sq, Strides4 sk, Strides4 sv, Strides4 so,
                                const AttnShape& a, hipStream_t s) {
  const AttnF32Route route = attention_f32_route(a, sk, sv);
  if (route == AttnF32Route::kFewRows) return launch_attention_f32_few(q, k, v, o, sq, sk, sv, so, a, s);
  const bool two = route == AttnF32Route::kTwoTiles;
  const int n_qtiles = two ? (a.Lq + 31) / 32 : (a.Lq + 15) / 16;
  const int64_t grid = (int64_t)n_qtiles * a.B * a.Hq;
  if (grid > INT32_MAX) return hipErrorInvalidValue;
  const float sl2 = a.scale * kLog2e;
#define RF_LAUNCH_F32(DD, NW, QT)                                                                       \
  hipLaunchKernelGGL((attention_f32_kernel<DD, NW, QT>), dim3((unsigned)grid), dim3(NW * kWave), 0, s, q, k, v, o, \
                     sq, sk, sv, so, a.Hq, a.Hkv, a.Lq, a.Lk, sl2, a.causal, n_qtiles)
  if (a.d == 64) {
    if (two) RF_LAUNCH_F32(64, 8, 2);
    else if (route == AttnF32Route::kWaves16) RF_LAUNCH_F32(64, 16, 1);
    else RF_LAUNCH_F32(64, 8, 1);
  } else {
    if (two) RF_LAUNCH_F32(128, 8, 2);
    else if (route == AttnF32Route::kWaves8) RF_LAUNCH_F32(128, 8, 1);
    else RF_LAUNCH_F32(128, 4, 1);
  }
#undef RF_LAUNCH_F32
  return hipGetLastError();
}

}  // namespace rf
