// Causal GQA attention of a prefill chunk (bf16): many rows of one sequence over its cache, which already holds the
// chunk's own K/V.
//
// The block-verification kernel gives 16 query vectors a workgroup and streams the cache through every workgroup's
// registers: right for the few queries of a verified block, but with a chunk's thousands it is bound by the L2's
// bandwidth (512 bytes of K/V per 16 queries and position).  This kernel computes the same results bit for bit (so a
// row's cached K/V do not depend on the chunk it was computed in): wave w takes the 32-position steps w, w + 8, ... in
// order, and the waves' partial results are added in wave order, per query in the same operations.  But a workgroup
// holds kQT tiles of 16 query vectors (rows x the heads that share a KV head), so that a step's K and V, loaded once
// into a wave's registers, serve kQT times as many.  A step's K registers take the next step's as soon as the tiles'
// scores are computed, and the V registers after the last product; the queries' fragments sit in LDS.
// Positions are masked only in the steps that reach a tile's diagonal, accumulators rescaled only where some query's
// maximum rises (the factor is 1 otherwise).  Later query blocks see more positions and are launched first.
// Measured, block kernel -> this, one layer of a prompt in one chunk (Qwen3-32B / Qwen2.5-7B heads): 66-96 rows 18 / 17 ->
// 12 / 12 us, 256 rows 35 / 35 -> 21 / 14, 1024 rows 156 / 136 -> 78 / 41, 4096 rows 1092 / 905 -> 623 / 268.  What bounds it:
// a wave takes 1.8 us per step of three tiles, 0.3 us of them MFMAs: the softmax on the vector units, with two waves per
// SIMD to cover the loads (three tiles take 244 registers; four spill); below a thousand rows a workgroup's start and the
// combination of its waves.  Sharing a step's K/V between waves through LDS (a wave per 32 queries, positions in one
// sequence) takes 42 us for 1024 rows and 356 for 4096, but adds a query's positions in another order.
#include "gemm.h"

namespace sdd {
namespace {

constexpr int kWaves = kAttnWaves, kThreads = kWaves * kWave;

template <int HD, int QT>
__global__ void __launch_bounds__(kThreads, 1) attention_prefill_kernel(AttnPrefillArgs a) {
#pragma clang fp contract(off)  // rounds where the block kernel rounds
  constexpr int KK = HD / 32, DB = HD / 16;
  __shared__ __align__(16) float s_o[2][kWaves][16][HD + 4];
  __shared__ __align__(16) char s_q[QT * KK * 1024];
  __shared__ float s_m[QT][kWaves][16], s_l[QT][kWaves][16], s_f[QT][kWaves][16], s_L[QT][16];
  touch_kernargs<AttnPrefillArgs>();
  // KV head and query block: workgroups go to the XCDs round-robin by linear id, and a head's query blocks to as few
  // XCDs as give every XCD work (their L2s hold its K/V); the last query blocks, which see most positions, first.
  const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
  const int gh = a.heads_apart, per = a.hkv / gh, parts = kXcds / gh;
  const int kvh = xcd % gh + gh * (slot % per), rank = slot / per * parts + xcd / gh;
  if (rank >= a.qblocks) return;
  const int q_first = (a.qblocks - 1 - rank) * 16 * QT;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int QV = a.R * a.grp, g8 = 8 * (lane / 16);
  const RowInfo first = a.rows[0];
  // fragment f of the queries (tile f / KK, dimensions 32 (f % KK) ..) goes to LDS by wave f % kWaves
  for (int f = wave; f < QT * KK; f += kWaves) {
    const int qv = q_first + 16 * (f / KK) + lane % 16;
    const int r = qv < QV ? qv / a.grp : 0, h = qv < QV ? qv % a.grp : 0;
    *reinterpret_cast<uint4*>(s_q + f * 1024 + lane * 16) =
        load16(a.q + ((int64_t)r * a.hq + kvh * a.grp + h) * HD + 32 * (f % KK) + g8);
  }
  // the lane's query's position (-1: none); a tile's first position, the one past its last (a chunk's rows are consecutive)
  int qpos[QT], lo[QT], end[QT];
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    const int q0 = q_first + 16 * t, qv = q0 + lane % 16;
    qpos[t] = qv < QV ? first.pos + qv / a.grp : -1;
    lo[t] = __builtin_amdgcn_readfirstlane(q0 + 15 < QV ? first.pos + q0 / a.grp : -1);
    end[t] = __builtin_amdgcn_readfirstlane(first.valid && q0 < QV ? first.pos + min(a.R - 1, (q0 + 15) / a.grp) + 1 : 0);
  }
  int kv_end = 0;
#pragma unroll
  for (int t = 0; t < QT; ++t) kv_end = max(kv_end, end[t]);
  const int64_t head = (int64_t)first.seq * a.hkv + kvh;
  const uint16_t* K = a.kc + head * a.ld * HD + lane * 8;
  const uint16_t* V = a.vc + head * a.ld * HD + lane * 8;

  // A loaded step starts below kv_end <= ld and ld is a multiple of 64, so its blocks lie inside the head's cache.
  // Entries at positions at or past a tile's end may hold stale values: their scores are masked and their V values
  // zeroed (P is 0 there, and 0 times a stale non-finite value would not be).
  uint4 kf[2][KK], vf[DB];
  auto load_k = [&](int p) {
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) kf[b][kk] = load16(K + (int64_t)(p / 32) * 32 * HD + (b * KK + kk) * 512);
  };
  auto load_v = [&](int p) {
#pragma unroll
    for (int db = 0; db < DB; ++db) vf[db] = load16(V + (int64_t)(p / 32) * 32 * HD + db * 512);
  };
  f32x4 o[QT][DB];
  float m[QT], l[QT];  // running maximum, this lane's part of the sum
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    m[t] = -INFINITY;
    l[t] = 0.f;
#pragma unroll
    for (int db = 0; db < DB; ++db) o[t][db] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  constexpr int kStride = 32 * kWaves;
  const int p_last = kv_end > 0 ? (kv_end - 1) / 32 * 32 : 0;
  const bool any = kv_end > 32 * wave;
  if (any) {
    load_k(32 * wave);
    load_v(32 * wave);
  }
  __syncthreads();  // the queries are in LDS
#pragma unroll 1
  for (int p = 32 * wave; p < kv_end; p += kStride) {
    f32x4 sacc[QT][2];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      sacc[t][0] = sacc[t][1] = f32x4{0.f, 0.f, 0.f, 0.f};
      if (p < end[t]) {
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
          const bf16x8 q = *reinterpret_cast<const bf16x8*>(s_q + (t * KK + kk) * 1024 + lane * 16);
#pragma unroll
          for (int b = 0; b < 2; ++b)
            sacc[t][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kf[b][kk]), q, sacc[t][b], 0, 0, 0);
        }
      }
    }
    load_k(min(p + kStride, p_last));
    __builtin_amdgcn_sched_barrier(0);
    uint4 pf[QT];
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      pf[t] = make_uint4(0, 0, 0, 0);
      if (p >= end[t]) continue;
      // sacc[t][b][i]: position p + g8 + 4 b + i, query column lane % 16
      float sv[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) sv[i] = sacc[t][i / 4][i % 4] * a.scale;
      if (p + 31 > lo[t]) {
#pragma unroll
        for (int i = 0; i < 8; ++i) sv[i] = p + g8 + i <= qpos[t] ? sv[i] : -INFINITY;
      }
      float mloc = -INFINITY;
#pragma unroll
      for (int i = 0; i < 8; ++i) mloc = fmaxf(mloc, sv[i]);
      mloc = xor16_op(mloc, [](float x, float y) { return fmaxf(x, y); });
      mloc = xor32_op(mloc, [](float x, float y) { return fmaxf(x, y); });
      const float mnew = fmaxf(m[t], mloc);
      float lsum = 0.f;
      float e[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        e[i] = sv[i] == -INFINITY ? 0.f : __expf(sv[i] - mnew);
        lsum += e[i];
      }
      pf[t] = make_uint4(pack_bf16x2(e[0], e[1]), pack_bf16x2(e[2], e[3]), pack_bf16x2(e[4], e[5]), pack_bf16x2(e[6], e[7]));
      if (__any(mnew != m[t])) {
        const float alpha = m[t] == -INFINITY ? 0.f : __expf(m[t] - mnew);
        l[t] = __builtin_fmaf(l[t], alpha, lsum);
#pragma unroll
        for (int db = 0; db < DB; ++db) o[t][db] *= alpha;
        m[t] = mnew;
      } else {
        l[t] += lsum;
      }
    }
#pragma unroll
    for (int t = 0; t < QT; ++t) {
      if (p >= end[t]) continue;
      if (p + 32 > end[t]) {
        const int nv = end[t] - (p + g8);  // valid positions of the lane's 8 (may be <= 0 or >= 8)
        uint32_t mask[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) mask[i] = (2 * i < nv ? 0xFFFFu : 0u) | (2 * i + 1 < nv ? 0xFFFF0000u : 0u);
#pragma unroll
        for (int db = 0; db < DB; ++db) {
          const uint4 v = make_uint4(vf[db].x & mask[0], vf[db].y & mask[1], vf[db].z & mask[2], vf[db].w & mask[3]);
          o[t][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, v), __builtin_bit_cast(bf16x8, pf[t]),
                                                             o[t][db], 0, 0, 0);
        }
      } else {
#pragma unroll
        for (int db = 0; db < DB; ++db)
          o[t][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf[db]),
                                                             __builtin_bit_cast(bf16x8, pf[t]), o[t][db], 0, 0, 0);
      }
    }
    load_v(min(p + kStride, p_last));
  }
  // the waves' partial (max, sum, O) in wave order; O two tiles at a time through LDS
  auto publish = [&](int t) {
#pragma unroll
    for (int db = 0; db < DB; ++db)
      *reinterpret_cast<f32x4*>(&s_o[t % 2][wave][lane % 16][16 * db + 4 * (lane / 16)]) = o[t][db];
  };
#pragma unroll
  for (int t = 0; t < QT; ++t) {
    float ltot = xor16_op(l[t], [](float x, float y) { return x + y; });
    ltot = xor32_op(ltot, [](float x, float y) { return x + y; });
    if (lane < 16) {
      s_m[t][wave][lane] = m[t];
      s_l[t][wave][lane] = ltot;
    }
  }
#pragma unroll
  for (int t0 = 0; t0 < QT; t0 += 2) {
    if (t0 > 0) __syncthreads();
#pragma unroll
    for (int t = t0; t < min(QT, t0 + 2); ++t) publish(t);
    __syncthreads();
    if (t0 == 0) {
      const int i = threadIdx.x;
      if (i < 16 * QT) attn_factors(s_m[i / 16], s_l[i / 16], s_f[i / 16], s_L[i / 16], i % 16);
      __syncthreads();
    }
#pragma unroll
    for (int t = t0; t < min(QT, t0 + 2); ++t)
      attn_combine<HD>(s_o[t % 2], s_f[t], s_L[t], [&](int q, int dim, const float* y) {
        const int qv = q_first + 16 * t + q;
        if (qv < QV)
          *reinterpret_cast<uint2*>(a.out + xfrag_index<uint16_t>(qv / a.grp, (kvh * a.grp + qv % a.grp) * HD + dim,
                                                                  a.hq * HD / 32)) =
              make_uint2(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]));
      });
  }
}

}  // namespace

int launch_attention_prefill(AttnPrefillArgs a, int head_dim, hipStream_t st) {
  constexpr int QT = kAttnPrefillQueries / 16;
  a.qblocks = (int)ceil_div((int64_t)a.R * a.grp, 16 * QT);
  a.heads_apart = kXcds;  // the largest power of two up to 8 that divides the KV heads
  while (a.hkv % a.heads_apart) a.heads_apart /= 2;
  const int per = a.hkv / a.heads_apart, parts = kXcds / a.heads_apart;
  const dim3 grid(kXcds * per * (int)ceil_div(a.qblocks, parts));
  if (head_dim == 128)
    hipLaunchKernelGGL((attention_prefill_kernel<128, QT>), grid, dim3(kThreads), 0, st, a);
  else
    hipLaunchKernelGGL((attention_prefill_kernel<64, QT>), grid, dim3(kThreads), 0, st, a);
  return check_launch("attention_prefill_kernel");
}

}  // namespace sdd
