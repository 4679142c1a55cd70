// Causal GQA attention of a prefill chunk (bf16): many rows of one sequence over its cache, which already holds the
// chunk's own K/V.
//
// The block-verification kernel gives 16 query vectors a workgroup and streams the cache through every workgroup's
// registers: right for the few queries of a verified block, but with a chunk's thousands it is bound by the L2's
// bandwidth (512 bytes of K/V per 16 queries and position).  Here a workgroup of 4 waves takes 128 consecutive query
// vectors (rows x the heads that share a KV head), 32 per wave, and walks the positions in 32-position steps whose K
// and V go to LDS once for all four (direct-to-LDS loads, a ring of kRing steps; the cache's fragment-major blocks are
// the MFMA operands, so LDS reads are contiguous and conflict-free).  A wave holds its queries, its 32 x HD output
// accumulators and one step's operands in registers: two workgroups per CU, so that one's softmax runs beside the
// other's MFMAs.  The softmax is online, in base 2 with the scale folded into one multiply-add; the accumulators are
// rescaled only in steps where some query's maximum rises (the factor is 1 otherwise), and positions are masked only
// in the steps that reach a wave's diagonal.  Later query blocks see more positions and are launched first.
// Measured (Qwen3-32B heads, one layer, block kernel -> this): 1024 rows at position 0 153 -> 44 us, 4096 rows 1072 ->
// 344 us (0.2 -> 0.8 PFLOP/s of the unmasked half).  What bounds it: per 32-position step and SIMD, two waves' 64 MFMAs (0.45 us)
// and their softmax on the vector units take 1.3 us; alone on a CU a workgroup's step takes 0.8 us, a serial chain
// of LDS reads, MFMAs, exponentials and MFMAs.
#include "gemm.h"

namespace sdd {
namespace {

constexpr int kWaves = 4, kThreads = kWaves * kWave;
constexpr int kQT = 2;                           // query tiles of 16 per wave
constexpr int kQueries = kWaves * kQT * 16;      // query vectors per workgroup
constexpr int kRing = 4;                         // steps in LDS

// One step's K and V fragments from LDS address `a` (this lane's 16 bytes of the first block; 1 KiB apart).  The
// reads and their wait are one asm block: the compiler cannot tell them from reads of the slots that direct-to-LDS
// loads are still filling and would wait for all of those loads.
#define SDD_RD(o, a, ofs) "ds_read_b128 %" #o ", %" #a " offset:" #ofs "\n\t"
template <int HD>
__device__ inline void read_step(u32x4* f, uint32_t a) {
  if constexpr (HD == 128) {
    asm volatile(SDD_RD(0, 16, 0) SDD_RD(1, 16, 1024) SDD_RD(2, 16, 2048) SDD_RD(3, 16, 3072) SDD_RD(4, 16, 4096)
                     SDD_RD(5, 16, 5120) SDD_RD(6, 16, 6144) SDD_RD(7, 16, 7168) SDD_RD(8, 16, 8192) SDD_RD(9, 16, 9216)
                         SDD_RD(10, 16, 10240) SDD_RD(11, 16, 11264) SDD_RD(12, 16, 12288) SDD_RD(13, 16, 13312)
                             SDD_RD(14, 16, 14336) SDD_RD(15, 16, 15360) "s_waitcnt lgkmcnt(0)"
                 : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(f[4]), "=&v"(f[5]), "=&v"(f[6]),
                   "=&v"(f[7]), "=&v"(f[8]), "=&v"(f[9]), "=&v"(f[10]), "=&v"(f[11]), "=&v"(f[12]), "=&v"(f[13]),
                   "=&v"(f[14]), "=&v"(f[15])
                 : "v"(a)
                 : "memory");
  } else {
    asm volatile(SDD_RD(0, 8, 0) SDD_RD(1, 8, 1024) SDD_RD(2, 8, 2048) SDD_RD(3, 8, 3072) SDD_RD(4, 8, 4096)
                     SDD_RD(5, 8, 5120) SDD_RD(6, 8, 6144) SDD_RD(7, 8, 7168) "s_waitcnt lgkmcnt(0)"
                 : "=&v"(f[0]), "=&v"(f[1]), "=&v"(f[2]), "=&v"(f[3]), "=&v"(f[4]), "=&v"(f[5]), "=&v"(f[6]), "=&v"(f[7])
                 : "v"(a)
                 : "memory");
  }
}
#undef SDD_RD

template <int HD>
__global__ void __launch_bounds__(kThreads, 2) attention_prefill_kernel(AttnPrefillArgs a) {
  constexpr int KK = HD / 32, DB = HD / 16, NB = 2 * KK + DB;  // 1 KiB blocks of a step: 2 KK of K, then DB of V
  constexpr int LQ = NB / kWaves;                              // of them per wave
  constexpr int kStage = NB * 1024;
  static_assert(2 * KK == DB && LQ % 2 == 0, "K and V take the same number of loads of each wave");
  __shared__ __align__(16) char s_ring[kRing * kStage];
  touch_kernargs<AttnPrefillArgs>();
  // KV head and query block: workgroups go to the XCDs round-robin by linear id, and a head's query blocks to as few
  // XCDs as give every XCD work (their L2s hold its K/V); the last query blocks, which see most positions, first.
  const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
  const int gh = a.heads_apart, per = a.hkv / gh, parts = kXcds / gh;
  const int kvh = xcd % gh + gh * (slot % per), rank = slot / per * parts + xcd / gh;
  if (rank >= a.qblocks) return;
  const int qb = a.qblocks - 1 - rank;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int QV = a.R * a.grp, q_first = qb * kQueries, qw = q_first + wave * kQT * 16;
  const int r_hi = min(a.R - 1, (q_first + kQueries - 1) / a.grp);
  const RowInfo first = a.rows[0];
  const int pos_hi = a.rows[r_hi].pos;
  const int w_lo = min(a.R - 1, qw / a.grp), w_hi = min(a.R - 1, (qw + kQT * 16 - 1) / a.grp);
  const int wlo_pos = a.rows[w_lo].pos, whi_pos = a.rows[w_hi].pos;  // the wave's first and last row
  int qpos[kQT], qrow[kQT], qh[kQT];
  uint4 qf[kQT][KK];  // lanes past the last query vector hold row 0's (not stored)
#pragma unroll
  for (int t = 0; t < kQT; ++t) {
    const int qv = qw + 16 * t + lane % 16;
    qrow[t] = qv < QV ? qv / a.grp : 0;
    qh[t] = kvh * a.grp + (qv < QV ? qv % a.grp : 0);
    qpos[t] = a.rows[qrow[t]].pos;
    const uint16_t* Q = a.q + ((int64_t)qrow[t] * a.hq + qh[t]) * HD;
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) qf[t][kk] = load16(Q + 32 * kk + 8 * (lane / 16));
  }
  const int kv_end = __builtin_amdgcn_readfirstlane(first.valid ? pos_hi + 1 : 0);
  const int wave_lo = __builtin_amdgcn_readfirstlane(wlo_pos);
  const int wave_end = __builtin_amdgcn_readfirstlane(min(whi_pos + 1, kv_end));
  const int n = (kv_end + 31) / 32;  // steps; (kv_end - 1) / 32 * 32 + 32 <= ld, a multiple of 64
  const int64_t head = (int64_t)first.seq * a.hkv + kvh;
  const int hbytes = a.ld * HD * 2;  // < 2^31: checked on the host
  char* const K = const_cast<char*>(reinterpret_cast<const char*>(a.kc + head * a.ld * HD));
  char* const V = const_cast<char*>(reinterpret_cast<const char*>(a.vc + head * a.ld * HD));
  // the query loads complete before the ring's go out, so that no wait in the loop is for them
  __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);

  // Step t's loads: wave w takes blocks w, w + 4, ... (K first, then V).  Every call issues the same ones, so that
  // the memory-counter waits count alike; past the last step the descriptors have no range.
  int slot_b = 0, st = 0;
  auto issue = [&]() {
    const int range = st < n ? hbytes : 0;
    const __amdgpu_buffer_rsrc_t krs = __builtin_amdgcn_make_buffer_rsrc(K, 0, range, kBufferRsrcWord3);
    const __amdgpu_buffer_rsrc_t vrs = __builtin_amdgcn_make_buffer_rsrc(V, 0, range, kBufferRsrcWord3);
    const int ofs = st * (NB / 2) * 1024 + wave * 1024;
#pragma unroll
    for (int i = 0; i < LQ / 2; ++i) {
      load_lds16<0>(krs, s_ring + slot_b + (wave + kWaves * i) * 1024, lane * 16, ofs + i * kWaves * 1024);
      load_lds16<0>(vrs, s_ring + slot_b + (NB / 2 + wave + kWaves * i) * 1024, lane * 16, ofs + i * kWaves * 1024);
    }
    slot_b = slot_b + kStage == kRing * kStage ? 0 : slot_b + kStage;
    ++st;
  };
#pragma unroll
  for (int i = 0; i < kRing - 1; ++i) issue();

  f32x4 o[kQT][DB];
  float m[kQT], l[kQT];  // running maximum (scaled, base 2) and this lane's part of the sum
#pragma unroll
  for (int t = 0; t < kQT; ++t) {
    m[t] = -INFINITY;
    l[t] = 0.f;
#pragma unroll
    for (int db = 0; db < DB; ++db) o[t][db] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const float c = a.scale * 1.44269504088896340736f;
  const int g8 = 8 * (lane / 16);
  const uint32_t ring = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)(s_ring) + lane * 16;
  uint32_t so = 0;
#pragma unroll 1
  for (int s = 0; s < n; ++s) {
    __builtin_amdgcn_s_waitcnt(wait_vmcnt((kRing - 2) * LQ));  // this wave's loads of step s have landed
    phase_barrier();  // everyone's have, and the slot of step s - 1 has been read by every wave
    issue();
    u32x4 f[NB];
    read_step<HD>(f, ring + so);
    so = so + kStage == kRing * kStage ? 0 : so + kStage;
    const int p = 32 * s;
    if (p >= wave_end) continue;  // past all of this wave's queries
    f32x4 sc[kQT][2];
#pragma unroll
    for (int t = 0; t < kQT; ++t)
#pragma unroll
      for (int b = 0; b < 2; ++b) {
        sc[t][b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < KK; ++kk)
          sc[t][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f[b * KK + kk]),
                                                             __builtin_bit_cast(bf16x8, qf[t][kk]), sc[t][b], 0, 0, 0);
      }
    // sc[t][b][i]: position p + g8 + 4 b + i of the lane's query
    if (p + 31 > wave_lo) {  // the step reaches past the wave's first row's position
#pragma unroll
      for (int t = 0; t < kQT; ++t)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            if (p + g8 + 4 * b + i > qpos[t]) sc[t][b][i] = -INFINITY;
      // entries past the wave's last position may hold stale values, and 0 times a non-finite one is not 0
      const int nv = wave_end - (p + g8);
      uint32_t mask[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) mask[i] = (2 * i < nv ? 0xFFFFu : 0u) | (2 * i + 1 < nv ? 0xFFFF0000u : 0u);
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int i = 0; i < 4; ++i) f[2 * KK + db][i] &= mask[i];
    }
    uint4 pf[kQT];
#pragma unroll
    for (int t = 0; t < kQT; ++t) {
      float mx = fmaxf(fmaxf(fmaxf(sc[t][0][0], sc[t][0][1]), fmaxf(sc[t][0][2], sc[t][0][3])),
                       fmaxf(fmaxf(sc[t][1][0], sc[t][1][1]), fmaxf(sc[t][1][2], sc[t][1][3])));
      mx = xor16_op(mx, [](float x, float y) { return fmaxf(x, y); });
      mx = xor32_op(mx, [](float x, float y) { return fmaxf(x, y); }) * c;
      if (__any(mx > m[t])) {
        const float mnew = fmaxf(m[t], mx);
        const float alpha = m[t] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m[t] - mnew);
        m[t] = mnew;
        l[t] *= alpha;
#pragma unroll
        for (int db = 0; db < DB; ++db) o[t][db] *= alpha;
      }
      const float mm = m[t] == -INFINITY ? 0.f : m[t];  // (a query with no position so far: every term is 2^-inf)
      float e[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) e[i] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[t][i / 4][i % 4], c, -mm));
      l[t] += ((e[0] + e[1]) + (e[2] + e[3])) + ((e[4] + e[5]) + (e[6] + e[7]));
      pf[t] = make_uint4(pack_bf16x2(e[0], e[1]), pack_bf16x2(e[2], e[3]), pack_bf16x2(e[4], e[5]), pack_bf16x2(e[6], e[7]));
    }
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int t = 0; t < kQT; ++t)
        o[t][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, f[2 * KK + db]),
                                                           __builtin_bit_cast(bf16x8, pf[t]), o[t][db], 0, 0, 0);
  }
  __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);  // the loads past the end (no memory access) before the block may end
  // o[t][db][i]: dimension 16 db + 4 (lane / 16) + i of query lane % 16
#pragma unroll
  for (int t = 0; t < kQT; ++t) {
    float L = xor16_op(l[t], [](float x, float y) { return x + y; });
    L = xor32_op(L, [](float x, float y) { return x + y; });
    const float inv = 1.f / L;
    if (qw + 16 * t + lane % 16 < QV) {
#pragma unroll
      for (int db = 0; db < DB; ++db)
        *reinterpret_cast<uint2*>(a.out + xfrag_index<uint16_t>(qrow[t], qh[t] * HD + 16 * db + 4 * (lane / 16), a.hq * HD / 32)) =
            L > 0.f ? make_uint2(pack_bf16x2(o[t][db][0] * inv, o[t][db][1] * inv),
                                 pack_bf16x2(o[t][db][2] * inv, o[t][db][3] * inv))
                    : make_uint2(0, 0);
    }
  }
}

}  // namespace

int launch_attention_prefill(AttnPrefillArgs a, int head_dim, hipStream_t st) {
  if ((int64_t)a.ld * head_dim * 2 >= (int64_t(1) << 31))
    return fail(SDD_EUNSUPPORTED, "a cache of %d positions exceeds the 32-bit buffer offsets", a.ld);
  a.qblocks = (int)ceil_div((int64_t)a.R * a.grp, kQueries);
  a.heads_apart = kXcds;  // the largest power of two up to 8 that divides the KV heads
  while (a.hkv % a.heads_apart) a.heads_apart /= 2;
  const int per = a.hkv / a.heads_apart, parts = kXcds / a.heads_apart;
  const dim3 grid(kXcds * per * (int)ceil_div(a.qblocks, parts));
  if (head_dim == 128)
    hipLaunchKernelGGL(attention_prefill_kernel<128>, grid, dim3(kThreads), 0, st, a);
  else
    hipLaunchKernelGGL(attention_prefill_kernel<64>, grid, dim3(kThreads), 0, st, a);
  return check_launch("attention_prefill_kernel");
}

}  // namespace sdd
