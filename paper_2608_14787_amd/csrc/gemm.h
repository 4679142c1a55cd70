// GEMM building blocks shared by the 33-row stream-K kernels (decoder.hip) and
// the many-row kernel (tiles.hip): launch arguments, the fragment-major K/V
// cache and activation indexing, and the fused epilogues that run on a
// [rows][C] output tile.
#pragma once

#include <algorithm>
#include <type_traits>
#include <cmath>

#include "model.h"

namespace sdd {

enum Epi { EPI_QKV = 0, EPI_RESID = 1, EPI_SWIGLU = 2, EPI_LOGITS = 3 };

constexpr int kGemmThreads = 256;
constexpr int kXcds = 8;  // XCDs of the MI355X (32 CUs each); workgroups go to them round-robin by linear id
constexpr int kMaxPassRows = 64;  // rows per GEMM pass (TB <= 4 row tiles of 16)
constexpr int kMaxBlockRows = 65; // rows of one sequence in a verify call (gamma <= 64)
// Arrival counters of split column groups sit one 128-byte line apart: the groups of a launch finish
// together, and device-scope atomics on one line serialize.
constexpr int kCntStride = 32;

struct GemmArgs {
  const char* W;  // tiled weights
  int KT;         // k-tiles per row strip
  int G;          // column groups
  int N;          // valid output columns
  const char* X;  // activations, element type T, fragment-major (xfrag_index) with KT k-tiles
  int m0, M;      // rows of this pass
  int mp;         // padded row stride of per-row scratch
  int n_wg;
  int segc;       // virtual units per column group of the plan (cost-balanced shares; 0: equal)
  int share;      // longest share (units): the stored matrix holds share x n_wg slots
  float* part;    // partial tiles [n_wg][2][M][NG*16] (many-row kernel: partial or running sums by place)
  int32_t* err;   // the KV cache's sticky error word (bit3: a workgroup's internal hand-off gave up)
  int* cnt;       // arrival counter per column group (group g at cnt[g * kCntStride])
  const RowInfo* rows;
  // RMSNorm of the input rows: r_m = 1/sqrt(sum_g ss_in[g][m] / d_in + eps),
  // from per-column-group sums of squares written by the producer (NULL: none)
  const float* ss_in;
  int ss_groups, d_in;
  float eps;
  // EPI_QKV
  char* q_out;
  int hq, hkv, hd, qk_norm;
  const float* qn;
  const float* kn;
  const float* rope;
  int kv_ld;  // position stride of the K / V^T caches
  char* kc;
  char* vc;
  // EPI_RESID
  float* x;
  char* xa;
  int d;
  const float* g_next;
  float* ss_part;  // sums of squares of this GEMM's output rows per column group
  // EPI_SWIGLU
  char* ffh;
  int dff;
  // EPI_LOGITS
  float* logits;
  int V;
  float* amax_v;
  int* amax_i;
  // the forward's next GEMM (NULL: none), whose first k-steps a workgroup that
  // only contributed a partial loads into L2 before it ends
  const char* Wn;
  int KTn, Gn, ngn, nwg_n, cn;
  // many-row kernel: column tiles per column group; this launch's column blocks from cb0, row blocks, contributors per
  // tile, K segments (SumPlan), partial sums per tile, places of running sums per row block
  int ng, cb0, ncb, nrb, ksplit;
  int sg, sG, sn, sc, nslot, nch, compact;
};

template <typename T>
__device__ inline void mma_tile(const uint4& a, const uint4& b, f32x4& acc) {
  if constexpr (sizeof(T) == 2) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0,
                                                  0, 0);
  } else {
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, a.x), __builtin_bit_cast(float, b.x), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, a.y), __builtin_bit_cast(float, b.y), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, a.z), __builtin_bit_cast(float, b.z), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__builtin_bit_cast(float, a.w), __builtin_bit_cast(float, b.w), acc, 0, 0, 0);
  }
}

// bf16 K / V caches, fragment-major.  Per (sequence, KV head) a cache holds ld positions (a multiple of
// 64) as 32-position steps of 32 x HD elements.  A step is the list of 1 KB blocks that one attention step
// loads, one block per 16-byte-per-lane load, lane-major (lane l holds elements 8 l .. 8 l + 7), so every
// load reads whole cache lines:
//   K block b * HD/32 + kk, lane 16 g + rho: K[32 s + kv_row(rho, b)][32 kk + 8 g + e],  e = 0..7
//   V block db,             lane 16 g + rho: V[32 s + 8 g + e][16 db + rho],             e = 0..7
// kv_row(rho, b) is the position that K sub-tile b feeds to MFMA row rho; it leaves the scores of lane
// group g on positions 8 g .. 8 g + 7 of the step, the positions of that lane's V block entries.
__device__ inline int kv_row(int rho, int b) { return 8 * (rho / 4) + 4 * b + rho % 4; }
__device__ inline int64_t kfrag_index(int p, int d, int HD) {
  const int i = p % 32, rho = 4 * (i / 8) + i % 4, b = (i / 4) % 2;
  return (int64_t)(p / 32) * 32 * HD + (b * (HD / 32) + d / 32) * 512 + (16 * ((d % 32) / 8) + rho) * 8 + d % 8;
}
__device__ inline int64_t vfrag_index(int p, int d, int HD) {
  const int i = p % 32;
  return (int64_t)(p / 32) * 32 * HD + (d / 16) * 512 + (16 * (i / 8) + d % 16) * 8 + i % 8;
}

// GEMM inputs (the normed residual stream, the attention output, the FFN hidden rows) are fragment-major
// too: 1 KiB tiles of 16 rows x 32 bf16 (16 fp32) columns, what one fragment load of an MFMA B operand takes, tile
// (row tile, k-tile) at (row tile * KT + k-tile) KiB; inside a tile row after row, 64 bytes each, of which lane
// 16 g + rho loads the EPL = 16 / sizeof(T) columns from g EPL of row rho.
// Why: a fragment load of row-major activations touched 16 lines and used half of each, and every column group
// re-reads them; as one contiguous KiB the same loads take half the line requests.  Measured (Qwen3-32B width,
// 2 layers + LM head, before -> after): 1056-token recompute 4.43 -> 3.74 ms, 264-row verify 1.78 -> 1.59 ms, 99
// rows 981 -> 896 us; 33 rows (4 layers) 1098 -> 1072 us.  Rows inside a tile rather than the lanes' order, in which a
// tile of one row (a decode step, the 33rd row of a block) took 4 lines instead of 1: 33 rows 1074 -> 1068 us
// (Qwen2.5-7B width 707 -> 703), a 1-row step 604 -> 601 us (row-major: 599), with the row argmax's loads batched.
// Element index of (row, col); EPL consecutive columns from a multiple of EPL are contiguous (16 bytes).
template <typename T>
__device__ inline int64_t xfrag_index(int row, int col, int KT) {
  constexpr int EPL = 16 / (int)sizeof(T), KTL = 4 * EPL;
  return ((int64_t)(row / 16) * KT + col / KTL) * (64 * EPL) + row % 16 * KTL + col % KTL;
}
// Byte offset of this lane's 16 bytes of the fragment (row tile, k-tile 0) for a buffer load; lanes of rows at
// or past `rows` get an offset past every descriptor (rows pad to whole tiles; a padded row's lanes read zero
// without a memory access).
__device__ inline int xfrag_lane(int row_tile, int KT, int rows, int lane) {
  return 16 * row_tile + lane % 16 < rows ? row_tile * KT * 1024 + lane % 16 * 64 + lane / 16 * 16 : 0x7ffffff0;
}
// bytes of whole row tiles holding `rows` rows: the range of a descriptor over them
__device__ inline int xfrag_bytes(int rows, int KT) { return (rows + 15) / 16 * KT * 1024; }

template <typename T>
__device__ inline void store_t(char* base, int64_t idx, float v) {
  reinterpret_cast<T*>(base)[idx] = Elem<T>::from_f32(v);
}

// Eight consecutive columns (from a multiple of 8) of a row of a fragment-major GEMM input of K columns.
template <typename T>
__device__ inline void store_x8(char* base, int row, int col, int K, const float* y) {
  if constexpr (sizeof(T) == 2) {
    *reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(base) + xfrag_index<T>(row, col, K / 32)) =
        make_uint4(pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]), pack_bf16x2(y[4], y[5]), pack_bf16x2(y[6], y[7]));
  } else {
#pragma unroll
    for (int h = 0; h < 2; ++h)
      *reinterpret_cast<f32x4*>(reinterpret_cast<float*>(base) + xfrag_index<T>(row, col + 4 * h, K / 16)) =
          f32x4{y[4 * h], y[4 * h + 1], y[4 * h + 2], y[4 * h + 3]};
  }
}

// Stream-K bookkeeping (unit_start, unit_owner: model.h) is 32-bit unsigned
// arithmetic: 64-bit division is a long software sequence on this GPU.

// Loads into L2 the k-steps st0 .. st0 + NS - 1 that workgroup w of a GEMM launch
// (weights Wn stored in the order of their plan: workgroup w's i-th unit of
// ngn tiles at slot i * nwg + w) streams, wave `wave` (0..3) the k-steps that
// wave streams (local units wave + 4 st, st0 <= st < st0 + NS).  Called from a
// workgroup on XCD w mod 8: workgroups are dispatched to the XCDs round-robin,
// so the lines land in the L2 that serves them.  Plain (cached) loads whose
// values are consumed by an empty asm statement.
template <int NS = 3>
__device__ inline void prefetch_gemm_start(const char* Wn, int KTn, int Gn, int cn, int ngn, int nwg, int w_,
                                           int wave, int lane, int st0 = 0) {
  const uint32_t n = (uint32_t)nwg, w = (uint32_t)w_;
  const int nloc = (int)(unit_start(w + 1, KTn, Gn, cn, n) - unit_start(w, KTn, Gn, cn, n));
  const int nk = nloc > wave ? (nloc - wave + 3) / 4 : 0;  // this wave's units
  if (nk <= st0) return;
  const uint4* base = reinterpret_cast<const uint4*>(Wn) + (int64_t)w * ngn * kWave + lane;
  uint4 v[NS][8];  // unconditional loads (unit clamped to the wave's last, tile to the group's last)
#pragma unroll
  for (int st = 0; st < NS; ++st) {
    const int64_t i = wave + 4 * min(st0 + st, nk - 1);
#pragma unroll
    for (int nt = 0; nt < 8; ++nt) v[st][nt] = base[(i * nwg * ngn + min(nt, ngn - 1)) * kWave];
  }
  uint32_t x = 0;
#pragma unroll
  for (int st = 0; st < NS; ++st)
#pragma unroll
    for (int nt = 0; nt < 8; ++nt) x ^= v[st][nt].x ^ v[st][nt].w;
  asm volatile("" ::"v"(x));
}

// the same for the workgroup of the same index of the forward's next GEMM
__device__ inline void prefetch_next(const GemmArgs& a, int wave, int lane) {
  prefetch_gemm_start(a.Wn, a.KTn, a.Gn, a.cn, a.ngn, a.nwg_n, blockIdx.x, wave, lane);
}

// Epilogues run on the final [rows][C] tile of one column group (LDS, row
// stride C + 4), on the 4 waves of a workgroup.  Each wave owns rows wave,
// wave + 4, ... (R / 4 of them, the padded ones included: their results are
// computed and not stored), so the rows' work is straight-line code that the
// compiler interleaves.  A row's
// reductions run over its columns lane, lane + 64 and then across the wave,
// in an order that does not depend on the number of rows, so a row's result
// is the same whatever block it is verified in (floating-point contraction is
// off here, so that the compiler cannot fuse a row's operations differently in
// instantiations for different row counts).  Every global load a wave needs is
// issued before any of them is used.
// Sum over the n lanes of each aligned group of n (n in 1, 2, 4, 8, 16) by DPP row permutations, the same
// butterfly in every lane (the wave must be fully active).
template <int N>
__device__ inline float group_sum(float v) {
  if constexpr (N >= 2) v += dpp_f<kDppXor1>(v);
  if constexpr (N >= 4) v += dpp_f<kDppXor2>(v);
  if constexpr (N >= 8) v += dpp_f<kDppHalfMirror>(v);
  if constexpr (N >= 16) v += dpp_f<kDppMirror>(v);
  return v;
}

// The Q / K epilogue works on 8 consecutive dimensions per lane: LPR = C / 8
// lanes hold a row, RPI = 64 / LPR rows per pass, NIT passes over the wave's
// R / 4 rows (row wave + 4 j, j = it * RPI + lane / LPR).
template <int NG, int R>
struct QkvShape {
  static constexpr int C = NG * 16, RPW = R / 4, LPR = C / 8, RPI = kWave / LPR, NIT = (RPW + RPI - 1) / RPI;
};
// Global inputs of the Q / K epilogue of column group g (head g): the QK-norm
// gains of the lane's 8 dimensions and, for each pass, the RoPE (cos, sin) of
// those dimensions at its row's position (table [pos][C/2] of float2; dimension
// d uses entry d mod C/2), all loaded before any is used.
template <int NG, int R>
struct QkvPre {
  f32x4 gn[2];
  f32x4 cs[QkvShape<NG, R>::NIT][4];  // (cos, sin) pairs of dimensions d0 .. d0 + 7
};
template <int NG, int R>
__device__ inline void qkv_pre_load(const GemmArgs& a, int g, const RowInfo* ri_s, QkvPre<NG, R>& p) {
  using S = QkvShape<NG, R>;
  constexpr int C = S::C;
  if constexpr (C == 64 || C == 128) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
    const int rsub = lane / S::LPR, d0 = 8 * (lane % S::LPR);
    const bool is_q = g < a.hq;
    p.gn[0] = p.gn[1] = f32x4{1.f, 1.f, 1.f, 1.f};
    if (g >= a.hq + a.hkv) return;  // V head: no inputs
    if (a.qk_norm) {
      const float* gp = (is_q ? a.qn : a.kn) + d0;
      p.gn[0] = *reinterpret_cast<const f32x4*>(gp);
      p.gn[1] = *reinterpret_cast<const f32x4*>(gp + 4);
    }
#pragma unroll
    for (int it = 0; it < S::NIT; ++it) {
      const int mm = wave + 4 * min(it * S::RPI + rsub, S::RPW - 1);
      const RowInfo ri = ri_s[mm < a.M ? mm : 0];
      const f32x4* t = reinterpret_cast<const f32x4*>(a.rope + ((size_t)(ri.valid ? ri.pos : 0) * (C / 2) + d0 % (C / 2)) * 2);
#pragma unroll
      for (int k = 0; k < 4; ++k) p.cs[it][k] = t[k];
    }
  }
}

template <typename T, int NG, int R>
__device__ void epilogue_qkv(const GemmArgs& a, const float* tile, int g, const float* rsl, const RowInfo* ri_s) {
  // no contraction: every instantiation (row count) must round each row alike
#pragma clang fp contract(off)
  constexpr int C = NG * 16;  // == head_dim
  constexpr int CP = C + 4, RPW = R / 4;
  if constexpr (C == 64 || C == 128) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
    const int h = g;
    const bool is_q = h < a.hq, is_k = !is_q && h < a.hq + a.hkv;
    if (!is_q && !is_k) {
      // V head: lane = row, so that consecutive positions of a cached
      // dimension are written together (adjacent in both cache layouts)
      const int mm = lane;
      const bool ok = mm < a.M && ri_s[mm < a.M ? mm : 0].valid;
      const RowInfo ri = ri_s[mm < a.M ? mm : 0];
      const float r = rsl[mm < a.M ? mm : 0];
      const int64_t head = (int64_t)ri.seq * a.hkv + (h - a.hq - a.hkv);
      constexpr int DPW = C / 4;  // dimensions per wave
#pragma unroll 8
      for (int dd = 0; dd < DPW; ++dd) {
        const int dim = wave * DPW + dd;
        const float y = tile[(mm < R ? mm : 0) * CP + dim] * r;
        if (ok) {
          if constexpr (sizeof(T) == 2)
            store_t<T>(a.vc, head * a.kv_ld * C + vfrag_index(ri.pos, dim, C), y);
          else
            store_t<T>(a.vc, (head * C + dim) * a.kv_ld + ri.pos, y);  // fp32: V^T rows
        }
      }
      return;
    }
    using S = QkvShape<NG, R>;
    QkvPre<NG, R> pp;
    qkv_pre_load<NG, R>(a, g, ri_s, pp);
    const int rsub = lane / S::LPR, d0 = 8 * (lane % S::LPR);
    const bool lo = d0 < C / 2;  // the rotation pairs dimension d with d + C/2
#pragma unroll
    for (int it = 0; it < S::NIT; ++it) {
      const int j = it * S::RPI + rsub, mm = wave + 4 * j;
      const int mt = wave + 4 * min(j, RPW - 1);  // tile row (a valid one for the last pass's spare lanes)
      const float r = rsl[mt < a.M ? mt : 0];
      const f32x4 t0 = *reinterpret_cast<const f32x4*>(&tile[mt * CP + d0]);
      const f32x4 t1 = *reinterpret_cast<const f32x4*>(&tile[mt * CP + d0 + 4]);
      float y[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        y[e] = t0[e] * r;
        y[4 + e] = t1[e] * r;
      }
      if (a.qk_norm) {
        float ss = 0.f;
#pragma unroll
        for (int e = 0; e < 8; ++e) ss += y[e] * y[e];
        ss = group_sum<S::LPR>(ss);
        const float inv = 1.f / sqrtf(ss / (float)C + a.eps);
#pragma unroll
        for (int e = 0; e < 8; ++e) y[e] *= inv * (e < 4 ? pp.gn[0][e] : pp.gn[1][e - 4]);
      }
      // the partner dimensions (d +- C/2) sit LPR / 2 lanes away in the row's lane group
      float o[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        if constexpr (C == 128)
          o[e] = dpp_f<kDppRor8>(y[e]);
        else
          o[e] = __shfl_xor(y[e], S::LPR / 2);
      }
      float z[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float c = pp.cs[it][e / 2][2 * (e % 2)], sn = pp.cs[it][e / 2][2 * (e % 2) + 1];
        z[e] = lo ? y[e] * c - o[e] * sn : y[e] * c + o[e] * sn;
      }
      if (j < RPW && mm < a.M && ri_s[mm].valid) {
        const RowInfo ri = ri_s[mm];
        int64_t off;  // element offset of the lane's 8 dimensions (16-byte aligned, contiguous)
        char* base;
        if (is_q) {
          base = a.q_out;
          off = ((int64_t)(a.m0 + mm) * a.hq + h) * C + d0;
        } else if constexpr (sizeof(T) == 2) {
          base = a.kc;
          off = ((int64_t)ri.seq * a.hkv + (h - a.hq)) * a.kv_ld * C + kfrag_index(ri.pos, d0, C);
        } else {
          base = a.kc;
          off = (((int64_t)ri.seq * a.hkv + (h - a.hq)) * a.kv_ld + ri.pos) * C + d0;  // fp32: [pos][hd]
        }
        if constexpr (sizeof(T) == 2) {
          *reinterpret_cast<uint4*>(reinterpret_cast<uint16_t*>(base) + off) =
              make_uint4(pack_bf16x2(z[0], z[1]), pack_bf16x2(z[2], z[3]), pack_bf16x2(z[4], z[5]), pack_bf16x2(z[6], z[7]));
        } else {
          float* dst = reinterpret_cast<float*>(base) + off;
          *reinterpret_cast<f32x4*>(dst) = f32x4{z[0], z[1], z[2], z[3]};
          *reinterpret_cast<f32x4*>(dst + 4) = f32x4{z[4], z[5], z[6], z[7]};
        }
      }
    }
  }
}


// Residual epilogue, 8 consecutive columns per lane: LPR = C / 8 lanes hold a row (16-byte loads and
// stores), RPI = 64 / LPR rows per pass; a row's sum of squares adds the lane's 8 squares in column order,
// then the LPR lanes by a fixed butterfly.
template <typename T, int NG, int R>
__device__ void epilogue_resid(const GemmArgs& a, const float* tile, int g) {
  // no contraction: every instantiation (row count) must round each row alike
#pragma clang fp contract(off)
  constexpr int C = NG * 16, CP = C + 4, RPW = R / 4;
  constexpr int LPR = C / 8, RPI = kWave / LPR, NIT = (RPW + RPI - 1) / RPI;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int rsub = lane / LPR, c0 = 8 * (lane % LPR);
  const int64_t n0 = (int64_t)g * C + c0;
  const f32x4 gv0 = *reinterpret_cast<const f32x4*>(a.g_next + n0), gv1 = *reinterpret_cast<const f32x4*>(a.g_next + n0 + 4);
  // every pass's residual loads first (padded rows read row 0)
  f32x4 xa0[NIT], xa1[NIT];
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int j = it * RPI + rsub, mm = wave + 4 * j;
    const int mc = (j < RPW && mm < a.M) ? mm : 0;
    const float* xr = a.x + (int64_t)(a.m0 + mc) * a.d + n0;
    xa0[it] = *reinterpret_cast<const f32x4*>(xr);
    xa1[it] = *reinterpret_cast<const f32x4*>(xr + 4);
  }
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int j = it * RPI + rsub, mm = wave + 4 * j;
    const int mt = wave + 4 * min(j, RPW - 1);  // tile row (a valid one for the last pass's spare lanes)
    const f32x4 t0 = *reinterpret_cast<const f32x4*>(&tile[mt * CP + c0]);
    const f32x4 t1 = *reinterpret_cast<const f32x4*>(&tile[mt * CP + c0 + 4]);
    float xv[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      xv[e] = xa0[it][e] + t0[e];
      xv[4 + e] = xa1[it][e] + t1[e];
    }
    float ss = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) ss += xv[e] * xv[e];
    ss = group_sum<LPR>(ss);
    if (j < RPW && mm < a.M) {
      const int m = a.m0 + mm;
      float* xr = a.x + (int64_t)m * a.d + n0;
      *reinterpret_cast<f32x4*>(xr) = f32x4{xv[0], xv[1], xv[2], xv[3]};
      *reinterpret_cast<f32x4*>(xr + 4) = f32x4{xv[4], xv[5], xv[6], xv[7]};
      float y[8];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        y[e] = xv[e] * gv0[e];
        y[4 + e] = xv[4 + e] * gv1[e];
      }
      store_x8<T>(a.xa, m, (int)n0, a.d, y);
      if (lane % LPR == 0) a.ss_part[(int64_t)g * a.mp + m] = ss;
    }
  }
}

// SwiGLU epilogue: the group's C columns are P = NG / 2 pairs of 16 gate and 16 up columns, i.e. P * 16
// hidden outputs per row; a lane computes 8 consecutive ones (LPR = NG lanes per row, RPI = 64 / LPR rows
// per pass) and stores them with one 16-byte store.
template <typename T, int NG, int R>
__device__ void epilogue_swiglu(const GemmArgs& a, const float* tile, int g, const float* rsl) {
  // no contraction: every instantiation (row count) must round each row alike
#pragma clang fp contract(off)
  constexpr int C = NG * 16, CP = C + 4, P = NG / 2, RPW = R / 4;
  constexpr int LPR = P * 2, RPI = kWave / LPR, NIT = (RPW + RPI - 1) / RPI;
  static_assert(NG % 2 == 0, "gate/up groups hold whole pairs");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int rsub = lane / LPR, h0 = 8 * (lane % LPR);      // first hidden column of the lane
  const int cg = (h0 / 16) * 32 + h0 % 16, cu = cg + 16;  // its gate and up tile columns
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int j = it * RPI + rsub, mm = wave + 4 * j;
    const int mt = wave + 4 * min(j, RPW - 1);
    const float r = rsl[mt];
    const f32x4 g0 = *reinterpret_cast<const f32x4*>(&tile[mt * CP + cg]);
    const f32x4 g1 = *reinterpret_cast<const f32x4*>(&tile[mt * CP + cg + 4]);
    const f32x4 u0 = *reinterpret_cast<const f32x4*>(&tile[mt * CP + cu]);
    const f32x4 u1 = *reinterpret_cast<const f32x4*>(&tile[mt * CP + cu + 4]);
    float hv[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float gt = (e < 4 ? g0[e] : g1[e - 4]) * r;
      const float up = (e < 4 ? u0[e] : u1[e - 4]) * r;
      hv[e] = gt / (1.f + expf(-gt)) * up;
    }
    if (j < RPW && mm < a.M) {
      store_x8<T>(a.ffh, a.m0 + mm, g * P * 16 + h0, a.dff, hv);
    }
  }
}

__device__ inline bool arg_better(float v2, int i2, float v1, int i1) {
  if (i2 < 0 || v2 != v2) return false;
  if (i1 < 0) return true;
  return v2 > v1 || (v2 == v1 && i2 < i1);
}

// Best (value, lowest index) over the n lanes of each aligned group of n (n in 1, 2, 4, 8, 16), left in
// every lane of the group; the combine is associative and commutative, so the butterfly's order is free.
template <int N>
__device__ inline void group_argmax(float& bv, int& bi) {
  auto step = [&](auto ctrl) {
    constexpr int CTRL = decltype(ctrl)::value;
    const float v2 = dpp_f<CTRL>(bv);
    const int i2 = dpp_i<CTRL>(bi);
    if (arg_better(v2, i2, bv, bi)) {
      bv = v2;
      bi = i2;
    }
  };
  if constexpr (N >= 2) step(std::integral_constant<int, kDppXor1>{});
  if constexpr (N >= 4) step(std::integral_constant<int, kDppXor2>{});
  if constexpr (N >= 8) step(std::integral_constant<int, kDppHalfMirror>{});
  if constexpr (N >= 16) step(std::integral_constant<int, kDppMirror>{});
}

// LM-head epilogue: fp32 logits of the valid rows and each row's best (value, index) over the group's
// columns below V.  A lane takes 8 consecutive columns (LPR = C / 8 lanes per row, RPI = 64 / LPR rows per
// pass): 16-byte stores where V keeps rows 16-byte aligned and the 8 columns are all below V.
template <int NG, int R>
__device__ void epilogue_logits(const GemmArgs& a, const float* tile, int g, const float* rsl, const RowInfo* ri_s) {
  // no contraction: every instantiation (row count) must round each row alike
#pragma clang fp contract(off)
  constexpr int C = NG * 16, CP = C + 4, RPW = R / 4;
  constexpr int LPR = C / 8, RPI = kWave / LPR, NIT = (RPW + RPI - 1) / RPI;
  static_assert(LPR <= 16, "a row's lanes must lie in one DPP row");
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int rsub = lane / LPR, c0 = 8 * (lane % LPR), n0 = g * C + c0;
  const bool vec = (a.V & 3) == 0 && n0 + 8 <= a.V;
  float bv[NIT];
  int bi[NIT];
#pragma unroll
  for (int it = 0; it < NIT; ++it) {
    const int j = it * RPI + rsub, mm = wave + 4 * j;
    const int mt = wave + 4 * min(j, RPW - 1);
    const float r = rsl[mt < a.M ? mt : 0];
    const f32x4 t0 = *reinterpret_cast<const f32x4*>(&tile[mt * CP + c0]);
    const f32x4 t1 = *reinterpret_cast<const f32x4*>(&tile[mt * CP + c0 + 4]);
    float v[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] = t0[e] * r;
      v[4 + e] = t1[e] * r;
    }
    bv[it] = -INFINITY;
    bi[it] = -1;
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (n0 + e < a.V && arg_better(v[e], n0 + e, bv[it], bi[it])) {
        bv[it] = v[e];
        bi[it] = n0 + e;
      }
    if (j < RPW && mm < a.M && ri_s[mm].valid) {
      float* lr = a.logits + (int64_t)(a.m0 + mm) * a.V + n0;
      if (vec) {
        *reinterpret_cast<f32x4*>(lr) = f32x4{v[0], v[1], v[2], v[3]};
        *reinterpret_cast<f32x4*>(lr + 4) = f32x4{v[4], v[5], v[6], v[7]};
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (n0 + e < a.V) lr[e] = v[e];
      }
    }
    group_argmax<LPR>(bv[it], bi[it]);
  }
  // one lane per row, so the rows' candidates take two store instructions, not
  // two per row: with the next segment's loads in flight, a wave's outstanding
  // memory operations would otherwise exceed the 63 the counter holds, and
  // issue would stall until those loads land
  float av = 0.f;
  int ai = -1;
#pragma unroll
  for (int it = 0; it < NIT; ++it)
#pragma unroll
    for (int q = 0; q < RPI; ++q) {
      const int j = it * RPI + q;
      if (j < RPW) {
        const float v2 = lane_f(bv[it], q * LPR);
        const int i2 = __builtin_amdgcn_readlane(bi[it], q * LPR);
        if (lane == j) {
          av = v2;
          ai = i2;
        }
      }
    }
  const int mm = wave + 4 * lane;
  if (lane < RPW && mm < a.M) {
    a.amax_v[(int64_t)g * a.mp + a.m0 + mm] = av;
    a.amax_i[(int64_t)g * a.mp + a.m0 + mm] = ai;
  }
}

// A 16-byte-per-lane direct-to-LDS buffer load: lane l's 16 bytes at `lds` + 16 l.
template <int AUX>
__device__ inline void load_lds16(__amdgpu_buffer_rsrc_t rs, void* lds, int voffset, int soffset) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void*)(lds), 16, voffset, soffset, 0,
                                           AUX);
}
// s_waitcnt operand: vector memory count <= n (0..63), the other counters unconstrained (gfx9 encoding:
// vmcnt in bits 3:0 and 15:14, expcnt 6:4, lgkmcnt 11:8)
constexpr int kWaitLgkm0 = 0xC07F;  // every LDS operation, nothing else
constexpr int wait_vmcnt(int n) { return (n & 0xF) | ((n >> 4) << 14) | (0x7 << 4) | (0xF << 8); }
// A workgroup barrier without a memory fence (a fence would wait for every load in flight); nothing is scheduled
// across it.
__device__ inline void phase_barrier() {
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
  __atomic_signal_fence(__ATOMIC_SEQ_CST);
}

// The order of a row's sums over K in the many-row kernel.  The K x column-group units of a matrix, G groups of `tiles`
// column tiles each, are shared out among n owners (unit_start with c virtual units); inside a group every share is one
// segment: the k-steps of a segment are added one after another, from zero, and the segments' sums in order.  It is a
// property of the matrix alone: a row's result does not depend on the rows, tiles and splits of the launch it is in.
// The groups and shares are those of the storage plan, or equal shares of pairs of 8-tile groups (gate/up and the LM
// head, whose tiles are mostly one segment).
struct SumPlan {
  int tiles, G, n, c;
  int nseg;      // segments per group (uniform), or a bound
  bool uniform;  // every group has the same segments
};
SumPlan sum_plan(const MatPlan& mp, bool pairs);
// Many-row GEMM (tiles.hip): bf16 weights, column groups of 8 or 4 tiles, rows [0, a.M); fused epilogue `epi`.  A plan
// fixes the tile (128 wc columns x 128 rtw / wc rows per workgroup), the number of column and row blocks and the
// workgroups that share a tile's segments.
struct TilePlan {
  int wc, rtw;            // wave columns (1 or 2) of the workgroup's 8 waves, row tiles per wave
  int ncb, nrb;           // column blocks, row blocks
  int per, ksplit;        // column blocks per launch, workgroups per tile
  int slots;              // partial sums per split tile
  bool compact;           // one running sum per segment boundary of the matrix (else one per 64 columns)
  SumPlan sums;
  double us;              // estimated time
};
// Best plan for M rows of a matrix of plan `mp` (pairs: gate/up or LM head) on n_cu compute units, with `part_bytes` for
// partial and running sums and arrival counters for max_split tiles.
TilePlan plan_tiles(const MatPlan& mp, bool pairs, int M, int n_cu, size_t part_bytes, int64_t max_split);
// Index arithmetic of a many-row launch (host and device: the tests replay it on the CPU).
// Launch fields of column blocks from cb0 on.
inline void tile_launch(GemmArgs& a, const TilePlan& p, int cb0) {
  a.cb0 = cb0;
  a.ncb = std::min(p.per, p.ncb - cb0);
  a.nrb = p.nrb;
  a.ksplit = p.ksplit;
  a.sg = p.sums.tiles;
  a.sG = p.sums.G;
  a.sn = p.sums.n;
  a.sc = p.sums.c;
  a.nslot = p.slots;
  a.nch = a.ncb * 2 * p.wc;
  a.compact = p.compact;
}
inline int tile_grid(const GemmArgs& a) { return kXcds * (int)ceil_div((int64_t)a.ncb * a.ksplit, kXcds) * a.nrb; }
// A workgroup's item: column block (of the launch and of the matrix), row block, contributor; cbl < 0: none.
// One XCD's workgroups are 8 apart; the row blocks of a column block run there next to each other.
struct TileItem {
  int cbl, cb, rb, sp;
};
__host__ __device__ inline TileItem tile_item(const GemmArgs& a, int block, int S) {
  const int slot = block / kXcds, cs = block % kXcds + kXcds * (slot / a.nrb);
  return cs < a.ncb * S ? TileItem{cs / S, a.cb0 + cs / S, slot % a.nrb, cs % S} : TileItem{-1, 0, 0, 0};
}
// First unit of the sum group of column tile ct (past the matrix: of the last group).
__host__ __device__ inline uint32_t sum_base(const GemmArgs& a, int ct) {
  const int g = ct / a.sg;
  return (uint32_t)(g < a.sG ? g : a.sG - 1) * (uint32_t)a.KT;
}
__host__ __device__ inline int sum_owner(const GemmArgs& a, uint32_t u) {
  return unit_owner(u, (uint32_t)a.KT, (uint32_t)a.sG, (uint32_t)a.sc, (uint32_t)a.sn);
}
// k-step (of the group with first unit `base`) at which owner o's share starts
__host__ __device__ inline int sum_start(const GemmArgs& a, uint32_t base, int o) {
  return (int)(unit_start((uint32_t)o, (uint32_t)a.KT, (uint32_t)a.sG, (uint32_t)a.sc, (uint32_t)a.sn) - base);
}
// Contributor sp's part of a split tile at column tile ct: segments from seg0, k-steps [kb, ke).  The first contributor
// adds its n0 segments up, so a tile's partial sums take nseg - n0 + 1 slots (part_slot).
struct TileRange {
  int kb, ke, own0, nseg, seg0, n0, E;  // own0: owner of the group's first segment; E: contributors (sp >= E has none)
};
__host__ __device__ inline TileRange tile_range(const GemmArgs& a, int ct, int sp) {
  TileRange r{0, a.KT, 0, 1, 0, 1, 1};
  const uint32_t u0 = sum_base(a, ct);
  r.own0 = sum_owner(a, u0);
  r.nseg = sum_owner(a, u0 + (uint32_t)a.KT - 1) - r.own0 + 1;
  r.E = r.nseg < a.ksplit ? r.nseg : a.ksplit;
  r.n0 = (r.nseg + r.E - 1) / r.E;
  if (sp >= r.E) return r;
  const int s1 = (r.nseg * (sp + 1) + r.E - 1) / r.E;
  r.seg0 = (r.nseg * sp + r.E - 1) / r.E;
  if (r.seg0 > 0) r.kb = sum_start(a, u0, r.own0 + r.seg0);
  if (s1 < r.nseg) r.ke = sum_start(a, u0, r.own0 + s1);
  return r;
}
__host__ __device__ inline int part_slot(const TileRange& r, int seg) { return seg < r.n0 ? 0 : seg - r.n0 + 1; }
// Byte offset of the running sums of four column tiles from ct (a multiple of four) of row block rb, RT row tiles of 4
// KiB: one place per 64 columns and row block, or per boundary where a group has at most one (own: the owner before it).
__host__ __device__ inline int chain_place(const GemmArgs& a, int rb, int ct, int own, int CG, int RT) {
  const int q = a.sg / 4;
  return (a.compact ? (rb * a.sn + own) * q + ct / 4 % q : rb * a.nch + ct / 4 - a.cb0 * CG / 4) * RT * 4096;
}
// Byte offset of partial sums `slot` of row tile rt and wave column wcol (8 KiB), for tile rb * ncb + cbl.
__host__ __device__ inline int part_place(const GemmArgs& a, int tile, int slot, int rt, int wcol, int RT, int WC) {
  return (((tile * a.nslot + slot) * RT + rt) * WC + wcol) * 8192;
}
// Where the matrix's streaming plan stores k-step k of column group g: unit g KT + k of owner o, at slot
// (g KT + k - start(o)) n_wg + o.  Follows one group's owners as k rises.
struct TileTrk {
  int g, o, kend, base;  // group, owner, first k-step past its share, slot of k-step 0
};
__host__ __device__ inline void trk_set(const GemmArgs& a, TileTrk& t, int o) {
  const uint32_t KT = (uint32_t)a.KT, u = (uint32_t)t.g * KT;
  const uint32_t us = unit_start((uint32_t)o, KT, (uint32_t)a.G, (uint32_t)a.segc, (uint32_t)a.n_wg);
  const uint32_t ue = unit_start((uint32_t)o + 1, KT, (uint32_t)a.G, (uint32_t)a.segc, (uint32_t)a.n_wg);
  t.o = o;
  t.kend = (int)(ue - u);
  t.base = ((int)u - (int)us) * a.n_wg + o;
}

// ---- attention (bf16) -----------------------------------------------------------------------------------
constexpr int kAttnWaves = 8;  // waves of a workgroup; wave w takes the 32-position steps w, w + kAttnWaves, ...

// Combining the waves' partial (max, sum, O) of 16 queries, published to LDS, in wave order.  First, for query q: the common
// max, each wave's rescale factor and the total sum.
__device__ inline void attn_factors(const float (*s_m)[16], const float (*s_l)[16], float (*s_f)[16], float* s_L, int q) {
  float M = -INFINITY;
#pragma unroll
  for (int w = 0; w < kAttnWaves; ++w) M = fmaxf(M, s_m[w][q]);
  float L = 0.f;
#pragma unroll
  for (int w = 0; w < kAttnWaves; ++w) {
    const float ms = s_m[w][q];
    const float f = (M == -INFINITY || ms == -INFINITY) ? 0.f : __expf(ms - M);
    s_f[w][q] = f;
    L += s_l[w][q] * f;
  }
  s_L[q] = L;
}
// Then (a barrier later) the outputs: put(query, dim, y) receives four consecutive dimensions.
template <int HD, typename Put>
__device__ inline void attn_combine(const float (*s_o)[16][HD + 4], const float (*s_f)[16], const float* s_L, Put put) {
  for (int e = threadIdx.x; e < 16 * HD / 4; e += kAttnWaves * kWave) {
    const int q = e / (HD / 4), dim = 4 * (e % (HD / 4));
    f32x4 O = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kAttnWaves; ++w) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(&s_o[w][q][dim]);
      const float f = s_f[w][q];
#pragma unroll
      for (int i = 0; i < 4; ++i) O[i] += v[i] * f;
    }
    const float L = s_L[q];
    float y[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) y[i] = L > 0.f ? O[i] / L : 0.f;
    put(q, dim, y);
  }
}

// Attention of a prefill chunk (attn_prefill.hip, bf16): R rows of one sequence, rows[0, R), over its cache.
struct AttnPrefillArgs {
  const uint16_t* q;   // [rows][hq][head_dim]
  const uint16_t* kc;  // layer base, per (seq, hkv) ld x head_dim elements, fragment-major
  const uint16_t* vc;
  uint16_t* out;       // rows of hq * head_dim columns, fragment-major
  const RowInfo* rows;
  int R, hq, hkv, grp, ld;
  float scale;
  int qblocks, heads_apart;  // set by the launch
};
constexpr int kAttnPrefillQueries = 48;  // query vectors per workgroup
int launch_attention_prefill(AttnPrefillArgs a, int head_dim, hipStream_t st);
int launch_gemm_tiles(const TilePlan& p, int epi, GemmArgs a, hipStream_t st);

}  // namespace sdd
