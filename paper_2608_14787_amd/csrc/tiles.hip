// Many-row GEMM on gfx950: the projections over more than 64 rows (prefill chunks, the full-recompute verifier,
// the blocks of several sequences verified together; Sec. 3.1 per sequence).
//
// At a few hundred rows and more a projection is bound by the matrix cores and by what feeds them: every
// fragment a wave multiplies comes through LDS, so the LDS reads of one k-step have to hide behind the MFMAs
// of another.  Design:
//  - a workgroup of 8 waves computes an output tile of 16 CG columns x 16 RT rows: WC x WR waves, each NTW column
//    tiles x RTW row tiles of accumulators.  Weights and activations are both stored as MFMA fragments of one
//    contiguous KiB, so a k-step is CG + RT direct-to-LDS loads (no registers, no bank conflicts), RS stages deep;
//  - waves 0-3 and 4-7 (one of each on every SIMD) run half a k-step apart: while one half reads its fragments from
//    LDS and issues loads, the other half multiplies, and they swap at a workgroup barrier.  With all 8 waves in
//    step, every SIMD idled through the LDS reads of each k-step;
//  - the epilogues run on the accumulators in registers (lane l: row l % 16, four consecutive columns of each
//    tile), so no staging in LDS and no barrier follows the k-loop.  A wave holds 128 whole columns, which is what
//    the per-head norm, the rotation (partner dimension in the same lane) and the per-group statistics need;
//  - a launch is (column block, row block, k-split) items, one per workgroup.  The row blocks of one column block
//    run on one XCD next to each other, so its L2 serves the weights to all but the first of them.  Where the
//    tiles leave compute units idle, K is split: partials go through 16-byte device-coherent stores and are added
//    in split order, the tile's row tiles shared out among its contributors.  A row's sums depend on its launch's
//    plan but not on the other rows' values.
//  - tiles that fill the chip several times and leave a few over pay a whole round for those few: the column blocks of
//    the whole rounds run unsplit, those left over follow in the same launch with K split over all compute units.
// Measured (Qwen3-32B width, with the chunked launches of 288 rows and 4 loading waves this kernel replaced): gate/up
// over 1024 rows 4 x 148 -> 498 us (1.08 PFLOP/s; the library's product at this size 0.99), over 264 rows 186 -> 151;
// down 125 -> 89, qkv 76 -> 58, o_proj 45 -> 47, LM head 546 -> 463 us.  What bounds it: a k-step of 8 + RTW fragment
// reads and 8 RTW MFMAs per wave takes 0.33 us + 14.2 ns per MFMA, about 1.6 times the matrix cores' own time at RTW 4.
#include "gemm.h"

namespace sdd {
namespace {

constexpr int kTileThreads = 512;
constexpr int kTilePolls = 1 << 11;  // polls for a split item's other contributors (about 2 ms)
constexpr size_t kTileRing = 148 * 1024;  // LDS for the ring (the rest: row scales and their partial sums)

// A wave's fragments of one k-step from LDS: 8 weight tiles from address aw and RTW row tiles from ax (this lane's 16
// bytes of the first; tiles 1 KiB apart).  The reads and their wait are one asm block: the compiler cannot tell them
// from reads of the slots the wave's own direct-to-LDS loads are still filling and would wait for all of those loads.
template <int RTW>
__device__ inline void lds_read_frags(u32x4* w, u32x4* x, uint32_t aw, uint32_t ax) {
  static_assert(RTW >= 1 && RTW <= 5, "row tiles per wave");
  if constexpr (RTW == 1) {
    asm volatile(
        "ds_read_b128 %0, %9\n\t"
        "ds_read_b128 %1, %9 offset:1024\n\t"
        "ds_read_b128 %2, %9 offset:2048\n\t"
        "ds_read_b128 %3, %9 offset:3072\n\t"
        "ds_read_b128 %4, %9 offset:4096\n\t"
        "ds_read_b128 %5, %9 offset:5120\n\t"
        "ds_read_b128 %6, %9 offset:6144\n\t"
        "ds_read_b128 %7, %9 offset:7168\n\t"
        "ds_read_b128 %8, %10\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]),
          "=&v"(w[4]), "=&v"(w[5]), "=&v"(w[6]), "=&v"(w[7]),
          "=&v"(x[0])
        : "v"(aw), "v"(ax)
        : "memory");
  } else if constexpr (RTW == 2) {
    asm volatile(
        "ds_read_b128 %0, %10\n\t"
        "ds_read_b128 %1, %10 offset:1024\n\t"
        "ds_read_b128 %2, %10 offset:2048\n\t"
        "ds_read_b128 %3, %10 offset:3072\n\t"
        "ds_read_b128 %4, %10 offset:4096\n\t"
        "ds_read_b128 %5, %10 offset:5120\n\t"
        "ds_read_b128 %6, %10 offset:6144\n\t"
        "ds_read_b128 %7, %10 offset:7168\n\t"
        "ds_read_b128 %8, %11\n\t"
        "ds_read_b128 %9, %11 offset:1024\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]),
          "=&v"(w[4]), "=&v"(w[5]), "=&v"(w[6]), "=&v"(w[7]),
          "=&v"(x[0]), "=&v"(x[1])
        : "v"(aw), "v"(ax)
        : "memory");
  } else if constexpr (RTW == 3) {
    asm volatile(
        "ds_read_b128 %0, %11\n\t"
        "ds_read_b128 %1, %11 offset:1024\n\t"
        "ds_read_b128 %2, %11 offset:2048\n\t"
        "ds_read_b128 %3, %11 offset:3072\n\t"
        "ds_read_b128 %4, %11 offset:4096\n\t"
        "ds_read_b128 %5, %11 offset:5120\n\t"
        "ds_read_b128 %6, %11 offset:6144\n\t"
        "ds_read_b128 %7, %11 offset:7168\n\t"
        "ds_read_b128 %8, %12\n\t"
        "ds_read_b128 %9, %12 offset:1024\n\t"
        "ds_read_b128 %10, %12 offset:2048\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]),
          "=&v"(w[4]), "=&v"(w[5]), "=&v"(w[6]), "=&v"(w[7]),
          "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2])
        : "v"(aw), "v"(ax)
        : "memory");
  } else if constexpr (RTW == 4) {
    asm volatile(
        "ds_read_b128 %0, %12\n\t"
        "ds_read_b128 %1, %12 offset:1024\n\t"
        "ds_read_b128 %2, %12 offset:2048\n\t"
        "ds_read_b128 %3, %12 offset:3072\n\t"
        "ds_read_b128 %4, %12 offset:4096\n\t"
        "ds_read_b128 %5, %12 offset:5120\n\t"
        "ds_read_b128 %6, %12 offset:6144\n\t"
        "ds_read_b128 %7, %12 offset:7168\n\t"
        "ds_read_b128 %8, %13\n\t"
        "ds_read_b128 %9, %13 offset:1024\n\t"
        "ds_read_b128 %10, %13 offset:2048\n\t"
        "ds_read_b128 %11, %13 offset:3072\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]),
          "=&v"(w[4]), "=&v"(w[5]), "=&v"(w[6]), "=&v"(w[7]),
          "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3])
        : "v"(aw), "v"(ax)
        : "memory");
  } else {
    asm volatile(
        "ds_read_b128 %0, %13\n\t"
        "ds_read_b128 %1, %13 offset:1024\n\t"
        "ds_read_b128 %2, %13 offset:2048\n\t"
        "ds_read_b128 %3, %13 offset:3072\n\t"
        "ds_read_b128 %4, %13 offset:4096\n\t"
        "ds_read_b128 %5, %13 offset:5120\n\t"
        "ds_read_b128 %6, %13 offset:6144\n\t"
        "ds_read_b128 %7, %13 offset:7168\n\t"
        "ds_read_b128 %8, %14\n\t"
        "ds_read_b128 %9, %14 offset:1024\n\t"
        "ds_read_b128 %10, %14 offset:2048\n\t"
        "ds_read_b128 %11, %14 offset:3072\n\t"
        "ds_read_b128 %12, %14 offset:4096\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]),
          "=&v"(w[4]), "=&v"(w[5]), "=&v"(w[6]), "=&v"(w[7]),
          "=&v"(x[0]), "=&v"(x[1]), "=&v"(x[2]), "=&v"(x[3]),
          "=&v"(x[4])
        : "v"(aw), "v"(ax)
        : "memory");
  }
}
// ---- epilogues of one row tile in the accumulator layout --------------------------------------------------
// v[nt][e]: row `m`, column 16 (ct + nt) + 4 (lane / 16) + e.  No contraction: a row rounds alike everywhere.

template <int NT>
__device__ inline void tile_resid(const GemmArgs& a, const f32x4* v, int ct, int m, bool ok, int lane) {
#pragma clang fp contract(off)
  const int c0 = 16 * ct + 4 * (lane / 16), mr = ok ? m : 0;
  float* xr = a.x + (int64_t)mr * a.d + c0;
  f32x4 xo[NT], gv[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    xo[nt] = *reinterpret_cast<const f32x4*>(xr + 16 * nt);
    gv[nt] = *reinterpret_cast<const f32x4*>(a.g_next + c0 + 16 * nt);
  }
  float ss = 0.f;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      xo[nt][e] += v[nt][e];
      ss += xo[nt][e] * xo[nt][e];
    }
  ss = xor16_op(ss, [](float x, float y) { return x + y; });
  ss = xor32_op(ss, [](float x, float y) { return x + y; });
  if (!ok) return;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    *reinterpret_cast<f32x4*>(xr + 16 * nt) = xo[nt];
    *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.xa) + xfrag_index<uint16_t>(m, c0 + 16 * nt, a.d / 32)) =
        make_uint2(pack_bf16x2(xo[nt][0] * gv[nt][0], xo[nt][1] * gv[nt][1]),
                   pack_bf16x2(xo[nt][2] * gv[nt][2], xo[nt][3] * gv[nt][3]));
  }
  if (lane < 16) a.ss_part[(int64_t)(ct / NT) * a.mp + m] = ss;
}

template <int NT>
__device__ inline void tile_swiglu(const GemmArgs& a, const f32x4* v, int ct, int m, bool ok, float r, int lane) {
#pragma clang fp contract(off)
  if (!ok) return;
#pragma unroll
  for (int t = 0; t < NT / 2; ++t) {
    float hv[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float gt = v[2 * t][e] * r, up = v[2 * t + 1][e] * r;
      hv[e] = gt / (1.f + expf(-gt)) * up;
    }
    *reinterpret_cast<uint2*>(reinterpret_cast<uint16_t*>(a.ffh) +
                              xfrag_index<uint16_t>(m, 8 * ct + 16 * t + 4 * (lane / 16), a.dff / 32)) =
        make_uint2(pack_bf16x2(hv[0], hv[1]), pack_bf16x2(hv[2], hv[3]));
  }
}

template <int NT>
__device__ inline void tile_logits(const GemmArgs& a, const f32x4* v, int ct, int m, bool ok, bool valid, float r, int lane) {
#pragma clang fp contract(off)
  float bv = -INFINITY;
  int bi = -1;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int n0 = 16 * (ct + nt) + 4 * (lane / 16);
    float x[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) x[e] = v[nt][e] * r;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (n0 + e < a.V && arg_better(x[e], n0 + e, bv, bi)) {
        bv = x[e];
        bi = n0 + e;
      }
    if (ok && valid) {
      float* lr = a.logits + (int64_t)m * a.V + n0;
      if ((a.V & 3) == 0 && n0 + 4 <= a.V) {
        *reinterpret_cast<f32x4*>(lr) = f32x4{x[0], x[1], x[2], x[3]};
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (n0 + e < a.V) lr[e] = x[e];
      }
    }
  }
#pragma unroll
  for (int o = 16; o <= 32; o *= 2) {
    const float v2 = __shfl_xor(bv, o);
    const int i2 = __shfl_xor(bi, o);
    if (arg_better(v2, i2, bv, bi)) {
      bv = v2;
      bi = i2;
    }
  }
  if (lane < 16 && ok) {
    a.amax_v[(int64_t)(ct / NT) * a.mp + m] = bv;
    a.amax_i[(int64_t)(ct / NT) * a.mp + m] = bi;
  }
}

// One head of HD = 16 NT columns: row scale, QK-norm, rotation, store (Q rows, or the fragment-major K / V caches).
template <int NT>
__device__ inline void tile_qkv(const GemmArgs& a, const f32x4* v, int h, int m, bool ok, float r, const RowInfo& ri,
                                int lane) {
#pragma clang fp contract(off)
  constexpr int C = 16 * NT;
  const int d0 = 4 * (lane / 16);
  const bool is_q = h < a.hq;
  f32x4 y[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int e = 0; e < 4; ++e) y[nt][e] = v[nt][e] * r;
  if (h >= a.hq + a.hkv) {
    if (!ok) return;
    uint16_t* vc = reinterpret_cast<uint16_t*>(a.vc) + ((int64_t)ri.seq * a.hkv + (h - a.hq - a.hkv)) * a.kv_ld * C;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int e = 0; e < 4; ++e) vc[vfrag_index(ri.pos, 16 * nt + d0 + e, C)] = f32_to_bf16(y[nt][e]);
    return;
  }
  if (a.qk_norm) {
    const float* gp = (is_q ? a.qn : a.kn) + d0;
    float ss = 0.f;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int e = 0; e < 4; ++e) ss += y[nt][e] * y[nt][e];
    ss = xor16_op(ss, [](float x, float z) { return x + z; });
    ss = xor32_op(ss, [](float x, float z) { return x + z; });
    const float inv = 1.f / sqrtf(ss / (float)C + a.eps);
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      const f32x4 gn = *reinterpret_cast<const f32x4*>(gp + 16 * nt);
#pragma unroll
      for (int e = 0; e < 4; ++e) y[nt][e] *= inv * gn[e];
    }
  }
  // rotation: dimension d pairs with d + C/2, NT / 2 tiles away in the same lane
#pragma unroll
  for (int nt = 0; nt < NT / 2; ++nt) {
    const float* t = a.rope + ((int64_t)(ok ? ri.pos : 0) * (C / 2) + 16 * nt + d0) * 2;
    const f32x4 c0 = *reinterpret_cast<const f32x4*>(t), c1 = *reinterpret_cast<const f32x4*>(t + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float c = e < 2 ? c0[2 * e] : c1[2 * e - 4], s = e < 2 ? c0[2 * e + 1] : c1[2 * e - 3];
      const float lo = y[nt][e], hi = y[nt + NT / 2][e];
      y[nt][e] = lo * c - hi * s;
      y[nt + NT / 2][e] = hi * c + lo * s;
    }
  }
  if (!ok) return;
  uint16_t* dst = is_q ? reinterpret_cast<uint16_t*>(a.q_out) + ((int64_t)m * a.hq + h) * C
                       : reinterpret_cast<uint16_t*>(a.kc) + ((int64_t)ri.seq * a.hkv + (h - a.hq)) * a.kv_ld * C;
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const int d = 16 * nt + d0;
    *reinterpret_cast<uint2*>(dst + (is_q ? d : kfrag_index(ri.pos, d, C))) =
        make_uint2(pack_bf16x2(y[nt][0], y[nt][1]), pack_bf16x2(y[nt][2], y[nt][3]));
  }
}

// MODE: what a launch's items are.  (A kernel that holds both kinds of item spills registers in its epilogues, outside
// the k-loop, so the launches of one kind keep kernels of their own.)
enum Mode { UNSPLIT = 0, SPLIT = 1, MIXED = 2 };

template <int WC, int RTW, int EPI, int MODE>
__global__ void __launch_bounds__(kTileThreads, 1) gemm_tile_kernel(GemmArgs a) {
  constexpr int NTW = 8, WR = 8 / WC, CG = NTW * WC, RT = WR * RTW, ROWS = 16 * RT;
  constexpr int kStage = (CG + RT) * 1024;
  constexpr int RS = std::min<int>(8, (int)(kTileRing / kStage));  // ring stages; RS - 1 k-steps in flight
  constexpr int NL = CG + RT, LQ = NL / 8, LR = NL % 8;            // a wave issues LQ + (wave < LR) loads per k-step
  constexpr int NWT = CG / 8;                                      // of them the first NWT are weight tiles
  static_assert(RS >= 3 && (RS - 2) * (LQ + 1) <= 63, "ring depth within the memory counter");
  __shared__ __align__(16) char s_ring[(size_t)RS * kStage];
  __shared__ float s_part[4][ROWS];
  __shared__ float s_rs[ROWS];
  __shared__ int s_flag, s_left;
  touch_kernargs<GemmArgs>();
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = threadIdx.x % kWave;
  const int wc = wv % WC, wr = wv / WC;  // this wave's column and row position
  const bool lateh = wv >= 4;            // the half that runs half a k-step behind
  // item: column block and k-split cs (one XCD's items are 8 apart), row block fastest within an XCD
  const int slot = blockIdx.x / kXcds, cs = blockIdx.x % kXcds + kXcds * (slot / a.nrb), rb = slot % a.nrb;
  if (cs >= a.ncb1 + (a.ncb - a.ncb1) * a.ksplit) return;
  const int S = MODE == SPLIT || (MODE == MIXED && cs >= a.ncb1) ? a.ksplit : 1;  // the first ncb1 column blocks are not split
  const int cb = S == 1 ? cs : a.ncb1 + (cs - a.ncb1) / S, sp = S == 1 ? 0 : (cs - a.ncb1) % S;
  const int kb = (int)((int64_t)a.KT * sp / S), nk = (int)((int64_t)a.KT * (sp + 1) / S) - kb;
  const int row0 = rb * ROWS, nrows = min(ROWS, a.M - row0);
  const uint32_t KT = (uint32_t)a.KT, G = (uint32_t)a.G, SC = (uint32_t)a.segc, NW = (uint32_t)a.n_wg;
  const int ng = a.ng, unit_b = ng * 1024;

  // The wave's loads of a k-step: fragments wv, wv + 8, ... of [CG weight tiles][RT row tiles].  A weight tile
  // is read where the matrix's streaming plan stores it: k-step k of group g is unit g KT + k of owner o, at slot
  // (g KT + k - start(o)) n_wg + o; one tracker per weight tile follows its group's owners as k rises.
  struct Trk {
    int g, o, kend, base;  // group, owner, first k-step past its share, slot of k-step 0
  };
  constexpr int kOob = 0x7ffffff0;  // a lane offset past every descriptor: zero without a memory access
  Trk trk[NWT];
  auto trk_set = [&](Trk& t, int o) {
    const uint32_t us = unit_start((uint32_t)o, KT, G, SC, NW), ue = unit_start((uint32_t)o + 1, KT, G, SC, NW);
    t.o = __builtin_amdgcn_readfirstlane(o);
    t.kend = __builtin_amdgcn_readfirstlane((int)(ue - (uint32_t)t.g * KT));
    t.base = __builtin_amdgcn_readfirstlane(((int)((uint32_t)t.g * KT) - (int)us) * (int)NW + o);
  };
  int wtile[NWT], fl[LQ + 1];  // byte offset of a weight tile inside its unit; this lane's offset of each fragment
#pragma unroll
  for (int i = 0; i < NWT; ++i) {
    const int ct = cb * CG + wv + 8 * i, g = ct / ng;
    trk[i].g = __builtin_amdgcn_readfirstlane(min(g, (int)G - 1));
    wtile[i] = __builtin_amdgcn_readfirstlane(ct % ng * 1024);
    fl[i] = g < (int)G ? lane * 16 : kOob;
    trk_set(trk[i], unit_owner((uint32_t)trk[i].g * KT + (uint32_t)kb, KT, G, SC, NW));
  }
#pragma unroll
  for (int i = NWT; i <= LQ; ++i) fl[i] = xfrag_lane(row0 / 16 + wv + 8 * i - CG, a.KT, a.M, lane);
  // Issues the next k-step's loads.  Every call issues the same ones, so that the memory-counter waits count alike;
  // past the last k-step the descriptors have no range (zero without a memory access).  Scalar state advances by
  // constants (this code shares the read phase with the LDS reads); only where a tile's owner changes are its offset
  // and the distance to the next change computed again.  Weights that no other row block reads are streamed past
  // the caches.
  const int wrange = (int)((uint32_t)a.share * NW * (uint32_t)unit_b), xrange = xfrag_bytes(a.M, a.KT);
  const int wstep = (int)NW * unit_b;
  int wofs[NWT], until = 0, ki = 0, slot_b = 0;
  auto retrack = [&]() {
    until = 0x7fffffff;
    const int k = kb + min(ki, nk - 1);
#pragma unroll
    for (int i = 0; i < NWT; ++i) {
      while (k >= trk[i].kend) trk_set(trk[i], trk[i].o + 1);
      wofs[i] = __builtin_amdgcn_readfirstlane((trk[i].base + k * (int)NW) * unit_b + wtile[i]);
      if (ki < nk) until = min(until, trk[i].kend - k);
    }
  };
  auto issue_as = [&](auto policy) {
    constexpr int kPolicy = decltype(policy)::value;
    const bool in = ki < nk;
    const __amdgpu_buffer_rsrc_t wrs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(a.W), 0, in ? wrange : 0, kBufferRsrcWord3);
    const __amdgpu_buffer_rsrc_t xrs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(a.X), 0, in ? xrange : 0, kBufferRsrcWord3);
    char* st = s_ring + slot_b + wv * 1024;
#pragma unroll
    for (int i = 0; i < NWT; ++i) {
      load_lds16<kPolicy>(wrs, st + i * 8192, fl[i], wofs[i]);
      wofs[i] += wstep;
    }
#pragma unroll
    for (int i = NWT; i <= LQ; ++i)
      if (i < LQ || wv < LR) load_lds16<0>(xrs, st + i * 8192, fl[i], (kb + ki) * 1024);
  };
  const bool once = a.nrb == 1;
  auto issue = [&]() {
    if (until == 0) retrack();
    if (once)
      issue_as(std::integral_constant<int, kNtCpol>{});
    else
      issue_as(std::integral_constant<int, 0>{});
    slot_b = slot_b + kStage == RS * kStage ? 0 : slot_b + kStage;
    ++ki;
    --until;
  };
  auto wait_next = [&]() {  // this wave's loads of the next k-step have landed (RS - 2 later ones may be in flight)
    if (LR > 0 && wv < LR)
      __builtin_amdgcn_s_waitcnt(wait_vmcnt((RS - 2) * (LQ + 1)));
    else
      __builtin_amdgcn_s_waitcnt(wait_vmcnt((RS - 2) * LQ));
  };

  // RMSNorm row scales of the block's rows: the producer's per-group sums of squares in the 33-row kernels' order
  // (every fourth group in group order, then (s0 + s1) + (s2 + s3)).  The loads go out ahead of the ring's (they
  // complete in order), the sums are taken while the first k-steps load.
  constexpr int kIt = EPI == EPI_RESID ? 0 : (4 * ROWS + kTileThreads - 1) / kTileThreads, kPre = 20;
  const int ng_in = EPI != EPI_RESID && a.ss_in ? a.ss_groups : 0;
  float pre[kIt > 0 ? kIt : 1][kPre];
  if (ng_in > 0) {
#pragma unroll
    for (int it = 0; it < kIt; ++it) {
      const int idx = min((int)threadIdx.x + it * kTileThreads, 4 * ROWS - 1), q4 = idx / ROWS, row = min(idx % ROWS, nrows - 1);
#pragma unroll
      for (int j = 0; j < kPre; ++j) pre[it][j] = a.ss_in[(int64_t)min(q4 + 4 * j, ng_in - 1) * a.mp + row0 + row];
    }
  }
#pragma unroll
  for (int kt = 0; kt < RS - 1; ++kt) issue();
  if constexpr (EPI != EPI_RESID) {
#pragma unroll
    for (int it = 0; it < kIt; ++it) {
      const int idx = (int)threadIdx.x + it * kTileThreads, q4 = idx / ROWS, row = idx % ROWS;
      float ssum = 0.f;
#pragma unroll
      for (int j = 0; j < kPre; ++j)
        if (q4 + 4 * j < ng_in) ssum += pre[it][j];
      for (int g0 = q4 + 4 * kPre; g0 < ng_in; g0 += 4) ssum += a.ss_in[(int64_t)g0 * a.mp + row0 + min(row, nrows - 1)];
      if (idx < 4 * ROWS) s_part[q4][row] = ssum;
    }
    __builtin_amdgcn_s_waitcnt(kWaitLgkm0);
    phase_barrier();
    for (int r = threadIdx.x; r < ROWS; r += kTileThreads) {
      const float tot = (s_part[0][r] + s_part[1][r]) + (s_part[2][r] + s_part[3][r]);
      s_rs[r] = ng_in ? 1.f / sqrtf(tot / (float)a.d_in + a.eps) : 1.f;  // read after the loop's barriers
    }
  }

  f32x4 acc[RTW][NTW];
#pragma unroll
  for (int j = 0; j < RTW; ++j)
#pragma unroll
    for (int nt = 0; nt < NTW; ++nt) acc[j][nt] = f32x4{0.f, 0.f, 0.f, 0.f};

  const uint32_t ring = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char*)(s_ring);
  const uint32_t rd_w = ring + (uint32_t)(wc * NTW * 1024 + lane * 16);
  const uint32_t rd_x = ring + (uint32_t)((CG + wr * RTW) * 1024 + lane * 16);
  wait_next();
  phase_barrier();  // k-step 0 is whole
  if (lateh) phase_barrier();
  uint32_t so = 0;
#pragma unroll 1
  for (int t = 0; t < nk; ++t) {
    // read phase (the other half multiplies): the loads of k-step t + RS - 1 into the slot of k-step t - 1, which
    // both halves have read, and this k-step's fragments
    issue();
    u32x4 wf[NTW], xf[RTW];
    lds_read_frags<RTW>(wf, xf, rd_w + so, rd_x + so);
    so = so + kStage == (uint32_t)(RS * kStage) ? 0 : so + kStage;
    if (lateh) wait_next();
    phase_barrier();
    // multiply phase (the other half reads)
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int j = 0; j < RTW; ++j)
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt)
        mma_tile<uint16_t>(__builtin_bit_cast(uint4, wf[nt]), __builtin_bit_cast(uint4, xf[j]), acc[j][nt]);
    __builtin_amdgcn_s_setprio(0);
    if (!lateh) wait_next();
    phase_barrier();
  }
  if (!lateh) phase_barrier();
  __builtin_amdgcn_s_waitcnt(wait_vmcnt(0));  // the loads past the end (no memory access) before the block may end

  const int ntiles = (nrows + 15) / 16;  // row tiles that hold rows
  // epilogue of row tile rt (of the block) and the NTW column tiles of wave column wcol: column groups of NT tiles
  auto epilogue = [&](auto ntc, const f32x4* v, int rt, int wcol) {
    constexpr int NT = decltype(ntc)::value;
    const int lr = rt * 16 + lane % 16, m = row0 + lr, ct = cb * CG + wcol * NTW;
    const bool ok = lr < nrows;
    const float r = EPI == EPI_RESID ? 1.f : s_rs[ok ? lr : 0];
    RowInfo ri{0, 0, 1, 0};
    if constexpr (EPI == EPI_QKV || EPI == EPI_LOGITS) ri = a.rows[ok ? m : 0];
#pragma unroll
    for (int h = 0; h < NTW / NT; ++h) {
      const int c = ct + h * NT;
      if (16 * c < a.N) {  // (a column block's end may lie past the matrix)
        if constexpr (EPI == EPI_QKV) tile_qkv<NT>(a, v + h * NT, c / NT, m, ok && ri.valid, r, ri, lane);
        if constexpr (EPI == EPI_RESID) tile_resid<NT>(a, v + h * NT, c, m, ok, lane);
        if constexpr (EPI == EPI_SWIGLU) tile_swiglu<NT>(a, v + h * NT, c, m, ok, r, lane);
        if constexpr (EPI == EPI_LOGITS) tile_logits<NT>(a, v + h * NT, c, m, ok, ri.valid, r, lane);
      }
    }
  };
  auto with_nt = [&](auto f) {
    if (NTW == 8 && ng == 8)
      f(std::integral_constant<int, NTW>{});
    else
      f(std::integral_constant<int, 4>{});
  };
  if (MODE == UNSPLIT || (MODE == MIXED && S == 1)) {
    with_nt([&](auto ntc) {
#pragma unroll
      for (int j = 0; j < RTW; ++j)
        if (wr * RTW + j < ntiles) {
          epilogue(ntc, acc[j], wr * RTW + j, wc);
          if constexpr (MODE == MIXED) __builtin_amdgcn_sched_barrier(0);  // one row tile's loads at a time: registers
        }
    });
    return;
  }
  if constexpr (MODE != UNSPLIT) {

  // Split item: every contributor stores its accumulators (16-byte device-coherent stores) and the item is
  // finished in ksplit shares of (row tile, wave column) units, each summed in split order.  A contributor waits
  // for the others for a bounded time (a split launch has at most one workgroup per compute unit, so all of them
  // are normally running) and finishes its own share; whoever arrives last also takes the shares that nobody
  // claimed, so the item completes whether or not the others waited.  The last one to leave zeroes the counters.
  // (Unsplit items, launched first, wait for nobody, so the split ones behind them are always reached.)
  // Measured against the last arriver adding all partials: 264 rows of down_proj 125 -> 93 us, o_proj 61 -> 50.
  const __amdgpu_buffer_rsrc_t prs = __builtin_amdgcn_make_buffer_rsrc(a.part, 0, 0x7fffffff, kBufferRsrcWord3);
  const int item = rb * (a.ncb - a.ncb1) + cb - a.ncb1;
  auto part_off = [&](int sq, int rt, int wcol) {  // bytes (< 2^31: checked on the host)
    return (((item * S + sq) * RT + rt) * WC + wcol) * NTW * 1024 + lane * 16;
  };
#pragma unroll
  for (int j = 0; j < RTW; ++j)
    if (wr * RTW + j < ntiles)
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt)
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[j][nt]), prs,
                                               part_off(sp, wr * RTW + j, wc) + nt * 1024, 0, kCoherentCpol);
  wait_stores();
  __syncthreads();
  int* const cnt = &a.cnt[item * kCntStride];  // arrivals, claimed shares (bits), departures
  if (threadIdx.x == 0) {
    int st = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == S - 1 ? 2 : 0;
    for (int it = 0; st == 0 && it < kTilePolls; ++it) {
      __builtin_amdgcn_s_sleep(2);
      if (ld_coherent(cnt) == S) st = 1;
    }
    if (st == 1 && (__hip_atomic_fetch_or(cnt + 1, 1 << sp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >> sp & 1)) st = 0;
    // the last arriver claims its own share, and what is left once that is done
    s_flag = st;
  }
  __syncthreads();
  const int st = s_flag;  // 0: leave, 1: own share, 2: last arriver
  auto units = [&](int first, int step) {  // this wave's units of the share: one per (row tile, wave column)
    for (int un = first + step * wv; un < ntiles * WC; un += 8 * step) {
      const int rt = un / WC, wcol = un % WC;
      f32x4 sum[NTW];
#pragma unroll
      for (int nt = 0; nt < NTW; ++nt) sum[nt] = f32x4{0.f, 0.f, 0.f, 0.f};
      constexpr int kB = 3;  // partials in flight
      for (int s0 = 0; s0 < S; s0 += kB) {
        f32x4 pv[kB][NTW];
#pragma unroll
        for (int q = 0; q < kB; ++q)
#pragma unroll
          for (int nt = 0; nt < NTW; ++nt)
            pv[q][nt] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                      prs, part_off(min(s0 + q, S - 1), rt, wcol) + nt * 1024, 0, kCoherentCpol));
#pragma unroll
        for (int q = 0; q < kB; ++q)
          if (s0 + q < S)
#pragma unroll
            for (int nt = 0; nt < NTW; ++nt) sum[nt] += pv[q][nt];
      }
      with_nt([&](auto ntc) { epilogue(ntc, sum, rt, wcol); });
    }
  };
  if (st != 0) {
    units(sp, S);
    if (st == 2) {
      if (threadIdx.x == 0) {
        const int all = (1 << S) - 1;
        s_left = all & ~__hip_atomic_fetch_or(cnt + 1, all, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & ~(1 << sp);
      }
      __syncthreads();
      for (int q = 0; q < S; ++q)
        if (s_left >> q & 1) units(q, S);
    }
  }
  if (threadIdx.x == 0 &&
      __hip_atomic_fetch_add(cnt + 2, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == S - 1) {
    st_coherent(cnt, 0);
    st_coherent(cnt + 1, 0);
    st_coherent(cnt + 2, 0);
  }
  }
}

template <int EPI, int MODE>
void launch_shape(const TilePlan& p, const GemmArgs& a, hipStream_t st) {
  const dim3 grid(kXcds * (int)ceil_div(p.ncb1 + (int64_t)(p.ncb - p.ncb1) * p.ksplit, kXcds) * p.nrb), block(kTileThreads);
#define SDD_TILE(WC, RTW) \
  case WC * 10 + RTW: hipLaunchKernelGGL((gemm_tile_kernel<WC, RTW, EPI, MODE>), grid, block, 0, st, a); break
  switch (p.wc * 10 + p.rtw) {
    SDD_TILE(2, 2);
    SDD_TILE(2, 3);
    SDD_TILE(2, 4);
  }
  if constexpr (MODE != MIXED) {
    switch (p.wc * 10 + p.rtw) {
      SDD_TILE(2, 5);
      SDD_TILE(1, 1);
      SDD_TILE(1, 2);
      SDD_TILE(1, 3);
    }
  }
#undef SDD_TILE
}

template <int EPI>
void launch_tile(const TilePlan& p, const GemmArgs& a, hipStream_t st) {
  if (p.ksplit == 1)
    launch_shape<EPI, UNSPLIT>(p, a, st);
  else if (p.ncb1 == 0)
    launch_shape<EPI, SPLIT>(p, a, st);
  else
    launch_shape<EPI, MIXED>(p, a, st);
}

}  // namespace

// The launch's estimated time, fitted to measurements of every shape and split at 99-1792 rows of the Qwen3-32B and
// Qwen2.5-7B widths: a k-step takes 0.33 us (two barriers, the LDS reads' latency, load issue) + 14.2 ns per MFMA of
// a wave; weights stream at 6 TB/s at best, round by round; a split writes and reads its partial tiles once at about
// 6 TB/s and costs 3 us more, 15 us more again behind unsplit rounds.  Workgroups go to the XCDs round-robin, so rounds
// and the split workgroups that can run at once are counted per XCD.  (Counted over the whole chip, plans with 33-35
// waiting workgroups on an XCD of 32 compute units ran into the bound of the wait: down_proj of Qwen2.5-7B over 1136
// rows 250 -> 152 us, over 528 rows 142 -> 88.)
// Splitting only the column blocks left over after whole rounds: LM head of 99 rows 338 -> 310 us, gate/up of 1024 rows
// 474 -> 446 (Qwen3-32B width).  With 5 row tiles per wave that kernel spills in its k-loop and is not used.
TilePlan plan_tiles(const MatPlan& mp, int M, int n_cu, size_t part_bytes, int64_t max_split) {
  const int CT = mp.G * mp.ng, RTM = (int)ceil_div(M, 16), xcd_cus = std::max(1, n_cu / kXcds);
  TilePlan best{};
  best.us = 1e30;
  const size_t cap = std::min<size_t>(part_bytes, (size_t(1) << 31) - 1);
  const double hbm = (double)CT * mp.KT * 1024 / 6.0e6;
  constexpr int kShapes[][2] = {{1, 1}, {1, 2}, {1, 3}, {2, 2}, {2, 3}, {2, 4}, {2, 5}};
  for (const auto& sh : kShapes) {
    const int wc = sh[0], rtw = sh[1], CG = 8 * wc, RT = 8 / wc * rtw;
    const int ncb = (int)ceil_div(CT, CG), nrb = (int)ceil_div(RTM, RT);
    const double kstep = 0.33 + 0.0142 * 8 * rtw, tile_bytes = 1024.0 * CG * RTM / nrb;
    const auto round_us = [&](int s) { return (double)ceil_div(mp.KT, s) * kstep + 1.0; };
    const auto consider = [&](int ncb1, int s, double us) {
      if (us < best.us) best = TilePlan{wc, rtw, ncb, nrb, ncb1, s, us};
    };
    // the workgroups of n (column block, k-range) pairs on the XCD that gets most of them
    const auto per_xcd = [&](int64_t n) { return ceil_div(n, kXcds) * nrb; };
    const int full = (int)(per_xcd(ncb) / xcd_cus);  // whole rounds, each no faster than its weights stream
    const double full_us = std::max(round_us(1), hbm * xcd_cus / per_xcd(ncb));
    const double part = hbm - std::min(hbm, full * hbm * xcd_cus / per_xcd(ncb));
    // (unsplit: the last round's epilogue is exposed)
    consider(0, 1, 6.0 + full * full_us + (per_xcd(ncb) % xcd_cus ? std::max(part, round_us(1)) : 0.0) + tile_bytes / 50e3);
    // `rounds` whole rounds of every XCD's compute units unsplit, the column blocks left over split behind them
    for (int rounds : {0, full}) {
      const int ncb1 = kXcds * (rounds * xcd_cus / nrb);
      if (ncb1 >= ncb || (rounds > 0 && (ncb1 == 0 || wc != 2 || rtw > 4))) continue;
      const int64_t left = ncb - ncb1;
      for (int s = 2; s <= 16 && s * 8 <= mp.KT; ++s) {
        // a split tile's workgroups wait for each other: no more of them on an XCD than it can run at once
        if (per_xcd(left * s) > xcd_cus || (size_t)(left * nrb * s) * CG * RT * 1024 > cap || left * nrb > max_split) break;
        const double last = std::max(hbm * left / ncb, round_us(s)) + 2.0 * left * nrb * s * tile_bytes / 6.0e6;
        consider(ncb1, s, 9.0 + (rounds > 0 ? rounds * full_us + 15.0 : 0.0) + last);
      }
    }
  }
  return best;
}

int launch_gemm_tiles(const TilePlan& p, int epi, GemmArgs a, hipStream_t st) {
  a.ncb = p.ncb;
  a.ncb1 = p.ncb1;
  a.nrb = p.nrb;
  a.ksplit = p.ksplit;
  switch (epi) {
    case EPI_QKV: launch_tile<EPI_QKV>(p, a, st); break;
    case EPI_RESID: launch_tile<EPI_RESID>(p, a, st); break;
    case EPI_SWIGLU: launch_tile<EPI_SWIGLU>(p, a, st); break;
    default: launch_tile<EPI_LOGITS>(p, a, st); break;
  }
  return check_launch("gemm_tile_kernel");
}

}  // namespace sdd
