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
//  - the order of a row's sums is the matrix's, not the launch's (SumPlan): K is cut into segments, each summed k-step by
//    k-step from zero, and the segments' sums are added in order.  So a sequence's logits do not depend on the other
//    sequences of its call, nor a prompt's cached K/V on its chunks, bit for bit.  The price is what a free split
//    over K would gain where the segments do not suit the launch: 99 rows of o_proj 31 -> 46 us, down_proj 56 -> 69, qkv 36 -> 41,
//    LM head 310 -> 353, 264 rows of o_proj 47 -> 59 (Qwen3-32B width; no other product of 99, 264 or 1024 rows by more
//    than 7%);
//  - a launch is (column block, row block, contributor) items, one per workgroup.  The row blocks of one column block
//    run on one XCD next to each other, so its L2 serves the weights to all but the first of them.  Where the
//    tiles fill the chip a workgroup walks a tile's segments in order, keeping the sum so far in memory while it
//    multiplies the next one (a few us per segment); where they leave compute units idle, the segments are shared out:
//    partials go through 16-byte device-coherent stores and are added in segment order, the tile's row tiles shared
//    out among its contributors.
// Measured (Qwen3-32B width; with the chunked launches of 288 rows and 4 loading waves this kernel replaced): gate/up
// over 1024 rows 4 x 148 -> 455 us (1.18 PFLOP/s; the library's product at this size 0.99), over 264 rows 186 -> 136;
// down 125 -> 95, qkv 76 -> 53, o_proj 45 -> 59, LM head 546 -> 490 us; over 1024 rows down 244 (1.10 PFLOP/s), qkv 131,
// o_proj 95.  What bounds it: a k-step of 8 + RTW fragment
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

// Sum of squares of a row's 16 NT columns (y in the accumulator layout), in the order of the 33-row kernels: eight
// consecutive columns one after another, then those sums pairwise.  The first four of eight lie in an even lane group,
// the last four in the next one.  The result is in every lane of the row.
template <int NT>
__device__ inline float row_sum_squares(const f32x4* y) {
#pragma clang fp contract(off)
  float n[NT];
#pragma unroll
  for (int nt = 0; nt < NT; ++nt) {
    const f32x4 q = y[nt] * y[nt];
    float c = xor16_op(((q[0] + q[1]) + q[2]) + q[3], [](float lo, float) { return lo; });  // the even group's
#pragma unroll
    for (int e = 0; e < 4; ++e) c += q[e];
    n[nt] = xor32_op(c, [](float lo, float hi) { return lo + hi; });  // (right in the odd groups)
  }
#pragma unroll
  for (int o = 1; o < NT; o *= 2)
#pragma unroll
    for (int nt = 0; nt < NT; nt += 2 * o) n[nt] += n[nt + o];
  return xor16_op(n[0], [](float, float hi) { return hi; });
}

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
#pragma unroll
  for (int nt = 0; nt < NT; ++nt)
#pragma unroll
    for (int e = 0; e < 4; ++e) xo[nt][e] += v[nt][e];
  const float ss = row_sum_squares<NT>(xo);
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
    const float ss = row_sum_squares<NT>(y);
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

// MODE: how a launch's items sum over K.  WHOLE: the matrix has one segment per column group, one workgroup per tile.
// CHAIN: one workgroup per tile, which walks the segments in order.  SPLIT: a tile's segments are shared out.  (Kernels of
// their own: one that holds both the unsplit and the split epilogue spills registers.)
enum Mode { WHOLE = 0, CHAIN = 1, SPLIT = 2 };

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
  const int S = MODE == SPLIT ? a.ksplit : 1;
  const TileItem it = tile_item(a, blockIdx.x, S);
  if (it.cbl < 0) return;
  const int cb = it.cb, rb = it.rb, sp = it.sp;
  // k-steps, and the K segments (SumPlan) they are: those of the block's first sum group, which are the block's wherever
  // it is split
  TileRange rg{0, a.KT, 0, 1, 0, 1, 1};
  if constexpr (MODE == SPLIT) {
    rg = tile_range(a, cb * CG, sp);
    if (sp >= rg.E) return;
  }
  const int kb = __builtin_amdgcn_readfirstlane(rg.kb), ke = __builtin_amdgcn_readfirstlane(rg.ke), nk = ke - kb;
  const int E = rg.E, nslot = rg.nseg - rg.n0 + 1;
  const int row0 = rb * ROWS, nrows = min(ROWS, a.M - row0);
  const uint32_t KT = (uint32_t)a.KT, G = (uint32_t)a.G, SC = (uint32_t)a.segc, NW = (uint32_t)a.n_wg;
  const int ng = a.ng, unit_b = ng * 1024;

  // The wave's loads of a k-step: fragments wv, wv + 8, ... of [CG weight tiles][RT row tiles]; one tracker per weight
  // tile follows its group's owners as k rises.
  constexpr int kOob = 0x7ffffff0;  // a lane offset past every descriptor: zero without a memory access
  TileTrk trk[NWT];
  auto track = [&](TileTrk& t, int o) {
    trk_set(a, t, o);
    t.o = __builtin_amdgcn_readfirstlane(t.o);
    t.kend = __builtin_amdgcn_readfirstlane(t.kend);
    t.base = __builtin_amdgcn_readfirstlane(t.base);
  };
  int wtile[NWT], fl[LQ + 1];  // byte offset of a weight tile inside its unit; this lane's offset of each fragment
#pragma unroll
  for (int i = 0; i < NWT; ++i) {
    const int ct = cb * CG + wv + 8 * i, g = ct / ng;
    trk[i].g = __builtin_amdgcn_readfirstlane(min(g, (int)G - 1));
    wtile[i] = __builtin_amdgcn_readfirstlane(ct % ng * 1024);
    fl[i] = g < (int)G ? lane * 16 : kOob;
    track(trk[i], unit_owner((uint32_t)trk[i].g * KT + (uint32_t)kb, KT, G, SC, NW));
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
      while (k >= trk[i].kend) track(trk[i], trk[i].o + 1);
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

  const int ntiles = (nrows + 15) / 16;  // row tiles that hold rows
  // Ends of K segments inside this workgroup's range.  The wave's two halves of four column tiles (h) follow their sum
  // group's segments: its current one's owner, the k-step past it, whether an earlier one's sum is in memory, and where.
  const __amdgpu_buffer_rsrc_t prs = __builtin_amdgcn_make_buffer_rsrc(a.part, 0, 0x7fffffff, kBufferRsrcWord3);
  constexpr int kNoEnd = 0x7fffffff;
  struct Seg {
    uint32_t base;  // sum group's first unit (k-step 0)
    int own, end, chain, at;
  } sg[2];
  int t_end = kNoEnd;  // next k-step at whose end a segment ends
  auto seg_end = [&](Seg& s) {  // of segment s.own, none for the last one
    const int e = sum_start(a, s.base, s.own + 1);
    s.end = __builtin_amdgcn_readfirstlane(e < ke ? e : kNoEnd);
  };
  if constexpr (MODE != WHOLE) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const int ct = cb * CG + wc * NTW + 4 * h;
      sg[h].base = sum_base(a, MODE == SPLIT ? cb * CG : ct);
      sg[h].chain = 0;
      sg[h].own = MODE == SPLIT ? rg.own0 + rg.seg0 : sum_owner(a, sg[h].base);
      sg[h].at = MODE == CHAIN ? __builtin_amdgcn_readfirstlane(chain_place(a, rb, ct, sg[h].own, CG, RT)) : 0;
      seg_end(sg[h]);
      if (MODE == CHAIN && 16 * ct >= a.N) sg[h].end = kNoEnd;  // past the matrix
    }
    t_end = min(sg[0].end, sg[1].end);
  }
  const int tile = rb * a.ncb + it.cbl;
  auto part_off = [&](int slot, int rt, int wcol) {  // (< 2^31: checked on the host)
    return part_place(a, tile, slot, rt, wcol, RT, WC) + lane * 16;
  };
  // Adds the accumulators to the partial sum that is in `slot` (fresh: to zero).
  auto store_part = [&](int slot, bool fresh) {
#pragma unroll
    for (int j = 0; j < RTW; ++j)
      if (wr * RTW + j < ntiles) {
        const int at = part_off(slot, wr * RTW + j, wc);
        if (!fresh) {
          f32x4 v[NTW];
#pragma unroll
          for (int nt = 0; nt < NTW; ++nt)
            v[nt] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(prs, at + nt * 1024, 0, kCoherentCpol));
#pragma unroll
          for (int nt = 0; nt < NTW; ++nt) acc[j][nt] = v[nt] + acc[j][nt];
        }
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt)
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[j][nt]), prs, at + nt * 1024, 0, kCoherentCpol);
      }
  };
  auto store_seg = [&]() {  // the segment that the accumulators hold
    const int seg = sg[0].own - rg.own0;
    store_part(part_slot(rg, seg), seg == 0 || seg >= rg.n0);
  };
  // the sum of the segments before the accumulators' one, for row tile j and half h
  auto chain_load = [&](int h, int j, f32x4* v) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      v[i] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                           prs, lane * 16 + ((wr * RTW + j) * 4 + i) * 1024, sg[h].at, 0));
  };
  // After k-step `k`: the segments that end there leave the accumulators, which start again from zero.
  auto flush = [&](int k) {
    if constexpr (MODE == SPLIT) {
      store_seg();
#pragma unroll
      for (int j = 0; j < RTW; ++j)
#pragma unroll
        for (int nt = 0; nt < NTW; ++nt) acc[j][nt] = f32x4{0.f, 0.f, 0.f, 0.f};
      ++sg[0].own;
      seg_end(sg[0]);
      t_end = sg[0].end;
    } else {
#pragma unroll
      for (int h = 0; h < 2; ++h)
        if (k == sg[h].end) {
#pragma unroll
          for (int j = 0; j < RTW; ++j)
            if (wr * RTW + j < ntiles) {
              f32x4 v[4];
#pragma unroll
              for (int i = 0; i < 4; ++i) v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
              if (sg[h].chain) chain_load(h, j, v);
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                v[i] += acc[j][4 * h + i];
                __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v[i]), prs,
                                                       lane * 16 + ((wr * RTW + j) * 4 + i) * 1024, sg[h].at, 0);
                acc[j][4 * h + i] = f32x4{0.f, 0.f, 0.f, 0.f};
              }
            }
          sg[h].chain = 1;
          ++sg[h].own;
          seg_end(sg[h]);
        }
      t_end = min(sg[0].end, sg[1].end);
    }
  };

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
    if constexpr (MODE != WHOLE) {
      if (kb + t + 1 == t_end) flush(t_end);
    }
    if (!lateh) wait_next();
    phase_barrier();
  }
  if (!lateh) phase_barrier();
  __builtin_amdgcn_s_waitcnt(wait_vmcnt(0));  // the loads past the end (no memory access) before the block may end

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
  if constexpr (MODE != SPLIT) {
    with_nt([&](auto ntc) {
#pragma unroll
      for (int j = 0; j < RTW; ++j)
        if (wr * RTW + j < ntiles) {
          if constexpr (MODE == CHAIN) {
#pragma unroll
            for (int h = 0; h < 2; ++h)
              if (sg[h].chain) {
                f32x4 v[4];
                chain_load(h, j, v);
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[j][4 * h + i] = v[i] + acc[j][4 * h + i];
              }
          }
          epilogue(ntc, acc[j], wr * RTW + j, wc);
        }
    });
  } else {
  // Split item: every contributor stores its segments' sums (16-byte device-coherent stores) and the item is finished in E
  // shares of (row tile, wave column) units, each summed in segment order.  A contributor waits for the others for a
  // bounded time (a split launch has at most one workgroup per compute unit, so all of them are normally running; where
  // other work holds compute units, a waiting contributor holds its own until then) and finishes its own share; whoever
  // arrives last also takes the shares that nobody claimed, so the item completes whether or not the others waited.  The
  // last one to leave zeroes the counters.
  // Measured against the last arriver adding all partials: 264 rows of down_proj 125 -> 93 us, o_proj 61 -> 50.
  // Beside a stream that keeps the chip full of another program's products (as a drafter would) the 264-row call of 2 layers
  // takes 2.17 ms (alone 1.38) and the other stream's product 73 -> 112 us; with a kernel whose contributors left after
  // publishing, 2.36 ms (alone 1.78) and 73 -> 120.
  store_seg();
  wait_stores();
  __syncthreads();
  int* const cnt = &a.cnt[tile * kCntStride];  // arrivals, claimed shares (bits), departures
  if (threadIdx.x == 0) {
    int st = __hip_atomic_fetch_add(cnt, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == E - 1 ? 2 : 0;
    for (int i = 0; st == 0 && i < kTilePolls; ++i) {
      __builtin_amdgcn_s_sleep(2);
      if (ld_coherent(cnt) == E) st = 1;
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
      for (int s0 = 0; s0 < nslot; s0 += kB) {
        f32x4 pv[kB][NTW];
#pragma unroll
        for (int q = 0; q < kB; ++q)
#pragma unroll
          for (int nt = 0; nt < NTW; ++nt)
            pv[q][nt] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                      prs, part_off(min(s0 + q, nslot - 1), rt, wcol) + nt * 1024, 0, kCoherentCpol));
#pragma unroll
        for (int q = 0; q < kB; ++q)
          if (s0 + q < nslot)
#pragma unroll
            for (int nt = 0; nt < NTW; ++nt) sum[nt] += pv[q][nt];
      }
      with_nt([&](auto ntc) { epilogue(ntc, sum, rt, wcol); });
    }
  };
  if (st != 0) {
    units(sp, E);
    if (st == 2) {
      if (threadIdx.x == 0) {
        const int all = (1 << E) - 1;
        s_left = all & ~__hip_atomic_fetch_or(cnt + 1, all, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & ~(1 << sp);
      }
      __syncthreads();
      for (int q = 0; q < E; ++q)
        if (s_left >> q & 1) units(q, E);
    }
  }
  if (threadIdx.x == 0 &&
      __hip_atomic_fetch_add(cnt + 2, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == E - 1) {
    st_coherent(cnt, 0);
    st_coherent(cnt + 1, 0);
    st_coherent(cnt + 2, 0);
  }
  }
}

template <int EPI, int MODE>
void launch_shape(const TilePlan& p, const GemmArgs& a, hipStream_t st) {
  const dim3 grid(tile_grid(a)), block(kTileThreads);
#define SDD_TILE(WC, RTW) \
  case WC * 10 + RTW: hipLaunchKernelGGL((gemm_tile_kernel<WC, RTW, EPI, MODE>), grid, block, 0, st, a); break
  switch (p.wc * 10 + p.rtw) {
    SDD_TILE(1, 1);
    SDD_TILE(1, 2);
    SDD_TILE(1, 3);
    SDD_TILE(2, 2);
    SDD_TILE(2, 3);
    SDD_TILE(2, 4);
    SDD_TILE(2, 5);
  }
#undef SDD_TILE
}

template <int EPI>
void launch_tile(const TilePlan& p, const GemmArgs& a, hipStream_t st) {
  if (p.ksplit > 1)
    launch_shape<EPI, SPLIT>(p, a, st);
  else if (p.sums.nseg > 1)
    launch_shape<EPI, CHAIN>(p, a, st);
  else
    launch_shape<EPI, WHOLE>(p, a, st);
}

}  // namespace

SumPlan sum_plan(const MatPlan& mp, bool pairs) {
  SumPlan s{mp.ng, mp.G, mp.n_wg, mp.c, 1, true};
  if (pairs && mp.ng == 8) {
    s.tiles = 16;
    s.G = (mp.G + 1) / 2;
    s.n = s.G >= mp.n_wg ? mp.n_wg : s.G * std::min(mp.n_wg / s.G, mp.KT);
    s.c = 0;
  }
  s.uniform = s.c == 0 && s.n % s.G == 0;
  s.nseg = s.uniform ? s.n / s.G : s.n <= s.G ? 2 : s.n / s.G + 2;
  return s;
}

// The launch's estimated time, fitted to measurements of every shape and split at 99-1792 rows of the Qwen3-32B and
// Qwen2.5-7B widths: a k-step takes 0.33 us (two barriers, the LDS reads' latency, load issue) + 14.2 ns per MFMA of
// a wave; weights stream at 6 TB/s at best, round by round; a segment that ends in a workgroup's walk costs 2 us and
// 5 us per 256 x 256 tile; a split writes and reads its partial tiles once at about 6 TB/s and costs 3 us more.  A last
// round is the shorter the emptier it is (gate/up over 1024 rows, 3.1 rounds, takes 3.6 rounds' time).  Workgroups go to the XCDs round-robin, so rounds and the split workgroups that can run at
// once are counted per XCD.  (Counted over the whole chip, plans with 33-35 waiting workgroups on an XCD of 32 compute
// units had to wait for a second round: down_proj of Qwen2.5-7B over 1136 rows 250 -> 152 us, over 528 rows 142 -> 88.)
TilePlan plan_tiles(const MatPlan& mp, bool pairs, int M, int n_cu, size_t part_bytes, int64_t max_split) {
  const SumPlan sums = sum_plan(mp, pairs);
  const int CT = mp.G * mp.ng, RTM = (int)ceil_div(M, 16), xcd_cus = std::max(1, n_cu / kXcds);
  TilePlan best{};
  best.us = 1e30;
  const size_t cap = std::min<size_t>(part_bytes, (size_t(1) << 31) - 1);
  const double hbm = (double)CT * mp.KT * 1024 / 6.0e6;
  const double seg_avg = sums.uniform ? sums.nseg : 1.0 + (double)(sums.n - 1) / sums.G;  // segments per column group
  constexpr int kShapes[][2] = {{1, 1}, {1, 2}, {1, 3}, {2, 2}, {2, 3}, {2, 4}, {2, 5}};
  for (const auto& sh : kShapes) {
    const int wc = sh[0], rtw = sh[1], CG = 8 * wc, RT = 8 / wc * rtw;
    const int ncb = (int)ceil_div(CT, CG), nrb = (int)ceil_div(RTM, RT);
    const double kstep = 0.33 + 0.0142 * 8 * rtw, tile_bytes = 1024.0 * CG * RTM / nrb;
    const auto per_xcd = [&](int64_t n) { return ceil_div(n, kXcds) * nrb; };  // workgroups of n (column block, contributor) pairs on the XCD that gets most of them
    // one workgroup per tile, in as many launches as the running sums need; rounds no faster than their weights stream
    {
      // running sums: one place per 64 columns and row block, or one per boundary where shares are longer than groups
      const size_t place = (size_t)RT * 4096;
      const bool compact = !sums.uniform && sums.n <= sums.G && (size_t)nrb * sums.n * (sums.tiles / 4) * place <= cap;
      int per = ncb;  // column blocks per launch
      if (sums.nseg > 1 && !compact) per = (int)std::min<int64_t>(ncb, (int64_t)(cap / (place * nrb * 2 * wc)));
      if (per < 1) continue;
      const double chain = (seg_avg - 1.0) * (2.0 + 5.0 * CG * RT / 256);
      double us = 0.0;
      for (int c0 = 0; c0 < ncb; c0 += per) {
        const int n = std::min(per, ncb - c0), full = (int)(per_xcd(n) / xcd_cus);  // whole rounds
        const double round_us = mp.KT * kstep + 1.0 + chain, share = hbm * n / ncb;
        const double part = share - std::min(share, full * share * xcd_cus / per_xcd(n));
        // (the last round's epilogue is exposed)
        const double left = (double)(per_xcd(n) % xcd_cus) / xcd_cus;  // of a last round, which runs faster the emptier it is
        us += 6.0 + full * std::max(round_us, share * xcd_cus / per_xcd(n)) +
              (left > 0 ? std::max(part, round_us * (full ? 0.5 + 0.5 * left : 1.0)) : 0.0) + tile_bytes / 50e3;
      }
      if (us < best.us) best = TilePlan{wc, rtw, ncb, nrb, per, 1, 0, compact, sums, us};
    }
    // a tile's segments shared out, where every group has the same ones.  (Measured for groups with one or two, the LM head's:
    // its 594 tiles of 99 rows in segments on 1188 workgroups, a tile's second one to finish adding both, 465 us against 353.)
    if (!sums.uniform) continue;
    for (int s = 2; s <= std::min(16, sums.nseg); ++s) {
      const int slots = sums.nseg - (int)ceil_div(sums.nseg, s) + 1;
      if ((size_t)ncb * nrb * slots * CG * RT * 1024 > cap || (int64_t)ncb * nrb > max_split) continue;
      // a split tile's workgroups wait for each other: no more of them on an XCD than it can run at once
      if (per_xcd((int64_t)ncb * s) > xcd_cus) break;
      const double run = (double)ceil_div(sums.nseg, s) / sums.nseg * mp.KT * kstep + 1.0;
      const double us = 9.0 + std::max(hbm, run) + 2.0 * ncb * nrb * slots * tile_bytes / 6.0e6;
      if (us < best.us) best = TilePlan{wc, rtw, ncb, nrb, ncb, s, slots, false, sums, us};
    }
  }
  return best;
}

int launch_gemm_tiles(const TilePlan& p, int epi, GemmArgs a, hipStream_t st) {
  if (p.per < 1)  // (room for the running sums of 128 columns always plans)
    return fail(SDD_EUNSUPPORTED, "many-row GEMM: no plan for %d rows in this workspace", a.M);
  for (int cb0 = 0; cb0 < p.ncb; cb0 += p.per) {
    tile_launch(a, p, cb0);
    switch (epi) {
      case EPI_QKV: launch_tile<EPI_QKV>(p, a, st); break;
      case EPI_RESID: launch_tile<EPI_RESID>(p, a, st); break;
      case EPI_SWIGLU: launch_tile<EPI_SWIGLU>(p, a, st); break;
      default: launch_tile<EPI_LOGITS>(p, a, st); break;
    }
    const int rc = check_launch("gemm_tile_kernel");
    if (rc) return rc;
  }
  return SDD_OK;
}

}  // namespace sdd
