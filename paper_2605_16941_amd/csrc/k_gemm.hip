// GEMM C = A * W^T on gfx950 matrix cores (v_mfma_f32_32x32x16_bf16, or the
// _f16 form when activations and weights are fp16), with the epilogues of the
// WINO forward fused in:
//   QKV projection + rotate-half RoPE at the WINO position ids,
//   residual add into the fp32 stream (O projection, FFN down projection),
//   SwiGLU of interleaved gate/up tiles,
//   LM head + per-tile softmax statistics (max, sum-exp, best non-mask id,
//   logit of the current token) so the logits never reach memory,
//   plain fp32 store (+bias) for the test entry point.
//
// The LM-head epilogues read the final hidden rows as two 16-bit parts (hi and
// lo of the fp32 value) and multiply both with the same W tile, so the logits
// carry ~16 (bf16) or ~22 (fp16) mantissa bits of the hidden state.
//
// Tiling: a workgroup owns a BM x BN output tile and walks K in steps of 64.
// A and W tiles go straight from global memory into LDS (gfx950 LDS-DMA,
// global_load_lds_dwordx4: no staging registers), double-buffered so the next
// K step streams in while the matrix cores consume the current one.  Within a
// tile row the 16-byte chunks are XOR-swizzled by the row index, so the
// fragment reads of 8 consecutive rows hit distinct bank groups.  Waves form a WM x WN grid, each owning a
// (BM/WM) x (BN/WN) sub-tile of 32x32 MFMA blocks.  Workgroups are renumbered
// so that each XCD works on one contiguous range of tiles (shared W tiles stay
// in that XCD's L2).
#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdlib>
#include <mutex>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace wino {
namespace {

constexpr int BK = 64;

// SwiGLU virtual columns come in blocks of WTN: the first half of a block is
// gate rows f0..f0+WTN/2-1, the second half the up rows of the same f range,
// so each lane holds both factors of its outputs.
template <int WTN>
__device__ __forceinline__ int swiglu_row(int vc, int F) {
  constexpr int half = WTN / 2;
  const int blk = vc / WTN, c = vc - blk * WTN;
  const int f = blk * half + (c < half ? c : c - half);
  return c < half ? f : F + f;
}

// Row of W_qkv for virtual column vc when a wave owns half of a 128-wide head:
// each 128-row head is taken as (elements 0..31, 64..95), (32..63, 96..127), so a
// lane holds both elements of its rotate-half pairs.
__device__ __forceinline__ int qkv_half_row(int vc) {
  const int c = vc & 127, j = c >> 6, r = c & 63;
  return (vc & ~127) + 32 * j + r + (r & 32);
}

template <int FM, int FN>
__device__ __forceinline__ void epi_store(const GemmCall& c, f32x16 (&acc)[FM][FN], int rowb,
                                          int colb, int lane) {
  float bias[FN];
#pragma unroll
  for (int fn = 0; fn < FN; ++fn) bias[fn] = c.bias ? c.bias[colb + fn * 32 + (lane & 31)] : 0.f;
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int row = rowb + fm * 32 + mfma_row(i, lane);
      if (row >= c.M) continue;
      float* dst = c.outf + (size_t)row * c.ldc + colb + (lane & 31);
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) dst[fn * 32] = acc[fm][fn][i] + bias[fn];
    }
}

// The fp32 epilogues through the wave's LDS region (free once the K loop has
// drained): one 32-row block of accumulators at a time goes to LDS in the
// MFMA layout and comes back as 16-byte row chunks, so x (residual: read, add,
// write) or the partial buffer moves in 16-byte accesses - a quarter of the
// memory instructions of the 4-byte accesses straight from the MFMA layout.
// op(row, col, float4 v) gets 4 consecutive columns of one row.
template <int FM, int FN, class Op>
__device__ __forceinline__ void epi_rows16(f32x16 (&acc)[FM][FN], int lane, float* ws, Op op) {
  constexpr int WTN = FN * 32, C4 = WTN / 4;
#pragma unroll
  for (int fm = 0; fm < FM; ++fm) {
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int i = 0; i < 16; ++i) ws[mfma_row(i, lane) * WTN + fn * 32 + (lane & 31)] = acc[fm][fn][i];
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int it = 0; it < 32 * C4 / 64; ++it) {
      const int idx = it * 64 + lane, r = idx / C4, c4 = idx - (idx / C4) * C4;
      op(fm * 32 + r, c4 * 4, *reinterpret_cast<const float4*>(ws + r * WTN + c4 * 4));
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  }
}

// x += acc for a wave tile whose rows all lie below M, through the wave's LDS
// region like epi_rows16: a 32-row block's x loads all go out before its
// adds and stores (in program order, so the compiler need not prove the
// runtime-strided stores and loads apart, and one memory round trip covers
// the block instead of one per 16-byte chunk).  xb: the tile's x at
// (rowb, colb), the same in every lane.
template <int FM, int FN>
__device__ __forceinline__ void epi_residual_full(f32x16 (&acc)[FM][FN], int lane, float* ws, float* xb,
                                                  int ldc) {
  constexpr int WTN = FN * 32, C4 = WTN / 4, IT = 32 * C4 / 64;
  const int r0 = lane / C4, c4 = lane % C4;
  float* xl = xb + (size_t)r0 * ldc + c4 * 4;
#pragma unroll
  for (int fm = 0; fm < FM; ++fm) {
    float4 xv[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it)
      xv[it] = *reinterpret_cast<const float4*>(xl + (size_t)(fm * 32 + it * (64 / C4)) * ldc);
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int i = 0; i < 16; ++i) ws[mfma_row(i, lane) * WTN + fn * 32 + (lane & 31)] = acc[fm][fn][i];
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const float4 v = *reinterpret_cast<const float4*>(ws + (it * (64 / C4) + r0) * WTN + c4 * 4);
      float4 x = xv[it];
      x.x += v.x; x.y += v.y; x.z += v.z; x.w += v.w;
      *reinterpret_cast<float4*>(xl + (size_t)(fm * 32 + it * (64 / C4)) * ldc) = x;
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  }
}

// out = silu(gate) * up = g u / (1 + 2^(-g log2 e)), with the hardware exp2
// and reciprocal (about 1 ulp of fp32 each, far below the bf16 rounding that
// follows; an IEEE divide is ~10 VALU instructions per element, and the
// epilogue runs while the matrix cores of the CU idle).  Stores are buffer
// stores: the row offset of each accumulator register is wave-uniform and
// goes in a scalar register, the lane's column in the vector offset.  In a
// tile that crosses the last row, rows past it get an offset beyond the
// buffer range, which drops their stores.
template <class A, int FM, int FN>
__device__ __forceinline__ void epi_swiglu(const GemmCall& c, f32x16 (&acc)[FM][FN], int rowb,
                                           int colb, int lane) {
  constexpr int H2 = FN / 2, WTM = FM * 32;
  // wave-uniform: the resource and the row offsets live in scalar registers
  rowb = __builtin_amdgcn_readfirstlane(rowb);
  colb = __builtin_amdgcn_readfirstlane(colb);
  if (rowb >= c.M) return;
  const int nrows = min(c.M - rowb, WTM), ld2 = c.ldc * 2;
  const auto rs = __builtin_amdgcn_make_buffer_rsrc(c.outh + (size_t)rowb * c.ldc + colb / 2, (short)0,
                                                    nrows * ld2, kBufferDword3);
  const int lrow = 4 * (lane >> 5);
  const int voff = lrow * ld2 + (lane & 31) * 2;
  auto body = [&](auto full) {
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int srow = fm * 32 + 8 * (i >> 2) + (i & 3);
        int vo = voff;
        if constexpr (!decltype(full)::value) vo = srow + lrow < nrows ? voff : kBufferOffNone;
#pragma unroll
        for (int fn = 0; fn < H2; ++fn) {
          const float g = acc[fm][fn][i], u = acc[fm][fn + H2][i];
          const float sg = __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(g * -1.44269504088896341f));
          __builtin_amdgcn_raw_buffer_store_b16(A::cvt(g * u * sg), rs, vo + fn * 64, srow * ld2, 0);
        }
      }
  };
  if (nrows == WTM) body(std::true_type{});
  else body(std::false_type{});
}

// Sequence b and position t of row rowb + lr of a wave's tile (rows are
// sequence-major, T per sequence).  TWO: the sequences are at least as long
// as the tile, so it spans at most two of them - one division per wave and a
// compare per row instead of a division per row.
template <bool TWO>
struct TileRows {
  int b0, t0, T;
  __device__ __forceinline__ TileRows(int rowb, int T_) : T(T_) {
    b0 = rowb / T;
    t0 = rowb - b0 * T;
  }
  __device__ __forceinline__ void at(int lr, int& b, int& t) const {
    if constexpr (TWO) {
      t = t0 + lr;
      const bool nx = t >= T;
      t = nx ? t - T : t;
      b = b0 + (int)nx;
    } else {
      const int r = b0 * T + t0 + lr;
      b = r / T;
      t = r - b * T;
    }
  }
};

// Wave columns = one head (WTN == hd): lane holds columns e and e + hd/2 of
// the rotate-half pair in fragments fn and fn + FN/2.  The wave's rotated q/k
// rows (or its v columns, transposed) are staged in the wave's own LDS region
// of WTM x hd bf16 and leave in 16-byte stores: whole q/k rows of hd elements,
// and runs of 8 consecutive positions of v^T.  Storing v^T straight from the
// MFMA layout would scatter 2-byte writes over hd rows of the transposed
// buffer.  16-byte chunks are XOR-swizzled by the row index, so the
// half-waves' writes (4 rows apart) land in distinct banks.
// HR = 2: the wave owns half of a 128-wide head, elements 32j..32j+31 of each half
// of it (qkv_half_row orders the W rows so), and its local element e is element
// e + 32j (+ 32 from e = 32 on) of the head.  64-wide wave tiles then serve every
// head size: with whole heads only, 128-wide heads had no 192-row tile and few small
// ones (1444 x 12288 x 4096 201 -> 177 us, 1260 x 7680 x 2560 75 -> 65, 776 x 3072 x
// 1024 23 -> 17, 130 x 1536 x 512 9.5 -> 6.6).
template <class A, int FM, int FN, bool TWO, int HR>
__device__ __forceinline__ void epi_qkv_rope(const GemmCall& c, f32x16 (&acc)[FM][FN], int rowb,
                                             int colb, int lane, uint16_t* ws) {
  constexpr int H2 = FN / 2;
  constexpr int WTM = FM * 32, HDL = FN * 32, HD = HDL * HR;
  static_assert(HR == 1 || HDL == 64, "half heads of 128-wide ones");
  constexpr int QCH = HDL / 8;  // 16-byte chunks per staged q/k row (power of two)
  constexpr int VCH = WTM / 8;  // 16-byte chunks per v^T row
  // v^T rows are 2*VCH slots of 8 bytes; slot s of row e sits at s ^ m(e),
  // m(e) = (e >> 1) & SMASK, so 32 consecutive rows written at one slot
  // cover 64 distinct banks.  A 16-byte chunk stays whole (its halves swap
  // when m(e) is odd).
  constexpr int SL = 2 * VCH;
  constexpr int SMASK = SL % 16 == 0 ? 15 : SL % 8 == 0 ? 7 : SL % 4 == 0 ? 3 : 1;
  static_assert((QCH & (QCH - 1)) == 0 && 64 % QCH == 0, "q/k chunking");
  static_assert((HDL * VCH) % 64 == 0, "v^T chunking");
  const RopeOut& ro = c.rope;
  const StepGeom& g = c.geom;
  // wave-uniform: store bases and row offsets live in scalar registers
  rowb = __builtin_amdgcn_readfirstlane(rowb);
  colb = __builtin_amdgcn_readfirstlane(colb);
  const int half = HDL / 2;
  const int d = ro.H * HD;
  const int hj = HR == 2 ? (colb / HDL) & 1 : 0;  // which half of the head
  // element of the head that local element e is (e in steps of up to 32)
  auto elem = [&](int e) { return HR == 2 ? e + 32 * hj + (e & 32) : e; };
  const int which = colb / d;               // 0 q, 1 k, 2 v
  const int head = (colb - which * d) / HD;
  if (rowb >= c.M) return;  // a wave wholly past the last row
  const TileRows<TWO> tr(rowb, g.T);
  // the wave's first sequence and position, marked uniform (the division
  // runs on the vector unit) so the store bases below stay scalar
  const int b0u = __builtin_amdgcn_readfirstlane(tr.b0), t0u = __builtin_amdgcn_readfirstlane(tr.t0);
  // A wave whose rows are all normal rows of one sequence has position = t:
  // its table rows follow one base pointer at constant offsets, and each lane
  // writes its two rotated values (elements e and e + 64) as 16-bit stores.
  // The staged layout is the general path's: element e of row r in 16-byte
  // chunk (e >> 3) ^ (r & 15).  With r = lrc + 4*g (lrc the row's constant
  // part, g = lane / 32) that chunk is c8 | ((fn ^ g) << 2) | (q ^ (i & 3)),
  // q = (lane & 31) / 8, c8 = bit 3 of lrc, and element e + 64 flips bit 3:
  // a per-lane base and a compile-time offset for every store.
  bool plain = false;
  if constexpr (TWO && HDL == 128) plain = which < 2 && tr.t0 + WTM <= g.S;
  if (plain) {
    const int g4 = lane >> 5, q8 = (lane & 31) >> 3;
    const float* tb = ro.tab + ((size_t)(t0u + 4 * g4) * 32 + (lane & 31)) * 4;
    uint16_t* wl = ws + 4 * g4 * HD + (lane & 7);
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int i3 = i & 3, c8 = 8 * ((i >> 2) & 1);
        const int lrc = fm * 32 + 8 * (i >> 2) + i3;
        const float4 t4 = *reinterpret_cast<const float4*>(tb + (size_t)lrc * 128);
        const float cst[4] = {t4.x, t4.y, t4.z, t4.w};
#pragma unroll
        for (int fn = 0; fn < 2; ++fn) {
          const float cs = cst[2 * fn], sn = cst[2 * fn + 1];
          const float x1 = acc[fm][fn][i], x2 = acc[fm][fn + 2][i];
          const float r1 = fmaf(x1, cs, -(x2 * sn));  // element e
          const float r2 = fmaf(x2, cs, x1 * sn);     // element e + hd/2
          const uint32_t pk = A::pack2(r1, r2);
          uint16_t* row = wl + lrc * HD + (((((fn ^ g4) << 2) | (q8 ^ i3))) << 3);
          row[c8 << 3] = (uint16_t)pk;
          row[(c8 ^ 8) << 3] = (uint16_t)(pk >> 16);
        }
      }
  } else if (which < 2) {
    // block starts of the wave's first two sequences (the second clamped to
    // the batch: rows past the last compute a valid but unused position)
    const int cs0 = cur_start(g, tr.b0), cs1 = cur_start(g, min(tr.b0 + 1, g.B - 1));
#pragma unroll
    for (int fm = 0; fm < FM; ++fm)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        // rows past the last are staged too (their q/k never leave LDS)
        const int lr = fm * 32 + mfma_row(i, lane);
        int b, t;
        tr.at(lr, b, t);
        int pos = t;
        if (t >= g.S) {
          if constexpr (TWO) pos = (b == tr.b0 ? cs0 : cs1) + (t - g.S);
          else pos = cur_start(g, min(b, g.B - 1)) + (t - g.S);
        }
        uint16_t* wr = ws + lr * HDL;
        const int sw = lr & (QCH - 1);
        float cst[2 * H2];  // (cos, sin) of elements fn*32 + (lane & 31)
        const float* tp = ro.tab + ((size_t)pos * 32 + (lane & 31)) * (2 * H2 * HR) + 2 * hj;
        if constexpr (H2 == 2) {
          const float4 t4 = *reinterpret_cast<const float4*>(tp);
          cst[0] = t4.x; cst[1] = t4.y; cst[2] = t4.z; cst[3] = t4.w;
        } else {
#pragma unroll
          for (int j = 0; j < H2; ++j) {
            const float2 t2 = *reinterpret_cast<const float2*>(tp + 2 * j);
            cst[2 * j] = t2.x; cst[2 * j + 1] = t2.y;
          }
        }
#pragma unroll
        for (int fn = 0; fn < H2; ++fn) {
          const int e = fn * 32 + (lane & 31);
          const float cs = cst[2 * fn], sn = cst[2 * fn + 1];
          const float x1 = acc[fm][fn][i], x2 = acc[fm][fn + H2][i];
          // explicit FMAs: the rounding does not depend on how the compiler
          // contracts the products
          const float r1 = fmaf(x1, cs, -(x2 * sn));  // element e
          const float r2 = fmaf(x2, cs, x1 * sn);     // element e + hd/2
          // lane pairs trade one value: the even lane stores elements e, e+1,
          // the odd lane elements e+hd/2-1, e+hd/2 (one 4-byte write each)
          const bool odd = lane & 1;
          // (lane ^ 1 by a DPP quad swap, no LDS round trip)
          const float got = __uint_as_float(dpp_mov<0xB1>(__float_as_uint(odd ? r1 : r2)));
          const int ee = odd ? e + half - 1 : e;
          const uint32_t pk = odd ? A::pack2(got, r2) : A::pack2(r1, got);
          *reinterpret_cast<uint32_t*>(wr + (((ee >> 3) ^ sw) << 3) + (ee & 7)) = pk;
        }
      }
  }
  if (which < 2) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    uint16_t* base = which == 0 ? ro.q : ro.k;
    constexpr int RPI = 64 / QCH;  // rows per pass
    if (tr.t0 + WTM <= g.T && rowb + WTM <= c.M) {
      // the wave's rows are one contiguous block of one sequence: 16-byte
      // stores from a wave-uniform base at per-lane plus constant offsets
      // (no per-row position, address or bounds arithmetic).  Not buffer
      // stores with the row offset in a scalar register: after such a 16-byte
      // store the compiler let the next instruction overwrite its data
      // register with no wait state, and one dword of it was lost.
      const size_t bh = (size_t)b0u * ro.H + head;
      uint16_t* dst = uniform_ptr(base + (bh * g.Tp + t0u) * HD);
      const int lrl = lane / QCH, ch = lane & (QCH - 1);
      uint16_t* dl = dst + lrl * HD + elem(ch * 8);
#pragma unroll
      for (int it = 0; it < WTM / RPI; ++it) {
        const int lr = it * RPI + lrl;
        const uint4 v = *reinterpret_cast<const uint4*>(ws + lr * HDL + ((ch ^ (lr & (QCH - 1))) << 3));
        *reinterpret_cast<uint4*>(dl + it * RPI * HD) = v;
      }
    } else {
#pragma unroll
    for (int it = 0; it < WTM / RPI; ++it) {
      const int lr = it * RPI + lane / QCH, ch = lane & (QCH - 1);
      if (rowb + lr >= c.M) continue;
      int b, t;
      tr.at(lr, b, t);
      const size_t bh = (size_t)b * ro.H + head;
      const uint4 v = *reinterpret_cast<const uint4*>(ws + lr * HDL + ((ch ^ (lr & (QCH - 1))) << 3));
      *reinterpret_cast<uint4*>(base + (bh * g.Tp + t) * HD + elem(ch * 8)) = v;
    }
    }
  } else {
    // v^T staging: LDS row e holds the WTM positions of this wave; lane writes
    // the 4 consecutive positions 8*(i/4) + 4*(lane/32) + 0..3 of fragment fm.
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
      const int e = fn * 32 + (lane & 31);
      uint16_t* wr = ws + e * WTM;
#pragma unroll
      for (int fm = 0; fm < FM; ++fm)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int tl = fm * 32 + 8 * q + 4 * (lane >> 5);
          uint2 v;
          v.x = A::pack2(acc[fm][fn][4 * q], acc[fm][fn][4 * q + 1]);
          v.y = A::pack2(acc[fm][fn][4 * q + 2], acc[fm][fn][4 * q + 3]);
          const int slot = (tl >> 2) ^ ((e >> 1) & SMASK);
          *reinterpret_cast<uint2*>(wr + slot * 4) = v;
        }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    if (tr.t0 + WTM <= g.T && rowb + WTM <= c.M && (tr.t0 & 7) == 0) {
      // one sequence, no row past M, 16-byte aligned runs: the head's v^T
      // rows from a wave-uniform base (position t0) at per-lane offsets
      const size_t bh = (size_t)b0u * ro.H + head;
      uint16_t* dst = uniform_ptr(ro.vt + bh * HD * g.Tp + t0u);
#pragma unroll
      for (int it = 0; it < HDL * VCH / 64; ++it) {
        int e, ch;
        if constexpr ((VCH & (VCH - 1)) == 0) {
          e = it * (64 / VCH) + lane / VCH;  // (a lane part and a constant part)
          ch = lane % VCH;
        } else {
          e = (it * 64 + lane) / VCH;
          ch = it * 64 + lane - e * VCH;
        }
        const int m = (e >> 1) & SMASK;
        uint4 v = *reinterpret_cast<const uint4*>(ws + e * WTM + ((ch ^ (m >> 1)) << 3));
        if (m & 1) v = make_uint4(v.z, v.w, v.x, v.y);
        *reinterpret_cast<uint4*>(dst + (size_t)elem(e) * g.Tp + ch * 8) = v;
      }
      return;
    }
#pragma unroll
    for (int it = 0; it < HDL * VCH / 64; ++it) {
      const int idx = it * 64 + lane;
      const int e = idx / VCH, ch = idx - (idx / VCH) * VCH;
      const int m = (e >> 1) & SMASK;
      uint4 v = *reinterpret_cast<const uint4*>(ws + e * WTM + ((ch ^ (m >> 1)) << 3));
      if (m & 1) v = make_uint4(v.z, v.w, v.x, v.y);
      const int r0 = rowb + ch * 8;
      if (r0 >= c.M) continue;
      int b, t0;
      tr.at(ch * 8, b, t0);
      if (r0 + 7 < c.M && t0 + 7 < g.T && (t0 & 7) == 0) {
        const size_t bh = (size_t)b * ro.H + head;
        *reinterpret_cast<uint4*>(ro.vt + (bh * HD + elem(e)) * g.Tp + t0) = v;
      } else {
        // run crosses a sequence end or the last row, or T is not a multiple
        // of 8: element stores
        const uint16_t* h = reinterpret_cast<const uint16_t*>(&v);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const int r = r0 + j;
          if (r >= c.M) break;
          const int bj = r / g.T, tj = r - bj * g.T;
          ro.vt[(((size_t)bj * ro.H + head) * HD + elem(e)) * g.Tp + tj] = h[j];
        }
      }
    }
  }
}

// LM head epilogue: per row of the tile, statistics over the BN columns.  The
// kernel multiplies with the operands swapped (W rows as the MFMA's A), so lane
// l holds row l % 32 of each 32-row block and, in register i of block fn, the
// id colb + fn*32 + mfma_row(i, l): a row's statistics are reductions inside
// the lane and over the pair (l, l ^ 32).  With the ids across the lanes every
// row took four 32-lane reductions: 16 rows x 4096 ids (K = 256) 14.8 -> 6.8
// us, 128 x 126464 (K = 4096) 272 -> 251 us, 836 rows 1630 -> 1486 us.
template <int BM, int WM, int WN, int FM, int FN>
__device__ __forceinline__ void epi_lmstats(const GemmCall& c, f32x16 (&acc)[FM][FN], int m0,
                                            int tn, int colb, int lane, int wm, int wn,
                                            uint16_t* smem_raw) {
  const LmStatsOut& lm = c.lm;
  float* red_m = reinterpret_cast<float*>(smem_raw);
  float* red_s = red_m + WN * BM;
  float* red_b = red_s + WN * BM;
  float* red_t = red_b + WN * BM;
  int* red_i = reinterpret_cast<int*>(red_t + WN * BM);
  float* red_z = reinterpret_cast<float*>(red_i + WN * BM);  // entropy term (pz only)
  constexpr int WTN = FN * 32;
  colb = __builtin_amdgcn_readfirstlane(colb);
  const int id0 = colb + 4 * (lane >> 5);  // register i of block fn: id0 + fn*32 + 8*(i/4) + i%4
  if (lm.bias) {
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        struct __attribute__((packed, aligned(4))) F4 { float v[4]; };  // (a 16-byte load at any 4-byte address)
        const F4 bz = *reinterpret_cast<const F4*>(lm.bias + id0 + fn * 32 + 8 * q);
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[fm][fn][4 * q + e] += bz.v[e];
      }
  }
  const bool mask_here = lm.mask_id >= colb && lm.mask_id < colb + WTN;
  __syncthreads();  // LDS is reused
#pragma unroll
  for (int fm = 0; fm < FM; ++fm) {
    const int lrow = wm * (BM / WM) + fm * 32 + (lane & 31);
    const int row = m0 + lrow;
    const int tgt = row < c.M ? lm.target[row] : -1;
    float mx = kNegBig;
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int i = 0; i < 16; ++i) mx = fmaxf(mx, acc[fm][fn][i]);
    mx = max_xor32(mx);
    // best value over non-mask ids: differs from mx only where the mask id is
    float bz = mx;
    if (mask_here) {
      bz = kNegBig;
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          bz = id0 + fn * 32 + 8 * (i >> 2) + (i & 3) == lm.mask_id ? bz : fmaxf(bz, acc[fm][fn][i]);
      bz = max_xor32(bz);
    }
    // its lowest id (ids grow with fn, then i, within a lane)
    int bi = INT_MAX;
#pragma unroll
    for (int fn = FN - 1; fn >= 0; --fn)
#pragma unroll
      for (int i = 15; i >= 0; --i) bi = acc[fm][fn][i] == bz ? id0 + fn * 32 + 8 * (i >> 2) + (i & 3) : bi;
    if (mask_here && bi == lm.mask_id) {  // the mask id ties with the best other id: look past it
      bi = INT_MAX;
#pragma unroll
      for (int fn = FN - 1; fn >= 0; --fn)
#pragma unroll
        for (int i = 15; i >= 0; --i) {
          const int id = id0 + fn * 32 + 8 * (i >> 2) + (i & 3);
          bi = acc[fm][fn][i] == bz && id != lm.mask_id ? id : bi;
        }
    }
    bi = min_xor32(bi);
    float tz = kNegBig;
    const int trel = tgt - id0;  // this lane's ids: bit 2 of trel clear
    if (__any(trel >= 0 && trel < WTN && !(trel & 4))) {
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
#pragma unroll
        for (int i = 0; i < 16; ++i) tz = trel == fn * 32 + 8 * (i >> 2) + (i & 3) ? acc[fm][fn][i] : tz;
      tz = max_xor32(tz);
    }
    float se4[4] = {0.f, 0.f, 0.f, 0.f}, sz4[4] = {0.f, 0.f, 0.f, 0.f};
    if (lm.pz) {
      // sum exp(z - m) * (z - m): the entropy's expectation term, relative
      // to the tile max so nothing cancels against a large m
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float u = acc[fm][fn][i] - mx;
          const float e = __expf(u);
          se4[i & 3] += e;
          sz4[i & 3] += e * u;
        }
    } else {
#pragma unroll
      for (int fn = 0; fn < FN; ++fn)
#pragma unroll
        for (int i = 0; i < 16; ++i) se4[i & 3] += __expf(acc[fm][fn][i] - mx);
    }
    const float se = sum_xor32((se4[0] + se4[1]) + (se4[2] + se4[3]));
    const float sz = sum_xor32((sz4[0] + sz4[1]) + (sz4[2] + sz4[3]));
    if (lane < 32) {
      red_m[wn * BM + lrow] = mx;
      red_s[wn * BM + lrow] = se;
      red_b[wn * BM + lrow] = bz;
      red_t[wn * BM + lrow] = tz;
      red_i[wn * BM + lrow] = bi;
      if (lm.pz) red_z[wn * BM + lrow] = sz;
    }
  }
  __syncthreads();
  for (int r = threadIdx.x; r < BM; r += WM * WN * 64) {
    const int row = m0 + r;
    if (row >= c.M) continue;
    float m = kNegBig;
#pragma unroll
    for (int w = 0; w < WN; ++w) m = fmaxf(m, red_m[w * BM + r]);
    float s = 0.f, z = 0.f, bz = kNegBig, tz = kNegBig;
    int bi = INT_MAX;
#pragma unroll
    for (int w = 0; w < WN; ++w) {
      const float dm = red_m[w * BM + r] - m, f = __expf(dm);
      s += red_s[w * BM + r] * f;
      // sum e^{z-m}(z-m) = e^{m_w-m} (sum e^{z-m_w}(z-m_w) + (m_w-m) sum e^{z-m_w})
      if (lm.pz) z += f * (red_z[w * BM + r] + dm * red_s[w * BM + r]);
      const float ob = red_b[w * BM + r];
      const int oi = red_i[w * BM + r];
      if (ob > bz || (ob == bz && oi < bi)) { bz = ob; bi = oi; }
      tz = fmaxf(tz, red_t[w * BM + r]);
    }
    const size_t o = (size_t)row * lm.n_part + tn;
    if (lm.pz) lm.pz[o] = z;
    lm.pm[o] = m;
    lm.ps[o] = s;
    lm.pb[o] = bz;
    lm.pi[o] = bi;
    lm.pt[o] = tz;
  }
}

// Physical 16-byte position of chunk kc of LDS tile row r: rows of KB bf16
// (KB/8 chunks) are XOR-swizzled so the fragment reads of 8 or 16
// consecutive rows at one chunk hit distinct bank groups.
//   KB = 64 (128-byte rows): kc ^ ((r ^ (r >> 3)) & 7): any 8 consecutive rows
//     use 8 positions, any 16 rows 16 (row parity, position) pairs.
//   KB = 32 (64-byte rows, 4 per 64 banks): kc ^ ((r >> 2) & 3): 16
//     consecutive rows give 16 distinct (r mod 4, position) pairs.
template <int KB>
__device__ __forceinline__ int lds_swz(int r) {
  if constexpr (KB == 64) return (r ^ (r >> 3)) & 7;
  else return (r >> 2) & 3;
}

// OCC workgroups per CU: the launch bound asks for OCC * waves / 4 waves per
// SIMD, which caps the registers per wave accordingly.  XW > 0 gives the W
// tiles XW more LDS stages than the two of A, so W copies have 1 + XW K
// steps to land instead of one (for weights that few row tiles share, whose
// copies mostly miss L2).
template <int BM, int BN, int WM, int WN, int EPI, int KB, int NST, int OCC, int XW, class A>
__global__ __launch_bounds__(WM* WN * 64, (OCC * WM * WN + 3) / 4) void gemm_kernel(const GemmCall c) {
  static_assert(KB == 32 || KB == 64, "K step");
  static_assert(NST >= 2, "pipeline stages");
  static_assert(XW == 0 || (XW <= 2 && NST == 2), "extra W stages beside two A stages");
  constexpr int NW = WM * WN;
  constexpr int WTM = BM / WM, WTN = BN / WN;
  constexpr int FM = WTM / 32, FN = WTN / 32;
  // LM-head epilogues multiply W with both bf16 parts (hi, lo) of the fp32 rows
  constexpr bool SPLIT = EPI == EPI_LMSTATS || EPI == EPI_LOGITS;
  constexpr int AROWS = SPLIT ? 2 * BM : BM;
  // one LDS-DMA instruction moves 64 lanes x 16 bytes = 1 KB = RPI tile rows
  constexpr int CPR = KB / 8;    // 16-byte chunks per tile row
  constexpr int RPI = 64 / CPR;  // tile rows per DMA instruction
  constexpr int A_INS = AROWS / (RPI * NW);
  constexpr int B_INS = BN / (RPI * NW);
  constexpr int INS = A_INS + B_INS;
  static_assert(A_INS * RPI * NW == AROWS && B_INS * RPI * NW == BN, "loader split");
  static_assert(FM >= 1 && FN >= 1, "wave tile");
  constexpr int NSB = NST + XW;  // W stages
  constexpr int A_STAGE = AROWS * KB, B_STAGE = BN * KB;  // bf16 elements per stage
  constexpr int LDS_ELEMS = NST * A_STAGE + NSB * B_STAGE;  // A stages, then W stages

  __shared__ __attribute__((aligned(1024))) uint16_t smem[LDS_ELEMS];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave - (wave / WN) * WN;
  // Tile order: each XCD takes a contiguous range of logical tiles, walked in
  // groups of GM M-tiles so the ~32 workgroups an XCD runs at once cover
  // GM A tiles x (32/GM) W tiles and reuse both from its L2.
  // Work units: whole-K tiles of the full row tiles first, then the rest:
  // with the residual epilogue and splits > 1, `splits` K-slices of each
  // tile from split_row0 on (a last partial round of whole tiles becomes a
  // full round of thin slices); otherwise the partial last row tile, whose
  // waves past M skip their MFMAs - these finish early, so they go last and
  // fill the CUs the full tiles leave free.
  constexpr int GM = 8;
  const int nTM = (c.M + BM - 1) / BM, nTN = c.N / BN;
  const bool ksplit = EPI == EPI_RESIDUAL && c.splits > 1;
  const int mainTM = ksplit ? c.split_row0 / BM : c.M / BM;
  const int n_main = mainTM * nTN;
  const bool tail = (int)blockIdx.x >= n_main;
  const int tailTM = nTM - mainTM;
  const int u = tail ? xcd_remap(blockIdx.x - n_main, gridDim.x - n_main)
                     : xcd_remap(blockIdx.x, n_main);
  const int split = tail ? u / (tailTM * nTN) : 0;
  const int t = tail ? u - split * (tailTM * nTN) : u;
  const int rTM = tail ? tailTM : mainTM;
  const int first_m = (t / (GM * nTN)) * GM;
  const int gsz = min(rTM - first_m, GM);
  const int tm = (tail ? mainTM : 0) + first_m + (t % (GM * nTN)) % gsz;
  const int tn = (t % (GM * nTN)) / gsz;
  // K steps of this unit (the slices of a tile differ by at most one 64-deep step)
  const int nkt = c.K / KB;
  const int k0 = ksplit && tail ? (int)((long)split * (c.K / BK) / c.splits) * (BK / KB) : 0;
  const int k1 = ksplit && tail ? (int)((long)(split + 1) * (c.K / BK) / c.splits) * (BK / KB) : nkt;
  const int m0 = tm * BM, n0 = tn * BN;

  // The lane that fills position (lane % CPR) of row RPI*i + lane/CPR of a
  // tile fetches the chunk that belongs there: position ^ lds_swz(row).
  const int lrow = lane / CPR, lpos = lane % CPR;
  const int kbase = k0 * KB;  // first K column of this unit
  // In a partial row tile (8-wave shapes; the 4-wave ones would need more
  // registers for the extra code paths) a wave skips the MFMAs of its rows
  // past M and the copies of A rows past M (they feed only output rows past
  // M); with two stages every later wait is for all of a wave's copies, so
  // only the first wait changes.
  constexpr bool CAN_SKIP = NST == 2 && !SPLIT && NW == 8;  // (W copies are never skipped)
  constexpr bool BIG2 = NW == 8 && BM == 256 && BN == 256 && XW == 0 && NST == 2;
  constexpr int CROSS = BIG2 ? 3 : 1;
  static_assert(CROSS != 3 || (XW == 0 && NST == 2), "the W-first crossing relies on waiting for every copy");
  bool alive[A_INS];
  const uint16_t* asrc[A_INS];
#pragma unroll
  for (int i = 0; i < A_INS; ++i) {
    alive[i] = m0 + (wave * A_INS + i) * RPI < c.M;
    const int gi = wave * A_INS + i;
    const int row = gi * RPI + lrow;
    const int lkc = lpos ^ lds_swz<KB>(row);
    const bool lo = SPLIT && row >= BM;
    const int gm = min(m0 + (lo ? row - BM : row), c.M - 1);
    asrc[i] = (lo ? c.A2 : c.A) + (size_t)gm * c.lda + kbase + lkc * 8;
  }
  const uint16_t* bsrc[B_INS];
#pragma unroll
  for (int i = 0; i < B_INS; ++i) {
    const int gi = wave * B_INS + i;
    const int lkc = lpos ^ lds_swz<KB>(gi * RPI + lrow);
    const int vc = n0 + gi * RPI + lrow;
    const int wr = EPI == EPI_SWIGLU ? swiglu_row<WTN>(vc, c.F) : EPI == EPI_QKV_HALF ? qkv_half_row(vc) : vc;
    bsrc[i] = c.W + (size_t)wr * c.ldw + kbase + lkc * 8;
  }

  // A wave's copies land in consecutive 1 KB blocks; groups of four share
  // one LDS base (M0) and differ in the instruction offset.
  auto stage_a = [&](int s) { return smem + s * A_STAGE; };
  auto stage_b = [&](int s) { return smem + NST * A_STAGE + s * B_STAGE; };
  auto issue_a = [&](int kt, int stage, auto skip_tag) {
    uint16_t* sA = stage_a(stage);
#pragma unroll
    for (int i = 0; i < A_INS; ++i)
      if (!decltype(skip_tag)::value || alive[i])
        dma16(asrc[i] + kt * KB - (i & 3) * 512, sA + (wave * A_INS + (i & ~3)) * 512, i & 3);
  };
  auto issue_b = [&](int kt, int stage) {
    uint16_t* sB = stage_b(stage);
#pragma unroll
    for (int i = 0; i < B_INS; ++i)
      dma16(bsrc[i] + kt * KB - (i & 3) * 512, sB + (wave * B_INS + (i & ~3)) * 512, i & 3);
  };

  f32x16 acc[FM][FN];
#pragma unroll
  for (int fm = 0; fm < FM; ++fm)
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[fm][fn][i] = 0.f;

  const int nk = k1 - k0;
  const int arow = wm * WTM + (lane & 31), brow = wn * WTN + (lane & 31);
  // swizzle of each fragment row this lane reads (fixed over the K loop)
  int aswz[FM], alswz[SPLIT ? FM : 1], bswz[FN];
#pragma unroll
  for (int fm = 0; fm < FM; ++fm) {
    const int r = arow + fm * 32;
    aswz[fm] = lds_swz<KB>(r);
    if constexpr (SPLIT) alswz[fm] = lds_swz<KB>(BM + r);
  }
#pragma unroll
  for (int fn = 0; fn < FN; ++fn) {
    const int r = brow + fn * 32;
    bswz[fn] = lds_swz<KB>(r);
  }
  constexpr int KS = KB / 16;
  static_assert(KS % 2 == 0, "fragment buffers alternate per step");
  typename A::v8 af[2][FM], bf[2][FN], al[2][SPLIT ? FM : 1];

  // The K loop for a wave whose first FMV of its FM 32-row blocks hold rows
  // below M (FMV = FM everywhere but in a partial last row tile): the other
  // blocks' fragment reads and MFMAs are skipped; the wave still issues its
  // share of the tile copies and meets every barrier.
  auto pipeline = [&](auto fmv_tag, auto skip_tag) {
  constexpr int FMV = decltype(fmv_tag)::value;
  constexpr bool SKIP = decltype(skip_tag)::value;
  constexpr int NR = FMV ? FMV + FN + (SPLIT ? FMV : 0) : 0;  // LDS fragment reads per 16-deep step
  constexpr int NM = FMV * FN * (SPLIT ? 2 : 1);              // MFMAs per step
  constexpr int RI = NR < NM ? NR : NM;                       // reads interleaved with MFMAs
  auto load_frags = [&](const uint16_t* sA, const uint16_t* sB, int ks, int buf) {
    if constexpr (FMV > 0) {
    const int kc = ks * 2 + (lane >> 5);
#pragma unroll
    for (int fm = 0; fm < FMV; ++fm)
      af[buf][fm] = A::frag(*reinterpret_cast<const uint4*>(
          sA + (arow + fm * 32) * KB + ((kc ^ aswz[fm]) << 3)));
#pragma unroll
    for (int fn = 0; fn < FN; ++fn)
      bf[buf][fn] = A::frag(*reinterpret_cast<const uint4*>(
          sB + (brow + fn * 32) * KB + ((kc ^ bswz[fn]) << 3)));
    if constexpr (SPLIT) {
#pragma unroll
      for (int fm = 0; fm < FMV; ++fm)
        al[buf][fm] = A::frag(*reinterpret_cast<const uint4*>(
            sA + (BM + arow + fm * 32) * KB + ((kc ^ alswz[fm]) << 3)));
    }
    }
  };
  // (EPI_LMSTATS: operands swapped, so that a lane holds one row and many ids)
  auto mma1 = [&](const typename A::v8& a, const typename A::v8& b, const f32x16& cc) {
    if constexpr (EPI == EPI_LMSTATS) return A::mma(b, a, cc);
    else return A::mma(a, b, cc);
  };
  auto mfmas = [&](int buf) {
#pragma unroll
    for (int fm = 0; fm < FMV; ++fm)
#pragma unroll
      for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = mma1(af[buf][fm], bf[buf][fn], acc[fm][fn]);
    if constexpr (SPLIT) {
#pragma unroll
      for (int fm = 0; fm < FMV; ++fm)
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) acc[fm][fn] = mma1(al[buf][fm], bf[buf][fn], acc[fm][fn]);
    }
  };
  // steps 0..KS-2 of a tile: the reads of step ks+1 go between the MFMAs of ks
  auto inner_steps = [&](const uint16_t* sA, const uint16_t* sB) {
#pragma unroll
    for (int ks = 0; ks + 1 < KS; ++ks) {
      load_frags(sA, sB, ks + 1, (ks + 1) & 1);
      mfmas(ks & 1);
    }
    if constexpr (NR > 0) {
#pragma unroll
    for (int ks = 0; ks + 1 < KS; ++ks) {
#pragma unroll
      for (int r = 0; r < RI; ++r) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
      }
      if (NR > RI) __builtin_amdgcn_sched_group_barrier(0x100, NR - RI, 0);
      if (NM > RI) __builtin_amdgcn_sched_group_barrier(0x008, NM - RI, 0);
    }
    }
  };

  // Pipeline over NST LDS stages: K tile t sits in stage t % NST and its DMA
  // is issued NST tiles ahead.  Crossing from tile t to t+1, each wave (1)
  // waits for its copies of tile t+1 (the NST-2 later tiles may still be in
  // flight), (2) meets the others at the barrier - after which every wave
  // has read all of tile t, (3) issues the first fragment reads of tile t+1
  // and tile t+NST's copy into tile t's stage, and (4) runs the last MFMAs
  // of tile t, which cover the latency of those reads.  The order of the
  // reads, the copies and the MFMAs at that crossing (CROSS) is measured per
  // tile against copies-then-reads: 1 = reads, copies, MFMAs (544-row
  // gate/up 112 -> 100 us); 3 = W copy, reads, A copy, MFMAs for the
  // two-stage 8-wave 256x256 tile (8704 rows, runs alternating with 1:
  // gate/up 1359 -> 1339 us, QKV 724 -> 711 us, down 713 -> 702 us).  3 needs the wait for every copy of
  // the two-stage tile: with a third W stage the waits count on A copies
  // being issued before W copies at each crossing.  Tiles past
  // the end are refetches of the last one, which keeps the wait counts fixed.
  // With XW extra W stages the crossing issues the A copy of tile t+2 and the
  // W copy of tile t+2+XW, and the copies are ordered so that one wait for
  // all but the last W copies covers both operands of tile t+1: A0, W0..WXW,
  // A1, W(XW+1) up front, then A(t+2) W(t+2+XW) per crossing (copies
  // complete in issue order).
  auto kclamp = [&](int k) { return k < nk ? k : nk - 1; };
  if constexpr (XW == 0) {
#pragma unroll
    for (int s0 = 0; s0 < NST; ++s0) {
      issue_a(kclamp(s0), s0, skip_tag);
      issue_b(kclamp(s0), s0);
    }
  } else {
    issue_a(0, 0, skip_tag);
#pragma unroll
    for (int s0 = 0; s0 <= XW; ++s0) issue_b(kclamp(s0), s0);
    issue_a(kclamp(1), 1, skip_tag);
    issue_b(kclamp(XW + 1), XW + 1);
  }
  // (a wave that may have skipped copies has fewer in flight: it waits for all)
  if constexpr (SKIP) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  else if constexpr (XW == 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 1) * INS) : "memory");
  else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(A_INS + (XW + 1) * B_INS) : "memory");
  __syncthreads();
  load_frags(stage_a(0), stage_b(0), 0, 0);
  int ca = 0, cb = 0;  // stages of tile kt
  for (int kt = 0; kt + 1 < nk; ++kt) {
    inner_steps(stage_a(ca), stage_b(cb));
    if constexpr (XW == 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 2) * INS) : "memory");
    else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(B_INS) : "memory");
    __syncthreads();
    const int na = ca + 1 == NST ? 0 : ca + 1, nb = cb + 1 == NSB ? 0 : cb + 1;
    if constexpr (CROSS == 3) issue_b(kclamp(kt + NSB), cb);
    load_frags(stage_a(na), stage_b(nb), 0, 0);
    if constexpr (CROSS == 1) issue_a(kclamp(kt + NST), ca, skip_tag);
    if constexpr (CROSS == 1) issue_b(kclamp(kt + NSB), cb);
    if constexpr (CROSS == 3) issue_a(kclamp(kt + NST), ca, skip_tag);
    mfmas((KS - 1) & 1);
    if constexpr (NR > 0) {
      __builtin_amdgcn_sched_group_barrier(0x100, NR, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, NM, 0);
    }
    ca = na;
    cb = nb;
  }
  inner_steps(stage_a(ca), stage_b(cb));
  mfmas((KS - 1) & 1);
  };  // pipeline

  using Full = std::integral_constant<int, FM>;
  using Keep = std::false_type;
  const int vrows = c.M - (m0 + wm * WTM);  // rows of this wave's tile below M
  if constexpr (CAN_SKIP) {
    using Skip = std::true_type;
    if (m0 + BM <= c.M) pipeline(Full{}, Keep{});
    else if (vrows <= 0) pipeline(std::integral_constant<int, 0>{}, Skip{});
    else if (FM > 1 && vrows <= 32) pipeline(std::integral_constant<int, 1>{}, Skip{});
    else pipeline(Full{}, Skip{});
  } else {
    pipeline(Full{}, Keep{});
  }
  // the refetch issued last may still be landing: finish it before the
  // epilogue reuses LDS
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();

  const int rowb = m0 + wm * WTM, colb = n0 + wn * WTN;
  if constexpr (EPI == EPI_RESIDUAL) {
    // a wave's LDS region holds one 32-row fp32 block of its tile; the batched x
    // loads need 64 registers beside the accumulators of at most 8 MFMA blocks
    static_assert(NW * 32 * WTN * 2 <= LDS_ELEMS && FM * FN <= 8, "residual staging");
    float* ws = reinterpret_cast<float*>(smem + wave * (32 * WTN * 2));
    if (!(ksplit && tail) && rowb + WTM <= c.M) {
      const int rbu = __builtin_amdgcn_readfirstlane(rowb), cbu = __builtin_amdgcn_readfirstlane(colb);
      epi_residual_full<FM, FN>(acc, lane, ws, c.outf + (size_t)rbu * c.ldc + cbu, c.ldc);
    } else if (!(ksplit && tail)) {
      epi_rows16<FM, FN>(acc, lane, ws, [&](int lr, int lc, float4 v) {
        const int row = rowb + lr;
        if (row >= c.M) return;
        float4* dst = reinterpret_cast<float4*>(c.outf + (size_t)row * c.ldc + colb + lc);
        float4 x = *dst;
        x.x += v.x; x.y += v.y; x.z += v.z; x.w += v.w;
        *dst = x;
      });
    } else {
      // K-slice `split` of a tile from split_row0 on: fp32 partial
      // part[split][m - split_row0][n] (row stride N), summed into x later
      const size_t mt = (size_t)(c.M - c.split_row0);
      epi_rows16<FM, FN>(acc, lane, ws, [&](int lr, int lc, float4 v) {
        const int row = rowb + lr;
        if (row >= c.M) return;
        *reinterpret_cast<float4*>(c.part + (split * mt + (row - c.split_row0)) * c.N + colb + lc) = v;
      });
    }
  }
  else if constexpr (EPI == EPI_STORE_F32 || EPI == EPI_LOGITS) epi_store<FM, FN>(c, acc, rowb, colb, lane);
  else if constexpr (EPI == EPI_SWIGLU) epi_swiglu<A, FM, FN>(c, acc, rowb, colb, lane);
  else if constexpr (EPI == EPI_QKV_ROPE || EPI == EPI_QKV_HALF) {
    constexpr int HR = EPI == EPI_QKV_HALF ? 2 : 1;
    // each wave stages its WTM x WTN tile in its own LDS region
    static_assert(BM * BN <= LDS_ELEMS, "QKV staging fits the pipeline LDS");
    if (c.geom.T >= WTM) epi_qkv_rope<A, FM, FN, true, HR>(c, acc, rowb, colb, lane, smem + wave * (WTM * WTN));
    else epi_qkv_rope<A, FM, FN, false, HR>(c, acc, rowb, colb, lane, smem + wave * (WTM * WTN));
  }
  else epi_lmstats<BM, WM, WN, FM, FN>(c, acc, m0, tn, colb, lane, wm, wn, smem);
}

// A tile shape: BM x BN by WM x WN waves, NST stages of KB-deep K steps (xw more
// for W), occ workgroups per CU, and its measured times in microseconds: a unit
// of n 64-deep K steps takes fix + n * (lat + (load + cold / r) * u), u the share
// of the chip's 256 workgroup slots in use (what the copies share) or, where a CU
// holds several, of the fullest CU's, and r the row tiles that read each W strip
// (one of them from HBM).
struct TileCfg {
  int BM, BN, WM, WN, KB, NST, occ, xw;
  float fix, lat, load, cold;
};

// fix / lat / load / cold: least squares over 119 shapes (24-8704 rows, N
// 256-24576, K 256-12288, both types, weights from HBM), LM head tiles over 11
// (16-1024 rows x 4096-126464 ids).  On gate/up products the model is within 4-12%
// rms per tile where the tile is competitive (18% for the smallest), and the plans
// are 1.7% behind the fastest measured choice on those shapes and 2.4% on 478 others
// in the mean.  RoPE at sequence lengths that are not a multiple of 8 takes 15-35%
// longer than modelled on every tile (v^T leaves in 2-byte stores), so it moves no
// choice much.  What each shape is for:
//  - few units, bound by the latency of the copies: small tiles that keep many
//    stages in flight (entries 8-12; 64 rows x 24576 x 4096 58 -> 45 us, 128 x
//    17408 x 3072 62 -> 37, 32 x 256 x 704 9.5 -> 5.9)
//  - many units: 256x256, or the 192-row tiles where those round better (1444 x
//    24576 x 4096 316 -> 272 us, 870 x 12288 x 4096 102 -> 93)
//  - a third W stage (xw): the weights of few row tiles come from HBM, not L2
constexpr TileCfg kTiles[] = {
    {128, 128, 2, 2, 64, 2, 2, 0, 0.57f, 0.587f, 0.401f, 0.117f},  // 0
    {32, 256, 1, 4, 64, 2, 2, 0, 0.40f, 1.037f, 0.247f, 0.000f},  // 1: LM head
    {256, 256, 4, 2, 64, 2, 1, 0, 4.58f, 1.130f, 0.415f, 0.000f},  // 2
    {256, 256, 4, 2, 64, 2, 1, 1, 5.07f, 1.041f, 0.521f, 0.000f},  // 3
    {128, 256, 4, 2, 64, 3, 1, 0, 3.51f, 0.686f, 0.243f, 0.159f},  // 4
    {128, 256, 4, 2, 64, 2, 1, 1, 2.57f, 0.770f, 0.160f, 0.105f},  // 5
    {128, 256, 2, 4, 64, 2, 1, 0, 3.07f, 1.379f, 0.379f, 0.000f},  // 6: LM head
    {256, 256, 4, 2, 32, 3, 1, 0, 9.45f, 1.309f, 1.628f, 0.000f},  // 7: LM head
    {64, 64, 2, 1, 64, 6, 1, 0, 1.58f, 0.245f, 0.036f, 0.095f},  // 8
    {64, 128, 2, 2, 64, 4, 1, 0, 1.48f, 0.335f, 0.049f, 0.271f},  // 9
    {32, 64, 1, 1, 64, 6, 1, 0, 1.63f, 0.169f, 0.000f, 0.287f},  // 10
    {64, 128, 2, 2, 64, 3, 2, 0, 0.90f, 0.158f, 0.526f, 0.000f},  // 11
    {128, 128, 4, 2, 64, 4, 1, 0, 2.08f, 0.397f, 0.182f, 0.139f},  // 12
    {128, 128, 4, 1, 64, 2, 2, 0, 0.50f, 0.700f, 0.312f, 0.002f},  // 13
    {192, 256, 2, 4, 64, 2, 1, 1, 4.08f, 0.870f, 0.376f, 0.000f},  // 14
    {192, 128, 2, 2, 64, 2, 2, 0, 1.50f, 0.611f, 0.760f, 0.000f},  // 15
    {256, 256, 2, 4, 64, 2, 1, 0, 6.57f, 1.116f, 0.450f, 0.000f},  // 16: QKV of 64-wide heads
};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);

// Which epilogues each tile is built for.  The LM-head epilogues double the A
// tile (hi and lo parts): with 64-deep stages that fits LDS only for BM <= 128,
// the 256-row tile takes 32-deep ones (per MFMA it moves a quarter less than a
// plain 256x256 tile: 1024 rows x 126464 ids 1688 -> 1561 us against 128x256,
// 836 rows 1486 -> 1532), and 32 rows two per CU serve few rows (32 x 126464
// 168 us against 229).  RoPE needs a wave to own one head or half of a 128-wide
// one (checked per call); the 256x256 tile with 64-wide wave tiles serves only it.
constexpr bool tile_epi(int BM, int BN, int WM, int WN, int KB, int EPI) {
  const int WTN = BN / WN;
  if ((BM == 32 && BN == 256) || (BM == 128 && BN == 256 && WM == 2))
    return EPI == EPI_LMSTATS || EPI == EPI_LOGITS;
  if (KB == 32) return EPI == EPI_LMSTATS;
  if (EPI == EPI_LMSTATS || EPI == EPI_LOGITS) return false;
  if (EPI == EPI_QKV_ROPE) return WTN == 64 || WTN == 128;
  if (EPI == EPI_QKV_HALF) return WTN == 64;
  return !(BM == 256 && WN == 4);
}

bool tile_ok(const GemmCall& c, const TileCfg& t) {
  // (N in whole 128-column tiles whatever the tile: the 64-wide ones choose
  // among the same shapes)
  if (c.N % std::max(t.BN, 128) || c.K % BK) return false;
  if (!tile_epi(t.BM, t.BN, t.WM, t.WN, t.KB, c.epi)) return false;
  const int WTN = t.BN / t.WN;
  // (RoPE: heads in pairs, like the 128-column rule)
  if (c.epi == EPI_QKV_ROPE) {
    const int d = c.rope.H * c.rope.hd;
    return (WTN == c.rope.hd || WTN * 2 == c.rope.hd) && d % t.BN == 0 && d % (2 * c.rope.hd) == 0;
  }
  if (c.epi == EPI_SWIGLU) return (c.F % (WTN / 2)) == 0;
  return true;
}

int env_int(const char* name, int dflt) {
  const char* e = std::getenv(name);
  return e ? std::atoi(e) : dflt;
}

// Launch overhead (us), the rate weights stream from HBM (bytes/us), and what
// split-K partials cost: bytes/us over their write in the GEMM (about 5.5) and
// their read in the norm kernel that adds them (about 4.2), and a fixed time.
constexpr double kLaunchUs = 2.2, kWRate = 5.6e6, kPartRate = 2.4e6, kPartUs = 1.3;

double unit_us(const GemmCall& c, const TileCfg& t, double ksteps, double units) {
  const double cu = t.occ > 1 ? std::ceil(units / 256.0) : units / 256.0;
  const double u = std::min(1.0, cu / t.occ), r = (c.M + t.BM - 1) / t.BM;
  return t.fix + ksteps * (t.lat + (t.load + t.cold / r) * u);
}

// Time of n_main units of length T followed by n_units units of length U on the 8
// workgroup slots per `occ` of one shader engine, each started on the slot that
// frees first.
double engine_makespan(long n_main, double T, long n_units, double U, long slots) {
  const long R = n_main / slots, r = n_main % slots;
  const double main_end = (R + (r ? 1 : 0)) * T;
  if (n_units == 0) return main_end;
  const long early = slots - r;  // slots free at R*T; the other r at (R+1)*T
  double best = 0;
  for (long j = 1;; ++j) {
    const double X = R * T + j * U;
    const long late = r ? (long)std::floor(std::max(0.0, (X - (R + 1) * T) / U) + 1e-9) : 0;
    if (early * j + r * late >= n_units) { best = X; break; }
  }
  if (r) {
    for (long j = 1;; ++j) {
      const double X = (R + 1) * T + j * U;
      if (X >= best) break;
      const long e = (long)std::floor((X - R * T) / U + 1e-9);
      if (early * e + r * j >= n_units) { best = X; break; }
    }
  }
  return std::max(main_end, best);
}

// Time of the partial last row tile (rem = M mod BM rows) relative to a full
// one.  8-wave two-stage shapes skip the MFMAs of rows past M per wave (the
// kernel's rule: a wave keeps all its 32-row blocks, only the first, or none), so
// the busiest SIMD's remaining share, at least kPartialFloor, sets two thirds of the
// time; the W copies and the barriers stay (192-row tiles with 96 and 128 rows, half
// and two thirds of the MFMAs, ran 0.66 and 0.78 of a full tile beside full ones).
// A tile alone on its CU still waits for its copies, kPartialLat of an idle chip's
// time.  Other shapes: a full tile.
constexpr double kPartialFloor = 0.3, kPartialLat = 0.75;
double partial_share(const GemmCall& c, const TileCfg& t, int rem) {
  const bool lm = c.epi == EPI_LMSTATS || c.epi == EPI_LOGITS;
  if (rem == 0) return 0.0;
  if (lm || t.WM * t.WN != 8 || t.NST != 2) return 1.0;  // (xw tiles skip too)
  const int WTM = t.BM / t.WM, FM = WTM / 32;
  double load[4] = {0, 0, 0, 0};
  for (int w = 0; w < 8; ++w) {
    const int v = rem - (w / t.WN) * WTM;
    const int fmv = v <= 0 ? 0 : (FM > 1 && v <= 32 ? 1 : FM);
    load[w % 4] += (double)fmv / FM;
  }
  const double busiest = std::max(std::max(load[0], load[1]), std::max(load[2], load[3])) / 2.0;
  return (1.0 + 2.0 * std::max(busiest, kPartialFloor)) / 3.0;
}

// Time of the partial last row tile's unit next to full ones of time T.
double partial_us(const GemmCall& c, const TileCfg& t, double ksteps, double T) {
  return std::max(partial_share(c, t, c.M % t.BM) * T, kPartialLat * (t.fix + ksteps * t.lat));
}

// Estimated time (us) of whole-K tiles: rounds of 256 * occ units, then what is
// left and the partial last row tile at their own load; never less than reading W
// once.
double tile_time(const GemmCall& c, const TileCfg& t) {
  const long nTN = c.N / t.BN, slots = 256L * t.occ;
  const double ks = c.K / BK;
  const long n_full = (c.M / t.BM) * nTN, n_part = c.M % t.BM ? nTN : 0;
  const long rounds = n_full / slots, rest = n_full % slots;
  double time = rounds * unit_us(c, t, ks, slots);
  if (rest + n_part) {
    const double T = unit_us(c, t, ks, rest + n_part);
    time += dispatch_makespan(rest, T, n_part, n_part ? partial_us(c, t, ks, T) : T, t.occ);
  }
  return std::max(kLaunchUs + time, 2.0 + 2.0 * c.N * (double)c.K / kWRate);
}

// Residual GEMM whose last tail_tm > 0 row tiles are computed as `splits` K-slices
// that write fp32 partials for the next norm kernel; HUGE_VAL if this, and so more
// slices too, cannot take less than `limit` (an even spread of the units over the
// slots, which grows with the slices, already does not).
double residual_time(const GemmCall& c, const TileCfg& t, int nTM, int nTN, int tail_tm, int splits, double limit) {
  const long n_main = (long)(nTM - tail_tm) * nTN, n_slices = (long)tail_tm * nTN * splits;
  const double ks = (double)c.K / BK, tail_rows = c.M - (double)(nTM - tail_tm) * t.BM;
  const double rest = kLaunchUs + kPartUs + splits * tail_rows * c.N * (4.0 / kPartRate);
  const double T = unit_us(c, t, ks, n_main + n_slices), U = t.fix + (T - t.fix) / splits;
  if (rest + (n_main * T + n_slices * U) / (256 * t.occ) >= limit) return HUGE_VAL;
  // (a partial row tile's slices count as whole ones: the renumbering of a split
  // tail's units spreads them among the others)
  return rest + dispatch_makespan(n_main, T, n_slices, U, t.occ);
}

// Plans of the calls seen last, by the values that decide them: working one out takes
// 1-2 us of host time (3-16 with the slices of a residual call), finding it 0.1.
struct PlanEntry {
  int epi, M, N, K, p0, p1;  // p0, p1: heads and head size (RoPE), F (SwiGLU)
  size_t part_elems;         // (residual)
  int tile, splits, split_row0;  // tile: index + 1, 0 = none fits
  bool same(const PlanEntry& o) const {
    return epi == o.epi && M == o.M && N == o.N && K == o.K && p0 == o.p0 && p1 == o.p1 &&
           part_elems == o.part_elems;
  }
};
constexpr int kMaxPlans = 64;
std::mutex g_plan_mu;
PlanEntry g_plans[kMaxPlans];
int g_n_plans = 0, g_next_plan = 0;  // (the oldest makes room)

PlanEntry plan_key(const GemmCall& c, size_t part_elems) {
  PlanEntry e{c.epi, c.M, c.N, c.K, 0, 0, part_elems, 0, 1, c.M};
  if (c.epi == EPI_QKV_ROPE) { e.p0 = c.rope.H; e.p1 = c.rope.hd; }
  if (c.epi == EPI_SWIGLU) e.p0 = c.F;
  return e;
}

bool find_plan(PlanEntry& e) {
  std::lock_guard<std::mutex> lk(g_plan_mu);
  for (int i = 0; i < g_n_plans; ++i)
    if (g_plans[i].same(e)) { e = g_plans[i]; return true; }
  return false;
}

void keep_plan(const PlanEntry& e) {
  std::lock_guard<std::mutex> lk(g_plan_mu);
  g_plans[g_next_plan] = e;
  g_next_plan = (g_next_plan + 1) % kMaxPlans;
  g_n_plans = std::min(g_n_plans + 1, kMaxPlans);
}

int pick_tile(const GemmCall& c) {
  const int f = env_int("WINO_GEMM_TILE", -1);
  if (f >= 0 && f < kNumTiles && tile_ok(c, kTiles[f])) return f;
  PlanEntry e = plan_key(c, 0);
  if (find_plan(e)) return e.tile - 1;
  double best_t = 0;
  for (int i = 0; i < kNumTiles; ++i) {
    if (!tile_ok(c, kTiles[i])) continue;
    const double time = tile_time(c, kTiles[i]);
    if (e.tile == 0 || time < best_t) { e.tile = i + 1; best_t = time; }
  }
  keep_plan(e);
  return e.tile - 1;
}

template <int BM, int BN, int WM, int WN, int EPI, int KB, int NST, int OCC, int XW, class A>
hipError_t launch_one(const GemmCall& c, hipStream_t st) {
  constexpr bool split = EPI == EPI_LMSTATS || EPI == EPI_LOGITS;
  constexpr int arows = split ? 2 * BM : BM;
  constexpr int lds = (NST * arows + (NST + XW) * BN) * KB * 2;
  constexpr bool qkv_fits = (EPI != EPI_QKV_ROPE && EPI != EPI_QKV_HALF) || BM * BN * 2 <= lds;
  if constexpr (tile_epi(BM, BN, WM, WN, KB, EPI)) {
    static_assert(lds * OCC <= 160 * 1024 && qkv_fits && (XW == 0 || !split), "tile fits LDS");
    const int nTM = (c.M + BM - 1) / BM, nTN = c.N / BN;
    int units = nTM * nTN;
    if (EPI == EPI_RESIDUAL && c.splits > 1) {
      const int mainTM = c.split_row0 / BM;
      units = mainTM * nTN + (nTM - mainTM) * nTN * c.splits;
    }
    gemm_kernel<BM, BN, WM, WN, EPI, KB, NST, OCC, XW, A><<<dim3(units), dim3(WM * WN * 64), 0, st>>>(c);
    return hipGetLastError();
  } else {
    return hipErrorInvalidValue;
  }
}

template <int BM, int BN, int WM, int WN, int KB, int NST, int OCC, int XW, class A>
hipError_t launch_cfg_t(const GemmCall& c, hipStream_t st) {
  switch (c.epi) {
    case EPI_QKV_ROPE:
      if (c.rope.hd == 2 * (BN / WN)) return launch_one<BM, BN, WM, WN, EPI_QKV_HALF, KB, NST, OCC, XW, A>(c, st);
      return launch_one<BM, BN, WM, WN, EPI_QKV_ROPE, KB, NST, OCC, XW, A>(c, st);
    case EPI_QKV_HALF: break;  // (chosen above)
    case EPI_RESIDUAL: return launch_one<BM, BN, WM, WN, EPI_RESIDUAL, KB, NST, OCC, XW, A>(c, st);
    case EPI_SWIGLU: return launch_one<BM, BN, WM, WN, EPI_SWIGLU, KB, NST, OCC, XW, A>(c, st);
    case EPI_LMSTATS: return launch_one<BM, BN, WM, WN, EPI_LMSTATS, KB, NST, OCC, XW, A>(c, st);
    case EPI_STORE_F32: return launch_one<BM, BN, WM, WN, EPI_STORE_F32, KB, NST, OCC, XW, A>(c, st);
    case EPI_LOGITS: return launch_one<BM, BN, WM, WN, EPI_LOGITS, KB, NST, OCC, XW, A>(c, st);
  }
  return hipErrorInvalidValue;
}

template <int BM, int BN, int WM, int WN, int KB, int NST, int OCC, int XW = 0>
hipError_t launch_cfg(const GemmCall& c, hipStream_t st) {
  return c.f16 ? launch_cfg_t<BM, BN, WM, WN, KB, NST, OCC, XW, ActF16>(c, st)
               : launch_cfg_t<BM, BN, WM, WN, KB, NST, OCC, XW, ActBf16>(c, st);
}

}  // namespace

// Workgroups go to the 32 shader engines (8 XCDs of 4, 8 CUs each) in turn, in
// launch order, and wait there for a slot while another engine may have free ones.
// Units just over a round therefore cost a whole further unit (192x256 tiles, K =
// 2560: 240 units 55 us, 240 and 30 partial ones of 16 rows 75, where slots shared
// by the whole chip would give 55; planned so, 1620 x 7680 x 2560 took 108 us and
// 1800 x 3328 x 8640 168, in the tiles chosen now 82 and 129).
double dispatch_makespan(long n_main, double T, long n_units, double U, int occ) {
  constexpr long E = 32;
  double end = 0;
  // an engine's counts change at engines n_main and n_main + n_units (mod 32)
  for (const long e : {0L, n_main % E, (n_main + n_units) % E}) {
    const long m = (n_main - e + E - 1) / E, all = (n_main + n_units - e + E - 1) / E;
    end = std::max(end, engine_makespan(m, T, all - m, U, 8L * occ));
  }
  return end;
}

void plan_residual_gemm(GemmCall& c, size_t part_elems) {
  const int f_tile = env_int("WINO_GEMM_TILE", -1);
  const int f_split = env_int("WINO_GEMM_SPLIT", 0), f_tail = env_int("WINO_GEMM_TAIL", -1);
  const bool forced = f_tile >= 0 || f_split > 0 || f_tail >= 0;
  c.epi = EPI_RESIDUAL;
  PlanEntry e = plan_key(c, part_elems);
  if (!forced && find_plan(e)) {
    c.tile = e.tile; c.splits = e.splits; c.split_row0 = e.split_row0;
    return;
  }
  const int nk = c.K / BK;
  int best = -1, best_s = 1, best_tail = 0;
  double best_t = HUGE_VAL;
  auto consider = [&](int i, int tail, int splits, double time) {
    if (time < best_t) { best = i; best_t = time; best_s = splits; best_tail = tail; }
  };
  // whole-K tiles and the split of every row tile first: they bound the rest
  for (const bool some : {false, true})
    for (int i = 0; i < kNumTiles; ++i) {
      const TileCfg& t = kTiles[i];
      if (!tile_ok(c, t) || (f_tile >= 0 && i != f_tile)) continue;
      const int nTM = (c.M + t.BM - 1) / t.BM, nTN = c.N / t.BN;
      if (!some && (f_tail < 0 || f_tail == 0)) consider(i, 0, 1, tile_time(c, t));
      // (a few trailing row tiles, or all)
      for (int tail = some ? 1 : nTM; tail <= (some ? std::min(8, nTM - 1) : nTM); ++tail) {
        if (f_tail >= 0 && tail != std::min(f_tail, nTM)) continue;
        const double tail_rows = c.M - (double)(nTM - tail) * t.BM;
        // (with five and seven slices 52 of 1048 plans changed, GEMM and norm together
        // by 1% in the mean, 16 of them slower; not worth two more instances of each
        // norm kernel - 544 x 4096 x 12288: 72.9 us with three, 71.8 with five)
        for (const int s : {2, 3, 4, 6, 8}) {
          if (nk / s < 4 || s * tail_rows * c.N > (double)part_elems) break;
          if (f_split > 0 && s != f_split) continue;
          const double time = residual_time(c, t, nTM, nTN, tail, s, best_t);
          if (time == HUGE_VAL) break;
          consider(i, tail, s, time);
        }
      }
    }
  if (best < 0) {  // no candidate under the overrides (or at all): whole-K tiles
    c.tile = 0; c.splits = 1; c.split_row0 = c.M;
    return;
  }
  const int nTM = (c.M + kTiles[best].BM - 1) / kTiles[best].BM;
  c.tile = best + 1;
  c.splits = best_tail ? best_s : 1;
  c.split_row0 = best_tail ? (nTM - best_tail) * kTiles[best].BM : c.M;
  if (!forced) {
    e.tile = c.tile; e.splits = c.splits; e.split_row0 = c.split_row0;
    keep_plan(e);
  }
}

int gemm_tile_n(const GemmCall& c) {
  const int i = pick_tile(c);
  return i < 0 ? 0 : kTiles[i].BN;
}

hipError_t launch_gemm(const GemmCall& c, hipStream_t st) {
  const int i = (c.tile > 0 && c.tile <= kNumTiles) ? c.tile - 1 : pick_tile(c);
  if (i < 0 || !tile_ok(c, kTiles[i])) return hipErrorInvalidValue;
  if (c.M <= 0) return hipSuccess;
  if (c.epi == EPI_RESIDUAL && c.splits > 1) {
    const int nk = c.K / BK;
    if (!c.part || c.split_row0 < 0 || c.split_row0 >= c.M || c.split_row0 % kTiles[i].BM ||
        nk < c.splits)
      return hipErrorInvalidValue;
  }
  switch (i) {
    case 0: return launch_cfg<128, 128, 2, 2, 64, 2, 2>(c, st);
    case 1: return launch_cfg<32, 256, 1, 4, 64, 2, 2>(c, st);
    case 2: return launch_cfg<256, 256, 4, 2, 64, 2, 1>(c, st);
    case 3: return launch_cfg<256, 256, 4, 2, 64, 2, 1, 1>(c, st);
    case 4: return launch_cfg<128, 256, 4, 2, 64, 3, 1>(c, st);
    case 5: return launch_cfg<128, 256, 4, 2, 64, 2, 1, 1>(c, st);
    case 6: return launch_cfg<128, 256, 2, 4, 64, 2, 1>(c, st);
    case 7: return launch_cfg<256, 256, 4, 2, 32, 3, 1>(c, st);
    case 8: return launch_cfg<64, 64, 2, 1, 64, 6, 1>(c, st);
    case 9: return launch_cfg<64, 128, 2, 2, 64, 4, 1>(c, st);
    case 10: return launch_cfg<32, 64, 1, 1, 64, 6, 1>(c, st);
    case 11: return launch_cfg<64, 128, 2, 2, 64, 3, 2>(c, st);
    case 12: return launch_cfg<128, 128, 4, 2, 64, 4, 1>(c, st);
    case 13: return launch_cfg<128, 128, 4, 1, 64, 2, 2>(c, st);
    case 14: return launch_cfg<192, 256, 2, 4, 64, 2, 1, 1>(c, st);
    case 15: return launch_cfg<192, 128, 2, 2, 64, 2, 2>(c, st);
    case 16: return launch_cfg<256, 256, 2, 4, 64, 2, 1>(c, st);
  }
  return hipErrorInvalidValue;
}

}  // namespace wino
