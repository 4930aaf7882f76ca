// Embedding gather and RMSNorm kernels: one workgroup per row, the row held in
// registers (16-byte chunks of 8 elements per thread) so that all its loads -
// the row, every split-K partial, the gain - are in flight at once; fp32 sum of
// squares; output in the activation type A (bf16 or fp16) rounded to nearest
// even.  Gains and the embedding table are bf16 weights.
#include <algorithm>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace wino {

namespace {

// A row's 8-element chunks held by a workgroup of NT threads, CPT per thread
// (chunk c * NT + tid; chunks past d hold zeros): sum of squares over the
// workgroup, then the normed row in 16-byte stores (and its rounding remainder
// to out_lo, if given).
template <class A, int NT, int CPT>
__device__ __forceinline__ void row_norm_store(float (&v)[CPT][8], const uint4 (&graw)[CPT], float eps, int d,
                                               uint16_t* out, uint16_t* out_lo = nullptr) {
  __shared__ float red[NT / 64];
  const int tid = threadIdx.x, nch = d >> 3;
  float ss = 0.f;
#pragma unroll
  for (int c = 0; c < CPT; ++c)
#pragma unroll
    for (int e = 0; e < 8; ++e) ss += v[c][e] * v[c][e];
  ss = valu_sum(ss);
  if constexpr (NT > 64) {
    if ((tid & 63) == 0) red[tid >> 6] = ss;
    __syncthreads();
    if constexpr (NT == 128) ss = red[0] + red[1];
    else ss = (red[0] + red[1]) + (red[2] + red[3]);
  }
  const float rs = rsqrtf(ss / (float)d + eps);
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int ch = c * NT + tid;
    if (ch >= nch) continue;
    const uint16_t* gp = reinterpret_cast<const uint16_t*>(&graw[c]);
    float y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = v[c][e] * rs * bf2f(gp[e]);
    uint4 o;
    uint32_t* op = reinterpret_cast<uint32_t*>(&o);
#pragma unroll
    for (int e = 0; e < 4; ++e) op[e] = A::pack2(y[2 * e], y[2 * e + 1]);
    *reinterpret_cast<uint4*>(out + ch * 8) = o;
    if (out_lo) {
      const uint16_t* hi = reinterpret_cast<const uint16_t*>(&o);
      uint4 lo;
      uint32_t* lp = reinterpret_cast<uint32_t*>(&lo);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        lp[e] = A::pack2(y[2 * e] - A::val(hi[2 * e]), y[2 * e + 1] - A::val(hi[2 * e + 1]));
      *reinterpret_cast<uint4*>(out_lo + ch * 8) = lo;
    }
  }
}

// Gain chunks of a row (zeros past d).
template <int NT, int CPT>
__device__ __forceinline__ void load_gain(const uint16_t* gain, int d, uint4 (&graw)[CPT]) {
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int ch = c * NT + (int)threadIdx.x;
    graw[c] = ch < (d >> 3) ? *reinterpret_cast<const uint4*>(gain + ch * 8) : make_uint4(0, 0, 0, 0);
  }
}

// fp32 row chunks (zeros past d).
template <int NT, int CPT>
__device__ __forceinline__ void load_row(const float* xr, int d, float (&v)[CPT][8]) {
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int ch = c * NT + (int)threadIdx.x;
    float4 a = make_float4(0, 0, 0, 0), b = a;
    if (ch < (d >> 3)) {
      const float4* xi = reinterpret_cast<const float4*>(xr + ch * 8);
      a = xi[0];
      b = xi[1];
    }
    v[c][0] = a.x; v[c][1] = a.y; v[c][2] = a.z; v[c][3] = a.w;
    v[c][4] = b.x; v[c][5] = b.y; v[c][6] = b.z; v[c][7] = b.w;
  }
}

template <int NT, int CPT>
__device__ __forceinline__ void store_row(float* xr, int d, const float (&v)[CPT][8]) {
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int ch = c * NT + (int)threadIdx.x;
    if (ch >= (d >> 3)) continue;
    float4* xo = reinterpret_cast<float4*>(xr + ch * 8);
    xo[0] = make_float4(v[c][0], v[c][1], v[c][2], v[c][3]);
    xo[1] = make_float4(v[c][4], v[c][5], v[c][6], v[c][7]);
  }
}

template <class A, int NT, int CPT>
__global__ __launch_bounds__(NT) void embed_norm_kernel(StepGeom g, const int32_t* __restrict__ tokens,
                                                        const uint16_t* __restrict__ emb, int vocab,
                                                        const uint16_t* __restrict__ gain, float eps,
                                                        int d, float* __restrict__ x,
                                                        uint16_t* __restrict__ h) {
  const int m = blockIdx.x;
  const int b = m / g.T, t = m - b * g.T;
  uint4 graw[CPT];
  load_gain<NT, CPT>(gain, d, graw);
  int tok = t < g.S ? tokens[(size_t)b * g.S + t] : g.mask_id;
  tok = tok < 0 ? 0 : (tok >= vocab ? vocab - 1 : tok);  // ids outside [0,V) are clamped
  const uint16_t* src = emb + (size_t)tok * d;
  float v[CPT][8];
#pragma unroll
  for (int c = 0; c < CPT; ++c) {
    const int ch = c * NT + (int)threadIdx.x;
    const uint4 raw = ch < (d >> 3) ? *reinterpret_cast<const uint4*>(src + ch * 8) : make_uint4(0, 0, 0, 0);
    const uint16_t* p = reinterpret_cast<const uint16_t*>(&raw);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[c][e] = bf2f(p[e]);
  }
  store_row<NT, CPT>(x + (size_t)m * d, d, v);
  row_norm_store<A, NT, CPT>(v, graw, eps, d, h + (size_t)m * d);
}

// RMSNorm, a workgroup per row.  NP is the number of split-K partials, known at
// compile time so that their loads are all issued before the first wait (a runtime
// loop over them took one round trip each); they are added in split order.  Rows
// carrying partials are the slow ones: taken first.
template <class A, int NT, int CPT, int NP>
__global__ __launch_bounds__(NT) void rmsnorm_kernel(float* __restrict__ x, const uint16_t* __restrict__ gain,
                                                     float eps, int M, int d, uint16_t* __restrict__ h,
                                                     const float* __restrict__ part, int part_row0) {
  const int r = blockIdx.x;
  const int n_tail = NP ? M - part_row0 : 0;
  const int m = r < n_tail ? part_row0 + r : r - n_tail;
  float* xr = x + (size_t)m * d;
  float v[CPT][8];
  uint4 graw[CPT];
  load_row<NT, CPT>(xr, d, v);
  load_gain<NT, CPT>(gain, d, graw);
  if constexpr (NP > 0) {
    if (m >= part_row0) {
      const float* pr = part + (size_t)(m - part_row0) * d;
      const size_t pstride = (size_t)(M - part_row0) * d;
      float pa[NP][CPT][8];
#pragma unroll
      for (int s = 0; s < NP; ++s) load_row<NT, CPT>(pr + s * pstride, d, pa[s]);
#pragma unroll
      for (int s = 0; s < NP; ++s)
#pragma unroll
        for (int c = 0; c < CPT; ++c)
#pragma unroll
          for (int e = 0; e < 8; ++e) v[c][e] += pa[s][c][e];
      store_row<NT, CPT>(xr, d, v);
    }
  }
  row_norm_store<A, NT, CPT>(v, graw, eps, d, h + (size_t)m * d);
}

// x += the NP split-K partials in split order, four elements per thread.  n4:
// float4s of one split (rows * d / 4).
template <int NP>
__global__ __launch_bounds__(256) void residual_reduce_kernel(float4* __restrict__ x,
                                                              const float4* __restrict__ part, size_t n4) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= n4) return;
  float4 v = x[i], pa[NP];
#pragma unroll
  for (int s = 0; s < NP; ++s) pa[s] = part[s * n4 + i];
#pragma unroll
  for (int s = 0; s < NP; ++s) { v.x += pa[s].x; v.y += pa[s].y; v.z += pa[s].z; v.w += pa[s].w; }
  x[i] = v;
}

template <class A, int NT, int CPT>
__global__ __launch_bounds__(NT) void select_norm_kernel(StepGeom g, int mode,
                                                         const int32_t* __restrict__ tokens,
                                                         const float* __restrict__ x,
                                                         const uint16_t* __restrict__ gain,
                                                         float eps, int d, uint16_t* __restrict__ hf,
                                                         uint16_t* __restrict__ hf_lo,
                                                         int32_t* __restrict__ target,
                                                         const int32_t* __restrict__ tgt_in, int compact) {
  const int rows_per_seq = mode == 0 ? g.Lb : mode == 1 ? 2 * g.Lb : g.G;
  const int r = blockIdx.x;  // row of the flattened [B, rows_per_seq] selection
  const int b = r / rows_per_seq, j = r - b * rows_per_seq;
  uint4 graw[CPT];
  load_gain<NT, CPT>(gain, d, graw);
  const bool lead = threadIdx.x == 0;
  int src;
  if (mode == 2) {  // response row j (WINO+ training state, no shadow block)
    src = g.P + j;
    if (lead) target[r] = tgt_in[r];
  } else if (mode == 0) {
    const int c0 = cur_start(g, b);
    const int tok = tokens[(size_t)b * g.S + c0 + j];
    // Eq. 4: draft reads Y_cur, verify reads Y_shad (without shadow rows no
    // position is verified; the current row's statistics then go unused)
    const bool verify = tok != g.mask_id && g.Ls > 0;
    src = verify ? g.S + j : c0 + j;
    if (compact) src = verify ? g.Lb + j : j;  // gathered rows: current block, then shadow
    if (lead) target[r] = verify ? tok : -1;
  } else {
    src = j < g.Lb ? cur_start(g, b) + j : g.S + (j - g.Lb);
    if (lead) target[r] = -1;
  }
  float v[CPT][8];
  const size_t xrow = compact ? (size_t)b * (g.Lb + g.Ls) + src : (size_t)b * g.T + src;
  load_row<NT, CPT>(x + xrow * d, d, v);
  row_norm_store<A, NT, CPT>(v, graw, eps, d, hf + (size_t)r * d, hf_lo + (size_t)r * d);
}

// Copy of the current-block and shadow rows of every sequence (fp32).
__global__ __launch_bounds__(256) void gather_block_rows_kernel(StepGeom g, const float* __restrict__ x,
                                                                int d, float* __restrict__ xc) {
  const int nq = g.Lb + g.Ls;
  const int r = blockIdx.x;  // b * nq + i
  const int b = r / nq, i = r - b * nq;
  const int t = i < g.Lb ? cur_start(g, b) + i : g.S + (i - g.Lb);
  const float4* src = reinterpret_cast<const float4*>(x + ((size_t)b * g.T + t) * d);
  float4* dst = reinterpret_cast<float4*>(xc + (size_t)r * d);
  for (int c = threadIdx.x; c < d / 4; c += 256) dst[c] = src[c];
}

// Weights bf16 -> fp16 (round to nearest even), 8 elements per thread; n is
// a multiple of 8.
__global__ __launch_bounds__(256) void bf16_to_f16_kernel(const uint16_t* __restrict__ in,
                                                          uint16_t* __restrict__ out, size_t n8,
                                                          int* __restrict__ overflow) {
  bool bad = false;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n8; i += (size_t)gridDim.x * 256) {
    const uint4 raw = reinterpret_cast<const uint4*>(in)[i];
    const uint32_t* w = &raw.x;
    uint4 o;
    uint32_t* op = &o.x;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      op[e] = ActF16::pack2(__uint_as_float(w[e] << 16), __uint_as_float(w[e] & 0xFFFF0000u));
      // an all-ones exponent: the value overflowed fp16 (or was not finite)
      bad |= (op[e] & 0x7C00u) == 0x7C00u || (op[e] & 0x7C000000u) == 0x7C000000u;
    }
    reinterpret_cast<uint4*>(out)[i] = o;
  }
  if (bad) *overflow = 1;
}

}  // namespace

void launch_bf16_to_f16(const uint16_t* in, uint16_t* out, size_t n, int* overflow, hipStream_t st) {
  const size_t n8 = n / 8;
  if (n8 == 0) return;
  const size_t blocks = std::min<size_t>((n8 + 255) / 256, 8192);
  bf16_to_f16_kernel<<<blocks, 256, 0, st>>>(in, out, n8, overflow);
}

// Runs f(threads per row, chunks per thread) for a row of d <= 4096 elements
// (the library's limit): the smallest workgroup whose threads cover the row in
// one or two 8-element chunks each.  These kernels are bound by HBM at many
// rows and by their chain of loads at few; a wave per row with up to eight
// chunks per lane had fewer loads in flight per CU (d = 4096, us per launch:
// embedding + norm 70 -> 55 at 8704 rows, 13.0 -> 9.5 at 544; partials
// added to the stream 14.3 -> 8.2 at 544 rows, 25 -> 15 at 512 of 8704).
template <class F>
void with_row_shape(int d, F f) {
  using std::integral_constant;
  if (d <= 512) f(integral_constant<int, 64>{}, integral_constant<int, 1>{});
  else if (d <= 1024) f(integral_constant<int, 128>{}, integral_constant<int, 1>{});
  else if (d <= 2048) f(integral_constant<int, 256>{}, integral_constant<int, 1>{});
  else f(integral_constant<int, 256>{}, integral_constant<int, 2>{});
}

void launch_embed_norm(const StepGeom& g, const int32_t* tokens, const uint16_t* emb, int vocab,
                       const uint16_t* gain, float eps, int d, float* x, uint16_t* h,
                       hipStream_t st) {
  const int M = g.B * g.T;
  with_row_shape(d, [&](auto nt, auto cpt) {
    constexpr int NT = decltype(nt)::value, CPT = decltype(cpt)::value;
    if (g.f16) embed_norm_kernel<ActF16, NT, CPT><<<M, NT, 0, st>>>(g, tokens, emb, vocab, gain, eps, d, x, h);
    else embed_norm_kernel<ActBf16, NT, CPT><<<M, NT, 0, st>>>(g, tokens, emb, vocab, gain, eps, d, x, h);
  });
}

// Runs f(split count) for the counts the residual planner uses; false for others.
template <class F>
bool with_splits(int n, F f) {
  using std::integral_constant;
  switch (n) {
    case 2: f(integral_constant<int, 2>{}); return true;
    case 3: f(integral_constant<int, 3>{}); return true;
    case 4: f(integral_constant<int, 4>{}); return true;
    case 6: f(integral_constant<int, 6>{}); return true;
    case 8: f(integral_constant<int, 8>{}); return true;
  }
  return false;
}

hipError_t launch_rmsnorm(float* x, const uint16_t* gain, float eps, int M, int d, uint16_t* h,
                          const float* part, int n_part, int part_row0, hipStream_t st, bool f16) {
  bool ok = true;
  with_row_shape(d, [&](auto nt, auto cpt) {
    constexpr int NT = decltype(nt)::value, CPT = decltype(cpt)::value;
    auto go = [&](auto np) {
      constexpr int NP = decltype(np)::value;
      if (f16) rmsnorm_kernel<ActF16, NT, CPT, NP><<<M, NT, 0, st>>>(x, gain, eps, M, d, h, part, part_row0);
      else rmsnorm_kernel<ActBf16, NT, CPT, NP><<<M, NT, 0, st>>>(x, gain, eps, M, d, h, part, part_row0);
    };
    if (!part || n_part == 0) go(std::integral_constant<int, 0>{});
    else ok = with_splits(n_part, go);
  });
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}

hipError_t launch_residual_reduce(float* x, const float* part, int n_part, int part_row0, int M, int d,
                                  hipStream_t st) {
  if (M - part_row0 <= 0) return hipSuccess;
  const size_t n4 = (size_t)(M - part_row0) * (d / 4);
  float4* x4 = reinterpret_cast<float4*>(x + (size_t)part_row0 * d);
  const float4* p4 = reinterpret_cast<const float4*>(part);
  const unsigned grid = (unsigned)((n4 + 255) / 256);
  const bool ok = with_splits(n_part, [&](auto np) {
    residual_reduce_kernel<decltype(np)::value><<<grid, 256, 0, st>>>(x4, p4, n4);
  });
  return ok ? hipGetLastError() : hipErrorInvalidValue;
}

void launch_select_norm(const StepGeom& g, int mode, const int32_t* tokens, const float* x,
                        const uint16_t* gain, float eps, int d, uint16_t* hf, uint16_t* hf_lo,
                        int32_t* target, hipStream_t st, const int32_t* tgt_in, bool compact) {
  const int n = g.B * (mode == 0 ? g.Lb : mode == 1 ? 2 * g.Lb : g.G);
  if (mode != 0) compact = false;
  const int cp = compact ? 1 : 0;
  with_row_shape(d, [&](auto nt, auto cpt) {
    constexpr int NT = decltype(nt)::value, CPT = decltype(cpt)::value;
    if (g.f16) select_norm_kernel<ActF16, NT, CPT><<<n, NT, 0, st>>>(g, mode, tokens, x, gain, eps, d, hf, hf_lo, target, tgt_in, cp);
    else select_norm_kernel<ActBf16, NT, CPT><<<n, NT, 0, st>>>(g, mode, tokens, x, gain, eps, d, hf, hf_lo, target, tgt_in, cp);
  });
}

void launch_gather_block_rows(const StepGeom& g, const float* x, int d, float* xc, hipStream_t st) {
  const int rows = g.B * (g.Lb + g.Ls);
  if (rows > 0) gather_block_rows_kernel<<<rows, 256, 0, st>>>(g, x, d, xc);
}

}  // namespace wino
