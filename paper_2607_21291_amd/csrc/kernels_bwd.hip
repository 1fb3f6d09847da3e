// Backward of the routed layer (the training side of Section 3.4) on gfx950:
// the kernels of the block's adjoint on the kept rows that are not projection
// GEMMs (those run on the forward's GEMM kernels with backward epilogues) nor
// weight gradients (kernels_wgrad.hip).
//
//   - transposes of the weights;
//   - gather of the output gradient at the kept rows, scaled by the gate;
//   - LayerNorm / RMSNorm adjoints with the gradients of gain and bias;
//   - causal attention backward over the kept tokens in two passes, both on
//     v_mfma_f32_16x16x32_bf16 and both deterministic (no atomics): one pass
//     per query block for dQ (and the softmax statistics), one per key block
//     for dK and dV, which adds the query heads of a GQA group in order;
//     both turn RoPE back and write token-major rows;
//   - the final scatter: dx = dy, plus the block's gradient at the kept rows.
#include <hip/hip_ext.h>

#include "attn_tiles.h"
#include "dsf_device.h"
#include "dsf_internal.h"

namespace dsf {

// ----------------------------------------------------------- transposes

// out[c][r] = in[r][c] of up to four dense matrices in one launch, a 64 x 64
// tile per workgroup: the weights, which the adjoint GEMMs read along their
// other dimension. R and C are multiples of 8 and the bases 16-byte aligned: a
// thread loads 8 columns of an input row and stores 8 rows of an output row.
// (With a launch each, 5 us apiece, of which the copying takes one.)
struct TransposeBatch {
  TransposeArgs m[kTransposeMax];
  int tile0[kTransposeMax + 1], n;
};

__global__ __launch_bounds__(256) void transpose_kernel(TransposeBatch g) {
  __shared__ float tile[64][65];
  int k = 0;
  while (k + 1 < g.n && int(blockIdx.x) >= g.tile0[k + 1]) ++k;
  const int R = g.m[k].R, C = g.m[k].C;
  const auto* in = (const uint16_t*)g.m[k].in;
  auto* out = (uint16_t*)g.m[k].out;
  const int ntc = (C + 63) / 64, t = int(blockIdx.x) - g.tile0[k];
  const int c0 = (t % ntc) * 64, r0 = (t / ntc) * 64;
  const int v = threadIdx.x & 7, q = threadIdx.x >> 3;  // vector index, row (column) within a pass
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int rr = q + 32 * i, r = r0 + rr, c = c0 + 8 * v;
    if (r < R && c < C) {
      float x[8];
      load_vec(in + int64_t(r) * C + c, x);
#pragma unroll
      for (int e = 0; e < 8; ++e) tile[rr][8 * v + e] = x[e];
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int cc = q + 32 * i, c = c0 + cc, r = r0 + 8 * v;
    if (c < C && r < R) {
      float x[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) x[e] = tile[8 * v + e][cc];
      store_vec(out + int64_t(c) * R + r, x);
    }
  }
}

hipError_t launch_transpose(const TransposeArgs* m, int n, hipStream_t s) {
  if (n > kTransposeMax) return hipErrorInvalidValue;
  TransposeBatch g{};
  for (g.n = 0; g.n < n; ++g.n) {
    const TransposeArgs& t = m[g.n];
    if (t.R <= 0 || t.C <= 0 || t.R % 8 != 0 || t.C % 8 != 0) return hipErrorInvalidValue;
    g.m[g.n] = t;
    g.tile0[g.n + 1] = g.tile0[g.n] + ((t.R + 63) / 64) * ((t.C + 63) / 64);
  }
  transpose_kernel<<<g.tile0[g.n], 256, 0, s>>>(g);
  return hipGetLastError();
}

// ------------------------------------------------- gather of the gradient

// out[m][:] = g_m * dy[b][idx[m]][:], m = b * kk + j, with g_m = sigmoid of
// the token's router score (gate) or 1. 16-byte vectors; d % 8 == 0.
__global__ __launch_bounds__(256) void gather_scale_kernel(const uint16_t* __restrict__ dy, int T, int d,
                                                           const int32_t* __restrict__ idx, int kk, int M,
                                                           const float* __restrict__ scores,
                                                           uint16_t* __restrict__ out) {
  const int nv = d / 8;
  const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (e >= int64_t(M) * nv) return;
  const int m = int(e / nv), c = int(e - int64_t(m) * nv) * 8;
  const int b = m / kk;
  const int p = clamp_pos(idx[m], T);
  float v[8];
  load_vec(dy + (int64_t(b) * T + p) * d + c, v);
  if (scores) {
    const float g = 1.f / (1.f + expf(-scores[int64_t(b) * T + p]));
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] *= g;
  }
  store_vec(out + int64_t(m) * d + c, v);
}

hipError_t launch_gather_scale(const void* dy, int B, int T, int d, const int32_t* idx, int kk, const float* scores,
                               void* out, hipStream_t s) {
  const int64_t n = int64_t(B) * kk * (d / 8);
  if (n == 0) return hipSuccess;
  gather_scale_kernel<<<int((n + 255) / 256), 256, 0, s>>>((const uint16_t*)dy, T, d, idx, kk, B * kk, scores,
                                                           (uint16_t*)out);
  return hipGetLastError();
}

// ------------------------------------------------------ norm adjoints

// Row m of x [M, d] (the norm's input) and dyn [M, d] (the gradient at the
// norm's output), gain w [d]:
//   LayerNorm: xhat = (x - mean) * rstd, g = dyn * w,
//              dx = rstd * (g - mean(g) - xhat * mean(g * xhat));
//   RMSNorm:   xhat = x * rstd, dx = rstd * (g - xhat * mean(g * xhat)).
// dx goes to acc (fp32 [M, d]): acc = dx, or acc += dx with accumulate. With
// add and sum_out (both bf16 [M, d]): sum_out = add + dx (Qwen's
// d(attention output) = d(delta) + d(h)).
//
// With partial, the gradients of gain (sum of dyn * xhat over the rows) and
// bias (sum of dyn) ride along: a workgroup takes `rows` consecutive rows and
// keeps the sums of its columns in registers, partial[workgroup][0, d) for
// the gain, [d, 2d) for the bias, which norm_sums_kernel adds. Column sums of
// their own read x and dyn once more and ended in a kernel of a few
// workgroups. Every order is fixed by the shape.
//
// A lane holds VC vectors of 8 columns of a row, the next row's on the way
// while it works on one. BLOCK false: one wavefront per row (d <= 512 VC),
// wave w taking rows w, w + 4, ...; true: the workgroup's four waves share a
// row (d <= 2048 VC), so that the sums of 8192 columns still fit registers.
// kNormBwdChunks bounds the partial sums to what the scratch holds.
// kNormBwdRows: few rows leave norm_sums_kernel more to add, many leave CUs
// idle; training step of a layer with 4 / 8 / 16 / 32 / 64: NeoX-160M 300 rows 199 / 203 /
// 208 / 219 / 239 us, 1400 rows 313 / 313 / 316 / 326 / 346, 12504 rows 1094 / 1098 / 1099 /
// 1102 / 1117; Qwen2.5-1.5B 6000 rows 2345 / 2342 / 2349 / 2348 / 2406.
constexpr int kNormBwdChunks = 512;  // workgroups, at most
constexpr int kNormBwdRows = 16;     // rows per workgroup, at least

static int norm_bwd_rows(int M) { return std::max(kNormBwdRows, (M + kNormBwdChunks - 1) / kNormBwdChunks); }
int norm_bwd_partials(int M) { return (M + norm_bwd_rows(M) - 1) / norm_bwd_rows(M); }

template <bool RMS, int VC, bool BLOCK>
__global__ __launch_bounds__(256) void norm_bwd_kernel(const uint16_t* __restrict__ x,
                                                       const uint16_t* __restrict__ dyn,
                                                       const uint16_t* __restrict__ w, int M, int d, float eps,
                                                       float* __restrict__ acc, int accumulate,
                                                       const uint16_t* __restrict__ add, uint16_t* __restrict__ sum_out,
                                                       int rows, float* __restrict__ partial) {
  constexpr int kStep = BLOCK ? 1 : 4;
  __shared__ float red[BLOCK ? 16 : 4 * VC * 512];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int v0 = BLOCK ? int(threadIdx.x) : lane;  // this lane's vectors: v0 + kVecStep c
  constexpr int kVecStep = BLOCK ? 256 : 64;
  // the sum over a row, in every lane that holds a part of it; slot: the
  // row's place among its sums (the four waves' parts are read behind one
  // barrier, and a slot is written again two barriers later)
  auto row_sum = [&](float v, int slot) {
    v = wave_sum_fast(v);
    if constexpr (BLOCK) {
      if (lane == 0) red[slot * 4 + wave] = v;
      __syncthreads();
      v = (red[slot * 4] + red[slot * 4 + 1]) + (red[slot * 4 + 2] + red[slot * 4 + 3]);
    }
    return v;
  };
  const int m0 = int(blockIdx.x) * rows + (BLOCK ? 0 : wave), m1 = min(M, (int(blockIdx.x) + 1) * rows);
  const u32x4 zero{0u, 0u, 0u, 0u};
  auto load_row = [&](const uint16_t* src, u32x4(&r)[VC]) {
#pragma unroll
    for (int c = 0; c < VC; ++c) {
      const int col = (v0 + kVecStep * c) * 8;
      r[c] = col < d ? *reinterpret_cast<const u32x4*>(src + col) : zero;
    }
  };
  auto unpack = [](const u32x4& r, float(&v)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      v[2 * i] = __uint_as_float(r[i] << 16);
      v[2 * i + 1] = __uint_as_float(r[i] & 0xffff0000u);
    }
  };
  float gw[VC][8], gb[RMS ? 1 : VC][8];
#pragma unroll
  for (int c = 0; c < VC; ++c)
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      gw[c][i] = 0.f;
      if constexpr (!RMS) gb[c][i] = 0.f;
    }
  u32x4 wv[VC], xv[VC], gv[VC];
  load_row(w, wv);
  if (m0 < m1) {
    load_row(x + int64_t(m0) * d, xv);
    load_row(dyn + int64_t(m0) * d, gv);
  }
  for (int m = m0; m < m1; m += kStep) {
    u32x4 xn[VC], gn[VC];
    const int mn = min(m + kStep, M - 1);  // (the last row's successor is loaded but not used)
    load_row(x + int64_t(mn) * d, xn);
    load_row(dyn + int64_t(mn) * d, gn);
    float s1 = 0.f, s2 = 0.f;
#pragma unroll
    for (int c = 0; c < VC; ++c) {
      float v[8];
      unpack(xv[c], v);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        s1 += v[i];
        s2 += v[i] * v[i];
      }
    }
    if constexpr (!RMS) s1 = row_sum(s1, 0);
    s2 = row_sum(s2, 1);
    const float mean = RMS ? 0.f : s1 / float(d);
    const float var = RMS ? s2 / float(d) : fmaxf(s2 / float(d) - mean * mean, 0.f);
    const float rstd = 1.f / sqrtf(var + eps);
    float sg = 0.f, sgx = 0.f;
#pragma unroll
    for (int c = 0; c < VC; ++c) {
      float v[8], g[8], ww[8];
      unpack(xv[c], v);
      unpack(gv[c], g);
      unpack(wv[c], ww);
#pragma unroll
      for (int i = 0; i < 8; ++i) {  // columns past d: g = 0
        const float gi = g[i] * ww[i], xh = (v[i] - mean) * rstd;
        sg += gi;
        sgx += gi * xh;
        gw[c][i] += g[i] * xh;
        if constexpr (!RMS) gb[c][i] += g[i];
      }
    }
    if constexpr (!RMS) sg = row_sum(sg, 2) / float(d);
    sgx = row_sum(sgx, 3) / float(d);
#pragma unroll
    for (int c = 0; c < VC; ++c) {
      const int col = (v0 + kVecStep * c) * 8;
      if (col >= d) continue;
      float v[8], g[8], ww[8], dx[8];
      unpack(xv[c], v);
      unpack(gv[c], g);
      unpack(wv[c], ww);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const float xh = (v[i] - mean) * rstd;
        dx[i] = rstd * (g[i] * ww[i] - (RMS ? 0.f : sg) - xh * sgx);
      }
      f32x4* ar = reinterpret_cast<f32x4*>(acc + int64_t(m) * d + col);
      f32x4 o0{dx[0], dx[1], dx[2], dx[3]}, o1{dx[4], dx[5], dx[6], dx[7]};
      if (accumulate) {
        o0 += ar[0];
        o1 += ar[1];
      }
      ar[0] = o0;
      ar[1] = o1;
      if (sum_out) {
        float a[8];
        load_vec(add + int64_t(m) * d + col, a);
#pragma unroll
        for (int i = 0; i < 8; ++i) a[i] += dx[i];
        store_vec(sum_out + int64_t(m) * d + col, a);
      }
    }
#pragma unroll
    for (int c = 0; c < VC; ++c) {
      xv[c] = xn[c];
      gv[c] = gn[c];
    }
  }
  if (!partial) return;
  float* dst = partial + int64_t(blockIdx.x) * 2 * d;
  auto put = [&](const float(*g)[8], float* to) {
    if constexpr (BLOCK) {
#pragma unroll
      for (int c = 0; c < VC; ++c) {
        const int col = (v0 + kVecStep * c) * 8;
        if (col >= d) continue;
        f32x4* o = reinterpret_cast<f32x4*>(to + col);
        o[0] = f32x4{g[c][0], g[c][1], g[c][2], g[c][3]};
        o[1] = f32x4{g[c][4], g[c][5], g[c][6], g[c][7]};
      }
    } else {
      __syncthreads();
#pragma unroll
      for (int c = 0; c < VC; ++c) {
        f32x4* o = reinterpret_cast<f32x4*>(red + wave * VC * 512 + (lane + 64 * c) * 8);
        o[0] = f32x4{g[c][0], g[c][1], g[c][2], g[c][3]};
        o[1] = f32x4{g[c][4], g[c][5], g[c][6], g[c][7]};
      }
      __syncthreads();
      for (int col = threadIdx.x; col < d; col += 256)
        to[col] = (red[col] + red[VC * 512 + col]) + (red[2 * VC * 512 + col] + red[3 * VC * 512 + col]);
    }
  };
  put(gw, dst);
  if constexpr (!RMS) put(gb, dst + d);
}

// out0[c] = sum over chunks of partial[chunk][c], out1[c] of [chunk][d + c]
// (either nullable): 16 columns by 16 chunk lanes per workgroup, lane j adding
// chunks j, j + 16, ... in order, then the lanes in order.
__global__ __launch_bounds__(256) void norm_sums_kernel(const float* __restrict__ partial, int chunks, int d,
                                                        float* __restrict__ out0, float* __restrict__ out1) {
  __shared__ float red[16][17];
  const int cl = threadIdx.x & 15, kl = threadIdx.x >> 4, c = blockIdx.x * 16 + cl;
  float s = 0.f;
  if (c < 2 * d) {
    constexpr int U = 8;  // partials loaded before they are added
    for (int k = kl; k < chunks; k += 16 * U) {
      float v[U];
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] = k + 16 * u < chunks ? partial[int64_t(k + 16 * u) * 2 * d + c] : 0.f;
#pragma unroll
      for (int u = 0; u < U; ++u) s += v[u];
    }
  }
  red[kl][cl] = s;
  __syncthreads();
  if (kl != 0 || c >= 2 * d) return;
#pragma unroll
  for (int j = 1; j < 16; ++j) s += red[j][cl];
  float* out = c < d ? out0 : out1;
  if (out) out[c < d ? c : c - d] = s;
}

template <int VC, bool BLOCK>
static void launch_norm_bwd_t(bool rms, const uint16_t* x, const uint16_t* dyn, const uint16_t* w, int M, int d,
                              float eps, float* acc, bool accumulate, const uint16_t* add, uint16_t* sum_out,
                              float* partial, hipStream_t s) {
  const int rows = norm_bwd_rows(M), grid = norm_bwd_partials(M);
  if (rms)
    norm_bwd_kernel<true, VC, BLOCK><<<grid, 256, 0, s>>>(x, dyn, w, M, d, eps, acc, accumulate, add, sum_out, rows,
                                                          partial);
  else
    norm_bwd_kernel<false, VC, BLOCK><<<grid, 256, 0, s>>>(x, dyn, w, M, d, eps, acc, accumulate, add, sum_out, rows,
                                                           partial);
}

hipError_t launch_norm_bwd(bool rms, const void* x, const void* dyn, const void* w, int M, int d, float eps, float* acc,
                           bool accumulate, const void* add, void* sum_out, float* dw, float* db, float* partial,
                           hipStream_t s) {
  if (M == 0) return hipSuccess;
  const auto *xx = (const uint16_t*)x, *g = (const uint16_t*)dyn, *ww = (const uint16_t*)w, *ad = (const uint16_t*)add;
  auto* so = (uint16_t*)sum_out;
  float* part = dw || db ? partial : nullptr;
  auto run = [&](auto vc, auto block) {
    launch_norm_bwd_t<decltype(vc)::value, decltype(block)::value>(rms, xx, g, ww, M, d, eps, acc, accumulate, ad, so,
                                                                   part, s);
  };
  using std::integral_constant;
  if (d <= 512) run(integral_constant<int, 1>{}, std::false_type{});
  else if (d <= 1024) run(integral_constant<int, 2>{}, std::false_type{});
  else if (d <= 2048) run(integral_constant<int, 4>{}, std::false_type{});
  else if (d <= 4096) run(integral_constant<int, 2>{}, std::true_type{});
  else run(integral_constant<int, 4>{}, std::true_type{});  // d <= 8192
  // RMSNorm has no bias: its half of the partials is not written and not read
  if (part)
    norm_sums_kernel<<<((rms ? 1 : 2) * d + 15) / 16, 256, 0, s>>>(part, norm_bwd_partials(M), d, dw,
                                                                  rms ? nullptr : db);
  return hipGetLastError();
}

// ----------------------------------------------------- the final scatter

// x_grad[b][idx[m]][:] = dy[b][idx[m]][:] + acc[m][:] (fp32 add, one rounding);
// the other rows of x_grad were copied from dy before.
__global__ __launch_bounds__(256) void scatter_grad_kernel(const uint16_t* __restrict__ dy,
                                                           const float* __restrict__ acc, int T, int d,
                                                           const int32_t* __restrict__ idx, int kk, int M,
                                                           uint16_t* __restrict__ dx) {
  const int nv = d / 8;
  const int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x;
  if (e >= int64_t(M) * nv) return;
  const int m = int(e / nv), c = int(e - int64_t(m) * nv) * 8;
  const int b = m / kk;
  const int64_t row = (int64_t(b) * T + clamp_pos(idx[m], T)) * d + c;
  float v[8];
  load_vec(dy + row, v);
  const float* a = acc + int64_t(m) * d + c;
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] += a[i];
  store_vec(dx + row, v);
}

hipError_t launch_scatter_grad(const void* dy, const float* acc, int B, int T, int d, const int32_t* idx, int kk,
                               void* dx, hipStream_t s) {
  const int64_t n = int64_t(B) * kk * (d / 8);
  if (n == 0) return hipSuccess;
  scatter_grad_kernel<<<int((n + 255) / 256), 256, 0, s>>>((const uint16_t*)dy, acc, T, d, idx, kk, B * kk,
                                                           (uint16_t*)dx);
  return hipGetLastError();
}

// ------------------------------------------------- attention backward

// Shapes: q [B, Hq, n, HD], k and v [B, Hkv, n, HD] (bf16, RoPE applied, as
// the forward's QKV epilogue writes them); o and dout [B n, Hq HD] (bf16,
// token-major: the attention output and its gradient); lse [B, Hq, n], the
// log of each query's softmax normaliser as the forward computed it. Query
// head h reads kv head h / (Hq / Hkv). scale = 1 / sqrt(HD).
//
// MFMA operand layout (v_mfma_f32_16x16x32_bf16): lane l supplies row l % 16
// of each operand and its 8 consecutive k slots 8 (l / 16) .. + 7; output
// element e of lane l is D[4 (l / 16) + e][l % 16]. A contraction may assign
// its 32 summed indices to the k slots in any order, the same for both
// operands: the probabilities and score gradients are used in the order a
// lane holds them after the score MFMA (index 16 blk + 4 grp + e of the two
// 16-blocks of the step), and the other operand is read with the LDS
// transpose load in that order (AttnTrans).
//
// Tiles of 64 rows go global -> LDS by buffer DMA into a ring of two stages
// (attn_tiles.h): the next tile's DMA is issued after the barrier that
// publishes the current one, and runs under its products.

constexpr int kAB = kAttnTileRows;  // queries or keys per block

__device__ __forceinline__ bf16x8 pack8(const float* v) {
  bf16x8 r;
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i] = (__bf16)v[i];
  return r;
}

// Both passes are bound by their vector instructions per score (exponential,
// difference, products, conversion) and by LDS reads, not by the matrix cores
// (a fifth of the time). Scores enter the exponential as one fused
// multiply-add in base 2, the causal test runs only in blocks that the
// diagonal crosses, and the scale is left to the accumulators. With 16 queries
// (keys) per wave every fragment read feeds one MFMA; G = 2 gives a wave two
// groups of 16 that share the fragments: for head dimensions up to 64 (the
// accumulators of 128 do not fit) where the larger blocks still give every CU
// two workgroups (kAttnBwdWide). Blocks are launched longest first, all heads
// of a block index together, so the short ones fill the end and, with heads in
// multiples of 8, an XCD's L2 keeps its heads' tiles. 96 heads of 64, 1563
// tokens: 100 -> 82 us (pass 1) and 170 -> 98 us (pass 2).
constexpr float kLog2e = 1.4426950408889634f;
constexpr int kAttnBwdWide = 512;  // workgroups of 128 queries (keys) from which they are used

// The gradients at q, k and v leave as the rows of dqkv [B n, (Hq + 2 Hkv) HD]
// (bf16, token-major), q and k turned back through the rotary embedding: a
// rotated pair (i, i + R/2) at position p was turned by the angle
// a = p * theta^(-2i/R); its gradient turns back,
//   d_i' = d_i cos a + d_{i+R/2} sin a, d_{i+R/2}' = d_{i+R/2} cos a - d_i sin a.
// A pair's halves lie in different lanes, so the fp32 rows go through the LDS
// of the finished tiles. (As a kernel of its own behind fp32 head-major
// outputs the turn read 115 MB and wrote 58 MB again at 12504 NeoX-160M rows:
// 29 us.) table: [T][R/2][2] (cos, sin).
struct RopeOut {
  const float* table; const int32_t* idx;  // positions [B, n]
  int T, R;
  uint16_t* out;
  int cols;
};

// Four columns 4 c4 .. + 3 of row r of the staged [rows][HD] fp32 gradients.
template <int HD>
__device__ __forceinline__ float* staged4(float* stage, int r, int c4) {
  return stage + r * HD + ((c4 ^ (r & 7)) << 2);
}

// Rows `first` .. of `rows` staged rows (those below n) to columns col .. of dqkv.
template <int HD>
__device__ __forceinline__ void store_rows(float* stage, int rows, int first, int n, int b, int col, bool rope,
                                           const RopeOut& o) {
  constexpr int V = HD / 8;
  const int half = o.R / 2;
  for (int t = threadIdx.x; t < rows * V; t += 256) {
    const int r = t / V, c0 = (t % V) * 8, tok = first + r;
    if (tok >= n) break;  // (r grows with t)
    const int64_t m = int64_t(b) * n + tok;
    float v[8];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const f32x4 x = *reinterpret_cast<const f32x4*>(staged4<HD>(stage, r, c0 / 4 + q));
#pragma unroll
      for (int e = 0; e < 4; ++e) v[4 * q + e] = x[e];
    }
    if (rope && c0 < o.R) {
      const float* tab = o.table + int64_t(clamp_pos(o.idx[m], o.T)) * o.R;
      if (o.R % 16 == 0) {  // the eight columns lie in one half, their partners are eight columns too
        const bool lo = c0 < half;
        const int pc = lo ? c0 + half : c0 - half;
        const f32x4* cs = reinterpret_cast<const f32x4*>(tab + 2 * (lo ? c0 : pc));
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const f32x4 x = *reinterpret_cast<const f32x4*>(staged4<HD>(stage, r, pc / 4 + q));
          const f32x4 t0 = cs[2 * q], t1 = cs[2 * q + 1];
          const float c[4] = {t0[0], t0[2], t1[0], t1[2]}, sn[4] = {t0[1], t0[3], t1[1], t1[3]};
#pragma unroll
          for (int e = 0; e < 4; ++e)
            v[4 * q + e] = lo ? v[4 * q + e] * c[e] + x[e] * sn[e] : v[4 * q + e] * c[e] - x[e] * sn[e];
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int dim = c0 + e;
          if (dim >= o.R) continue;
          const bool lo = dim < half;
          const int pc = lo ? dim + half : dim - half, i = lo ? dim : pc;
          const float x = staged4<HD>(stage, r, pc >> 2)[pc & 3];
          v[e] = lo ? v[e] * tab[2 * i] + x * tab[2 * i + 1] : v[e] * tab[2 * i] - x * tab[2 * i + 1];
        }
      }
    }
    store_vec(o.out + m * o.cols + col + c0, v);
  }
}

// Pass 1: one workgroup per (sequence, query head, block of 64 G queries);
// wave w owns queries q0 + 16 G w .. + 16 G - 1 (lane l: query l % 16 of each
// group). Scores are formed transposed (S^T = K Q^T, keys as MFMA rows), so a
// lane holds 16 scores of each of its queries per 64-key block. With
// P = exp(S scale - lse): writes D = sum_c dout * o for pass 2, and
// dQ = scale * sum_keys dS K with dS = P (dP - D), dP = dout V^T. Queries past
// the end are columns of their own that are not stored.
template <int HD, int G>
__global__ __launch_bounds__(256, HD == 64 && G == 2 ? 3 : 1) void attn_bwd_dq_kernel(const uint16_t* __restrict__ Q,
                                                          const uint16_t* __restrict__ K,
                                                          const uint16_t* __restrict__ V,
                                                          const uint16_t* __restrict__ O,
                                                          const uint16_t* __restrict__ dO, int n, int Hq, int Hkv,
                                                          int nbh, const float* __restrict__ lse,
                                                          float* __restrict__ dvec_out, RopeOut ro) {
  using A = AttnTile<HD>;
  constexpr int NS = HD / 32, NC = HD / 16;
  __shared__ __attribute__((aligned(16))) char smem[2 * 2 * A::kTileBytes];  // stage: K tile, then V tile
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, grp = lane >> 4;
  const int nqb = (n + kAB * G - 1) / (kAB * G);
  const int qb = nqb - 1 - int(blockIdx.x) / nbh, bh = int(blockIdx.x) % nbh;
  const int h = bh % Hq, b = bh / Hq, kvh = h / (Hq / Hkv);
  const int qw = (qb * 4 + wave) * 16 * G;  // the wave's first query
  const float scale = 1.f / sqrtf(float(HD)), scale2 = scale * kLog2e;
  const uint16_t* Kh = K + (int64_t(b) * Hkv + kvh) * n * HD;
  const uint16_t* Vh = V + (int64_t(b) * Hkv + kvh) * n * HD;
  const int nkb = min((n + kAB - 1) / kAB, (qb + 1) * G);
  auto issue = [&](int kt) {
    char* st = smem + (kt & 1) * 2 * A::kTileBytes;
    attn_tile_dma<HD>(Kh, HD, kt * kAB, n, st, wave, lane);
    attn_tile_dma<HD>(Vh, HD, kt * kAB, n, st + A::kTileBytes, wave, lane);
  };
  issue(0);

  // this lane's queries as MFMA B operand: Q and dout rows, k slots 32 s + 8 grp ..
  bf16x8 qf[G][NS], df[G][NS];
  float Dq[G], lq[G];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const int query = qw + 16 * g + r16;
    const bool qok = query < n;
    const int64_t orow = (int64_t(b) * n + (qok ? query : 0)) * (int64_t(Hq) * HD) + int64_t(h) * HD;
    float dsum = 0.f;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      u32x4 z = {0u, 0u, 0u, 0u};
      u32x4 qv = z, dv = z, ov = z;
      if (qok) {
        qv = *reinterpret_cast<const u32x4*>(Q + ((int64_t(bh) * n + query) * HD) + 32 * s + 8 * grp);
        dv = *reinterpret_cast<const u32x4*>(dO + orow + 32 * s + 8 * grp);
        ov = *reinterpret_cast<const u32x4*>(O + orow + 32 * s + 8 * grp);
      }
      qf[g][s] = __builtin_bit_cast(bf16x8, qv);
      df[g][s] = __builtin_bit_cast(bf16x8, dv);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        dsum += __uint_as_float(dv[i] << 16) * __uint_as_float(ov[i] << 16);
        dsum += __uint_as_float(dv[i] & 0xffff0000u) * __uint_as_float(ov[i] & 0xffff0000u);
      }
    }
    Dq[g] = rows4_sum(dsum);
    lq[g] = qok ? lse[int64_t(bh) * n + query] * kLog2e : 0.f;
    if (qok && grp == 0) dvec_out[int64_t(bh) * n + query] = Dq[g];
  }

  // dQ^T[c][query] = scale * sum_keys K^T[c][key] dS^T[key][query]
  const AttnTrans<HD> tr(lane);
  f32x4 acc[G][NC];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) acc[g][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int kt = 0; kt < nkb; ++kt) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's share of tile kt has landed
    __syncthreads();                                   // ... and every wave's; tile kt - 1 is retired
    if (kt + 1 < nkb) issue(kt + 1);
    if (kt * kAB > qw + 16 * G - 1) continue;  // every key after the wave's queries
    const char* Kt = smem + (kt & 1) * 2 * A::kTileBytes;
    const char* Vt = Kt + A::kTileBytes;
    const bool edge = kt * kAB + kAB - 1 > qw;  // some of the block's keys come after some of the queries
    bf16x8 dsb[G][2];
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
      float ds[G][8];
#pragma unroll
      for (int hb = 0; hb < 2; ++hb) {
        const int blk = 2 * s2 + hb;
        f32x4 st[G], dp[G];
#pragma unroll
        for (int g = 0; g < G; ++g) st[g] = dp[g] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const bf16x8 kf = attn_row_frag<HD>(Kt, 16 * blk + r16, 4 * s + grp);
          const bf16x8 vf = attn_row_frag<HD>(Vt, 16 * blk + r16, 4 * s + grp);
#pragma unroll
          for (int g = 0; g < G; ++g) {
            st[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf, qf[g][s], st[g], 0, 0, 0);
            dp[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, df[g][s], dp[g], 0, 0, 0);
          }
        }
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float p = __builtin_amdgcn_exp2f(fmaf(st[g][e], scale2, -lq[g]));
            if (edge && kt * kAB + 16 * blk + 4 * grp + e > qw + 16 * g + r16) p = 0.f;
            ds[g][4 * hb + e] = p * (dp[g][e] - Dq[g]);
          }
      }
#pragma unroll
      for (int g = 0; g < G; ++g) dsb[g][s2] = pack8(ds[g]);
    }
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) {
      bf16x8 kt2[2];
      tr.read(Kt, cb, kt2);
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int g = 0; g < G; ++g)
          acc[g][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kt2[s2], dsb[g][s2], acc[g][cb], 0, 0, 0);
    }
  }
  // lane holds dQ^T[16 cb + 4 grp + e][query] / scale
  float* stage = reinterpret_cast<float*>(smem);
  __syncthreads();  // every wave is done with the tiles
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int cb = 0; cb < NC; ++cb)
      *reinterpret_cast<f32x4*>(staged4<HD>(stage, 16 * (G * wave + g) + r16, 4 * cb + grp)) = acc[g][cb] * scale;
  __syncthreads();
  store_rows<HD>(stage, kAB * G, qb * kAB * G, n, b, h * HD, true, ro);
}

// Pass 2: one workgroup per (sequence, kv head, block of 64 G keys); wave w
// owns keys k0 + 16 G w .. + 16 G - 1 (lane l: key l % 16 of each group). For
// every query head of the kv head's group and every query block that reaches
// the key block (one work item each, in that order), scores are formed with
// keys as MFMA columns (S = Q K^T), so a lane holds the probabilities of its
// own keys, and
//   dV^T[c][key] += sum_queries dout^T[c][query] P[query][key],
//   dK^T[c][key] += scale * sum_queries Q^T[c][query] dS[query][key].
// Each item's lse and D come with its tiles, by DMA (as register loads their
// arrival was waited for, and with it the DMA in flight). Queries past the
// end are zero rows of Q and dout, masked so that an infinite key (whose
// product with a zero row is NaN) keeps its own gradient; keys past it are not
// stored.
template <int HD, int G>
__global__ __launch_bounds__(256) void attn_bwd_dkv_kernel(const uint16_t* __restrict__ Q,
                                                           const uint16_t* __restrict__ K,
                                                           const uint16_t* __restrict__ V,
                                                           const uint16_t* __restrict__ dO,
                                                           const float* __restrict__ lse,
                                                           const float* __restrict__ dvec, int n, int Hq, int Hkv,
                                                           int nbkv, RopeOut ro) {
  using A = AttnTile<HD>;
  constexpr int NS = HD / 32, NC = HD / 16;
  // stage: Q tile, then dout tile; then per stage lse and D of its queries.
  // One object: with several, the compiler orders every LDS read behind the
  // DMA in flight.
  __shared__ __attribute__((aligned(16))) char smem[2 * 2 * A::kTileBytes + 2 * 2 * kAB * 4];
  float* stats = reinterpret_cast<float*>(smem + 2 * 2 * A::kTileBytes);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r16 = lane & 15, grp = lane >> 4;
  const int kb = int(blockIdx.x) / nbkv, bkv = int(blockIdx.x) % nbkv;
  const int kvh = bkv % Hkv, b = bkv / Hkv;
  const int R = Hq / Hkv;
  const int kw = (kb * 4 + wave) * 16 * G;  // the wave's first key
  const float scale = 1.f / sqrtf(float(HD)), scale2 = scale * kLog2e;
  const uint16_t* Kh = K + int64_t(bkv) * n * HD;
  const uint16_t* Vh = V + int64_t(bkv) * n * HD;
  const int qb0 = kb * G, nq = (n + kAB - 1) / kAB - qb0;  // query blocks that reach the key block
  const int items = R * nq;
  // item i: query head kvh R + i / nq, query block qb0 + i % nq
  auto issue = [&](int i) {
    const int h = kvh * R + i / nq, qb = qb0 + i % nq;
    const int64_t bh = int64_t(b) * Hq + h;
    char* st = smem + (i & 1) * 2 * A::kTileBytes;
    attn_tile_dma<HD>(Q + bh * n * HD, HD, qb * kAB, n, st, wave, lane);
    attn_tile_dma<HD>(dO + int64_t(b) * n * (int64_t(Hq) * HD) + int64_t(h) * HD, int64_t(Hq) * HD, qb * kAB, n,
                      st + A::kTileBytes, wave, lane);
    if (wave == 0) {  // lane: query of the item; zeros past the end
      const auto lr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(lse + bh * n), (short)0, n * 4, 0x00020000);
      const auto dr =
          __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(dvec + bh * n), (short)0, n * 4, 0x00020000);
      const int voff = (qb * kAB + lane) * 4;
      float* sp = stats + (i & 1) * 2 * kAB;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(lr, (__attribute__((address_space(3))) void*)(sp), 4, voff, 0, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(dr, (__attribute__((address_space(3))) void*)(sp + kAB), 4, voff, 0, 0,
                                               0);
    }
  };
  issue(0);

  bf16x8 kf[G][NS], vf[G][NS];
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const int key = kw + 16 * g + r16;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
      u32x4 z = {0u, 0u, 0u, 0u}, kv = z, vv = z;
      if (key < n) {
        kv = *reinterpret_cast<const u32x4*>(Kh + int64_t(key) * HD + 32 * s + 8 * grp);
        vv = *reinterpret_cast<const u32x4*>(Vh + int64_t(key) * HD + 32 * s + 8 * grp);
      }
      // wait for them here: left to their first use, the wait would sit in the
      // loop, behind the DMA of the next item
      asm volatile("" : "+v"(kv), "+v"(vv));
      kf[g][s] = __builtin_bit_cast(bf16x8, kv);
      vf[g][s] = __builtin_bit_cast(bf16x8, vv);
    }
  }
  const AttnTrans<HD> tr(lane);
  f32x4 adk[G][NC], adv[G][NC];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) adk[g][cb] = adv[g][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int i = 0; i < items; ++i) {
    const int slot = i & 1;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's share of item i's tiles has landed
    __syncthreads();                                   // ... and every wave's; item i - 1 is retired
    if (i + 1 < items) issue(i + 1);
    const int q0 = (qb0 + i % nq) * kAB;
    if (q0 + kAB - 1 < kw) continue;  // every query before the wave's keys
    // some of the block's queries come before some of the keys, or past the end
    const bool edge = q0 < kw + 16 * G - 1 || q0 + kAB > n;
    const char* Qt = smem + slot * 2 * A::kTileBytes;
    const char* Dt = Qt + A::kTileBytes;
    bf16x8 pb[G][2], db[G][2];
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
      float p[G][8], ds[G][8];
#pragma unroll
      for (int hb = 0; hb < 2; ++hb) {
        const int blk = 2 * s2 + hb;
        f32x4 st[G], dp[G];
#pragma unroll
        for (int g = 0; g < G; ++g) st[g] = dp[g] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < NS; ++s) {
          const bf16x8 qa = attn_row_frag<HD>(Qt, 16 * blk + r16, 4 * s + grp);
          const bf16x8 da = attn_row_frag<HD>(Dt, 16 * blk + r16, 4 * s + grp);
#pragma unroll
          for (int g = 0; g < G; ++g) {
            st[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qa, kf[g][s], st[g], 0, 0, 0);
            dp[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(da, vf[g][s], dp[g], 0, 0, 0);
          }
        }
        const f32x4 l4 = *reinterpret_cast<const f32x4*>(stats + slot * 2 * kAB + 16 * blk + 4 * grp) * kLog2e;
        const f32x4 d4 = *reinterpret_cast<const f32x4*>(stats + slot * 2 * kAB + kAB + 16 * blk + 4 * grp);
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float pv = __builtin_amdgcn_exp2f(fmaf(st[g][e], scale2, -l4[e]));
            // key <= query < n, as one unsigned comparison of their distances
            const int key = kw + 16 * g + r16;
            if (edge && uint32_t(q0 + 16 * blk + 4 * grp + e - key) >= uint32_t(n - key)) pv = 0.f;
            p[g][4 * hb + e] = pv;
            ds[g][4 * hb + e] = pv * (dp[g][e] - d4[e]);
          }
      }
#pragma unroll
      for (int g = 0; g < G; ++g) {
        pb[g][s2] = pack8(p[g]);
        db[g][s2] = pack8(ds[g]);
      }
    }
#pragma unroll
    for (int cb = 0; cb < NC; ++cb) {
      bf16x8 dt2[2], qt2[2];
      tr.read(Dt, cb, dt2);
      tr.read(Qt, cb, qt2);
#pragma unroll
      for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
        for (int g = 0; g < G; ++g) {
          adv[g][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(dt2[s2], pb[g][s2], adv[g][cb], 0, 0, 0);
          adk[g][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qt2[s2], db[g][s2], adk[g][cb], 0, 0, 0);
        }
    }
  }
  float* stage = reinterpret_cast<float*>(smem);
  auto put = [&](const f32x4(&acc)[G][NC], float mul, int col, bool rope) {
    __syncthreads();  // every wave is done with the tiles (with the rows staged before)
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
      for (int cb = 0; cb < NC; ++cb)
        *reinterpret_cast<f32x4*>(staged4<HD>(stage, 16 * (G * wave + g) + r16, 4 * cb + grp)) = acc[g][cb] * mul;
    __syncthreads();
    store_rows<HD>(stage, kAB * G, kb * kAB * G, n, b, col, rope, ro);
  };
  put(adk, scale, (Hq + kvh) * HD, true);
  put(adv, 1.f, (Hq + Hkv + kvh) * HD, false);
}

hipError_t launch_attention_bwd(const void* q, const void* k, const void* v, const void* o, const void* dout, int B,
                                int Hq, int Hkv, int n, int hd, const float* lse, float* dvec, const float* table,
                                const int32_t* idx, int T, int R, void* dqkv, hipStream_t s) {
  if (B == 0 || n == 0) return hipSuccess;
  const RopeOut ro{table, idx, T, R, (uint16_t*)dqkv, (Hq + 2 * Hkv) * hd};
  const auto *Qp = (const uint16_t*)q, *Kp = (const uint16_t*)k, *Vp = (const uint16_t*)v;
  const auto *Op = (const uint16_t*)o, *Dp = (const uint16_t*)dout;
  auto run_dq = [&](auto hdc, auto gc) {
    constexpr int HD = decltype(hdc)::value, G = decltype(gc)::value;
    attn_bwd_dq_kernel<HD, G><<<B * Hq * ((n + kAB * G - 1) / (kAB * G)), 256, 0, s>>>(Qp, Kp, Vp, Op, Dp, n, Hq, Hkv,
                                                                                       B * Hq, lse, dvec, ro);
  };
  auto run_dkv = [&](auto hdc, auto gc) {
    constexpr int HD = decltype(hdc)::value, G = decltype(gc)::value;
    attn_bwd_dkv_kernel<HD, G><<<B * Hkv * ((n + kAB * G - 1) / (kAB * G)), 256, 0, s>>>(
        Qp, Kp, Vp, Dp, lse, dvec, n, Hq, Hkv, B * Hkv, ro);
  };
  std::integral_constant<int, 1> one;
  std::integral_constant<int, 2> two;
  const int64_t wide = (n + 2 * kAB - 1) / (2 * kAB);
  auto run = [&](auto hdc) {
    if (B * Hq * wide >= kAttnBwdWide) run_dq(hdc, two);
    else run_dq(hdc, one);
    if (B * Hkv * wide >= kAttnBwdWide) run_dkv(hdc, two);
    else run_dkv(hdc, one);
  };
  switch (hd) {
    case 32: run(std::integral_constant<int, 32>{}); break;
    case 64: run(std::integral_constant<int, 64>{}); break;
    case 128:
      run_dq(std::integral_constant<int, 128>{}, one);
      run_dkv(std::integral_constant<int, 128>{}, one);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace dsf
