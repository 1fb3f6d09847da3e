// Device-side pieces of the router that more than one kernel uses: the
// decode-time routing of a scored token, and the scores of up to 16 rows by
// one workgroup of eight wavefronts (decode steps).
#pragma once

#include "dsf_device.h"
#include "dsf_internal.h"

namespace dsf {

// Decode-time routing of token t with score v (RouteArgs).
__device__ __forceinline__ void route_token(const RouteArgs& ra, int64_t t, float v, float thr, int len) {
  const bool want = v >= thr;
  const bool room = len < ra.cap;
  const int k = want && room;
  ra.keep[t] = k;
  ra.len_in[t] = len;
  ra.gate[t] = k ? INFINITY : -INFINITY;
  if (ra.keep_out) ra.keep_out[t] = want ? (room ? 1 : 2) : 0;
}

// Scores of rows row0 .. row0 + 15 (< r.n) with the arithmetic of
// router_bf16_kernel (wave w takes the 32-wide column slices w, w + 8, ...;
// the wave partials are added in wave order), so the scores are bitwise
// those of the router kernel. part: 8 x 16 x (d_r + 1) + 128 floats of LDS.
// One workgroup scores a whole decode batch's block of rows, so its time is
// the latency of its loads: eight slices' loads are in flight per wave, and
// what the scores need at the end is requested first.
__device__ __forceinline__ void router_rows16(const RouterRows& r, int row0, float* part) {
  constexpr int NW = 8, U = 8;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int r16 = lane & 15, g = lane >> 4, nb_n = r.d_r / 16, ld = r.d_r + 1;
  const uint16_t* x = (const uint16_t*)r.x + int64_t(min(row0 + r16, r.n - 1)) * r.d;
  const uint16_t* w1 = (const uint16_t*)r.w1 + int64_t(r16) * r.d;
  // output weights and biases of the units, and the token's threshold and cache length
  float* unit = part + NW * 16 * ld;
  if (tid < r.d_r) {
    unit[tid] = bf2f(((const uint16_t*)r.w2)[tid]);
    unit[64 + tid] = r.b1 ? bf2f(((const uint16_t*)r.b1)[tid]) : 0.f;
  }
  float thr = 0.f;
  int len = 0;
  if (tid < 64 && row0 + (tid >> 2) < r.n && r.route.thr) {
    thr = r.route.thr[row0 + (tid >> 2)];
    len = r.route.len[row0 + (tid >> 2)];
  }
  const bf16x8 zero = {};
  for (int n0 = 0; n0 < nb_n; n0 += 2) {  // two blocks of 16 units at a time
    const bool two = n0 + 1 < nb_n;
    const uint16_t* wr = w1 + int64_t(16 * n0) * r.d;
    const int64_t wo = two ? int64_t(16) * r.d : 0;
    f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
    for (int k0 = 32 * w; k0 < r.d; k0 += 32 * NW * U) {
      bf16x8 xa[U], wb[U][2];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = k0 + 32 * NW * u + 8 * g;
        const bool ok = k < r.d;  // d is a multiple of 8
        xa[u] = ok ? *reinterpret_cast<const bf16x8*>(x + k) : zero;
        wb[u][0] = ok ? *reinterpret_cast<const bf16x8*>(wr + k) : zero;
        wb[u][1] = ok ? *reinterpret_cast<const bf16x8*>(wr + wo + k) : zero;
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (k0 + 32 * NW * u >= r.d) break;
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
          acc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xa[u], wb[u][nb], acc[nb], 0, 0, 0);
      }
    }
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
      if (nb == 0 || two)
#pragma unroll
        for (int i = 0; i < 4; ++i) part[(w * 16 + 4 * g + i) * ld + 16 * (n0 + nb) + r16] = acc[nb][i];
  }
  __syncthreads();
  // threads 0..63: token t / 4, a quarter of its units each, as in the router kernel
  if (tid >= 64) return;
  const int t = tid >> 2, q = tid & 3, per = r.d_r / 4;
  float v = 0.f;
  for (int jj = 0; jj < per; ++jj) {
    const int j = q * per + jj;
    float h = unit[64 + j];
#pragma unroll
    for (int ww = 0; ww < NW; ++ww) h += part[(ww * 16 + t) * ld + j];
    v = fmaf(unit[j], h > 0.f ? h : 0.f, v);
  }
  v += __shfl_xor(v, 1);
  v += __shfl_xor(v, 2);
  if (q == 0 && row0 + t < r.n) {
    r.scores[row0 + t] = v + r.b2;
    if (r.route.thr) route_token(r.route, row0 + t, v + r.b2, thr, len);
  }
}

}  // namespace dsf
