// Few-row projections: C[M, N] = A[M, K] . B[N, K]^T with the block's fused
// epilogues for M <= 64 rows (decode steps, the shortest prompts), gfx950.
//
// With so few rows a projection is a stream over its weights: at 8 rows the
// GPT-NeoX-160M QKV projection is 3.5 MB for 28 MFLOP. The 128 x 128 tile
// grid puts N / 128 workgroups on 256 CUs (28 of them for the Qwen2.5-7B down
// projection: 253 us at 32 rows, against 27 us for its 136 MB at the copy
// rate), and splitting K over workgroups ends in a hand-over of partial sums
// through memory whose stores, counter and reloads cost more than the
// weights. Here a workgroup of eight wavefronts takes 16 NB output columns
// over the whole of K: each wave multiplies one contiguous range of k-steps,
// operands straight from global memory into the MFMA (16 bytes per lane; the
// next group's loads are issued before the current group's MFMAs), and the
// eight partial tiles meet in LDS, added in wave order (deterministic).
// Nothing is handed over between workgroups (but see SPLIT).
//
// Column groups. An epilogue item is one row of a 16-column group, held by
// one thread as two chunks of 8 columns, chosen so that whatever the epilogue
// combines is in the group: 8 gate units with their 8 up units (SwiGLU), 8
// rotated dims with their 8 partners (RoPE), otherwise 16 neighbours.
//
// The launch can also normalise its input rows (NORM): the workgroups read
// the raw hidden states, take every row's statistics themselves and
// normalise each A fragment on its way into the MFMA, so that a decode layer
// needs no launch for it; run two projections of the same rows side by side
// (GPT-NeoX QKV and FFN up); and score the rows with the router in extra
// workgroups at the head of the grid.
//
// Above 16 rows of a deep reduction every workgroup re-reads all of A for its
// 16 columns (32 rows: twice the weights), so the tile is made 64 (17-32
// rows) or 32 columns (33-64) wide and K split over workgroups again (SPLIT).
//
// Measured (kernel trace, weights from memory): GPT-NeoX-160M layer at 8
// rows, router, norm, FFN up and QKV 6.8 + 3.6 + 9.5 + 10.3 us as four
// launches (up and QKV split along K over workgroups), 10.5 us as this one;
// down 10.9 -> 10.5. Qwen2.5-7B layer at 32 rows: QKV 54 -> 24 us with the
// router's 19 us inside, O 51 -> 19, down 253 -> 51 (2.7 TB/s). What is left
// at 8 rows is latency: arguments, statistics, weights, LDS and stores, one
// after the other.
#include <algorithm>
#include <cstdlib>

#include "dsf_device.h"
#include "dsf_internal.h"
#include "router_device.h"

namespace dsf {

namespace {
// What a workgroup reads of one projection. The arguments arrive over the
// scalar cache from the launch's argument buffer, about a microsecond a line
// on first use, so they are packed and every line is touched at once.
struct RowProb {
  const void* a; const void* b; const void* a2; const void* b2;
  const void* bias; const void* bias2;
  // QKV: out q, aux0 k, aux1 v, aux2 the RoPE table; GELU, SwiGLU: out;
  // residual store: out, aux0 x; residual scatter: out x, aux0 res, aux1 gate
  void* out; void* aux0; void* aux1; const void* aux2;
  const int32_t* idx;
  int M, N, K, K1, lda, lda2, ldb, ldb2, epi, kk, T, f, ldo, Hq, Hkv, hd, R, nsub;
};
// Where the forms change. The figures are microseconds per layer of a decode
// step over 300 keys, with the form / without it.
//
// 16-column groups from which a workgroup takes two, which halves the re-reads
// of A and, below some count, leaves CUs idle. 16 rows: Qwen2.5-7B gate|up
// (2368 groups) 201 / 226, 1.5B (1120) 90 / 92; below the line NeoX-1.4B QKV
// and up (896) 64 / 69, Qwen2.5-0.5B (608) 63 / 64, NeoX-160M (336) 35 / 35. 4 rows:
// 165 / 172, 77 / 77, 56 / 57, 56 / 55, 28.5 / 27.7.
constexpr int kRowWideMin = 1024;
// Groups up to which groups of 8 columns double the workgroups of a down or O
// projection. 16 rows: NeoX-160M (48 groups) 35 / 37, Qwen2.5-0.5B (56) 64 / 66,
// 1.5B (96) 90 / 94, NeoX-1.4B (128) 69 / 73; beyond, Qwen2.5-7B (224) 227 / 201.
constexpr int kRowNarrowMax = 128;
// k-steps from which more than 16 rows split K. 48 rows: 120 steps (NeoX-160M
// down) 44 / 53, 152 (Qwen2.5-0.5B) 71 / 83, 64 and 320 (NeoX-1.4B) 100 / 121, of
// which the 64 give nothing; 24 rows: 38 / 41, 64 / 69, 72 / 82 (the 64: 72 / 73).
// Below, 48 steps (Qwen2.5-1.5B QKV): 102 -> 98 at 48 rows, 88 -> 90 at 24.
constexpr int kRowSplitMinSteps = 64;
// Workgroups that a split aims at, two per CU. 128 / 256 / 512 / 1024 at 24 rows:
// NeoX-1.4B 74 / 68 / 72 / 79, Qwen2.5-1.5B 87 / 84 / 88 / 88, 7B 204 / 166 / 179 /
// 185; at 48 rows 109 / 97 / 100 / 110, 113 / 99 / 102 / 110, 245 / 214 / 209 / 231;
// the small models the same throughout.
constexpr int kRowSplitWgs = 512;
// Pieces of a tile, at most: the last adds them all. 4 / 8 / 16 / 32 at 24 rows:
// NeoX-160M 39 / 38 / 38 / 38, Qwen2.5-0.5B 65 / 63 / 64 / 64, 1.5B 89 / 84 / 88 / 89,
// 7B 172 / 180 / 179 / 179; at 48 rows within 4 % of each other.
constexpr int kRowSplitMax = 16;
// fp32: workgroups below which a smaller tile is taken. A layer of one sequence,
// line at 96 / 192 / 300: NeoX-160M 100 rows 94 / 89 / 92, 307 rows 128 / 118 / 116,
// 600 rows 200 / 176 / 187; Qwen2.5-1.5B 307 rows 468 / 410 / 440, 600 rows 674 / 674 /
// 726; Qwen2.5-0.5B 307 rows 200 / 222 / 222, 600 rows 312 / 337 / 336; from 1200 rows
// on the same.
constexpr int kRowTilesF32 = 192;
struct RowGemmArgs {
  int router_wgs;
  int tiles0;    // tiles of the first projection
  int rms;
  int narrow;    // 1: column groups of 8
  int splits;    // workgroups per tile, each a slice of K
  int mtiles;    // tiles of 16 MB rows (fp32; 1 in bf16)
  float eps;
  const void* norm_w[2]; const void* norm_b[2];
  float* part; uint32_t* count;
  RowProb p[2];
  RouterRows r;
};

// One k-step: a 16-byte vector per lane, 4 lanes along K.
template <typename T>
struct RowElem {
  static constexpr int kVec = 16 / int(sizeof(T));
  static constexpr int kStep = 4 * kVec;
};

// acc += A(16 rows) . B(16 rows)^T over one k-step. bf16: one MFMA. fp32:
// element e of every lane's vector forms one 4-deep MFMA; A and B use the
// same assignment of k to slots, so the contraction is unchanged.
template <typename T>
__device__ __forceinline__ void row_mma(f32x4& acc, const u32x4& a, const u32x4& b) {
  if constexpr (sizeof(T) == 2) {
    acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0,
                                                  0, 0);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[e]), __uint_as_float(b[e]), acc, 0, 0, 0);
  }
}

// The two 8-column chunks of column group s: first output column of each
// (lo, hi), whether they are rotation partners, and whether hi exists.
struct RowCols {
  int lo, hi;
  bool rot, has_hi;
};
__device__ __forceinline__ RowCols row_cols(const RowProb& g, int s, int narrow) {
  RowCols c;
  c.rot = false;
  c.has_hi = true;
  if (narrow) {  // 8 columns: the hi lanes repeat the lo rows
    c.lo = c.hi = 8 * s;
    c.has_hi = false;
    return c;
  }
  if (g.epi == EPI_SWIGLU) {
    c.lo = 8 * s;  // gate units; hi holds the matching up units
    c.hi = g.f + 8 * s;
    return c;
  }
  c.lo = 16 * s;
  if (g.epi == EPI_QKV_ROPE) {
    const int sh = 31 - __clz(g.hd / 16), head = s >> sh, t = s - (head << sh);  // hd is a power of two
    if (head < g.Hq + g.Hkv && t < g.R / 16) {
      c.rot = true;
      c.lo = head * g.hd + 8 * t;
      c.hi = c.lo + g.R / 2;
      return c;
    }
  }
  c.hi = c.lo + 8;
  c.has_hi = c.hi < g.N;
  return c;
}

// What the epilogue of row m and one column group reads besides the sums.
// The row's position and the first words are requested ahead of the main
// loop (row_touch: they bring the lines in), the vectors after it.
template <typename T>
struct RowPre {
  Raw8<T> bias[2], bias2[2], res[2], x[2];
  float4 cs[4];
  float gate;
  int bq, jq, pq;
  uint32_t t[5];
};
__device__ __forceinline__ bool row_scatters(const RowProb& g) {
  return g.epi == EPI_RESID_SCATTER || g.epi == EPI_RESID_SCATTER_GATE;
}
__device__ __forceinline__ const void* row_x(const RowProb& g) { return row_scatters(g) ? g.out : g.aux0; }
template <typename T>
__device__ __forceinline__ void row_place(const RowProb& g, int m, RowPre<T>& e) {
  e.bq = g.kk == 1 ? m : m / g.kk;
  e.jq = m - e.bq * g.kk;
  e.pq = epi_uses_positions(g.epi) && g.idx ? clamp_pos(g.idx[m], g.T) : e.jq;
}
template <typename T>
__device__ __forceinline__ void row_touch(const RowProb& g, int m, const RowCols& c, RowPre<T>& e) {
  auto word = [](const void* p, int64_t i) { return *reinterpret_cast<const uint32_t*>((const T*)p + i); };
#pragma unroll
  for (int i = 0; i < 5; ++i) e.t[i] = 0u;
  if (g.epi == EPI_SWIGLU) return;
  const bool scatter = row_scatters(g);
  if (g.bias) e.t[0] = word(g.bias, c.lo);
  if (scatter && g.bias2) e.t[1] = word(g.bias2, c.lo);
  if (scatter && g.aux0) e.t[2] = word(g.aux0, int64_t(m) * g.N + c.lo);
  if (g.kk == 1 && !g.idx) {  // decode rows: the position is the row
    if (scatter || g.epi == EPI_RESID_STORE) e.t[3] = word(row_x(g), int64_t(m) * g.T * g.N + c.lo);
    if (g.epi == EPI_RESID_SCATTER_GATE) e.t[4] = __float_as_uint(((const float*)g.aux1)[int64_t(m) * g.T]);
  }
}
template <typename T>
__device__ __forceinline__ void row_prefetch(const RowProb& g, int m, const RowCols& c, RowPre<T>& e) {
#pragma unroll
  for (int i = 0; i < 5; ++i) asm volatile("" ::"v"(e.t[i]));
  if (g.epi == EPI_SWIGLU) return;
  const int64_t xrow = int64_t(e.bq) * g.T + e.pq;
  const bool scatter = row_scatters(g), resid = scatter || g.epi == EPI_RESID_STORE;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (h == 1 && !c.has_hi) break;
    const int n = h ? c.hi : c.lo;
    if (g.bias) e.bias[h] = load_raw8((const T*)g.bias + n);
    if (scatter && g.bias2) e.bias2[h] = load_raw8((const T*)g.bias2 + n);
    if (scatter && g.aux0) e.res[h] = load_raw8((const T*)g.aux0 + int64_t(m) * g.N + n);
    if (resid && (!(scatter && g.aux0) || g.epi == EPI_RESID_SCATTER_GATE))
      e.x[h] = load_raw8((const T*)row_x(g) + xrow * g.N + n);
  }
  if (g.epi == EPI_RESID_SCATTER_GATE) e.gate = ((const float*)g.aux1)[xrow];
  if (c.rot) {
    const int half = g.R / 2, dim = c.lo & (g.hd - 1);  // hd is a power of two
    const float4* cs = reinterpret_cast<const float4*>((const float*)g.aux2 + (int64_t(e.pq) * half + dim) * 2);
#pragma unroll
    for (int p = 0; p < 4; ++p) e.cs[p] = cs[p];
  }
}

// Finish row m of one column group: v[0..8) are the sums of its lo chunk,
// v[8..16) of its hi chunk. The arithmetic and its order are those of the
// tile GEMMs' epilogues.
template <typename T>
__device__ __forceinline__ void row_epilogue(const RowProb& g, int m, const RowCols& c, float* v,
                                             const RowPre<T>& e) {
  if (g.epi == EPI_SWIGLU) {
    float y[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) y[i] = (sizeof(T) == 2 ? silu_bf16(v[i]) : silu(v[i])) * v[8 + i];
    store8((T*)g.out + int64_t(m) * g.ldo + c.lo, y);
    return;
  }
  const bool scatter = row_scatters(g);
  float bias[16];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int i = 0; i < 8; ++i) bias[8 * h + i] = 0.f;
    if (h == 1 && !c.has_hi) break;
    if (g.bias) unpack8(e.bias[h], bias + 8 * h);
    if (scatter && g.bias2) {
      float b2[8];
      unpack8(e.bias2[h], b2);
#pragma unroll
      for (int i = 0; i < 8; ++i) bias[8 * h + i] += b2[i];
    }
  }
  if (g.epi == EPI_QKV_ROPE) {
    // columns: Q heads, then K heads, then V heads; written head-major [B, H, kk, hd]
    int col = c.lo, heads = g.Hq;
    T* sec = (T*)g.out;
    if (col >= g.Hq * g.hd) {
      col -= g.Hq * g.hd;
      heads = g.Hkv;
      sec = (T*)g.aux0;
      if (col >= g.Hkv * g.hd) {
        col -= g.Hkv * g.hd;
        sec = (T*)g.aux1;
      }
    }
    const int hs = 31 - __clz(g.hd), head = col >> hs, dim = col & (g.hd - 1);
    T* dst = sec + ((int64_t(e.bq) * heads + head) * g.kk + e.jq) * g.hd + dim;
#pragma unroll
    for (int i = 0; i < 16; ++i) v[i] += bias[i];
    if (c.rot) {
      float lo[8], hi[8];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const float4 a = e.cs[p];
        lo[2 * p] = v[2 * p] * a.x - v[8 + 2 * p] * a.y;
        lo[2 * p + 1] = v[2 * p + 1] * a.z - v[8 + 2 * p + 1] * a.w;
        hi[2 * p] = v[8 + 2 * p] * a.x + v[2 * p] * a.y;
        hi[2 * p + 1] = v[8 + 2 * p + 1] * a.z + v[2 * p + 1] * a.w;
      }
      store8(dst, lo);
      store8(dst + g.R / 2, hi);
    } else {
      store8(dst, v);
      store8(dst + 8, v + 8);
    }
    return;
  }
  const int64_t xrow = int64_t(e.bq) * g.T + e.pq;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (h == 1 && !c.has_hi) break;
    const int n = h ? c.hi : c.lo;
    float* w = v + 8 * h;
    const float* bi = bias + 8 * h;
    if (g.epi == EPI_BIAS_GELU) {
#pragma unroll
      for (int i = 0; i < 8; ++i) w[i] = sizeof(T) == 2 ? gelu_bf16(w[i] + bi[i]) : gelu_erf(w[i] + bi[i]);
      store8((T*)g.out + int64_t(m) * g.ldo + n, w);
      continue;
    }
    const bool has_res = scatter && g.aux0;
    float r[8];
    unpack8(has_res ? e.res[h] : e.x[h], r);
    if (g.epi == EPI_RESID_SCATTER_GATE) {
      const float sg = 1.f / (1.f + expf(-e.gate));
      if (has_res) {
        float o[8];
        unpack8(e.x[h], o);
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = o[i] + sg * ((w[i] + bi[i]) + (r[i] - o[i]));
      } else {
#pragma unroll
        for (int i = 0; i < 8; ++i) w[i] = r[i] + sg * (w[i] + bi[i]);
      }
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) w[i] = w[i] + bi[i] + r[i];
    }
    if (g.epi == EPI_RESID_STORE) store8((T*)g.out + int64_t(m) * g.ldo + n, w);
    else store8((T*)g.out + xrow * g.N + n, w);
  }
}

// Mean and 1 / standard deviation of one row of x by one wave (LayerNorm;
// RMSNorm: mean 0): the row's loads (at most kNormVecs vectors per lane), then
// the sums.
constexpr int kNormVecs = kRowGemmNormVecs;
template <typename T>
__device__ __forceinline__ void stat_load(const T* row, int nv, u32x4* raw) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int c = 0; c < kNormVecs; ++c)
    if (64 * c < nv)
      raw[c] = 64 * c + lane < nv ? *reinterpret_cast<const u32x4*>(row + (64 * c + lane) * RowElem<T>::kVec)
                                  : u32x4{0u, 0u, 0u, 0u};
}
template <typename T>
__device__ __forceinline__ void stat_finish(const u32x4* raw, int nv, int d, float eps, bool rms, float* mean,
                                            float* rstd) {
  constexpr int V = RowElem<T>::kVec;
  const int lane = threadIdx.x & 63;
  float mu = 0.f;
  if (!rms) {
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < kNormVecs; ++c)
      if (64 * c < nv) {
        float f[V];
        load_vec(reinterpret_cast<const T*>(&raw[c]), f);
#pragma unroll
        for (int i = 0; i < V; ++i) s += f[i];
      }
    mu = wave_sum_fast(s) / float(d);
  }
  float q = 0.f;
#pragma unroll
  for (int c = 0; c < kNormVecs; ++c)
    if (64 * c < nv) {
      float f[V];
      load_vec(reinterpret_cast<const T*>(&raw[c]), f);
      if (64 * c + lane < nv)
#pragma unroll
        for (int i = 0; i < V; ++i) {
          const float t = f[i] - mu;
          q += t * t;
        }
    }
  q = wave_sum_fast(q);
  if (lane == 0) {
    *mean = mu;
    *rstd = 1.0f / sqrtf(q / float(d) + eps);
  }
}

// y = (x - mean) rstd w + b on one 16-byte vector, rounded to T.
template <typename T>
__device__ __forceinline__ u32x4 row_norm(const u32x4& x, float mean, float rstd, const u32x4& w, const u32x4& b,
                                          bool has_b) {
  constexpr int V = RowElem<T>::kVec;
  float f[V], wf[V], bf[V];
  load_vec(reinterpret_cast<const T*>(&x), f);
  load_vec(reinterpret_cast<const T*>(&w), wf);
  load_vec(reinterpret_cast<const T*>(&b), bf);
#pragma unroll
  for (int i = 0; i < V; ++i) {
    f[i] = (f[i] - mean) * rstd * wf[i];
    if (has_b) f[i] += bf[i];
  }
  u32x4 out;
  store_vec(reinterpret_cast<T*>(&out), f);
  return out;
}
}  // namespace

// MB blocks of 16 rows, NB groups of 16 columns per workgroup, NW waves
// (four resident per SIMD; two for the fp32 tiles, whose accumulators and
// operands take more registers).
template <typename T, int MB, int NB, int NW, bool NORM, bool SPLIT>
__global__ __launch_bounds__(64 * NW, MB * NB >= 16 || (sizeof(T) == 4 && MB * NB >= 4 && NB > 1) ? 2 : 4) void rowgemm_kernel(RowGemmArgs a) {
  using E = RowElem<T>;
  constexpr int VEC = E::kVec, STEP = E::kStep;
  constexpr int LD = 16 * NB + 4;  // 4 rows apart: 16 banks apart
  // k-steps whose loads are in flight together (two groups are: the next
  // one's loads precede the current one's MFMAs), within the register budget
  constexpr int kStepVecs = MB + NB + (NORM ? 2 : 0);
  constexpr int G = kStepVecs <= 2 ? 4 : kStepVecs <= 5 ? 2 : 1;
  constexpr int kRedBytes = NW * 16 * MB * LD * 4;
  constexpr int kRouteBytes = sizeof(T) == 2 && NW == 8 ? (8 * 16 * (64 + 1) + 128) * 4 : 0;
  constexpr int kSmem = kRedBytes > kRouteBytes ? kRedBytes : kRouteBytes;
  __shared__ __attribute__((aligned(16))) char smem[kSmem];
  __shared__ float mean_s[16], rstd_s[16];
  __shared__ int is_last;
  int blk = int(blockIdx.x);
  {  // every line of the arguments at once
    const uint32_t* w = reinterpret_cast<const uint32_t*>(&a);
    constexpr int kLines = int(sizeof(RowGemmArgs)) / 64;
#pragma unroll
    for (int i = 0; i < kLines; ++i) asm volatile("" ::"s"(w[16 * i]));
  }
  if constexpr (sizeof(T) == 2 && NW == 8) {
    if (blk < a.router_wgs) {
      router_rows16(a.r, 16 * blk, reinterpret_cast<float*>(smem));
      return;
    }
  }
  blk -= a.router_wgs;
  int gt = SPLIT ? blk / a.splits : blk, m0 = 0;  // column tile, first row
  const int sl = SPLIT ? blk - gt * a.splits : 0;   // slice of K
  if constexpr (NW == 8 && !NORM && !SPLIT && MB >= 2 && NB >= 2) {  // the row-tile forms
    const int t = gt / a.mtiles;
    m0 = 16 * MB * (gt - t * a.mtiles);
    gt = t;
  }
  const int pi = gt >= a.tiles0 ? 1 : 0;
  const RowProb& g = a.p[pi];
  const int tile = pi ? gt - a.tiles0 : gt;
  const int nsub = g.nsub;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r16 = lane & 15, grp = lane >> 4;
  const int eb = sizeof(T);

  // byte offsets of this lane's rows (rows past the end repeat the last one)
  uint32_t oa[MB], oa2[MB], ob[NB], ob2[NB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    const int m = min(m0 + 16 * mb + r16, g.M - 1);
    oa[mb] = uint32_t(m * g.lda + VEC * grp) * eb;
    oa2[mb] = uint32_t(m * g.lda2 + VEC * grp) * eb;
  }
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const RowCols c = row_cols(g, min(tile * NB + nb, nsub - 1), a.narrow);
    const int row = r16 < 8 ? c.lo + r16 : (c.has_hi ? c.hi : c.lo) + r16 - 8;
    ob[nb] = uint32_t(row * g.ldb + VEC * grp) * eb;
    ob2[nb] = uint32_t(row * g.ldb2 + VEC * grp) * eb;
  }
  const int nst_all = g.K / STEP;
  const int b0 = SPLIT ? int(int64_t(nst_all) * sl / a.splits) : 0;
  const int nst = (SPLIT ? int(int64_t(nst_all) * (sl + 1) / a.splits) : nst_all) - b0, spw = (nst + NW - 1) / NW;
  const int s0 = b0 + wave * spw, cnt = max(0, min(nst - wave * spw, spw));

  struct Frags {
    u32x4 a[G][MB], b[G][NB], w[NORM ? G : 1], c[NORM ? G : 1];
  };
  auto load = [&](Frags& f, int i0) {
#pragma unroll
    for (int i = 0; i < G; ++i) {
      const int k = (s0 + min(i0 + i, cnt - 1)) * STEP;  // past the end: repeat the last step (not used)
      const bool second = k >= g.K1;
      const int kk = second ? k - g.K1 : k;
      const char* pa = (const char*)(second ? g.a2 : g.a) + kk * eb;
      const char* pb = (const char*)(second ? g.b2 : g.b) + kk * eb;
#pragma unroll
      for (int nb = 0; nb < NB; ++nb) f.b[i][nb] = *reinterpret_cast<const u32x4*>(pb + (second ? ob2[nb] : ob[nb]));
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) f.a[i][mb] = *reinterpret_cast<const u32x4*>(pa + (second ? oa2[mb] : oa[mb]));
      if constexpr (NORM) {
        const T* w = (const T*)a.norm_w[pi] + k + VEC * grp;
        const T* b = a.norm_b[pi] ? (const T*)a.norm_b[pi] + k + VEC * grp : w;
        f.w[i] = *reinterpret_cast<const u32x4*>(w);
        f.c[i] = *reinterpret_cast<const u32x4*>(b);
      }
    }
  };
  f32x4 acc[MB][NB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) acc[mb][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  float mu = 0.f, rs = 0.f;
  auto mma = [&](const Frags& f, int i0) {
#pragma unroll
    for (int i = 0; i < G; ++i) {
      if (i0 + i >= cnt) break;
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) {
        u32x4 av = f.a[i][mb];
        if constexpr (NORM) av = row_norm<T>(av, mu, rs, f.w[i], f.c[i], a.norm_b[pi] != nullptr);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) row_mma<T>(acc[mb][nb], av, f.b[i][nb]);
      }
    }
  };
  // one epilogue item per thread: row em of column group tile * NB + en
  static_assert(16 * MB * NB <= 64 * NW, "one item per thread");
  const int em = tid / NB, en = tid - em * NB, es = tile * NB + en;
  const int er = m0 + em;  // its row
  const bool live = er < g.M && es < nsub && tid < 16 * MB * NB;
  const RowCols ec = row_cols(g, min(es, nsub - 1), a.narrow);
  RowPre<T> pre;
  // the rows for the statistics are requested ahead of the weights: loads
  // return in order, and the weights come from memory
  u32x4 raw[NORM ? kNormVecs : 1];
  const int nv = g.K / VEC;
  if constexpr (NORM) stat_load<T>((const T*)g.a + int64_t(min(wave, g.M - 1)) * g.lda, nv, raw);
  Frags f0, f1;
  if (cnt > 0) load(f0, 0);
  if (live) {
    row_place<T>(g, er, pre);
    row_touch<T>(g, er, ec, pre);
  }
  if constexpr (NORM) {
    for (int m = wave; m < g.M; m += NW) {
      if (m != wave) stat_load<T>((const T*)g.a + int64_t(m) * g.lda, nv, raw);
      stat_finish<T>(raw, nv, g.K, a.eps, a.rms != 0, mean_s + m, rstd_s + m);
    }
    __syncthreads();
    const int m = min(r16, g.M - 1);
    mu = mean_s[m];
    rs = rstd_s[m];
  }
  for (int i = 0; i < cnt; i += 2 * G) {
    if (i + G < cnt) load(f1, i + G);
    mma(f0, i);
    if (i + 2 * G < cnt) load(f0, i + 2 * G);
    if (i + G < cnt) mma(f1, i + G);
  }
  if (live) row_prefetch<T>(g, er, ec, pre);
  // lane holds C[16 mb + 4 grp + e][16 nb + r16] of its wave's k range
  float* red = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int e = 0; e < 4; ++e)
        red[(wave * 16 * MB + 16 * mb + 4 * grp + e) * LD + 16 * nb + r16] = acc[mb][nb][e];
  __syncthreads();
  float v[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = 0.f;
  if (live) {
#pragma unroll 2
    for (int w = 0; w < NW; ++w) {
      const f32x4* p = reinterpret_cast<const f32x4*>(red + (w * 16 * MB + em) * LD + 16 * en);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const f32x4 x = p[i];
#pragma unroll
        for (int e = 0; e < 4; ++e) v[4 * i + e] += x[e];
      }
    }
  }
  if constexpr (SPLIT) {
    if (a.splits > 1) {
      // Hand-over between the tile's slices, as in the split-K QKV kernel:
      // device-coherent stores complete, a device-scope counter moves, and
      // the last slice to arrive (which resets the counter) adds all of them
      // in slice order. No workgroup waits for another.
      constexpr int kItems = 16 * MB * NB, kCoherent = 16;  // cache policy: sc1
      const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(a.part, (short)0, 0x7fffffff, 0x00020000);
      const int base = (gt * a.splits) * (kItems * 64) + tid * 64;
      if (live) {
        const int at = base + sl * (kItems * 64);
#pragma unroll
        for (int i = 0; i < 4; ++i)
          __builtin_amdgcn_raw_buffer_store_b128(
              u32x4{__float_as_uint(v[4 * i]), __float_as_uint(v[4 * i + 1]), __float_as_uint(v[4 * i + 2]),
                    __float_as_uint(v[4 * i + 3])},
              rsrc, at + 16 * i, 0, kCoherent);
      }
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (tid == 0) {
        const uint32_t old = __hip_atomic_fetch_add(a.count + gt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        is_last = old == uint32_t(a.splits - 1);
        if (is_last) __hip_atomic_store(a.count + gt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
      __syncthreads();
      if (!is_last || !live) return;
#pragma unroll
      for (int i = 0; i < 16; ++i) v[i] = 0.f;
      for (int s4 = 0; s4 < a.splits; s4 += 4) {
        u32x4 x[4][4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            x[j][i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, base + min(s4 + j, a.splits - 1) * (kItems * 64) + 16 * i,
                                                            0, kCoherent);
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (s4 + j < a.splits)
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
              for (int e = 0; e < 4; ++e) v[4 * i + e] += __uint_as_float(x[j][i][e]);
      }
    }
  }
  if (live) row_epilogue<T>(g, er, ec, v, pre);
}

bool rowgemm_ok(const GemmArgs& g) {
  const int eb = g.dtype == DSF_BF16 ? 2 : 4, step = 4 * (16 / eb);
  if (g.M < 1 || g.epi >= EPI_STORE || g.K % step || g.K1 % step || g.K < 1) return false;
  if (g.lda % 8 || g.ldb % 8 || (g.a2 && g.lda2 % 8) || (g.b2 && g.ldb2 % 8) || g.N % 8) return false;
  if (g.epi == EPI_SWIGLU && g.f % 8) return false;
  if (g.epi == EPI_QKV_ROPE && (g.R % 16 || g.hd % 16)) return false;
  // 32-bit byte offsets
  if (g.dtype == DSF_BF16 && g.M > kRowGemmMaxRows) return false;
  const int64_t rows_b = g.epi == EPI_SWIGLU ? 2 * int64_t(g.f) : g.N, lim = (int64_t(1) << 31) - 1;
  return rows_b * g.ldb * eb < lim && (!g.b2 || rows_b * g.ldb2 * eb < lim) &&
         int64_t(std::max(g.M, kRowGemmMaxRows)) * std::max(g.lda, g.lda2) * eb < lim;
}

static RowProb row_prob(const GemmArgs& g) {
  RowProb r{};
  r.a = g.a; r.b = g.b; r.a2 = g.a2; r.b2 = g.b2;
  r.bias = g.bias; r.bias2 = g.bias2;
  r.idx = g.idx;
  r.M = g.M; r.N = g.N; r.K = g.K; r.K1 = g.K1;
  r.lda = g.lda; r.lda2 = g.lda2; r.ldb = g.ldb; r.ldb2 = g.ldb2;
  r.epi = g.epi; r.kk = g.kk; r.T = g.T; r.f = g.f; r.ldo = g.ldo;
  r.Hq = g.Hq; r.Hkv = g.Hkv; r.hd = g.hd; r.R = g.R;
  r.nsub = g.epi == EPI_SWIGLU ? g.f / 8 : (g.N + 15) / 16;
  r.out = g.out;
  if (g.epi == EPI_QKV_ROPE) {
    r.out = g.q; r.aux0 = g.k; r.aux1 = g.v; r.aux2 = g.rope;
  } else if (g.epi == EPI_RESID_STORE) {
    r.aux0 = g.x;
  } else if (g.epi == EPI_RESID_SCATTER || g.epi == EPI_RESID_SCATTER_GATE) {
    r.out = g.x; r.aux0 = const_cast<void*>(g.res); r.aux1 = const_cast<float*>(g.gate);
  }
  return r;
}

// fp32 projections of more rows, on the fp32 matrix cores: the same kernel
// over tiles of 16 MB x 16 NB outputs, K split between the tile's eight waves.
// One MFMA step of a 64 x 64 tile is 2048 cycles of a SIMD's matrix core for
// 8 KB of operands, so they come straight from L1/L2 without staging. The
// largest tile that still gives most CUs a workgroup is taken. GPT-NeoX-160M
// layer, 307 rows: 26 (QKV) and 37 us (up) side by side and 34 us (down),
// against 73, 71 and 320 us of the scalar kernel (a chain of 3840 products
// per output in the last).
static hipError_t launch_row_tiles_f32(const GemmArgs* p, int np, hipStream_t s) {
  int nsub = 0;
  for (int i = 0; i < np; ++i) nsub += row_prob(p[i]).nsub;
  const int M = p[0].M;
  auto tiles = [&](int mb, int nb) { return int64_t((M + 16 * mb - 1) / (16 * mb)) * ((nsub + nb - 1) / nb); };
  const int mb = tiles(4, 4) >= kRowTilesF32 ? 4 : 2;
  const int nb = mb == 4 || tiles(2, 4) >= kRowTilesF32 ? 4 : 2;
  RowGemmArgs a{};
  for (int i = 0; i < np; ++i) a.p[i] = row_prob(p[i]);
  a.splits = 1;
  a.mtiles = (M + 16 * mb - 1) / (16 * mb);
  a.tiles0 = (a.p[0].nsub + nb - 1) / nb;
  const int nt = a.tiles0 + (np > 1 ? (a.p[1].nsub + nb - 1) / nb : 0);
  const dim3 grid(unsigned(nt) * unsigned(a.mtiles)), block(512);
  if (mb == 4) launch_with_timing(rowgemm_kernel<float, 4, 4, 8, false, false>, grid, block, s, a);
  else if (nb == 4) launch_with_timing(rowgemm_kernel<float, 2, 4, 8, false, false>, grid, block, s, a);
  else launch_with_timing(rowgemm_kernel<float, 2, 2, 8, false, false>, grid, block, s, a);
  return hipGetLastError();
}

// the split forms' tiles are 128 items of 64 bytes (32 x 64 or 64 x 32 outputs)
size_t rowgemm_split_bytes() { return size_t(kRowSplitWgs) * 128 * 64; }

hipError_t launch_rowgemm(const GemmArgs* p, int np, const RowGemmNorm* norm, const RouterRows* router,
                          const RowGemmSplit* split, hipStream_t s) {
  const int M = p[0].M, epi = p[0].epi;
  const bool bf = p[0].dtype == DSF_BF16;
  if (!bf && M > kRowGemmMaxRows) return launch_row_tiles_f32(p, np, s);
  if (norm && M > kRowGemmNormRows) return hipErrorInvalidValue;
  RowGemmArgs a{};
  for (int i = 0; i < np; ++i) a.p[i] = row_prob(p[i]);
  if (norm) {
    for (int i = 0; i < np; ++i) {
      a.norm_w[i] = norm->w[i];
      a.norm_b[i] = norm->b[i];
    }
    a.eps = norm->eps;
    a.rms = norm->rms;
  }
  if (router) {
    a.r = *router;
    a.router_wgs = int((router->n + 15) / 16);
  }
  // few columns for the depth of the reduction: groups of 8, twice the workgroups
  if (np == 1 && !norm && M <= 16 && epi != EPI_SWIGLU && epi != EPI_QKV_ROPE && a.p[0].nsub <= kRowNarrowMax) {
    a.narrow = 1;
    a.p[0].nsub = p[0].N / 8;
  }
  a.splits = 1;
  a.mtiles = 1;
  const int nsub = a.p[0].nsub + (np > 1 ? a.p[1].nsub : 0), nst = p[0].K / (bf ? 32 : 16);
  int nb = bf && nsub >= kRowWideMin ? 2 : 1;
  auto set_tiles = [&]() {
    a.tiles0 = (a.p[0].nsub + nb - 1) / nb;
    return a.tiles0 + (np > 1 ? (a.p[1].nsub + nb - 1) / nb : 0);
  };
  int tiles = set_tiles();
  // More than 16 rows of a deep reduction: wider tiles, split along K.
  const int mb = M <= 16 ? 1 : M <= 32 ? 2 : 4;
  bool wide = false;
  if (bf && mb > 1 && split && split->part && nst >= kRowSplitMinSteps) {
    const int nb1 = nb;
    nb = mb == 2 ? 4 : 2;
    tiles = set_tiles();
    int sp = std::min(std::min(kRowSplitWgs / tiles, kRowSplitMax), nst / 16);
    const size_t tile_bytes = size_t(16 * mb * nb) * 64;
    sp = int(std::min<size_t>(size_t(std::max(sp, 1)), split->part_bytes / (tile_bytes * size_t(tiles))));
    if (sp >= 2 && tiles <= split->counts && size_t(tiles) * sp * tile_bytes < (size_t(1) << 31)) {
      wide = true;
      a.splits = sp;
      a.part = (float*)split->part;
      a.count = split->count;
    } else {
      nb = nb1;
      tiles = set_tiles();
    }
  }
  // a grid that leaves CUs with one workgroup or none: sixteen waves each
  const bool deep = !wide && nb == 1 && tiles <= 256 && !norm && !router;
  const dim3 grid(unsigned(a.router_wgs + tiles * a.splits)), block(deep ? 1024 : 512);
#define DSF_ROWGEMM(T, MB, NB, NW, NORM, SPLIT) \
  launch_with_timing(rowgemm_kernel<T, MB, NB, NW, NORM, SPLIT>, grid, block, s, a)
#define DSF_ROWGEMM_T(T, NB)                                   \
  do {                                                         \
    if (norm) DSF_ROWGEMM(T, 1, NB, 8, true, false);           \
    else if (mb == 1) DSF_ROWGEMM(T, 1, NB, 8, false, false);  \
    else if (mb == 2) DSF_ROWGEMM(T, 2, NB, 8, false, false);  \
    else DSF_ROWGEMM(T, 4, NB, 8, false, false);               \
  } while (0)
#define DSF_ROWGEMM_DEEP(T)                                    \
  do {                                                         \
    if (mb == 1) DSF_ROWGEMM(T, 1, 1, 16, false, false);       \
    else if (mb == 2) DSF_ROWGEMM(T, 2, 1, 16, false, false);  \
    else DSF_ROWGEMM(T, 4, 1, 16, false, false);               \
  } while (0)
  if (bf) {
    if (wide && mb == 2) DSF_ROWGEMM(uint16_t, 2, 4, 8, false, true);
    else if (wide) DSF_ROWGEMM(uint16_t, 4, 2, 8, false, true);
    else if (deep) DSF_ROWGEMM_DEEP(uint16_t);
    else if (nb == 2) DSF_ROWGEMM_T(uint16_t, 2);
    else DSF_ROWGEMM_T(uint16_t, 1);
  } else {
    if (deep) DSF_ROWGEMM_DEEP(float);
    else DSF_ROWGEMM_T(float, 1);
  }
#undef DSF_ROWGEMM_DEEP
#undef DSF_ROWGEMM_T
#undef DSF_ROWGEMM
  return hipGetLastError();
}

}  // namespace dsf
