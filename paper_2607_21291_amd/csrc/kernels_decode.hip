// Incremental decoding with per-layer caches of the kept tokens' keys and
// values (the paper treats prefill only; the decode-time routing rule is a
// threshold on the new token's router score, and a kept token attends
// causally over the layer's cached kept tokens).
//
// The projections of a decode step run on the few-row GEMM and the routing
// flags come from the router (bf16: workgroups of that GEMM's first launch);
// the kernels here are the other pieces decoding adds:
// - attention of one query per (sequence, head) over its cache and the new
//   token, split into chunks of keys whose last-arriving workgroup combines
//   them in chunk order (memory-bound: it reads the cache once), which also
//   appends the kept tokens' keys and values to the caches;
// - for a prefill: copying each layer's kept keys/values into the caches and
//   the lowest kept score per sequence (the threshold that continues the
//   prompt's selection).
#include <algorithm>

#include "dsf_device.h"
#include "dsf_internal.h"

namespace dsf {

// ------------------------------------------------------- decode attention

template <typename T>
__device__ __forceinline__ T round_to(float v) {
  if constexpr (sizeof(T) == 2) return f2bf(v);
  else return v;
}

__device__ __forceinline__ float wave_max_dec(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// Block-wide max over 256 threads (4 wavefronts) through LDS.
__device__ __forceinline__ float block4_max(float v, float* red) {
  v = wave_max_dec(v);
  const int w = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  const float r = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  __syncthreads();
  return r;
}
constexpr int kDecChunk = 256;  // keys per workgroup of the decode attention

// Sum over the lanes of a wavefront that share lane % L (L a power of two
// from 4 to 32): DPP row rotations within 16-lane rows, row swaps beyond.
template <int L>
__device__ __forceinline__ float strided_sum(float v) {
  if constexpr (L <= 4) v += DSF_DPP(v, 0x124);  // row_ror:4
  if constexpr (L <= 8) v += DSF_DPP(v, 0x128);  // row_ror:8
  if constexpr (L <= 16) return rows4_sum(v);
  auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}
// N 32-bit words at p (aligned to their size, 16 bytes at most), and the
// elements they hold as fp32.
template <int N>
__device__ __forceinline__ void load_words(const void* p, uint32_t* w) {
  if constexpr (N == 1) {
    w[0] = *reinterpret_cast<const uint32_t*>(p);
  } else if constexpr (N == 2) {
    const u32x2 t = *reinterpret_cast<const u32x2*>(p);
    w[0] = t[0];
    w[1] = t[1];
  } else {
#pragma unroll
    for (int j = 0; j < N / 4; ++j) {
      const u32x4 t = reinterpret_cast<const u32x4*>(p)[j];
#pragma unroll
      for (int i = 0; i < 4; ++i) w[4 * j + i] = t[i];
    }
  }
}
template <typename T, int N>
__device__ __forceinline__ void widen_words(const uint32_t* w, float* v) {
#pragma unroll
  for (int i = 0; i < N; ++i)
    v[i] = sizeof(T) == 4 ? __uint_as_float(w[i * int(sizeof(T)) / 4])
                          : __uint_as_float(i & 1 ? w[i / 2] & 0xffff0000u : w[i / 2] << 16);
}
__device__ __forceinline__ float row16_max(float v) {
  v = fmaxf(v, DSF_DPP(v, 0xB1));   // quad_perm [1,0,3,2]
  v = fmaxf(v, DSF_DPP(v, 0x4E));   // quad_perm [2,3,0,1]
  v = fmaxf(v, DSF_DPP(v, 0x141));  // row_half_mirror
  return fmaxf(v, DSF_DPP(v, 0x140));  // row_mirror
}

// Attention of one new token per sequence over its cache. Workgroup (chunk c,
// block of up to GB query heads of one kv head, sequence b): keys c * 256 ..
// of the len = len_in[b] (+ 1 if kept) valid slots, read once for all of the
// block's heads (grouped-query attention: a workgroup per query head re-read
// the cache Hq / Hkv times; Qwen2.5-7B heads, 32 sequences of 1.8k keys: 243
// us). Wave w takes 64 keys. Scores are MFMA products, the heads as the 16
// rows of A and 16 keys as B, both loaded from global memory in the operand
// layout (16 bytes per lane); every key and value vector is requested before
// the first is used where the registers allow. Each wave takes its own
// maximum m and sum l of exp(s - m), p = exp(s - m) goes through LDS, and
// o = sum_t p_t v_t stays in fp32: for one or two heads on the vector ALUs, a
// lane owning one 16-byte vector of dims; for more (GB = 16) as fp32 MFMA
// products of 4 keys, lane (r16, grp) holding HD / 16 neighbouring dims of key
// grp as they come from memory, element e of every lane forming one product
// (on the vector ALUs eight heads took 64 accumulators, their sums over the
// row groups and one wave per SIMD: 149 us on the shape above, 44 this way). The four
// waves combine through LDS in wave order. A sequence of one chunk is finished there; otherwise the
// chunk publishes {m, l, o[0..HD)} per head with device-coherent stores and
// counts itself on the head block's counter, and the last of the sequence's
// ceil(len / 256) chunks resets the counter and combines them in chunk
// order. No workgroup waits for another; chunks past len leave at once.
//
// With keep non-null the launch also appends the step's new key and value
// rows (knew, vnew [B, Hkv, HD]) of every kept sequence: attention reads them
// from there as slot len_in[b], the first head block of each kv head copies
// them into that slot (read by nobody here), and one workgroup sets
// cache_len[b]. len_in is the router's copy of the lengths, so no workgroup
// reads cache_len.
template <typename T, int HD, int GB>
__global__ __launch_bounds__(256, 2) void decode_attn_kernel(const T* __restrict__ q, const T* __restrict__ ck,
                                                          const T* __restrict__ cv, int32_t* __restrict__ cache_len,
                                                          const int32_t* __restrict__ len_in,
                                                          const T* __restrict__ knew, const T* __restrict__ vnew,
                                                          const int32_t* __restrict__ keep, int Hq, int Hkv, int cap,
                                                          int nch_max, float* __restrict__ part,
                                                          uint32_t* __restrict__ count, T* __restrict__ out) {
  constexpr int VEC = 16 / int(sizeof(T));  // elements per 16-byte vector
  constexpr int STEP = 4 * VEC;             // dims per k-step of the score product
  constexpr int NK = HD / STEP;             // k-steps
  constexpr bool kMfmaPV = GB == 16;
  constexpr int LPR = kMfmaPV ? 16 : HD / VEC;  // lanes per value row
  constexpr int DPL = HD / LPR;             // dims per lane
  constexpr int NWD = DPL * int(sizeof(T)) / 4;  // 32-bit words of them
  constexpr int RPP = 64 / LPR;             // value rows per pass of a wave
  constexpr int NPV = 64 / RPP;             // passes over a wave's 64 keys
  // key and value vectors all in flight at once, or the values after the scores
  constexpr bool kBoth = 16 * NK + NPV * NWD <= 128;
  static_assert(GB <= 16, "heads are the rows of one MFMA operand");
  // probabilities of a wave's 64 keys: [key][head], or [head][key] (rows 4 banks apart)
  constexpr int kPs = kMfmaPV ? 16 * 68 : 64 * GB;
  __shared__ __attribute__((aligned(16))) float ps[4][kPs];
  auto ps_at = [](int h, int key) { return kMfmaPV ? h * 68 + key : key * GB + h; };
  __shared__ float osum[4][GB][HD];
  __shared__ float wm[4][GB], wl[4][GB];
  __shared__ int is_last;
  const int c = blockIdx.y;
  const int group = Hq / Hkv, nhb = (group + GB - 1) / GB;
  const int b = int(blockIdx.x) / (Hkv * nhb), kh = int(blockIdx.x) - b * (Hkv * nhb);
  const int kvh = kh / nhb, hb = kh - kvh * nhb;
  const int h0 = kvh * group + hb * GB, ng = min(GB, group - hb * GB);
  const int len_old = min(len_in[b], cap);
  const int kp = keep && keep[b] && len_old < cap ? 1 : 0;  // the new token joins at slot len_old
  const int len = len_old + kp;
  const int nch = max(1, (len + kDecChunk - 1) / kDecChunk);
  if (c >= nch) return;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int r16 = lane & 15, grp = lane >> 4, sub = lane % LPR, row = lane / LPR;
  const int64_t kv0 = (int64_t(b) * Hkv + kvh) * cap;
  const T* kbase = ck + kv0 * HD;
  const T* vbase = cv + kv0 * HD;
  const T* knb = knew + (int64_t(b) * Hkv + kvh) * HD;
  const T* vnb = vnew + (int64_t(b) * Hkv + kvh) * HD;
  // row `key` (clamped below len; an empty cache reads nothing): a cached slot, or the new token at slot len_old
  auto krow = [&](int key) { return key < len_old ? kbase + int64_t(key) * HD : knb; };
  auto vrow = [&](int key) { return key < len_old ? vbase + int64_t(key) * HD : vnb; };
  const int k0 = c * kDecChunk + 64 * w;
  const u32x4 zero = {0u, 0u, 0u, 0u};
  // heads as the rows of A; rows past the block's heads are zero
  u32x4 qf[NK], kf[4][NK];
  uint32_t vf[NPV][NWD];
#pragma unroll
  for (int s = 0; s < NK; ++s)
    qf[s] = r16 < ng ? *reinterpret_cast<const u32x4*>(q + (int64_t(b) * Hq + h0 + r16) * HD + STEP * s + VEC * grp)
                     : zero;
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    const int key = k0 + 16 * kb + r16;
    const T* kr = krow(key) + VEC * grp;
#pragma unroll
    for (int s = 0; s < NK; ++s) kf[kb][s] = key < len ? *reinterpret_cast<const u32x4*>(kr + STEP * s) : zero;
  }
  auto load_v = [&]() {
#pragma unroll
    for (int p = 0; p < NPV; ++p) {
      const int key = k0 + p * RPP + row;
      if (key < len) {
        load_words<NWD>(vrow(key) + sub * DPL, vf[p]);
      } else {
#pragma unroll
        for (int i = 0; i < NWD; ++i) vf[p][i] = 0u;
      }
    }
  };
  if constexpr (kBoth) load_v();
  if (kp && hb == 0 && c == len_old / kDecChunk) {
    // the new rows into slot len_old, 16 bytes a lane
    if (tid < HD / VEC) {
      *reinterpret_cast<u32x4*>(const_cast<T*>(kbase) + int64_t(len_old) * HD + tid * VEC) =
          *reinterpret_cast<const u32x4*>(knb + tid * VEC);
      *reinterpret_cast<u32x4*>(const_cast<T*>(vbase) + int64_t(len_old) * HD + tid * VEC) =
          *reinterpret_cast<const u32x4*>(vnb + tid * VEC);
    }
    if (kvh == 0 && tid == 0) cache_len[b] = len;
  }
  const float scale = 1.0f / sqrtf(float(HD));
  float s[4][4];  // scores of heads 4 grp + i, keys k0 + 16 kb + r16
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int t = 0; t < NK; ++t) {
      if constexpr (sizeof(T) == 2) {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, qf[t]),
                                                      __builtin_bit_cast(bf16x8, kf[kb][t]), acc, 0, 0, 0);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(qf[t][e]), __uint_as_float(kf[kb][t][e]), acc, 0,
                                                     0, 0);
      }
    }
    const bool ok = k0 + 16 * kb + r16 < len;
#pragma unroll
    for (int i = 0; i < 4; ++i) s[kb][i] = ok ? acc[i] * scale : -INFINITY;
  }
  if constexpr (!kBoth) load_v();
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int h = 4 * grp + i;
    const float m = row16_max(fmaxf(fmaxf(s[0][i], s[1][i]), fmaxf(s[2][i], s[3][i])));
    float l = 0.f;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      const float p = s[kb][i] == -INFINITY ? 0.f : expf(s[kb][i] - m);
      l += p;
      if (h < GB) ps[w][ps_at(h, 16 * kb + r16)] = p;
    }
    l = row16_sum(l);
    if (r16 == 0 && h < GB) {
      wm[w][h] = m;
      wl[w][h] = l;
    }
  }
  // a wave reads back only its own probabilities
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0)
  __builtin_amdgcn_wave_barrier();
  if constexpr (kMfmaPV) {
    f32x4 o[DPL];  // o[e]: heads 4 grp + i, dim DPL r16 + e
#pragma unroll
    for (int e = 0; e < DPL; ++e) o[e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int p = 0; p < NPV; ++p) {
      const float pa = ps[w][ps_at(r16, 4 * p + grp)];
      float v[DPL];
      widen_words<T, DPL>(vf[p], v);
#pragma unroll
      for (int e = 0; e < DPL; ++e) o[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(pa, v[e], o[e], 0, 0, 0);
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (4 * grp + i < ng)
#pragma unroll
        for (int e = 0; e < DPL; ++e) osum[w][4 * grp + i][DPL * r16 + e] = o[e][i];
  } else {
    float o[GB][DPL];
#pragma unroll
    for (int h = 0; h < GB; ++h)
#pragma unroll
      for (int i = 0; i < DPL; ++i) o[h][i] = 0.f;
#pragma unroll
    for (int p = 0; p < NPV; ++p) {
      float v[DPL];
      widen_words<T, DPL>(vf[p], v);
#pragma unroll
      for (int h = 0; h < GB; ++h) {
        const float pp = ps[w][ps_at(h, p * RPP + row)];
#pragma unroll
        for (int i = 0; i < DPL; ++i) o[h][i] = fmaf(pp, v[i], o[h][i]);
      }
    }
#pragma unroll
    for (int h = 0; h < GB; ++h)
#pragma unroll
      for (int i = 0; i < DPL; ++i) {
        const float t = strided_sum<LPR>(o[h][i]);
        if (row == 0) osum[w][h][sub * DPL + i] = t;
      }
  }
  __syncthreads();
  // combine the four waves in order: element (head, dim)
  constexpr int kItems = GB * HD;
  for (int e = tid; e < kItems; e += 256) {
    const int h = e / HD, dim = e - h * HD;
    if (h >= ng) break;
    const float M = fmaxf(fmaxf(wm[0][h], wm[1][h]), fmaxf(wm[2][h], wm[3][h]));
    float O = 0.f, L = 0.f;
    if (M != -INFINITY) {
#pragma unroll
      for (int ww = 0; ww < 4; ++ww) {
        const float f = wm[ww][h] == -INFINITY ? 0.f : expf(wm[ww][h] - M);
        O = fmaf(osum[ww][h][dim], f, O);
        L = fmaf(wl[ww][h], f, L);
      }
    }
    const int64_t bh = int64_t(b) * Hq + h0 + h;
    if (nch == 1) {
      out[bh * HD + dim] = round_to<T>(L > 0.f ? O / L : 0.f);
    } else {
      float* dst = part + (bh * nch_max + c) * (HD + 2);
      __hip_atomic_store(dst + 2 + dim, O, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (dim == 0) {
        __hip_atomic_store(dst, M, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(dst + 1, L, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
  if (nch == 1) return;
  // the device-coherent stores complete before the counter moves; the last
  // chunk reads them back with device-coherent loads
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) {
    uint32_t* cnt = count + int64_t(b) * Hq + h0;
    const uint32_t old = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    is_last = old == uint32_t(nch - 1);
    if (is_last) __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (!is_last) return;
  // combine in chunk order, elements (head, dim) of this thread four at a
  // time: all loads of eight chunks of them are in flight together
  const float* pb = part + (int64_t(b) * Hq + h0) * nch_max * (HD + 2);
  constexpr int IT = (kItems + 255) / 256, IG = IT < 4 ? IT : 4;
  for (int i0 = 0; i0 < IT && tid + 256 * i0 < ng * HD; i0 += IG) {
    float M[IG], L[IG], O[IG];
#pragma unroll
    for (int i = 0; i < IG; ++i) {
      M[i] = -INFINITY;
      L[i] = O[i] = 0.f;
    }
    for (int c0 = 0; c0 < nch; c0 += 8) {
      float v[IG][8], m[IG][8], l[IG][8];
#pragma unroll
      for (int i = 0; i < IG; ++i) {
        const int e = min(tid + 256 * (i0 + i), ng * HD - 1);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float* p = pb + (int64_t(e / HD) * nch_max + min(c0 + j, nch - 1)) * (HD + 2);
          m[i][j] = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          l[i][j] = __hip_atomic_load(p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          v[i][j] = __hip_atomic_load(p + 2 + e % HD, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      }
#pragma unroll
      for (int i = 0; i < IG; ++i) {
        float mx = M[i];
#pragma unroll
        for (int j = 0; j < 8; ++j) mx = fmaxf(mx, m[i][j]);  // past the end: the last chunk again
        if (mx == -INFINITY) continue;
        const float f0 = M[i] == -INFINITY ? 0.f : expf(M[i] - mx);
        O[i] *= f0;
        L[i] *= f0;
        M[i] = mx;
#pragma unroll
        for (int j = 0; j < 8; ++j)
          if (c0 + j < nch && m[i][j] != -INFINITY) {
            const float f = expf(m[i][j] - mx);
            O[i] = fmaf(v[i][j], f, O[i]);
            L[i] = fmaf(l[i][j], f, L[i]);
          }
      }
    }
#pragma unroll
    for (int i = 0; i < IG; ++i) {
      const int e = tid + 256 * (i0 + i);
      if (e < ng * HD)
        out[(int64_t(b) * Hq + h0) * HD + e] = round_to<T>(L[i] > 0.f ? O[i] / L[i] : 0.f);
    }
  }
}

int decode_attn_chunks(int cap) { return (cap + kDecChunk - 1) / kDecChunk; }

hipError_t launch_decode_attention(int dtype, const void* q, const void* ck, const void* cv, int32_t* cache_len,
                                   const int32_t* len_in, const void* knew, const void* vnew, const int32_t* keep,
                                   int B, int Hq, int Hkv, int hd, int cap, float* part, uint32_t* count, void* out,
                                   hipStream_t s) {
  if (B == 0) return hipSuccess;
  if (cap > kDecodeMaxCap) return hipErrorInvalidValue;
  const int nch = decode_attn_chunks(cap), group = Hq / Hkv;
  auto run = [&](auto tag, auto hdc, auto gbc) -> hipError_t {
    using T = decltype(tag);
    constexpr int HD = decltype(hdc)::value, GB = decltype(gbc)::value;
    // chunks outermost: the chunks past a sequence's length, which leave at
    // once, are dispatched last (with the chunk innermost they alternated with
    // the others and the dispatch put all the work on half of the CUs: 77 us
    // for 1.8k keys in caches of 4096 slots)
    const dim3 grid(unsigned(B) * Hkv * ((group + GB - 1) / GB), nch);
    decode_attn_kernel<T, HD, GB><<<grid, 256, 0, s>>>((const T*)q, (const T*)ck, (const T*)cv, cache_len, len_in,
                                                       (const T*)knew, (const T*)vnew, keep, Hq, Hkv, cap, nch, part,
                                                       count, (T*)out);
    return hipGetLastError();
  };
  // heads per workgroup: the vector-ALU forms for one or two, the MFMA form for more (blocks of 16)
  auto run_g = [&](auto tag, auto hdc) -> hipError_t {
    if (group == 1) return run(tag, hdc, std::integral_constant<int, 1>());
    if (group == 2) return run(tag, hdc, std::integral_constant<int, 2>());
    return run(tag, hdc, std::integral_constant<int, 16>());
  };
  auto run_t = [&](auto tag) -> hipError_t {
    switch (hd) {
      case 32: return run_g(tag, std::integral_constant<int, 32>());
      case 64: return run_g(tag, std::integral_constant<int, 64>());
      case 128: return run_g(tag, std::integral_constant<int, 128>());
      default: return hipErrorInvalidValue;
    }
  };
  return dtype == DSF_BF16 ? run_t(uint16_t()) : run_t(float());
}

// ------------------------------------------------------------- prefill

// Rows j < k of src [B, Hkv, k, hd] -> slots 0..k-1 of the caches [B, Hkv, cap, hd];
// cache_len[b] = k for every sequence (written by the first workgroup).
__global__ void kv_fill_kernel(const u32x4* __restrict__ ks, const u32x4* __restrict__ vs, u32x4* __restrict__ ck,
                               u32x4* __restrict__ cv, int32_t* __restrict__ cache_len, int B, int Hkv, int k, int cap,
                               int row_vecs) {
  const int64_t n = int64_t(B) * Hkv * k * row_vecs;
  for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x) {
    const int64_t e = i % row_vecs, r = i / row_vecs;  // r = (b * Hkv + h) * k + j
    const int64_t j = r % k, bh = r / k;
    ck[(bh * cap + j) * row_vecs + e] = ks[i];
    cv[(bh * cap + j) * row_vecs + e] = vs[i];
  }
  if (blockIdx.x == 0)
    for (int b = threadIdx.x; b < B; b += blockDim.x) cache_len[b] = k;
}

hipError_t launch_kv_fill(int dtype, const void* ks, const void* vs, void* ck, void* cv, int32_t* cache_len, int B,
                          int Hkv, int hd, int k, int cap, hipStream_t s) {
  if (B == 0) return hipSuccess;
  const int row_vecs = hd * (dtype == DSF_BF16 ? 2 : 4) / 16;
  const int64_t n = int64_t(B) * Hkv * k * row_vecs;
  const int blocks = int(std::min<int64_t>(std::max<int64_t>((n + 255) / 256, 1), 4096));
  kv_fill_kernel<<<blocks, 256, 0, s>>>((const u32x4*)ks, (const u32x4*)vs, (u32x4*)ck, (u32x4*)cv, cache_len, B, Hkv,
                                        k, cap, row_vecs);
  return hipGetLastError();
}

// thr[b] = min over the kept tokens of scores[b, idx[b, j]] (+inf for k = 0).
__global__ __launch_bounds__(256) void kept_min_score_kernel(const float* __restrict__ scores,
                                                             const int32_t* __restrict__ idx, int T, int k,
                                                             float* __restrict__ thr) {
  __shared__ float red[4];
  const int b = blockIdx.x;
  float v = INFINITY;
  for (int j = threadIdx.x; j < k; j += 256) v = fminf(v, scores[int64_t(b) * T + clamp_pos(idx[int64_t(b) * k + j], T)]);
  v = -block4_max(-v, red);
  if (threadIdx.x == 0) thr[b] = v;
}

hipError_t launch_kept_min_score(const float* scores, const int32_t* idx, int B, int T, int k, float* thr,
                                 hipStream_t s) {
  if (B == 0) return hipSuccess;
  kept_min_score_kernel<<<B, 256, 0, s>>>(scores, idx, T, k, thr);
  return hipGetLastError();
}

}  // namespace dsf
