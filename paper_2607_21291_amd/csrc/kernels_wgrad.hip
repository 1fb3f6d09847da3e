// Weight gradients of the layer's backward: dW[M, N] = sum_t P[t, m] Q[t, n]
// (fp32) over the kept tokens t, with P the gradient at a projection's output
// and Q its input, both bf16 and token-major as the rest of the backward
// leaves them, and optionally the column sums of P (the bias gradient).
//
// A reduction over tokens contracts the slow dimension of both operands.
// The forward's GEMM kernels read rows along the reduction, which took a
// transposed copy of every operand first; here tiles of 64 tokens go to LDS
// row-major by buffer DMA (the layout of attn_tiles.h) and both MFMA operands
// come from LDS with the transpose load, so nothing is copied. The column
// sums ride along as one more MFMA per P fragment, against ones, in the
// workgroups of the first column tile.
//
// A GPT-NeoX layer has 36-144 tiles of 128 x 128 with reductions of 10k
// tokens: the tokens are split between workgroups. All but the last slice of a
// tile store their partial tiles with device-coherent stores and raise a flag;
// the last slice adds them in order (deterministic). Only last slices wait,
// and the workgroups of an XCD that never wait are dispatched before those
// that do, so the waits end; a bounded spin guards them (status word on a
// give-up). (The stream-K grid this replaces ended in a chain of up to
// fourteen flag waits and serial adds per tile: 99 us for each of the four
// gradients of the NeoX-160M layer at 12504 rows, whatever their size.)
#include <algorithm>

#include "attn_tiles.h"
#include "dsf_device.h"
#include "dsf_internal.h"

namespace dsf {

namespace {
constexpr int kWgK = kAttnTileRows;      // tokens per LDS tile
constexpr int kWgSub = 128;              // columns per LDS subtile
constexpr int kWgSubBytes = kWgK * kWgSub * 2;
// Token tiles per slice, at least: a hand-over costs a few of them. Training
// step of a NeoX-160M layer, 300 rows, with 1 / 2 / 4 / 8: 249 / 226 / 209 / 209 us; 1400
// rows 330 / 328 / 317 / 310; 12504 rows 1099 / 1098 / 1103 / 1103.
constexpr int kWgMinTiles = 4;
// 256 x 256 tiles from which they are taken: more than a round of the CUs, as
// their grids are not split. Training step of a layer with large / small tiles:
// Qwen2.5-1.5B, 6000 rows (420 for the up projection) 2370 / 2390 us; at 256 tiles
// (NeoX-1.4B, 6000 rows), where the line keeps the small ones, 2087 / 2145.
constexpr int kWgLargeMin = 320;

struct WgArgs {
  const uint16_t* p; const uint16_t* q;
  int ldp, ldq, T, M, N;
  float* out;                  // nullable (only the sums)
  float* bias;                 // nullable
  float* part; float* bpart;   // splits > 1: partial tiles, partial column sums [splits - 1][ntm * BM]
  uint32_t* flags; uint32_t* status;
  uint32_t epoch;
  int spin_limit;
  int ntn, nt, splits;
};

// 16-byte chunk c of row r lies at chunk c ^ wg_swz(r): the sixteen rows of a
// transpose load, 32 bytes each, then cover the 64 banks twice, the minimum
// (with the attention tiles' swizzle half of the LDS cycles were conflicts:
// 84 against 81 us for 768 x 3072 outputs over 12504 tokens).
__device__ __forceinline__ int wg_swz(int r) { return (r & 7) << 1; }

// LDS byte addresses of the transpose loads of a subtile (the lane's part as
// in AttnTrans, with this swizzle).
struct WgTrans {
  uint32_t base, u;
  __device__ __forceinline__ explicit WgTrans(int lane) {
    const int row = 4 * (lane >> 4) + ((lane >> 2) & 3);
    base = uint32_t(row * kWgSub * 2 + (lane & 1) * 8);
    u = uint32_t(((lane & 3) >> 1) ^ wg_swz(row));
  }
  __device__ __forceinline__ uint32_t addr(const char* tile, int blk) const {
    return uint32_t(size_t((__attribute__((address_space(3))) const char*)(tile))) + base +
           ((uint32_t(2 * blk) ^ u) * 16);
  }
};

// Tokens r0 .. r0 + 63, columns c0 .. c0 + 127 of src [T, ld] into a subtile.
// The resource ends with the matrix, so rows past T land as zeros; columns
// past ld hold the next row's values and only reach outputs that are dropped.
__device__ __forceinline__ void wg_dma(const uint16_t* src, int ld, int T, int r0, int c0, char* lds, int wave,
                                       int lane) {
  using A = AttnTile<kWgSub>;
  const int64_t left = (int64_t(T - r0) * ld - c0) * 2;
  const int bytes = int(left < 0 ? 0 : left > 0x7fffffff ? 0x7fffffff : left);
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(src + int64_t(r0) * ld + c0), (short)0,
                                                      bytes, 0x00020000);
#pragma unroll
  for (int e = 0; e < A::kDmaPerWave; ++e) {
    const int byte = 1024 * (wave * A::kDmaPerWave + e) + 16 * lane;
    const int r = byte / A::kRowBytes, c = (byte % A::kRowBytes) / 16;
    const uint32_t voff = uint32_t(r) * uint32_t(ld) * 2u + uint32_t((c ^ wg_swz(r)) * 16);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        rsrc, (__attribute__((address_space(3))) void*)(lds + 1024 * (wave * A::kDmaPerWave + e)), 16, int(voff), 0,
        0, 0);
  }
}

// The transposed fragments (two k-steps of 32 tokens) of two column blocks:
// eight transpose loads and their wait in one statement (see lds_read_tr4).
__device__ __forceinline__ void wg_read2(uint32_t a0, uint32_t a1, bf16x8 (&f0)[2], bf16x8 (&f1)[2]) {
  u32x2 v[8];
  asm volatile(
      "ds_read_b64_tr_b16 %0, %8\n\t"
      "ds_read_b64_tr_b16 %1, %8 offset:%10\n\t"
      "ds_read_b64_tr_b16 %2, %8 offset:%11\n\t"
      "ds_read_b64_tr_b16 %3, %8 offset:%12\n\t"
      "ds_read_b64_tr_b16 %4, %9\n\t"
      "ds_read_b64_tr_b16 %5, %9 offset:%10\n\t"
      "ds_read_b64_tr_b16 %6, %9 offset:%11\n\t"
      "ds_read_b64_tr_b16 %7, %9 offset:%12\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3]), "=&v"(v[4]), "=&v"(v[5]), "=&v"(v[6]), "=&v"(v[7])
      : "v"(a0), "v"(a1), "n"(16 * kWgSub * 2), "n"(32 * kWgSub * 2), "n"(48 * kWgSub * 2)
      : "memory");
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    f0[s] = __builtin_bit_cast(bf16x8, u32x4{v[2 * s][0], v[2 * s][1], v[2 * s + 1][0], v[2 * s + 1][1]});
    f1[s] = __builtin_bit_cast(bf16x8, u32x4{v[4 + 2 * s][0], v[4 + 2 * s][1], v[5 + 2 * s][0], v[5 + 2 * s][1]});
  }
}
}  // namespace

// LARGE: 256 x 256 tiles of eight 64 x 128 waves, one workgroup per CU; else
// 128 x 128 tiles of four 64 x 64 waves, two per CU. Two LDS stages; one
// barrier per 64 tokens.
template <bool LARGE>
__global__ __launch_bounds__(LARGE ? 512 : 256, 2) void wgrad_kernel(WgArgs g) {
  constexpr int BM = LARGE ? 256 : 128, WN = LARGE ? 128 : 64, MI = 4, NI = WN / 16;
  constexpr int NSUB = BM / kWgSub;               // subtiles of each operand
  constexpr int kStage = 2 * NSUB * kWgSubBytes;
  constexpr int kWaves = LARGE ? 8 : 4;
  constexpr int kFrags = MI * NI, kSlot = kWaves * kFrags * 1024;
  __shared__ __attribute__((aligned(1024))) char smem[2 * kStage];
  __shared__ int n_seen;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1, r16 = lane & 15, grp = lane >> 4;
  // each XCD takes a contiguous range of (slice, tile): neighbouring tiles of
  // one token range share its rows in the XCD's L2
  const int w = xcd_remap(int(blockIdx.x), int(gridDim.x));
  const int sl = w / g.nt, tile = w - sl * g.nt, tm = tile / g.ntn, tn = tile - tm * g.ntn;
  const int nk = (g.T + kWgK - 1) / kWgK;
  const int kb = int(int64_t(nk) * sl / g.splits), ke = int(int64_t(nk) * (sl + 1) / g.splits);

  auto issue = [&](int kt) {
    char* st = smem + (kt & 1) * kStage;
    // four waves fill a subtile; with eight, the second four take the Q subtiles
    if constexpr (LARGE) {
      const bool q = wave >= 4;
#pragma unroll
      for (int u = 0; u < NSUB; ++u)
        wg_dma(q ? g.q : g.p, q ? g.ldq : g.ldp, g.T, kt * kWgK, (q ? tn : tm) * BM + u * kWgSub,
               st + ((q ? NSUB : 0) + u) * kWgSubBytes, wave & 3, lane);
    } else {
      wg_dma(g.p, g.ldp, g.T, kt * kWgK, tm * BM, st, wave, lane);
      wg_dma(g.q, g.ldq, g.T, kt * kWgK, tn * BM, st + kWgSubBytes, wave, lane);
    }
  };
  f32x4 acc[MI][NI], accb[MI];
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    accb[i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NI; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const bool sums = g.bias && tn == 0 && wn == 0;
  bf16x8 ones;
#pragma unroll
  for (int i = 0; i < 8; ++i) ones[i] = (__bf16)1.0f;

  const WgTrans tr(lane);
  // subtile and first 16-column block of this wave's rows and columns
  const int ps = (wm * 64) / kWgSub, pb = (wm * 4) % 8, qs = (wn * WN) / kWgSub, qb = (wn * NI) % 8;
  if (kb < ke) issue(kb);
  for (int kt = kb; kt < ke; ++kt) {
    // this wave's share of tile kt has landed; behind the barrier so has every
    // wave's, and all are done reading tile kt - 1, whose stage is refilled
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (kt + 1 < ke) issue(kt + 1);
    const char* st = smem + (kt & 1) * kStage;
    const char* pt = st + ps * kWgSubBytes;
    const char* qt = st + (NSUB + qs) * kWgSubBytes;
    bf16x8 bf[NI][2];
#pragma unroll
    for (int j = 0; j < NI; j += 2) wg_read2(tr.addr(qt, qb + j), tr.addr(qt, qb + j + 1), bf[j], bf[j + 1]);
#pragma unroll
    for (int i = 0; i < MI; i += 2) {
      bf16x8 af[2][2];
      wg_read2(tr.addr(pt, pb + i), tr.addr(pt, pb + i + 1), af[0], af[1]);
#pragma unroll
      for (int ii = 0; ii < 2; ++ii)
#pragma unroll
        for (int s = 0; s < 2; ++s) {
#pragma unroll
          for (int j = 0; j < NI; ++j)
            acc[i + ii][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[ii][s], bf[j][s], acc[i + ii][j], 0, 0, 0);
          if (sums) accb[i + ii] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[ii][s], ones, accb[i + ii], 0, 0, 0);
        }
    }
  }
  // lane holds dW[wm*64 + 16 i + 4 grp + e][wn*WN + 16 j + r16]; accb the same rows' sums in every column
  const int mrow = tm * BM + wm * 64 + 4 * grp, ncol = tn * BM + wn * WN + r16;
  if constexpr (!LARGE) {  // (large grids are not split)
    if (g.splits > 1) {
      constexpr int kCoherent = 16;  // cache policy: sc1
      const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(g.part, (short)0, 0x7fffffff, 0x00020000);
      const int lane_off = wave * (kFrags * 1024) + lane * 16;
      const int np = g.splits - 1, slot = tile * np + sl;  // slots of a tile's pieces before the last
      const int bstride = (g.nt / g.ntn) * BM;
      if (sl < np) {
#pragma unroll
        for (int f = 0; f < kFrags; ++f)
          __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[f / NI][f % NI]), rsrc,
                                                 slot * kSlot + lane_off + f * 1024, 0, kCoherent);
        if (sums && r16 == 0)
#pragma unroll
          for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              __hip_atomic_store(g.bpart + int64_t(sl) * bstride + mrow + 16 * i + e, accb[i][e], __ATOMIC_RELAXED,
                                 __HIP_MEMORY_SCOPE_AGENT);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();  // every wave's stores have completed
        if (tid == 0) __hip_atomic_store(g.flags + slot, g.epoch, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
      }
      if (tid == 0) {
        int seen = 0;
        for (; seen < np; ++seen) {
          int it = 0;
          while (it < g.spin_limit && __hip_atomic_load(g.flags + tile * np + seen, __ATOMIC_RELAXED,
                                                        __HIP_MEMORY_SCOPE_AGENT) != g.epoch) {
            __builtin_amdgcn_s_sleep(2);
            ++it;
          }
          if (it == g.spin_limit) break;
        }
        n_seen = seen;
        if (seen < np)
          __hip_atomic_fetch_or(g.status, uint32_t(DSF_WS_STATUS_SK_TIMEOUT), __ATOMIC_RELAXED,
                                __HIP_MEMORY_SCOPE_AGENT);
      }
      __syncthreads();  // the loads below are issued after their flags were seen
      const int seen = __builtin_amdgcn_readfirstlane(n_seen);
      for (int s = 0; s < seen; ++s) {
        const int at = (tile * np + s) * kSlot + lane_off;
#pragma unroll
        for (int f = 0; f < kFrags; ++f)
          acc[f / NI][f % NI] += __builtin_bit_cast(
              f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc, at + f * 1024, 0, kCoherent));
        if (sums && r16 == 0)
#pragma unroll
          for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e)
              accb[i][e] += __hip_atomic_load(g.bpart + int64_t(s) * bstride + mrow + 16 * i + e, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int m = mrow + 16 * i + e;
      if (m >= g.M) continue;
      float* row = g.out + int64_t(m) * g.N;
#pragma unroll
      for (int j = 0; j < NI; ++j)
        if (g.out && ncol + 16 * j < g.N) row[ncol + 16 * j] = acc[i][j][e];
      if (sums && r16 == 0) g.bias[m] = accb[i][e];
    }
}

hipError_t launch_wgrad(const void* p, int ldp, int M, const void* q, int ldq, int N, int T, float* out, float* bias,
                        const WgradScratch& ws, hipStream_t s) {
  if (M <= 0 || N <= 0 || T <= 0 || (!out && !bias)) return hipSuccess;
  if (!out) {  // the sums alone: one column tile, of P itself, that is not stored
    q = p;
    ldq = ldp;
    N = 1;
  }
  WgArgs g{};
  g.p = (const uint16_t*)p;
  g.q = (const uint16_t*)q;
  g.ldp = ldp;
  g.ldq = ldq;
  g.T = T;
  g.M = M;
  g.N = N;
  g.out = out;
  g.bias = bias;
  g.part = ws.part;
  g.bpart = ws.bias_part;
  g.flags = ws.flags;
  g.status = ws.status;
  g.epoch = ws.epoch;
  g.spin_limit = spin_limit();
  auto tiles = [&](int b, int* ntn) {
    *ntn = (N + b - 1) / b;
    return ((M + b - 1) / b) * *ntn;
  };
  const bool large = tiles(256, &g.ntn) >= kWgLargeMin;
  const int bm = large ? 256 : 128;
  g.nt = tiles(bm, &g.ntn);
  // slices of the tokens: as many workgroups as two per CU hold (one of the
  // large tiles, whose grids fill the chip without)
  const int nk = (T + kWgK - 1) / kWgK, slots = 512;
  int sp = large ? 1 : std::max(1, std::min(std::min(kWgradMaxSplit, slots / g.nt), nk / kWgMinTiles));
  while (sp > 1 && (size_t(sp) * g.nt * (128 * 128 * 4) > ws.part_bytes || size_t(sp) * g.nt > size_t(ws.nflags) ||
                    size_t(sp) * (g.nt / g.ntn) * bm * 4 > ws.bias_bytes))
    --sp;
  g.splits = sp;
  if (large) wgrad_kernel<true><<<g.nt, 512, 0, s>>>(g);
  else wgrad_kernel<false><<<g.nt * sp, 256, 0, s>>>(g);
  return hipGetLastError();
}

}  // namespace dsf
