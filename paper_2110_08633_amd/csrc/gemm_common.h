// Shared by the GEMM kernels: argument block, tile numbering, epilogues and their write-out, buffer descriptors.
#pragma once
#include <type_traits>

#include "kernels.h"
#include "once_per_gpu.h"
#include "tile_ops.h"

namespace hydra {

struct GemmArgs {
  const void *A, *B;
  int M, N, K;
  int64_t lda, ldb, ldc;
  int nb2;
  int64_t sA1, sA2, sB1, sB2, sC1, sC2;
  const float *bias, *resid;
  float *out_f32;
  void *out_act, *out_act2;
  const void *aux;
  int epi, causal;
  int tiles_m, tiles_n;
  float alpha;  // kept among the 32-bit fields: next to a pointer the compiler fused both into one 16-byte load and
  int grp;      // parked it in scratch memory, and a kernel that uses scratch pays microseconds per launch
                // grp: tile rows per group of the tile numbering (see xcd_group_rows)
};

// Tiles are numbered so that the run of tiles an XCD works on (consecutive workgroup ids go round-robin to the 8
// XCDs, each with its own L2) is a block of grp tile rows by a few tile columns: every XCD then fetches grp row
// panels of A and those few column panels of B once.  grp minimises the operand rows + columns such a block
// spans; a fixed 8 made the XCDs of an N = 768 product fetch 60 MB for 17 MB of operands, 4 rows give 44 MB.
// What shares an L2 in time is the set of tiles in flight on the XCD (32 CUs x blocks per CU), not its whole run:
// a launch of several rounds is sized for that set, walked column by column so that the row panels stay (the
// 4096 x 16384 x 1024 weight gradient: 16 rows per group 588, 8 rows 605 TFLOP/s; 16384 x 4096: 527 -> 604).
static inline int xcd_group_rows(int tiles_m, int tiles_n, int bm, int bn, int inflight_per_xcd = 64) {
  long per = ((long)tiles_m * tiles_n + 7) / 8;  // tiles per XCD
  if (per > inflight_per_xcd) per = inflight_per_xcd;
  int best = 1;
  long best_cost = -1;
  for (int g = 1; g <= 16 && g <= tiles_m; ++g) {
    const long cols = (per + g - 1) / g;
    const long cost = (long)g * bm + (cols < tiles_n ? cols : tiles_n) * bn;
    if (best_cost < 0 || cost <= best_cost) { best = g; best_cost = cost; }
  }
  return best;
}

template <typename T> __device__ __forceinline__ float ld_act(const void *p, int64_t i);
template <> __device__ __forceinline__ float ld_act<float>(const void *p, int64_t i) { return ((const float *)p)[i]; }
template <> __device__ __forceinline__ float ld_act<bf16_t>(const void *p, int64_t i) { return bf2f(((const bf16_t *)p)[i]); }
template <typename T> __device__ __forceinline__ void st_act(void *p, int64_t i, float v);
template <> __device__ __forceinline__ void st_act<float>(void *p, int64_t i, float v) { ((float *)p)[i] = v; }
template <> __device__ __forceinline__ void st_act<bf16_t>(void *p, int64_t i, float v) { ((bf16_t *)p)[i] = f2bf(v); }

// tanh-form GELU and its derivative (fp32)
__device__ __forceinline__ float gelu_f(float u) {
  const float c = 0.7978845608028654f;
  float t = tanhf(c * (u + 0.044715f * u * u * u));
  return 0.5f * u * (1.f + t);
}
__device__ __forceinline__ float dgelu_f(float u) {
  const float c = 0.7978845608028654f;
  float t = tanhf(c * (u + 0.044715f * u * u * u));
  float dt = (1.f - t * t) * c * (1.f + 3.f * 0.044715f * u * u);
  return 0.5f * (1.f + t) + 0.5f * u * dt;
}

template <typename ActT>
__device__ __forceinline__ void epilogue_store(const GemmArgs &g, int64_t coff, int row, int col, float acc) {
  float v = acc * g.alpha;
  if (g.bias) v += g.bias[col];
  const int64_t idx = coff + (int64_t)row * g.ldc + col;
  if (g.epi == EPI_GELU) {
    st_act<ActT>(g.out_act, idx, v);
    st_act<ActT>(g.out_act2, idx, gelu_f(v));
    return;
  }
  if (g.epi == EPI_DGELU) v *= dgelu_f(ld_act<ActT>(g.aux, idx));
  if (g.resid) v += g.resid[idx];
  if (g.out_f32) g.out_f32[idx] = v;
  if (g.out_act) st_act<ActT>(g.out_act, idx, v);
}

// 4 consecutive columns of one row of C
template <typename ActT>
__device__ __forceinline__ void epilogue_store4(const GemmArgs &g, int64_t coff, int row, int col, const f32x4_t acc,
                                                bool vec) {
  if (!vec || col + 3 >= g.N) {
#pragma unroll 1
    for (int e = 0; e < 4; ++e) {
      // chosen by comparison, not by address: an indexed local array would live in scratch memory, and a kernel
      // that uses scratch pays several microseconds per launch for its set-up
      const float x = e == 0 ? acc[0] : e == 1 ? acc[1] : e == 2 ? acc[2] : acc[3];
      if (col + e < g.N) epilogue_store<ActT>(g, coff, row, col + e, x);
    }
    return;
  }
  float v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = acc[e] * g.alpha;
  if (g.bias) {
    const f32x4_t b = *(const f32x4_t *)(g.bias + col);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += b[e];
  }
  const int64_t idx = coff + (int64_t)row * g.ldc + col;
  if (g.epi == EPI_GELU) {
    u32x2_t u, h;
    u.x = (uint32_t)f2bf(v[0]) | ((uint32_t)f2bf(v[1]) << 16);
    u.y = (uint32_t)f2bf(v[2]) | ((uint32_t)f2bf(v[3]) << 16);
    h.x = (uint32_t)f2bf(gelu_f(v[0])) | ((uint32_t)f2bf(gelu_f(v[1])) << 16);
    h.y = (uint32_t)f2bf(gelu_f(v[2])) | ((uint32_t)f2bf(gelu_f(v[3])) << 16);
    *(u32x2_t *)((bf16_t *)g.out_act + idx) = u;
    *(u32x2_t *)((bf16_t *)g.out_act2 + idx) = h;
    return;
  }
  if (g.epi == EPI_DGELU) {
    const u32x2_t a = *(const u32x2_t *)((const bf16_t *)g.aux + idx);
    v[0] *= dgelu_f(__uint_as_float(a.x << 16));
    v[1] *= dgelu_f(__uint_as_float(a.x & 0xffff0000u));
    v[2] *= dgelu_f(__uint_as_float(a.y << 16));
    v[3] *= dgelu_f(__uint_as_float(a.y & 0xffff0000u));
  }
  if (g.resid) {
    const f32x4_t r = *(const f32x4_t *)(g.resid + idx);
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] += r[e];
  }
  if (g.out_f32) {
    f32x4_t o = {v[0], v[1], v[2], v[3]};
    *(f32x4_t *)(g.out_f32 + idx) = o;
  }
  if (g.out_act) {
    u32x2_t o;
    o.x = (uint32_t)f2bf(v[0]) | ((uint32_t)f2bf(v[1]) << 16);
    o.y = (uint32_t)f2bf(v[2]) | ((uint32_t)f2bf(v[3]) << 16);
    *(u32x2_t *)((bf16_t *)g.out_act + idx) = o;
  }
}

// tanh(x) = 1 - 2 / (exp(2x) + 1): exact limits at both infinities; the absolute error of about 1e-7 near zero
// is far below what a bf16 result keeps
__device__ __forceinline__ float tanh_fast(float x) {
  return 1.f - 2.f * __builtin_amdgcn_rcpf(__expf(2.f * x) + 1.f);
}
__device__ __forceinline__ float gelu_fast(float u) {
  const float c = 0.7978845608028654f;
  return 0.5f * u * (1.f + tanh_fast(c * (u + 0.044715f * u * u * u)));
}
__device__ __forceinline__ float dgelu_fast(float u) {
  const float c = 0.7978845608028654f;
  const float t = tanh_fast(c * (u + 0.044715f * u * u * u));
  const float dt = (1.f - t * t) * c * (1.f + 3.f * 0.044715f * u * u);
  return 0.5f * (1.f + t) + 0.5f * u * dt;
}

// Row-wise write-out of a wavefront's staged [32][WTN] fp32 patch (LDS, pitch WTN + 4) to rows row0.. and columns
// col0.. of C.  LPR lanes cover a row with 4 columns each, so one instruction stores whole row segments.  With one
// wavefront per SIMD nothing hides latency here, so the work is batched: the epilogue kind is a template
// parameter, addresses advance by addition, and the rows are handled four instructions' worth at a time - all LDS
// reads and all global loads (residual, GELU pre-activation) of a batch are issued before the first is used, and
// all its stores follow together (a load issued after a store has to wait until that store has completed).
// bf16 packing is the hardware conversion.  Needs: 16-byte aligned fp32 pointers, 8-byte aligned bf16 pointers,
// ldc % 4 == 0, col0 + WTN <= N, row0 + 32 <= M.
template <int WTN, int EPI, int PR>
__device__ __forceinline__ void store_patch_rows(const GemmArgs &g, int64_t coff, const float *patch, int row0,
                                                 int col0, int lane) {
  // LPR lanes per row; when that is no power of two, a wavefront instruction covers rows and a part of one
  constexpr int SP = WTN + 4, LPR = WTN / 4, NIT = PR * LPR / 64, U = NIT % 4 == 0 ? 4 : NIT % 3 == 0 ? 3 : NIT % 2 == 0 ? 2 : 1;
  constexpr bool P2 = 64 % LPR == 0;
  constexpr int RPI = P2 ? 64 / LPR : 1;
  static_assert(NIT * 64 == PR * LPR, "whole instructions");
  const float alpha = g.alpha;
  const int c0 = (lane % LPR) * 4, r0 = lane / LPR;
  const int64_t tile0 = coff + (int64_t)row0 * g.ldc + col0;
  const int64_t step = (int64_t)RPI * g.ldc;
  int64_t idx0 = tile0 + (int64_t)r0 * g.ldc + c0;
  const float *pp0 = patch + r0 * SP + c0;
  f32x4_t b0 = {0.f, 0.f, 0.f, 0.f};
  if (P2 && g.bias) b0 = *(const f32x4_t *)(g.bias + col0 + c0);
  const bool has_resid = g.resid != nullptr, has_f32 = g.out_f32 != nullptr, has_act = g.out_act != nullptr;
#pragma unroll 1
  for (int p0 = 0; p0 < NIT; p0 += U) {
    f32x4_t v[U], r[U], b4[U];
    u32x2_t a[U];
    int64_t idx[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (P2) {
        idx[u] = idx0 + u * step;
        v[u] = *(const f32x4_t *)(pp0 + u * RPI * SP);
        b4[u] = b0;
      } else {
        const int id = (p0 + u) * 64 + lane, row = id / LPR, c = (id % LPR) * 4;
        idx[u] = tile0 + (int64_t)row * g.ldc + c;
        v[u] = *(const f32x4_t *)(patch + row * SP + c);
        b4[u] = g.bias ? *(const f32x4_t *)(g.bias + col0 + c) : b0;
      }
    }
    idx0 += U * step;
    pp0 += U * RPI * SP;
    if (EPI == EPI_DGELU) {
#pragma unroll
      for (int u = 0; u < U; ++u) a[u] = *(const u32x2_t *)((const bf16_t *)g.aux + idx[u]);
    }
    if (EPI != EPI_GELU && has_resid) {
#pragma unroll
      for (int u = 0; u < U; ++u) r[u] = *(const f32x4_t *)(g.resid + idx[u]);
    }
#pragma unroll
    for (int u = 0; u < U; ++u) v[u] = v[u] * alpha + b4[u];
    if (EPI == EPI_GELU) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        u32x2_t o, h;
        o.x = pack_bf16(v[u][0], v[u][1]);
        o.y = pack_bf16(v[u][2], v[u][3]);
        h.x = pack_bf16(gelu_fast(v[u][0]), gelu_fast(v[u][1]));
        h.y = pack_bf16(gelu_fast(v[u][2]), gelu_fast(v[u][3]));
        *(u32x2_t *)((bf16_t *)g.out_act + idx[u]) = o;
        *(u32x2_t *)((bf16_t *)g.out_act2 + idx[u]) = h;
      }
      continue;
    }
    if (EPI == EPI_DGELU) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        v[u][0] *= dgelu_fast(__uint_as_float(a[u].x << 16));
        v[u][1] *= dgelu_fast(__uint_as_float(a[u].x & 0xffff0000u));
        v[u][2] *= dgelu_fast(__uint_as_float(a[u].y << 16));
        v[u][3] *= dgelu_fast(__uint_as_float(a[u].y & 0xffff0000u));
      }
    }
    if (has_resid) {
#pragma unroll
      for (int u = 0; u < U; ++u) v[u] += r[u];
    }
    if (has_f32) {
#pragma unroll
      for (int u = 0; u < U; ++u) *(f32x4_t *)(g.out_f32 + idx[u]) = v[u];
    }
    if (has_act) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        u32x2_t o;
        o.x = pack_bf16(v[u][0], v[u][1]);
        o.y = pack_bf16(v[u][2], v[u][3]);
        *(u32x2_t *)((bf16_t *)g.out_act + idx[u]) = o;
      }
    }
  }
}

template <int WTN, int PR, bool COALESCE>
__device__ __forceinline__ void store_patch(const GemmArgs &g, int64_t coff, const float *patch, int row0, int col0,
                                            int lane, bool vec) {
  if (vec && col0 + WTN <= g.N && row0 + PR <= g.M) {  // uniform over the wavefront
    if (g.epi == EPI_GELU) store_patch_rows<WTN, EPI_GELU, PR>(g, coff, patch, row0, col0, lane);
    else if (g.epi == EPI_DGELU) store_patch_rows<WTN, EPI_DGELU, PR>(g, coff, patch, row0, col0, lane);
    else store_patch_rows<WTN, EPI_NONE, PR>(g, coff, patch, row0, col0, lane);
    return;
  }
  constexpr int SP = WTN + 4, LPR = WTN / 4;
  if (COALESCE && !vec && g.epi == EPI_NONE) {
    // rows that vector stores cannot address (an LM head's gradient has an odd number of columns): neighbouring lanes
    // store neighbouring columns, eight instructions' worth at a time (768x50257x2048 tn: 233 -> 208 us)
    constexpr int U = PR * WTN % 512 == 0 ? 8 : 4;
    static_assert(PR * WTN % (64 * U) == 0, "whole batches");
    const int end = min(PR, g.M - row0) * WTN;
#pragma unroll 1
    for (int p0 = 0; p0 < end; p0 += 64 * U) {
      float v[U];
      int64_t idx[U];
      bool in[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int r = (p0 + u * 64 + lane) / WTN, cc = (p0 + u * 64 + lane) % WTN;
        in[u] = row0 + r < g.M && col0 + cc < g.N;
        idx[u] = coff + (int64_t)(row0 + r) * g.ldc + col0 + cc;
        v[u] = patch[r * SP + cc] * g.alpha;
        if (g.bias && in[u]) v[u] += g.bias[col0 + cc];
        if (g.resid && in[u]) v[u] += g.resid[idx[u]];
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (in[u]) {
          if (g.out_f32) g.out_f32[idx[u]] = v[u];
          if (g.out_act) ((bf16_t *)g.out_act)[idx[u]] = f2bf(v[u]);
        }
    }
    return;
  }
  // ragged edge, or an unaligned GELU: one copy of the code
#pragma unroll 1
  for (int p = 0; p < PR * LPR / 64; ++p) {
    const int r = (p * 64 + lane) / LPR, c = ((p * 64 + lane) % LPR) * 4;
    const f32x4_t v4 = *(const f32x4_t *)(patch + r * SP + c);
    const int row = row0 + r, col = col0 + c;
    if (row < g.M && col < g.N) epilogue_store4<bf16_t>(g, coff, row, col, v4, vec);
  }
}


// Adds a wavefront's staged patch to the results in memory, neighbouring lanes to neighbouring columns.
template <int WTN, int PR>
__device__ __forceinline__ void add_patch(const GemmArgs &g, const float *patch, int row0, int col0, int lane) {
  constexpr int SP = WTN + 4;
  static_assert(PR * WTN % 64 == 0, "whole instructions");
#pragma unroll 4
  for (int p0 = 0; p0 < PR * WTN; p0 += 64) {
    const int r = (p0 + lane) / WTN, c = (p0 + lane) % WTN;
    if (row0 + r < g.M && col0 + c < g.N)
      unsafeAtomicAdd(g.out_f32 + (int64_t)(row0 + r) * g.ldc + col0 + c, patch[r * SP + c] * g.alpha);
  }
}

// descriptor of 2 GB from p on (offsets are 32 bits wide: the base moves with the slice)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_at(const void *p) {
  return __builtin_amdgcn_make_buffer_rsrc((void *)p, 0, 0x7ffffff0, 0x00020000);
}

template <int n> __device__ __forceinline__ void wait_loads_le() {
  // vmcnt (outstanding vector-memory loads) is split over bits 3:0 and 15:14; lgkmcnt(0): this wavefront's LDS
  // reads have returned; expcnt is left alone
  static_assert(n >= 0 && n <= 63, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((n & 15) | ((n >> 4) << 14) | 0x0070);
}

// lets a kernel have `bytes` of dynamic LDS on the current GPU; once: one object per kernel
inline hipError_t allow_lds(OncePerGpu &once, const void *kern, size_t bytes) {
  int gpu = -1;
  const hipError_t e = hipGetDevice(&gpu);
  if (e != hipSuccess) return e;
  return (hipError_t)once.run(gpu, [&] { return (int)hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes); });
}

constexpr int GEMM_GROUP_MAX = 4;
// the single-product kernel (gemm_plain.hip): any layout, any K, no batching and no causal short-cut
bool gemm_plain_ok(const GemmDesc &d);
hipError_t launch_gemm_plain(const GemmDesc &d, hipStream_t s);
// n products with both operands stored contraction-strided, in one launch
hipError_t launch_gemm_plain_group(const GemmDesc *d, int n, hipStream_t s);
// the kernel for products with few tiles (gemm_split.hip); shape: index into split_shapes
hipError_t launch_gemm_split(const GemmDesc &d, int shape, hipStream_t s);
void gemm_fill_args(GemmArgs &a, const GemmDesc &d);
double gemm_flops(const GemmDesc &d);

}  // namespace hydra
