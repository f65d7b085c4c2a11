// bf16 products with few tiles: small tiles, the contraction shared out over the eight wavefronts of a block.
#include "gemm16_ops.h"
#include "gemm_shapes.h"

namespace hydra {

// ---------------------------------------------------------------------------
// A short sample, a narrow layer or the gradient of a small matrix has fewer
// 64x64 tiles than the chip has CUs, and a launch lasts as long as one CU needs
// to load a tile's operands: 128 bytes per contraction step and row of both at
// 64x64, of which a CU gets 50 to 150 a nanosecond.  Hence tiles of 16x16 to
// 64x32 (a quarter of the bytes per CU and step at 16x16), and to keep eight
// wavefronts busy on so small a tile each takes slices of BKW contraction steps
// of its own: slice w, w + 8, w + 16, ...  Nothing a wavefront loads is read by
// another one, so the loop has no barrier: a wavefront waits for its slice, reads
// all its fragments, hands the LDS back to the loads of its next slice and
// multiplies while they fly; 96 to 160 KB per CU are in flight.  At the end the
// eight partial tiles are added through LDS, in ascending order of the wavefront,
// and written out like the other kernels' tiles.
// Bound: loads of operands that come from the 256 MB cache (rows of 128 bytes: 110 bytes per nanosecond and CU measured, 154
// from the L2), and for tens of tiles the latency of a launch (about 2.5 us before the first result is written).
// Counters (matrix pipes 1 to 11 % busy, LDS 4 to 15 %, 0.8 to 1.8 wavefronts per SIMD) show nothing else that is busy.
// us, launched one after another, 64x64 tiles with slices split over two groups / here (MxNxK, n: contraction-contiguous): nt 152x168x6120 23.9 / 7.9
// (16x16 tiles), 201x768x2304 9.4 / 6.0 (32x32), 64x704x9768 37 / 10.9 (16x16), 876x520x13592 50 / 49 (64x32), tn 248x408x2174
// 13.8 / 9.5 (16x32), nn 117x216x2896 15.9 / 6.3 (16x32).
// ---------------------------------------------------------------------------
template <int BM, int BN, int TA, int TB, int BKW>
__device__ __forceinline__ void split_tile(const GemmArgs &g, const int bid, const int nt, bf16_t *const lds) {
  constexpr int NW = 8, MI = BM / 16, NJ = BN / 16, SLICE = (BM + BN) * BKW, KS = BKW / 32;
  typedef LdsMover<BM, TA, BKW, 1> MA;
  typedef LdsMover<BN, TB, BKW, 1> MB;
  constexpr int NL = MA::N + MB::N, NM = KS * MI * NJ, PER = (NL + NM - 1) / NM;  // loads, MFMAs, loads per MFMA
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int m0, n0;
  tile_origin<BM, BN>(g, bid, nt, m0, n0);
  const int nk = (g.K + BKW - 1) / BKW;

  MA ma;
  MB mb;
  ma.init((const bf16_t *)g.A, g.lda, m0, g.M, lane);
  mb.init((const bf16_t *)g.B, g.ldb, n0, g.N, lane);
  Frag16<BM, TA, MI, BKW, KS> fa;
  Frag16<BN, TB, NJ, BKW, KS> fb;
  fa.init(0, lane, 0);
  fb.init(0, lane, 0);
  bf16_t *const as = lds + wave * SLICE, *const bs = as + BM * BKW;  // this wavefront's slice
  const uint32_t dst = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) bf16_t *)as);
  // load l (first A's, then B's) of slice t; slices past K are zeros without a memory access
  auto issue = [&](int l, int t) {
    if (l < MA::N) ma.issue(l, t, g.K - t * BKW, dst, 0);
    else mb.issue(l - MA::N, t, g.K - t * BKW, dst + BM * BKW * 2, 0);
  };
  f32x4_t acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int l = 0; l < NL; ++l) issue(l, wave);
  for (int t = wave; t < nk; t += NW) {
    wait_loads_le<0>();
    asm volatile("" ::: "memory");
    bf16x8_t af[KS][MI], bfr[KS][NJ];
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
#pragma unroll
      for (int i = 0; i < MI; ++i) af[kk][i] = fa.get(as, i, kk);
#pragma unroll
      for (int j = 0; j < NJ; ++j) bfr[kk][j] = fb.get(bs, j, kk);
    }
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the slice is in registers, its LDS may be overwritten
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kk = 0; kk < KS; ++kk)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int q = (kk * MI + i) * NJ + j;
#pragma unroll
          for (int l = q * PER; l < (q + 1) * PER && l < NL; ++l) issue(l, t + NW);
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[kk][j], af[kk][i], acc[i][j], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
        }
  }
  wait_loads_le<0>();

  const bool vec = ((g.ldc & 3) == 0) &&
                   ((((uintptr_t)g.out_f32 | (uintptr_t)g.resid | (uintptr_t)g.bias) & 15) == 0) &&
                   ((((uintptr_t)g.out_act | (uintptr_t)g.out_act2 | (uintptr_t)g.aux) & 7) == 0);
  // patches [wavefront][BM][SP] of partial sums; wavefront w < BM / PR adds rows w * PR .. up and stores them
  constexpr int SP = BN + 4, PR = BN % 32 ? 16 : 8;
  float *const patch = (float *)lds;
  __syncthreads();
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
      *(f32x4_t *)(patch + (wave * BM + i * 16 + (lane & 15)) * SP + j * 16 + (lane >> 4) * 4) = acc[i][j];
  __syncthreads();
  if (wave < BM / PR) {
#pragma unroll
    for (int u = 0; u < PR * BN / 256; ++u) {
      const int id = u * 64 + lane;
      float *const p = patch + (wave * PR + id / (BN / 4)) * SP + id % (BN / 4) * 4;
      f32x4_t v = *(const f32x4_t *)p;
#pragma unroll
      for (int k = 1; k < NW; ++k) v += *(const f32x4_t *)(p + k * BM * SP);
      *(f32x4_t *)p = v;
    }
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_wave_barrier();
    store_patch<BN, PR, true>(g, 0, patch + wave * PR * SP, m0 + wave * PR, n0, lane, vec);
  }
}

template <int BM, int BN, int TA, int TB, int BKW, int OCC>
__global__ __launch_bounds__(512, OCC * 2) void gemm_split_kernel(const GemmArgs g) {
  extern __shared__ __attribute__((aligned(16))) bf16_t lds_dyn[];
  split_tile<BM, BN, TA, TB, BKW>(g, blockIdx.x, gridDim.x, lds_dyn);
}

template <int SHAPE, int BKW, int OCC>
static hipError_t launch_split(const GemmDesc &d, hipStream_t s) {
  constexpr int BM = split_shapes[SHAPE].bm, BN = split_shapes[SHAPE].bn;
  constexpr size_t slices = (size_t)8 * (BM + BN) * BKW * 2, patches = (size_t)8 * BM * (BN + 4) * 4, lds = slices > patches ? slices : patches;
  static_assert(lds * OCC <= 160 * 1024, "LDS per CU");
  GemmArgs a;
  gemm_fill_args(a, d);
  a.tiles_m = (a.M + BM - 1) / BM;
  a.tiles_n = (a.N + BN - 1) / BN;
  a.grp = xcd_group_rows(a.tiles_m, a.tiles_n, BM, BN, 32 * OCC);
#define HYDRA_SPLIT(TA_, TB_)                                                       \
  do {                                                                              \
    auto kern = gemm_split_kernel<BM, BN, TA_, TB_, BKW, OCC>;                       \
    static OncePerGpu once;                                                         \
    const hipError_t attr = allow_lds(once, (const void *)kern, lds);               \
    if (attr != hipSuccess) return attr;                                            \
    hipLaunchKernelGGL(kern, dim3(a.tiles_m * a.tiles_n), dim3(512), lds, s, a);     \
  } while (0)
  if (d.ta && d.tb) HYDRA_SPLIT(1, 1);
  else if (d.ta) HYDRA_SPLIT(1, 0);
  else if (d.tb) HYDRA_SPLIT(0, 1);
  else HYDRA_SPLIT(0, 0);
#undef HYDRA_SPLIT
  return hipGetLastError();
}

hipError_t launch_gemm_split(const GemmDesc &d, int shape, hipStream_t s) {
  static const char *const names[N_SPLIT][4] = {
#define HYDRA_N(X) {"gemm_bf16_" X "_nt", "gemm_bf16_" X "_nn", "gemm_bf16_" X "_tt", "gemm_bf16_" X "_tn"}
      HYDRA_N("64x64k2"), HYDRA_N("64x32w8"), HYDRA_N("48x32w8"), HYDRA_N("32x32w8"), HYDRA_N("16x32w8"), HYDRA_N("16x16w8")};
#undef HYDRA_N
  ProfScope ps(names[shape][d.ta * 2 + d.tb], s, gemm_flops(d), 0);
  switch (shape) {
    case 1: return launch_split<1, 64, 1>(d, s);
    case 2: return launch_split<2, 64, 2>(d, s);
    case 3: return launch_split<3, 64, 2>(d, s);
    case 4: return launch_split<4, 64, 2>(d, s);
    case 5: return launch_split<5, 128, 2>(d, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace hydra
