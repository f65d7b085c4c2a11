// bf16 products of single matrices - the linear layers of a block, their input and weight gradients, the LM head - and
// the choice of their tile shape.
#include "gemm16_ops.h"
#include "gemm_shapes.h"
#include "result_memory.h"

namespace hydra {

// ---------------------------------------------------------------------------
// bf16 MFMA kernel for single products of any layout: v_mfma_f32_16x16x32_bf16,
// operand slices moved from global memory straight into LDS.
//
// What bounds a bf16 product here, per CU: the matrix pipes (4096 flop per
// clock), the vector-memory path (about 60 bytes per clock, 43 for rows of 64
// bytes) and, at a few thousand rows, the 256 CUs themselves - a launch lasts as
// long as the CU with the most tiles.  So the kernel is written for many tile
// shapes (multiples of 16 either way) and the launcher picks the shape by those
// three terms (shape_cost).  Per tile:
//   - WM x WN wavefronts, each (BM/WM) x (BN/WN) results; at least two
//     wavefronts per SIMD are resident (one block of eight or several blocks of
//     four), so that one computes while another waits;
//   - buffer loads with the LDS flag (16 bytes per lane, lane l fills LDS base +
//     16*l), S stages of BK contraction steps.  Chunks that start past the matrix
//     or past K are fetched from an out-of-range offset, which writes zeros: no
//     branches, and the ragged end of K needs no code of its own.  A chunk of a
//     contraction-contiguous operand holds eight steps: where K is no multiple of
//     eight, its elements past K are read as they are, and the caller keeps them
//     zero;
//   - the only barrier of a slice sits before its last contraction step: every
//     wavefront has read the slice by then, its stage is handed to the loads of
//     slice t + S, and the first fragments of slice t + 1 are read while the last
//     MFMAs of slice t run;
//   - operands sit in LDS as in memory.  Contraction-contiguous ones are read
//     with ds_read_b128, the others with the transposing ds_read_b64_tr_b16; XOR
//     swizzles spread both over the banks (applied on the global side: which 16
//     bytes a lane fetches).  Counted conflict cycles: 2 to 8 % of the LDS cycles
//     with slices of 64, but half of them where contraction-contiguous operands
//     sit in slices of 128 (16 rows there fall into 8 slots, see swz_kc).
// Measured, us, the kernels this one replaced / now (MxNxK; n: operand contraction-contiguous, t: not):
//   nt 201x768x2304 13.4 / 9.4, 2048x2304x768 14.7 / 12.7, 1000x3072x768 11.1 / 9.9, 1024x16384x4096 115 / 100,
//   4096^3 116 / 104; tn 768x2304x2048 20.1 / 17.1, 3072x768x2048 28.8 / 19.0, 1600x6400x1000 41 / 34,
//   4096x4096x1024 53 / 40, 4096^3 204 / 124; nn 2048x768x50257 437 / 272, 4096^3 188 / 111;
//   tn 768x50257x2048 270 / 208.
// 720 random products: 1.40 times as fast on average (nt 1.56, tn 1.22, nn 1.25), 7 of them more than 5 % slower, 0.83 at
// worst.
// With both operands contraction-strided the 256x256 shape takes slices of 32 steps (large_tn); "tt" products, which no caller
// of the library has, take 64 and spill 5 registers (24 bytes of scratch per lane), reloaded inside the loop.
// What bounds the large ones now: with loads, LDS reads and MFMAs switched off in turn, 1024x16384x4096 takes 71 us of
// loads alone (25 bytes per clock and CU), 73 us of MFMAs alone at the clock the chip holds for them, 100 us together.
// HALVES: this workgroup multiplies one half of the contraction and adds its results to a cleared C (see best_half_shape).
// ---------------------------------------------------------------------------
template <int BM, int BN, int WM, int WN, int KW, int TA, int TB, int BK_, int S, bool HALVES = false>
__device__ __forceinline__ void gemm16_tile(const GemmArgs &g, const int bid, const int nt, bf16_t *const lds) {
  constexpr int NG = WM * WN, NW = NG * KW, WTM = BM / WM, WTN = BN / WN, MI = WTM / 16, NJ = WTN / 16;
  static_assert(WTM % 16 == 0 && WTN % 16 == 0 && MI * 16 * WM == BM && NJ * 16 * WN == BN, "wavefront tiles");
  constexpr int STAGE = (BM + BN) * BK_, KS = BK_ / 32 / KW;  // steps of a slice per wavefront
  static_assert(KS * KW * 32 == BK_ && (KS % 2 == 0 || KS == 1), "the groups share a slice evenly, one step or an even number each");
  typedef LdsMover<BM, TA, BK_, NW> MA;
  typedef LdsMover<BN, TB, BK_, NW> MB;
  constexpr int NL = MA::N + MB::N;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = wave / NG, wm = (wave / WN) % WM, wn = wave % WN;
  int m0, n0;
  int K = g.K;
  const bf16_t *A = (const bf16_t *)g.A, *B = (const bf16_t *)g.B;
  if constexpr (HALVES) {
    const int K0 = ((K + BK_ - 1) / BK_ + 1) / 2 * BK_;  // steps of the first half
    if (tile_origin<BM, BN, true>(g, bid, nt, m0, n0)) {
      K -= K0;
      A += (int64_t)K0 * (TA ? g.lda : 1);
      B += (int64_t)K0 * (TB ? g.ldb : 1);
    } else {
      K = K0;
    }
  } else {
    tile_origin<BM, BN>(g, bid, nt, m0, n0);
  }
  const int nk = (K + BK_ - 1) / BK_;

  MA ma;
  MB mb;
  ma.init(A, g.lda, m0, g.M, tid);
  mb.init(B, g.ldb, n0, g.N, tid);
  Frag16<BM, TA, MI, BK_, KS> fa;
  Frag16<BN, TB, NJ, BK_, KS> fb;
  fa.init(wm * WTM, lane, kg * KS);
  fb.init(wn * WTN, lane, kg * KS);
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) bf16_t *)lds);
  // load l (first A's, then B's) of slice t into stage st  (a whole contraction's length is read from the arguments: kept in a
  // variable it costs the largest shapes registers they do not have)
  auto issue = [&](int l, int t, int st) {
    const uint32_t b = lds0 + st * STAGE * 2;
    const int left = (HALVES ? K : g.K) - t * BK_;
    if (l < MA::N) ma.issue(l, t, left, b, wave);
    else mb.issue(l - MA::N, t, left, b + BM * BK_ * 2, wave);
  };
  f32x4_t acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int p = 0; p < S; ++p)
#pragma unroll
    for (int l = 0; l < NL; ++l) issue(l, p, p);
  // a slice has landed when at most the loads of the S - 1 younger ones are in flight
  wait_loads_le<(S - 1) * NL>();
  block_barrier();
  bf16x8_t af[2][MI], bfr[2][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i) af[0][i] = fa.get(lds, i, 0);
#pragma unroll
  for (int j = 0; j < NJ; ++j) bfr[0][j] = fb.get(lds + BM * BK_, j, 0);

  // one slice from stage st; its first step sits in fragment set P0
  auto slice = [&](int t, int st, auto parity) {
    constexpr int P0 = decltype(parity)::value;
    const bf16_t *const as = lds + st * STAGE;
    const int st_next = st + 1 == S ? 0 : st + 1;
#pragma unroll
    for (int kk = 0; kk < KS; ++kk) {
      constexpr int NR = MI + NJ, NS = MI * NJ;
      const int c = (kk + P0) & 1, nx = c ^ 1, nkk = kk + 1 < KS ? kk + 1 : 0;
      const bf16_t *na = as;
      if (kk + 1 == KS) {
        // slice t + 1 has landed, and this wavefront's reads of slice t are complete before anybody overwrites it
        wait_loads_le<(S - 2) * NL>();
        block_barrier();
        na = lds + st_next * STAGE;
      }
      const bf16_t *const nb = na + BM * BK_;
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const int q = i * NJ + j;
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bfr[c][j], af[c][i], acc[i][j], 0, 0, 0);
          __builtin_amdgcn_sched_barrier(0);
          // the next step's fragments one by one between the MFMAs, in the order it needs them
#pragma unroll
          for (int r = 0; r < NR; ++r)
            if ((NS >= NR ? r : r * NS / NR) == q) {
              if (r == 0) af[nx][0] = fa.get(na, 0, nkk);
              else if (r <= NJ) bfr[nx][r - 1] = fb.get(nb, r - 1, nkk);
              else af[nx][r - NJ] = fa.get(na, r - NJ, nkk);
            }
          // the loads of slice t + S into the stage slice t has left, spread over the last step
          if (kk + 1 == KS) {
#pragma unroll
            for (int l = 0; l < NL; ++l)
              if (l * NS / NL == q) issue(l, t + S, st);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
    }
  };
  typedef std::integral_constant<int, 0> even;
  typedef std::integral_constant<int, KS & 1> odd;  // slices of one step: the fragment sets change places from slice to slice
  for (int t = 0, st = 0; t < nk;) {
    slice(t, st, even());
    if (++st == S) st = 0;
    if (++t >= nk || KS > 1) continue;
    slice(t, st, odd());
    if (++st == S) st = 0;
    ++t;
  }
  wait_loads_le<0>();
  block_barrier();  // the write-out reuses the stages

  const bool vec = ((g.ldc & 3) == 0) &&
                   ((((uintptr_t)g.out_f32 | (uintptr_t)g.resid | (uintptr_t)g.bias) & 15) == 0) &&
                   ((((uintptr_t)g.out_act | (uintptr_t)g.out_act2 | (uintptr_t)g.aux) & 7) == 0);
  constexpr int SP = WTN + 4, PR = MI % (2 * KW) == 0 ? 32 : 16;  // rows staged at a time
  constexpr int MG = MI / KW;  // groups of 16 rows that a wavefront writes out
  if constexpr (KW > 1) {
    // every group of wavefronts holds a partial sum of the tile; group kg writes out rows kg*MG*16 .. of each
    // wavefront's part and receives them from the others through LDS, each in a fixed order
    static_assert(MG * KW == MI && KW * (KW - 1) * NG * MG * NJ * 64 * 16 <= S * STAGE * 2, "exchange fits the stages");
    f32x4_t *const xch = (f32x4_t *)lds;
    auto area = [&](int to, int from) { return ((to * (KW - 1) + (from < to ? from : from - 1)) * NG + wave % NG) * MG * NJ * 64 + lane; };
#pragma unroll
    for (int to = 0; to < KW; ++to)
      if (to != kg) {
#pragma unroll
        for (int i = 0; i < MG; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) xch[area(to, kg) + (i * NJ + j) * 64] = acc[to * MG + i][j];
      }
    __syncthreads();
    f32x4_t mine[MG][NJ];
#pragma unroll
    for (int to = 0; to < KW; ++to)
      if (to == kg) {
#pragma unroll
        for (int i = 0; i < MG; ++i)
#pragma unroll
          for (int j = 0; j < NJ; ++j) mine[i][j] = acc[to * MG + i][j];
      }
#pragma unroll
    for (int d = 1; d < KW; ++d) {
      const int from = (kg + d) % KW;
#pragma unroll
      for (int i = 0; i < MG; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j) mine[i][j] += xch[area(kg, from) + (i * NJ + j) * 64];
    }
#pragma unroll
    for (int i = 0; i < MG; ++i)
#pragma unroll
      for (int j = 0; j < NJ; ++j) acc[i][j] = mine[i][j];
    __syncthreads();  // the staging patches overlap the exchange area
  }
  static_assert(NW * PR * SP * 4 <= S * STAGE * 2, "staging patches must fit the stages");
  float *const patch = (float *)lds + wave * PR * SP;
#pragma unroll
  for (int i = 0; i < MG; i += PR / 16) {
#pragma unroll
    for (int h = 0; h < PR / 16; ++h)
#pragma unroll
      for (int j = 0; j < NJ; ++j)
        *(f32x4_t *)(patch + (h * 16 + (lane & 15)) * SP + j * 16 + (lane >> 4) * 4) = acc[i + h][j];
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_wave_barrier();
    if constexpr (HALVES) add_patch<WTN, PR>(g, patch, m0 + wm * WTM + (kg * MG + i) * 16, n0 + wn * WTN, lane);
    else store_patch<WTN, PR, true>(g, 0, patch, m0 + wm * WTM + (kg * MG + i) * 16, n0 + wn * WTN, lane, vec);
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_wave_barrier();
  }
}

template <int BM, int BN, int WM, int WN, int KW, int TA, int TB, int BK_, int S, int OCC>
__global__ __launch_bounds__(64 * WM * WN * KW, OCC * WM * WN * KW / 4) void gemm_plain_kernel(const GemmArgs g) {
  extern __shared__ __attribute__((aligned(16))) bf16_t lds_dyn[];
  gemm16_tile<BM, BN, WM, WN, KW, TA, TB, BK_, S>(g, blockIdx.x, gridDim.x, lds_dyn);
}

template <int BM, int BN, int WM, int WN, int BK_, int S>
__global__ __launch_bounds__(64 * WM * WN, WM * WN / 4) void gemm_halves_kernel(const GemmArgs g) {
  extern __shared__ __attribute__((aligned(16))) bf16_t lds_dyn[];
  gemm16_tile<BM, BN, WM, WN, 1, 0, 1, BK_, S, true>(g, blockIdx.x, gridDim.x, lds_dyn);
}

// the M x N results are cleared before the halves add to them
__global__ __launch_bounds__(256) void clear_result_kernel(float *__restrict__ c, int64_t ldc, int M, int N) {
  const int col = blockIdx.x * 256 + threadIdx.x;
  if (col >= N) return;
  for (int row = blockIdx.y; row < M; row += gridDim.y) c[row * ldc + col] = 0.f;
}

template <int SHAPE, int WM, int WN, int BK_, int S>
static hipError_t launch_halves(const GemmDesc &d, hipStream_t s) {
  constexpr int BM = half_shapes[SHAPE].bm, BN = half_shapes[SHAPE].bn;
  constexpr size_t lds = (size_t)S * (BM + BN) * BK_ * 2;
  GemmArgs a;
  gemm_fill_args(a, d);
  a.tiles_m = (a.M + BM - 1) / BM;
  a.tiles_n = (a.N + BN - 1) / BN;
  a.grp = xcd_group_rows(a.tiles_m, a.tiles_n, BM, BN, 32);
  auto kern = gemm_halves_kernel<BM, BN, WM, WN, BK_, S>;
  static OncePerGpu once;
  const hipError_t attr = allow_lds(once, (const void *)kern, lds);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL(clear_result_kernel, dim3((d.N + 255) / 256, d.M < 4096 ? d.M : 4096), dim3(256), 0, s, d.out_f32, d.ldc, d.M, d.N);
  hipLaunchKernelGGL(kern, dim3(2 * a.tiles_m * a.tiles_n), dim3(64 * WM * WN), lds, s, a);
  return hipGetLastError();
}

// A product that may be computed in two halves: fp32 results alone, nothing added to them, in memory that takes the additions
static bool halves_ok(const GemmDesc &d) {
  if (!d.out_f32 || d.out_act || d.resid || d.bias || d.epi != EPI_NONE) return false;
  hipPointerAttribute_t at;
  int gpu;
  if (hipPointerGetAttributes(&at, d.out_f32) != hipSuccess || hipGetDevice(&gpu) != hipSuccess) {
    (void)hipGetLastError();
    return false;
  }
  return atomic_adds_ok(at, gpu);
}

// Several products of one layout in one launch (the weight-gradient products of a block: each alone may leave most of
// the chip idle, together they fill it): workgroups tile0[i] .. tile0[i+1]-1 work on product i.
struct GemmGroup {
  GemmArgs p[GEMM_GROUP_MAX];
  int tile0[GEMM_GROUP_MAX + 1];
  int n;
};

template <int BM, int BN, int WM, int WN, int KW, int TA, int TB, int BK_, int S, int OCC>
__global__ __launch_bounds__(64 * WM * WN * KW, OCC * WM * WN * KW / 4) void gemm_plain_group_kernel(const GemmGroup gg) {
  extern __shared__ __attribute__((aligned(16))) bf16_t lds_dyn[];
  int i = 0;
#pragma unroll 1
  while (i + 1 < gg.n && (int)blockIdx.x >= gg.tile0[i + 1]) ++i;  // uniform over the workgroup
  gemm16_tile<BM, BN, WM, WN, KW, TA, TB, BK_, S>(gg.p[i], blockIdx.x - gg.tile0[i], gg.tile0[i + 1] - gg.tile0[i], lds_dyn);
}

// d[0..n): one product, or a group of contraction-strided ones.  LAYOUTS: the kernels for these alone are built
enum { ALL_LAYOUTS, TN_ONLY, ALL_BUT_TN };
template <int BM, int BN, int WM, int WN, int KW, int BK_, int S, int OCC, int LAYOUTS = ALL_LAYOUTS>
static hipError_t launch_shape(const GemmDesc *d, int n, hipStream_t s) {
  constexpr size_t lds = (size_t)S * (BM + BN) * BK_ * 2;
  constexpr int threads = 64 * WM * WN * KW;
  static_assert(lds * OCC <= 160 * 1024, "LDS per CU");
  GemmGroup gg;
  int tiles = 0;
  for (int i = 0; i < n; ++i) {
    GemmArgs &a = gg.p[i];
    gemm_fill_args(a, d[i]);
    a.tiles_m = (a.M + BM - 1) / BM;
    a.tiles_n = (a.N + BN - 1) / BN;
    a.grp = xcd_group_rows(a.tiles_m, a.tiles_n, BM, BN, 32 * OCC);
    gg.tile0[i] = tiles;
    tiles += a.tiles_m * a.tiles_n;
  }
#define HYDRA_SET_LDS(KERN_)                                        \
  static OncePerGpu once;                                           \
  const hipError_t attr = allow_lds(once, (const void *)KERN_, lds); \
  if (attr != hipSuccess) return attr
#define HYDRA_PLAIN(TA_, TB_)                                                                  \
  do {                                                                                         \
    auto kern = gemm_plain_kernel<BM, BN, WM, WN, KW, TA_, TB_, BK_, S, OCC>;                   \
    HYDRA_SET_LDS(kern);                                                                       \
    hipLaunchKernelGGL(kern, dim3(tiles), dim3(threads), lds, s, gg.p[0]);                      \
  } while (0)
  if (d->ta && d->tb) {
    if constexpr (LAYOUTS == ALL_BUT_TN) {
      return hipErrorInvalidValue;
    } else if (n > 1) {
      for (int i = n; i <= GEMM_GROUP_MAX; ++i) gg.tile0[i] = tiles;
      gg.n = n;
      auto kern = gemm_plain_group_kernel<BM, BN, WM, WN, KW, 1, 1, BK_, S, OCC>;
      HYDRA_SET_LDS(kern);
      hipLaunchKernelGGL(kern, dim3(tiles), dim3(threads), lds, s, gg);
    } else {
      HYDRA_PLAIN(1, 1);
    }
  } else if constexpr (LAYOUTS == TN_ONLY) {
    return hipErrorInvalidValue;
  } else if (d->ta) {
    HYDRA_PLAIN(1, 0);
  } else if (d->tb) {
    HYDRA_PLAIN(0, 1);
  } else {
    HYDRA_PLAIN(0, 0);
  }
#undef HYDRA_PLAIN
#undef HYDRA_SET_LDS
  return hipGetLastError();
}

static GemmDims dims_of(const GemmDesc &d) { return {d.M, d.N, d.K, d.ta != 0, d.tb != 0, (d.ldc & 3) == 0}; }

static hipError_t launch_best(const GemmDesc *d, int n, int shape, hipStream_t s) {
  static const char *const names[N_SHAPES][5] = {
#define HYDRA_N(X) {"gemm_bf16_" X "_nt", "gemm_bf16_" X "_nn", "gemm_bf16_" X "_tt", "gemm_bf16_" X "_tn", "gemm_bf16_" X "_tn_group"}
      HYDRA_N("256x256"), HYDRA_N("128x256"), HYDRA_N("128x192"), HYDRA_N("128x128"), HYDRA_N("128x64"),
      HYDRA_N("64x96"), HYDRA_N("64x64"), HYDRA_N("64x64k2"), HYDRA_N("128x64k2"), HYDRA_N("64x96k2"), HYDRA_N("128x128x2"), HYDRA_N("128x256x2")};
#undef HYDRA_N
  double flops = 0;
  for (int i = 0; i < n; ++i) flops += gemm_flops(d[i]);
  ProfScope ps(names[shape][n > 1 ? 4 : d->ta * 2 + d->tb], s, flops, 0);
  switch (shape) {
    case SHAPE_256X256:
      if (d->ta && d->tb) return launch_shape<256, 256, 2, 4, 1, 32, 4, 1, TN_ONLY>(d, n, s);  // see large_tn
      return launch_shape<256, 256, 2, 4, 1, 64, 2, 1, ALL_BUT_TN>(d, n, s);
    case 1: return launch_shape<128, 256, 2, 4, 1, 64, 3, 1>(d, n, s);
    case 2: return launch_shape<128, 192, 2, 4, 1, 64, 3, 1>(d, n, s);
    case 3: return launch_shape<128, 128, 2, 4, 1, 64, 4, 1>(d, n, s);
    case 4: return launch_shape<128, 64, 2, 2, 1, 64, 3, 2>(d, n, s);
    case 5: return launch_shape<64, 96, 2, 2, 1, 64, 3, 2>(d, n, s);
    case 6: return launch_shape<64, 64, 2, 2, 1, 64, 3, 3>(d, n, s);
    case 7: return launch_shape<64, 64, 2, 2, 2, 128, 4, 1>(d, n, s);
    case 8: return launch_shape<128, 64, 2, 2, 2, 128, 3, 1>(d, n, s);
    case 9: return launch_shape<64, 96, 2, 2, 2, 128, 3, 1>(d, n, s);
    case 10: return launch_shape<128, 128, 2, 2, 1, 64, 2, 2, TN_ONLY>(d, n, s);
    case SHAPE_128X256X2: return launch_shape<128, 256, 2, 2, 1, 32, 3, 2, TN_ONLY>(d, n, s);
    default: return hipErrorInvalidValue;
  }
}

bool gemm_plain_ok(const GemmDesc &d) {
  // 256 lines of a slice stay within a 32-bit byte offset
  return d.dtype == DT_BF16 && d.causal == CAUSAL_NONE && d.nb1 * d.nb2 == 1 && d.lda < 4000000 && d.ldb < 4000000;
}

hipError_t launch_gemm_plain(const GemmDesc &d, hipStream_t s) {
  const GemmDims x = dims_of(d);
  float cost;
  if (few_tiles(x)) {
    const int split = best_split_shape(x);
    return split >= 0 ? launch_gemm_split(d, split, s) : launch_best(&d, 1, SHAPE_64X64K2, s);
  }
  const int shape = best_shape(&x, 1, &cost), half = best_half_shape(x, cost);
  if (half >= 0 && halves_ok(d)) {
    static const char *const names[] = {"gemm_bf16_128x128_halves_nn", "gemm_bf16_128x192_halves_nn", "gemm_bf16_128x256_halves_nn"};
    ProfScope ps(names[half], s, gemm_flops(d), 0);
    switch (half) {
      case 0: return launch_halves<0, 2, 4, 64, 4>(d, s);
      case 1: return launch_halves<1, 2, 4, 64, 3>(d, s);
      case 2: return launch_halves<2, 2, 4, 64, 3>(d, s);
    }
  }
  return launch_best(&d, 1, shape, s);
}

// One launch wherever a grid holds it: of 950 groups (the four gradients of a block, width 32 to 4096, 8 to 8192 tokens) four
// launches were faster twice (by 2 and 3 %) and take 1.55 times as long at the median (us, together / alone: 792 wide, 238
// tokens 19.2 / 29.5, 1192 wide, 1144 tokens 67.8 / 83.1).
hipError_t launch_gemm_plain_group(const GemmDesc *d, int n, hipStream_t s) {
  GemmDims x[GEMM_GROUP_MAX];
  for (int i = 0; i < n; ++i) x[i] = dims_of(d[i]);
  float cost;
  const int shape = best_shape(x, n, &cost);
  if (n > 1 && shape_fits(plain_shapes[shape], x, n)) return launch_best(d, n, shape, s);
  for (int i = 0; i < n; ++i) {
    const hipError_t e = launch_gemm_plain(d[i], s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace hydra
