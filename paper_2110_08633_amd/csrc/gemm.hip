// GEMM kernels for gfx950: register-staged bf16 MFMA (batched and causal products, and the single ones that
// gemm_plain.hip leaves) and fp32 MFMA, both with the same fused epilogues (bias, residual, GELU, GELU', scale) and the
// same causal short-cuts for attention operands.
//
// The linear layers of a block (y = x*W + b), their input gradients
// (dx = dy*W^T) and weight gradients (dW = x^T*dy) and the batched attention
// products are all instances of C = alpha * op(A) * op(B) with a row-major C.
#include "gemm_common.h"

namespace hydra {

// ---------------------------------------------------------------------------
// Register-staged bf16 MFMA kernel.  256 threads = 4 wavefronts arranged WM x WN
// over a BM x BN tile of C.  K is consumed in slices of BK = 64:
//   global -> registers : 16-byte loads, issued D slices ahead
//   registers -> LDS    : one slice ahead, two LDS buffers, one barrier per slice
//   LDS -> MFMA operands: ds_read_b128 for operands whose contraction index is
//                         contiguous in memory, ds_read_tr16_b64 (transposing
//                         read) for operands stored with it strided, so both
//                         kinds sit in LDS exactly as they sit in memory
// LDS tiles carry no padding; their 16-byte chunks are XOR-swizzled so that the
// operand reads of 16 neighbouring lanes fall into distinct banks.
// The MFMA is issued with the B fragment as first operand, which leaves every
// lane with runs of 4 consecutive columns of one row of C: the epilogue then
// stores 16-byte (fp32) or 8-byte (bf16) vectors.
// ---------------------------------------------------------------------------
// One tile of one product: g describes the product, bid is the workgroup's index among the nt workgroups that
// work on it, z its batch index.
template <int BM, int BN, int WM, int WN, int TA, int TB, int D>
__device__ __forceinline__ void gemm_bf16_tile(const GemmArgs &g, const int bid, const int nt, const int z) {
  static_assert(D >= 2 && D % 2 == 0, "slices in flight");
  constexpr int WTM = BM / WM, WTN = BN / WN;
  constexpr int MI = WTM / 32, NJ = WTN / 32;
  // one LDS block: two buffers per operand during the K loop, per-wavefront staging of C in the epilogue
  __shared__ __attribute__((aligned(16))) bf16_t lds_all[2 * (BM + BN) * BK];
  bf16_t *const As[2] = {lds_all, lds_all + BM * BK};
  bf16_t *const Bs[2] = {lds_all + 2 * BM * BK, lds_all + 2 * BM * BK + BN * BK};

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  // consecutive workgroup ids are dealt round-robin to the 8 XCDs; renumber so that each XCD (own L2)
  // works on a contiguous run of tiles, which share operand rows
  const int xcd = bid & 7, per = nt >> 3, rem = nt & 7;
  const int tile = xcd * per + min(xcd, rem) + (bid >> 3);
  // ... and within the run, groups of up to g.grp tile rows are walked column by column: the tiles an XCD works on
  // at any time then share a few row panels of A and a few column panels of B instead of one A panel and all of B
  const int gsz = g.grp * g.tiles_n;
  const int grp = tile / gsz, in_grp = tile - grp * gsz;
  const int rows_in_grp = min(g.grp, g.tiles_m - grp * g.grp);
  const int tm = grp * g.grp + in_grp % rows_in_grp, tn = in_grp / rows_in_grp;
  const int m0 = tm * BM, n0 = tn * BN;
  if (g.causal == CAUSAL_SKIP_UPPER && n0 > m0 + BM - 1) return;
  const int z1 = z / g.nb2, z2 = z % g.nb2;
  const bf16_t *A = (const bf16_t *)g.A + z1 * g.sA1 + z2 * g.sA2;
  const bf16_t *B = (const bf16_t *)g.B + z1 * g.sB1 + z2 * g.sB2;
  const int64_t coff = z1 * g.sC1 + z2 * g.sC2;

  int kbeg = 0, kend = g.K;
  if (g.causal == CAUSAL_K_END) kend = min(g.K, m0 + BM);
  if (g.causal == CAUSAL_K_BEGIN) kbeg = m0;
  const int nk = (kend - kbeg + BK - 1) / BK;

  Mover<BM, TA> ma;
  Mover<BN, TB> mb;
  ma.init(A, g.lda, m0, g.M, kbeg, tid);
  mb.init(B, g.ldb, n0, g.N, kbeg, tid);
  u32x4_t ra[D][Mover<BM, TA>::N], rb[D][Mover<BN, TB>::N];

  int ao[MI][BK / 16][2], bo[NJ][BK / 16][2];
#pragma unroll
  for (int kk = 0; kk < BK / 16; ++kk) {
#pragma unroll
    for (int i = 0; i < MI; ++i) fragment_offsets<BM, TA>(wm * WTM + i * 32, kk, lane, ao[i][kk][0], ao[i][kk][1]);
#pragma unroll
    for (int j = 0; j < NJ; ++j) fragment_offsets<BN, TB>(wn * WTN + j * 32, kk, lane, bo[j][kk][0], bo[j][kk][1]);
  }

  f32x16_t acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int klen = kend - kbeg;
#pragma unroll
  for (int p = 0; p < D; ++p) {
    ma.load_tail(ra[p], p, klen - p * BK);
    mb.load_tail(rb[p], p, klen - p * BK);
  }
  ma.store(ra[0], As[0]);
  mb.store(rb[0], Bs[0]);
  __syncthreads();

  // All operand fragments of a slice are requested from LDS before the first MFMA: with one wavefront per SIMD
  // nothing else hides the LDS latency, and LDS returns data in order, so the MFMAs start as the first arrive.
  auto compute = [&](const bf16_t *as, const bf16_t *bs) {
    bf16x8_t af[BK / 16][MI], bfr[BK / 16][NJ];
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
#pragma unroll
      for (int i = 0; i < MI; ++i) af[kk][i] = fragment<TA>(as, ao[i][kk][0], ao[i][kk][1]);
#pragma unroll
      for (int j = 0; j < NJ; ++j) bfr[kk][j] = fragment<TB>(bs, bo[j][kk][0], bo[j][kk][1]);
    }
    __builtin_amdgcn_sched_barrier(0);  // keep the scheduler from sinking the reads between the MFMAs
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk)
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[kk][j], af[kk][i], acc[i][j], 0, 0, 0);
  };

  // Step for slice u = t + j: request slice u + D into the register set that slice u left, move slice u + 1 from
  // registers to the other LDS buffer, multiply slice u out of LDS buffer u & 1.  D slices are in flight.  Both
  // loops are free of conditions around the MFMAs, so the accumulators never move; the drain loop zero-fills
  // slices past the end of the contraction range (at most D - 1 all-zero slices are multiplied).
  int t = 0;
  if (nk <= 1) {  // a single slice (the head-width contractions of attention): nothing to pipeline
    compute(As[0], Bs[0]);
    t = nk;
    __syncthreads();  // the epilogue reuses the operand buffers: every wavefront must be done reading them
  }
  for (; t + 2 * D + 1 <= nk; t += D) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
      ma.load_full(ra[j], t + j + D);
      mb.load_full(rb[j], t + j + D);
      ma.store(ra[(j + 1) % D], As[(j + 1) & 1]);
      mb.store(rb[(j + 1) % D], Bs[(j + 1) & 1]);
      compute(As[j & 1], Bs[j & 1]);
      __syncthreads();
    }
  }
  for (; t < nk; t += D) {
#pragma unroll
    for (int j = 0; j < D; ++j) {
      ma.load_tail(ra[j], t + j + D, klen - (t + j + D) * BK);
      mb.load_tail(rb[j], t + j + D, klen - (t + j + D) * BK);
      ma.store(ra[(j + 1) % D], As[(j + 1) & 1]);
      mb.store(rb[(j + 1) % D], Bs[(j + 1) & 1]);
      compute(As[j & 1], Bs[j & 1]);
      __syncthreads();
    }
  }
  // Epilogue through LDS.  Lane L of a 32x32 result (B fragment first) holds row L%32 and columns
  // (r/4)*8 + (L/32)*4 + r%4: storing that directly would touch 32 different rows per instruction.  Each
  // wavefront instead parks 32 rows of its sub-tile in a private LDS patch [32][WTN + 4] (fp32) and reads it
  // back row-wise, so every store instruction covers whole row segments of C.
  const bool vec = ((g.ldc & 3) == 0) && ((coff & 3) == 0) &&
                   ((((uintptr_t)g.out_f32 | (uintptr_t)g.resid | (uintptr_t)g.bias) & 15) == 0) &&
                   ((((uintptr_t)g.out_act | (uintptr_t)g.out_act2 | (uintptr_t)g.aux) & 7) == 0);
  constexpr int SP = WTN + 4;                 // patch pitch in floats
  static_assert(4 * 32 * SP * 4 <= 2 * (BM + BN) * BK * 2, "staging patches must fit the operand buffers");
  float *const patch = (float *)lds_all + wave * 32 * SP;
  // every wavefront has passed the last barrier of the K loop, so nobody reads the operand buffers any more
#pragma unroll
  for (int i = 0; i < MI; ++i) {
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        f32x4_t v = {acc[i][j][q * 4 + 0], acc[i][j][q * 4 + 1], acc[i][j][q * 4 + 2], acc[i][j][q * 4 + 3]};
        *(f32x4_t *)(patch + (lane & 31) * SP + j * 32 + q * 8 + (lane >> 5) * 4) = v;
      }
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the patch is written (LDS serves a wavefront in order)
    __builtin_amdgcn_wave_barrier();
    store_patch<WTN, 32, false>(g, coff, patch, m0 + wm * WTM + i * 32, n0 + wn * WTN, lane, vec);
    __builtin_amdgcn_s_waitcnt(0xc07f);
    __builtin_amdgcn_wave_barrier();
  }
}

template <int BM, int BN, int WM, int WN, int TA, int TB, int D>
__global__ __launch_bounds__(256, 2) void gemm_bf16_kernel(const GemmArgs g) {
  gemm_bf16_tile<BM, BN, WM, WN, TA, TB, D>(g, blockIdx.x, gridDim.x, blockIdx.y);
}

// ---------------------------------------------------------------------------
// fp32 kernel: v_mfma_f32_32x32x2_f32 and 16x16x4 (full fp32 products and sums,
// no reduced-precision split; each is a chain of fused multiply-adds over its
// contraction steps in ascending order).  The instruction needs 64 clocks for 4096 flop, so
// LDS and the load path are far from binding (a 32x32 result per wavefront
// reads 8 bytes of LDS per clock, 32 on a CU's four SIMDs); what costs is everything that keeps
// the matrix pipes waiting: too few tiles for 256 CUs and trips to memory.
// Hence small tiles, operands requested two slices ahead (16-byte loads into
// registers where alignment allows), two LDS buffers and one barrier per slice.
//   64x64 tiles: 2x2 wavefronts, 32 contraction steps per slice
//   32x32 tiles: 2x2 wavefronts of 16x16 results, 64 steps per slice - four times
//                the tiles where 64x64 ones would leave CUs idle
// A result is one chain of fused multiply-adds over ascending k, whatever the
// tile: the sum does not depend on the shape, and parameters whose gradient is
// zero but for rounding (the key bias) see the same rounding everywhere.
// An operand sits in LDS as it sits in memory: [row][k] when its contraction
// index is contiguous (steps regrouped so that a lane's four are neighbours),
// else [k][row].  A lane feeds row L%MT and steps e * KG + L/MT, e = 0..3, of
// every group of 4 * KG.
// Bank conflicts of 32x32 tiles: those of [k][row] (reads: 40 % of the LDS cycles) are gone with the swizzle of at(), those of
// [row][k] (stores: half of the cycles) are a third with that of place(): 768x3072x1000 tn 50.4 -> 47.2 us, 1024x1024x4096 tn
// 85 -> 79, 4096x1024x1024 nt 75 -> 72.
// Measured against the former vector-ALU kernel (64x64 tiles, 4-byte loads, no
// prefetch): 1000x3072x768 265 -> 51 us, 128x128x512 34 -> 6 us, 4096^3 at 128
// TFLOP/s of the 157 the matrix pipes offer; the results are the same to the bit.
// ---------------------------------------------------------------------------
// Global -> registers -> LDS mover of one operand: R rows x BKF contraction steps per slice.  Buffer loads, so that
// elements outside the operand are fetched from an out-of-range offset (zero) instead of behind a branch: a register
// that is cleared under a condition makes the compiler wait for every load in flight before it reuses the register.
// LD_VEC: 16-byte loads; LD_SCALAR: 4-byte loads for operands whose alignment does not allow them; LD_WIDE: leading
// dimensions that a 32-bit offset within a slice cannot hold
enum { LD_VEC = 0, LD_SCALAR = 1, LD_WIDE = 2 };
template <int R, int BKF, int RC, int KG, int MODE>
struct MoverF {
  static constexpr int LEN = RC ? R : BKF;           // elements per line of memory (row of [row][k] / [k][row])
  // LDS pitch in floats: 16 bytes of padding spread the banks of [row][k]; [k][row] is swizzled instead, see at()
  static constexpr int PITCH = RC ? LEN : LEN + 4;
  static constexpr int SIZE = (RC ? BKF : R) * PITCH;
  static constexpr int W = MODE == LD_VEC ? 4 : 1;   // elements per load
  static constexpr int NL = R * BKF / 256 / W;       // loads per thread and slice
  static constexpr int N = R * BKF / 256 / 4;        // 4-element registers per thread and slice
  static constexpr int LS = 256 * W / LEN;           // lines between a thread's loads
  static_assert(NL >= 1 && NL * 256 * W == R * BKF && 256 * W % LEN == 0, "the slice divides evenly over the threads");
  const float *base;  // the tile's first row, contraction step 0
  int64_t ld;
  int rows, line, c;  // rows from the tile's first to the matrix's end; this thread's first line and its place in a line
  __device__ __forceinline__ void init(const float *mat, int64_t ld_, int row0, int rows_, int tid) {
    ld = ld_;
    base = RC ? mat + row0 : mat + (int64_t)row0 * ld;
    rows = rows_ - row0;
    line = tid / (LEN / W);
    c = (tid % (LEN / W)) * W;
  }
  // contraction steps k0 .. k0 + BKF - 1; steps from kend on and rows past the matrix read as zero
  __device__ __forceinline__ void load(f32x4_t (&r)[N], int k0, int kend) const {
    const float *const b = base + (RC ? k0 * ld : (int64_t)k0);
    const __amdgpu_buffer_rsrc_t rs = buffer_at(b);
    const int off = (int)((line * ld + c) * 4);
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int l = line + j * LS;
      const bool in = (RC ? c : l) < rows && k0 + (RC ? l : c) < kend;
      if (MODE == LD_VEC) {
        union { u32x4_t u; f32x4_t f; } x;
        x.u = __builtin_amdgcn_raw_buffer_load_b128(rs, in ? off + (int)(j * LS * ld * 4) : BUF_OUT, 0, 0);
        r[j] = x.f;
      } else if (MODE == LD_SCALAR) {
        r[j / 4][j % 4] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, in ? off + (int)(j * LS * ld * 4) : BUF_OUT, 0, 0));
      } else {
        r[j / 4][j % 4] = in ? b[l * ld + c] : 0.f;
      }
    }
  }
  // position of contraction step k in a line of [row][k]: within every 4 * KG steps, those of one lane group together; of
  // four runs of sixteen steps the last two change their pairs of groups, so that a store's lanes fall into distinct banks
  static __device__ __forceinline__ int group(int k, int kq) { return KG == 4 ? kq ^ (k >> 4 & 2) : kq; }
  static __device__ __forceinline__ int place(int k) { return k / (4 * KG) * (4 * KG) + group(k, k % KG) * 4 + k % (4 * KG) / KG; }
  // [k][row]: the lane groups of a read, neighbouring steps, fall into distinct halves or quarters of the banks
  static __device__ __forceinline__ int at(int k, int row) {
    return k * PITCH + (row ^ (KG == 4 ? ((k ^ k >> 1) & 1) << 4 : (k & 1) << 5));
  }
  __device__ __forceinline__ void store(const f32x4_t (&r)[N], float *lds) const {
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      float *const p = lds + (line + j * LS) * PITCH;
      if (RC) {
        float *const q = lds + at(line + j * LS, c);
        if (MODE != LD_VEC) *q = r[j / 4][j % 4];
        else *(f32x4_t *)q = r[j];
      } else if (MODE != LD_VEC) {
        p[place(c)] = r[j / 4][j % 4];
      } else if (KG == 2) {  // steps c, c + 2 and c + 1, c + 3 are neighbours
        *(f32x2_t *)(p + place(c)) = f32x2_t{r[j][0], r[j][2]};
        *(f32x2_t *)(p + place(c) + 4) = f32x2_t{r[j][1], r[j][3]};
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) p[place(c + e)] = r[j][e];
      }
    }
  }
  // lane group kq's four of the 4 * KG steps that start at k, of row: steps k + e * KG + kq, e = 0..3
  static __device__ __forceinline__ f32x4_t frag(const float *lds, int row, int k, int kq) {
    if (!RC) return *(const f32x4_t *)(lds + row * PITCH + k + group(k, kq) * 4);
    f32x4_t v;
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = lds[at(k + e * KG + kq, row)];
    return v;
  }
};

// four consecutive columns of one row of C
__device__ __forceinline__ void epilogue_store4_f32(const GemmArgs &g, int64_t coff, int row, int col, const f32x4_t acc,
                                                    bool vec) {
  if (!vec || col + 3 >= g.N) {
#pragma unroll 1
    for (int e = 0; e < 4; ++e) {
      const float x = e == 0 ? acc[0] : e == 1 ? acc[1] : e == 2 ? acc[2] : acc[3];  // see epilogue_store4
      if (col + e < g.N) epilogue_store<float>(g, coff, row, col + e, x);
    }
    return;
  }
  const int64_t idx = coff + (int64_t)row * g.ldc + col;
  f32x4_t v = acc * g.alpha;
  if (g.bias) v += *(const f32x4_t *)(g.bias + col);
  if (g.epi == EPI_GELU) {
    const f32x4_t h = {gelu_f(v[0]), gelu_f(v[1]), gelu_f(v[2]), gelu_f(v[3])};
    *(f32x4_t *)((float *)g.out_act + idx) = v;
    *(f32x4_t *)((float *)g.out_act2 + idx) = h;
    return;
  }
  if (g.epi == EPI_DGELU) {
    const f32x4_t a = *(const f32x4_t *)((const float *)g.aux + idx);
    const f32x4_t dg = {dgelu_f(a[0]), dgelu_f(a[1]), dgelu_f(a[2]), dgelu_f(a[3])};
    v *= dg;
  }
  if (g.resid) v += *(const f32x4_t *)(g.resid + idx);
  if (g.out_f32) *(f32x4_t *)(g.out_f32 + idx) = v;
  if (g.out_act) *(f32x4_t *)((float *)g.out_act + idx) = v;
}

template <int MT, int BKF, int TA, int TB, int MODE>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const GemmArgs g) {
  constexpr int BM = 2 * MT, BN = 2 * MT;  // 2x2 wavefronts, one MT x MT result each
  constexpr int KG = 64 / MT;              // lane groups = contraction steps of one MFMA
  constexpr int NR = MT * MT / 64;         // accumulator registers
  typedef MoverF<BM, BKF, TA, KG, MODE> MA;
  typedef MoverF<BN, BKF, TB, KG, MODE> MB;
  typedef __attribute__((ext_vector_type(NR))) float acc_t;
  constexpr int STAGE = MA::SIZE + MB::SIZE;
  static_assert(BKF % (4 * KG) == 0, "whole groups of steps");
  __shared__ __attribute__((aligned(16))) float lds[2 * STAGE];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  // tile numbering as in the bf16 kernels: contiguous runs per XCD, groups of g.grp tile rows walked column by column
  const int nt = gridDim.x, bid = blockIdx.x, xcd = bid & 7, per = nt >> 3, rem = nt & 7;
  const int tile = xcd * per + min(xcd, rem) + (bid >> 3);
  const int gsz = g.grp * g.tiles_n;
  const int grp = tile / gsz, in_grp = tile - grp * gsz;
  const int rows_in_grp = min(g.grp, g.tiles_m - grp * g.grp);
  const int m0 = (grp * g.grp + in_grp % rows_in_grp) * BM, n0 = (in_grp / rows_in_grp) * BN;
  if (g.causal == CAUSAL_SKIP_UPPER && n0 > m0 + BM - 1) return;
  const int z = blockIdx.y, z1 = z / g.nb2, z2 = z % g.nb2;
  const int64_t coff = z1 * g.sC1 + z2 * g.sC2;
  int kbeg = 0, kend = g.K;
  if (g.causal == CAUSAL_K_END) kend = min(g.K, m0 + BM);
  if (g.causal == CAUSAL_K_BEGIN) kbeg = m0;
  const int nk = kend > kbeg ? (kend - kbeg + BKF - 1) / BKF : 0;

  MA ma;
  MB mb;
  ma.init((const float *)g.A + z1 * g.sA1 + z2 * g.sA2, g.lda, m0, g.M, tid);
  mb.init((const float *)g.B + z1 * g.sB1 + z2 * g.sB2, g.ldb, n0, g.N, tid);
  f32x4_t ra[2][MA::N], rb[2][MB::N];
  acc_t acc;
#pragma unroll
  for (int r = 0; r < NR; ++r) acc[r] = 0.f;

  const int arow = wm * MT + lane % MT, brow = wn * MT + lane % MT, kq = lane / MT;
  auto compute = [&](const float *as, const float *bs) {
#pragma unroll
    for (int k = 0; k < BKF; k += 4 * KG) {
      const f32x4_t a = MA::frag(as, arow, k, kq), b = MB::frag(bs, brow, k, kq);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (MT == 32) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(b[e], a[e], acc, 0, 0, 0);
        else acc = __builtin_amdgcn_mfma_f32_16x16x4f32(b[e], a[e], acc, 0, 0, 0);
      }
    }
  };
  // slice t travels in register set t & 1 and LDS buffer t & 1
  auto step = [&](int t, auto setc) {
    constexpr int S = decltype(setc)::value;
    ma.load(ra[S], kbeg + (t + 2) * BKF, kend);  // past the end: zeros, without a memory access
    mb.load(rb[S], kbeg + (t + 2) * BKF, kend);
    compute(lds + S * STAGE, lds + S * STAGE + MA::SIZE);
    if (t + 1 < nk) {
      ma.store(ra[S ^ 1], lds + (S ^ 1) * STAGE);
      mb.store(rb[S ^ 1], lds + (S ^ 1) * STAGE + MA::SIZE);
    }
    __syncthreads();
  };
  if (nk > 0) {
    ma.load(ra[0], kbeg, kend);
    mb.load(rb[0], kbeg, kend);
    ma.load(ra[1], kbeg + BKF, kend);
    mb.load(rb[1], kbeg + BKF, kend);
    ma.store(ra[0], lds);
    mb.store(rb[0], lds + MA::SIZE);
  }
  __syncthreads();
  for (int t = 0; t < nk; t += 2) {
    step(t, std::integral_constant<int, 0>());
    if (t + 1 < nk) step(t + 1, std::integral_constant<int, 1>());
  }

  const bool vec = ((g.ldc & 3) == 0) && ((coff & 3) == 0) &&
                   ((((uintptr_t)g.out_f32 | (uintptr_t)g.resid | (uintptr_t)g.bias | (uintptr_t)g.out_act |
                      (uintptr_t)g.out_act2 | (uintptr_t)g.aux) & 15) == 0);
  const int row = m0 + arow, col = n0 + wn * MT + kq * 4;
  if (row < g.M) {
#pragma unroll
    for (int q = 0; q < NR / 4; ++q) {
      const f32x4_t v = {acc[q * 4 + 0], acc[q * 4 + 1], acc[q * 4 + 2], acc[q * 4 + 3]};
      epilogue_store4_f32(g, coff, row, col + q * 8, v, vec);
    }
  }
}

template <int MT, int BKF, int MODE>
static hipError_t launch_f32_cfg(GemmArgs &a, int ta, int tb, int nbatch, hipStream_t s) {
  constexpr int BT = 2 * MT;
  a.tiles_m = (a.M + BT - 1) / BT;
  a.tiles_n = (a.N + BT - 1) / BT;
  a.grp = xcd_group_rows(a.tiles_m, a.tiles_n, BT, BT);
  dim3 grid(a.tiles_m * a.tiles_n, nbatch);
  if (ta == 0 && tb == 0) hipLaunchKernelGGL((gemm_f32_kernel<MT, BKF, 0, 0, MODE>), grid, dim3(256), 0, s, a);
  else if (ta == 0 && tb == 1) hipLaunchKernelGGL((gemm_f32_kernel<MT, BKF, 0, 1, MODE>), grid, dim3(256), 0, s, a);
  else if (ta == 1 && tb == 1) hipLaunchKernelGGL((gemm_f32_kernel<MT, BKF, 1, 1, MODE>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((gemm_f32_kernel<MT, BKF, 1, 0, MODE>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

// 16-byte loads of an fp32 operand: aligned rows and no chunk that straddles the end of the contiguous extent (rows
// of a row-contiguous operand, contraction range of the other kind - a causal range ends at a multiple of 32 or at K)
static bool f32_vec_ok(const void *p, int64_t ld, int64_t s1, int64_t s2, int extent) {
  return (((uintptr_t)p) & 15) == 0 && !((ld | s1 | s2 | extent) & 3);
}

constexpr int64_t F32_LD_MAX = 0x70000000 / (64 * 4);  // 64 lines of a slice stay below 2 GB
static hipError_t launch_gemm_f32(GemmArgs &a, const GemmDesc &d, int nbatch, hipStream_t s) {
  const bool vec = f32_vec_ok(d.A, d.lda, d.sA1, d.sA2, d.ta ? d.M : d.K) && f32_vec_ok(d.B, d.ldb, d.sB1, d.sB2, d.tb ? d.N : d.K);
  const long t64 = (long)((d.M + 63) / 64) * ((d.N + 63) / 64) * nbatch;
  const bool wide = d.lda >= F32_LD_MAX || d.ldb >= F32_LD_MAX;
  // 64x64 tiles once they go round the 256 CUs two and a half times: below that the last round leaves too many idle
  // (us, 64x64 / 32x32 tiles: 192 tiles 72 / 57 at 1000x768x3072, 384 tiles 83 / 75 at 2048x768x2304, 768 tiles
  // 51 / 56 at 1000x3072x768, 4096 tiles 1074 / 1192 at 4096^3)
  if (t64 >= 640)
    return wide  ? launch_f32_cfg<32, 32, LD_WIDE>(a, d.ta, d.tb, nbatch, s)
           : vec ? launch_f32_cfg<32, 32, LD_VEC>(a, d.ta, d.tb, nbatch, s)
                 : launch_f32_cfg<32, 32, LD_SCALAR>(a, d.ta, d.tb, nbatch, s);
  if (wide) return launch_f32_cfg<16, 64, LD_WIDE>(a, d.ta, d.tb, nbatch, s);
  return vec ? launch_f32_cfg<16, 64, LD_VEC>(a, d.ta, d.tb, nbatch, s)
             : launch_f32_cfg<16, 64, LD_SCALAR>(a, d.ta, d.tb, nbatch, s);
}

template <int BM, int BN, int WM, int WN, int D>
static hipError_t launch_bf16_cfg(const GemmArgs &a, int ta, int tb, dim3 grid, hipStream_t s) {
  if (ta == 0 && tb == 0) {
    // (both operands contraction-contiguous: only ever 128x64 tiles)
    if constexpr (BM == 128 && BN == 64) hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, WM, WN, 0, 0, D>), grid, dim3(256), 0, s, a);
    else return hipErrorInvalidValue;
  } else if (ta == 0) {
    hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, WM, WN, 0, 1, D>), grid, dim3(256), 0, s, a);
  } else if (tb == 1) {
    hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, WM, WN, 1, 1, D>), grid, dim3(256), 0, s, a);
  } else {
    hipLaunchKernelGGL((gemm_bf16_kernel<BM, BN, WM, WN, 1, 0, D>), grid, dim3(256), 0, s, a);
  }
  return hipGetLastError();
}

// algorithmic flops of a launch: causal products only count the triangle
double gemm_flops(const GemmDesc &d) {
  const double nb = (double)d.nb1 * d.nb2;
  if (d.causal == CAUSAL_SKIP_UPPER) return nb * 2.0 * d.K * (0.5 * d.M * (d.M + 1.0));
  if (d.causal == CAUSAL_K_END || d.causal == CAUSAL_K_BEGIN) return nb * 2.0 * d.N * (0.5 * d.M * (d.M + 1.0));
  return nb * 2.0 * d.M * d.N * d.K;
}

static const char *gemm_name(int bn, int ta, int tb) {
  static const char *n128[4] = {"gemm_bf16_staged_128x128_nt", "gemm_bf16_staged_128x128_nn",
                                "gemm_bf16_staged_128x128_tt", "gemm_bf16_staged_128x128_tn"};
  static const char *n64[4] = {"gemm_bf16_staged_x64_nt", "gemm_bf16_staged_x64_nn", "gemm_bf16_staged_x64_tt",
                               "gemm_bf16_staged_x64_tn"};
  return (bn == 128 ? n128 : n64)[ta * 2 + tb];
}

void gemm_fill_args(GemmArgs &a, const GemmDesc &d) {
  a.A = d.A; a.B = d.B; a.M = d.M; a.N = d.N; a.K = d.K;
  a.lda = d.lda; a.ldb = d.ldb; a.ldc = d.ldc;
  a.nb2 = d.nb2;
  a.sA1 = d.sA1; a.sA2 = d.sA2; a.sB1 = d.sB1; a.sB2 = d.sB2; a.sC1 = d.sC1; a.sC2 = d.sC2;
  a.alpha = d.alpha; a.bias = d.bias; a.resid = d.resid;
  a.out_f32 = d.out_f32; a.out_act = d.out_act; a.out_act2 = d.out_act2; a.aux = d.aux;
  a.epi = d.epi; a.causal = d.causal;
  a.grp = 8;
}

// operand alignment the vector loads of the bf16 kernels rely on
static bool bf16_operands_ok(const GemmDesc &d) {
  return !((d.lda & 7) || (d.ldb & 7) || (((uintptr_t)d.A) & 15) || (((uintptr_t)d.B) & 15) || (d.sA1 & 7) || (d.sA2 & 7) ||
           (d.sB1 & 7) || (d.sB2 & 7));
}

// Single products whose contraction fits one slice of the register-staged kernel: there is nothing to pipeline, a launch
// is its write-out, and that kernel's shorter way to the first MFMA wins with both operands contraction-contiguous and
// otherwise once 128x64 tiles go round the CUs; not where rows are unaligned, which the other kernel stores better.
// us at K 64, staged / direct to LDS: nt 1000x1000 6.4 / 6.8, 201x2304 4.1 / 4.3, 2048x4096 8.3 / 9.4; tn 1024x4096 6.4 /
// 7.0, 1600x6400 11.0 / 12.3, 4096x4096 14.4 / 15.2, but 768x2304 4.6 / 4.3; nn 2048x4096 8.5 / 9.6, but 1000x1000 6.4 / 4.8;
// rows of 1001: nn 1000x1001 11.1 / 5.1
static bool one_slice(const GemmDesc &d) {
  return d.K <= BK && !(d.ldc & 3) && ((!d.ta && !d.tb) || (long)((d.M + 127) / 128) * ((d.N + 63) / 64) > 256);
}

hipError_t launch_gemm(const GemmDesc &d, hipStream_t s) {
  if (d.M <= 0 || d.N <= 0 || d.nb1 * d.nb2 <= 0) return hipSuccess;
  GemmArgs a;
  gemm_fill_args(a, d);
  const int nbatch = d.nb1 * d.nb2;
  if (d.dtype == DT_F32) {
    ProfScope ps("gemm_f32", s, gemm_flops(d), 0);
    return launch_gemm_f32(a, d, nbatch, s);
  }
  if (!bf16_operands_ok(d)) return hipErrorInvalidValue;
  if (gemm_plain_ok(d) && !one_slice(d)) return launch_gemm_plain(d, s);
  // batched and causal products (attention at head widths without a fused kernel), one-slice products, and leading
  // dimensions beyond what the single-product kernel addresses.  128x128 tiles for many rounds of them, 64x64 ones when 128x64 tiles would
  // not occupy half the CUs (a third faster there); neither where both operands are contraction-contiguous (scores of
  // 64 pairs of T 1024, head width 32, causal: 52 us with 128x64 tiles, 55 with 128x128)
  const bool nt = !d.ta && !d.tb;
  const long t128 = (long)((d.M + 127) / 128) * ((d.N + 127) / 128) * nbatch;
  int tile = (!nt && d.N > 64 && t128 >= 2048) ? 1 : 2;
  if (tile == 2 && !nt && (long)((d.M + 127) / 128) * ((d.N + 63) / 64) * nbatch < 128 && d.M > 64) tile = 3;
  // slices in flight: a deeper pipeline pays once the contraction is long enough to amortise filling it (of the products
  // that come here, those with leading dimensions beyond the single-product kernel's)
  const int D = (d.causal == CAUSAL_NONE && d.K >= 24 * BK) ? 4 : 2;
#define HYDRA_LAUNCH(BM_, BN_, DD_)                                                                      \
  do {                                                                                                    \
    a.tiles_m = (d.M + BM_ - 1) / BM_;                                                                    \
    a.tiles_n = (d.N + BN_ - 1) / BN_;                                                                    \
    a.grp = xcd_group_rows(a.tiles_m, a.tiles_n, BM_, BN_);                                               \
    ProfScope ps(gemm_name(BN_, d.ta, d.tb), s, gemm_flops(d), 0);                                        \
    return launch_bf16_cfg<BM_, BN_, 2, 2, DD_>(a, d.ta, d.tb, dim3(a.tiles_m * a.tiles_n, nbatch), s); \
  } while (0)
  if (tile == 1) HYDRA_LAUNCH(128, 128, 2);
  if (tile == 3) {
    if (D == 4) HYDRA_LAUNCH(64, 64, 4);
    HYDRA_LAUNCH(64, 64, 2);
  }
  if (D == 4) HYDRA_LAUNCH(128, 64, 4);
  HYDRA_LAUNCH(128, 64, 2);
#undef HYDRA_LAUNCH
}

hipError_t launch_gemm_group(const GemmDesc *d, int n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  bool group = n <= GEMM_GROUP_MAX;
  for (int i = 0; i < n && group; ++i)
    group = d[i].dtype == DT_BF16 && d[i].ta == 1 && d[i].tb == 1 && d[i].M > 0 && d[i].N > 0 && bf16_operands_ok(d[i]) &&
            gemm_plain_ok(d[i]);
  if (group) return launch_gemm_plain_group(d, n, s);
  for (int i = 0; i < n; ++i) {  // other layouts and dtypes: one launch each
    const hipError_t e = launch_gemm(d[i], s);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace hydra
