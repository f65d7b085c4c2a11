// Fused causal self-attention for the bf16 path (gfx950): scores, mask,
// softmax and the product with V in one kernel, and the matching backward
// kernels, so that no T x T matrix ever reaches HBM.  Only what lies on or
// below the diagonal is computed.
//
// The attention of one (sample, head): s[i,j] = q_i . k_j / sqrt(dh) for
// j <= i, p = softmax_j(s), o_i = sum_j p[i,j] v_j.  The forward kernel keeps,
// per row, only the log-sum-exp L_i = log sum_j exp(s[i,j]); the backward
// kernels rebuild p[i,j] = exp(s[i,j] - L_i) from q and k.
//
// Operand conventions: v_mfma_f32_32x32x16_bf16 with the column operand first, so a
// lane holds row L%32 of a 32x32 result and columns (r/4)*8 + (L/32)*4 + r%4 for
// r = 0..15.  Tiles of 32 or 64 rows go straight to LDS (one copy, read both along
// the head dimension and, transposing, along the rows); probabilities stay in the
// registers they are computed in.
#include <cfloat>

#include "attn_forms.h"
#include "gemm_common.h"

namespace hydra {

namespace {

// A block: KW groups of RW wavefronts.  It owns 32 * RW rows (queries, or keys in the dK/dV kernel), 32 per wavefront of a
// group, and walks over tiles of TK rows (keys, or queries in the dK/dV kernel), which its groups share out.
constexpr float LOG2E = 1.4426950408889634f, LN2 = 0.6931471805599453f;

// value of the lane 32 away and the lane's own, in either order
__device__ __forceinline__ void halves(float x, float &a, float &b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  a = __uint_as_float(r[0]);
  b = __uint_as_float(r[1]);
}
__device__ __forceinline__ float sum_halves(float x) { float a, b; halves(x, a, b); return a + b; }
__device__ __forceinline__ float max_halves(float x) { float a, b; halves(x, a, b); return __builtin_fmaxf(a, b); }

__device__ __forceinline__ bf16x8_t load_frag_global(const bf16_t *p) {
  union { u32x4_t u; bf16x8_t f; } x;
  x.u = *(gvec_ptr)p;
  return x.f;
}

// s + the products of eight bf16 elements
__device__ __forceinline__ float dot8(const u32x4_t a, const u32x4_t b, float s) {
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    s = __builtin_fmaf(__uint_as_float(a[e] << 16), __uint_as_float(b[e] << 16), s);
    s = __builtin_fmaf(__uint_as_float(a[e] & 0xffff0000u), __uint_as_float(b[e] & 0xffff0000u), s);
  }
  return s;
}

// Results r = 8*s .. 8*s + 7 of a lane (row L%32, columns (r/4)*8 + (L/32)*4 + r%4) as the row operand of a product
// that contracts over those columns: rounded to bf16, they already sit in the right lane - lane half h holds steps
// 4h .. 4h+3 and 8+4h .. 11+4h of the sixteen, and RowTile::tr feeds the other operand's steps in the same order.  So
// probabilities never leave the registers.
__device__ __forceinline__ bf16x8_t row_operand(const float (&p)[16], int s) {
  union { uint32_t u[4]; bf16x8_t f; } x;
#pragma unroll
  for (int e = 0; e < 4; ++e) x.u[e] = pack_bf16(p[s * 8 + 2 * e], p[s * 8 + 2 * e + 1]);
  return x.f;
}

// A [TK rows][DH] bf16 tile of a row-major matrix in LDS, loaded by RW wavefronts: DH/64 slices [row][64] whose 16-byte
// chunks are swizzled so that both ways of reading it are free of bank conflicts - as operand of a product over the head
// dimension (16 bytes per lane: rows of one parity need distinct slots) and, through the transposing read, of a product
// over the rows (32 bytes of rows k..k+3 each, two column groups at a time).  One copy serves both.
template <int DH, int RW, int TK>
struct RowTile {
  static constexpr int SIZE = TK * DH;            // elements
  static constexpr int N = SIZE / 8 / (64 * RW);  // 16-byte loads per lane
  static constexpr int RP = 8 * RW, PS = TK / RP;  // rows per load, loads per slice
  static_assert(PS * RP == TK && N == PS * DH / 64, "whole loads");
  int off, row;  // byte offset and row of this lane's first chunk; the others are RP rows and 64 columns further on
  int64_t ld;
  static __device__ __forceinline__ int swz(int r) { return ((r >> 1) & 1) << 2 | ((r >> 2) & 1) << 1 | ((r >> 3) & 1); }
  __device__ __forceinline__ void init(int64_t ld_, int tid) {  // tid within the RW wavefronts
    ld = ld_;
    row = tid >> 3;
    off = (int)((row * ld + ((tid & 7) ^ swz(row)) * 8) * 2);
  }
  // base: element (first row of the tile, first column of the head), uniform; rows from `valid` on read as zero.
  // DIRECT: straight to LDS, which wants aligned addresses; else through registers, whose loads take any
  template <bool DIRECT>
  __device__ __forceinline__ void load(const bf16_t *base, int valid, uint32_t lds, int wave) const {
    int o[PS];
#pragma unroll
    for (int i = 0; i < PS; ++i) o[i] = row + i * RP < valid ? off : BUF_OUT;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const bf16_t *const b = base + (i % PS) * RP * ld + (i / PS) * 64;
      const uint32_t dst = lds + (i * 64 * RW + wave * 64) * 16;
      if constexpr (DIRECT) {
        load_to_lds(b, o[i % PS], dst);
      } else {
        u32x4_t v = {0u, 0u, 0u, 0u};
        if (o[i % PS] != BUF_OUT) v = *(gvec_ptr)((const char *)b + o[i % PS]);
        *(__attribute__((address_space(3))) u32x4_t *)(uintptr_t)(dst + (threadIdx.x & 63) * 16) = v;
      }
    }
  }
};
// a wavefront's operand fragments of such a tile
template <typename TILE, int TK>
struct RowFrag {
  int kc[4], t0[2], t1[2];
  __device__ __forceinline__ void init(int lane) {
    const int r = lane & 31, hi = lane >> 5;
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) kc[kk] = r * 64 + ((kk * 2 + hi) ^ TILE::swz(r)) * 8;
    const int G = lane >> 4, sl = lane & 15, k = 4 * hi + (sl >> 2);
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      const int m = q * 32 + 16 * (G & 1) + 4 * (sl & 3);
      t0[q] = k * 64 + ((m >> 3) ^ TILE::swz(k)) * 8 + ((m >> 2) & 1) * 4;
      t1[q] = (k + 8) * 64 + ((m >> 3) ^ TILE::swz(k + 8)) * 8 + ((m >> 2) & 1) * 4;
    }
  }
  // rows 32*nt .. +31, head dimensions 16*kk .. +15
  __device__ __forceinline__ bf16x8_t rows(const bf16_t *t, int nt, int kk) const {
    return *(const bf16x8_t *)(t + (kk >> 2) * TK * 64 + nt * 2048 + kc[kk & 3]);
  }
  // rows 16*kk .. +15 (in the order of row_operand) as contraction steps, head dimensions 32*nd .. +31
  __device__ __forceinline__ bf16x8_t tr(const bf16_t *t, int nd, int kk) const {
    const int c = (nd >> 1) * TK * 64 + kk * 1024;
    return fragment<1>(t, c + t0[nd & 1], c + t1[nd & 1]);
  }
};

// a lane's 32x32 result tile (row L%32) -> bf16 row segment at dst (already offset to the row and the tile)
__device__ __forceinline__ void store_tile_row(bf16_t *dst, int lane, const f32x16_t &a) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    u32x2_t w;
    w.x = pack_bf16(a[q * 4 + 0], a[q * 4 + 1]);
    w.y = pack_bf16(a[q * 4 + 2], a[q * 4 + 3]);
    *(u32x2_t *)(dst + q * 8 + (lane >> 5) * 4) = w;
  }
}

__device__ __forceinline__ void landed_barrier() {
  wait_loads_le<0>();  // this wavefront's tiles have landed and its LDS traffic is done
  block_barrier();
}
__device__ __forceinline__ uint32_t lds_addr(const void *p) {
  return __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void *)p);
}

// Block -> (sample and head, row block): all pairs' row blocks of one index before those of the next, the ones with the
// most tiles first (the longest ones would otherwise be started last and run alone).  Consecutive block ids go
// round-robin to the 8 XCDs, so with a multiple of 8 pairs a pair's keys and values stay in one XCD's L2.
// False for blocks that only fill up the last row of a two-dimensional grid (see HYDRA_ATTN).
__device__ __forceinline__ bool block_place(int pairs, int nb, int &z, int &rb) {
  const uint32_t id = blockIdx.y * gridDim.x + blockIdx.x;
  rb = id / (uint32_t)pairs;
  z = id - rb * (uint32_t)pairs;
  return rb < nb;
}

// ---------------------------------------------------------------------------
// forward: RW wavefronts = 32 RW query rows of one (sample, head); wavefront w owns
// rows r0 = q0 + 32 w .. + 31 and keeps its Q fragments in registers.  One
// sweep over the key tiles up to the diagonal with a running row maximum and
// sum (the output is rescaled when the maximum grows and divided by the sum at
// the end).  Tiles go straight from global memory to LDS, one ahead; one barrier
// per tile.  KW groups of RW wavefronts share the rows: group g takes key
// tiles g, g + KW, ... and the partial results are merged through LDS at the end
// (launches that would leave CUs without work; which form when: attn_forms.h).
// Bound: per 64 keys and wavefront 1024 clocks of MFMAs at head width 128 (512 at 64) and 960 of vector ALU, which overlap
// only between the wavefronts of a SIMD; counters at B 4, H 16, T 2048, dh 128: matrix pipes 0.44 busy, vector ALU 0.48,
// LDS 0.22 (with tiles of 64 keys and two blocks per CU 0.43, 0.41, 0.22).  That launch, in a row of such: 82 us with tiles
// of 64 keys, 79 with 32, whose LDS lets three blocks share a CU (165 registers; held to 128 for a fourth block it spills:
// 132 us).  Measured without gain: tiles two and three ahead, raised wavefront priority around the MFMAs, MFMAs and
// exponentials interleaved by scheduling directives (spills).
// ---------------------------------------------------------------------------
template <int DH, int RW, int KW, int TK, bool DIRECT>
__global__ __launch_bounds__(64 * RW * KW, 2) void attn_fwd_kernel(const bf16_t *__restrict__ qkv, bf16_t *__restrict__ o,
                                                               float *__restrict__ lse, int T, int H, int d, int nb, int pairs,
                                                               float scale_log2e) {
  constexpr int ND = DH / 32;  // 32-wide column tiles of the output
  typedef RowTile<DH, RW, TK> tile_t;
  constexpr int AQ = 32 * RW, NT = TK / 32;  // rows of the block, 32-row parts of a tile
  constexpr int TILE = tile_t::SIZE, STAGE = 2 * TILE * KW;
  constexpr int FOLLOW = 4;  // tiles of a group in which the reference maximum follows the maximum, see below
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];  // [2 stages][KW][K, V]
  const int tid = threadIdx.x % (64 * RW), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = KW > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / (64 * RW)) : 0;
  int z, qb;
  if (!block_place(pairs, nb, z, qb)) return;
  qb = nb - 1 - qb;
  const int b = z / H, h = z % H;
  const int q0 = qb * AQ, r0 = q0 + wave * 32;
  const int64_t ld = 3 * (int64_t)d;
  const bf16_t *qp = qkv + (int64_t)b * T * ld + h * DH, *kp = qp + d, *vp = qp + 2 * d;
  const int myrow = r0 + (lane & 31);
  const int ldrow = min(myrow, T - 1);  // rows past the sequence compute on a valid row and store nothing

  tile_t tile;
  tile.init(ld, tid);
  const uint32_t lds0 = lds_addr(smem) + grp * 2 * TILE * 2;
  const int kend = min(T, q0 + AQ);  // keys any row of the block can see
  const int nstep = (kend + TK * KW - 1) / (TK * KW);
  const int my_last = r0 + 31;       // tiles starting beyond it hold nothing for this wavefront
  auto load = [&](int it) {
    const int j0 = (it * KW + grp) * TK;
    const uint32_t s = lds0 + (it & 1) * STAGE * 2;
    tile.template load<DIRECT>(kp + (int64_t)j0 * ld, T - j0, s, wave);
    tile.template load<DIRECT>(vp + (int64_t)j0 * ld, T - j0, s + TILE * 2, wave);
  };
  load(0);
  bf16x8_t qf[DH / 16];
#pragma unroll
  for (int kk = 0; kk < DH / 16; ++kk) qf[kk] = load_frag_global(qp + ldrow * ld + kk * 16 + (lane >> 5) * 8);
  RowFrag<tile_t, TK> fr;
  fr.init(lane);

  // the reference maximum starts at the lowest finite value: a row whose scores of a tile are all -inf then adds
  // exp2(-inf) = 0, where -inf - -inf would be NaN
  float m = -FLT_MAX, l = 0.f, part = 0.f;
  f32x16_t acc[ND];
#pragma unroll
  for (int nd = 0; nd < ND; ++nd)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[nd][r] = 0.f;

  for (int it = 0; it < nstep; ++it) {
    landed_barrier();
    if (it + 1 < nstep) load(it + 1);
    const int j0 = (it * KW + grp) * TK;
    const bf16_t *const ks = smem + (it & 1) * STAGE + grp * 2 * TILE, *const vs = ks + TILE;
    if (j0 > my_last) continue;
    f32x16_t s[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
      for (int r = 0; r < 16; ++r) s[nt][r] = 0.f;
#pragma unroll
      for (int kk = 0; kk < DH / 16; ++kk)
        s[nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.rows(ks, nt, kk), qf[kk], s[nt], 0, 0, 0);
    }
    // Vector-ALU work per score is kept to a maximum, a fused multiply-add, an exponential, an add and half a
    // conversion: the scores stay unscaled (the scale is positive, so it commutes with the maximum and is folded into
    // the exponent's multiply-add), and the causal mask is applied only in tiles that reach above the wavefront's
    // first row.
    if (j0 + TK - 1 > r0) {
      const int over = j0 + (lane >> 5) * 4 - myrow;  // key - row of this lane's first column
#pragma unroll
      for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (over + nt * 32 + (r >> 2) * 8 + (r & 3) > 0) s[nt][r] = -INFINITY;
    }
    float tmax = s[0][0];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
      for (int r = 0; r < 16; ++r) tmax = __builtin_fmaxf(tmax, s[nt][r]);
    tmax = max_halves(tmax);
    // The reference maximum m of a row (log2 domain) only has to keep the exponentials in range, so it is moved -
    // and the sum and the output rescaled - only when some row's maximum has outgrown it by more than 2^8.  Except in
    // the first FOLLOW tiles: a weight equal to the reference is exactly 1, every other one carries a bf16 rounding, and
    // the heaviest weight of a row is the one whose rounding counts.  Error of o against 64 bits, B 4, H 16, T 2048, dh 128:
    // 1.009 times that of 64-key tiles with the first tile's maximum as reference, now 0.985 times; B 3, H 32, T 392 1.029
    // times that of two groups with such tiles, now 0.999; B 1, H 16, T 2048 (two groups) 1.006, now 0.982.  77.5 -> 79 us,
    // 16.1 -> 16.8 and no change.
    const float tm = tmax * scale_log2e, room = it < FOLLOW ? 0.f : 8.f;
    if (__builtin_amdgcn_ballot_w64(tm > m + room)) {
      const float mn = __builtin_fmaxf(m, tm);
      const float alpha = __builtin_amdgcn_exp2f(m - mn);
      m = mn;
      l *= alpha;
      part *= alpha;
#pragma unroll
      for (int nd = 0; nd < ND; ++nd)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[nd][r] *= alpha;
    }
    // of 64 keys, whatever the tile: half as many additions to l (error of lse 1.055 -> 0.96)
    float sum = NT == 1 ? part : 0.f;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      float p[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        p[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[nt][r], scale_log2e, -m));
        sum += p[r];
      }
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2) {
        const bf16x8_t pf = row_operand(p, k2);
#pragma unroll
        for (int nd = 0; nd < ND; ++nd)
          acc[nd] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.tr(vs, nd, nt * 2 + k2), pf, acc[nd], 0, 0, 0);
      }
    }
    if (NT > 1 || (it & 1)) {
      l += sum;
      part = 0.f;
    } else {
      part = sum;
    }
  }
  l = sum_halves(NT > 1 ? l : l + part);
#pragma unroll
  for (int n = KW / 2; n > 0; n /= 2) {
    // groups n .. 2n - 1 hand their maximum, sum and output to groups 0 .. n - 1; [group][value][wavefront][lane]
    constexpr int VALS = 2 + ND * 16;
    float *const x = (float *)smem + (grp % n) * VALS * 64 * RW + wave * 64 + lane;
    __syncthreads();
    if (grp >= n && grp < 2 * n) {
      x[0] = m;
      x[64 * RW] = l;
#pragma unroll
      for (int nd = 0; nd < ND; ++nd)
#pragma unroll
        for (int r = 0; r < 16; ++r) x[(2 + nd * 16 + r) * 64 * RW] = acc[nd][r];
    }
    __syncthreads();
    if (grp < n) {
      const float m1 = x[0], mn = __builtin_fmaxf(m, m1);
      const float a0 = __builtin_amdgcn_exp2f(m - mn), a1 = __builtin_amdgcn_exp2f(m1 - mn);
      m = mn;
      l = l * a0 + x[64 * RW] * a1;
#pragma unroll
      for (int nd = 0; nd < ND; ++nd)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[nd][r] = acc[nd][r] * a0 + x[(2 + nd * 16 + r) * 64 * RW] * a1;
    }
  }
  if (KW > 1 && grp > 0) return;
  const float inv_l = 1.f / l;
  if (myrow < T) {
    if (lane < 32) lse[(int64_t)z * T + myrow] = (m + log2f(l)) * LN2;
    bf16_t *op = o + ((int64_t)b * T + myrow) * d + h * DH;
#pragma unroll
    for (int nd = 0; nd < ND; ++nd) {
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[nd][r] *= inv_l;
      store_tile_row(op + nd * 32, lane, acc[nd]);
    }
  }
}

// adds what the groups of a block hold into group 0's accumulators, in pairs; false for the wavefronts of the other groups
template <int RW, int KW, int NA>
__device__ __forceinline__ bool merge_groups(f32x16_t (&acc)[NA], int grp, float *smem, int wave, int lane) {
#pragma unroll
  for (int n = KW / 2; n > 0; n /= 2) {
    float *const x = smem + (grp % n) * NA * 16 * 64 * RW + wave * 64 + lane;
    __syncthreads();
    if (grp >= n && grp < 2 * n) {
#pragma unroll
      for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) x[(i * 16 + r) * 64 * RW] = acc[i][r];
    }
    __syncthreads();
    if (grp < n) {
#pragma unroll
      for (int i = 0; i < NA; ++i)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[i][r] += x[(i * 16 + r) * 64 * RW];
    }
  }
  return grp == 0;
}

// ---------------------------------------------------------------------------
// backward, part 1: dQ.  Same decomposition as the forward kernel.  Per tile:
// p = exp(s - L), dP = dO V^T, dS = p (dP - D) / sqrt(dh) with
// D_i = sum_c dO[i,c] O[i,c] (OWN_D: summed here and written out), dQ += dS K.  B 4, H 16, T 2048, dh 128, launched alone: 117 us,
// whether with 64 or with 32 keys per tile (three blocks per CU would need 168 registers: 180 us with the spills); among
// other kernels 121 to 126.
// ---------------------------------------------------------------------------
template <int DH, int RW, int KW, int TK, bool DIRECT, bool OWN_D>
__device__ __forceinline__ void attn_bwd_dq(const bf16_t *__restrict__ qkv, const bf16_t *__restrict__ o, const bf16_t *__restrict__ d_o,
                                            const float *__restrict__ lse, float *__restrict__ dsum, bf16_t *__restrict__ dqkv, int T,
                                            int H, int d, const int z, const int qb, float scale) {
  constexpr int ND = DH / 32;
  typedef RowTile<DH, RW, TK> tile_t;
  constexpr int AQ = 32 * RW, NT = TK / 32;  // rows of the block, 32-row parts of a tile
  constexpr int TILE = tile_t::SIZE, STAGE = 2 * TILE * KW;
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];
  const int tid = threadIdx.x % (64 * RW), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = KW > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / (64 * RW)) : 0;
  const int b = z / H, h = z % H;
  const int q0 = qb * AQ, r0 = q0 + wave * 32;
  const int64_t ld = 3 * (int64_t)d;
  const bf16_t *qp = qkv + (int64_t)b * T * ld + h * DH, *kp = qp + d, *vp = qp + 2 * d;
  const int myrow = r0 + (lane & 31);
  const int ldrow = min(myrow, T - 1);

  tile_t tile;
  tile.init(ld, tid);
  const uint32_t lds0 = lds_addr(smem) + grp * 2 * TILE * 2;
  const int kend = min(T, q0 + AQ);
  const int nstep = (kend + TK * KW - 1) / (TK * KW);
  const int my_last = r0 + 31;
  auto load = [&](int it) {
    const int j0 = (it * KW + grp) * TK;
    const uint32_t s = lds0 + (it & 1) * STAGE * 2;
    tile.template load<DIRECT>(kp + (int64_t)j0 * ld, T - j0, s, wave);
    tile.template load<DIRECT>(vp + (int64_t)j0 * ld, T - j0, s + TILE * 2, wave);
  };
  load(0);
  bf16x8_t qf[DH / 16], dof[DH / 16];
  float dsum_part = 0.f;
  {
    const bf16_t *dop = d_o + ((int64_t)b * T + ldrow) * d + h * DH, *op = o + ((int64_t)b * T + ldrow) * d + h * DH;
#pragma unroll
    for (int kk = 0; kk < DH / 16; ++kk) {
      const int c = kk * 16 + (lane >> 5) * 8;
      qf[kk] = load_frag_global(qp + ldrow * ld + c);
      dof[kk] = load_frag_global(dop + c);
      if constexpr (OWN_D) {
        const bf16x8_t of = load_frag_global(op + c);
#pragma unroll
        for (int e = 0; e < 8; ++e) dsum_part += (float)dof[kk][e] * (float)of[e];
      }
    }
  }
  const float Di = OWN_D ? sum_halves(dsum_part) : dsum[(int64_t)z * T + ldrow];
  const float L2 = lse[(int64_t)z * T + ldrow] * LOG2E;
  if (OWN_D && grp == 0 && lane < 32 && myrow < T) dsum[(int64_t)z * T + myrow] = Di;
  const float scale_log2e = scale * LOG2E;
  const float nL2 = -L2, nDs = -Di * scale;
  RowFrag<tile_t, TK> fr;
  fr.init(lane);

  f32x16_t acc[ND];
#pragma unroll
  for (int nd = 0; nd < ND; ++nd)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[nd][r] = 0.f;

  for (int it = 0; it < nstep; ++it) {
    landed_barrier();
    if (it + 1 < nstep) load(it + 1);
    const int j0 = (it * KW + grp) * TK;
    const bf16_t *const ks = smem + (it & 1) * STAGE + grp * 2 * TILE, *const vs = ks + TILE;
    if (j0 > my_last) continue;
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) {
      f32x16_t s, dp;
#pragma unroll
      for (int r = 0; r < 16; ++r) s[r] = dp[r] = 0.f;
#pragma unroll
      for (int kk = 0; kk < DH / 16; ++kk) {
        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.rows(ks, nt, kk), qf[kk], s, 0, 0, 0);
        dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.rows(vs, nt, kk), dof[kk], dp, 0, 0, 0);
      }
      // as in the forward kernel the vector-ALU work per score is kept minimal: the mask only where the tile
      // reaches above the wavefront's first row (a masked score of -inf gives p = 0 exactly), the scale folded
      // into two fused multiply-adds
      if (j0 + nt * 32 + 31 > r0) {
        const int over = j0 + nt * 32 + (lane >> 5) * 4 - myrow;
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (over + (r >> 2) * 8 + (r & 3) > 0) s[r] = -INFINITY;
      }
      float ds[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], scale_log2e, nL2));
        ds[r] = p * __builtin_fmaf(dp[r], scale, nDs);
      }
#pragma unroll
      for (int k2 = 0; k2 < 2; ++k2) {
        const bf16x8_t df = row_operand(ds, k2);
#pragma unroll
        for (int nd = 0; nd < ND; ++nd)
          acc[nd] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.tr(ks, nd, nt * 2 + k2), df, acc[nd], 0, 0, 0);
      }
    }
  }
  if constexpr (KW > 1) {
    if (!merge_groups<RW, KW>(acc, grp, (float *)smem, wave, lane)) return;
  }
  if (myrow < T) {
    bf16_t *dq = dqkv + ((int64_t)b * T + myrow) * ld + h * DH;
#pragma unroll
    for (int nd = 0; nd < ND; ++nd) store_tile_row(dq + nd * 32, lane, acc[nd]);
  }
}

template <int DH, int RW, int KW, int TK, bool DIRECT>
__global__ __launch_bounds__(64 * RW * KW, 2) void attn_bwd_dq_kernel(const bf16_t *__restrict__ qkv, const bf16_t *__restrict__ o,
                                                                  const bf16_t *__restrict__ d_o, const float *__restrict__ lse,
                                                                  float *__restrict__ dsum, bf16_t *__restrict__ dqkv, int T,
                                                                  int H, int d, int nb, int pairs, float scale) {
  int z, qb;
  if (!block_place(pairs, nb, z, qb)) return;
  attn_bwd_dq<DH, RW, KW, TK, DIRECT, true>(qkv, o, d_o, lse, dsum, dqkv, T, H, d, z, nb - 1 - qb, scale);
}

// ---------------------------------------------------------------------------
// backward, part 2: dK and dV.  RW wavefronts = 32 RW keys of one (sample, head),
// wavefront w owns keys kr0 = k0 + 32 w .. + 31 and keeps their K and V
// fragments in registers.  It walks the query tiles from the diagonal
// to the end of the sequence, computing the transposed quantities directly:
// s^T = K Q^T, p^T = exp(s^T - L), dP^T = V dO^T, dS^T = p^T (dP^T - D)/sqrt(dh),
// dV += p^T dO, dK += dS^T Q.  No atomics: every key row has one owner.  At head width 128, launched alone, it is 157 us
// at B 4, H 16, T 2048 with two blocks per CU and tiles of 64 queries, 173 with 32; among other kernels 170 to 180.
// ---------------------------------------------------------------------------
template <int DH, int RW, int KW, int TK, bool DIRECT, bool OWN_D>
__device__ __forceinline__ void attn_bwd_dkv(const bf16_t *__restrict__ qkv, const bf16_t *__restrict__ o,
                                             const bf16_t *__restrict__ d_o, const float *__restrict__ lse,
                                             const float *__restrict__ dsum, bf16_t *__restrict__ dqkv, int T, int H, int d,
                                             const int z, const int kb, float scale) {
  constexpr int ND = DH / 32;
  typedef RowTile<DH, RW, TK> tile_t;
  constexpr int AQ = 32 * RW, NT = TK / 32;  // rows of the block, 32-row parts of a tile
  constexpr int TILE = tile_t::SIZE, STAGE = 2 * TILE * KW;
  extern __shared__ __attribute__((aligned(16))) bf16_t smem[];  // [2 stages][KW][Q, dO], then the statistics
  float *const Ls = (float *)(smem + 2 * STAGE);  // [2][KW][2 * TK]: -log-sum-exp (log2 domain) and -D / sqrt(dh) of a tile's queries
  const int tid = threadIdx.x % (64 * RW), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int grp = KW > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / (64 * RW)) : 0;
  const int b = z / H, h = z % H;
  const int k0 = kb * AQ, kr0 = k0 + wave * 32;
  const int64_t ld = 3 * (int64_t)d;
  const bf16_t *qp = qkv + (int64_t)b * T * ld + h * DH, *kp = qp + d, *vp = qp + 2 * d;
  const bf16_t *dop = d_o + (int64_t)b * T * d + h * DH, *op = o + (int64_t)b * T * d + h * DH;
  const int mykey = kr0 + (lane & 31);
  const int ldkey = min(mykey, T - 1);

  tile_t tq, to;
  tq.init(ld, tid);
  to.init(d, tid);
  const uint32_t lds0 = lds_addr(smem) + grp * 2 * TILE * 2;
  const int nstep = (T - k0 + TK * KW - 1) / (TK * KW);
  auto first = [&](int it) { return k0 + (it * KW + grp) * TK; };  // first query of this group's tile
  auto load = [&](int it) {
    const int i0 = first(it);
    const uint32_t s = lds0 + (it & 1) * STAGE * 2;
    tq.template load<DIRECT>(qp + (int64_t)i0 * ld, T - i0, s, wave);
    to.template load<DIRECT>(dop + (int64_t)i0 * d, T - i0, s + TILE * 2, wave);
  };
  // The statistics of a tile's queries.  OWN_D: D is summed here, by PR threads per query, from loads that fly while the tile
  // before is worked on; else the first 2 TK threads fetch what part 1 left.
  constexpr int PR = 64 * RW / TK, NV = DH / 8 / PR;  // threads per query, 16-byte loads of O and dO per thread
  static_assert(!OWN_D || (PR >= 2 && PR * TK == 64 * RW && NV * PR * 8 == DH), "every thread has a part of a query");
  struct Stat { float x; u32x4_t a[OWN_D ? NV : 1], b[OWN_D ? NV : 1]; };
  auto load_stat = [&](int i0, Stat &st) {
    if constexpr (OWN_D) {
      const int qi = i0 + tid / PR, part = tid % PR;
      const bool in = qi < T;
      const int64_t at = (int64_t)min(qi, T - 1) * d + part * 8;
      st.x = in && part == 0 ? -lse[(int64_t)z * T + qi] * LOG2E : 0.f;
#pragma unroll
      for (int v = 0; v < NV; ++v) {
        st.a[v] = *(gvec_ptr)(dop + at + v * PR * 8);
        st.b[v] = *(gvec_ptr)(op + at + v * PR * 8);
      }
    } else {
      const int qi = i0 + tid % TK;
      st.x = 0.f;
      if (tid >= 2 * TK || qi >= T) return;
      st.x = tid < TK ? -lse[(int64_t)z * T + qi] * LOG2E : -dsum[(int64_t)z * T + qi] * scale;
    }
  };
  // of the tile from query i0 on, to ls
  auto store_stat = [&](const Stat &st, int i0, float *ls) {
    if constexpr (OWN_D) {
      float s = 0.f;
#pragma unroll
      for (int v = 0; v < NV; ++v) s = dot8(st.a[v], st.b[v], s);
#pragma unroll
      for (int x = 1; x < PR; x *= 2) s += __shfl_xor(s, x);
      const int r = tid / PR, part = tid % PR;
      if (part < 2) ls[part * TK + r] = part ? (i0 + r < T ? -s * scale : 0.f) : st.x;
    } else {
      if (tid < 2 * TK) ls[tid] = st.x;
    }
  };
  load(0);
  Stat stat;
  load_stat(first(0), stat);
  bf16x8_t kf[DH / 16], vf[DH / 16];
#pragma unroll
  for (int kk = 0; kk < DH / 16; ++kk) {
    const int c = kk * 16 + (lane >> 5) * 8;
    kf[kk] = load_frag_global(kp + ldkey * ld + c);
    vf[kk] = load_frag_global(vp + ldkey * ld + c);
  }
  store_stat(stat, first(0), Ls + grp * 2 * TK);
  const float scale_log2e = scale * LOG2E;
  RowFrag<tile_t, TK> fr;
  fr.init(lane);

  f32x16_t acc[2 * ND];  // dK, dV
#pragma unroll
  for (int nd = 0; nd < 2 * ND; ++nd)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[nd][r] = 0.f;

  for (int it = 0; it < nstep; ++it) {
    landed_barrier();
    const bool more = it + 1 < nstep;
    if (more) {
      load_stat(first(it + 1), stat);
      load(it + 1);
    }
    const int i0 = first(it);
    const bf16_t *const qs = smem + (it & 1) * STAGE + grp * 2 * TILE, *const os = qs + TILE;
    const float *const ls = Ls + ((it & 1) * KW + grp) * 2 * TK;
    if (i0 + TK - 1 >= kr0 && i0 < T) {  // else no query of the tile comes after a key of this wavefront
      // one half tile at a time: unrolled, the two halves' results do not fit the 256 registers two wavefronts per SIMD
      // leave at head width 128 (the two backward kernels at B 4, H 16, T 2048, dh 128: 289 -> 270 us).  Even so one register
      // is spilled there where part 2 has a launch of its own (8 bytes of scratch per lane; two off the 16-byte grid); for one
      // launch of both parts see attn_bwd_kernel
#pragma unroll 1
      for (int nt = 0; nt < NT; ++nt) {
        f32x16_t s, dp;
#pragma unroll
        for (int r = 0; r < 16; ++r) s[r] = dp[r] = 0.f;
#pragma unroll
        for (int kk = 0; kk < DH / 16; ++kk) {
          s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.rows(qs, nt, kk), kf[kk], s, 0, 0, 0);
          dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.rows(os, nt, kk), vf[kk], dp, 0, 0, 0);
        }
        // The mask is needed only where the tile holds queries that precede keys of this wavefront; queries past the
        // end of the sequence need none (their Q and dO rows are zero-filled and their statistics zero, so they
        // contribute exact zeros).
        if (i0 + nt * 32 < kr0 + 31) {
          const int under = mykey - (i0 + nt * 32 + (lane >> 5) * 4);  // key - query of this lane's first column
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if (under - ((r >> 2) * 8 + (r & 3)) > 0) s[r] = -INFINITY;
        }
        float p[16], ds[16];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const int qc = nt * 32 + q * 8 + (lane >> 5) * 4;  // first of this lane's four queries within the tile
          const f32x4_t nl = *(const f32x4_t *)(ls + qc), nd4 = *(const f32x4_t *)(ls + TK + qc);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int r = q * 4 + e;
            p[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], scale_log2e, nl[e]));
            ds[r] = p[r] * __builtin_fmaf(dp[r], scale, nd4[e]);
          }
        }
#pragma unroll
        for (int k2 = 0; k2 < 2; ++k2) {
          const bf16x8_t pf = row_operand(p, k2), df = row_operand(ds, k2);
#pragma unroll
          for (int nd = 0; nd < ND; ++nd)
            acc[ND + nd] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.tr(os, nd, nt * 2 + k2), pf, acc[ND + nd], 0, 0, 0);
#pragma unroll
          for (int nd = 0; nd < ND; ++nd) {
            acc[nd] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr.tr(qs, nd, nt * 2 + k2), df, acc[nd], 0, 0, 0);
          }
        }
      }
    }
    if (more) store_stat(stat, first(it + 1), Ls + (((it + 1) & 1) * KW + grp) * 2 * TK);
  }
  if constexpr (KW > 1) {
    if (!merge_groups<RW, KW>(acc, grp, (float *)smem, wave, lane)) return;
  }
  if (mykey < T) {
    bf16_t *dkp = dqkv + ((int64_t)b * T + mykey) * ld + d + h * DH, *dvp = dkp + d;
#pragma unroll
    for (int nd = 0; nd < ND; ++nd) {
      store_tile_row(dkp + nd * 32, lane, acc[nd]);
      store_tile_row(dvp + nd * 32, lane, acc[ND + nd]);
    }
  }
}

template <int DH, int RW, int KW, int TK, bool DIRECT>
__global__ __launch_bounds__(64 * RW * KW, DH == 64 ? 3 : 2) void attn_bwd_dkv_kernel(const bf16_t *__restrict__ qkv,
                                                                   const bf16_t *__restrict__ d_o,
                                                                   const float *__restrict__ lse,
                                                                   const float *__restrict__ dsum, bf16_t *__restrict__ dqkv,
                                                                   int T, int H, int d, int nb, int pairs, float scale) {
  int z, kb;
  if (!block_place(pairs, nb, z, kb)) return;
  attn_bwd_dkv<DH, RW, KW, TK, DIRECT, false>(qkv, nullptr, d_o, lse, dsum, dqkv, T, H, d, z, kb, scale);
}

// D alone, where part 2 does not sum it: 16 bytes of dO and O per lane, samples blockIdx.y, + gridDim.y, ...  Bound: HBM, and a
// launch (us, traced: 13 for the 52 MB of B 8, H 25, T 512, dh 128 or T 1024, dh 64; 5.3 for 6 MB).
template <int DH>
__global__ __launch_bounds__(256) void attn_dsum_kernel(const bf16_t *__restrict__ o, const bf16_t *__restrict__ d_o,
                                                        float *__restrict__ dsum, int B, int T, int H) {
  constexpr uint32_t L = DH / 8;  // lanes per row
  const uint32_t i = blockIdx.x * 256 + threadIdx.x, row = i / L, t = row / (uint32_t)H, h = row - t * H;
  if (t >= (uint32_t)T) return;  // whole rows of lanes
  for (int b = blockIdx.y; b < B; b += gridDim.y) {
    const int64_t at = ((int64_t)b * T * H * L + i) * 8;
    float s = dot8(*(gvec_ptr)(d_o + at), *(gvec_ptr)(o + at), 0.f);
#pragma unroll
    for (int n = 1; n < (int)L; n *= 2) s += __shfl_xor(s, n);
    if (i % L == 0) dsum[((int64_t)b * H + h) * T + t] = s;
  }
}

// ---------------------------------------------------------------------------
// backward, both parts in one launch: 2 * pairs blocks per row block, those of part 2, which take longer, first; MIXED: see
// attn_bwd_place.  Bound: at a few hundred row blocks the chain of tiles of a block, 0.6 to 0.9 us per 64 rows, which the other
// part's blocks now share the CUs with; at thousands the matrix pipes, as for the parts alone, less the tails of two launches, until
// both parts' tensors no longer fit the caches together (attn_bwd_mode).  us, two launches / one: B 4, H 12, T 512, dh 64 23.4 /
// 18.7, B 1, H 12, T 512 19.7 / 13.2, B 8, H 25, T 1024 143 / 133, dh 128 B 1, H 16, T 512 35 / 24; mixed H 16, T 3792, dh 64
// 142 / 131 (151 in the other order).
// At head width 64 three blocks share a CU (168 registers; off the 16-byte grid one form spills 4) unless they sum D (213 to 249
// registers: two); at 128 two, with 2 to 10 registers spilled, 41 where they sum D.  (Another spelling of the loop's last statement,
// with 4 instead of 10 spilled, made the two-group form 3 to 8 % slower.)
// ---------------------------------------------------------------------------
template <int DH, int RW, int KW, int TK, bool DIRECT, bool OWN_D, int OCC, bool MIXED>
__global__ __launch_bounds__(64 * RW * KW, OCC) void attn_bwd_kernel(const bf16_t *__restrict__ qkv, const bf16_t *__restrict__ o,
                                                               const bf16_t *__restrict__ d_o, const float *__restrict__ lse,
                                                               float *__restrict__ dsum, bf16_t *__restrict__ dqkv, int T, int H,
                                                               int d, int nb, int pairs, float scale) {
  if constexpr (MIXED) {
    const AttnBwdPlace at = attn_bwd_place(blockIdx.y * gridDim.x + blockIdx.x, pairs);
    if (at.rb >= nb) return;
    if (at.dq) attn_bwd_dq<DH, RW, KW, TK, DIRECT, OWN_D>(qkv, o, d_o, lse, dsum, dqkv, T, H, d, at.z, nb - 1 - at.rb, scale);
    else attn_bwd_dkv<DH, RW, KW, TK, DIRECT, OWN_D>(qkv, o, d_o, lse, dsum, dqkv, T, H, d, at.z, at.rb, scale);
    return;
  }
  int z, rb;
  if (!block_place(2 * pairs, nb, z, rb)) return;
  if (z < pairs) attn_bwd_dkv<DH, RW, KW, TK, DIRECT, OWN_D>(qkv, o, d_o, lse, dsum, dqkv, T, H, d, z, rb, scale);
  else attn_bwd_dq<DH, RW, KW, TK, DIRECT, OWN_D>(qkv, o, d_o, lse, dsum, dqkv, T, H, d, z - pairs, nb - 1 - rb, scale);
}

}  // namespace

bool attention_fused_supported(int dtype, int dh) { return dtype == DT_BF16 && (dh == 64 || dh == 128); }

// bytes of LDS: two stages of two tiles per group, and room for the merge of the groups (nacc 32-column accumulators
// and `extra` values per row)
static constexpr size_t attn_lds(int dh, int rw, int kw, int tk, int nacc, int extra, size_t stats) {
  const size_t tiles = (size_t)2 * kw * 2 * tk * dh * 2 + stats, merge = (size_t)(kw / 2) * (nacc * 16 + extra) * 64 * rw * 4;
  return tiles > merge ? tiles : merge;
}

// (a row of the grid holds at most 2^32 threads)
#define HYDRA_ATTN(KERN_, BLOCKS_, LDS_, ...)                                      \
  do {                                                                             \
    auto kern = KERN_;                                                             \
    static OncePerGpu once;                                                        \
    const hipError_t attr = allow_lds(once, (const void *)kern, LDS_);             \
    if (attr != hipSuccess) return attr;                                           \
    const uint32_t blocks = BLOCKS_, gx = blocks < (1u << 22) ? blocks : 1u << 22; \
    hipLaunchKernelGGL(kern, dim3(gx, (blocks + gx - 1) / gx), dim3(64 * RW * KW), LDS_, s, __VA_ARGS__); \
  } while (0)

template <int DH, int RW, int KW, int TK, bool DIRECT>
static hipError_t attn_fwd(const bf16_t *qkv, bf16_t *o, float *lse, int B, int H, int T, hipStream_t s) {
  const int nb = (T + 32 * RW - 1) / (32 * RW), d = H * DH;
  HYDRA_ATTN((attn_fwd_kernel<DH, RW, KW, TK, DIRECT>), (uint32_t)nb * B * H, attn_lds(DH, RW, KW, TK, DH / 32, 2, 0), qkv, o, lse, T, H, d, nb, B * H,
             LOG2E / sqrtf((float)DH));
  return hipGetLastError();
}

template <int DH, int RW, int KW, int TK, int MODE, bool DIRECT>
static hipError_t attn_bwd(const bf16_t *qkv, const bf16_t *o, const bf16_t *d_o, const float *lse, float *dsum, bf16_t *dqkv,
                           int B, int H, int T, hipStream_t s) {
  const int nb = (T + 32 * RW - 1) / (32 * RW), d = H * DH;
  const float scale = 1.0f / sqrtf((float)DH);
  constexpr size_t lds_dkv = attn_lds(DH, RW, KW, TK, DH / 16, 0, KW * 2 * 2 * TK * 4);
  const uint32_t blocks1 = (uint32_t)nb * B * H;  // of one part
  if constexpr (MODE != BWD_TWO) {  // see attn_bwd_mode
    constexpr bool OWN_D = MODE == BWD_ONE || MODE == BWD_MIXED, MIXED = MODE == BWD_MIXED || MODE == BWD_MIXED_AFTER_D;
    if constexpr (!OWN_D) {
      const uint32_t lanes = (uint32_t)T * H * (DH / 8);  // of a sample
      hipLaunchKernelGGL((attn_dsum_kernel<DH>), dim3((lanes + 255) / 256, B < 32768 ? B : 32768), dim3(256), 0, s, o, d_o, dsum, B, T, H);
    }
    HYDRA_ATTN((attn_bwd_kernel<DH, RW, KW, TK, DIRECT, OWN_D, OWN_D || DH == 128 ? 2 : 3, MIXED>), MIXED ? attn_bwd_grid(blocks1) : 2 * blocks1,
               lds_dkv, qkv, o, d_o, lse, dsum, dqkv, T, H, d, nb, B * H, scale);
  } else {
    HYDRA_ATTN((attn_bwd_dq_kernel<DH, RW, KW, TK, DIRECT>), blocks1, attn_lds(DH, RW, KW, TK, DH / 32, 0, 0), qkv, o, d_o, lse, dsum,
               dqkv, T, H, d, nb, B * H, scale);
    HYDRA_ATTN((attn_bwd_dkv_kernel<DH, RW, KW, TK, DIRECT>), blocks1, lds_dkv, qkv, d_o, lse, dsum, dqkv, T, H, d, nb, B * H, scale);
  }
  return hipGetLastError();
}
#undef HYDRA_ATTN

// One launch of form F of a table (attn_forms.h).  Tensors off the 16-byte grid (qkv or d_o; heads and rows are multiples of
// it) move their tiles through registers.
template <int DH, int F, bool DIRECT>
static hipError_t attn_fwd_form(const bf16_t *qkv, bf16_t *o, float *lse, int B, int H, int T, hipStream_t s) {
  constexpr AttnForm f = DH == 64 ? attn_forms_fwd64[F] : attn_forms_fwd128[F < 3 ? F : 0];
  return attn_fwd<DH, f.rw, f.kw, f.tk, DIRECT>(qkv, o, lse, B, H, T, s);
}
template <int DH, int F, bool DIRECT>
static hipError_t attn_bwd_form(const bf16_t *qkv, const bf16_t *o, const bf16_t *d_o, const float *lse, float *dsum, bf16_t *dqkv,
                                int B, int H, int T, hipStream_t s) {
  constexpr AttnForm f = DH == 64 ? attn_forms_bwd64[F] : attn_forms_bwd128[F < 3 ? F : 0];
  const AttnBwdMode mode = attn_bwd_mode(DH, F, B * H, T);
#define HYDRA_MODE(M_) \
  if (mode == M_) return attn_bwd<DH, f.rw, f.kw, f.tk, M_, DIRECT>(qkv, o, d_o, lse, dsum, dqkv, B, H, T, s)
  if constexpr (DH == 64 || F == 1) HYDRA_MODE(BWD_ONE);
  if constexpr (DH == 128 || F == 0 || F == 2) HYDRA_MODE(BWD_ONE_AFTER_D);
  if constexpr (DH == 64 && (F == 0 || F == 2)) HYDRA_MODE(BWD_MIXED);
  if constexpr (F < 3) HYDRA_MODE(BWD_MIXED_AFTER_D);
  if constexpr (F < 2) HYDRA_MODE(BWD_TWO);
#undef HYDRA_MODE
  return hipErrorInvalidValue;
}
#define HYDRA_ATTN_FORM(FN_, DH_, F_, ...) \
  return direct ? FN_<DH_, F_, true>(__VA_ARGS__) : FN_<DH_, F_, false>(__VA_ARGS__)
#define HYDRA_ATTN_FORMS3(FN_, DH_, ...)                  \
  case 0: HYDRA_ATTN_FORM(FN_, DH_, 0, __VA_ARGS__);      \
  case 1: HYDRA_ATTN_FORM(FN_, DH_, 1, __VA_ARGS__);      \
  case 2: HYDRA_ATTN_FORM(FN_, DH_, 2, __VA_ARGS__)

hipError_t launch_attention_fwd(const void *qkv, void *o, float *lse, int B, int H, int T, int dh, hipStream_t s) {
  if (!attention_fused_supported(DT_BF16, dh)) return hipErrorInvalidValue;
  // causal half of both products
  ProfScope ps("attention_fwd", s, 2.0 * B * H * dh * ((double)T * (T + 1.0)), 0);
  const bool direct = ((uintptr_t)qkv & 15) == 0;
  const int form = attn_form_fwd(dh, B * H, T);
#define HYDRA_ARGS (const bf16_t *)qkv, (bf16_t *)o, lse, B, H, T, s
  if (dh == 128) {
    switch (form) { HYDRA_ATTN_FORMS3(attn_fwd_form, 128, HYDRA_ARGS); }
  } else {
    switch (form) {
      HYDRA_ATTN_FORMS3(attn_fwd_form, 64, HYDRA_ARGS);
      case 3: HYDRA_ATTN_FORM(attn_fwd_form, 64, 3, HYDRA_ARGS);
      case 4: HYDRA_ATTN_FORM(attn_fwd_form, 64, 4, HYDRA_ARGS);
    }
  }
#undef HYDRA_ARGS
  return hipErrorInvalidValue;
}

hipError_t launch_attention_bwd(const void *qkv, const void *o, const void *d_o, const float *lse, float *dsum,
                                void *dqkv, int B, int H, int T, int dh, hipStream_t s) {
  if (!attention_fused_supported(DT_BF16, dh)) return hipErrorInvalidValue;
  // five causal products of T x T x dh each (s and dP in both kernels count once: the recomputation is overhead)
  ProfScope ps("attention_bwd", s, 5.0 * B * H * dh * ((double)T * (T + 1.0)), 0);
  const bool direct = (((uintptr_t)qkv | (uintptr_t)d_o) & 15) == 0;
  const int form = attn_form_bwd(dh, B * H, T);
#define HYDRA_ARGS (const bf16_t *)qkv, (const bf16_t *)o, (const bf16_t *)d_o, lse, dsum, (bf16_t *)dqkv, B, H, T, s
  if (dh == 128) {
    switch (form) { HYDRA_ATTN_FORMS3(attn_bwd_form, 128, HYDRA_ARGS); }
  } else {
    switch (form) {
      HYDRA_ATTN_FORMS3(attn_bwd_form, 64, HYDRA_ARGS);
      case 3: HYDRA_ATTN_FORM(attn_bwd_form, 64, 3, HYDRA_ARGS);
    }
  }
#undef HYDRA_ARGS
  return hipErrorInvalidValue;
}
#undef HYDRA_ATTN_FORMS3
#undef HYDRA_ATTN_FORM

}  // namespace hydra
