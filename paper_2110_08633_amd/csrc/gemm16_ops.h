// Shared by the bf16 kernels for single products (v_mfma_f32_16x16x32_bf16, operand slices straight to LDS): tile numbering,
// the global -> LDS mover of one operand and the fragment reads.
#pragma once
#include "gemm_common.h"

namespace hydra {

// first row and column of the tile of workgroup bid of nt: contiguous runs of tiles per XCD, see xcd_group_rows.  HALVES: every
// tile has two workgroups, one per half of the contraction, numbered so that all but one XCD, at most, work on one half; the half is returned
template <int BM, int BN, bool HALVES = false>
__device__ __forceinline__ int tile_origin(const GemmArgs &g, int bid, int nt, int &m0, int &n0) {
  const int xcd = bid & 7, per = nt >> 3, rem = nt & 7;
  int tile = xcd * per + min(xcd, rem) + (bid >> 3);
  int half = 0;
  if (HALVES && tile >= nt / 2) {
    half = 1;
    tile -= nt / 2;
  }
  const int gsz = g.grp * g.tiles_n;
  const int grp = tile / gsz, in_grp = tile - grp * gsz;
  const int rows_in_grp = min(g.grp, g.tiles_m - grp * g.grp);
  m0 = (grp * g.grp + in_grp % rows_in_grp) * BM;
  n0 = (in_grp / rows_in_grp) * BN;
  return half;
}

// 16-byte chunk position within a line of LDS.  [row][BK]: 16 rows at one chunk index should fall into distinct slots
// of the 256-byte bank period (at BK 128, lines of 256 bytes, they fall into 8).  [k][R]: a read takes two neighbouring
// chunks of lines k..k+3 and k+8..k+11.
template <int BK_> __device__ __forceinline__ int swz_kc(int row) { return (BK_ >= 128 ? row : row >> 1) & (BK_ >= 64 ? 7 : 3); }
template <int R> __device__ __forceinline__ int swz_rc(int k) {
  // lines too short or too odd to swizzle: conflicts are a third of the LDS cycles, 2 to 4 % of the kernel's (counted for the
  // 48x32 and 16x16 tiles of gemm_split.hip)
  if (R % 32) return 0;
  const int hi = ((k >> 3) & 1) << 1;
  if (R % 128 == 0) return ((k & 3) << 2) ^ hi;                     // lines a multiple of 256 bytes
  if (R % 64 == 0) return (R / 64) % 2 ? (((k >> 1) & 1) << 2) ^ hi : 0;  // odd multiples of 128 bytes
  return hi;                                                         // odd multiples of 64 bytes (R = 96)
}

template <int R, int RCL, int BK_, int NW>
struct LdsMover {
  static constexpr int CPL = (RCL ? R : BK_) / 8;        // chunks per line
  static constexpr int NCH = R * BK_ / 8;                // chunks per slice
  static constexpr int N = NCH / (64 * NW);              // loads per wavefront
  static_assert(NCH == N * 64 * NW, "every wavefront loads alike");
  const bf16_t *base;
  int64_t kstep;   // elements per slice
  int off[N];      // byte offset within a slice, BUF_OUT for rows past the matrix
  int kloc[N];     // first contraction step of the chunk
  __device__ __forceinline__ void init(const bf16_t *mat, int64_t ld, int row0, int rows, int tid) {
    const int lane = tid & 63, wave = tid >> 6;
    base = RCL ? mat + row0 : mat + (int64_t)row0 * ld;
    kstep = RCL ? (int64_t)BK_ * ld : BK_;
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const int p = (i * NW + wave) * 64 + lane, line = p / CPL, pos = p % CPL;
      if (!RCL) {
        const int kc = pos ^ swz_kc<BK_>(line);
        off[i] = row0 + line < rows ? (int)((line * ld + kc * 8) * 2) : BUF_OUT;
        kloc[i] = kc * 8;
      } else {
        const int c = pos ^ swz_rc<R>(line);
        off[i] = row0 + c * 8 < rows ? (int)((line * ld + c * 8) * 2) : BUF_OUT;
        kloc[i] = line;
      }
    }
  }
  // chunk i of slice t into the operand's tile at lds; krem: contraction steps left from the start of the slice
  __device__ __forceinline__ void issue(int i, int t, int krem, uint32_t lds, int wave) const {
    load_to_lds(base + t * kstep, kloc[i] < krem ? off[i] : BUF_OUT, lds + (i * NW + wave) * 64 * 16);
  }
};

// LDS addresses of a wavefront's fragments for v_mfma_f32_16x16x32_bf16: NF groups of 16 rows from row rb on; lane L
// holds row L%16, contraction steps (L/16)*8 .. +7 of a step of 32
template <int R, int RCL, int NF, int BK_, int KS>
struct Frag16 {
  static constexpr int CPL = (RCL ? R : BK_) / 8;
  static constexpr int NO = RCL ? NF : KS;
  int o[NO];
  // KS steps of 32 from step k0 of the slice on
  __device__ __forceinline__ void init(int rb, int lane, int k0) {
    const int G = lane >> 4, sl = lane & 15;
    if (!RCL) {
      const int row = rb + sl;
#pragma unroll
      for (int kk = 0; kk < NO; ++kk) o[kk] = (row * CPL + (((k0 + kk) * 4 + G) ^ swz_kc<BK_>(row))) * 8;
    } else {
      const int k = k0 * 32 + G * 8 + (sl >> 2);
#pragma unroll
      for (int f = 0; f < NO; ++f) {
        const int m = rb + f * 16 + 4 * (sl & 3);
        o[f] = (k * CPL + ((m >> 3) ^ swz_rc<R>(k))) * 8 + ((m >> 2) & 1) * 4;
      }
    }
  }
  __device__ __forceinline__ bf16x8_t get(const bf16_t *lds, int f, int kk) const {
    if (!RCL) return fragment<0>(lds, o[kk] + f * 16 * CPL * 8, 0);  // 16 further rows leave the swizzle unchanged
    const int b = o[f] + kk * 32 * CPL * 8;                          // and so do 32 further contraction steps, or 4
    return fragment<1>(lds, b, b + 4 * CPL * 8);
  }
};

}  // namespace hydra
