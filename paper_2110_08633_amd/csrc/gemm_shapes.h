// Choice of the tile shape of a bf16 product (host only, no HIP).
#pragma once
#include <stdint.h>

#include <cmath>

namespace hydra {

struct GemmDims {
  int M, N, K;
  bool ta, tb;    // operand stored with the contraction index strided
  bool vec_rows;  // leading dimension of the result is a multiple of 4
};

// The tile shapes, and what a launch of each costs in us:
//   t0 + rounds * (nk * a + c) + tiles / 256 * (nk * b + e)
// with nk = contraction / 64 (rounded up) and rounds = tiles / 256 rounded up: the tiles of the busiest CU one after the
// other, plus what all of them take from the caches and from memory together.  With transposing LDS reads of both a block of four
// wavefronts alone leaves its CU half idle, so there a round is as many tiles as the CUs hold blocks.  The constants are
// least-squares fits (weighted towards the products for which a shape is among the fastest) to 200 products of the four
// models' widths at 201 to 4096 tokens, LM heads included: one set for operands that are both contraction-contiguous and
// one for products that read both through the transposing LDS read; products with one of each take the middle.
struct PlainShape {
  int bm, bn, occ, threads;  // tile, blocks per CU, threads per block
  float t0[2], a[2], b[2], c[2], e[2];
};
constexpr PlainShape plain_shapes[] = {
    {256, 256, 1, 512, {0.f, 0.f}, {0.830f, 1.272f}, {0.538f, 0.538f}, {7.196f, 7.679f}, {5.990f, 5.423f}},
    {128, 256, 1, 512, {0.700f, 2.841f}, {0.542f, 0.588f}, {0.215f, 0.251f}, {4.376f, 2.872f}, {3.607f, 3.663f}},
    {128, 192, 1, 512, {0.698f, 4.614f}, {0.470f, 0.506f}, {0.150f, 0.154f}, {3.797f, 0.f}, {2.403f, 4.969f}},
    {128, 128, 1, 512, {1.171f, 2.835f}, {0.323f, 0.332f}, {0.137f, 0.171f}, {3.051f, 1.382f}, {0.878f, 2.316f}},
    {128, 64, 2, 256, {3.621f, 3.814f}, {0.258f, 0.307f}, {0.025f, 0.135f}, {0.f, 0.f}, {0.751f, 1.514f}},
    {64, 96, 2, 256, {3.906f, 3.841f}, {0.231f, 0.272f}, {0.012f, 0.112f}, {0.f, 0.f}, {0.578f, 1.421f}},
    {64, 64, 3, 256, {3.788f, 3.715f}, {0.193f, 0.124f}, {0.f, 0.147f}, {0.f, 0.f}, {0.500f, 0.668f}},
    {64, 64, 1, 512, {1.535f, 1.619f}, {0.147f, 0.166f}, {0.027f, 0.f}, {2.522f, 2.463f}, {0.088f, 0.294f}},  // slices split over two groups of wavefronts
    {128, 64, 1, 512, {1.761f, 2.516f}, {0.215f, 0.222f}, {0.071f, 0.075f}, {3.127f, 2.300f}, {0.f, 0.936f}},  // the same
    {64, 96, 1, 512, {2.014f, 2.093f}, {0.186f, 0.186f}, {0.043f, 0.075f}, {2.271f, 2.622f}, {0.677f, 0.415f}},  // the same
    {128, 128, 2, 256, {0.f, 3.209f}, {0.f, 0.432f}, {0.f, 0.223f}, {0.f, 0.879f}, {0.f, 2.244f}},  // two blocks of four wavefronts: see best_shape
    {128, 256, 2, 256, {0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}, {0.f, 0.f}},  // the same, large_tn only
};
constexpr int N_SHAPES = sizeof(plain_shapes) / sizeof(plain_shapes[0]);

inline float shape_cost(const PlainShape &p, const GemmDims *d, int n) {
  // one transposed operand: half way between the two
  const float x = d->ta == d->tb ? (float)d->ta : 0.5f;
  auto at = [x](const float (&v)[2]) { return v[0] + x * (v[1] - v[0]); };
  float tiles = 0.f;
  int K = 0;
  for (int i = 0; i < n; ++i) {
    tiles += (float)((d[i].M + p.bm - 1) / p.bm) * (float)((d[i].N + p.bn - 1) / p.bn);
    K = d[i].K > K ? d[i].K : K;
  }
  const float nk = (float)((K + 63) / 64), u = tiles * (1.f / 256.f);
  const float rounds = ceilf(x == 1.f ? u / (float)p.occ : u);
  return at(p.t0) + rounds * (nk * at(p.a) + at(p.c)) + u * (nk * at(p.b) + at(p.e));
}

// a launch of this shape stays below the 2^32 threads of a grid (small tiles have the least estimated cost per result at
// short contractions, and with them a result of some 7e10 elements would not)
inline bool shape_fits(const PlainShape &p, const GemmDims *d, int n) {
  uint64_t tiles = 0;
  for (int i = 0; i < n; ++i) tiles += ((uint64_t)d[i].M + p.bm - 1) / p.bm * (((uint64_t)d[i].N + p.bn - 1) / p.bn);
  return tiles * p.threads < (uint64_t)1 << 32;
}

// Large products whose operands are both read through the transposing LDS read (weight gradients of wide layers, an LM
// head's): what they wait for is the write-out of a tile that nothing overlaps, and operands.  With slices of 32 steps - whole
// lines of such an operand all the same - 256x256 tiles fit the registers (with 64 they spill) and four slices fit the LDS; and
// two blocks of four wavefronts with 128x256 tiles fit a CU, one writing out while the other multiplies.  Constants as above
// (rounds of twice 256 tiles where two blocks share a CU), fitted to 1340 products and groups of random layers launched one
// after another with operands that are not in the L2s.
struct LargeShape {
  int shape;  // of plain_shapes
  float t0, a, b, c, e;
  float f;  // us per MB of fp32 results beyond the 220 that stay in the 256 MB cache
};
constexpr int SHAPE_256X256 = 0, SHAPE_64X64K2 = 7, SHAPE_128X256X2 = N_SHAPES - 1;
constexpr LargeShape tn_shapes[] = {{SHAPE_256X256, 4.386f, 0.934f, 0.622f, 9.367f, 0.776f, 0.063f},
                                 {1, 3.069f, 0.546f, 0.341f, 5.485f, 1.107f, 0.051f},
                                 {2, 3.256f, 0.308f, 0.429f, 5.147f, 0.f, 0.031f},
                                 {10, 4.982f, 0.484f, 0.239f, 2.171f, 1.423f, 0.114f},
                                 {SHAPE_128X256X2, 11.030f, 0.603f, 0.561f, 0.668f, 2.700f, 0.159f}};
static_assert(plain_shapes[SHAPE_128X256X2].bn == 256 && plain_shapes[SHAPE_64X64K2].bm == 64 && plain_shapes[SHAPE_64X64K2].threads == 512, "");

// at least 128 tiles of 256x256 with nothing narrow, and enough steps for the rounds to count
inline bool large_tn(const GemmDims *d, int n) {
  int64_t tiles = 0;
  for (int i = 0; i < n; ++i) {
    if (!d[i].ta || !d[i].tb || d[i].M < 512 || d[i].N < 512 || d[i].K < 256) return false;
    tiles += ((int64_t)d[i].M + 255) / 256 * (((int64_t)d[i].N + 255) / 256);
  }
  return tiles >= 128;
}
// Large products whose operands are both contraction-contiguous (forward, input gradients).  At short contractions the estimate
// for all products misses what thousands of small tiles read again and write, and takes 128x64 where 256x256 are up to 1.8 times
// as fast.  Constants as above, f = 0: fits to 539 products with more than 256 tiles of 256x256 (contractions of 128 to 6000
// steps, results of up to 200 million, fp32 and bf16), operands not in the L2s.
constexpr LargeShape nt_shapes[] = {{SHAPE_256X256, 8.001f, 1.171f, 0.524f, 2.448f, 9.053f, 0.f},
                                    {1, 7.700f, 0.458f, 0.617f, 1.009f, 4.738f, 0.f},
                                    {2, 5.271f, 0.297f, 0.586f, 1.018f, 3.906f, 0.f},
                                    {3, 2.967f, 0.492f, 0.149f, 0.f, 3.591f, 0.f},
                                    {4, 5.219f, 0.298f, 0.204f, 0.f, 1.374f, 0.f}};

// more than one round of 256x256 tiles (with 192 to 256 of them the choice gave 1 % and 21 of 248 were more than 3 % slower),
// contractions and results of the fitted sizes stored by vectors as theirs, and a second operand of more than 6 MB: a smaller one
// stays in an XCD's L2, and small tiles may read it again (16280x7280x256, 3.7 MB, 128x64 153 us, 256x256 177)
inline bool large_nt(const GemmDims *d, int n) {
  int64_t tiles = 0;
  for (int i = 0; i < n; ++i) {
    if (d[i].ta || d[i].tb || d[i].K < 128 || d[i].K > 6000 || !d[i].vec_rows || d[i].M < 256 ||
        (int64_t)d[i].M * d[i].N > 200000000 || (int64_t)d[i].N * d[i].K <= 3 << 20) return false;
    tiles += ((int64_t)d[i].M + 255) / 256 * (((int64_t)d[i].N + 255) / 256);
  }
  return tiles > 256;
}
inline float large_cost(const LargeShape &t, const GemmDims *d, int n) {
  const PlainShape &p = plain_shapes[t.shape];
  float tiles = 0.f, mb = 0.f;
  int K = 0;
  for (int i = 0; i < n; ++i) {
    tiles += (float)((d[i].M + p.bm - 1) / p.bm) * (float)((d[i].N + p.bn - 1) / p.bn);
    mb += (float)d[i].M * (float)d[i].N * 4e-6f;
    K = d[i].K > K ? d[i].K : K;
  }
  const float nk = (float)((K + 63) / 64), u = tiles * (1.f / 256.f);
  return t.t0 + ceilf(u / (float)p.occ) * (nk * t.a + t.c) + u * (nk * t.b + t.e) + (mb > 220.f ? (mb - 220.f) * t.f : 0.f);
}

// index of the cheapest shape, and its cost
inline int best_shape(const GemmDims *d, int n, float *cost) {
  // 128x128x2 gains where two blocks write out and multiply in turn, which needs many tiles, transposing reads and vector
  // stores (768x50257x2048 with its odd rows: 256 us against 208 with 128x256)
  bool tn = true, x2 = true;
  for (int i = 0; i < n; ++i) {
    tn = tn && d[i].ta && d[i].tb;
    x2 = x2 && d[i].vec_rows;
  }
  // (256x256 tiles of two strided operands, whose constants date from slices of 64: with slices of 32 they take 1.06 times the
  // estimate where they are among the best of the products below large_tn, the shapes chosen take 1.14 times theirs; over 2310
  // products and groups they were chosen 26 times, 1.04 times as fast as the next choice)
  int best = 0;
  for (int i = 0; i < SHAPE_128X256X2 - (tn && x2 ? 0 : 1); ++i) {
    const float c = shape_cost(plain_shapes[i], d, n);
    if (i == 0 || (c < *cost && shape_fits(plain_shapes[i], d, n))) { best = i; *cost = c; }
  }
  // Large: another shape has to be estimated 4 % below the one that all products would choose.  The 1340 of two strided operands
  // take 0.938 times as long as with that one, 1.6 % more than with the best shape; 42 are more than 3 % (9 more than 5 %) slower
  // than before there was a second table (with constants fitted to 106 products launched alone, and without the margin: 0.965, 255
  // and 172).  us, launched one after another, the first choice / now: 4096x16384x1024 175 / 157, 4096^3 126 / 112, 768x50257x2048
  // 213 / 199, 3728x3288x5556 159 / 127, 16384x4096x1024 157 / 147, 1600x6400x1000 33.9 / 32.6, 1024x50257x1024 197 / 175.
  // Contraction-contiguous: of 75 products that the constants were not fitted to and that take another shape here, 0.81 times as
  // long, two more than 3 % slower (6992x24656x224 220 / 233, 8395x19080x384 260 / 272); 1547x45480x512 199 / 132, 1087x38984x392
  // 101 / 75, 2215x35944x360 160 / 143.  (A first choice that is not in the table, 64x96, stays: 306x49616x768.)
  const bool nt = large_nt(d, n);
  if (!nt && !large_tn(d, n)) return best;
  const int first = best;
  float least = 0.f, own = 0.f;
  auto among = [&](const LargeShape &t) {
    const float c = large_cost(t, d, n);
    if (t.shape == first) own = c;
    if (least == 0.f || (c < least && shape_fits(plain_shapes[t.shape], d, n))) { best = t.shape; least = c; }
  };
  if (nt) for (const LargeShape &t : nt_shapes) among(t);
  else for (const LargeShape &t : tn_shapes) among(t);
  if (own == 0.f || least >= 0.96f * own) return first;
  *cost = least;
  return best;
}

// Input gradients of an LM head (results tokens x width, contraction over the vocabulary, weights stored [vocabulary][width]):
// what they wait for is lines that miss the L2s, which arrive at 3 TB/s, and small tiles - a few thousand tokens by a thousand
// columns - read every operand 8 to 32 times.  With two workgroups per tile, one per half of the contraction, the tiles are twice
// as large and all but one XCD read half of the lines; both add their results to a cleared C, one atomic addition each (0 + a + b =
// 0 + b + a: the bits repeat).  Cost in us: n * (a + u * b) + c * results / 10^6, u = two workgroups per tile / 256, n = K / 128;
// fits to 211 products (128 to 4096 tokens, widths 256 to 1600, vocabularies from 5000).  us, whole / halves: 2048x768x50257
// 313 / 224, 1024x4096x50400 470 / 391, 512x4096x50400 361 / 248, 1976x944x65803 453 / 296, 8576x120x59837 500 / 309.
// Contraction-contiguous operands of 4096 to 16384 steps: 3 of 30 more than 5 % shorter, hence the one layout.
struct HalfShape {
  int bm, bn;
  float a, b, c;
};
constexpr HalfShape half_shapes[] = {{128, 128, 0.496f, 0.118f, 6.36f}, {128, 192, 0.603f, 0.100f, 7.61f}, {128, 256, 0.744f, 0.064f, 8.38f}};

// index into half_shapes, -1: whole.  (whole_cost: estimate of best_shape, which for these products is 0.6 to 0.9 of the measured
// time, hence the factor.)  Only where all workgroups run at once: with a second round of them 21 of 21 products are 4 to 35 %
// slower than whole (8841x264x52499 405 / 546).  And only where 8 us are estimated to be gained, the clearing among them: without,
// 2039x576x10673 43.9 / 47.6, 1003x1392x11952 55.6 / 59.9; 128x256 tiles gain nothing over whole ones of 128x128 below 11520 steps
// (10 products, 0.92 to 1.105).  Of 531 products (128 to 33000 rows, 72 to 8192 columns, up to 200000 steps) 416 are computed in
// halves, 0.47 to 1.005 times as long, 0.79 on average, clearing and adding included.
inline int best_half_shape(const GemmDims &d, float whole_cost) {
  if (d.ta || !d.tb || d.K < 10240) return -1;
  const float n = (float)((d.K + 127) / 128);
  int best = -1;
  float cost = 1.35f * whole_cost - 8.f;
  for (int i = 0; i < 3; ++i) {
    const HalfShape &p = half_shapes[i];
    const int64_t groups = 2 * (((int64_t)d.M + p.bm - 1) / p.bm) * (((int64_t)d.N + p.bn - 1) / p.bn);
    if (groups > 256 || (p.bn == 256 && d.K < 11520)) continue;
    const float c = n * (p.a + (float)groups * (1.f / 256.f) * p.b) + p.c * 1e-6f * (float)d.M * (float)d.N;
    if (c < cost) { best = i; cost = c; }
  }
  return best;
}

// Products that 64x64 tiles would leave half of the CUs idle for, or a quarter with a long contraction: smaller tiles whose
// contraction eight wavefronts share out (gemm_split.hip).  Cost as above, with
// rounds = tiles / 256 rounded up also where two blocks share a CU; fits to 443 products of random layers (64 to 8192 tokens,
// widths 128 to 16384) with operands that are not in the L2s; the shape taken costs 0.2 % more than the best one on average.  800 narrow products (up
// to 256 rows or columns) against the 64x64 tiles before: 10 more than 3 % slower, the worst 33 / 44 us (tn 3776x80x10959).
// The first entry is the 64x64 shape of plain_shapes with its slices split over two groups of wavefronts.  Before / now: both
// operands contraction-contiguous 1.59 times as fast (181 products), one of each 1.44, both strided 1.29; 152x168x6120 nt
// 23.9 -> 7.9 us, 201x768x2304 nt 9.4 -> 6.0, 417x896x7784 nt 29.6 -> 23.5, 360x448x2719 tn 14.7 -> 10.4.
struct SplitShape {
  int bm, bn;
  float t0[2], a[2], b[2], c[2], e[2];
};
constexpr SplitShape split_shapes[] = {
    {64, 64, {3.612f, 3.172f}, {0.178f, 0.232f}, {0.050f, 0.013f}, {0.f, 0.f}, {0.149f, 1.512f}},
    {64, 32, {1.455f, 1.642f}, {0.149f, 0.199f}, {0.010f, 0.019f}, {1.284f, 0.584f}, {0.865f, 1.780f}},
    {48, 32, {2.752f, 2.218f}, {0.118f, 0.188f}, {0.021f, 0.020f}, {0.f, 0.f}, {0.483f, 1.353f}},
    {32, 32, {2.709f, 2.307f}, {0.087f, 0.147f}, {0.026f, 0.041f}, {0.f, 0.f}, {0.287f, 0.575f}},
    {16, 32, {2.545f, 2.402f}, {0.047f, 0.129f}, {0.041f, 0.044f}, {0.144f, 0.f}, {0.000f, 0.120f}},
    {16, 16, {2.676f, 2.586f}, {0.040f, 0.084f}, {0.007f, 0.068f}, {0.037f, 0.f}, {0.407f, 0.273f}},
};
constexpr int N_SPLIT = sizeof(split_shapes) / sizeof(split_shapes[0]);

// below 384 contraction steps a launch is its latency, whatever the tile
inline bool few_tiles(const GemmDims &d) {
  const int64_t t = ((int64_t)d.M + 63) / 64 * (((int64_t)d.N + 63) / 64);
  return (t <= 128 && d.K >= 384) || (t <= 192 && d.K >= 1024);
}

// index into split_shapes, -1 for its first entry
inline int best_split_shape(const GemmDims &d) {
  const float x = d.ta == d.tb ? (float)d.ta : 0.5f;  // one transposed operand: half way between the two
  auto at = [x](const float (&v)[2]) { return v[0] + x * (v[1] - v[0]); };
  const float nk = (float)((d.K + 63) / 64);
  int best = 0;
  float cost = 0.f;
  for (int i = 0; i < N_SPLIT; ++i) {
    const SplitShape &p = split_shapes[i];
    const float u = (float)((d.M + p.bm - 1) / p.bm) * (float)((d.N + p.bn - 1) / p.bn) * (1.f / 256.f);
    const float c = at(p.t0) + ceilf(u) * (nk * at(p.a) + at(p.c)) + u * (nk * at(p.b) + at(p.e));
    if (i == 0 || c < cost) { best = i; cost = c; }
  }
  return best > 0 ? best : -1;
}

}  // namespace hydra
