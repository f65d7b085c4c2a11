// Choice of the block form of the fused attention kernels (host only, no HIP).
#pragma once
#include <stdint.h>

#include <cmath>

namespace hydra {

// A block of kw groups of rw wavefronts owns 32 * rw rows and walks over tiles of tk rows, which its groups share out.  What a
// launch costs in us: a + sqrt((b * steps of the longest block)^2 + (c * steps of all blocks / 256)^2) - the chain of tiles
// that the longest block walks, and what all of them keep the CUs busy with.  Least-squares fits to 114 calls of 64 to 2048
// positions, 4 to 256 pairs of sample and head; the form taken is within 1 % of the best one on average.
struct AttnForm {
  int rw, kw, tk;
  float a, b, c;
};
// Large launches: one group of four wavefronts, two to four blocks per CU; tiles of 64 rows, forward at head width 128 of 32
// (three blocks per CU; at 64 the two are within 1 %: B 8, H 25, T 1024 forward and backward 176 us with 64, 178 with 32).
// Few rows: 64-row blocks, twice as many, whose tiles two or four groups share.  The former forms (128-row blocks and 64-row
// tiles, one or two groups) / these, us, launched one after another, forward then backward:
//   B 4, H 12, T 512, dh 64 10.6 / 9.3, 28.3 / 24.5;  B 4, H 12, T 1024, dh 64 17.9 / 16.2, 49.1 / 48.8;
//   B 1, H 16, T 2048, dh 128 41.7 / 35.8, 116 / 106;  B 4, H 16, T 2048, dh 128 82 / 79, 258 / 258;
//   600 random calls: 1.12 times as fast at head width 64 either way, 1.17 and 1.16 at 128
constexpr AttnForm attn_forms_fwd64[] = {{4, 1, 64, 3.147f, 0.762f, 0.666f},
                                         {2, 1, 32, 2.866f, 0.495f, 0.193f},
                                         {2, 2, 32, 3.569f, 0.455f, 0.388f},
                                         {2, 2, 64, 3.828f, 0.728f, 0.868f},
                                         {2, 4, 32, 4.803f, 0.440f, 0.908f}};
constexpr AttnForm attn_forms_fwd128[] = {{4, 1, 32, 3.860f, 0.667f, 0.572f},
                                          {2, 1, 32, 3.347f, 0.668f, 0.368f},
                                          {2, 2, 32, 4.604f, 0.620f, 0.804f}};
// (backward at head width 64: fitted to 340 calls with the launches of attn_bwd_mode, to the choice rather than the times)
constexpr AttnForm attn_forms_bwd64[] = {{4, 1, 64, 3.557f, 3.333f, 1.875f},
                                         {2, 1, 32, 2.999f, 1.706f, 0.618f},
                                         {2, 2, 32, 7.170f, 0.823f, 1.938f},
                                         {2, 2, 64, 7.611f, 0.983f, 4.965f}};
constexpr AttnForm attn_forms_bwd128[] = {{4, 1, 64, 11.223f, 4.395f, 3.716f},
                                          {2, 1, 32, 9.295f, 2.444f, 1.181f},
                                          {2, 2, 32, 14.782f, 2.022f, 2.582f}};

inline float attn_form_cost(const AttnForm &f, int pairs, int T) {
  const float R = 32.f * f.rw, W = (float)f.kw * f.tk, nb = ceilf(T / R);
  const float chain = ceilf(T / W), all = pairs * nb * ((nb + 1.f) * R / (2.f * W) + 0.5f) / 256.f;
  return f.a + sqrtf(f.b * chain * f.b * chain + f.c * all * f.c * all);
}

// index of the cheapest form.  Several groups per block only while the blocks are resident at once or nearly so (what a second
// round of them costs is not in the estimate): B 5, H 25, T 368, dh 128 (750 blocks) 16.6 with one group, 22.9 with two; long
// sequences gain even then: B 1, H 25, T 1960 (775) 50 / 46; head width 64 has room for more: B 3, H 12, T 2016 (1152) 39 / 31,
// but B 5, H 25, T 456 (1000) 13.2 / 15.9.
// For the same reason, from one block of 128 rows per CU on, another form has to be estimated below `whole` times the first
// one: us, forward B 3, H 25, T 1024, dh 64 22.0 with the first form, 26.2 with two groups (estimates 22.3, 21.5), backward
// B 7, H 25, T 328, dh 64 31.8 / 35.0 with 64-row blocks (30.0, 29.7), B 7, H 12, T 672, dh 128 70.6 / 75.3 (84.4, 83.3).  Of
// 2400 random calls, forward and backward (then in two launches), 174 were more than 3 % (73 more than 5 %) slower than with the two
// forms before this table, with it 48 (23); the form taken was 0.2 to 0.3 % off the best one on average.
template <int N>
inline int best_attn_form(const AttnForm (&f)[N], int dh, int pairs, int T, float whole) {
  const int64_t blocks = ((int64_t)T + 63) / 64 * pairs, limit = dh == 64 ? (T >= 576 ? 1280 : 900) : (T >= 768 ? 900 : 512);
  const bool filled = ((int64_t)T + 127) / 128 * pairs >= 256;
  int best = 0;
  float cost = 0.f;
  for (int i = 0; i < N; ++i) {
    const float c = attn_form_cost(f[i], pairs, T) * (i == 0 && filled ? whole : 1.f);
    if (i == 0 || (c < cost && (f[i].kw == 1 || blocks <= limit))) { best = i; cost = c; }
  }
  return best;
}
inline int attn_form_fwd(int dh, int pairs, int T) {
  return dh == 64 ? best_attn_form(attn_forms_fwd64, dh, pairs, T, 0.92f)
                  : best_attn_form(attn_forms_fwd128, dh, pairs, T, 1.f);
}
// head width 64, backward: a sequence of one 64-row tile is one step of the first form and two of the others, up to 32 rows it is
// one of each and the smaller block is done sooner.  In two launches that showed (B 4, H 12, T 56 9.4 / 9.9, T 24 7.9 / 6.8), in one
// they are alike (5.7 / 5.7, 5.8 / 5.6), and from some 250 pairs on the second form would be the faster one (B 25, H 16, T 56 11.6 /
// 10.4, T 40 10.5 / 8.7).
inline int attn_form_bwd(int dh, int pairs, int T) {
  if (dh == 64) return T > 32 && T <= 64 ? 0 : best_attn_form(attn_forms_bwd64, dh, pairs, T, 0.954f);
  const int form = best_attn_form(attn_forms_bwd128, dh, pairs, T, 0.95f);
  // head width 128, thousands of 64-row blocks of a few tiles: in one launch those lose what two had (B 27, H 32, T 408 397 / 441,
  // B 28, H 16, T 576 298 / 318), two of 128-row blocks do not (361 and 277)
  return form == 1 && ((int64_t)T + 63) / 64 * pairs >= (T > 512 ? 2500 : T >= 256 ? 4500 : INT64_MAX) ? 0 : form;
}

// The launches of the backward pass, whose two parts are dQ and dK/dV: two (part 2 reads the D = rowsum(dO * O) that part 1
// wrote); one, in which the blocks of part 2 sum D themselves; or one after a small launch that sums D.  (The figures above are
// those of two launches, and so are the constants of head width 128.)  Most calls wait for chains of tiles, those of one part as
// long as the other's, and have room for both at once: two / one, us: B 4, H 12, T 512, dh 64 23.9 / 18.7; B 1, H 12, T 1024
// 30.3 / 24.6; B 2, H 4, T 64 9.0 / 5.4; B 8, H 25, T 1024 143 / 133; B 1, H 16, T 1024, dh 128 57 / 44.  Over 340 random calls
// of 16 to 2048 positions form and mode are within 2 % of the best at head width 64, over 310 within 2 % at 128.
enum AttnBwdMode { BWD_TWO, BWD_ONE, BWD_ONE_AFTER_D, BWD_MIXED, BWD_MIXED_AFTER_D };
constexpr AttnBwdMode attn_bwd_mode(int dh, int form, int pairs, int T) {
  const int rows = 32 * (dh == 64 ? attn_forms_bwd64[form] : attn_forms_bwd128[form]).rw;
  const int64_t blocks = ((int64_t)T + rows - 1) / rows * pairs;  // of each part
  // long sequences, and each part's blocks of a row a multiple of 8 or both parts' a divisor of it: see attn_bwd_place
  const bool lopsided = T > 2048 && (pairs % 8 == 0 || pairs == 4 || pairs < 3);
  if (dh == 64) {
    // Two launches remain where the tensors (a KB per position and pair) exceed the 256 MB cache and both parts would fetch them at
    // once: B 8, H 32, T 3792 1824 us, in one 2089; T 2656 923 / 982; B 4, H 32, T 2216 329 / 342; B 44, H 16, T 936 470 / 481; not
    // for short sequences, whose tiles are read again soon (B 28, H 16, T 656 203 / 178).
    if (form == 0 && T >= 800 && (int64_t)pairs * T >= (T > 2048 ? 240000 : T >= 1200 ? 320000 : 600000)) return BWD_TWO;
    if (form == 1) {
      // thousands of single tiles, of which a CU takes more while they are of part 1 alone (T 16, 9376 blocks 71.6 / 77.4 in one)
      if (T <= 32) return blocks > (T <= 16 ? 4096 : 6000) ? BWD_TWO : BWD_ONE;
      // the 256 MB cache as above (B 109, H 16, T 448 509 / mixed 539)
      if (T >= 384 && (int64_t)pairs * T >= 600000) return BWD_TWO;
      // one / mixed after D: 1476 blocks 35 / 37, 1580 42 / 43, 2448 55 / 50, 7200 296 / 249, two launches 258
      return blocks > 1536 ? BWD_MIXED_AFTER_D : BWD_ONE;
    }
    // Summing D takes registers: two such blocks fit a CU, of the others three.  With more blocks than the chip holds that is
    // worth the 2.5 us of the launch before (us, one / after D, 64-row blocks of two groups: 512 blocks 18.2 / 18.9, 640 29.9 /
    // 28.5, 1056 50.5 / 44.6; 128-row: 525 32.7 / 33.9, 672 54 / 50.5); 64-row tiles shared by two groups are for few blocks anyway.
    const bool after = blocks > 512 && form != 3;
    // H 16, T 3792 150 / mixed 126 (two launches 139), T 2904 89 / 79 (85), B 2, H 2, T 7944 190 / 160 (185)
    if (lopsided && form != 3) return after ? BWD_MIXED_AFTER_D : BWD_MIXED;
    return after ? BWD_ONE_AFTER_D : BWD_ONE;
  }
  // Head width 128: with D to sum 40 registers are spilled, which only few sequences of one tile do not feel (64 of T 24 7.4 / after
  // D 8.2 us, 256 of T 16 9.1 / 8.6).  Two launches remain where 128-row blocks abound: D is summed beside part 1's other work, and
  // nobody waits for a chain (B 4, H 16, T 2048 271 us, after D 282; B 4, H 12, T 2224, 864 blocks, 249 / 258; with fewer blocks
  // B 3, H 25, T 1584, 975, 224 / 218, B 8, H 25, T 512, 800, 106 / 98).
  if (form == 0 && blocks >= (T > 2048 ? 850 : 1000)) return BWD_TWO;
  if (form == 1) {
    if (T <= 32 && blocks <= 256) return BWD_ONE;
    // thousands of short sequences, whose tiles both parts then fetch once: after D / mixed (two launches) 3008 of T 64 161 / 136
    // (159), 9376 of T 16 136 / 126 (127), 1300 of T 40 47 / 44 (51); at T 536 136 / 143.  Two launches for one-tile blocks whose
    // number fits two rounds of part 1 alone (996 of T 40 33.6, mixed 36.7, 736 of T 16 14.1 / 15.0)
    if (T <= 48 && blocks >= 640 && blocks <= 1024) return BWD_TWO;
    return T <= 48 || (blocks > 1024 && T <= 512) ? BWD_MIXED_AFTER_D : BWD_ONE_AFTER_D;
  }
  // H 16, T 3416 248 / mixed 202 (two launches 211), B 2, H 4, T 11944 1091 / 1000 (1013); others B 2, H 3, T 5632 209 / 234
  return lopsided && blocks > 512 ? BWD_MIXED_AFTER_D : BWD_ONE_AFTER_D;
}

// The mixed launch of both parts: block id -> part, pair of sample and head, row block.  (In the other one all pairs' dK/dV blocks
// of a row come before their dQ blocks.)  Ids go round-robin to the 8 XCDs and from there round-robin to the groups of CUs: with
// 16 pairs, say, half of the CUs see the longer dK/dV blocks alone.  Here ids 16 q + x and 16 q + 8 + x are both parts of one
// pair's row block, which thus share an XCD's L2, in the order of the Thue-Morse sequence: whatever power of two the CUs are taken
// in, each gets as many of one part as of the other.  Not for few rounds of blocks, where the longest had better be first (B 7,
// H 32, T 248, dh 128 49.6 / 54.7).
struct AttnBwdPlace {
  bool dq;
  int z, rb;
};
constexpr AttnBwdPlace attn_bwd_place(uint32_t id, uint32_t pairs) {
  const uint32_t k = id >> 3, m = (k >> 1) * 8 + (id & 7), rb = m / pairs;
  return {(__builtin_popcount(k) & 1) != 0, (int)(m - rb * pairs), (int)rb};
}
constexpr uint32_t attn_bwd_grid(uint32_t row_blocks) { return (row_blocks + 7) / 8 * 16; }

}  // namespace hydra
