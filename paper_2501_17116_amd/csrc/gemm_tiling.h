// Which tiles an FP4 GEMM is cut into: host arithmetic on its sizes, types and the number of compute units.
#pragma once
#include <stdint.h>

#include <algorithm>

struct GemmTiling {
  int tile;      // 32 (whose waves share a contraction), 64, 128 or 256: rows and columns of an output tile
  int rest;      // 256: tiles of the last round that are cut into 128 x 128 ones
  int stagger;   // 256: how much later than the one before each quarter of the workgroups begins, in 512 cycles
};

// Codes up to which every sum of products is a multiple of 1/4 below 2^22 (a product is 36 at most), so exact in fp32 in any order.
constexpr int64_t GEMM_EXACT_CODES = (1 << 22) / 36;
// Offset past the end of any tile's buffer descriptor while the tile's rows take no more bytes than this.
constexpr uint32_t GEMM_OUT_OF_RANGE = 0xf0000000u;
constexpr int GEMM_K_STEP = 128;   // bytes of a row that one stage of the staged tilings holds

// Whether the 64 x 64 tiles, whose operands go straight to registers, beat the 128 x 128 ones, whose go through a ring in LDS.  What
// bounds a call with few tiles is one tile's chain of steps: theirs is shorter to start and slower a step, so the line is a
// length of the contraction, and it moves with
//  - whether a row of codes is whole 128-byte lines.  Where it is, all rows of a tile come to the end of a line in the same step
//    and their next lines are waited for together; where it is not, a few do in every step;
//  - the rounds of tiles that a CU takes (the smaller tile is the first to need a second one);
//  - the factor, which asks for many threads.
// In us as 64 / 128 tiles, bf16 out with fp32 addend or fp32 out, one round: rows of whole lines, 1024 codes (64 x 2048) 6.9 / 7.0,
// 2048 9.7 / 8.8; others, 1056 (64 x 2048) 5.1 / 7.7, 4640 (512 x 512) 0.85 of the 128 tiles' time, 6176 1.00.  Two rounds, whole
// lines, 256 / 512 codes 0.91 / 1.13, others 1056 / 1312 0.92 / 1.00; three rounds, others, 416 / 544 0.96 / 1.01.  With the factor, one
// round, whole lines, 3072 / 4096 codes 0.95 / 1.04, others 8224 / 10272 0.92 / 1.06; two rounds, 768 / 1024 0.98 / 1.05 and 2080 / 2592
// 0.85 / 1.04; three, 256 / 512 0.90 / 1.06 and 1056 / 1312 0.92 / 1.00, with fp32 weights 1312 / 1568 0.86 / 1.0 and, four rounds,
// 384 0.62, 800 1.02.
inline bool gemm_small_tiles_win(int64_t P, int64_t Q, int64_t Kc, bool factor, bool w_bf16, int n_cu) {
  const int64_t tp = (P + 63) / 64, tq = (Q + 63) / 64, tiles = tp * tq, rounds = (tiles + n_cu - 1) / n_cu, Kb = Kc / 2;
  if (rounds > 4) return false;
  const int r = (int)std::max<int64_t>(rounds, 1) - 1;
  if (Kb % GEMM_K_STEP == 0) {
    static constexpr int plain[4] = {1280, 256, 0, 0}, with_factor[4] = {3072, 768, 256, 0};
    return Kc <= (factor ? with_factor : plain)[r];
  }
  static constexpr int plain[4] = {6144, 1088, 448, 0}, with_factor[4] = {8448, 2336, 1184, 0}, with_f32_factor[4] = {8448, 2336, 1376, 640};
  if (Kc > (factor ? (w_bf16 ? with_factor : with_f32_factor) : plain)[r]) return false;
  if (Kc <= 1024 || tp == 1 || tq == 1) return true;
  // An operand row is read once for every tile that needs it, so the rows that an XCD's tiles need (they are dealt round, column by
  // column) have to stay in its 4 MiB of L2: 320 x 3200, 2592 / 3616 codes, 3.0 / 4.3 MB: 0.92 / 1.13; 512 x 2048, 3104 / 4640, 3.3 / 4.9
  // MB: 0.83 / 1.25.  With the factor 512 x 2048, 3616 / 5152, 3.8 / 5.4 MB: 0.90 / 1.09, and where a CU takes more than one
  // round 512 x 4096, 1312 / 1824, 2.7 / 3.8 MB: 0.87 / 1.15.
  int64_t stride = 8;
  while (tp % stride) stride /= 2;   // of the tiles of a column, each XCD has every stride-th
  const int64_t share = (tiles + 7) / 8, rows = 64 * (std::min(tq, share) + std::min(tp / stride, share));
  return rows * Kb <= (!factor ? 15 << 18 : r == 0 ? 18 << 18 : 10 << 18);
}

// Whether 32 x 32 tiles, whose four waves share the contraction, beat both: what they save are round trips, up to two workgroups a CU (one with
// rings of four steps, two with rings of two), so they win from two steps of whole lines on, and where rows are no whole lines, so
// that a step's lines are half another's, from four on.  With the factor from one, because they have more threads for it.  In us,
// 64 or 128 tiles / these, bf16 with fp32 addend: 64 x 2048, 256 codes 4.4 / 4.7, 512 5.4 / 4.4, 1024 7.0 / 4.6, 2048 9.7 / 5.0, 8192 20.9 / 6.8, 544
// 4.6 / 4.5, 1376 5.8 / 4.9; two a CU, 64 x 8192, 512 5.5 / 5.1, 2048 9.6 / 6.0, 8192 22 / 10.8, 544 4.6 / 5.4, 1376 6.0 / 5.7; factor, 512 x 512,
// 128 5.5 / 5.3, 256 5.9 / 5.2, 512 x 1024, 128 5.6 / 6.2, 256 6.2 / 6.0.  Another half round: 96 x 8192, 1024 7.4 / 7.2, 2048 10.2 / 8.1, 8192 23 /
// 13.8, 2080 7.5 / 8.4, 3168 12.9 / 9.5.  Beyond, the operands' second and third reading counts: 1024 tiles, 4096 codes 13.5 / 11.3 to 13.4 / 13.0, 2048
// tiles 13.8 / 18.8.  Only while sums are exact, or the waves' four would not add up to the bits of the others' one chain.
inline bool gemm_split_tiles_win(int64_t P, int64_t Q, int64_t Kc, bool factor, int n_cu) {
  const int64_t tiles = ((P + 31) / 32) * ((Q + 31) / 32);
  const bool whole = Kc / 2 % GEMM_K_STEP == 0;
  if (Kc > GEMM_EXACT_CODES) return false;
  if (tiles <= 2 * (int64_t)n_cu) return Kc >= (factor ? 256 : whole ? 512 : 1120);
  return tiles <= 3 * (int64_t)n_cu && !factor && Kc >= (whole ? 1024 : 3072);
}

inline GemmTiling gemm_tiling(int64_t P, int64_t Q, int64_t Kc, bool factor, bool w_bf16, bool addend, bool out_bf16, int n_cu) {
  GemmTiling t = {256, 0, 0};
  const int64_t Kb = Kc / 2;
  if (gemm_split_tiles_win(P, Q, Kc, factor, n_cu)) {
    t.tile = 32;
    return t;
  }
  const bool few = gemm_small_tiles_win(P, Q, Kc, factor, w_bf16, n_cu);
  // 128 x 128, up to two per CU: 4096 x 2048, 1024 / 8192 codes, fp32 with addend, as 64 / 128 / 256 tiles in us: 40 / 22.6 / 24.8 and
  // 237 / 54 / 58; past it 2816 x 3072, 4096 140 / 48 / 38.  With the factor one (2048 x 4096 x 4096 bf16 172 / 87 / 86).  With fp32
  // masters, for which the big tiles have no branch-free epilogue, three with an addend (2016 x 4640, 1632 codes 128 / 256: 54 / 62;
  // 2800 x 3456, 3328 63 / 67) and two without (2872 x 3376, 8448 88 / 76; 1248 x 7344, 5600 79 / 67).
  const int64_t mid_tiles = ((P + 127) / 128) * ((Q + 127) / 128);
  const int mid_per_cu = !factor ? 2 : w_bf16 ? 1 : addend ? 3 : 2;
  // The larger tiles address their rows by 32-bit offsets into a descriptor; rows too long for that go to the next smaller
  // one, and the 64 x 64 ones have 64-bit addresses.
  const bool fits_big = Kb * 256 <= (int64_t)GEMM_OUT_OF_RANGE, fits_mid = Kb * 128 <= (int64_t)GEMM_OUT_OF_RANGE;
  // An empty contraction has no K step to request, which the staged tilings do ahead: the operands may be null.
  if (few || !fits_mid || Kb == 0) {
    t.tile = 64;
    return t;
  }
  if (mid_tiles <= mid_per_cu * (int64_t)n_cu || !fits_big) {
    t.tile = 128;
    return t;
  }
  // A last round of 256 x 256 tiles that no more than a quarter of the CUs have is cut into 128 x 128 ones, which go round the
  // chip once: 320 tiles, 13824 codes 166 -> 143 us (with fp32 addend 183 -> 160), 2048 codes 41 -> 38 (59 -> 54); 289, 512
  // codes 25.5 -> 23.6; 1080, 4096 codes 162 -> 153.  Two rounds of them take as long as the one they replace, or longer (352
  // tiles, 512 / 4096 / 13824 codes 26 / 62 / 166 -> 29 / 66 / 173).
  const int wgs = (n_cu / 8) * 8;
  const int64_t total = ((P + 255) / 256) * ((Q + 255) / 256);
  if (total > wgs && 4 * (total % wgs) <= wgs) t.rest = (int)(total % wgs);
  // Workgroups that start together come to their epilogues together: memory is idle while all multiply and the bound while all
  // add, convert and store.  Four quarters 3.4 us apart overlap the two where an epilogue moves much (addend, fp32
  // output) and a workgroup has enough tiles to make up for it, or those that have one less can be the late ones
  // (16384 x 12288 x 4096 with addend 603 -> 561 us, 16384 x 4096 x 2048 151 -> 137, 5120 x 13824 x 4096 fp32 258 -> 246, 4096 x
  // 11008 x 4096 131 -> 127; three full rounds 410 -> 415, bf16 without addend 353 -> 359).  It stays off where it lost: fp32
  // outputs in whole rounds with nothing behind them (1024 tiles, 256 / 512 / 1024 codes 66 -> 71, 74 -> 80, 89 -> 94; 1536, 2048 codes
  // with addend 262 -> 270; with 64 cut tiles behind, 1024 codes, 101 -> 85), the factor with fp32 weights (736 tiles, 256 codes 142 -> 148, else within 2 %), and at short contractions nearly three rounds (736
  // tiles, 256: bf16 with addend 62 -> 63, factor 94 -> 98, 1024: factor 107 -> 109) and the factor without addend (1088, 256: 141 -> 146).
  const int64_t full = total - t.rest;
  const bool whole = full % wgs == 0 && t.rest == 0, short_k = Kc < 1024;
  const bool rounds = full > 3 * wgs || (full > 2 * wgs && 8 * full <= (Kc < (factor ? 2048 : 1024) ? 21 : 23) * (int64_t)wgs);
  const bool gains = factor ? w_bf16 && (addend || !short_k) : out_bf16 ? addend : !whole;
  t.stagger = rounds && gains ? 15 : 0;
  return t;
}
