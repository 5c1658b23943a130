// Which tiles an FP4 GEMM is cut into: host arithmetic on its sizes, types and the number of compute units.
#pragma once
#include <stdint.h>

#include <algorithm>

struct GemmTiling {
  int tile;      // 64, 128 or 256: rows and columns of an output tile
  int rest;      // 256: tiles of the last round that are cut into 128 x 128 ones
  int stagger;   // 256: how much later than the one before each quarter of the workgroups begins, in 512 cycles
};

// Offset past the end of any tile's buffer descriptor while the tile's rows take no more bytes than this.
constexpr uint32_t GEMM_OUT_OF_RANGE = 0xf0000000u;
constexpr int GEMM_K_STEP = 128;   // bytes of a row that one stage of the staged tilings holds

inline GemmTiling gemm_tiling(int64_t P, int64_t Q, int64_t Kc, bool factor, bool w_bf16, bool addend, bool out_bf16, int n_cu) {
  GemmTiling t = {256, 0, 0};
  const int64_t Kb = Kc / 2;
  // What bounds a call with few tiles is one tile's chain of steps, so the smaller tile wins while there is no more than a
  // round or two of it.  Measured as 64 / 128 / 256 tiles, in us:
  //  64, up to 1024 codes and two tiles per CU: 512 x 2048, 512 codes 5.6 / 7.1 / 11.5; 512 x 1024, 1024 7.2 / 7.8 / 13.3;
  //   past that line 512 x 2048, 2048 10.7 / 9.5 / 17.5; 2048 x 2048, 256 9.7 / 7.6 / 11.4.
  //  64 with the factor, which asks for many threads: tiles x contraction up to 3072 codes per CU (the whole weight gradient
  //   without the clamp, fp32, 1024 x 1024, 2048 codes: 42 / 45 / 78; 1376 x 2080, 1056: 45 / 47 / 77; 2048 x 2048, 2048: 72 / 51 / 84).
  //  128, up to two per CU: 4096 x 2048, 1024 / 8192 codes, fp32 with addend 40 / 22.6 / 24.8 and 237 / 54 / 58; past it
  //   2816 x 3072, 4096 140 / 48 / 38.  With the factor one (2048 x 4096 x 4096 bf16 172 / 87 / 86), and with fp32 masters, for which
  //   the big tiles have no branch-free epilogue, three (2048 x 5504, 2048 codes 138 / 88 / 93; 4096 x 4096, 2048 180 / 107 / 99).
  const int64_t small_tiles = ((P + 63) / 64) * ((Q + 63) / 64), mid_tiles = ((P + 127) / 128) * ((Q + 127) / 128);
  const bool few = factor ? small_tiles <= 3 * (int64_t)n_cu && small_tiles * Kc <= 3072 * (int64_t)n_cu
                          : small_tiles <= 2 * (int64_t)n_cu && Kc <= 1024;
  // The larger tiles address their rows by 32-bit offsets into a descriptor; rows too long for that go to the next smaller
  // one, and the 64 x 64 ones have 64-bit addresses.
  const bool fits_big = Kb * 256 <= (int64_t)GEMM_OUT_OF_RANGE, fits_mid = Kb * 128 <= (int64_t)GEMM_OUT_OF_RANGE;
  // An empty contraction has no K step to request, which the staged tilings do ahead: the operands may be null.
  if (few || !fits_mid || Kb == 0) {
    t.tile = 64;
    return t;
  }
  if (mid_tiles <= (factor ? (w_bf16 ? 1 : 3) : 2) * (int64_t)n_cu || !fits_big) {
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
  // 11008 x 4096 131 -> 127; three full rounds 410 -> 415, bf16 without addend 353 -> 359).
  const int64_t full = total - t.rest;
  t.stagger = (addend || !out_bf16) && (full > 3 * wgs || (full > 2 * wgs && 8 * full <= 23 * (int64_t)wgs)) ? 15 : 0;
  return t;
}
