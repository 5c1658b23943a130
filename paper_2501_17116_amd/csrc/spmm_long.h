// Rows of a CSR matrix that are "long" (outlier channels, nearly dense among rows that are nearly empty): the
// kernels that walk many rows side by side leave them out (one such row holds up its whole workgroup), the
// long-row kernels of spmm.hip multiply them.
#pragma once
#include "fp4_common.h"

// What the packed product of spmm_mfma.hip leaves to the tiled kernel: bundle i has 16 * groups rows, and is left
// where steps[i] < 0 or redo[i] != 0.
struct SpmmRest {
  const int32_t* steps;
  const int32_t* redo;
  int groups;   // 1 to 3
};

#if defined(__HIPCC__)
// A row is long above a quarter of the columns, at most 2048 entries, but always above four times the mean row.  Measured
// against 2048 entries whatever the width (steps with one to ten dense channels): fp32 2048^3 1379 -> 429 us, fp32 256 x 512
// x 512 337 -> 256 us, bf16 1056 x 1376 x 2080 836 -> 403 us.
// With 64 columns or fewer no row is long, also not one that repeats columns and so has more entries than that: the
// long-row kernels are not launched then.
constexpr int64_t SPMM_LONG_MIN = 64;
FP4_D int64_t spmm_long_limit(const int64_t* row_ptr, int64_t P, int64_t Q, int64_t capacity) {
  if (Q <= SPMM_LONG_MIN) return INT64_MAX;
  const float mean = (float)(min(row_ptr[P], capacity) - row_ptr[0]) / (float)P;
  return max(min(max(Q / 4, SPMM_LONG_MIN), (int64_t)2048), (int64_t)(4.0f * mean));
}

// Rows in ascending order, by one workgroup of THREADS (ballot + scan), so the split between the long-row kernels
// does not depend on timing.  16 x THREADS rows a turn: all their row_ptr loads in flight at once, then one scan over
// the (round, wave) counts instead of a barrier-separated step per THREADS rows.
template <int THREADS>
FP4_D void find_long_rows(const int64_t* row_ptr, int64_t P, int64_t Q, int64_t capacity, int32_t* list, int32_t* count) {
  constexpr int W = THREADS / 64, PER = W / 4;   // counts a lane of the scanning wave holds
  static_assert(W % 4 == 0 && THREADS % 64 == 0, "whole waves, whole counts a lane");
  __shared__ int s_cnt[16 * W];   // [round][wave] counts, then their exclusive prefix in that order
  __shared__ int s_base;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t long_limit = spmm_long_limit(row_ptr, P, Q, capacity);
  if (tid == 0) s_base = 0;
  for (int64_t r0 = 0; r0 < P; r0 += 16 * THREADS) {
    uint32_t flags = 0;
#pragma unroll
    for (int it = 0; it < 16; ++it) {
      const int64_t row = r0 + it * THREADS + tid;
      const bool is_long = row < P && min(row_ptr[row + 1], capacity) - row_ptr[row] > long_limit;
      flags |= (is_long ? 1u : 0u) << it;
    }
#pragma unroll
    for (int it = 0; it < 16; ++it) {
      const unsigned long long m = __ballot((flags >> it) & 1u);
      if (lane == 0) s_cnt[it * W + wave] = __popcll(m);
    }
    __syncthreads();   // counts complete (and s_base of the turn before)
    if (wave == 0) {
      int c[PER], sum = 0;
#pragma unroll
      for (int j = 0; j < PER; ++j) { c[j] = s_cnt[lane * PER + j]; sum += c[j]; }
      int incl = sum;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int up = __shfl_up(incl, o, 64);
        if (lane >= o) incl += up;
      }
      int run = s_base + incl - sum;
#pragma unroll
      for (int j = 0; j < PER; ++j) { s_cnt[lane * PER + j] = run; run += c[j]; }
      if (lane == 63) s_base = run;
    }
    __syncthreads();
#pragma unroll
    for (int it = 0; it < 16; ++it) {
      const bool is_long = (flags >> it) & 1u;
      const unsigned long long m = __ballot(is_long);
      const int pos = s_cnt[it * W + wave] + __popcll(m & ((1ull << lane) - 1ull));
      if (is_long) list[pos] = (int32_t)(r0 + it * THREADS + tid);
    }
    __syncthreads();   // s_cnt is rewritten in the next turn
  }
  if (tid == 0) *count = P > 0 ? s_base : 0;
}
#endif
