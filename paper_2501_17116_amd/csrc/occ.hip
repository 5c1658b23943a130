// Outlier clamping and compensation (Sec. 3.2): exact per-tensor quantile thresholds by
// radix selection, and the ordering of the clamped-away residual of long rows into canonical
// CSR.  (The clamp itself is fused into the quantization pass; the transpose for the weight
// gradient and the sparse x dense product live with the sparse kernels.)
#include "fp4_common.h"
#include "fp4_measure.h"
#include "select.h"

#include <algorithm>
#include <cstddef>
#include <type_traits>

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));

// ---- bf16 tensors: thresholds and the rows' outlier counts out of one pass -------------------------------------------------
// The leading 11-bit digits of the thresholds, exactly (from a digit pass, up to 2^25 elements) or to within a few of 2048 (from a
// sample), leave few keys; the pass over all elements then needs bins only for the keys around them (three digits, 96 keys a
// threshold), counts what lies outside, and keeps every row's bins: with the thresholds known, a row's outliers are a sum over those.
// Where a sampled threshold turns out not to lie in its window, or a NaN is about, `done` stays 0 and the passes of the general path,
// launched behind, do their work; otherwise they leave at once.  Behind an exact digit the thresholds always come out of the bins, and
// what can fail (a NaN, zeros that are outliers) is that the rows' bins tell the rows' counts: those are taken from the elements then.
// Bound by the one read and, about as long, by vector instructions (nine an element, twelve where zeros are counted apart).
// 16384 x 11008, in us: sample 6.6, the pass 97, the general path's two launches 10, rows 6, together 119 (130 with picks in launches of
// their own, of 4.8 each); digit passes, picks and the count of the rows after them 249.  16384 x 4096: 65 against 107.  Half
// zeros, 16384 x 11008, with scan and emission, 250 against 540; a miss (a NaN), which took 466 with picks, now 367.  8192 x 2048, behind a digit pass of 14 us: the
// pass 19.5, rows 7.6, where a second digit pass and the count of the rows took 15 and 11 and two picks and the clearing 4.5 each; 1056 x
// 1376 7.2 + 8.1 + 4.2 against 7.1 + 4.4 + 7.3 + 4.0 + 4.2 and 2.2.
// 4096 runs of 512 elements, evenly spaced.  As many elements in 128 runs were a few hundred whole rows: of 216 tensors and alphas
// (large rows or channels, first tokens 1000 times as large, rows or channels that differ in scale) the windows missed 20, now 1.
__global__ __launch_bounds__(SEL_THREADS) void sel_sample_kernel(const u32x4* x, int64_t nvec, unsigned long long* hist) {
  __shared__ uint32_t h[8 * SEL_BINS];
  for (int i = threadIdx.x; i < 8 * SEL_BINS; i += SEL_THREADS) h[i] = 0;
  __syncthreads();
  uint32_t* const hrep = &h[(threadIdx.x & 7) * SEL_BINS];
  const int64_t run = (int64_t)blockIdx.x * (2 * SEL_THREADS / 64) + threadIdx.x / 64;
  auto vec = [&](int64_t c) { return x[c * (nvec - 64) / (SAMPLE_RUNS - 1) + (threadIdx.x & 63)]; };
  const u32x4 r[2] = {vec(run), vec(run + SEL_THREADS / 64)};
#pragma unroll
  for (int v = 0; v < 2; ++v)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      atomicAdd(&hrep[key_of<BF16>(r[v][e] & 0xffffu) >> 5], 1u);
      atomicAdd(&hrep[key_of<BF16>(r[v][e] >> 16) >> 5], 1u);
    }
  __syncthreads();
  for (int i = threadIdx.x; i < SEL_BINS; i += SEL_THREADS) {
    uint32_t v = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) v += h[q * SEL_BINS + i];
    if (v) atomicAdd(&hist[SAMPLE_AT + i], (unsigned long long)v);
  }
}

// A wave per row.
__global__ __launch_bounds__(1024) void win_count_kernel(const uint16_t* x, int64_t rows, int64_t cols, Ranks sample, const unsigned long long* digits,
                                                         SelState* st, unsigned long long* hist, uint16_t* row_bins) {
  __shared__ uint32_t tab[16][WIN_LDS];
  __shared__ uint32_t total[WIN_LDS + 2];
  uint32_t digit[2];
  Ranks left;
  find_bins<1024, SEL_BINS, 0>(digits, sample, digit, left);
  const Windows win(digit);
  if (blockIdx.x == 0 && threadIdx.x == 0) { st->window[0] = win.w0; st->window[1] = win.w1; }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t* const t = tab[wave];
#pragma unroll
  for (int j = 0; j < WIN_LDS / 64; ++j) t[lane + 64 * j] = 0;
  if (threadIdx.x < WIN_LDS + 2) total[threadIdx.x] = 0;
  __syncthreads();
  typedef short s16x2 __attribute__((ext_vector_type(2)));
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  uint32_t sum[WIN_LDS / 64] = {};
  u16x2 top = {0, 0};   // largest magnitude
  // Sums of 0 / 1 / 1 and of 0 / 1 / 2 for -0, +0 and the rest.  16 bits hold them: a half word meets 4 elements for every 512 begun of a row, in
  // ceil(rows / 8192) rows, rows have 500 elements or more (row_bins has to fit the entries' room) and the tensor fewer than 2^32: at most
  // 2^13 + 2^10 elements.
  u16x2 nz1 = {0, 0}, nz2 = {0, 0};
  const uint16_t lo1 = (uint16_t)(win.w0 - 1), hi1 = (uint16_t)(win.w1 - 1), most = WIN_KEYS + 1;
  const u16x2 lo = {lo1, lo1}, hi = {hi1, hi1}, lim = {most, most};
  auto all_rows = [&](auto zeros) {
    constexpr bool ZEROS = decltype(zeros)::value;
    auto visit = [&](uint32_t bin) {
      if (bin != WIN_KEYS + 1 && (!ZEROS || bin < WIN_BINS)) atomicAdd(&t[bin], 1u);
    };
    auto visit_vec = [&](const u32x4& r) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {   // two elements at a time: keys as key_of, then how far they are into either window
        const uint32_t p = r[e];
        const s16x2 sign = __builtin_bit_cast(s16x2, p) >> (short)15;
        const u16x2 key = __builtin_bit_cast(u16x2, p ^ (__builtin_bit_cast(uint32_t, sign) | 0x80008000u));
        top = __builtin_elementwise_max(top, __builtin_bit_cast(u16x2, p & 0x7fff7fffu));
        u16x2 bin = __builtin_elementwise_min(__builtin_elementwise_sub_sat(key, lo), lim) +
                    __builtin_elementwise_min(__builtin_elementwise_sub_sat(key, hi), lim);
        if constexpr (ZEROS) {   // half of the elements on one word of a table: the atomics would wait for each other
          const u16x2 d = key - (u16x2){KEY_NEG_ZERO, KEY_NEG_ZERO}, one = {1, 1}, two = {2, 2};
          const u16x2 d2 = __builtin_elementwise_min(d, two);
          nz1 += __builtin_elementwise_min(d, one);
          nz2 += d2;
          bin |= (d2 ^ two) << (u16x2){8, 8};   // past the bins
        }
        visit(bin.x);
        visit(bin.y);
        // a pair at a time, or the sums become trees and a CU has registers for one workgroup instead of two
        if constexpr (ZEROS) asm volatile("" : "+v"(nz1), "+v"(nz2));
      }
    };
    const int nvec = (int)(cols / 8);
    for (int64_t row = (int64_t)blockIdx.x * 16 + wave; row < rows; row += (int64_t)gridDim.x * 16) {
      const u32x4* const xr = reinterpret_cast<const u32x4*>(x + row * cols);
      int i = lane;
      for (; i + 3 * 64 < nvec; i += 4 * 64) {
        const u32x4 r0 = xr[i], r1 = xr[i + 64], r2 = xr[i + 128], r3 = xr[i + 192];
        visit_vec(r0); visit_vec(r1); visit_vec(r2); visit_vec(r3);
      }
      for (; i < nvec; i += 64) visit_vec(xr[i]);
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the table is this wave's own
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int j = 0; j < WIN_LDS / 64; ++j) {
        const uint32_t v = t[lane + 64 * j];
        t[lane + 64 * j] = 0;
        sum[j] += v;
        if (lane + 64 * j < WIN_BINS) row_bins[row * WIN_STRIDE + lane + 64 * j] = (uint16_t)v;
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      __builtin_amdgcn_wave_barrier();
    }
  };
  const bool zeros_apart = win.zeros_apart();
  if (zeros_apart) all_rows(std::true_type{});
  else all_rows(std::false_type{});
#pragma unroll
  for (int j = 0; j < WIN_LDS / 64; ++j)
    if (sum[j]) atomicAdd(&total[lane + 64 * j], sum[j]);
  if (zeros_apart) {
    atomicAdd(&total[WIN_LDS], (uint32_t)nz1.x + nz1.y);
    atomicAdd(&total[WIN_LDS + 1], (uint32_t)nz2.x + nz2.y);
  }
  if (max(top.x, top.y) > 0x7f80) st->nan = 1;
  __syncthreads();
  if (threadIdx.x < WIN_LDS + 2 && total[threadIdx.x]) atomicAdd(&hist[WIN_AT + threadIdx.x], (unsigned long long)total[threadIdx.x]);
}

template <class DT, int PASS, bool BEHIND>
__global__ __launch_bounds__(SEL_THREADS) void sel_hist_kernel(const void* x, int64_t rows, int64_t cols, int64_t ld, Ranks ranks,
                                                               SelState* st, unsigned long long* hist, float* thresholds) {
  __shared__ SelTable<DT, PASS> table;
  sel_hist<DT, PASS, BEHIND>(x, rows, cols, ld, ranks, st, hist, thresholds, blockIdx.x, gridDim.x, table);
}

// ---- Outliers of each row, and of each block of 4 << shift rows -----------------------------------------------------------
// Eight elements of a row as loaded.
template <class DT> struct Unit { u32x4 r[__is_same(DT, BF16) ? 1 : 2]; };
template <class DT>
FP4_D void load_unit(const void* x, int64_t off, int valid, Unit<DT>& u) {
  constexpr int E = __is_same(DT, BF16) ? 2 : 4;   // bytes an element
  const uint8_t* const p = reinterpret_cast<const uint8_t*>(x) + off * E;
  if (valid >= 8) {
#pragma unroll
    for (int q = 0; q < E / 2; ++q) u.r[q] = reinterpret_cast<const u32x4*>(p)[q];
  } else {
    uint32_t w[2 * E] = {};
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      if (e >= valid) continue;
      if constexpr (E == 2) w[e / 2] |= (uint32_t)reinterpret_cast<const uint16_t*>(p)[e] << (16 * (e & 1));
      else w[e] = reinterpret_cast<const uint32_t*>(p)[e];
    }
#pragma unroll
    for (int q = 0; q < 2 * E; ++q) u.r[q / 4][q % 4] = w[q];
  }
}
template <class DT>
FP4_D int count_unit(const Unit<DT>& u, int valid, float lo, float hi) {
  int cnt = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    float v;
    if constexpr (__is_same(DT, BF16)) v = u2f((e & 1) ? u.r[0][e / 2] & 0xffff0000u : u.r[0][e / 2] << 16);
    else v = u2f(u.r[e / 4][e % 4]);
    cnt += (e < valid && ((v < lo) | (v > hi))) ? 1 : 0;
  }
  return cnt;
}

struct RowCounts { int32_t *cnt, *sum; int shift; };   // sum[b]: of rows b * (4 << shift) ..

FP4_D int wave_sum(int v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// A wave per row and four at a time; find(thr) gives the thresholds to all threads, while the first elements are on their way.
template <class DT, class F>
FP4_D void count_rows(const void* x, int64_t rows, int64_t cols, int64_t ld, const RowCounts& out, F&& find) {
  __shared__ int s_sum[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, per = 1 << out.shift;
  const int64_t row0 = ((int64_t)blockIdx.x * 4 + wave) * per;
  const int nrows = (int)min((int64_t)per, rows - row0);   // may be <= 0
  const int64_t nunits = (cols + 7) / 8;
  const int steps = (int)((nunits + 255) / 256);           // of four units a lane
  auto valid_of = [&](int step, int q) {
    const int64_t unit = (int64_t)step * 256 + q * 64 + lane;
    return unit < nunits ? (int)min((int64_t)8, cols - unit * 8) : 0;
  };
  // whether a lane has anything of the wave's q-th units: a branch that all take, where a short row's three absent units of four cost
  // as much as the one it has (clamp alone, 32768 x 64 bf16 71.5 -> 62.0 us, 65536 x 64 111 -> 93)
  auto is_there = [&](int step, int q) { return (int64_t)step * 256 + q * 64 < nunits; };
  Unit<DT> u[4];
  auto fetch = [&](int row, int step) {
    if (row >= nrows) return;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (is_there(step, q)) load_unit<DT>(x, (row0 + row) * ld + ((int64_t)step * 256 + q * 64 + lane) * 8, valid_of(step, q), u[q]);
  };
  fetch(0, 0);
  float thr[2];
  find(thr);
  int sum = 0;
  for (int row = 0; row < nrows; ++row) {
    int cnt = 0;
    for (int step = 0; step < steps; ++step) {
      const Unit<DT> c[4] = {u[0], u[1], u[2], u[3]};
      if (step + 1 < steps) fetch(row, step + 1);
      else fetch(row + 1, 0);
#pragma unroll
      for (int q = 0; q < 4; ++q)
        if (is_there(step, q)) cnt += count_unit<DT>(c[q], valid_of(step, q), thr[0], thr[1]);
    }
    cnt = wave_sum(cnt);
    if (lane == 0) out.cnt[row0 + row] = cnt;
    sum += cnt;
  }
  if (lane == 0) s_sum[wave] = sum;
  __syncthreads();
  if (threadIdx.x == 0) out.sum[blockIdx.x] = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
}

// After the last digit pass: the thresholds, to memory as well, and the counts.
template <class DT>
FP4_D void find_thresholds(SelState* st, const unsigned long long* hist, const Ranks& ranks, float* thresholds, float (&thr)[2]) {
  uint32_t key[2];
  find_digit<DT, sel_digits<DT>(), 256>(st, hist, ranks, false, key);
  thr[0] = value_of<DT>(key[0]);
  thr[1] = value_of<DT>(key[1]);
  if (blockIdx.x == 0 && threadIdx.x < 2) thresholds[threadIdx.x] = thr[threadIdx.x];
}

// FOUND: sel_pick_kernel has found the thresholds.
template <class DT, bool FOUND>
__global__ __launch_bounds__(256) void sel_count_kernel(const void* x, int64_t rows, int64_t cols, int64_t ld, Ranks ranks, SelState* st,
                                                        const unsigned long long* hist, float* thresholds, RowCounts out) {
  count_rows<DT>(x, rows, cols, ld, out, [&](float (&thr)[2]) {
    if constexpr (FOUND) { thr[0] = thresholds[0]; thr[1] = thresholds[1]; }
    else find_thresholds<DT>(st, hist, ranks, thresholds, thr);
  });
}

// More rows than have their sums taken: a wave a row, nothing more (131072 x 64 bf16 25 us, with eight rows
// a wave and their sums, which nothing reads, 91).
template <class DT>
__global__ __launch_bounds__(256) void sel_count_apart_kernel(const void* x, int64_t rows, int64_t cols, int64_t ld, const float* thresholds,
                                                              int32_t* row_cnt) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const float lo = thresholds[0], hi = thresholds[1];
  int cnt = 0;
  for (int64_t unit = lane; unit < (cols + 7) / 8; unit += 64) {
    const int valid = (int)min((int64_t)8, cols - unit * 8);
    Unit<DT> u;
    load_unit<DT>(x, row * ld + unit * 8, valid, u);
    cnt += count_unit<DT>(u, valid, lo, hi);
  }
  cnt = wave_sum(cnt);
  if (lane == 0) row_cnt[row] = cnt;
}

template <class DT>
__global__ __launch_bounds__(256) void sel_pick_kernel(SelState* st, const unsigned long long* hist, Ranks ranks, float* thresholds) {
  float thr[2];
  find_thresholds<DT>(st, hist, ranks, thresholds, thr);
}

__global__ __launch_bounds__(256) void sel_clear_kernel(unsigned long long* clear, const float* src, float* dst, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (clear && i < SEL_CLEAR) clear[i] = 0;
  if (i < n) dst[i] = src[i];
}

// Outliers of each row: from its bins, or, where these don't tell, from its elements.  EXACT: the windows hold the thresholds, which are
// still to be found; otherwise the digit passes have run.
template <bool EXACT>
__global__ __launch_bounds__(256) void win_rows_kernel(const uint16_t* x, int64_t rows, int64_t cols, Ranks ranks, SelState* st,
                                                       const unsigned long long* hist, const uint16_t* row_bins, float* thresholds, RowCounts out) {
  uint32_t key[2] = {}, bin[2] = {st->bin[0], st->bin[1]};
  const bool ok = EXACT ? find_windowed(st, hist, ranks, rows * cols, key, bin) : st->done != 0;
  if (EXACT && blockIdx.x == 0 && threadIdx.x < 2) thresholds[threadIdx.x] = value_of<BF16>(threadIdx.x ? key[1] : key[0]);
  if (!ok) {
    count_rows<BF16>(x, rows, cols, cols, out, [&](float (&thr)[2]) {
      if constexpr (EXACT) { thr[0] = value_of<BF16>(key[0]); thr[1] = value_of<BF16>(key[1]); }
      else find_thresholds<BF16>(st, hist, ranks, thresholds, thr);
    });
    return;
  }
  __shared__ int s_sum[4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, per = 1 << out.shift;
  const int b0 = (int)bin[0], b1 = (int)bin[1];
  const int64_t row0 = ((int64_t)blockIdx.x * 4 + wave) * per;
  int sum = 0;
  for (int j = 0; j < per; ++j) {
    const int64_t row = row0 + j;
    int cnt = 0;
    if (row < rows)
#pragma unroll
      for (int q = 0; q < WIN_LDS / 64; ++q) {
        const int b = lane + 64 * q;
        if (b < b0 || (b > b1 && b < WIN_BINS)) cnt += row_bins[row * WIN_STRIDE + b];
      }
    cnt = wave_sum(cnt);
    if (lane == 0 && row < rows) out.cnt[row] = cnt;
    sum += cnt;
  }
  if (lane == 0) s_sum[wave] = sum;
  __syncthreads();
  if (threadIdx.x == 0) out.sum[blockIdx.x] = s_sum[0] + s_sum[1] + s_sum[2] + s_sum[3];
}

// ---- CSR finalisation ---------------------------------------------------------------------
// ptr[0] = 0, ptr[i+1] = sum cnt[0..i]; optional copy of the total.  A workgroup for 1024 counts, which adds up those before them
// for itself: up to 64 Ki counts, from L2, 16 bytes a thread at a time.  One workgroup for all of them wrote 16 strided runs a thread:
// 8192 counts 6.6 -> 4.9 us, 16384 11.0 -> 5.1.
constexpr int64_t SCAN_WIDE = 65536;
__global__ __launch_bounds__(1024) void scan_counts_wide_kernel(const int32_t* cnt, int64_t n, int64_t* ptr, int64_t* total_out) {
  __shared__ long long s_before[16], s_w[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t b0 = (int64_t)blockIdx.x * 1024, i = b0 + tid;
  const long long mine = i < n ? cnt[i] : 0;
  long long before = 0;
#pragma unroll 4
  for (int64_t j = (int64_t)tid * 4; j < b0; j += 4096) {   // b0 is a multiple of 4
    const i32x4 t = *reinterpret_cast<const i32x4*>(cnt + j);
    before += (long long)t.x + t.y + t.z + t.w;
  }
  long long incl = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const long long up = __shfl_up(incl, o, 64);
    if (lane >= o) incl += up;
    before += __shfl_xor(before, o, 64);
  }
  if (lane == 63) { s_w[wave] = incl; s_before[wave] = before; }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    const long long t = s_w[w];
    incl += s_before[w];
    if (w < wave) incl += t;
  }
  if (i < n) ptr[i + 1] = incl;
  if (i == 0) ptr[0] = 0;
  if (i == n - 1 && total_out) *total_out = incl;
}

// ptr[0] = 0, ptr[i+1] = sum cnt[0..i]; optional copy of the total.  One workgroup; a thread
// takes 16 consecutive counts, so one block scan covers 16384 of them.
__global__ __launch_bounds__(1024) void scan_counts_kernel(const int32_t* cnt, int64_t n, int64_t* ptr,
                                                           int64_t* total_out) {
  __shared__ long long s_w[16];
  __shared__ long long carry;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (threadIdx.x == 0) { carry = 0; ptr[0] = 0; }
  __syncthreads();
  for (int64_t base = 0; base < n; base += 16 * 1024) {
    const int64_t i0 = base + (int64_t)threadIdx.x * 16;
    int32_t c[16];
    if (i0 + 16 <= n) {   // 64 aligned bytes: four loads in flight instead of sixteen guarded ones in a row
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const i32x4 t = reinterpret_cast<const i32x4*>(cnt + i0)[q];
        c[4 * q] = t.x; c[4 * q + 1] = t.y; c[4 * q + 2] = t.z; c[4 * q + 3] = t.w;
      }
    } else {
#pragma unroll
      for (int j = 0; j < 16; ++j) c[j] = i0 + j < n ? cnt[i0 + j] : 0;
    }
    long long v[16];
    long long sum = 0;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      sum += c[j];
      v[j] = sum;   // inclusive inside the thread
    }
    long long incl = sum;   // inclusive over the wave
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const long long up = __shfl_up(incl, o, 64);
      if (lane >= o) incl += up;
    }
    if (lane == 63) s_w[wave] = incl;
    __syncthreads();
    long long before = carry + incl - sum;
    for (int w = 0; w < wave; ++w) before += s_w[w];
#pragma unroll
    for (int j = 0; j < 16; ++j)
      if (i0 + j < n) ptr[i0 + j + 1] = before + v[j];
    __syncthreads();
    if (threadIdx.x == 1023) carry = before + sum;
    __syncthreads();
  }
  if (threadIdx.x == 0 && total_out) *total_out = carry;
}

// One wave per row: move the row's temporary entries to their canonical place (same segment
// of the final arrays), ascending column order (rank of a column among the row's columns; columns are distinct).
__global__ __launch_bounds__(256) void csr_gather_kernel(const int32_t* tmp_col, const float* tmp_val,
                                                         const int64_t* row_ptr, int64_t rows, int64_t capacity,
                                                         int32_t* col_idx, float* val) {
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= rows) return;
  const int64_t src = row_ptr[row];
  const int64_t en = row_ptr[row + 1];
  if (en > capacity) return;  // truncated output, nnz tells
  const int L = (int)(en - src);
  for (int i = lane; i < L; i += 64) {
    const int32_t c = tmp_col[src + i];
    int rank = 0;
    for (int j = 0; j < L; ++j) rank += tmp_col[src + j] < c ? 1 : 0;
    col_idx[src + rank] = c;
    val[src + rank] = tmp_val[src + i];
  }
}

}  // namespace

// ---- internal launchers -----------------------------------------------------------------------
int fp4_row_sum_shift(int64_t rows);
int64_t fp4_row_sum_most();
size_t fp4_select_scratch_bytes() { return SEL_CLEAR * 8; }
int64_t fp4_select_clear_words() { return SEL_CLEAR; }

// Clears a selection's scratch (null: none) and copies n floats: what a layer does ahead of its passes, in one launch.
int fp4_launch_clear_select(void* scratch, const float* src, float* dst, int64_t n, hipStream_t s) {
  const int64_t most = std::max<int64_t>(scratch ? SEL_CLEAR : 0, n);
  if (most == 0) return FP4_OK;
  hipLaunchKernelGGL(sel_clear_kernel, dim3((unsigned)((most + 255) / 256)), dim3(256), 0, s, reinterpret_cast<unsigned long long*>(scratch),
                     src, dst, n);
  FP4_CHECK_LAUNCH();
  return FP4_OK;
}

// Which passes find the thresholds: bits of fp4_select_route (fp4_measure.h).
//
// The pass with windows has a wave a row and sixteen rows a workgroup, so few long rows leave most of the chip without one, and where zeros are
// counted apart (rectified tensors, whose lower threshold is zero) it takes half as long again; digit passes spread over the chip whatever
// the shape.  Clamp alone in us, N(0, 1) and rectified, windows / digits, and what both took when the digits' bins were picked in launches of their
// own: 64 x 2048 24 and 31 / 24 and 26, 31 and 34; 64 x 13824 42 and 59 / 39 and 41, 47 and 49; 256 x 8192 37 and 49 / 42 and 44, 47 and 49; 256 x
// 13824 47 and 63 / 49 and 51, 54 and 56; 1024 x 28672 106 and 150 / 121 and 159, 125 and 160.  From 2^25 elements on the sample takes a digit pass's
// place (16384 x 4096 above).
constexpr int64_t WIN_COLS_PER_ROW = 32;
static unsigned count_blocks(int64_t rows, int shift) { return (unsigned)((rows + (4 << shift) - 1) / (4 << shift)); }
int fp4_select_passes(int bf16, int64_t rows, int64_t cols, int64_t ld, int64_t rows_scratch_words) {
  const int64_t n = rows * cols;
  int route = 0;
  if (bf16 && ld == cols && cols % 8 == 0 && cols <= 65535 && n < ((int64_t)1 << 32) && rows * WIN_STRIDE <= 2 * rows_scratch_words) {
    if (n >= ((int64_t)1 << 25)) route |= FP4_SELECT_SAMPLE | FP4_SELECT_WINDOWS;
    else if (cols <= WIN_COLS_PER_ROW * rows) route |= FP4_SELECT_WINDOWS;
  }
  if (!route && rows > fp4_row_sum_most()) route |= FP4_SELECT_FOUND | FP4_SELECT_APART;
  if (bf16 && !route && count_blocks(rows, fp4_row_sum_shift(rows)) > SEL_FIND_BLOCKS) route |= FP4_SELECT_FOUND;
  return route;
}

// Whether the selection begins with a first digit pass over all elements, which may then be launched elsewhere.
bool fp4_select_begins_with_digits(int bf16, int64_t rows, int64_t cols, int64_t ld, int64_t rows_scratch_words) {
  return !(fp4_select_passes(bf16, rows, cols, ld, rows_scratch_words) & FP4_SELECT_SAMPLE);
}

// Thresholds lo = v[k], hi = v[n-1-k] of the ascending-sorted tensor into thresholds[0..1], then the outliers of each row (row_cnt) and
// of each block of 4 << shift rows (row_sum; up to fp4_row_sum_most() rows).  scratch: fp4_select_scratch_bytes(), cleared; first_done: but
// for the first digit's bins, whose pass has run.  rows_scratch: words that are free until
// the rows' entries are emitted.
int fp4_launch_thresholds_and_counts(const void* x, int bf16, int64_t rows, int64_t cols, int64_t ld, int64_t k, float* thresholds,
                                     void* scratch, void* rows_scratch, int64_t rows_scratch_words, int32_t* row_cnt, int32_t* row_sum,
                                     int shift, bool first_done, hipStream_t s) {
  SelState* const st = reinterpret_cast<SelState*>(scratch);
  unsigned long long* const hist = reinterpret_cast<unsigned long long*>(reinterpret_cast<uint8_t*>(scratch) + SEL_STATE_BYTES);
  const int64_t n = rows * cols;
  const Ranks ranks = {{(unsigned long long)k, (unsigned long long)(n - 1 - k)}};
  const RowCounts out = {row_cnt, row_sum, shift};
  const unsigned count_grid = count_blocks(rows, shift);
  const unsigned grid = sel_blocks(n);
  auto digit = [&](auto dt, auto pass, auto behind) {
    hipLaunchKernelGGL((sel_hist_kernel<decltype(dt), decltype(pass)::value, decltype(behind)::value>), dim3(grid), dim3(SEL_THREADS), 0, s, x,
                       rows, cols, ld, ranks, st, hist, thresholds);
  };
  using First = std::integral_constant<int, 0>;
  using Second = std::integral_constant<int, 1>;
  using Third = std::integral_constant<int, 2>;
  const int route = fp4_select_passes(bf16, rows, cols, ld, rows_scratch_words);
  if (route & FP4_SELECT_WINDOWS) {
    uint16_t* const bins = reinterpret_cast<uint16_t*>(rows_scratch);
    const uint16_t* const xp = reinterpret_cast<const uint16_t*>(x);
    auto window = [&](const Ranks& r, const unsigned long long* digits) {
      hipLaunchKernelGGL(win_count_kernel, dim3((unsigned)std::min<int64_t>((rows + 15) / 16, 512)), dim3(1024), 0, s, xp, rows, cols, r, digits,
                         st, hist, bins);
    };
    auto counts = [&](auto exact) {
      hipLaunchKernelGGL((win_rows_kernel<decltype(exact)::value>), dim3(count_grid), dim3(256), 0, s, xp, rows, cols, ranks, st, hist, bins,
                         thresholds, out);
    };
    if (route & FP4_SELECT_SAMPLE) {
      const int64_t ns = (int64_t)SAMPLE_RUNS * 64 * 8;
      const unsigned long long ks = (unsigned long long)((double)k / (double)n * (double)ns);
      hipLaunchKernelGGL(sel_sample_kernel, dim3(SAMPLE_BLOCKS), dim3(SEL_THREADS), 0, s, reinterpret_cast<const u32x4*>(x), n / 8, hist);
      window({{ks, (unsigned long long)ns - 1 - ks}}, hist + SAMPLE_AT);   // the sample's ranks
      digit(BF16{}, First{}, std::true_type{});
      digit(BF16{}, Second{}, std::true_type{});
      counts(std::false_type{});
    } else {
      if (!first_done) digit(BF16{}, First{}, std::false_type{});
      window(ranks, hist + SEL_AT[0]);
      counts(std::true_type{});
    }
  } else {
    auto count = [&](auto dt) {
      using DT = decltype(dt);
      if (route & FP4_SELECT_FOUND) hipLaunchKernelGGL((sel_pick_kernel<DT>), dim3(1), dim3(256), 0, s, st, hist, ranks, thresholds);
      if (route & FP4_SELECT_APART)
        hipLaunchKernelGGL((sel_count_apart_kernel<DT>), dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, x, rows, cols, ld, thresholds, row_cnt);
      else if (route & FP4_SELECT_FOUND)
        hipLaunchKernelGGL((sel_count_kernel<DT, true>), dim3(count_grid), dim3(256), 0, s, x, rows, cols, ld, ranks, st, hist, thresholds, out);
      else
        hipLaunchKernelGGL((sel_count_kernel<DT, false>), dim3(count_grid), dim3(256), 0, s, x, rows, cols, ld, ranks, st, hist, thresholds, out);
    };
    if (bf16) {
      if (!first_done) digit(BF16{}, First{}, std::false_type{});
      digit(BF16{}, Second{}, std::false_type{});
      count(BF16{});
    } else {
      if (!first_done) digit(F32{}, First{}, std::false_type{});
      digit(F32{}, Second{}, std::false_type{});
      digit(F32{}, Third{}, std::false_type{});
      count(F32{});
    }
  }
  FP4_CHECK_LAUNCH();
  return FP4_OK;
}

int fp4_launch_scan_rows(const int32_t* row_cnt, int64_t rows, int64_t* row_ptr, int64_t* nnz, hipStream_t s) {
  if (rows > 0 && rows <= SCAN_WIDE && aligned16(row_cnt))
    hipLaunchKernelGGL(scan_counts_wide_kernel, dim3((unsigned)((rows + 1023) / 1024)), dim3(1024), 0, s, row_cnt, rows, row_ptr, nnz);
  else
    hipLaunchKernelGGL(scan_counts_kernel, dim3(1), dim3(1024), 0, s, row_cnt, rows, row_ptr, nnz);
  FP4_CHECK_LAUNCH();
  return FP4_OK;
}

int fp4_launch_csr_gather(const int32_t* tmp_col, const float* tmp_val, int64_t rows, int64_t capacity,
                          const int64_t* row_ptr, int32_t* col_idx, float* val, hipStream_t s) {
  hipLaunchKernelGGL(csr_gather_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, tmp_col, tmp_val,
                     row_ptr, rows, capacity, col_idx, val);
  FP4_CHECK_LAUNCH();
  return FP4_OK;
}
