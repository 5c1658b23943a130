// Exact order statistics by radix selection on order-preserving keys: digit passes over the elements and what finds the bins behind them
// (occ.hip launches them; the first pass over a layer's activations also runs beside the quantization of its weights, quantize.hip).
#pragma once
#include "fp4_common.h"

#include <cstddef>

// A selection's first digit pass, launched beside something else.
struct SelFirst {
  const void* x;
  int64_t rows, cols, ld;
  unsigned long long* hist;   // cleared by an earlier launch
};

namespace {

constexpr int SEL_BINS = 2048;  // 11-bit digits
constexpr int SEL_THREADS = 1024;   // per workgroup: the 64 KiB of LDS tables allow two workgroups per CU,
                                    // so their size decides how many loads a CU has in flight

// A digit pass: a workgroup for every 8192 elements up to 256 of them, for every 65536 up to 512 (64 x 2048 bf16, one for
// every 8192 / 65536: 8.5 / 9.2 us; 1056 x 1376 7.1 / 10.2; 8192 x 2048, 512 / 256: 18.1 / 15.6, each adds its bins to the same words).
//
// The bins that hold the two ranks are found by whoever needs them next: every workgroup of the next digit's pass, and of the
// count behind the last, scans them again while its first elements are on their way: 2 to 3 us, where a launch of one workgroup took
// 4.5 and its gap.  So each digit has bins of its own in memory, all cleared before the first.  The count behind bf16's second digit
// does so with up to SEL_FIND_BLOCKS workgroups only: its 64 bins lie in four lines, and a thousand workgroups that ask for them at once take
// 20 us (clamp alone of 64 / 128 / 256 / 1024 / 8192 rows of 64, found by the count 20.6 / 22.9 / 25.2 / 34.1 / 43.7 us, in a launch of its own 21.0 /
// 21.8 / 22.0 / 22.2 / 31.7).  fp32's 1024 bins a threshold lie in many: 1024 rows of 64 27.3 / 28.1, 8192 of 2048 94.3 / 93.1, 16384 of 2048 145.6 / 147.8.
constexpr unsigned SEL_FIND_BLOCKS = 16;
constexpr int SEL_AT[3] = {0, SEL_BINS, 3 * SEL_BINS};      // where a digit's bins begin (the first's are shared by both targets)
constexpr int SEL_APART[3] = {0, SEL_BINS, SEL_BINS / 2};   // from one target's bins to the other's
constexpr int SEL_WORDS = 4 * SEL_BINS;
// bf16: 11 + 5 bits; fp32: 11 + 11 + 10
template <class DT> constexpr int sel_digits() { return __is_same(DT, BF16) ? 2 : 3; }
template <class DT> constexpr int sel_bits(int pass) { return pass == 0 ? 11 : __is_same(DT, BF16) ? 5 : pass == 1 ? 11 : 10; }
template <class DT> constexpr int sel_shift(int pass) {   // bits below a digit
  int at = __is_same(DT, BF16) ? 16 : 32;
  for (int p = 0; p <= pass; ++p) at -= sel_bits<DT>(p);
  return at;
}

// Workgroups of a digit pass (above).
inline unsigned sel_blocks(int64_t n) {
  const int64_t few = (n + 8191) / 8192 < 256 ? (n + 8191) / 8192 : 256, many = (n + 65535) / 65536 < 512 ? (n + 65535) / 65536 : 512;
  return (unsigned)(few > many ? few : many > 1 ? many : 1);
}

struct Ranks { unsigned long long v[2]; };   // 0-based, of the lo / hi order statistic

// Selection state kept in the workspace between passes.
struct SelState {
  unsigned long long rank[2];  // remaining ranks after the first digit
  uint32_t prefix[2];          // key bits fixed by then (right-aligned)
  // windows (below): their first keys; thresholds and row counts came out of one pass; a NaN was met; the thresholds' bins
  uint32_t window[2], unused, done, nan, bin[2];
  uint32_t prefix2[2];         // after the second digit
  unsigned long long rank2[2];
};
static_assert(offsetof(SelState, done) == 9 * 4, "the tests read it there");
constexpr int SEL_STATE_BYTES = 256;   // the state's place, before the bins
constexpr int SEL_CLEAR = (SEL_STATE_BYTES + SEL_WORDS * 8) / 8;   // 8-byte words, state and bins, that are 0 when a selection begins

template <class DT>
FP4_D uint32_t key_of(uint32_t raw) {   // raw: bf16 bits (low 16) or fp32 bits
  if constexpr (__is_same(DT, BF16)) return f32_order_key(raw << 16) >> 16;
  else return f32_order_key(raw);
}
template <class DT>
FP4_D float value_of(uint32_t key) {
  // 16-bit keys are the top half of the fp32 key of a bf16 value; undo the map on
  // 16 bits so the low half of the fp32 pattern stays zero
  if constexpr (__is_same(DT, BF16)) return u2f(((key & 0x8000u) ? (key & 0x7fffu) : (~key & 0xffffu)) << 16);
  else return u2f(f32_from_order_key(key));
}

template <class T>
FP4_D T scan_lanes(T v, int width) {   // inclusive, over groups of `width` lanes
  const int at = threadIdx.x & (width - 1);
#pragma unroll
  for (int o = 1; o < width; o <<= 1) {
    const T up = __shfl_up(v, o, width);
    if (at >= o) v += up;
  }
  return v;
}

// For each of the two targets the bin that holds its rank, of NB bins each (APART words from the other's, 0: they share one histogram),
// and its rank in there.  By all THREADS of a workgroup; of 32 bins by one wave of it (every wave for itself: 8192 x 2048, the count
// 22.1 us instead of 10.9; all that are under way ask one memory channel for the same two lines).
template <int THREADS, int NB, int APART>
FP4_D void find_bins(const unsigned long long* hist, const Ranks& ranks, uint32_t (&bin)[2], Ranks& left) {
  const int tid = threadIdx.x, lane = tid & 63;
  if constexpr (NB == 32) {
    __shared__ unsigned long long s_left[2];
    __shared__ uint32_t s_bin[2];
    if (tid < 64) {
      const unsigned long long v = hist[(lane >> 5) * APART + (lane & 31)], incl = scan_lanes(v, 32), excl = incl - v;
      const unsigned long long r = lane < 32 ? ranks.v[0] : ranks.v[1];
      // the bin whose range [excl, incl) holds the rank (the last, should the rank lie beyond the total)
      if ((excl <= r && r < incl) || ((lane & 31) == 31 && r >= incl)) { s_bin[lane >> 5] = (uint32_t)(lane & 31); s_left[lane >> 5] = r - excl; }
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < 2; ++s) { bin[s] = s_bin[s]; left.v[s] = s_left[s]; }
  } else {
    constexpr int PER = NB / THREADS, WAVES = THREADS / 64, SETS = APART ? 2 : 1;
    static_assert(PER >= 1 && NB % THREADS == 0, "a thread owns whole bins");
    __shared__ unsigned long long s_w[SETS][WAVES], s_left[2];
    __shared__ uint32_t s_bin[2];
    unsigned long long v[SETS][PER], sum[SETS], incl[SETS];
#pragma unroll
    for (int q = 0; q < SETS; ++q)
#pragma unroll
      for (int j = 0; j < PER; ++j) v[q][j] = hist[q * APART + tid * PER + j];
#pragma unroll
    for (int q = 0; q < SETS; ++q) {
      sum[q] = 0;
#pragma unroll
      for (int j = 0; j < PER; ++j) sum[q] += v[q][j];
      incl[q] = scan_lanes(sum[q], 64);
      if (lane == 63) s_w[q][tid >> 6] = incl[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < SETS; ++q)
#pragma unroll
      for (int w = 0; w < WAVES; ++w) {   // all of them requested at once
        const unsigned long long ws = s_w[q][w];
        if (w < (tid >> 6)) incl[q] += ws;
      }
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int q = SETS == 2 ? s : 0;
      const unsigned long long r = ranks.v[s], excl = incl[q] - sum[q];
      if ((excl <= r && r < incl[q]) || (tid == THREADS - 1 && r >= incl[q])) {
        unsigned long long cum = excl;
        int j = 0;
#pragma unroll
        for (int b = 0; b < PER - 1; ++b)
          if (j == b && cum + v[q][b] <= r) { cum += v[q][b]; ++j; }
        s_bin[s] = (uint32_t)(tid * PER + j);
        s_left[s] = r - cum;
      }
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < 2; ++s) { bin[s] = s_bin[s]; left.v[s] = s_left[s]; }
  }
}

// What digit pass PASS - 1 found: the keys' leading bits, and the ranks that remain.  keep: left in memory for the passes after this.
template <class DT, int PASS, int THREADS>
FP4_D void find_digit(SelState* st, const unsigned long long* hist, const Ranks& ranks, bool keep, uint32_t (&prefix)[2]) {
  constexpr int D = PASS - 1;
  Ranks in = ranks, left;
  if constexpr (D > 0)
    for (int s = 0; s < 2; ++s) in.v[s] = D == 1 ? st->rank[s] : st->rank2[s];
  uint32_t bin[2];
  find_bins<THREADS, 1 << sel_bits<DT>(D), SEL_APART[D]>(hist + SEL_AT[D], in, bin, left);
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    prefix[s] = D == 0 ? bin[s] : ((D == 1 ? st->prefix[s] : st->prefix2[s]) << sel_bits<DT>(D)) | bin[s];
    if (keep && threadIdx.x == 0) {
      if (D == 0) { st->prefix[s] = prefix[s]; st->rank[s] = left.v[s]; }
      else { st->prefix2[s] = prefix[s]; st->rank2[s] = left.v[s]; }
    }
  }
}

constexpr int WIN_KEYS = 96, WIN_BINS = 2 * WIN_KEYS + 3, WIN_LDS = 256, WIN_STRIDE = 200;   // bins; a wave's table; a row's in memory
// in memory: the sample's bins and the windows', beside the digits'
constexpr int SAMPLE_AT = SEL_AT[2], WIN_AT = SEL_AT[1] + 64;
constexpr uint32_t KEY_NEG_ZERO = 0x7fff, KEY_POS_ZERO = 0x8000;
constexpr int SAMPLE_BLOCKS = 128, SAMPLE_RUNS = SAMPLE_BLOCKS * 2 * (SEL_THREADS / 64);   // runs of 64 16-byte vectors

// First keys of the windows, from the digits that the sample's order statistics have.  Windows that would meet lie side by
// side, and either threshold may be in either.
struct Windows {
  uint32_t w0, w1;
  FP4_D explicit Windows(const uint32_t (&digit)[2]) {
    const int d0 = min(max((int)digit[0] - 1, 0), SEL_BINS - 6);
    w0 = max((uint32_t)d0 * 32u, 1u);   // bin 0 is what lies below: key 0 alone, then
    w1 = max((uint32_t)min(max((int)digit[1] - 1, d0 + 3), SEL_BINS - 3) * 32u, w0 + WIN_KEYS);
  }
  FP4_D explicit Windows(const SelState* st) : w0(st->window[0]), w1(st->window[1]) {}
  FP4_D bool side_by_side() const { return w0 + WIN_KEYS == w1; }
  // Bin 0: below the lower window, 1 .. 96 in it, 97 between the two (not kept), 98 .. 193 in the upper one, 194 above.
  FP4_D int bin(uint32_t key) const {
    return (key < w0 ? 0 : (int)min(key - w0 + 1, WIN_KEYS + 1u)) + (key < w1 ? 0 : (int)min(key - w1 + 1, WIN_KEYS + 1u));
  }
  // The two keys of zero, which may be most of a tensor, are counted apart where either is in a window.
  FP4_D bool zeros_apart() const {
    const int a = bin(KEY_NEG_ZERO), b = bin(KEY_POS_ZERO);
    return a % (WIN_KEYS + 1) != 0 || b % (WIN_KEYS + 1) != 0;
  }
};

// The thresholds' keys and bins from the bins' totals; false where rows' bins don't tell the rows' outliers, or the windows were missed.
// By all threads of a workgroup of 256 or more.
FP4_D bool find_windowed(const SelState* st, const unsigned long long* all_bins, const Ranks& ranks, unsigned long long n,
                         uint32_t (&key_out)[2], uint32_t (&bin_out)[2]) {
  const unsigned long long* const hist = all_bins + WIN_AT;
  __shared__ unsigned long long s_w[WIN_LDS / 64];
  __shared__ uint32_t key[2], bin[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const unsigned long long k = ranks.v[0];
  const Windows win(st);
  unsigned long long v = tid < WIN_BINS ? hist[tid] : 0, neg = 0, pos = 0;
  if (win.zeros_apart()) {   // the sums of win_count_kernel, undone
    const unsigned long long nz1 = hist[WIN_LDS], nz2 = hist[WIN_LDS + 1];
    neg = n - nz1;
    pos = 2 * nz1 - nz2;
    if (tid == win.bin(KEY_NEG_ZERO)) v += neg;
    if (tid == win.bin(KEY_POS_ZERO)) v += pos;
  }
  if (tid == WIN_KEYS + 1) v = 0;
  if (tid < 2) bin[tid] = WIN_BINS;
  unsigned long long incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long up = __shfl_up(incl, o, 64);
    if (lane >= o) incl += up;
  }
  if (lane == 63 && wave < WIN_LDS / 64) s_w[wave] = incl;
  __syncthreads();
  unsigned long long total = 0;   // without what lies between the windows
  for (int w = 0; w < WIN_LDS / 64; ++w) {
    if (w < wave) incl += s_w[w];
    total += s_w[w];
  }
  const unsigned long long below = incl - v, above = total - incl;
  const bool lower = (tid >= 1 || win.w0 == 1) && tid <= WIN_KEYS, upper = tid >= WIN_KEYS + 2 && tid < WIN_BINS - 1, both = win.side_by_side();
  const uint32_t mine = lower ? win.w0 + tid - 1 : win.w1 + tid - (WIN_KEYS + 2);
  if ((lower || (upper && both)) && below <= k && k < incl) { bin[0] = tid; key[0] = mine; }
  if ((upper || (lower && both)) && above <= k && k < above + v) { bin[1] = tid; key[1] = mine; }   // the (k + 1)-th from the top
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 2; ++q) { key_out[q] = key[q]; bin_out[q] = bin[q]; }
  // Rows' bins leave zeros out where they are counted apart: right while they are no outliers.
  return bin_out[0] < WIN_BINS && bin_out[1] < WIN_BINS && !st->nan &&
         !(neg + pos && (key_out[0] > KEY_POS_ZERO || key_out[1] < KEY_NEG_ZERO));
}

// One digit pass: histogram of the key's digit over the elements whose higher bits equal the prefix found so far (first pass: all
// elements, one shared histogram).
// The workgroup histogram is replicated (by lane) to thin out same-address LDS atomics: real
// tensors put most of their mass in a few dozen exponent bins.
// BEHIND: launched behind the one pass of large tensors (below), which may have left nothing to do.
template <class DT, int PASS>
struct SelTable {
  static constexpr int BINS = 1 << sel_bits<DT>(PASS), TABLE = PASS == 0 ? BINS : 2 * BINS, REPLICAS = PASS == 0 ? 8 : 4;
  uint32_t h[REPLICAS * TABLE];
};
// By SEL_THREADS threads, workgroup `block` of `blocks`.
template <class DT, int PASS, bool BEHIND>
FP4_D void sel_hist(const void* x, int64_t rows, int64_t cols, int64_t ld, const Ranks& ranks, SelState* st, unsigned long long* hist,
                    float* thresholds, unsigned block, unsigned blocks, SelTable<DT, PASS>& table) {
  constexpr bool first = PASS == 0;
  constexpr int BINS = 1 << sel_bits<DT>(PASS), SHIFT = sel_shift<DT>(PASS), HS = SHIFT + sel_bits<DT>(PASS);
  constexpr int TABLE = SelTable<DT, PASS>::TABLE, REPLICAS = SelTable<DT, PASS>::REPLICAS;
  constexpr int EPV = __is_same(DT, BF16) ? 8 : 4;   // elements per 16-byte load
  uint32_t (&h)[REPLICAS * TABLE] = table.h;
  const bool flat = (ld == cols) && (cols % EPV) == 0;
  const int64_t nvec = flat ? rows * cols / EPV : 0, stride = (int64_t)blocks * SEL_THREADS;
  const u32x4* const xv = reinterpret_cast<const u32x4*>(x);
  int64_t i = (int64_t)block * SEL_THREADS + threadIdx.x;
  // four loads in flight per lane, the first four before anything else: with the LDS tables limiting a CU to two workgroups, one
  // load at a time leaves the memory pipe mostly idle
  u32x4 r[4];
  auto fetch = [&](int64_t at) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (at + j * stride < nvec) r[j] = xv[at + j * stride];
  };
  if constexpr (!BEHIND) fetch(i);
  for (int b = threadIdx.x; b < REPLICAS * TABLE; b += SEL_THREADS) h[b] = 0;
  uint32_t p[2] = {0, 0};
  if constexpr (BEHIND) {
    if constexpr (first) {
      uint32_t key[2], bin[2];
      const bool ok = find_windowed(st, hist, ranks, rows * cols, key, bin);
      if (block == 0 && threadIdx.x < 2) {
        if (ok) thresholds[threadIdx.x] = value_of<DT>(threadIdx.x ? key[1] : key[0]);
        st->bin[threadIdx.x] = threadIdx.x ? bin[1] : bin[0];
        st->done = ok;
      }
      if (ok) return;
    } else if (st->done) {
      return;
    }
    fetch(i);
  }
  if constexpr (!first) find_digit<DT, PASS, SEL_THREADS>(st, hist, ranks, block == 0, p);
  __syncthreads();
  const int lane = threadIdx.x & 63;
  uint32_t* const hrep = &h[(lane & (REPLICAS - 1)) * TABLE];
  auto visit = [&](uint32_t raw) {
    const uint32_t key = key_of<DT>(raw);
    const uint32_t d = (key >> SHIFT) & (BINS - 1);
    if constexpr (first) {
      atomicAdd(&hrep[d], 1u);
    } else {
      const uint32_t hi_bits = key >> HS;
      if (hi_bits == p[0]) atomicAdd(&hrep[d], 1u);
      if (hi_bits == p[1]) atomicAdd(&hrep[BINS + d], 1u);
    }
  };
  if (flat) {
    auto visit_vec = [&](const u32x4& v) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if constexpr (__is_same(DT, BF16)) { visit(v[e] & 0xffffu); visit(v[e] >> 16); }
        else visit(v[e]);
      }
    };
    while (i < nvec) {
      const u32x4 c[4] = {r[0], r[1], r[2], r[3]};
      fetch(i + 4 * stride);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (i + j * stride < nvec) visit_vec(c[j]);
      i += 4 * stride;
    }
  } else {
    const int64_t n = rows * cols;
    for (; i < n; i += stride) {
      const int64_t row = i / cols, c = i - row * cols;
      if constexpr (__is_same(DT, BF16)) visit(reinterpret_cast<const uint16_t*>(x)[row * ld + c]);
      else visit(reinterpret_cast<const uint32_t*>(x)[row * ld + c]);
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < TABLE; b += SEL_THREADS) {
    uint32_t v = 0;
#pragma unroll
    for (int q = 0; q < REPLICAS; ++q) v += h[q * TABLE + b];
    if (v) atomicAdd(&hist[SEL_AT[PASS] + (b < BINS ? b : SEL_APART[PASS] + b - BINS)], (unsigned long long)v);
  }
}

}  // namespace
