// Outlier clamping and compensation (Sec. 3.2): exact per-tensor quantile thresholds by
// radix selection, and the ordering of the clamped-away residual of long rows into canonical
// CSR.  (The clamp itself is fused into the quantization pass; the transpose for the weight
// gradient and the sparse x dense product live with the sparse kernels.)
#include "fp4_common.h"
#include "last_block.h"

#include <algorithm>
#include <type_traits>

namespace {

struct BF16 {};
struct F32 {};

typedef int i32x4 __attribute__((ext_vector_type(4)));
constexpr int SEL_BINS = 2048;  // 11-bit digits
constexpr int SEL_THREADS = 1024;   // per workgroup: the 64 KiB of LDS tables allow two workgroups per CU,
                                    // so their size decides how many loads a CU has in flight

constexpr int SEL_PASSES = 3;   // digits, at most

// A digit pass: a workgroup for every 8192 elements up to 256 of them, for every 65536 up to 512 (64 x 2048 bf16, one for
// every 8192 / 65536: 8.5 / 9.2 us with the bins picked / without; 1056 x 1376 7.1 / 10.2; 8192 x 2048, 512 / 256: 18.1 /
// 15.6, each adds its bins to the same words).  Up to 64 of them the last one picks the bins: a launch of 4 us less; with
// more the arrivals cost more than that (8192 x 2048: 22.9 us against 15.6 + 4.9).
constexpr int SEL_PICK_HERE = 64;

// Selection state kept in the workspace between passes.
struct SelState {
  unsigned long long rank[2];  // remaining 0-based rank of the lo / hi order statistic
  uint32_t prefix[2];          // key bits fixed so far (right-aligned)
  uint32_t arrived[SEL_PASSES];   // workgroups done with a pass
  // windows (below): thresholds and row counts came out of one pass; a NaN was met; the thresholds' bins
  uint32_t done, nan, bin[2];
};

__global__ void sel_init_kernel(SelState* st, unsigned long long* hist, unsigned long long k,
                                unsigned long long n, unsigned long long* total) {
  int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < 2 * SEL_BINS) hist[i] = 0;
  if (i == 0) {
    st->rank[0] = k;
    st->rank[1] = n - 1 - k;
    st->prefix[0] = st->prefix[1] = 0;
    if (total) *total = 0;
    for (int a = 0; a < SEL_PASSES; ++a) st->arrived[a] = 0;
    st->done = st->nan = 0;
  }
}

// One digit pass: histogram of key digit (key >> shift) & (2^bits - 1) over the elements whose
// higher bits equal the prefix found so far (first pass: all elements, one shared histogram).
// The workgroup histogram is replicated (by lane) to thin out same-address LDS atomics: real
// tensors put most of their mass in a few dozen exponent bins.
template <class DT>
FP4_D uint32_t key_of(uint32_t raw) {   // raw: bf16 bits (low 16) or fp32 bits
  if constexpr (__is_same(DT, BF16)) return f32_order_key(raw << 16) >> 16;
  else return f32_order_key(raw);
}

// Pick, for each of the two targets, the bin that holds its rank; extend the prefix, reduce
// the rank, clear the histograms.  After the last pass the prefix is the full key: decode it.
// One workgroup: the one that finishes its part of the histogram last, or a launch of its own.
FP4_D void sel_pick(SelState* st, unsigned long long* hist, int bits, int first, int last, int key_bits, float* thresholds) {
  constexpr int PER = SEL_BINS / SEL_THREADS;   // bins a thread owns when all SEL_BINS are in use
  __shared__ unsigned long long s_w[SEL_THREADS / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nb = 1 << bits;
  const int per = (nb + SEL_THREADS - 1) / SEL_THREADS;
  // both targets' bins and ranks are requested before either scan starts
  unsigned long long vv[2][PER], rr[2];
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const unsigned long long* hsrc = hist + (first ? 0 : s * SEL_BINS);
    rr[s] = st->rank[s];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const int b = tid * per + j;
      vv[s][j] = (j < per && b < nb) ? load_device(hsrc + b) : 0;
    }
  }
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    unsigned long long (&v)[PER] = vv[s];
    unsigned long long sum = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) sum += v[j];
    // inclusive prefix of the threads' sums: the thread whose range [excl, incl) holds the rank
    // owns the bin (the last thread, should the rank lie beyond the total)
    unsigned long long incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const unsigned long long up = __shfl_up(incl, o, 64);
      if (lane >= o) incl += up;
    }
    if (lane == 63) s_w[wave] = incl;
    __syncthreads();
    for (int w = 0; w < wave; ++w) incl += s_w[w];
    const unsigned long long r = rr[s];
    const unsigned long long excl = incl - sum;
    if ((excl <= r && r < incl) || (tid == SEL_THREADS - 1 && r >= incl)) {
      unsigned long long cum = excl;
      int j = 0;
      const int jend = min(per, nb - tid * per);   // bins of this thread that exist (may be <= 0)
#pragma unroll
      for (int q = 0; q < PER - 1; ++q)
        if (j == q && q < jend - 1 && cum + v[q] <= r) { cum += v[q]; ++j; }
      const int b = min(tid * per + j, nb - 1);
      const uint32_t key = (st->prefix[s] << bits) | (uint32_t)b;
      st->rank[s] = r - cum;
      st->prefix[s] = key;
      if (last) {
        if (key_bits == 16) {
          // 16-bit keys are the top half of the fp32 key of a bf16 value; undo the map on
          // 16 bits so the low half of the fp32 pattern stays zero
          const uint32_t h = (key & 0x8000u) ? (key & 0x7fffu) : (~key & 0xffffu);
          thresholds[s] = u2f(h << 16);
        } else {
          thresholds[s] = u2f(f32_from_order_key(key));
        }
      }
    }
    __syncthreads();
  }
  for (int i = tid; i < 2 * SEL_BINS; i += SEL_THREADS) hist[i] = 0;
}

// PICK: the workgroup that is done last picks the bins.  BEHIND: launched behind the one pass of large tensors (below), which may
// have left nothing to do; elsewhere nothing is asked before the first element is requested.
template <class DT, bool FIRST, bool PICK, bool BEHIND>
__global__ __launch_bounds__(SEL_THREADS) void sel_hist_kernel(const void* x, int64_t rows, int64_t cols,
                                                       int64_t ld, int shift, int bits, int pass, int last, int key_bits,
                                                       SelState* st, unsigned long long* hist, float* thresholds) {
  constexpr bool first = FIRST;
  if constexpr (BEHIND) {
    if (st->done) return;
  }
  __shared__ uint32_t h[8 * SEL_BINS];   // first pass: 8 replicas; later: 4 replicas x 2 targets
  for (int i = threadIdx.x; i < 8 * SEL_BINS; i += SEL_THREADS) h[i] = 0;
  __syncthreads();
  const uint32_t mask = (1u << bits) - 1u;
  const uint32_t p0 = st->prefix[0], p1 = st->prefix[1];
  const int hs = shift + bits;
  const int lane = threadIdx.x & 63;
  uint32_t* const hrep = first ? &h[(lane & 7) * SEL_BINS] : &h[(lane & 3) * 2 * SEL_BINS];
  auto visit = [&](uint32_t raw) {
    const uint32_t key = key_of<DT>(raw);
    const uint32_t d = (key >> shift) & mask;
    if (first) {
      atomicAdd(&hrep[d], 1u);
    } else {
      const uint32_t hi_bits = hs >= 32 ? 0u : (key >> hs);
      if (hi_bits == p0) atomicAdd(&hrep[d], 1u);
      if (hi_bits == p1) atomicAdd(&hrep[SEL_BINS + d], 1u);
    }
  };
  constexpr int EPV = __is_same(DT, BF16) ? 8 : 4;   // elements per 16-byte load
  const bool flat = (ld == cols) && (cols % EPV) == 0;
  if (flat) {
    const int64_t nvec = rows * cols / EPV;
    const u32x4* xv = reinterpret_cast<const u32x4*>(x);
    auto visit_vec = [&](const u32x4& r) {
      if constexpr (__is_same(DT, BF16)) {
        visit(r.x & 0xffffu); visit(r.x >> 16); visit(r.y & 0xffffu); visit(r.y >> 16);
        visit(r.z & 0xffffu); visit(r.z >> 16); visit(r.w & 0xffffu); visit(r.w >> 16);
      } else {
        visit(r.x); visit(r.y); visit(r.z); visit(r.w);
      }
    };
    // four loads in flight per lane: with the LDS tables limiting a CU to two workgroups, one
    // load at a time leaves the memory pipe mostly idle
    const int64_t stride = (int64_t)gridDim.x * SEL_THREADS;
    int64_t i = (int64_t)blockIdx.x * SEL_THREADS + threadIdx.x;
    for (; i + 3 * stride < nvec; i += 4 * stride) {
      const u32x4 r0 = xv[i], r1 = xv[i + stride], r2 = xv[i + 2 * stride], r3 = xv[i + 3 * stride];
      visit_vec(r0); visit_vec(r1); visit_vec(r2); visit_vec(r3);
    }
    for (; i < nvec; i += stride) visit_vec(xv[i]);
  } else {
    const int64_t n = rows * cols;
    for (int64_t i = (int64_t)blockIdx.x * SEL_THREADS + threadIdx.x; i < n; i += (int64_t)gridDim.x * SEL_THREADS) {
      const int64_t r = i / cols, c = i - r * cols;
      if constexpr (__is_same(DT, BF16)) visit(reinterpret_cast<const uint16_t*>(x)[r * ld + c]);
      else visit(reinterpret_cast<const uint32_t*>(x)[r * ld + c]);
    }
  }
  __syncthreads();
  if (first) {
    for (int i = threadIdx.x; i < SEL_BINS; i += SEL_THREADS) {
      uint32_t v = 0;
#pragma unroll
      for (int r = 0; r < 8; ++r) v += h[r * SEL_BINS + i];
      if (v) atomicAdd(&hist[i], (unsigned long long)v);
    }
  } else {
    for (int i = threadIdx.x; i < 2 * SEL_BINS; i += SEL_THREADS) {
      uint32_t v = 0;
#pragma unroll
      for (int r = 0; r < 4; ++r) v += h[r * 2 * SEL_BINS + i];
      if (v) atomicAdd(&hist[i], (unsigned long long)v);
    }
  }
  if constexpr (PICK) {
    if (last_workgroup(&st->arrived[pass], gridDim.x)) sel_pick(st, hist, bits, first, last, key_bits, thresholds);
  }
}

__global__ __launch_bounds__(SEL_THREADS) void sel_pick_kernel(SelState* st, unsigned long long* hist, int bits, int first, int last,
                                                               int key_bits, float* thresholds) {
  sel_pick(st, hist, bits, first, last, key_bits, thresholds);
}

// ---- Large bf16 tensors: thresholds and the rows' outlier counts out of one pass ------------------------------------------
// A sample says where the thresholds are, to within a few of the 2048 leading 11-bit digits; the pass over all elements then
// needs bins only for the keys around them (three digits, 96 keys a threshold), counts what lies outside, and keeps every
// row's bins: with the thresholds known, a row's outliers are a sum over those.  Where a threshold turns out not to lie in
// its window, or a NaN is about, `done` stays 0 and the passes of the general path, launched behind, do their work; otherwise
// they leave at once.
// Bound by the one read and, about as long, by vector instructions (nine an element, twelve where zeros are counted apart).
// 16384 x 11008, in us: init 4.6, sample 6.6, picks 4.8 + 4.7, the pass 94.7, the general path's two launches 9, rows 4.9, together
// 130; digit passes, picks and the count of the rows after them 249.  16384 x 4096: 71 against 107.  With scan and emission: half
// zeros, 16384 x 11008, 250 against 540; a miss 419 against 353.  Below 2^25 elements the launches cost what the pass saves (8192 x
// 2048: digit passes, picks and count 43, of which this would leave 40).
constexpr int WIN_KEYS = 96, WIN_BINS = 2 * WIN_KEYS + 3, WIN_LDS = 256, WIN_STRIDE = 200;   // bins; a wave's table; a row's in memory
constexpr uint32_t KEY_NEG_ZERO = 0x7fff, KEY_POS_ZERO = 0x8000;
constexpr int SAMPLE_BLOCKS = 128, SAMPLE_RUNS = SAMPLE_BLOCKS * 2 * (SEL_THREADS / 64);   // runs of 64 16-byte vectors

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
    if (v) atomicAdd(&hist[i], (unsigned long long)v);
  }
}

// First keys of the windows, from the digits that the sample's order statistics have.  Windows that would meet lie side by
// side, and either threshold may be in either.  (The lowest digit is that of a negative NaN.)
struct Windows {
  uint32_t w0, w1;
  FP4_D explicit Windows(const SelState* st) {
    const int d0 = min(max((int)st->prefix[0] - 1, 1), SEL_BINS - 6);
    w0 = (uint32_t)d0 * 32u;
    w1 = (uint32_t)min(max((int)st->prefix[1] - 1, d0 + 3), SEL_BINS - 3) * 32u;
  }
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

// A wave per row.
__global__ __launch_bounds__(1024) void win_count_kernel(const uint16_t* x, int64_t rows, int64_t cols, SelState* st, unsigned long long* hist,
                                                         uint16_t* row_bins) {
  __shared__ uint32_t tab[16][WIN_LDS];
  __shared__ uint32_t total[WIN_LDS + 2];
  const Windows win(st);
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
  // Sums of 0 / 1 / 1 and of 0 / 1 / 2 for -0, +0 and the rest.  16 bits hold them: rows have 500 elements or more (row_bins has to fit
  // the entries' room) and the tensor fewer than 2^32, so a half word meets at most 2^13 + 2^7 of them.
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
  if (threadIdx.x < WIN_LDS + 2 && total[threadIdx.x]) atomicAdd(&hist[threadIdx.x], (unsigned long long)total[threadIdx.x]);
}

// The thresholds from the bins' totals, or the state that the general path starts from.
__global__ __launch_bounds__(WIN_LDS) void win_pick_kernel(SelState* st, unsigned long long* hist, unsigned long long k, unsigned long long n,
                                                           float* thresholds) {
  __shared__ unsigned long long s_w[WIN_LDS / 64];
  __shared__ uint32_t key[2], bin[2];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const Windows win(st);
  const bool zeros_apart = win.zeros_apart();
  unsigned long long v = tid < WIN_BINS ? hist[tid] : 0, neg = 0, pos = 0;
  if (zeros_apart) {   // the sums of win_count_kernel, undone
    const unsigned long long nz1 = hist[WIN_LDS], nz2 = hist[WIN_LDS + 1];
    neg = n - nz1;
    pos = 2 * nz1 - nz2;
    if (tid == win.bin(KEY_NEG_ZERO)) v += neg;
    if (tid == win.bin(KEY_POS_ZERO)) v += pos;
  }
  if (tid == WIN_KEYS + 1) v = 0;
  if (tid < 2) bin[tid] = 0;
  unsigned long long incl = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long up = __shfl_up(incl, o, 64);
    if (lane >= o) incl += up;
  }
  if (lane == 63) s_w[wave] = incl;
  __syncthreads();
  unsigned long long total = 0;   // without what lies between the windows
  for (int w = 0; w < WIN_LDS / 64; ++w) {
    if (w < wave) incl += s_w[w];
    total += s_w[w];
  }
  const unsigned long long below = incl - v, above = total - incl;
  const bool lower = tid >= 1 && tid <= WIN_KEYS, upper = tid >= WIN_KEYS + 2 && tid < WIN_BINS - 1, both = win.side_by_side();
  const uint32_t mine = lower ? win.w0 + tid - 1 : win.w1 + tid - (WIN_KEYS + 2);
  if ((lower || (upper && both)) && below <= k && k < incl) { bin[0] = tid; key[0] = mine; }
  if ((upper || (lower && both)) && above <= k && k < above + v) { bin[1] = tid; key[1] = mine; }   // the (k + 1)-th from the top
  __syncthreads();
  if (tid == 0) {
    // Rows' bins leave zeros out where they are counted apart: right while they are no outliers.
    const bool ok = bin[0] && bin[1] && !st->nan && !(neg + pos && (key[0] > KEY_POS_ZERO || key[1] < KEY_NEG_ZERO));
    if (ok)
      for (int s = 0; s < 2; ++s) thresholds[s] = u2f(((key[s] & 0x8000u) ? (key[s] & 0x7fffu) : (~key[s] & 0xffffu)) << 16);
    st->done = ok;
    st->bin[0] = bin[0];
    st->bin[1] = bin[1];
    st->rank[0] = k;
    st->rank[1] = n - 1 - k;
    st->prefix[0] = st->prefix[1] = 0;
  }
  hist[tid] = 0;
  if (tid < 2) hist[WIN_LDS + tid] = 0;
}

// Outliers of each row: from its bins, or, where the windows were missed, from its elements.  A wave per row.
__global__ __launch_bounds__(256) void win_rows_kernel(const uint16_t* x, int64_t rows, int64_t cols, const SelState* st, const uint16_t* row_bins,
                                                       const float* thr, int32_t* row_cnt) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  int cnt = 0;
  if (st->done) {
    const int b0 = (int)st->bin[0], b1 = (int)st->bin[1];
#pragma unroll
    for (int j = 0; j < WIN_LDS / 64; ++j) {
      const int b = lane + 64 * j;
      if (b < b0 || (b > b1 && b < WIN_BINS)) cnt += row_bins[row * WIN_STRIDE + b];
    }
  } else {
    const float lo = thr[0], hi = thr[1];
    const u32x4* const xr = reinterpret_cast<const u32x4*>(x + row * cols);
    for (int64_t i = lane; i < cols / 8; i += 64) {
      const u32x4 r = xr[i];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float a = u2f(r[e] << 16), b = u2f(r[e] & 0xffff0000u);
        cnt += (((a < lo) | (a > hi)) ? 1 : 0) + (((b < lo) | (b > hi)) ? 1 : 0);
      }
    }
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) cnt += __shfl_xor(cnt, o, 64);
  if (lane == 0) row_cnt[row] = cnt;
}

// ---- CSR finalisation ---------------------------------------------------------------------
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
size_t fp4_select_scratch_bytes() {
  return align_up(sizeof(SelState), 256) + align_up(2 * SEL_BINS * sizeof(unsigned long long), 256);
}

namespace {
// The digit passes, from the state that sel_init_kernel left, or (behind) win_pick_kernel.
void launch_digits(const void* x, int bf16, int64_t rows, int64_t cols, int64_t ld, float* thresholds, SelState* st, unsigned long long* hist,
                   bool behind, hipStream_t s) {
  const int64_t n = rows * cols;
  const int key_bits = bf16 ? 16 : 32;
  int digits[3];
  int nd;
  if (bf16) { digits[0] = 11; digits[1] = 5; nd = 2; }
  else { digits[0] = 11; digits[1] = 11; digits[2] = 10; nd = 3; }
  int shift = key_bits;
  const int64_t few = std::min<int64_t>((n + 8191) / 8192, 256), many = std::min<int64_t>((n + 65535) / 65536, 512);
  const unsigned grid = (unsigned)std::max<int64_t>(1, std::max(few, many));
  const bool pick_here = behind || grid <= SEL_PICK_HERE;   // launches that mostly leave at once: as few as there can be
  for (int p = 0; p < nd; ++p) {
    shift -= digits[p];
    auto launch = [&](auto dt, auto first, auto pick, auto after) {
      hipLaunchKernelGGL((sel_hist_kernel<decltype(dt), decltype(first)::value, decltype(pick)::value, decltype(after)::value>), dim3(grid),
                         dim3(SEL_THREADS), 0, s, x, rows, cols, ld, shift, digits[p], p, p == nd - 1, key_bits, st, hist, thresholds);
    };
    auto pass = [&](auto dt, auto first) {
      if constexpr (__is_same(decltype(dt), BF16)) {
        if (behind) return launch(dt, first, std::true_type{}, std::true_type{});
      }
      if (pick_here) launch(dt, first, std::true_type{}, std::false_type{});
      else launch(dt, first, std::false_type{}, std::false_type{});
    };
    if (p == 0) { if (bf16) pass(BF16{}, std::true_type{}); else pass(F32{}, std::true_type{}); }
    else { if (bf16) pass(BF16{}, std::false_type{}); else pass(F32{}, std::false_type{}); }
    if (!pick_here)
      hipLaunchKernelGGL(sel_pick_kernel, dim3(1), dim3(SEL_THREADS), 0, s, st, hist, digits[p], p == 0, p == nd - 1, key_bits,
                         thresholds);
  }
}
}  // namespace

// Thresholds lo = v[k], hi = v[n-1-k] of the ascending-sorted tensor into thresholds[0..1].
// Also zeroes *total (the residual entry counter) when given.
int fp4_launch_thresholds(const void* x, int bf16, int64_t rows, int64_t cols, int64_t ld, int64_t k,
                          float* thresholds, void* scratch, unsigned long long* total, hipStream_t s) {
  SelState* st = reinterpret_cast<SelState*>(scratch);
  unsigned long long* hist =
      reinterpret_cast<unsigned long long*>(reinterpret_cast<uint8_t*>(scratch) + align_up(sizeof(SelState), 256));
  const int64_t n = rows * cols;
  hipLaunchKernelGGL(sel_init_kernel, dim3(2 * SEL_BINS / 256), dim3(256), 0, s, st, hist,
                     (unsigned long long)k, (unsigned long long)n, total);
  launch_digits(x, bf16, rows, cols, ld, thresholds, st, hist, false, s);
  FP4_CHECK_LAUNCH();
  return FP4_OK;
}

// Thresholds and outlier counts of rows in one pass; 1 where that is not the better way (the caller then does one after the other).
// rows_scratch: words that are free until the rows' entries are emitted.
int fp4_launch_thresholds_and_counts(const void* x, int bf16, int64_t rows, int64_t cols, int64_t ld, int64_t k, float* thresholds,
                                     void* scratch, unsigned long long* total, void* rows_scratch, int64_t rows_scratch_words,
                                     int32_t* row_cnt, hipStream_t s) {
  const int64_t n = rows * cols;
  if (!bf16 || ld != cols || cols % 8 != 0 || cols > 65535 || n < ((int64_t)1 << 25) || n >= ((int64_t)1 << 32) ||
      rows * WIN_STRIDE > 2 * rows_scratch_words)
    return 1;
  SelState* st = reinterpret_cast<SelState*>(scratch);
  unsigned long long* hist =
      reinterpret_cast<unsigned long long*>(reinterpret_cast<uint8_t*>(scratch) + align_up(sizeof(SelState), 256));
  // the sample's ranks first
  const int64_t ns = (int64_t)SAMPLE_RUNS * 64 * 8;
  const unsigned long long ks = (unsigned long long)((double)k / (double)n * (double)ns);
  hipLaunchKernelGGL(sel_init_kernel, dim3(2 * SEL_BINS / 256), dim3(256), 0, s, st, hist, ks, (unsigned long long)ns, total);
  hipLaunchKernelGGL(sel_sample_kernel, dim3(SAMPLE_BLOCKS), dim3(SEL_THREADS), 0, s, reinterpret_cast<const u32x4*>(x), n / 8, hist);
  hipLaunchKernelGGL(sel_pick_kernel, dim3(1), dim3(SEL_THREADS), 0, s, st, hist, 11, 1, 0, 16, thresholds);
  uint16_t* const bins = reinterpret_cast<uint16_t*>(rows_scratch);
  const uint16_t* const xp = reinterpret_cast<const uint16_t*>(x);
  hipLaunchKernelGGL(win_count_kernel, dim3((unsigned)std::min<int64_t>((rows + 15) / 16, 512)), dim3(1024), 0, s, xp, rows, cols, st, hist, bins);
  hipLaunchKernelGGL(win_pick_kernel, dim3(1), dim3(256), 0, s, st, hist, (unsigned long long)k, (unsigned long long)n, thresholds);
  launch_digits(x, bf16, rows, cols, ld, thresholds, st, hist, true, s);
  hipLaunchKernelGGL(win_rows_kernel, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, s, xp, rows, cols, st, bins, thresholds, row_cnt);
  FP4_CHECK_LAUNCH();
  return FP4_OK;
}

int fp4_launch_scan_rows(const int32_t* row_cnt, int64_t rows, int64_t* row_ptr, int64_t* nnz, hipStream_t s) {
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
