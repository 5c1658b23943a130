// The residual product R[P x N] = S D of a small layer: one launch, no packing, no staging, no list of long rows.
//
// The packed and the tiled kernels (spmm_mfma.hip, spmm.hip) are four launches, and what they stage, plan and list pays where a
// row of D is used again and again.  In a small product the launches are most of it and D fits the L2s: here every entry
// gathers its piece of D from L2, GA_AHEAD requests of 1 KiB on their way a wave, and plain FMAs add it up.
#include "fp4_common.h"
#include "fp4_measure.h"
#include "spmm_long.h"

#include <algorithm>
#include <type_traits>

namespace {

constexpr int GA_AHEAD = 8;
constexpr int GA_LONG = 256;         // entries up to which no row is long
constexpr int GA_LONG_COLS = 4096;   // columns up to which long rows are as others
constexpr int GA_LONG_LANES = 8;

FP4_D uint64_t lane_value(uint64_t v, int l) {
  return (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), l) << 32 | (uint32_t)__builtin_amdgcn_readlane((int)v, l);
}
FP4_D uint64_t uniform(uint64_t v) { return lane_value(v, 0); }   // what all lanes have

template <class DT> constexpr int per_lane() { return __is_same(DT, BF16) ? 8 : 4; }   // elements of 16 bytes

// A wave's sums over the entries [b, e) for the columns n0 .., left in `sums` [64 / LANES][LANES x 16 bytes of elements].  LANES lanes have an
// entry's piece of D, 16 bytes each; a request of the wave brings the pieces of 64 / LANES entries.  What is requested together is
// added up by itself: an outlier channel's row in one chain, or in one for 64 entries, is further off than the sums it replaces (error
// against 64 bits, rows of 512 among sparse ones, fp32: 1.28e-7, now 8.7e-8, the kernels of large products 9.7e-8).
template <class DT, int LANES>
FP4_D void gather_entries(const int32_t* __restrict__ col_idx, const float* __restrict__ val, int64_t b, int64_t e, const uint8_t* D, int Q,
                          int64_t N, int64_t n0, float* sums) {
  constexpr int ES = __is_same(DT, BF16) ? 2 : 4, PER = per_lane<DT>(), SIDE = 64 / LANES;
  const int lane = threadIdx.x & 63, side = lane / LANES, l = lane % LANES;
  // What an entry past the last or a column past N would ask for lies past the descriptor's end and arrives as zero: no branch between
  // the requests, which would each wait for the one before.
  constexpr uint32_t NOWHERE = 0xf0000000u;
  const uint32_t rowb = (uint32_t)(N * ES);
  const __amdgpu_buffer_rsrc_t rsrc =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(D), 0, (int)((uint32_t)Q * rowb), 0x00020000);
  const bool in_n = n0 + l * PER < N;   // N is a multiple of 8
  const uint32_t at = in_n ? (uint32_t)(n0 + l * PER) * ES : NOWHERE;
  float sum[PER] = {};
  for (int64_t i0 = b; i0 < e; i0 += 64) {
    const int here = (int)min(e - i0, (int64_t)64);
    int c = -1;   // of no entry; other columns that D has not are left out like it
    float v = 0.0f;
    if (lane < here) {
      c = col_idx[i0 + lane];
      v = val[i0 + lane];
    }
    const bool is = (uint32_t)c < (uint32_t)Q;
    const uint32_t off = is ? (uint32_t)c * rowb : NOWHERE;
    if (!is) v = 0.0f;
    for (int j = 0; j < here; j += GA_AHEAD * SIDE) {
      u32x4 p[GA_AHEAD];
      float acc[PER] = {};
#pragma unroll
      for (int u = 0; u < GA_AHEAD; ++u) {
        if constexpr (SIDE == 1) {
          const uint32_t o = (uint32_t)__builtin_amdgcn_readlane((int)off, j + u);
          p[u] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, at | (o == NOWHERE ? NOWHERE : 0u), o == NOWHERE ? 0u : o, 0);
        } else {
          const uint32_t o = (uint32_t)__shfl((int)off, j + u * SIDE + side, 64);
          p[u] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, o == NOWHERE || !in_n ? NOWHERE : at + o, 0, 0);
        }
      }
#pragma unroll
      for (int u = 0; u < GA_AHEAD; ++u) {
        float vu;
        if constexpr (SIDE == 1) vu = u2f((uint32_t)__builtin_amdgcn_readlane((int)f2u(v), j + u));
        else vu = __shfl(v, j + u * SIDE + side, 64);
#pragma unroll
        for (int k = 0; k < PER; ++k) {
          float d;
          if constexpr (ES == 2) d = u2f((k & 1) ? p[u][k >> 1] & 0xffff0000u : p[u][k >> 1] << 16);
          else d = u2f(p[u][k]);
          acc[k] = fmaf(vu, d, acc[k]);
        }
      }
#pragma unroll
      for (int k = 0; k < PER; ++k) sum[k] += acc[k];
    }
  }
#pragma unroll
  for (int h = 0; h < PER / 4; ++h)
    *reinterpret_cast<f32x4*>(sums + (side * LANES + l) * PER + 4 * h) = f32x4{sum[4 * h], sum[4 * h + 1], sum[4 * h + 2], sum[4 * h + 3]};
}

// The i-th of `of` parts of the entries [b, b + n): the waves of a row take them in that order, and they are added in it.
template <class DT, int LANES>
FP4_D void gather_part(const int32_t* col_idx, const float* val, int64_t b, int64_t n, int i, int of, const uint8_t* D, int Q, int64_t N,
                       int64_t n0, float* sums) {
  gather_entries<DT, LANES>(col_idx, val, b + n * i / of, b + n * (i + 1) / of, D, Q, N, n0, sums);
}

// A column's sum over all waves and sides of a workgroup, two or four at a time.
template <int WAVES, int SIDE, int COLS>
FP4_D float add_up(const float* sums, int t) {
  float s = 0.0f;
#pragma unroll
  for (int w = 0; w < WAVES; w += 2) {
    const float *x = sums + w * SIDE * COLS + t, *y = x + SIDE * COLS;
    float q = x[0] + y[0];
#pragma unroll
    for (int h = 1; h < SIDE; ++h) q += x[h * COLS] + y[h * COLS];
    s += q;
  }
  return s;
}

// A workgroup has ROWS rows of a strip of columns, WAVES / ROWS waves a row; rows of more than four times the mean are shared by all its
// waves.  LONG: not if they have more than GA_LONG entries as well.  A CU has about 64 KiB of requests on their way, 60 GB/s, so a row that is
// full or nearly takes a workgroup 8.5 ns an entry while the chip waits: as long, from about 6000 columns on, as the kernels of large
// products take for everything.  Such rows are the first long_blocks workgroups', strips of 128 bytes and every long_slots-th row each.  In
// us, bf16, 1 % and none / one / eight full rows, without / with these workgroups / the other kernels: 512 x 8192 -> 512 10, 77, 143 / 11, 29,
// 30 / 60, 69, 72; 512 x 8192 -> 2048 15, 84, 152 / 15, 39, 68 / 61, 73, 78; fp32 512 x 8192 -> 512 9, 50, 96 / 9, 28, 30 / 106, 136, 141.  With
// fewer columns they cost 4 to 6 % where there are no such rows (2048^3, 6 % 48.2 / 51.3).
template <class DT, int LANES, int WAVES, int ROWS, bool LONG>
__global__ __launch_bounds__(WAVES * 64, LONG ? 7 : 8) void spmm_gather_kernel(const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                                                                const float* __restrict__ val, int64_t capacity, int64_t P, int row_blocks,
                                                                int items, int long_blocks, int long_slots, int Q,
                                                                const uint8_t* __restrict__ D, int64_t N, float* __restrict__ R) {
  static_assert(WAVES % ROWS == 0 && ROWS < 64, "whole waves a row, a lane a row");
  constexpr int PER = per_lane<DT>(), COLS = LANES * PER, SIDE = 64 / LANES, SHARE = WAVES / ROWS;
  __shared__ __attribute__((aligned(16))) float sums[WAVES][64 * PER];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  auto limits = [&](int64_t& shared_from, int64_t& long_from) {
    shared_from = max((int64_t)64, 4 * (min(row_ptr[P], capacity) - row_ptr[0]) / P);
    long_from = LONG ? max((int64_t)GA_LONG, shared_from) : INT64_MAX;
  };
  if constexpr (LONG) {
    if ((int)blockIdx.x < long_blocks) {
      constexpr int LCOLS = GA_LONG_LANES * PER;
      __shared__ uint64_t s_long[WAVES];
      const int64_t n0 = (int64_t)((int)blockIdx.x / long_slots) * LCOLS;
      if (n0 >= N) return;
      int64_t shared_from, long_from;
      limits(shared_from, long_from);
      for (int64_t first = (int)blockIdx.x % long_slots; first < P; first += (int64_t)long_slots * WAVES * 64) {
        const int64_t row = min(first + (int64_t)tid * long_slots, P);
        const int64_t end = min(row_ptr[min(row + 1, P)], capacity);
        const uint64_t mine = __ballot(end - row_ptr[row] > long_from);
        if (lane == 0) s_long[wave] = mine;
        __syncthreads();
        for (int w = 0; w < WAVES; ++w)
          for (uint64_t m = uniform(s_long[w]); m != 0; m &= m - 1) {
            const int64_t r = first + (int64_t)(w * 64 + __builtin_ctzll(m)) * long_slots, b = row_ptr[r];
            gather_part<DT, GA_LONG_LANES>(col_idx, val, b, min(row_ptr[r + 1], capacity) - b, wave, WAVES, D, Q, N, n0, sums[wave]);
            __syncthreads();
            if (tid < LCOLS && n0 + tid < N) R[r * N + n0 + tid] = add_up<WAVES, 64 / GA_LONG_LANES, LCOLS>(sums[0], tid);
            __syncthreads();   // the sums are read
          }
        __syncthreads();   // and the rows
      }
      return;
    }
  }
  // Workgroup i runs on XCD i % 8 (long_blocks is a multiple of that), and each XCD takes a contiguous run of items, rows inside columns:
  // its L2 then holds the one strip of D that its workgroups gather from.
  const int per_xcd = (items + 7) / 8, id = LONG ? (int)blockIdx.x - long_blocks : (int)blockIdx.x;
  // An XCD has 32 CUs and gives them its workgroups in turn.  Each turn starts 11 further, or rows a power of two apart, or one row's strips,
  // meet on one CU, and full ones wait for each other.  In us, eight full rows of 2048^3, 128 and 64 apart, in order / now: bf16 38, 29 /
  // 25, 25, fp32 46, 46 / 34, 38, 16 apart 34 / 35, side by side 31 / 36; one full row, 992 x 736 -> 2336, 6 % 25 / 22; no full rows the same.
  const uint32_t in_xcd = (uint32_t)id / 8, turn = in_xcd / 32, place = turn * 32 + ((in_xcd + 11 * turn) & 31);
  const int item = (int)((uint32_t)id % 8 * per_xcd + place);
  if ((int)place >= per_xcd || item >= items) return;
  // Of every eight rows that lie side by side a workgroup has one, and not always the same: outlier channels are often neighbours, or as
  // far apart as a head is wide, and rows that all waves share are taken one after another.  In us, bf16, 1 % and eight full rows side by
  // side, eight rows in order a workgroup / now / the kernels of large products: 2048^3 112 / 32 / 43, 512 x 2048 -> 512 108 / 20 / 35,
  // 1024^3 59 / 13 / 31, 4096 x 512 -> 1024 35 / 16 / 34; fp32 2048^3 85 / 38 / 56.  Without such rows up to 4 % slower (1056 x 1376 -> 2080, 6 %
  // 24.0 / 25.0; 2048^3 22.2 / 22.5), because the entries' lines are several workgroups'.
  const int rb = item % row_blocks;
  auto row_of = [&](int r) { return (int64_t)(rb / 8) * (8 * ROWS) + 8 * r + ((rb + r) & 7); };   // P or more: none
  const int64_t n0 = (int64_t)(item / row_blocks) * COLS;
  // The rows' ends, a lane each; every wave has them all, so all come to the same answer without a word.
  const int64_t my_row = min(row_of(min(lane, ROWS - 1)), P);
  const int64_t rp = min(row_ptr[my_row], capacity), next = min(row_ptr[min(my_row + 1, P)], capacity);
  const int n_lane = lane < ROWS ? (int)max(next - rp, (int64_t)0) : 0;
  int64_t shared_from, long_from;
  limits(shared_from, long_from);
  const uint64_t not_here = LONG ? __ballot(n_lane > long_from) : 0, shared_rows = __ballot(n_lane > shared_from) & ~not_here;
  auto part = [&](int r, int i, int of) {   // the i-th part of row r's entries
    gather_part<DT, LANES>(col_idx, val, (int64_t)lane_value((uint64_t)rp, r), __builtin_amdgcn_readlane(n_lane, r), i, of, D, Q, N, n0, sums[wave]);
  };
  for (uint64_t m = shared_rows; m != 0; m &= m - 1) {
    const int r = __builtin_ctzll(m);
    part(r, wave, WAVES);
    __syncthreads();
    for (int t = tid; t < COLS; t += WAVES * 64)
      if (n0 + t < N) R[row_of(r) * N + n0 + t] = add_up<WAVES, SIDE, COLS>(sums[0], t);
    __syncthreads();   // the sums are read
  }
  const int mine = wave / SHARE;
  const uint64_t done = shared_rows | not_here;
  const bool mine_done = (done >> mine) & 1;
  if (!mine_done) part(mine, wave % SHARE, SHARE);
  if constexpr (SHARE == 1) {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");   // the sums are this wave's own
    __builtin_amdgcn_wave_barrier();
    if (mine_done || row_of(mine) >= P) return;
#pragma unroll
    for (int t = lane * 4; t < COLS; t += 256) {
      f32x4 s = *reinterpret_cast<const f32x4*>(&sums[wave][t]);
#pragma unroll
      for (int h = 1; h < SIDE; ++h) s += *reinterpret_cast<const f32x4*>(&sums[wave][h * COLS + t]);
      if (n0 + t < N) *reinterpret_cast<f32x4*>(R + row_of(mine) * N + n0 + t) = s;
    }
  } else {
    __syncthreads();
#pragma unroll
    for (int t = tid * 4; t < ROWS * COLS; t += WAVES * 256) {
      const int r = t / COLS, c = t % COLS;
      f32x4 s = *reinterpret_cast<const f32x4*>(&sums[r * SHARE][c]);
#pragma unroll
      for (int h = 1; h < SHARE * SIDE; ++h) s += *reinterpret_cast<const f32x4*>(&sums[r * SHARE + h / SIDE][h % SIDE * COLS + c]);
      if (!((done >> r) & 1) && row_of(r) < P && n0 + c < N) *reinterpret_cast<f32x4*>(R + row_of(r) * N + n0 + c) = s;
    }
  }
}

}  // namespace

// Whether a product of `entries` entries, or at most so many, is gathered.
//
// The gathers move entries x N x the size of an element through the L2s, at 20 to 30 TB/s while a strip of D stays in one; the other kernels'
// time goes with what they stage, Q x N, and with the output.  What they take besides goes with the entries too, but in the packed kernel
// hardly (and a value of several terms may send its matrix to the tiled one: the lines are those of values that bf16 holds, at which it is
// fastest).  So there is a number of entries up to which gathering is faster.  In us, this / the others, and the bytes where they meet:
//   bf16  4096 x 512 -> 1024, 12 % 28 / 32, 20 % 38 / 35 (709 MB); 2048 x 1024 -> 1024, 12 % 27 / 34, 20 % 39 / 36 (762); 1056 x 1376 ->
//         2080, 6 % 24 / 35, 12 % 40 / 40 (704); 2048 x 2048 -> 1024, 12 % 45 / 50, 20 % 72 / 54 (1171); 2048^3, 2 % 23 / 37, 6 % 48 / 50, 9 %
//         67 / 56, 20 % 132 / 63 (1104); 1024 x 4096 -> 1024, 20 % 76 / 86 (2046); 512 x 8192 -> 1024, 20 % 109 / 153 (2918)
//   fp32  4096 x 512 -> 1024, 20 % 63 / 67, 50 % 145 / 122 (2060); 2048^3, 12 % 144 / 148, 20 % 229 / 214 (4737); 1056 x 1376 -> 2080, 2048 x
//         1024 -> 1024 and smaller outputs never, 100 % 418 / 491 and 277 / 367: there the tiled kernel has too few workgroups
// Beyond 2^33, 2^23 outputs (fp32 2^22) or 8192 columns the others are faster at 6 %, the densest residual in use: bf16 16384 x 128 -> 2048
// 63 / 52, 512 x 4096 -> 8192 103 / 75; fp32 4096 x 1024 -> 2048 76 / 60.  256 x 16384 -> 1024 with four full rows 306 / 149.
static bool gathers(int64_t P, int64_t Q, int64_t N, int bf16, int64_t entries) {
  const int es = bf16 ? 2 : 4;
  const double out = (double)P * (double)N, d_bytes = (double)Q * (double)N * es;
  if (out * (double)Q > 0x1p33 || out > (bf16 ? 0x1p23 : 0x1p22) || Q > 8192 || d_bytes > (double)0xe0000000u) return false;   // 32-bit offsets into D
  const double moved = std::min((double)entries, (double)P * (double)Q) * (double)N * es;
  if (bf16) return moved <= 0x1p28 + (double)Q * 0x1p18 + 64 * out;
  return out <= 5 * 0x1p19 || moved <= 0x1p30 + 1.5 * (double)Q * 0x1p20;
}

extern "C" int fp4_residual_spmm_gathers(int64_t P, int64_t Q, int64_t N, fp4_dtype dt, int64_t entries) {
  return gathers(P, Q, N, dt == FP4_BF16, entries);
}

// Returns 1 where the packed or the tiled kernel takes the product.  capacity: no more entries than that.
int fp4_launch_spmm_gather(const int64_t* row_ptr, const int32_t* col_idx, const float* val, int64_t capacity, int64_t P, int64_t Q,
                           const void* D, int bf16, int64_t N, float* R, hipStream_t s) {
  if (!gathers(P, Q, N, bf16, capacity)) return 1;
  const int es = bf16 ? 2 : 4;
  const uint8_t* const d = reinterpret_cast<const uint8_t*>(D);
  auto launch = [&](auto dt, auto lanes, auto waves, auto rows, auto with_long) {
    constexpr int L = decltype(lanes)::value, W = decltype(waves)::value, ROWS = decltype(rows)::value;
    constexpr bool LONG = decltype(with_long)::value;
    const int64_t cols = L * 16 / es, row_blocks = (P + 8 * ROWS - 1) / (8 * ROWS) * 8, items = (N + cols - 1) / cols * row_blocks;
    // long rows: a workgroup a CU
    const int64_t lcols = GA_LONG_LANES * 16 / es, strips = (N + lcols - 1) / lcols, slots = std::max<int64_t>(1, std::min(P, 256 / strips));
    const int64_t long_blocks = LONG ? (strips * slots + 7) / 8 * 8 : 0;
    hipLaunchKernelGGL((spmm_gather_kernel<decltype(dt), L, W, ROWS, LONG>), dim3((unsigned)(long_blocks + (items + 255) / 256 * 256)),
                       dim3(W * 64), 0, s, row_ptr, col_idx, val, capacity, P, (int)row_blocks, (int)items, (int)long_blocks, (int)slots,
                       (int)Q, d, N, R);
  };
  using I1 = std::integral_constant<int, 1>;
  using I8 = std::integral_constant<int, 8>;
  using I32 = std::integral_constant<int, 32>;
  using I64 = std::integral_constant<int, 64>;
  // Eight waves a row where eight rows a workgroup would leave half the chip without one (four: 64 x 2048 -> 2048 3.8 against 5.6 us, 256 x 512
  // -> 512 3.3 / 4.2; 1056 x 1376 -> 2080 25.5 / 21.7).  Four of them are as fast but where rows are full or nearly: 64 x 8192 -> 2048 bf16, 6 %, four /
  // eight 16.5 / 13.9, 1 % and one full row 156 / 91; 64 x 2048 -> 2048 36 / 27.
  const int64_t half = (int64_t)32 * 16 / es;
  const bool few = (P + 7) / 8 * ((N + half - 1) / half) < 128;
  auto shape = [&](auto dt, auto with_long) {
    if (few) launch(dt, I64{}, I8{}, I1{}, with_long); else launch(dt, I32{}, I8{}, I8{}, with_long);
  };
  // Of up to four rows none has more than four times the mean.
  const bool with_long = Q > GA_LONG_COLS && P > 4 && capacity > GA_LONG;
  auto type = [&](auto dt) { if (with_long) shape(dt, std::true_type{}); else shape(dt, std::false_type{}); };
  if (bf16) type(BF16{}); else type(F32{});
  FP4_CHECK_LAUNCH();
  return FP4_OK;
}
