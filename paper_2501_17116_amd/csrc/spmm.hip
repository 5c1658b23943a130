// The high-precision sparse product of outlier compensation (Sec. 3.2):
//   R[P x N] = S D,  S a P x Q CSR matrix with fp32 values (the clamped-away residual or its
//   transpose), D [Q x N] dense in the master dtype, fp32 accumulation.
// and the CSR transpose the weight-gradient pass needs (Delta_A^T dY).  bf16 D goes to the matrix cores
// (spmm_mfma.hip) as far as that path's 32-bit offsets and packing tables reach (24576 columns of S, 3.5 GiB of D) and
// as the matrix's entries are worth packing, which its packing decides on the device; the tiled kernel here takes fp32 D
// and the rest.  Small products of either type are one launch that gathers rows of D from L2 (spmm_gather.hip).
//
// S has density 2(1 - alpha) (about 2 %), scattered, plus a few nearly dense outlier channels.
// At that density and a large size neither a dense matrix-core product (50x wasted work) nor a row gather
// (every non-zero re-reads a row of D from L2) is acceptable, so the product of fp32 D is tiled the way
// a dense GEMM is, with plain fp32 FMAs:
//   * a workgroup of 1024 threads (512 where those go round the chip once) owns as many rows of R x 64 columns, one row per
//     thread, the 64 accumulators in registers;
//   * D is staged through LDS in slabs of 512 rows x 64 columns, widened to fp32 once per slab,
//     so a D element is fetched from L2 once per 1024 (512) output rows;
//   * a thread walks its row's entries (ascending columns) slab by slab: per non-zero 64 FMAs
//     against one LDS row.
// Rows much longer than the rest (the outlier channels of the transposed residual, spmm_long_limit) would
// stall their workgroup; they are left out of the tiled kernel and multiplied eight at a time as a dense matrix.
#include "fp4_common.h"
#include "fp4_measure.h"
#include "csr_mask.h"
#include "spmm_long.h"

#include <algorithm>
#include <type_traits>

namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));

constexpr int SP_ROWS = 1024;   // output rows per workgroup = threads, where there are rows enough
constexpr int SP_COLS = 64;     // output columns per workgroup
constexpr int SP_KS = 512;      // rows of D per LDS slab
// LDS chunk reads a lane has in flight before the FMAs that use them: more do not fit the 128 VGPRs of a 1024-thread
// workgroup, and on a full chip a smaller workgroup with more registers loses more through occupancy
constexpr int sp_rif(int rows) { return rows >= 1024 ? 4 : 8; }
constexpr int SP_WPR = SP_KS / 64;    // waves whose 64 x 64 tiles fit the slab at once
constexpr int SP_LD = SP_COLS;   // LDS row (floats), unpadded: see the lane swizzle in the kernel
constexpr int SP_XM = 15;        // lane bits that rotate the order in which a thread reads a D row

template <class DT>
FP4_D void load8g(const void* base, int64_t off, int valid, float (&v)[8]) {
  if (valid >= 8) {
    if constexpr (__is_same(DT, BF16)) {
      u32x4 r = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(base) + off);
      v[0] = u2f(r.x << 16); v[1] = u2f(r.x & 0xffff0000u);
      v[2] = u2f(r.y << 16); v[3] = u2f(r.y & 0xffff0000u);
      v[4] = u2f(r.z << 16); v[5] = u2f(r.z & 0xffff0000u);
      v[6] = u2f(r.w << 16); v[7] = u2f(r.w & 0xffff0000u);
    } else {
      const f32x4* p = reinterpret_cast<const f32x4*>(reinterpret_cast<const float*>(base) + off);
      f32x4 a = p[0], b = p[1];
      v[0] = a.x; v[1] = a.y; v[2] = a.z; v[3] = a.w;
      v[4] = b.x; v[5] = b.y; v[6] = b.z; v[7] = b.w;
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float f = 0.0f;
      if (e < valid) {
        if constexpr (__is_same(DT, BF16))
          f = bf16_bits_to_f32(reinterpret_cast<const uint16_t*>(base)[off + e]);
        else
          f = reinterpret_cast<const float*>(base)[off + e];
      }
      v[e] = f;
    }
  }
}

// A block of ROWS rows times the 64 columns of D from n0 on.  mine: whether the thread's row is to be written.
template <class DT, bool EARLY, int ROWS = SP_ROWS>
FP4_D void spmm_tile_block(const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col_idx,
                           const float* __restrict__ val, int64_t capacity, int64_t P, int64_t Q, const void* __restrict__ D,
                           int64_t N, float* __restrict__ R, int64_t block, int tid, bool mine, int64_t n0, float* slab, int* s_skip) {
  constexpr int RPP = ROWS / 8, RIF = sp_rif(ROWS);   // rows of D staged per pass (8 threads per row)
  static_assert(SP_KS % RPP == 0, "whole staging passes");
  const int64_t row = block * ROWS + tid;
  // Entry positions are kept as 32-bit offsets from the workgroup's first entry (a workgroup's
  // rows hold fewer than 2^31 entries: the launcher bounds Q); the base stays in scalar registers.
  const int64_t ebase = row_ptr[min(block * ROWS, P)];
  const int64_t long_limit = spmm_long_limit(row_ptr, P, Q, capacity);
  uint32_t cur = 0, end = 0;
  if (mine) {
    const int64_t b = row_ptr[row];
    int64_t e = max(min(row_ptr[row + 1], capacity), b);
    if (e - b > long_limit) e = b;   // long rows belong to the long-row kernels
    cur = (uint32_t)(b - ebase);
    end = (uint32_t)(e - ebase);
  }
  const int32_t* const cbase = col_idx + ebase;
  const float* const vbase = val + ebase;
  float acc[SP_COLS];
#pragma unroll
  for (int j = 0; j < SP_COLS; ++j) acc[j] = 0.0f;

  // staging map: 8 threads cover the 64 columns of a D row, RPP rows per pass
  const int s_unit = tid & 7, s_row = tid >> 3;
  const int64_t s_col = n0 + s_unit * 8;
  const int s_valid = s_col < N ? (int)min((int64_t)8, N - s_col) : 0;

  // The row's entries are fetched four at a time (one 16-byte request per array instead of
  // four 4-byte ones: every lane walks a different row, so requests, not bytes, are what the
  // cache path runs out of).  A quad may run past the row's end; what lies there is ignored.
  const uint32_t limit =   // entries that exist, as an offset
      (uint32_t)min(max(min(row_ptr[P], capacity) - ebase, (int64_t)0), (int64_t)0x7ffffff0);
  uint32_t qb = cur;
  int32_t cq[4] = {0x7fffffff, 0x7fffffff, 0x7fffffff, 0x7fffffff};
  float vq[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  auto load_quad = [&]() {
    if (qb + 4 <= limit) {
      const i32x4 c4 = *reinterpret_cast<const i32x4*>(cbase + qb);   // dword-aligned 16-byte loads
      const f32x4 v4 = *reinterpret_cast<const f32x4*>(vbase + qb);
      cq[0] = c4.x; cq[1] = c4.y; cq[2] = c4.z; cq[3] = c4.w;
      vq[0] = v4.x; vq[1] = v4.y; vq[2] = v4.z; vq[3] = v4.w;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        cq[i] = qb + i < limit ? cbase[qb + i] : 0x7fffffff;
        vq[i] = qb + i < limit ? vbase[qb + i] : 0.0f;
      }
    }
  };
  if (cur < end) load_quad();

  // Every lane gathers a different LDS row, so the bank a 16-byte read lands on cannot depend
  // on the row or the lanes collide at random.  Rows are unpadded (every row starts at bank 0)
  // and lane l reads the row's 16-byte chunks in the order j ^ (l & SP_XM): neighbouring lanes
  // always sit on different banks, whatever rows they read.  acc[4 j ..] of lane l therefore
  // holds columns 4 (j ^ (l & SP_XM)) ..; the final store undoes the permutation.
  const int swz = tid & SP_XM;
  // chunk j = jl + 8 jh sits at (jl ^ (swz & 7)) + 8 (jh ^ (swz >> 3)): eight lane constants
  // and two row bases instead of sixteen constants
  int xo[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) xo[j] = (j ^ (swz & 7)) * 4;
  const int hi_off = (swz >> 3) * 32;

  // EARLY (bf16 D, and workgroups with registers to spare): a wave requests its share of the next slab as soon as its own rows
  // are done with the current one (bf16: the registers of the read window are free then), so the round trip runs while
  // the slower waves finish instead of after the barrier.
  constexpr int UNIT = __is_same(DT, BF16) ? 1 : 2;   // 16-byte loads of eight elements
  static_assert(!EARLY || UNIT == 1 || ROWS < SP_ROWS, "registers");
  [[maybe_unused]] u32x4 nxt[SP_KS / RPP][UNIT];
  [[maybe_unused]] auto fetch_next = [&](int64_t k0n) {
#pragma unroll
    for (int ps = 0; ps < SP_KS / RPP; ++ps) {
      const int64_t r = k0n + ps * RPP + s_row;
      if constexpr (UNIT == 1) {
        nxt[ps][0] = u32x4{0u, 0u, 0u, 0u};
        if (r < Q && s_valid >= 8) nxt[ps][0] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(D) + r * N + s_col);
      } else {   // no branch: what stands in for rows past Q no entry names, and columns past N are not stored
        const u32x4* const at = reinterpret_cast<const u32x4*>(reinterpret_cast<const float*>(D) + min(r, Q - 1) * N + (s_valid >= 8 ? s_col : 0));
        nxt[ps][0] = at[0];
        nxt[ps][UNIT - 1] = at[1];
      }
    }
  };
  if constexpr (EARLY) {
    if (Q > 0) fetch_next(0);
  }

  for (int64_t k0 = 0; k0 < Q; k0 += SP_KS) {
    __syncthreads();
#pragma unroll
    for (int ps = 0; ps < SP_KS / RPP; ++ps) {
      const int r = ps * RPP + s_row;
      f32x4 a, b;
      if constexpr (EARLY && UNIT == 2) {
        a = __builtin_bit_cast(f32x4, nxt[ps][0]);
        b = __builtin_bit_cast(f32x4, nxt[ps][UNIT - 1]);
      } else if constexpr (EARLY) {
        const u32x4 u = nxt[ps][0];
        a = f32x4{u2f(u.x << 16), u2f(u.x & 0xffff0000u), u2f(u.y << 16), u2f(u.y & 0xffff0000u)};
        b = f32x4{u2f(u.z << 16), u2f(u.z & 0xffff0000u), u2f(u.w << 16), u2f(u.w & 0xffff0000u)};
      } else {
        float d[8];
        if (k0 + r < Q && s_valid > 0) load8g<DT>(D, (k0 + r) * N + s_col, s_valid, d);
        else {
#pragma unroll
          for (int e = 0; e < 8; ++e) d[e] = 0.0f;
        }
        a = f32x4{d[0], d[1], d[2], d[3]};
        b = f32x4{d[4], d[5], d[6], d[7]};
      }
      *reinterpret_cast<f32x4*>(&slab[r * SP_LD + s_unit * 8]) = a;
      *reinterpret_cast<f32x4*>(&slab[r * SP_LD + s_unit * 8 + 4]) = b;
    }
    __syncthreads();
    const int32_t k_end = (int32_t)min(k0 + SP_KS, Q);
    // The quad in registers always starts at the row's next entry, so its four entries are taken
    // with static indices and all lanes of a wave reload at the same point of the loop (one
    // wait per four entries instead of one in most iterations).  A lane that meets the slab's
    // end inside a quad fetches the quad at its new position right away: the request is in
    // flight while the next slab is staged.
    bool more = cur < end;
    while (more) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if (cur >= end || cq[i] >= k_end) { more = false; break; }
        ++cur;
        const float v = vq[i];
        const float* dr = &slab[(cq[i] - (int32_t)k0) * SP_LD];
        // A window of RIF chunk reads stays in flight: chunk g's FMAs are followed by the read
        // of chunk g + RIF into the registers they freed, in exactly this order.
        static_assert(SP_XM == 15 && SP_COLS == 64, "one chunk per swizzle constant");
        auto chunk = [&](int g) {
          return *reinterpret_cast<const f32x4*>(dr + ((g & 8) ? 32 - hi_off : hi_off) + xo[g & 7]);
        };
        f32x4 d4[RIF];
#pragma unroll
        for (int q = 0; q < RIF; ++q) d4[q] = chunk(q);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int g = 0; g < 16; ++g) {
          const f32x4 d = d4[g % RIF];
          acc[4 * g + 0] = fmaf(v, d.x, acc[4 * g + 0]);
          acc[4 * g + 1] = fmaf(v, d.y, acc[4 * g + 1]);
          acc[4 * g + 2] = fmaf(v, d.z, acc[4 * g + 2]);
          acc[4 * g + 3] = fmaf(v, d.w, acc[4 * g + 3]);
          if (g + RIF < 16) d4[g % RIF] = chunk(g + RIF);
          __builtin_amdgcn_sched_barrier(0);
        }
        // the sums are final here: the optimizer may not sink a step's FMAs into the block where
        // the exits of all four steps meet (it did, and kept all 16 chunks alive across it)
#pragma unroll
        for (int j = 0; j < SP_COLS; j += 16)
          asm volatile("" : "+v"(acc[j]), "+v"(acc[j + 1]), "+v"(acc[j + 2]), "+v"(acc[j + 3]), "+v"(acc[j + 4]),
                            "+v"(acc[j + 5]), "+v"(acc[j + 6]), "+v"(acc[j + 7]), "+v"(acc[j + 8]), "+v"(acc[j + 9]),
                            "+v"(acc[j + 10]), "+v"(acc[j + 11]), "+v"(acc[j + 12]), "+v"(acc[j + 13]),
                            "+v"(acc[j + 14]), "+v"(acc[j + 15]));
      }
      if (more) {
        if (cur < end) { qb = cur; load_quad(); }
        else more = false;
      }
    }
    if (cur < end && cur != qb) { qb = cur; load_quad(); }
    if constexpr (EARLY) {
      if (k0 + SP_KS < Q) fetch_next(k0 + SP_KS);
    }
  }
  // A lane's 64 sums belong to one row of R (lanes are N floats apart); they go through LDS once
  // more so that the stores run along rows: 16 lanes x 16 B per row, four rows per instruction.
  // A wave's 64 x 64 tile takes 16 KiB, so the workgroup stores in two rounds of eight waves.
  bool skip = !mine;   // rows outside the matrix, and rows that other kernels write (long ones)
  if (!skip) skip = min(row_ptr[row + 1], capacity) - row_ptr[row] > spmm_long_limit(row_ptr, P, Q, capacity);
  s_skip[tid] = skip ? 1 : 0;
  __syncthreads();   // everyone is done with the last slab
  const int lane = tid & 63, wave = tid >> 6;
  float* const tile = slab + (wave % SP_WPR) * (64 * SP_COLS);
#pragma unroll 1
  for (int round = 0; round < (ROWS / 64 + SP_WPR - 1) / SP_WPR; ++round) {
    if (wave / SP_WPR == round) {
#pragma unroll
      for (int j = 0; j < SP_COLS; j += 4)
        *reinterpret_cast<f32x4*>(&tile[lane * SP_COLS + (j ^ (swz * 4))]) = f32x4{acc[j], acc[j + 1], acc[j + 2], acc[j + 3]};
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      const int tc = lane & 15;
      const int64_t col = n0 + tc * 4;   // N is a multiple of 8: a 4-column chunk is inside or outside
      if (col < N) {
#pragma unroll 4
        for (int ps = 0; ps < 16; ++ps) {
          const int r = 4 * ps + (lane >> 4);
          if (!s_skip[wave * 64 + r]) {
            const f32x4 t = *reinterpret_cast<const f32x4*>(&tile[r * SP_COLS + tc * 4]);
            *reinterpret_cast<f32x4*>(R + (block * ROWS + wave * 64 + r) * N + col) = t;
          }
        }
      }
    }
    __syncthreads();
  }
}

template <class DT, int ROWS = SP_ROWS>
__global__ __launch_bounds__(ROWS) void spmm_tile_kernel(const int64_t* __restrict__ row_ptr,
                                                         const int32_t* __restrict__ col_idx,
                                                         const float* __restrict__ val, int64_t capacity,
                                                         int64_t P, int64_t Q, const void* __restrict__ D,
                                                         int64_t N, float* __restrict__ R) {
  __shared__ __attribute__((aligned(16))) float slab[SP_KS * SP_LD];
  __shared__ int s_skip[ROWS];
  spmm_tile_block<DT, __is_same(DT, BF16) || (ROWS < SP_ROWS), ROWS>(row_ptr, col_idx, val, capacity, P, Q, D, N, R, blockIdx.x, threadIdx.x,
                                                 (int64_t)blockIdx.x * ROWS + threadIdx.x < P, (int64_t)blockIdx.y * SP_COLS,
                                                 slab, s_skip);
}

// ---- long rows -------------------------------------------------------------------------------
// The list of long rows (spmm_long.h) as a launch of its own, for the fp32 kernel; the matrix-core path has one
// workgroup of its packing kernel make it.
__global__ __launch_bounds__(1024) void find_long_rows_kernel(const int64_t* row_ptr, int64_t P, int64_t Q, int64_t capacity,
                                                              int32_t* list, int32_t* count) {
  find_long_rows<1024>(row_ptr, P, Q, capacity, list, count);
}

// Long rows (outlier channels of the transposed residual: nearly dense) are multiplied as a small dense matrix so that D is
// streamed once per group of LD_LB of them instead of once per row: a workgroup takes a span of D's rows x 512 columns x
// LD_LB long rows, scatters those rows' values for as many rows of the span as fit into an LDS table V[row][long row] (zero
// where a row has no entry), and every lane keeps LD_LB x 8 accumulators for its 8 columns while the eight waves
// split the table's rows.  Partial sums per span go to a scratch array and are added in span
// order by a second kernel, so the result does not depend on scheduling.
constexpr int LD_LB = 8;         // long rows per workgroup pass (64 accumulators a lane: two workgroups share a CU)
constexpr int LD_SLICE = 512;    // most rows of D in the table, and in a slice
constexpr int LD_CAP = 32;       // long rows up to which a span is one slice; sizes the partial sums' scratch
constexpr int LD_COLS = 512;     // columns per workgroup (64 lanes x 8)
constexpr int LD_WAVES = 8;      // waves per workgroup; they split the slice's rows
// Rows of D per slice: 512, halved (to 64 at least) while that leaves fewer than 256 workgroups for a group of long rows,
// whose stream of D would then run on a part of the chip (512 against this: 1056 x 1376 x 2080 step, both products 35 -> 13
// us; 2048^3 fp32 44 -> 22).  Aiming at 512 workgroups gave nothing more and made the summing of the slices longer.
inline int ld_slice(int64_t Q, int64_t N) {
  int slice = LD_SLICE;
  while (slice > 64 && (Q + slice - 1) / slice * ((N + LD_COLS - 1) / LD_COLS) < 256) slice /= 2;
  return slice;
}
// Slices a span has with n_long long rows: as few as leave room for every row's sums of every span in the scratch, which has
// LD_CAP rows' for every slice.  A single span goes straight to R and takes none.  4096 x 2048 -> 2048, 40 long rows of 0.4,
// fp32: those beyond LD_CAP over the whole of D by four workgroups 148 us, row by row 117, this 68; 4096 x 4096 -> 4096, 256
// of 0.5, bf16: row by row 3162, all in the tiled kernel 1509, this 230.
FP4_D int ld_span(int n_long, int slices) {
  if (n_long <= LD_CAP) return 1;
  int m = (n_long + LD_CAP - 1) / LD_CAP;
  while (m < slices && (int64_t)((slices + m - 1) / m) * n_long > (int64_t)LD_CAP * slices) ++m;
  return max(1, min(m, slices));
}
constexpr int LD_TABLE = LD_SLICE * LD_LB > LD_WAVES * 2 * LD_COLS ? LD_SLICE * LD_LB : LD_WAVES * 2 * LD_COLS;   // floats

// Main loop of spmm_long_dense_kernel for NL accumulated long rows: adds the slice's products to the wave's sums.
template <class DT, int NL>
FP4_D void long_dense_add(int tid, const float* V, const void* D, int m0, int rows_here, int64_t N, float (&acc)[NL][8]) {
  const int lane = tid & 63, wave = tid >> 6;
  const int64_t col = (int64_t)blockIdx.x * LD_COLS + lane * 8;
  const int valid = col < N ? (int)min((int64_t)8, N - col) : 0;
  constexpr int UN = NL <= 4 ? 6 : 4;   // rows in flight per wave
  auto fma_row = [&](int row, const float (&d)[8]) {
    const f32x4* vr = reinterpret_cast<const f32x4*>(&V[row * LD_LB]);
#pragma unroll
    for (int q = 0; q < NL / 4; ++q) {
      const f32x4 v4 = vr[q];   // same address in every lane: an LDS broadcast
      const float v[4] = {v4.x, v4.y, v4.z, v4.w};
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[q * 4 + i][e] = fmaf(v[i], d[e], acc[q * 4 + i][e]);
    }
  };
  bool done = false;
  if constexpr (__is_same(DT, BF16)) {
    if (valid == 8) {
      // Whole 16-byte units of bf16: the rows of the next turn are requested before the FMAs of this
      // one, as raw words (four registers a row), so a wave always has a turn's loads in flight.
      done = true;
      const uint16_t* const base = reinterpret_cast<const uint16_t*>(D) + (int64_t)m0 * N + col;
      u32x4 cur[UN], nxt[UN];
      const u32x4 zero = {0u, 0u, 0u, 0u};
      auto request = [&](u32x4 (&dst)[UN], int r0) {
#pragma unroll
        for (int u = 0; u < UN; ++u) {
          const int row = r0 + LD_WAVES * u;   // wave-uniform
          dst[u] = row < rows_here ? *reinterpret_cast<const u32x4*>(base + (int64_t)row * N) : zero;
        }
      };
      request(cur, wave);
      for (int r = wave; r < rows_here; r += LD_WAVES * UN) {
        request(nxt, r + LD_WAVES * UN);
#pragma unroll
        for (int u = 0; u < UN; ++u) {
          const int row = r + LD_WAVES * u;
          if (row < rows_here) {
            const u32x4 w = cur[u];
            const float d[8] = {u2f(w.x << 16), u2f(w.x & 0xffff0000u), u2f(w.y << 16), u2f(w.y & 0xffff0000u),
                                u2f(w.z << 16), u2f(w.z & 0xffff0000u), u2f(w.w << 16), u2f(w.w & 0xffff0000u)};
            fma_row(row, d);
          }
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) cur[u] = nxt[u];
      }
    }
  }
  if (!done && valid > 0) {
    int r = wave;
    for (; r + LD_WAVES * (UN - 1) < rows_here; r += LD_WAVES * UN) {
      float d[UN][8];
#pragma unroll
      for (int u = 0; u < UN; ++u) load8g<DT>(D, (int64_t)(m0 + r + LD_WAVES * u) * N + col, valid, d[u]);
#pragma unroll
      for (int u = 0; u < UN; ++u) fma_row(r + LD_WAVES * u, d[u]);
    }
    for (; r < rows_here; r += LD_WAVES) {
      float d[8];
      load8g<DT>(D, (int64_t)(m0 + r) * N + col, valid, d);
      fma_row(r, d);
    }
  }
}

// Adds the waves' sums, two long rows at a time, in wave order, and hands out(long row, column, sum) the columns in range.
template <int NL, class Out>
FP4_D void long_dense_reduce(int tid, float* V, const float (&acc)[NL][8], int64_t N, int nl, Out out) {
  const int lane = tid & 63, wave = tid >> 6;
  float* red = V;   // [LD_WAVES][2 rows][512 columns]
  static_assert(LD_WAVES * 2 * LD_COLS <= LD_TABLE, "reduction buffer fits the table");
#pragma unroll
  for (int q = 0; q < NL / 2; ++q) {
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      float* dst = red + ((wave * 2 + i) * LD_COLS + lane * 8);
      *reinterpret_cast<f32x4*>(dst) = f32x4{acc[q * 2 + i][0], acc[q * 2 + i][1], acc[q * 2 + i][2], acc[q * 2 + i][3]};
      *reinterpret_cast<f32x4*>(dst + 4) = f32x4{acc[q * 2 + i][4], acc[q * 2 + i][5], acc[q * 2 + i][6], acc[q * 2 + i][7]};
    }
    __syncthreads();
    // 2 rows x 512 columns = 1024 sums: two per thread
    for (int t2 = tid; t2 < 2 * LD_COLS; t2 += LD_WAVES * 64) {
      const int ri = t2 / LD_COLS, c = t2 % LD_COLS;
      const int64_t gcol = (int64_t)blockIdx.x * LD_COLS + c;
      if (q * 2 + ri < nl && gcol < N) {
        float sum = 0.0f;
#pragma unroll
        for (int w = 0; w < LD_WAVES; ++w) sum += red[(w * 2 + ri) * LD_COLS + c];
        out(q * 2 + ri, gcol, sum);
      }
    }
  }
}

// Places the values of nl long rows for the D rows m0 .. m0 + rows_here - 1 into the zeroed table V[row][long row]; row
// l's entries of the slice begin at s_lo[l], and *s_rep is 0 on entry.  Columns ascend inside a row.  Where they are
// distinct, the entries of the slice are among the first `slice` from the start and every one has a word of its own:
// item j = (long row j / slice, offset j % slice), four items a thread at a time, their loads issued together.  A row that
// repeats a column is seen by an entry that equals the one before it (or by one more entry than there are columns): then
// the first entry of each run writes the run's sum, in the entries' order.
FP4_D void ld_place(int tid, float* V, const int32_t* col_idx, const float* val, const int64_t* s_lo, const int64_t* s_en,
                    int* s_rep, int nl, int m0, int rows_here, int slice) {
  constexpr int THREADS = LD_WAVES * 64;
  const int shift = 31 - __builtin_clz(slice);   // a power of two
  const int items = nl * slice;
  int32_t beyond = 0x7fffffff;   // the entry after as many as there are columns
  if (tid < nl && s_lo[tid] + slice < s_en[tid]) beyond = col_idx[s_lo[tid] + slice];
  for (int j0 = tid; j0 < items; j0 += 4 * THREADS) {
    int32_t c[4], before[4];
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int j = j0 + u * THREADS;
      const int l = min(j >> shift, nl - 1);
      const int64_t i = s_lo[l] + (j & (slice - 1));
      const bool ok = j < items && i < s_en[l];
      c[u] = ok ? col_idx[i] : 0x7fffffff;
      v[u] = ok ? val[i] : 0.0f;
      before[u] = ok && i > s_lo[l] ? col_idx[i - 1] : -1;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int r = c[u] - m0;
      if (r < 0 || r >= rows_here) continue;
      if (before[u] == c[u]) *s_rep = 1;
      else V[r * LD_LB + min((j0 + u * THREADS) >> shift, nl - 1)] = v[u];
    }
  }
  if (beyond < m0 + rows_here) *s_rep = 1;
  __syncthreads();
  if (*s_rep == 0) return;
  for (int l = 0; l < nl; ++l)
    for (int64_t i = s_lo[l] + tid; i < s_en[l]; i += THREADS) {
      const int32_t c = col_idx[i];
      const int r = c - m0;
      if (r >= rows_here) break;
      if (r < 0 || (i > s_lo[l] && col_idx[i - 1] == c)) continue;
      float sum = val[i];
      for (int64_t k = i + 1; k < s_en[l] && col_idx[k] == c; ++k) sum += val[k];
      V[r * LD_LB + l] = sum;
    }
  __syncthreads();
}

// The sums of nl long rows, at most NL, over the rows of D in the table: to[l][column], added to what is there unless `set`.
template <class DT, int NL>
FP4_D void long_dense_turn(int tid, float* V, const void* D, int m0, int rows_here, int64_t N, int nl, bool set, float* to,
                            const int32_t* rows) {
  float acc[NL][8];
#pragma unroll
  for (int l = 0; l < NL; ++l)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[l][e] = 0.0f;
  long_dense_add<DT>(tid, V, D, m0, rows_here, N, acc);
  long_dense_reduce(tid, V, acc, N, nl, [&](int l, int64_t col, float sum) {
    float* const at = to + (rows ? (int64_t)rows[l] : (int64_t)l) * N + col;
    *at = set ? sum : *at + sum;   // the thread that wrote it
  });
}

// Items (group of eight long rows, span), as many per column block as there are; blockIdx.y takes every gridDim.y-th.  The
// sums leave the registers after every turn of a span: kept across the next one's table they spill.
template <class DT>
__global__ __launch_bounds__(LD_WAVES * 64, 4) void spmm_long_dense_kernel(const int64_t* row_ptr, const int32_t* col_idx,
                                                              const float* val, int64_t capacity,
                                                              const int32_t* list, const int32_t* count,
                                                              const void* D, int Q, int64_t N, int slice, int slices,
                                                              float* part, float* R) {
  __shared__ __attribute__((aligned(16))) float V[LD_TABLE];   // 32 KiB, reused for the wave reduction
  __shared__ int64_t s_lo[LD_LB], s_en[LD_LB];
  __shared__ int s_rep;
  const int n_long = *count;
  if (n_long == 0) return;
  const int groups = (n_long + LD_LB - 1) / LD_LB;
  const int span = ld_span(n_long, slices), spans = span == 1 ? slices : (slices + span - 1) / span;
  int rows_a_turn = slice;   // what of a span the table takes at a time: a power of two
  while (2 * rows_a_turn <= min(LD_SLICE, span * slice)) rows_a_turn *= 2;
  for (int item = blockIdx.y; item < groups * spans; item += gridDim.y) {
    const int group = item < spans ? 0 : item / spans, at = item - group * spans;   // its span
    const int g0 = group * LD_LB, nl = min(LD_LB, n_long - g0);
    const int first = at * span * slice, last = min(first + span * slice, Q);   // Q < 2^21
#pragma unroll 1
    for (int m0 = first; m0 < last; m0 += rows_a_turn) {
      int tid = threadIdx.x;
      asm volatile("" : "+v"(tid));   // a lane's constants are formed again for each turn: kept across, they spill
      const int lane = tid & 63, wave = tid >> 6;
      const int rows_here = min(rows_a_turn, last - m0);
      __syncthreads();   // everyone is done with the table
      for (int i = tid; i < rows_a_turn * LD_LB; i += LD_WAVES * 64) V[i] = 0.0f;
      if (tid == 0) s_rep = 0;
      // A wave per long row finds where its entries for the turn begin, 64 probes a round (a bisection by one lane was a
      // chain of fourteen round trips, a third of the workgroup's time), from the row's start or the turn before's.
      static_assert(LD_LB <= LD_WAVES, "a wave per long row");
      if (wave < nl) {
        const int64_t row = list[g0 + wave];
        int64_t lo = m0 == first ? row_ptr[row] : s_lo[wave];
        const int64_t en = min(row_ptr[row + 1], capacity);
        int64_t hi = en;
        while (lo < hi) {   // the first entry with column >= m0 lies in [lo, hi]
          const int64_t step = (hi - lo + 63) / 64;
          const int64_t at = lo + lane * step;
          const int below = __popcll(__ballot(at < hi && col_idx[min(at, hi - 1)] < m0));   // columns ascend
          if (below == 0) hi = lo;
          else {
            hi = min(hi, lo + below * step);
            lo += (below - 1) * step + 1;
          }
        }
        if (lane == 0) {
          s_lo[wave] = lo;
          s_en[wave] = en;
        }
      }
      __syncthreads();   // table zeroed, starts known
      ld_place(tid, V, col_idx, val, s_lo, s_en, &s_rep, nl, m0, rows_here, rows_a_turn);
      float* const to = spans > 1 ? part + ((int64_t)at * n_long + g0) * N : R;
      const int32_t* const rows = spans > 1 ? nullptr : list + g0;
      if (nl <= 4)   // sums only for as many long rows as there are (4 or 8): usually a handful
        long_dense_turn<DT, 4>(tid, V, D, m0, rows_here, N, nl, m0 == first, to, rows);
      else
        long_dense_turn<DT, LD_LB>(tid, V, D, m0, rows_here, N, nl, m0 == first, to, rows);
    }
  }
}

// The 256 columns from `first` on of one long row from its entries alone: 32 columns at a time, 4 column groups of 8 x
// THREADS / 4 entry lanes; entry lane l takes every THREADS / 4-th entry from the l-th on; the lanes' sums are added in order.
template <class DT, int THREADS>
FP4_D void long_row_entries(const int64_t* row_ptr, const int32_t* col_idx, const float* val, int64_t capacity, int64_t row,
                            int64_t first, const void* D, int64_t N, float* R, float* part) {
  constexpr int LANES = THREADS / 4;
  const int cg = threadIdx.x & 3, el = threadIdx.x >> 2;
  const int64_t b = row_ptr[row], en = min(row_ptr[row + 1], capacity);
  for (int64_t n0 = first; n0 < min(first + 256, N); n0 += 32) {
    const int64_t col = n0 + cg * 8;
    const int valid = col < N ? (int)min((int64_t)8, N - col) : 0;
    float acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.0f;
    if (valid > 0) {
      for (int64_t i = b + el; i < en; i += LANES) {
        const int32_t c = col_idx[i];
        const float s = val[i];
        float d[8];
        load8g<DT>(D, (int64_t)c * N + col, valid, d);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = fmaf(s, d[e], acc[e]);
      }
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) part[el * 32 + cg * 8 + e] = acc[e];
    __syncthreads();
    if (threadIdx.x < 32) {
      float sum = 0.0f;
      for (int l = 0; l < LANES; ++l) sum += part[l * 32 + threadIdx.x];
      const int64_t c1 = n0 + threadIdx.x;
      if (c1 < N) R[row * N + c1] = sum;
    }
    __syncthreads();
  }
}

// What the dense path leaves to do for the 256 columns from `first` on, every rows_apart-th long row from row0 on: the
// spans' partial sums are added up (each 256 threads take every so many-th span, their sums are added in order), and where a
// row's sum is infinite or NaN the row's columns are summed from its entries instead, since the table's zeros times an
// infinity of D in a column the row has no entry in are NaN.  part: 8 THREADS floats.
template <class DT, int THREADS>
FP4_D void finish_long_rows(const int64_t* row_ptr, const int32_t* col_idx, const float* val, int64_t capacity,
                            const int32_t* list, int n_long, int row0, int rows_apart, const float* partial, int slices,
                            int64_t first, const void* D, int64_t N, float* R, float* part) {
  constexpr int PARTS = THREADS / 256;
  const int c = threadIdx.x & 255, q = threadIdx.x >> 8;
  const int64_t n = first + c;
  if (row0 >= n_long) return;
  const int span = ld_span(n_long, slices), spans = span == 1 ? slices : (slices + span - 1) / span;
  for (int li = row0; li < n_long; li += rows_apart) {
    float* const r = R + (int64_t)list[li] * N;
    float sum = 0.0f;
    if (n < N) {
      if (spans > 1) {
        const int64_t step = (int64_t)PARTS * n_long * N;
        const float* p = partial + ((int64_t)q * n_long + li) * N + n;
        for (int s0 = q; s0 < spans; s0 += 8 * PARTS) {   // eight loads in flight, added in span order
          float v[8];
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            v[k] = s0 + k * PARTS < spans ? *p : 0.0f;
            p += step;
          }
#pragma unroll
          for (int k = 0; k < 8; ++k) sum += v[k];
        }
      } else if (q == 0) {
        sum = r[n];
      }
    }
    if constexpr (PARTS > 1) {
      part[threadIdx.x] = sum;
      __syncthreads();
      if (q == 0) {
#pragma unroll
        for (int k = 1; k < PARTS; ++k) sum += part[k * 256 + c];
      }
    }
    if (n < N && q == 0 && spans > 1) r[n] = sum;
    if (__syncthreads_or(q == 0 && (f2u(sum) & 0x7f800000u) == 0x7f800000u))
      long_row_entries<DT, THREADS>(row_ptr, col_idx, val, capacity, list[li], first, D, N, R, part);
  }
}

constexpr int LF_ROWS = 32;   // long rows side by side
template <class DT>
__global__ __launch_bounds__(256) void spmm_finish_long_kernel(const int64_t* row_ptr, const int32_t* col_idx,
                                                               const float* val, int64_t capacity, const int32_t* list,
                                                               const int32_t* count, const float* partial, int slices,
                                                               const void* D, int64_t N, float* R) {
  __shared__ float part[8 * 256];
  finish_long_rows<DT, 256>(row_ptr, col_idx, val, capacity, list, *count, blockIdx.y, LF_ROWS, partial, slices,
                       (int64_t)blockIdx.x * 256, D, N, R, part);
}

// After the packed product and the dense path, one launch for what both leave.  The first long_blocks workgroups finish the
// long rows; the other tiles.x * tiles.y take the rows that the packed product left (usually none: the workgroup leaves at
// once), each every tiles.y-th column block.  512 of them, two rounds of one a CU: an idle launch is over in 5 us (one
// workgroup a block: 13), a full one takes about as long as with one a block (16384 x 4096 -> 12288, 6 % of two-term values,
// the product: 256 workgroups 3406 us, 384 4107, 512 3179, 1024 3151, one a block 3158; the tiled kernel alone 2890).
__global__ __launch_bounds__(SP_ROWS) void spmm_rest_kernel(const int64_t* __restrict__ row_ptr,
                                                            const int32_t* __restrict__ col_idx,
                                                            const float* __restrict__ val, int64_t capacity,
                                                            int64_t P, int64_t Q, const void* __restrict__ D,
                                                            int64_t N, float* __restrict__ R, SpmmRest rest, dim3 tiles,
                                                            unsigned long_blocks, const int32_t* list, const int32_t* count,
                                                            const float* partial, int slices) {
  __shared__ __attribute__((aligned(16))) float slab[SP_KS * SP_LD];
  __shared__ int s_skip[SP_ROWS];
  if (blockIdx.x < long_blocks) {
    const unsigned blocks = (unsigned)((N + 255) / 256), apart = long_blocks / blocks;
    finish_long_rows<BF16, SP_ROWS>(row_ptr, col_idx, val, capacity, list, *count, blockIdx.x / blocks, apart, partial, slices,
                                    (int64_t)(blockIdx.x % blocks) * 256, D, N, R, slab);
    return;
  }
  __shared__ bool s_mine[SP_ROWS];
  const unsigned tile = blockIdx.x - long_blocks;
  const int64_t block = tile % tiles.x;
  bool mine = false;
  if (block * SP_ROWS + threadIdx.x < P) {
    const uint32_t group = (uint32_t)((block * SP_ROWS + threadIdx.x) >> 4);   // P < 2^31: the list's rows have 32 bits
    const uint32_t bundle = rest.groups == 3 ? group / 3u : group >> (rest.groups - 1);
    mine = rest.steps[bundle] < 0 || rest.redo[bundle] != 0;
  }
  s_mine[threadIdx.x] = mine;
  if (!__syncthreads_or(mine)) return;
  for (int64_t n0 = (int64_t)(tile / tiles.x) * SP_COLS; n0 < N; n0 += (int64_t)tiles.y * SP_COLS) {
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));   // a lane's constants are formed again for each column block: kept across, they spill
    spmm_tile_block<BF16, false>(row_ptr, col_idx, val, capacity, P, Q, D, N, R, block, tid, s_mine[tid], n0, slab, s_skip);
  }
}

// ---- CSR transpose (P x Q -> Q x P) -----------------------------------------------------------
__global__ void fill_i32_kernel(int32_t* p, int64_t n, int32_t v) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Column counts with a workgroup-private LDS histogram when the column range fits.
constexpr int CNT_LDS = 16384;
__global__ __launch_bounds__(256) void csr_count_cols_kernel(const int32_t* col_idx, const int64_t* nnz,
                                                             int64_t capacity, int64_t Q, int32_t* cnt) {
  __shared__ int32_t h[CNT_LDS];
  const int64_t n = min((int64_t)*nnz, capacity);
  const bool use_lds = Q <= CNT_LDS;
  if (use_lds) {
    for (int i = threadIdx.x; i < Q; i += 256) h[i] = 0;
    __syncthreads();
  }
  for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (int64_t)gridDim.x * 256) {
    if (use_lds) atomicAdd(&h[col_idx[i]], 1);
    else atomicAdd(&cnt[col_idx[i]], 1);
  }
  if (use_lds) {
    __syncthreads();
    for (int i = threadIdx.x; i < Q; i += 256)
      if (h[i]) atomicAdd(&cnt[i], h[i]);
  }
}

// ptr[0] = 0, ptr[i+1] = sum cnt[0..i].  One workgroup.
__global__ __launch_bounds__(1024) void scan_counts32_kernel(const int32_t* cnt, int64_t n, int64_t* ptr) {
  __shared__ long long s[1024];
  __shared__ long long carry;
  if (threadIdx.x == 0) { carry = 0; ptr[0] = 0; }
  __syncthreads();
  for (int64_t base = 0; base < n; base += 1024) {
    const int64_t i = base + threadIdx.x;
    s[threadIdx.x] = i < n ? cnt[i] : 0;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
      long long add = threadIdx.x >= o ? s[threadIdx.x - o] : 0;
      __syncthreads();
      s[threadIdx.x] += add;
      __syncthreads();
    }
    if (i < n) ptr[i + 1] = carry + s[threadIdx.x];
    __syncthreads();
    if (threadIdx.x == 1023) carry += s[1023];
    __syncthreads();
  }
}

// Unordered fill: entry (row, col) goes to some slot of column col's segment.
__global__ __launch_bounds__(256) void csr_transpose_fill_kernel(const int64_t* row_ptr, const int32_t* col_idx,
                                                                 const float* val, int64_t rows, int64_t capacity,
                                                                 const int64_t* t_ptr, int32_t* cursor,
                                                                 int32_t* u_idx, float* u_val) {
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (row >= rows) return;
  const int64_t b = row_ptr[row], e = min(row_ptr[row + 1], capacity);
  for (int64_t i = b + lane; i < e; i += 64) {
    const int32_t c = col_idx[i];
    const int64_t pos = t_ptr[c] + atomicAdd(&cursor[c], 1);
    u_idx[pos] = (int32_t)row;
    u_val[pos] = val[i];
  }
}

// ---- transpose as a stable counting sort on the column (csr_mask.h), its three passes by themselves -------------------------
template <int QMAX>   // columns the LDS masks are laid out for (the launcher picks the smallest that fits)
__global__ __launch_bounds__(MB_THREADS) void csr_mask_count_kernel(MbArgs m) {
  __shared__ MbCountShared<QMAX> sh;
  mb_count<QMAX, MB_THREADS>(m, blockIdx.x, sh);
}

// 64 columns a workgroup; its four waves split the blocks into quarters: sum, exchange, rescan.
__global__ __launch_bounds__(256) void csr_mask_scan_kernel(MbArgs m) {
  const int lane = threadIdx.x & 63, quarter = threadIdx.x >> 6;
  const int64_t Q = m.Q, c = (int64_t)blockIdx.x * 64 + lane;
  const int per = (m.nblocks + 3) / 4;
  const int b0 = quarter * per, b1 = min(m.nblocks, b0 + per);
  __shared__ uint32_t s_q[4][64];
  uint32_t sum = 0;
  if (c < Q) {
    int bi = b0;
    for (; bi + 15 < b1; bi += 16) {   // sixteen independent loads at a time
      uint32_t v[16];
#pragma unroll
      for (int j = 0; j < 16; ++j) v[j] = m.cnt8[(int64_t)(bi + j) * Q + c];
#pragma unroll
      for (int j = 0; j < 16; ++j) sum += v[j];
    }
    for (; bi < b1; ++bi) sum += m.cnt8[(int64_t)bi * Q + c];
  }
  s_q[quarter][lane] = sum;
  __syncthreads();
  if (c >= Q) return;
  uint32_t run = 0;
  for (int q = 0; q < quarter; ++q) run += s_q[q][lane];
  if (quarter == 3) m.cnt[c] = (int32_t)(run + sum);
  int bi = b0;
  for (; bi + 15 < b1; bi += 16) {
    uint32_t v[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) v[j] = m.cnt8[(int64_t)(bi + j) * Q + c];
#pragma unroll
    for (int j = 0; j < 16; ++j) { m.ex[(int64_t)(bi + j) * Q + c] = run; run += v[j]; }
  }
  for (; bi < b1; ++bi) { m.ex[(int64_t)bi * Q + c] = run; run += m.cnt8[(int64_t)bi * Q + c]; }
}

template <int QMAX, MbFrom FROM>
__global__ __launch_bounds__(MB_THREADS) void csr_mask_fill_kernel(MbArgs m) {
  __shared__ MbFillShared<QMAX, FROM> sh;
  mb_fill<QMAX, FROM>(m, blockIdx.x, sh);
}

// Order every segment by index (the indices inside a segment are distinct): an entry's final
// slot is the number of smaller indices in its segment.  One thread per entry; the segment is
// found by bisection on t_ptr.  Makes the transposed matrix, and so the sums over it,
// independent of the order the atomics above happened to take.
__global__ __launch_bounds__(256) void csr_rank_sort_kernel(const int64_t* t_ptr, int64_t Q, const int32_t* u_idx,
                                                            const float* u_val, int32_t* t_idx, float* t_val) {
  const int64_t e = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int64_t total = t_ptr[Q];
  if (e >= total) return;
  int64_t lo = 0, hi = Q;   // largest seg with t_ptr[seg] <= e
  while (hi - lo > 1) {
    const int64_t mid = (lo + hi) >> 1;
    if (t_ptr[mid] <= e) lo = mid; else hi = mid;
  }
  const int64_t b = t_ptr[lo], en = t_ptr[lo + 1];
  const int32_t key = u_idx[e];
  int64_t rank = 0;
  for (int64_t j = b; j < en; ++j) rank += u_idx[j] < key ? 1 : 0;
  t_idx[b + rank] = key;
  t_val[b + rank] = u_val[e];
}

// Same ordering in linear time when the index range fits an LDS bitmap: one workgroup per
// segment marks the indices present, turns the bitmap's word counts into an exclusive prefix,
// and an entry's slot is the number of marked indices below its own.
constexpr int BM_WORDS = 8000;   // bitmap words (plus as many prefix words) within 64 KiB of LDS: indices < 256000
__global__ __launch_bounds__(256) void csr_bitmap_sort_kernel(const int64_t* seg_ptr, int64_t nidx, int64_t capacity,
                                                              const int32_t* u_idx, const float* u_val,
                                                              int32_t* t_idx, float* t_val) {
  extern __shared__ uint32_t bm_lds[];
  __shared__ uint32_t blk_sum[256];
  const int nwords = (int)((nidx + 31) / 32);
  uint32_t* const bits = bm_lds;            // [nwords]
  uint32_t* const pre = bm_lds + nwords;    // [nwords] marked indices before each word
  const int64_t seg = blockIdx.x;
  const int64_t b = seg_ptr[seg], en = seg_ptr[seg + 1];
  if (en > capacity) return;                // truncated output
  const int L = (int)(en - b);
  if (L == 0) return;
  if (L == 1) {
    if (threadIdx.x == 0) { t_idx[b] = u_idx[b]; t_val[b] = u_val[b]; }
    return;
  }
  for (int i = threadIdx.x; i < nwords; i += 256) bits[i] = 0;
  __syncthreads();
  for (int i = threadIdx.x; i < L; i += 256) {
    const uint32_t k = (uint32_t)u_idx[b + i];
    atomicOr(&bits[k >> 5], 1u << (k & 31));
  }
  __syncthreads();
  // exclusive prefix over words: each thread scans a contiguous run, then the runs are offset
  const int per = (nwords + 255) / 256;
  const int w0 = threadIdx.x * per, w1 = min(nwords, w0 + per);
  uint32_t run = 0;
  for (int w = w0; w < w1; ++w) { pre[w] = run; run += __popc(bits[w]); }
  blk_sum[threadIdx.x] = run;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t acc = 0;
    for (int t = 0; t < 256; ++t) { const uint32_t c = blk_sum[t]; blk_sum[t] = acc; acc += c; }
  }
  __syncthreads();
  const uint32_t off = blk_sum[threadIdx.x];
  for (int w = w0; w < w1; ++w) pre[w] += off;
  __syncthreads();
  for (int i = threadIdx.x; i < L; i += 256) {
    const uint32_t k = (uint32_t)u_idx[b + i];
    const int w = (int)(k >> 5);
    const uint32_t rank = pre[w] + __popc(bits[w] & ((1u << (k & 31)) - 1u));
    t_idx[b + rank] = (int32_t)k;
    t_val[b + rank] = u_val[b + i];
  }
}

}  // namespace

// ---- launchers ---------------------------------------------------------------------------------
int fp4_compute_units_of_current_device();
int fp4_trace_open(int kind, hipStream_t stream);
void fp4_trace_close(int slot, hipStream_t stream);
int64_t fp4_spmm_mfma_scratch_bytes(int64_t P, int64_t Q);
int fp4_launch_spmm_mfma(const int64_t* row_ptr, const int32_t* col_idx, const float* val, int64_t capacity, int64_t P,
                         int64_t Q, const void* D, int64_t N, float* R, void* scratch, int32_t* list, int32_t* count,
                         SpmmRest& rest, hipStream_t s);
int fp4_launch_spmm_gather(const int64_t* row_ptr, const int32_t* col_idx, const float* val, int64_t capacity, int64_t P, int64_t Q,
                           const void* D, int bf16, int64_t N, float* R, hipStream_t s);
// int32 words of scratch fp4_launch_spmm needs: count[64 (only [0] used)], list[P], then
// the fp32 partial sums of the dense long-row path, [spans][long rows][N], at most LD_CAP x slices rows of N, then (bf16 D)
// the packed matrix.
static int64_t spmm_list_words(int64_t P) { return 64 + (P + 63) / 64 * 64; }
// The partial sums' share, for this product and any smaller one: slices of fewer than 512 rows are only taken while twice as
// many rows leave fewer than 256 workgroups of 512 columns, so there are at most 510 of them.
static int64_t spmm_long_words(int64_t P, int64_t Q, int64_t N) {
  const int64_t most = std::max((Q + LD_SLICE - 1) / LD_SLICE * N, std::min<int64_t>((Q + 63) / 64 * N, 510 * LD_COLS));
  return spmm_list_words(P) + (most * LD_CAP + 63) / 64 * 64;
}
int64_t fp4_spmm_scratch_words(int64_t P, int64_t Q, int64_t N, int bf16) {
  return spmm_long_words(P, Q, N) + (bf16 ? (fp4_spmm_mfma_scratch_bytes(P, Q) + 3) / 4 : 0);
}

// general: by the kernels that large products take, whatever the size
int fp4_launch_spmm(const int64_t* row_ptr, const int32_t* col_idx, const float* val, int64_t capacity,
                    int64_t P, int64_t Q, const void* D, int bf16, int64_t N, float* R, int32_t* scratch,
                    hipStream_t s, bool general) {
  if (P == 0 || N == 0) return FP4_OK;
  if (Q >= ((int64_t)1 << 21)) return FP4_ERR_SHAPE;   // 32-bit entry offsets inside a workgroup's 1024 rows
  const bool may_be_long = Q > SPMM_LONG_MIN && capacity > SPMM_LONG_MIN;   // otherwise no row is
  int32_t* const count = scratch;
  int32_t* const list = scratch + 64;
  const dim3 grid((unsigned)((P + SP_ROWS - 1) / SP_ROWS), (unsigned)((N + SP_COLS - 1) / SP_COLS));
  const int trace_slot = fp4_trace_open(FP4_TRACE_SPMM, s);   // the whole product, as its entries are counted
  int rc = general ? 1 : fp4_launch_spmm_gather(row_ptr, col_idx, val, capacity, P, Q, D, bf16, N, R, s);
  if (rc != 1) {
    fp4_trace_close(trace_slot, s);
    return rc;
  }
  SpmmRest rest{nullptr, nullptr, 0};
  if (bf16)
    rc = fp4_launch_spmm_mfma(row_ptr, col_idx, val, capacity, P, Q, D, N, R, scratch + spmm_long_words(P, Q, N), list, count, rest, s);
  if (rc != 0 && rc != 1) {
    fp4_trace_close(trace_slot, s);
    return rc;
  }
  const bool packed = rc == 0;
  if (!packed) {
    if (bf16)
      hipLaunchKernelGGL((spmm_tile_kernel<BF16>), grid, dim3(SP_ROWS), 0, s, row_ptr, col_idx, val, capacity, P, Q, D, N, R);
    else {
      // Half as many rows a workgroup while those go round the chip once: the slab is staged as often as there are workgroups,
      // but a CU's gathers go twice as fast (1024 / 512 / 256 rows, with the long rows' launches, at 2 %: 2048^3 72 / 56 / 58 us,
      // 2500 x 2048 -> 3000 76 / 66 / 99, 1024^3 43 / 32 / 32; beyond one round 3072^3 104 / 142 / 184).
      const int64_t half = (P + SP_ROWS / 2 - 1) / (SP_ROWS / 2);
      if (half * grid.y <= fp4_compute_units_of_current_device())
        hipLaunchKernelGGL((spmm_tile_kernel<F32, SP_ROWS / 2>), dim3((unsigned)half, grid.y), dim3(SP_ROWS / 2), 0, s, row_ptr, col_idx, val,
                           capacity, P, Q, D, N, R);
      else
        hipLaunchKernelGGL((spmm_tile_kernel<F32>), grid, dim3(SP_ROWS), 0, s, row_ptr, col_idx, val, capacity, P, Q, D, N, R);
    }
    if (may_be_long)
      hipLaunchKernelGGL(find_long_rows_kernel, dim3(1), dim3(1024), 0, s, row_ptr, P, Q, capacity, list, count);
  }
  float* const part = reinterpret_cast<float*>(scratch + spmm_list_words(P));
  const int slice = ld_slice(Q, N);
  const int slices = (int)((Q + slice - 1) / slice);
  if (may_be_long) {
    // an item a workgroup for up to eight long rows, and two workgroups a CU for more; what finds no item leaves at once
    const unsigned blocks = (unsigned)((N + LD_COLS - 1) / LD_COLS);
    const dim3 dgrid(blocks, std::max((unsigned)slices, std::min((unsigned)slices * (LD_CAP / LD_LB), 512 / blocks)));
    if (bf16)
      hipLaunchKernelGGL((spmm_long_dense_kernel<BF16>), dgrid, dim3(LD_WAVES * 64), 0, s, row_ptr, col_idx, val, capacity, list,
                         count, D, (int)Q, N, slice, slices, part, R);
    else
      hipLaunchKernelGGL((spmm_long_dense_kernel<F32>), dgrid, dim3(LD_WAVES * 64), 0, s, row_ptr, col_idx, val, capacity, list,
                         count, D, (int)Q, N, slice, slices, part, R);
  }
  if (packed) {
    const dim3 tiles(grid.x, std::min(grid.y, std::max(1u, 512u / grid.x)));
    // up to eight long rows side by side, fewer where their column blocks are many: one workgroup fits a CU
    const unsigned blocks = (unsigned)((N + 255) / 256);
    const unsigned long_blocks = may_be_long ? blocks * std::max(1u, std::min(8u, 128u / blocks)) : 0;
    hipLaunchKernelGGL(spmm_rest_kernel, dim3(tiles.x * tiles.y + long_blocks), dim3(SP_ROWS), 0, s, row_ptr, col_idx, val,
                       capacity, P, Q, D, N, R, rest, tiles, long_blocks, list, count, part, slices);
  } else if (may_be_long) {
    const dim3 fgrid((unsigned)((N + 255) / 256), LF_ROWS);
    if (bf16)
      hipLaunchKernelGGL((spmm_finish_long_kernel<BF16>), fgrid, dim3(256), 0, s, row_ptr, col_idx, val, capacity, list, count, part,
                         slices, D, N, R);
    else
      hipLaunchKernelGGL((spmm_finish_long_kernel<F32>), fgrid, dim3(256), 0, s, row_ptr, col_idx, val, capacity, list, count, part,
                         slices, D, N, R);
  }
  fp4_trace_close(trace_slot, s);
  FP4_CHECK_LAUNCH();
  return FP4_OK;
}

int fp4_launch_scan_rows(const int32_t* row_cnt, int64_t rows, int64_t* row_ptr, int64_t* nnz, hipStream_t s);

// int32 words of scratch the transpose of a P x Q matrix needs.  Mask path (Q <= MB_MAXQ): cnt[Q], ex[blocks][Q] (uint32), cnt8[blocks][Q]
// (bytes).  Otherwise: cnt[Q], cursor[Q].  A matrix too wide for the masks counts as the widest that is not, or a wider one would need less.
int64_t fp4_csr_transpose_scratch_words(int64_t P, int64_t Q) {
  const int64_t columns = 2 * Q;
  Q = std::min<int64_t>(Q, MB_MAXQ);
  const int64_t blocks = (P + mb_rows(Q) - 1) / mb_rows(Q);
  return std::max(columns, Q + 64 + blocks * Q + (blocks * Q + 3) / 4 + 64);
}

int fp4_csr_transpose_from(int64_t P, int64_t Q) { return (int)mb_from(P, Q); }

// The passes that other launches have not taken along (m.counted, and the last unless fill_too; m.nblocks > 0).
int fp4_launch_csr_mask(const MbArgs& m, bool fill_too, hipStream_t s) {
  using Q4 = std::integral_constant<int, 4096>;
  using Q8 = std::integral_constant<int, 8192>;
  using Q16 = std::integral_constant<int, MB_MAXQ>;
  auto width = [&](auto go) {
    if (m.Q <= 4096) go(Q4{}); else if (m.Q <= 8192) go(Q8{}); else go(Q16{});
  };
  if (!m.counted)
    width([&](auto q) { hipLaunchKernelGGL((csr_mask_count_kernel<decltype(q)::value>), dim3(m.nblocks), dim3(MB_THREADS), 0, s, m); });
  if (m.from != MbFrom::FEW)
    hipLaunchKernelGGL(csr_mask_scan_kernel, dim3((unsigned)((m.Q + 63) / 64)), dim3(256), 0, s, m);
  FP4_CHECK_LAUNCH();
  if (!fill_too) return FP4_OK;
  if (m.from == MbFrom::TABLE) {
    const int rc = fp4_launch_scan_rows(m.cnt, m.Q, m.t_ptr, nullptr, s);
    if (rc) return rc;
  }
  auto fill = [&](auto from) {
    width([&](auto q) {
      hipLaunchKernelGGL((csr_mask_fill_kernel<decltype(q)::value, decltype(from)::value>), dim3(mb_fill_blocks(m.nblocks)), dim3(MB_THREADS), 0, s,
                         m);
    });
  };
  if (m.from == MbFrom::FEW) fill(std::integral_constant<MbFrom, MbFrom::FEW>{});
  else if (m.from == MbFrom::SCAN) fill(std::integral_constant<MbFrom, MbFrom::SCAN>{});
  else fill(std::integral_constant<MbFrom, MbFrom::TABLE>{});
  FP4_CHECK_LAUNCH();
  return FP4_OK;
}

// u_idx/u_val: unordered staging, capacity entries each (only the path for very wide matrices uses it)
// from: a MbFrom, or 0 for that of the sizes
int fp4_launch_csr_transpose(const int64_t* row_ptr, const int32_t* col_idx, const float* val,
                             const int64_t* nnz, int64_t P, int64_t Q, int64_t capacity, int64_t* t_ptr,
                             int32_t* t_idx, float* t_val, int32_t* u_idx, float* u_val, int32_t* scratch,
                             hipStream_t s, int from) {
  int32_t* cnt = scratch;
  if (Q <= MB_MAXQ) {
    if (from && from != (int)MbFrom::TABLE && !mb_positions(P, Q)) return FP4_ERR_ARG;
    MbArgs m = mb_args(row_ptr, col_idx, val, P, Q, capacity, t_ptr, t_idx, t_val, scratch);
    if (from) m.from = (MbFrom)from;
    return fp4_launch_csr_mask(m, true, s);
  }
  int32_t* cursor = scratch + Q;
  hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)((2 * Q + 255) / 256)), dim3(256), 0, s, scratch, 2 * Q, 0);
  const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((capacity + 4095) / 4096, 2048));
  hipLaunchKernelGGL(csr_count_cols_kernel, dim3(grid), dim3(256), 0, s, col_idx, nnz, capacity, Q, cnt);
  hipLaunchKernelGGL(scan_counts32_kernel, dim3(1), dim3(1024), 0, s, cnt, Q, t_ptr);
  hipLaunchKernelGGL(csr_transpose_fill_kernel, dim3((unsigned)((P + 3) / 4)), dim3(256), 0, s, row_ptr, col_idx, val,
                     P, capacity, t_ptr, cursor, u_idx, u_val);
  if (capacity > 0 && P <= (int64_t)BM_WORDS * 32)
    hipLaunchKernelGGL(csr_bitmap_sort_kernel, dim3((unsigned)Q), dim3(256), (size_t)((P + 31) / 32) * 8, s, t_ptr, P,
                       capacity, u_idx, u_val, t_idx, t_val);
  else if (capacity > 0)
    hipLaunchKernelGGL(csr_rank_sort_kernel, dim3((unsigned)((capacity + 255) / 256)), dim3(256), 0, s, t_ptr, Q, u_idx,
                       u_val, t_idx, t_val);
  FP4_CHECK_LAUNCH();
  return FP4_OK;
}

// Rows of a CSR matrix whose entries sit, unordered, in (u_idx, u_val): write them ordered by
// index to (idx, val).  nidx = number of columns.  Returns 1 if the index range is too large
// for the LDS bitmap (the caller then uses its own fallback).
int fp4_launch_order_rows(const int64_t* row_ptr, int64_t rows, int64_t nidx, int64_t capacity,
                          const int32_t* u_idx, const float* u_val, int32_t* idx, float* val, hipStream_t s) {
  if (nidx > (int64_t)BM_WORDS * 32) return 1;
  if (rows == 0) return FP4_OK;
  hipLaunchKernelGGL(csr_bitmap_sort_kernel, dim3((unsigned)rows), dim3(256), (size_t)((nidx + 31) / 32) * 8, s, row_ptr,
                     nidx, capacity, u_idx, u_val, idx, val);
  FP4_CHECK_LAUNCH();
  return FP4_OK;
}
