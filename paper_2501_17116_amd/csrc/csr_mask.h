// Transpose of a CSR matrix as a stable counting sort on the column, for column ranges that fit the LDS masks: passes 1 and 3, which run
// by themselves (spmm.hip, as pass 2 does) or beside the quantization passes of the backward pass (quantize.hip).
//
// The rows are cut into blocks of 64 (32, mb_rows).  Inside a block, column c's entries are described by a 64-bit
// mask of the rows that hold one (built with LDS atomic ORs: the result does not depend on their
// order).  Pass 1 writes the population count of every mask, cnt8[block][c].  Pass 2 scans those
// counts over the blocks of each column (exclusive, ex[block][c]) and leaves the column totals.
// After the scan of the totals into t_ptr, pass 3 rebuilds the masks and places entry (r, c) at
//   t_ptr[c] + ex[block][c] + popcount(mask[c] below bit r - r0),
// i.e. behind every entry of the column from an earlier row: the transposed matrix comes out with
// ascending indices inside every segment, without global atomics and without an ordering pass.
#pragma once
#include "fp4_common.h"

#include <algorithm>

// Rows per block = bits per mask: 64, above 8192 columns 32, whose masks leave the LDS room for the columns' positions.
constexpr int mb_rows(int64_t Q) { return Q > 8192 ? 32 : 64; }
constexpr int MB_THREADS = 1024;   // per workgroup in the two passes that walk entries: they are latency-bound
constexpr int MB_MAXQ = 16384;       // columns whose masks and positions (4 bytes each) fit 128 KiB of LDS

// Where pass 3 takes the positions from.  FEW: from the counts of all row blocks, at most MB_FEW_BYTES of them in MB_FEW_BLOCKS, which
// every workgroup adds up for itself, sixteen blocks at a time: as many rows of counts take as many round trips however few the
// columns are (fill alone, FEW / as SCAN with its launch before it, us: 16384 x 128 15 / 10, 65536 x 64 123 / 22, 131072 x 32 477 / 38; whole
// weight gradients with 64 blocks 53.6 / 53.9, with 128 51.5 / 50.5).  SCAN: from pass 2's ex and totals, which every workgroup scans over the columns.  Either way
// a column's position waits in LDS beside its mask, and the workgroup of the first row block writes t_ptr.  TABLE: with 2^32
// elements or more positions have no room in 32 bits; t_ptr comes from a scan of its own.  Bound by round trips to memory, so by the
// launches and by what a workgroup asks for one after another.
// Whole transposition at 2 % (count, scan over blocks, scan over columns and fill as four launches / now): 256 x 512 12.3 / 8.2 us,
// 1056 x 1376 at 6 % 28.7 / 19.3, 2048 x 2048 22.2 / 14.9, 8192 x 2048 25.0 / 19.3, 16384 x 4096 46.3 / 38.1,
// 16384 x 11008 the fill alone (blocks of 64 rows, from a table / of 32) 156 / 98.
enum class MbFrom { FEW = 1, SCAN, TABLE };
constexpr int64_t MB_FEW_BYTES = 64 * 1024, MB_FEW_BLOCKS = 64;

struct MbArgs {
  const int64_t* row_ptr;
  const int32_t* col_idx;
  const float* val;
  int64_t rows, Q, capacity;
  int64_t* t_ptr;
  int32_t* t_idx;
  float* t_val;
  uint32_t* ex;    // [blocks][Q]
  int32_t* cnt;    // [Q]
  uint8_t* cnt8;   // [blocks][Q]
  int nblocks;
  MbFrom from;
  bool counted;   // pass 1 has been launched elsewhere
};

inline int64_t mb_blocks(int64_t P, int64_t Q) { return std::max<int64_t>(1, (P + mb_rows(Q) - 1) / mb_rows(Q)); }
inline bool mb_positions(int64_t P, int64_t Q) { return Q % 4 == 0 && P * Q < ((int64_t)1 << 32); }
inline MbFrom mb_from(int64_t P, int64_t Q) {   // 0: no masks
  if (Q > MB_MAXQ) return (MbFrom)0;
  if (!mb_positions(P, Q)) return MbFrom::TABLE;
  const int64_t blocks = mb_blocks(P, Q);
  return blocks <= MB_FEW_BLOCKS && blocks * Q <= MB_FEW_BYTES ? MbFrom::FEW : MbFrom::SCAN;
}
// Each XCD takes a contiguous run of row blocks in pass 3: whole eighths.
inline unsigned mb_fill_blocks(int nblocks) { return (unsigned)((nblocks + 7) / 8 * 8); }
// scratch: fp4_csr_transpose_scratch_words(P, Q)
inline MbArgs mb_args(const int64_t* row_ptr, const int32_t* col_idx, const float* val, int64_t P, int64_t Q, int64_t capacity, int64_t* t_ptr,
                      int32_t* t_idx, float* t_val, int32_t* scratch) {
  MbArgs m = {};
  m.row_ptr = row_ptr; m.col_idx = col_idx; m.val = val;
  m.rows = P; m.Q = Q; m.capacity = capacity;
  m.t_ptr = t_ptr; m.t_idx = t_idx; m.t_val = t_val;
  m.from = mb_from(P, Q);
  m.nblocks = Q <= MB_MAXQ ? (int)mb_blocks(P, Q) : 0;
  m.cnt = scratch;
  m.ex = reinterpret_cast<uint32_t*>(scratch + Q + 64);
  m.cnt8 = reinterpret_cast<uint8_t*>(m.ex + (int64_t)m.nblocks * Q);
  return m;
}

int fp4_launch_csr_mask(const MbArgs& m, bool fill_too, hipStream_t s);

#if defined(__HIPCC__)
// first (entry offset, row) bookkeeping shared by pass 1 and pass 3: s_rp[0..MB_ROWS] = clipped row starts
template <int MB_ROWS>
FP4_D void mb_load_rows(const MbArgs& m, int64_t r0, long long* s_rp) {
  if (threadIdx.x <= MB_ROWS) {
    const int64_t r = min(r0 + (int64_t)threadIdx.x, m.rows);
    s_rp[threadIdx.x] = min(m.row_ptr[r], m.capacity);
  }
}
// row of entry e of the block: the last i with s_rp[i] <= e
template <int MB_ROWS>
FP4_D int mb_row_of(const long long* s_rp, long long e) {
  int lo = 0, hi = MB_ROWS;   // invariant: s_rp[lo] <= e < s_rp[hi]
#pragma unroll
  for (int it = 0; (1 << it) < MB_ROWS; ++it) {
    const int mid = (lo + hi) >> 1;
    if (s_rp[mid] <= e) lo = mid; else hi = mid;
  }
  return lo;
}

// sets, for every entry e of the block's range [b, e_end), bit (row of e) of its column's mask; AT_ONCE
// column loads a thread in flight
template <int MB_ROWS, int THREADS, int AT_ONCE>
FP4_D void mb_build_masks(const int32_t* col_idx, const long long* s_rp, long long b, long long e_end, uint32_t* mb_mask) {
  for (long long i0 = b + threadIdx.x; i0 < e_end; i0 += AT_ONCE * THREADS) {
    int32_t c[AT_ONCE];
#pragma unroll
    for (int u = 0; u < AT_ONCE; ++u) {
      const long long i = i0 + (long long)u * THREADS;
      c[u] = i < e_end ? col_idx[i] : -1;
    }
#pragma unroll
    for (int u = 0; u < AT_ONCE; ++u) {
      if (c[u] < 0) continue;
      const int r = mb_row_of<MB_ROWS>(s_rp, i0 + (long long)u * THREADS);
      atomicOr(&mb_mask[MB_ROWS / 32 * c[u] + (r >> 5)], 1u << (r & 31));
    }
  }
}

template <int QMAX>
struct MbCountShared {
  uint32_t mask[mb_rows(QMAX) / 32 * QMAX];   // rows 0..31 of the block in the first of a column's words
  long long rp[mb_rows(QMAX) + 1];
};

template <int QMAX, int THREADS>
FP4_D void mb_count(const MbArgs& m, unsigned block, MbCountShared<QMAX>& sh) {
  constexpr int MB_ROWS = mb_rows(QMAX), MW = MB_ROWS / 32;
  const int64_t r0 = (int64_t)block * MB_ROWS;
  for (int i = threadIdx.x; i < MW * m.Q; i += THREADS) sh.mask[i] = 0;
  mb_load_rows<MB_ROWS>(m, r0, sh.rp);
  __syncthreads();
  const long long b = sh.rp[0], e = sh.rp[MB_ROWS];
  mb_build_masks<MB_ROWS, THREADS, 4 * MB_THREADS / THREADS>(m.col_idx, sh.rp, b, e, sh.mask);
  __syncthreads();
  uint8_t* out = m.cnt8 + (int64_t)block * m.Q;
  for (int c = threadIdx.x; c < m.Q; c += THREADS)
    out[c] = (uint8_t)(__popc(sh.mask[MW * c]) + (MW > 1 ? __popc(sh.mask[MW * c + MW - 1]) : 0));
}

template <int QMAX, MbFrom FROM>
struct MbFillShared {
  uint32_t mask[mb_rows(QMAX) / 32 * QMAX];
  long long rp[mb_rows(QMAX) + 1];
  uint32_t pos[FROM == MbFrom::TABLE ? 1 : QMAX];   // fewer than 2^32 entries (the launcher's rule)
  uint32_t w[MB_THREADS / 64];
};

// By a workgroup of MB_THREADS; id: one of mb_fill_blocks, a multiple of 8 away from blockIdx.x.
template <int QMAX, MbFrom FROM>
FP4_D void mb_fill(const MbArgs& m, unsigned id, MbFillShared<QMAX, FROM>& sh) {
  constexpr bool TABLE = FROM == MbFrom::TABLE;
  constexpr int MB_ROWS = mb_rows(QMAX), MW = MB_ROWS / 32;
  constexpr int PER = QMAX / MB_THREADS;   // consecutive columns a thread forms positions of: a multiple of 4
  const int64_t Q = m.Q;
  // Each XCD takes a contiguous run of row blocks.  A block has one or two entries of a column, and its neighbours' lie beside
  // them: written from eight L2s they were partial lines of every one, from one L2 they are whole (16384 x 4096 at 2 %: 48.9
  // -> 29.3 us).
  const int nblocks = m.nblocks, per_xcd = (nblocks + 7) / 8;
  const int block = (int)(id % 8) * per_xcd + (int)(id / 8);
  if ((int)(id / 8) >= per_xcd || block >= nblocks) return;
  const int64_t r0 = (int64_t)block * MB_ROWS;
  const int c0 = (int)threadIdx.x * PER;
  uint32_t before[PER] = {}, total[PER] = {}, sum = 0, incl = 0;   // a column's entries in earlier blocks, and all of them
  mb_load_rows<MB_ROWS>(m, r0, sh.rp);
  for (int i = threadIdx.x; i < MW * Q; i += MB_THREADS) sh.mask[i] = 0;
  if constexpr (!TABLE) {
#pragma unroll
    for (int j = 0; j < PER; j += 4) {   // Q is a multiple of 4
      if (c0 + j >= Q) break;
      if constexpr (FROM == MbFrom::FEW) {
#pragma unroll 16
        for (int b = 0; b < nblocks; ++b) {
          const uint32_t four = *reinterpret_cast<const uint32_t*>(m.cnt8 + (int64_t)b * Q + c0 + j);
          const uint32_t early = b < block ? four : 0;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            before[j + q] += (early >> (8 * q)) & 0xffu;
            total[j + q] += (four >> (8 * q)) & 0xffu;
          }
        }
      } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          before[j + q] = m.ex[(int64_t)block * Q + c0 + j + q];
          total[j + q] = (uint32_t)m.cnt[c0 + j + q];
        }
      }
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) sum += total[j];
    incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t up = __shfl_up(incl, o, 64);
      if ((int)(threadIdx.x & 63) >= o) incl += up;
    }
    if ((threadIdx.x & 63) == 63) sh.w[threadIdx.x >> 6] = incl;
  }
  __syncthreads();
  if constexpr (!TABLE) {
    uint32_t at = incl - sum;
    for (int w = 0; w < (int)(threadIdx.x >> 6); ++w) at += sh.w[w];
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      if (c0 + j >= Q) break;
      sh.pos[c0 + j] = at + before[j];
      at += total[j];
      if (block == 0) m.t_ptr[c0 + j + 1] = at;
    }
    if (block == 0 && threadIdx.x == 0) m.t_ptr[0] = 0;
  }
  const long long b = sh.rp[0], e = sh.rp[MB_ROWS];
  mb_build_masks<MB_ROWS, MB_THREADS, 4>(m.col_idx, sh.rp, b, e, sh.mask);
  __syncthreads();
  // Placement, four entries a thread at a time: the steps of the chain column -> position -> store that go to memory are round
  // trips, so the four chains run side by side.
  const uint32_t* exb = m.ex + (int64_t)block * Q;
  for (long long i0 = b + threadIdx.x; i0 < e; i0 += 4 * MB_THREADS) {
    int32_t c[4];
    float v[4];
    int64_t pos[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const long long i = i0 + (long long)u * MB_THREADS;
      c[u] = i < e ? m.col_idx[i] : -1;
      v[u] = i < e ? m.val[i] : 0.0f;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if constexpr (TABLE) pos[u] = c[u] >= 0 ? m.t_ptr[c[u]] + exb[c[u]] : m.capacity;
      else pos[u] = c[u] >= 0 ? (int64_t)sh.pos[c[u]] : m.capacity;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (c[u] < 0) continue;
      const int r = mb_row_of<MB_ROWS>(sh.rp, i0 + (long long)u * MB_THREADS);
      const uint32_t lo = sh.mask[MW * c[u]], hi = sh.mask[MW * c[u] + MW - 1];
      const uint32_t below = r < 32 ? __popc(lo & ((1u << r) - 1u)) : __popc(lo) + __popc(hi & ((1u << (r - 32)) - 1u));
      const int64_t p = pos[u] + below;
      if (p < m.capacity) {
        m.t_idx[p] = (int32_t)(r0 + r);
        m.t_val[p] = v[u];
      }
    }
  }
}
#endif
