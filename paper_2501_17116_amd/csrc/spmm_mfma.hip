// The residual product R[P x N] = S D (Sec. 3.2) for bf16 D on the matrix cores.
//
// S has about 2 % scattered entries.  Sixteen rows of it together touch about 28 % of the columns, so a
// group of 16 rows is packed into "slots": one slot per column that any of the 16 rows has an entry in,
// holding that column's 16 values (zero where a row has none) in bf16.  32 slots make one step: A = the 16 x 32 packed values, B = the
// 32 rows of D that the slots name, gathered from LDS.  An fp32 value that is no bf16 number is the exact sum of two or three (down to
// 2^-110; rows with smaller values of more bits are left to the tiled kernel), and its column takes as many slots: products are
// exact, sums are fp32, nothing is rounded to 16 bits.
//
// A lane owns 8 adjacent columns of D, so a gathered row arrives as one 16-byte LDS read per lane, 256 contiguous bytes per
// quarter wave: free of bank conflicts whatever rows the slots name.  A register then holds two columns of one row, where the dense
// matrix instruction wants two rows of one column: v_perm_b32 turned eight rows x eight columns around, 32 a step.  The 2:4 sparse
// instruction (v_smfmac_f32_16x16x64_bf16) takes them as they came: of every four adjacent k values, here two columns of two rows, it
// multiplies two, the first column's or the second's as its index says, so that the same registers serve for both columns, and the
// eight registers of eight rows have only to be put side by side (30 v_mov_b32 a step; 12 v_swap_b32, or v_pk_mov_b32, take as long).
// A step of a SIMD alone, three waves of three groups: 155 -> 122 ns.  The product with its packing, at 2 %, us: 16384 x 4096 -> 12288
// 826 -> 813, 4096 x 16384 -> 12288 787 -> 764, 16384 x 11008 -> 4096 669 -> 652, 8192 x 4096 -> 11008 377 -> 360, 4096 x 8192 ->
// 11008 397 -> 377 (1 to 2 % of it from not waiting for operands at each phase, at `plan`).
//
// D passes through LDS as a ring of chunks (SM_KC rows x SM_NT columns, direct-to-LDS loads two chunks
// ahead, three with one group a wave).  A slot may be multiplied in any phase in which its chunk is resident, and the packing decides
// how many steps a group runs in each phase (a prefix of its slots, S[phase]): the steps stay full and the
// waves of a workgroup in step with each other although the entries of a chunk are few and random.
//
// Bound: a SIMD's vector instructions (38 a step beside the matrix core's 8, which have 16 cycles each) and the return of its LDS reads, which
// do not overlap: reads alone 62 ns a step, with the matrix core 84, with the moves 122.  Another 6 to 11 vector instructions a step
// are the sums' way to memory, the staging wave's and the phases'.  16384 x 4096 -> 12288 with its packing: 805 us at 2 % (650 without the stores of
// the sums, which mostly make the loads wait), 1364 at 6 % (1260), 514 at 0.2 % (384).  With plain fp32 FMAs fed from LDS (spmm.hip) 1423, 2961 and 609.
#include "fp4_common.h"
#include "spmm_long.h"

#include <algorithm>
#include <tuple>

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x8 __attribute__((ext_vector_type(8)));

constexpr int SM_STEPS_PAD = 12;   // step counts read past the last bundle (up to 12 waves)
constexpr int SM_KC = 128;       // rows of D per chunk
constexpr int SM_RING = 5;       // chunks in LDS (all 160 KiB): to multiply from, and on their way
// Chunks on their way.  With one group a wave a phase has so little to multiply that it lasts as long as a chunk takes to come, so three
// are, by two staging waves (a wave has 63 loads under way at most, a chunk is 32).
constexpr int sm_ahead(int g) { return g == 1 ? 3 : 2; }
constexpr int sm_stagers(int g) { return g == 1 ? 2 : 1; }
constexpr int sm_slack(int g) { return SM_RING - sm_ahead(g) - 1; }   // phases a chunk stays after the one it arrives in
constexpr int SM_PACE = 4;       // steps whose multiples bundles are paced by
constexpr int SM_DEEP = 3;       // steps of a single group requested ahead
constexpr int SM_NT = 128;       // columns of R per workgroup
constexpr int SM_ROWB = SM_NT * 2;
constexpr int SM_CHUNKB = SM_KC * SM_ROWB;
// Which two of four adjacent k values the 2:4 sparse instruction multiplies, two bits a value: the first and the third (low half), or the
// second and the fourth.
constexpr int SM_FIRST_OF_TWO = (int)0xdddd8888;
constexpr int SM_STRIP = 8;      // column blocks that an XCD works on side by side
// Packing threads per row: what fills a workgroup.  A row's entries are two chains of loads, so more threads shorten
// them (2048 rows of 164 entries, 16 / 32 / 64 threads a row: 20.1 / 17.8 / 16.7 us).
constexpr int pk_tpr(int g) { return g == 1 ? 64 : 16; }
constexpr int64_t SM_MAXQ = 24576;   // the packing keeps a nibble per column and group in LDS, within 64 KiB
constexpr int SM_PLANS = (int)((SM_MAXQ + 64 * SM_KC - 1) / (64 * SM_KC));   // registers that hold a step count for every phase
static_assert(SM_ROWB == 256, "a quarter wave covers a row of a chunk with 16 bytes a lane");

// Slots a column up to which a matrix is packed, at a share d of entries.  The packed product takes a time that goes with
// the slots, the tiled one's goes with the entries; they meet at 0.21 slots and 0.21 more per per cent of entries
// (8192 x 4096 -> 11008: 1 % and 0.45 slots 548 against 523 us, 2 % and 0.55 640 / 712, 2 % and 0.83 879 / 712, 4 % and 0.96
// 989 / 1097), at 0.10 in a smaller one (4096^3), where launches count.  A grid that does not fill the chip with the
// tiled kernel's workgroups is packed as far as there is room, with a margin (512 x 4096 -> 4096, 2 %, 0.83: 86 / 90).
constexpr float SM_ROOM_SLOTS = 1.15f, SM_EVEN_SLOTS = 0.14f, SM_EVEN_SHARE = 21.0f;
// steps a group of 16 rows has room for: every column once, and a quarter more for values of several terms
inline int64_t sm_cap(int64_t Q) { return (Q + 31) / 32 + (Q + 127) / 128 + 3; }
inline int64_t sm_phases(int64_t Q) { return (Q + SM_KC - 1) / SM_KC; }

// Byte of a step's packed values at which row r's value of slot p stands.  A lane gathers the eight rows of D of slots 8 q .. 8 q + 7, q its
// quarter of the wave; the instruction pairs the first four with values 4 (q & 1) .. of quarter q / 2, the others with those of quarter 2 + q / 2.
FP4_D int sm_a_at(int p, int r) {
  const int quarter = (p >> 1 & 2) | p >> 4, i = (p >> 1 & 4) | (p & 3);
  return (quarter * 16 + r) * 16 + i * 2;
}

FP4_D uint32_t bf16_nearest(float v) { return __builtin_bit_cast(uint16_t, (__bf16)v); }   // v_cvt_pk_bf16_f32

// v as the exact sum of up to three bf16 numbers (nearest first); returns how many, 4 if three are not enough: below
// 2^-110 the last of fp32's 24 bits can lie under the smallest bf16 number, 2^-133.
FP4_D int bf16_terms(float v, uint32_t (&t)[3]) {
  const uint32_t u = f2u(v);
  t[0] = bf16_nearest(v);
  if ((t[0] & 0x7f80u) == 0x7f80u) t[0] = (u >> 16) | ((u & 0x7fffffffu) > 0x7f800000u ? 1u : 0u);   // no rounding up to infinity
  const float r = (u & 0x7f800000u) == 0x7f800000u ? 0.0f : v - u2f(t[0] << 16);
  t[1] = bf16_nearest(r);
  const float r2 = r - u2f(t[1] << 16);
  t[2] = bf16_nearest(r2);
  return r2 != u2f(t[2] << 16) ? 4 : r2 != 0.0f ? 3 : r != 0.0f ? 2 : 1;
}

// Whether a matrix is worth packing, from 64 rows spread over it (every workgroup looks at the same ones and comes to the
// same answer, which depends on the matrix alone): the slots a column of a group needs on average, from the rows' entries
// and the number of terms of one value of each.  rows[0..3]: rows that are not long, their entries, those of values
// of two terms or more, of three.
FP4_D bool pk_worth(const int (&rows)[4], int Q, bool small_grid) {
  const float a_cell = __builtin_amdgcn_rcpf(fmaxf((float)rows[0], 1.0f) * (float)Q);
  float slots = 0.0f;
#pragma unroll
  for (int t = 1; t < 4; ++t) {
    float none = fmaxf(1.0f - (float)rows[t] * a_cell, 0.0f);   // no row of 16 has one
#pragma unroll
    for (int k = 0; k < 4; ++k) none *= none;
    slots += 1.0f - none;
  }
  return slots <= SM_ROOM_SLOTS && (small_grid || slots <= SM_EVEN_SLOTS + SM_EVEN_SHARE * (float)rows[1] * a_cell);
}

// One workgroup per bundle of G groups (the groups of one wave, which step together), or G of them (split), which all count and
// plan for the whole bundle and write one group each, up to two of these workgroups a CU: bundles of three groups that are fewer
// than two thirds of the CUs left the rest idle while each wrote some hundred KiB (4096 rows of 328 entries 53.5 -> 46.0 us, 2048 of 164 27.1 -> 22.4).  sched[bundle][phase]:
// steps done when the phase ends; steps[bundle]: steps in all, or -1 when the bundle is left to the tiled kernel (a
// matrix that is not worth it, more slots than there is room for, columns that repeat inside a row, or values that three
// bf16 terms do not make up); redo[bundle]: 0.
template <int G>
__global__ __launch_bounds__(16 * G * pk_tpr(G)) void spmm_pack_kernel(const int64_t* __restrict__ row_ptr,
                                                               const int32_t* __restrict__ col_idx,
                                                               const float* __restrict__ val, int64_t capacity, int64_t P,
                                                               int Q, int cap, int phases, bool small_grid, bool split, uint8_t* __restrict__ a_buf,
                                                               uint8_t* __restrict__ o_buf, int32_t* __restrict__ sched,
                                                               int32_t* __restrict__ steps, int32_t* __restrict__ redo, int32_t* list,
                                                               int32_t* count) {
  constexpr int ROWS = 16 * G, PK_TPR = pk_tpr(G), THREADS = ROWS * PK_TPR, SM_SLACK = sm_slack(G);
  extern __shared__ __attribute__((aligned(16))) uint32_t pk_lds[];
  const int words = phases * (SM_KC / 8);
  uint32_t* const nib = pk_lds;                                                // [G][words] a nibble per column: as many bits as slots
  uint16_t* const pre = reinterpret_cast<uint16_t*>(nib + G * words);      // [G][words] slots of the chunk before this word
  int32_t* const start = reinterpret_cast<int32_t*>(pre + G * words);       // [G][phases] slot count, then first slot
  __shared__ int64_t s_b[ROWS];
  __shared__ int s_n[ROWS];
  __shared__ int s_bad, s_total[G], s_steps, s_sample[4];
  const int tid = threadIdx.x;
  if (blockIdx.x == 0) {   // the first workgroup lists the long rows
    find_long_rows<THREADS>(row_ptr, P, Q, capacity, list, count);
    return;
  }
  const int64_t bundles = split ? (gridDim.x - 1) / G : gridDim.x - 1;
  const int64_t bundle = split ? (blockIdx.x - 1) / G : blockIdx.x - 1;
  const int part = (int)(blockIdx.x - 1 - bundle * G);   // split: the group to write
  auto entries = [&](int64_t row, int64_t& b) -> int64_t {
    b = row_ptr[row];
    return max(min(row_ptr[row + 1], capacity), b) - b;
  };
  // A row a thread, and in the last wave the sample's rows, all requests before the limit's.
  const bool sampler = tid >= THREADS - 64;
  static_assert(THREADS >= ROWS + 64, "a wave for the sample");
  int64_t b = 0, n = 0;
  if (tid < ROWS || sampler) {
    const int64_t row = sampler ? (int64_t)(tid & 63) * P / 64 : bundle * ROWS + tid;
    if (row < P) n = entries(row, b);
  }
  for (int i = tid; i < G * words; i += THREADS) nib[i] = 0;
  const int64_t long_limit = spmm_long_limit(row_ptr, P, Q, capacity);
  const bool is_long = n > long_limit;   // the long-row kernels' business
  if (tid < ROWS) {
    s_b[tid] = b;
    s_n[tid] = is_long ? 0 : (int)n;
  }
  float sample_v = 0.0f;   // on its way while the rows' entries are looked at
  if (sampler && n > 0 && !is_long) sample_v = val[b + n / 2];
  if (tid == 0) s_bad = 0;
  if (tid < G) s_total[tid] = 0;
  __syncthreads();
  int tpr = PK_TPR;
  int br = tid / PK_TPR, rt = tid % PK_TPR;   // row of the bundle, thread of the row
  int grp = br / 16, r = br % 16;
  int n_mine = s_n[br];
  const int32_t* cp = col_idx + s_b[br];
  const float* vp = val + s_b[br];
  for (int i0 = rt; i0 < n_mine; i0 += 4 * PK_TPR) {   // four entries a thread in flight
    int c[4], before[4];
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = min(i0 + u * PK_TPR, n_mine - 1);
      c[u] = cp[i];
      v[u] = vp[i];
      before[u] = i > 0 ? cp[i - 1] : -1;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      uint32_t t[3];
      const int nt = bf16_terms(v[u], t);
      if (i0 + u * PK_TPR >= n_mine) continue;
      if ((uint32_t)c[u] >= (uint32_t)Q || before[u] >= c[u] || nt > 3) { s_bad = 1; continue; }
      atomicOr(&nib[grp * words + (c[u] >> 3)], ((1u << nt) - 1u) << (4 * (c[u] & 7)));
    }
  }
  __syncthreads();
  if (sampler) {
    // more than one term: bits below bf16's; more than two: so has what the nearest bf16 number leaves
    const uint32_t u = f2u(sample_v);
    const float left = sample_v - u2f((u + 0x8000u) & 0xffff0000u);
    const uint64_t mine = is_long ? 0 : (uint64_t)min(n, (int64_t)Q);   // 21 bits hold the sum of 64
    uint64_t sum = mine | ((u & 0xffffu) ? mine << 21 : 0) | ((f2u(left) & 0xffffu) ? mine << 42 : 0);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) sum += __shfl_xor(sum, o, 64);
    const int rows = __popcll(__ballot(!is_long));
    if ((tid & 63) == 0) {
      s_sample[0] = rows;
      s_sample[1] = (int)(sum & 0x1fffff);
      s_sample[2] = (int)(sum >> 21 & 0x1fffff);
      s_sample[3] = (int)(sum >> 42);
    }
  }
  for (int i = tid; i < G * phases; i += THREADS) {
    int sum = 0;
#pragma unroll
    for (int w = 0; w < SM_KC / 8; w += 8) {
      const u32x4* const m = reinterpret_cast<const u32x4*>(nib + i * (SM_KC / 8) + w);
      const u32x4 m0 = m[0], m1 = m[1];
      u32x4 before;
#pragma unroll
      for (int h = 0; h < 4; ++h) {
        before[h] = (uint32_t)sum;
        sum += __popc(h < 2 ? m0[2 * h] : m1[2 * h - 4]);
        before[h] |= (uint32_t)sum << 16;
        sum += __popc(h < 2 ? m0[2 * h + 1] : m1[2 * h - 3]);
      }
      *reinterpret_cast<u32x4*>(pre + i * (SM_KC / 8) + w) = before;
    }
    start[i] = sum;
    atomicAdd(&s_total[i / phases], sum);
  }
  __syncthreads();
  if (tid < 64) {
    // S follows an even pace, between what must be done (chunk c - SM_SLACK leaves) and what fills whole steps, and takes no more steps in a
    // phase than the pace does, unless it must: the waves of a workgroup wait for each other at every phase, so that one which makes up for a
    // step it fell behind holds up all others.  The pace begins a phase late, when every bundle has the slots for it, and is that of the next
    // multiple of four steps, so that most bundles have the same (16384 x 4096 -> 12288 at 2 % 811 -> 777 us; counted over the phases, the fullest SIMD of a
    // workgroup has 6 % fewer steps).  Bundles of one group keep to their own pace, without a limit (2048 x 8192 -> 2048 90.6 us, 92.0 with).  One wave: a lane
    // holds the counts of every 64th chunk, the recurrence runs on scalars.
    constexpr bool EVEN = G > 1;
    int total = 0, e[G], ends[SM_SLACK + 1], S = 0, quot, rem, pace = 0, more = 0, left = 0;
    for (int j = 0; j < G; ++j) { total = max(total, (s_total[j] + 31) / 32); e[j] = 0; }
    total = __builtin_amdgcn_readfirstlane(total);
    if constexpr (EVEN) total = (total + SM_PACE) / SM_PACE * SM_PACE;
    quot = total / phases;
    rem = total % phases;
#pragma unroll
    for (int i = 0; i <= SM_SLACK; ++i) ends[i] = 0;
    int32_t* const sc = sched + bundle * phases;
    for (int c0 = 0; c0 < phases; c0 += 64) {
      int cnt[G], first[G], mine = 0;
#pragma unroll
      for (int j = 0; j < G; ++j) { cnt[j] = c0 + tid < phases ? start[j * phases + c0 + tid] : 0; first[j] = 0; }
      const int here = min(64, phases - c0);
      for (int i = 0; i < here; ++i) {
        int least = 0x7fffffff, most = 0;
#pragma unroll
        for (int j = 0; j < G; ++j) {
          const int st = max(e[j], 32 * S);
          first[j] = tid == i ? st : first[j];
          e[j] = st + __builtin_amdgcn_readlane(cnt[j], i);
          least = min(least, e[j]);
          most = max(most, e[j]);
        }
#pragma unroll
        for (int k = 0; k < SM_SLACK; ++k) ends[k] = ends[k + 1];
        ends[SM_SLACK] = most;
        const int lo = max(S, (ends[0] + 31) / 32);
        int next = pace;
        if constexpr (EVEN) next = min(pace, S + more);
        more = quot;   // pace: floor(total * c / phases) from here on
        left += rem;
        if (left >= phases) { left -= phases; ++more; }
        pace += more;
        if constexpr (!EVEN) next = pace + (left > 0 ? 1 : 0);
        S = c0 + i == phases - 1 ? max(lo, (most + 31) / 32) : max(min(next, least / 32), lo);
        mine = tid == i ? S : mine;
      }
      if (tid < here) {
        sc[c0 + tid] = mine;
#pragma unroll
        for (int j = 0; j < G; ++j) start[j * phases + c0 + tid] = first[j];
      }
    }
    const bool ok = !s_bad && S <= cap && pk_worth(s_sample, Q, small_grid);
    if (!ok)
      for (int c = tid; c < phases; c += 64) sc[c] = 0;
    if (bundle == bundles - 1 && tid < SM_STEPS_PAD) steps[bundles + tid] = -1;   // nothing packed past the last bundle
    if (tid == 0) {
      s_steps = ok ? S : 0;
      steps[bundle] = ok ? S : -1;
      redo[bundle] = 0;
    }
  }
  __syncthreads();
  const int T = s_steps;
  if (T == 0) return;
  int gt = tid % (16 * PK_TPR);   // thread of the group
  if (split) {   // all of them to the one group
    tpr = THREADS / 16;
    grp = part;
    r = tid / (THREADS / 16);
    rt = tid % (THREADS / 16);
    gt = tid;
    n_mine = s_n[grp * 16 + r];
    cp = col_idx + s_b[grp * 16 + r];
    vp = val + s_b[grp * 16 + r];
  }
  uint8_t* const ag = a_buf + (bundle * G + grp) * (int64_t)(cap + 1) * 1024;
  uint8_t* const og = o_buf + (bundle * G + grp) * (int64_t)(cap + 1) * 64;
  const u32x4 z = {0u, 0u, 0u, 0u};
  for (int i = gt; i < T * 64; i += 16 * tpr) *reinterpret_cast<u32x4*>(ag + (int64_t)i * 16) = z;
  for (int i = gt; i < T * 4; i += 16 * tpr) *reinterpret_cast<u32x4*>(og + (int64_t)i * 16) = z;
  __syncthreads();   // the zeros are written (a workgroup's stores reach L2 in order) before the values
  for (int i0 = rt; i0 < n_mine; i0 += 4 * tpr) {
    int cc[4];
    float v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int i = min(i0 + u * tpr, n_mine - 1);
      cc[u] = cp[i];
      v[u] = vp[i];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      if (i0 + u * tpr >= n_mine) continue;
      const int c = cc[u];
      uint32_t t[3];
      const int nt = bf16_terms(v[u], t);
      const int w = grp * words + (c >> 3);
      const int pos = start[grp * phases + c / SM_KC] + pre[w] + __popc(nib[w] & ((1u << (4 * (c & 7))) - 1u));
      const uint16_t at = (uint16_t)(c % (SM_RING * SM_KC));   // row of the ring
      for (int k = 0; k < nt; ++k) {
        const int p = pos + k;
        *reinterpret_cast<uint16_t*>(ag + (int64_t)(p >> 5) * 1024 + sm_a_at(p & 31, r)) = (uint16_t)t[k];
        *reinterpret_cast<uint16_t*>(og + (int64_t)p * 2) = at;
      }
    }
  }
}

// WV waves multiply, G groups of 16 rows each; one or two more stage D.  Bundles that are not packed are left out, and a
// bundle with a non-finite sum is marked in redo: a zero value times an infinite or NaN element of D
// reaches the other rows of the group.  The tiled kernel writes the rows of both afterwards, from their entries.
template <int G, int WV>
__global__ __launch_bounds__((WV + sm_stagers(G)) * 64) void spmm_mfma_kernel(const uint8_t* __restrict__ a_buf, const uint8_t* __restrict__ o_buf,
                                                            const int32_t* __restrict__ sched, const int32_t* __restrict__ steps,
                                                            int32_t* __restrict__ redo, int cap, int phases, int row_blocks,
                                                            int col_blocks, int64_t P, int64_t Q,
                                                            const uint16_t* __restrict__ D, int64_t N, float* __restrict__ R) {
  constexpr int SM_AHEAD = sm_ahead(G), STAGERS = sm_stagers(G);
  __shared__ __attribute__((aligned(16))) uint8_t ring[SM_RING * SM_CHUNKB];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Workgroup i runs on XCD i % 8; each XCD takes a contiguous run of tiles, ordered so that the workgroups
  // it runs at a time form four row blocks x eight column blocks and share D and the packed rows in its L2.
  const int total = row_blocks * col_blocks, per_xcd = (total + 7) / 8;
  const int id = (int)(blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8);
  if ((int)(blockIdx.x / 8) >= per_xcd || id >= total) return;
  const int strip = id / (SM_STRIP * row_blocks);
  const int width = min(SM_STRIP, col_blocks - SM_STRIP * strip);
  const int in_strip = id - SM_STRIP * strip * row_blocks;
  const int64_t n0 = (int64_t)(SM_STRIP * strip + in_strip % width) * SM_NT;
  const int rb = in_strip / width;
  const int64_t bundles = (P + 16 * G - 1) / (16 * G);
  // Nothing packed among the workgroup's bundles: every wave sees that alike (steps is written by the packing only) and
  // leaves.  Scalar loads, behind the first requests.
  auto nothing = [&]() {
    int32_t most = -1;
#pragma unroll
    for (int w = 0; w < WV; ++w) most = max(most, steps[(int64_t)rb * WV + w]);   // -1 past the last bundle
    return most < 0;
  };

  if (wave >= WV) {
    // The staging waves.  Their loads are their own business: a wave's loads return in order, so in a multiplying wave
    // every operand load would wait for the chunk requested before it.  One instruction fills 4 rows of a chunk;
    // rows past Q and columns past N read zero (offset out of range).
    constexpr int LD = SM_KC / 4 / STAGERS;
    static_assert(SM_AHEAD * LD <= 64, "a load more than can be counted waits for one");
    const int first = STAGERS == 1 ? 0 : (wave - WV) * LD;   // of the chunk's instructions
    const __amdgpu_buffer_rsrc_t rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(D) + n0, 0, (int)(uint32_t)((Q * N - n0) * 2), 0x00020000);
    const bool in_n = n0 + (lane & 15) * 8 < N;
    const uint32_t rowb = (uint32_t)(N * 2);
    const uint32_t voff = (uint32_t)(4 * first + (lane >> 4)) * rowb + (uint32_t)(lane & 15) * 16u;
    auto stage = [&](int c) {
      uint8_t* const slot = ring + (c % SM_RING) * SM_CHUNKB + first * 4 * SM_ROWB;
      const int rows = in_n ? (int)min((int64_t)SM_KC, Q - (int64_t)c * SM_KC) - 4 * first - (lane >> 4) : 0;
      uint32_t off = voff + (uint32_t)(c * SM_KC) * rowb;
#pragma unroll
      for (int j = 0; j < LD; ++j) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)(slot + j * 4 * SM_ROWB), 16,
                                                 4 * j < rows ? off : 0xf0000000u, 0, 0, 0);
        off += 4 * rowb;
      }
    };
#pragma unroll 1
    for (int c = 0; c < SM_AHEAD; ++c) stage(c);
    if (nothing()) {
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // as at the end
      return;
    }
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((SM_AHEAD - 1) * LD) : "memory");
    __builtin_amdgcn_s_barrier();
#pragma unroll 1
    for (int p = 0; p < phases; ++p) {
      stage(p + SM_AHEAD);   // past the end: zeros into a chunk nobody reads any more
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"((SM_AHEAD - 1) * LD) : "memory");   // chunk p + 1 is there
      __builtin_amdgcn_s_barrier();
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no load may land in LDS after the workgroup has given it back
    return;
  }

  f32x4 acc[G][8];
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[g][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  // The packed steps are read through scalar descriptors (a wave's groups lie one after another): the lane part
  // of an address is one register, whatever the group.
  const int64_t bundle = (int64_t)rb * WV + wave;
  const int64_t bl = min(bundle, bundles - 1);
  const uint32_t a_stride = (uint32_t)(cap + 1) * 1024u, o_stride = (uint32_t)(cap + 1) * 64u;
  const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(a_buf) + bl * G * (int64_t)a_stride, 0, (int)(a_stride * (uint32_t)G), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrc_o = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(o_buf) + bl * G * (int64_t)o_stride, 0, (int)(o_stride * (uint32_t)G), 0x00020000);
  const int32_t* const sp = sched + bl * phases;
  const uint32_t a_lane = (uint32_t)lane * 16u, o_lane = (uint32_t)(lane >> 4) * 16u;
  // Steps requested: the next one of each group; a single group's next SM_DEEP, which a phase or two have in all, or each would wait for
  // a round trip to L2 (steps past the last lie past the descriptors' ends or are another bundle's room, and are not used).
  constexpr int SETS = G == 1 ? SM_DEEP : G;
  u32x4 a[SETS], o[SETS];
  auto fetch = [&](int set, uint32_t step) {
    const uint32_t g = G == 1 ? 0u : (uint32_t)set;
    a[set] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_a, a_lane, g * a_stride + step * 1024u, 0);
    o[set] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_o, o_lane, g * o_stride + step * 64u, 0);
  };
#pragma unroll
  for (int set = 0; set < SETS; ++set) fetch(set, G == 1 ? (uint32_t)set : 0u);
  const uint32_t lbase = (uint32_t)(lane & 15) * 16u;
  const bool live = steps[bundle] >= 0;
  if (nothing()) return;
  __builtin_amdgcn_s_barrier();

  uint32_t done = 0;
  auto multiply = [&](int set, int g) {   // a step of group g
    u32x4 d[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      // row * 256 + the lane's bytes, in one instruction
      const uint32_t at = __builtin_amdgcn_perm(o[set][e >> 1], lbase, (e & 1) ? 0x0c070600u : 0x0c050400u);
      d[e] = *reinterpret_cast<const u32x4*>(ring + at);
    }
    const bf16x8 av = __builtin_bit_cast(bf16x8, a[set]);
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      u32x8 two;   // columns 2 w and 2 w + 1 of the lane's eight rows, as they came
#pragma unroll
      for (int e = 0; e < 8; ++e) two[e] = d[e][w];
      const bf16x16 dv = __builtin_bit_cast(bf16x16, two);
      acc[g][2 * w] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(av, dv, acc[g][2 * w], SM_FIRST_OF_TWO, 0, 0);
      acc[g][2 * w + 1] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(av, dv, acc[g][2 * w + 1], SM_FIRST_OF_TWO, 0, 1);
    }
    __builtin_amdgcn_sched_barrier(0);
    fetch(set, G == 1 ? done + SM_DEEP - 1 : done);   // into the registers this step is done with
    __builtin_amdgcn_sched_barrier(0);
  };
  int turn = 0;   // a single group's: the set of its next step
  auto rounds = [&](uint32_t upto) {
    if constexpr (G == 1) {
      static_assert(SM_DEEP == 3, "the turns below");
      while (done < upto) {
        if (turn == 0) { ++done; multiply(0, 0); turn = 1; if (done == upto) break; }
        if (turn == 1) { ++done; multiply(1, 0); turn = 2; if (done == upto) break; }
        ++done; multiply(2, 0); turn = 0;
      }
    } else {
      while (done < upto) {
        ++done;
#pragma unroll
        for (int g = 0; g < G; ++g) multiply(g, g);
      }
    }
  };
  // The steps done at the end of each phase, 64 phases a register, all of them loaded and waited for here: a load inside the loop, of
  // which there was one every 64 phases, made the compiler wait at every phase for whatever was under way, the next steps' operands above all.
  int plan[SM_PLANS];
#pragma unroll
  for (int i = 0; i < SM_PLANS; ++i) plan[i] = live ? sp[min(64 * i + lane, phases - 1)] : 0;
#pragma unroll
  for (int i = 0; i < SM_PLANS; ++i) asm volatile("" : "+v"(plan[i]));
  for (int p = 0; p < phases; ++p) {
    if (p > 0 && (p & 63) == 0)
#pragma unroll
      for (int i = 0; i + 1 < SM_PLANS; ++i) plan[i] = plan[i + 1];
    const uint32_t upto = (uint32_t)__builtin_amdgcn_readlane(plan[0], p & 63);
    // A single group's operands, on their way since the phase before, are waited for once a phase.  Where a step begins at any of three sets,
    // the compiler does not know how many requests came after the set's own and waits for all of them, at every step, a round trip to L2 each.
    // Without / with, us: 1536 x 8192 -> 2048 at 2 % 76.5 / 71.0, at 6 % 122.2 / 107.5; 2048 x 11008 -> 2048 98.8 / 91.8 and 161.2 / 143.0, at 0.2 %,
    // a step a phase at most, 75.4 / 75.2; 9312 x 11008 -> 512 147.0 / 140.4 and 246.4 / 232.2.
    if constexpr (G == 1) __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
    rounds(upto);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this wave's reads of the chunk that goes next are done
    __builtin_amdgcn_s_barrier();
  }

  if (!live) return;
#pragma unroll
  for (int g = 0; g < G; ++g) {
    const int64_t row0 = (bundle * G + g) * 16;
    if (row0 >= P) break;
    float nf = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; ++j)
#pragma unroll
      for (int i = 0; i < 4; ++i) nf = fmaf(acc[g][j][i], 0.0f, nf);
    if (__ballot(nf != 0.0f) != 0ull) {
      if (lane == 0) redo[bundle] = 1;
      continue;
    }
    // A lane holds 8 columns of 4 rows; four neighbours exchange 16-byte pieces so that each store instruction
    // writes whole 64-byte runs: lane q of four stores piece q, then piece q + 4, of their 32 columns.
    const int64_t col = n0 + (lane & 12) * 8 + (lane & 3) * 4;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      f32x4 st[2];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int k = 0; k < 4; ++k) {
          // quad_perm: every lane reads lane 0 0 1 1 (first half) or 2 2 3 3 of its four
          const int even = h ? __builtin_amdgcn_mov_dpp((int)f2u(acc[g][k][i]), 0xfa, 0xf, 0xf, true)
                             : __builtin_amdgcn_mov_dpp((int)f2u(acc[g][k][i]), 0x50, 0xf, 0xf, true);
          const int odd = h ? __builtin_amdgcn_mov_dpp((int)f2u(acc[g][4 + k][i]), 0xfa, 0xf, 0xf, true)
                            : __builtin_amdgcn_mov_dpp((int)f2u(acc[g][4 + k][i]), 0x50, 0xf, 0xf, true);
          st[h][k] = u2f((uint32_t)((lane & 1) ? odd : even));
        }
      const int64_t row = row0 + (lane >> 4) * 4 + i;
      float* const dst = R + row * N + col;
      if (row < P && col < N) *reinterpret_cast<f32x4*>(dst) = st[0];
      if (row < P && col + 16 < N) *reinterpret_cast<f32x4*>(dst + 16) = st[1];
    }
  }
}

template <int G, int WV>
struct Shape {   // of a workgroup: groups a wave, waves that multiply
  static constexpr int groups = G, waves = WV;
};

}  // namespace

int fp4_compute_units_of_current_device();

// bytes of scratch the packed form of a P x Q matrix takes, and that of any smaller one: a matrix too wide for this path
// counts as the widest that is not
int64_t fp4_spmm_mfma_scratch_bytes(int64_t P, int64_t Q) {
  Q = std::min(Q, SM_MAXQ);
  const int64_t groups = (P + 15) / 16 + 2;   // whole bundles of up to three
  return groups * ((sm_cap(Q) + 1) * (1024 + 64) + (sm_phases(Q) + 2) * 4) + 1024;
}

// Returns 1 when the product is left to the tiled kernel.  Otherwise that kernel has what remains: the rows of bundle i
// (16 rest.groups of them) where rest.steps[i] < 0 or rest.redo[i] != 0.
int fp4_launch_spmm_mfma(const int64_t* row_ptr, const int32_t* col_idx, const float* val, int64_t capacity, int64_t P,
                         int64_t Q, const void* D, int64_t N, float* R, void* scratch, int32_t* list, int32_t* count,
                         SpmmRest& rest, hipStream_t s) {
  if (Q > SM_MAXQ || Q <= 0 || (uint64_t)(Q + 4 * SM_KC) * (uint64_t)N * 2 > 0xe0000000ull) return 1;   // 32-bit offsets into D
  const int cap = (int)sm_cap(Q), phases = (int)sm_phases(Q);
  const int col_blocks = (int)((N + SM_NT - 1) / SM_NT);
  const bool small_grid = (P + 1023) / 1024 * ((N + 63) / 64) < 256;   // workgroups of the tiled kernel
  auto blocks = [&](int g, int wv) { return (P + 16 * g * wv - 1) / (16 * g * wv); };
  auto launch = [&](auto shape) {
    constexpr int G = decltype(shape)::groups, WV = decltype(shape)::waves;
    const int64_t bundles = (P + 16 * G - 1) / (16 * G);
    uint8_t* const a_buf = reinterpret_cast<uint8_t*>(scratch);
    uint8_t* const o_buf = a_buf + bundles * G * (int64_t)(cap + 1) * 1024;
    int32_t* const sched = reinterpret_cast<int32_t*>(o_buf + bundles * G * (int64_t)(cap + 1) * 64);
    int32_t* const steps = sched + bundles * phases;
    int32_t* const redo = steps + bundles + SM_STEPS_PAD;
    const size_t lds = (size_t)G * phases * (SM_KC / 8) * 6 + (size_t)G * phases * 4;
    const bool split = G > 1 && bundles * G <= 2 * fp4_compute_units_of_current_device();
    hipLaunchKernelGGL((spmm_pack_kernel<G>), dim3((unsigned)(bundles * (split ? G : 1)) + 1), dim3(16 * G * pk_tpr(G)), lds, s, row_ptr, col_idx,
                       val, capacity, P, (int)Q, cap, phases, small_grid, split, a_buf, o_buf, sched, steps, redo, list, count);
    const int row_blocks = (int)blocks(G, WV);
    const int per_xcd = (row_blocks * col_blocks + 7) / 8;
    hipLaunchKernelGGL((spmm_mfma_kernel<G, WV>), dim3((unsigned)(8 * per_xcd)), dim3((WV + sm_stagers(G)) * 64), 0, s, a_buf, o_buf, sched,
                       steps, redo, cap, phases, row_blocks, col_blocks, P, Q, reinterpret_cast<const uint16_t*>(D),
                       N, R);
    rest = SpmmRest{steps, redo, G};
    static_assert(G <= 3, "the rest's bundles");
  };
  // A phase takes a workgroup about as long as 300 of its rows do, whatever their number (staging, the barrier), and 256 workgroups run at
  // a time.  So: the shape with the fewest rounds x (300 + rows), but a smaller one only where it saves a tenth on the larger.  That tenth
  // decides between 528 and 384 rows alone, in grids of several rounds, where 384 save up to 4 % by this count: about as fast at 2 % of entries, slower
  // where they are few, which the sizes don't tell, faster where they are many.  528 / 384, us, at 0.2, 2 and 6 %: 5120 x 4096 -> 13824 208 / 226,
  // 308 / 307, 531 / 501; 12288 x 4096 -> 5504 192 / 214, 298 / 302, 541 / 506; 6144 x 5120 -> 13824 306 / 318, 442 / 428, 763 / 713; 5856 x 2048 ->
  // 13824 148 / 160, 202 / 206, 325 / 313.  Multiplying waves are whole numbers a SIMD beside the staging ones (8: two, 12: three, 11 + 1:
  // three), and rows come in the halves and quarters of which row counts are made; the sixteen rows that 128 and 192 have more than 112 and 176
  // cost nothing (within one round of either, 3584 x 8192 -> 1024 at 0.2, 2 and 6 % 61 / 61, 74 / 73, 117 / 114, 1408 x 8192 -> 4096 64 / 64, 80 / 78, 122 / 118).
  // Products, their packing and long rows included, 528 / 384 / 256 / 192 / 128 rows, us, the one taken in brackets; at 2 %
  // 2048 x 8192 -> 2048 123 / 110 / 95 / 83 / (76), 3072 x 8192 -> 2048 124 / 110 / 97 / (87) / 122, 4096 x 8192 -> 2048 126 / 112 / (100) / 140 /
  // 126, 5504 x 2048 -> 4096 92 / (84) / 93 / 103 / 120, 4096^3 (82) / 110 / 96 / 113 / 128, 4096 x 4096 -> 11008 (192) / 203 / 235 / 267 / 308,
  // 2048 x 8192 -> 5504 (147) / 208 / 180 / 160 / 190; at 0.2 % 4096 x 8192 -> 2048 81 / 81 / (74) / 107 / 100.
  const std::tuple<Shape<3, 11>, Shape<2, 12>, Shape<2, 8>, Shape<1, 12>, Shape<1, 8>> shapes;
  std::apply([&](auto... shape) {
    auto cost = [&](int g, int wv) { return (blocks(g, wv) * col_blocks + 255) / 256 * (300 + 16 * g * wv); };
    int64_t least = 0;
    int taken = -1, i = 0;
    for (const int64_t c : {cost(shape.groups, shape.waves)...}) {
      if (taken < 0 || 10 * c < 9 * least) { least = c; taken = i; }
      ++i;
    }
    i = 0;
    (void)((i++ == taken && (launch(shape), true)) || ...);
  }, shapes);
  FP4_CHECK_LAUNCH();
  return FP4_OK;
}
