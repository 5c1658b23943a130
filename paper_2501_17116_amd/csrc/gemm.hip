// FP4 x FP4 GEMM on the gfx950 F8F6F4 matrix cores with the scale-dequantizing epilogue
// (Fig. 2; App. C.2: the scaled quantized operands go through the GEMM and the 1/sf
// factors are applied to its result), optional fp32 addend (the sparse residual product
// of Sec. 3.2) and optional DGE factor (Sec. 3.1 Eq. 8) for the weight gradient.
//
// out[p, q] = sum_k v(L[p, k]) v(Rt[q, k]) * (1/gamma_l[p]) * (1/gamma_r[q]) (+ addend) (* f')
//
// Both operands are K-major packed E2M1 ("NT" GEMM).  Tile 256 x 256 per workgroup of eight
// wave64s (2 along rows x 4 along columns, 128 x 64 each), K step 256 codes (128 bytes per
// row), operands brought into two LDS stages by direct-to-LDS buffer loads, 32x32x64 MFMA with
// both operands in the FP4 format and the hardware block scales held at 2^0.  Workgroups are
// persistent (one per CU, walking an XCD-local run of tiles).  Every product of two E2M1 values
// is a multiple of 1/4 and bounded by 36, so the fp32 accumulator is exact for any contraction
// length below 2^22/36 and does not depend on summation order.
#include "fp4_common.h"
#include "gemm_tiling.h"
#include "fp4_measure.h"

#include <algorithm>
#include <type_traits>
#include <utility>

typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

namespace {

constexpr int BM = 256;          // rows of L per tile  (output rows)
constexpr int BN = 256;          // rows of Rt per tile (output columns)
constexpr int BKB = 128;         // bytes of K per step (256 codes)
constexpr int WQ = 4;            // waves along the output-column axis (x 2 along rows)
constexpr int NTHREADS = 2 * WQ * 64;
constexpr int NWAVES = NTHREADS / 64;
constexpr int QI = BN / WQ / 32;  // 32-column MFMA blocks per wave
constexpr int NLD = BM * 8 / NTHREADS;  // 16-byte chunks per thread, per operand, per K step
constexpr int GROUP_P = 8;       // tile-rows per L2 reuse group
constexpr int TILE_BYTES = BM * BKB;              // one operand, one stage (rows unpadded)
constexpr int EPI_LD = QI * 32 + 4;               // floats per row of the epilogue staging tile
constexpr int EPI_ROWS = 32;                      // rows of a wave's tile parked at a time
constexpr int EPI_BYTES = NWAVES * EPI_ROWS * EPI_LD * 4;
// Stage b of the operands sits at [b * 2 * TILE_BYTES, +2 * TILE_BYTES): L, then Rt.  The epilogue's
// staging area lies behind stage 0, over stage 1, so the next tile's stage 0 can be fetched while
// the epilogue of this one runs.
constexpr int STAGE_BYTES = 2 * TILE_BYTES;
constexpr int EPI_BASE = STAGE_BYTES;
constexpr int SMEM_BYTES = 2 * STAGE_BYTES > EPI_BASE + EPI_BYTES ? 2 * STAGE_BYTES : EPI_BASE + EPI_BYTES;
static_assert(SMEM_BYTES <= 160 * 1024, "LDS budget");
constexpr uint32_t OUT_OF_RANGE = GEMM_OUT_OF_RANGE;   // where a descriptor has nothing: arrives as zeros
static_assert(BKB == GEMM_K_STEP && BM == 256 && BN == 256, "as gemm_tiling has them");

// LDS layout of an operand stage: row r occupies bytes [128 r, 128 r + 128); its 16-byte
// chunk c sits in slot c ^ ((r >> 1) & 7).  Sixteen consecutive rows reading the same logical
// chunk then touch sixteen different 16-byte bank groups of the 256-byte bank period, and a
// wave's direct-to-LDS load (64 lanes x 16 B = 8 whole rows) stays one contiguous KiB.

struct GemmShape {
  int64_t P, Q, Kb, ldo, ldw;
  float dge_k, dge_cap;
  int tiles_p, tiles_q;
  int first, count;   // 256 x 256 tiles of this launch, in the order of tile_at
  int stagger;   // how much later than the one before each quarter of the workgroups begins, in 512 cycles
};

// Tile id of the order in which they are taken: eight tile-rows side by side.
FP4_D void tile_at(const GemmShape& g, int id, int& tp, int& tq) {
  const int in_group = GROUP_P * g.tiles_q;
  const int group = id / in_group;
  const int first_p = group * GROUP_P;
  const int gsz = min(g.tiles_p - first_p, GROUP_P);
  tp = first_p + (id % in_group) % gsz;
  tq = (id % in_group) / gsz;
}

template <class F, int... I>
FP4_D void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
FP4_D void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// two fp32 -> packed bf16 pair, round to nearest even (hardware conversion on gfx950)
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
FP4_D uint32_t pack_bf16x2(float a, float b) {
  f32x2_t f = {a, b};
  bf16x2_t h = __builtin_convertvector(f, bf16x2_t);
  union { bf16x2_t h; uint32_t u; } c;
  c.h = h;
  return c.u;
}

// OUT_BF16: output dtype; DGE: multiply by the DGE factor of W (dtype W_BF16).
template <bool OUT_BF16, bool DGE, bool W_BF16, bool KRAGGED>
__global__ __launch_bounds__(NTHREADS) void fp4_gemm_nt_kernel(
    const uint8_t* __restrict__ Lp, const uint8_t* __restrict__ Rp, const float* __restrict__ gl,
    const float* __restrict__ gr, const float* addend, void* outp, const void* __restrict__ Wp,
    const float* __restrict__ gamma_w, GemmShape g) {
  __shared__ __attribute__((aligned(16))) uint8_t smem[SMEM_BYTES];
  uint8_t* const sL = smem;                // stage b of L at sL + b * STAGE_BYTES
  uint8_t* const sR = smem + TILE_BYTES;   // stage b of Rt at sR + b * STAGE_BYTES

  // Workgroups are dealt round-robin to the 8 XCDs; give each XCD a contiguous run of the
  // tile sequence so that tiles sharing operand rows meet in the same L2.
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform, kept scalar
  const int wave_p = wave & 1;
  const int wave_q = wave >> 1;   // 0 .. WQ-1
  const int l32 = lane & 31;
  const int lhi = lane >> 5;

  // Persistent workgroups: the grid is at most one workgroup per CU and each walks a strided
  // share of its XCD's run of tiles, so a tile's stores drain while the next tile computes and
  // no workgroup relaunch sits between tiles.
  const int total = g.count;
  const int per_xcd = (total + 7) / 8;
  const int xcd = (int)(blockIdx.x % 8);
  const int wg_in_xcd = (int)(blockIdx.x / 8), wgs_per_xcd = (int)(gridDim.x / 8);
  const int run_end = min(total, (xcd + 1) * per_xcd);
  int lid = xcd * per_xcd + wg_in_xcd;
  if (lid >= run_end) return;
  for (int i = g.stagger * ((wg_in_xcd >> 3) & 3); i > 0; --i) __builtin_amdgcn_s_sleep(8);

  // Per-tile state.  The scalars (tile origin, base pointers, buffer descriptors) of the tile whose
  // operands are being fetched; they move on to the next tile as soon as this tile's main loop is
  // over, so the epilogue keeps its own copy of the origin.
  int64_t P0 = 0, Q0 = 0;
  const uint8_t* tileL = nullptr;
  const uint8_t* tileR = nullptr;
  __amdgpu_buffer_rsrc_t rsrcL, rsrcR;
  // Operand staging.  Load instruction j of wave w fills the KiB [(w*NLD + j) * 1024, +1024) of a
  // stage = tile rows 8*(w*NLD+j) .. +7; lane i owns slot i & 7 of row (i >> 3) of that group and
  // therefore fetches logical chunk (i & 7) ^ ((row >> 1) & 7) of its row.
  uint32_t goffL[NLD], goffR[NLD];   // byte offset of this lane's chunk from the tile's first row
  // tile base pointers are workgroup-uniform; say so, so descriptors and offsets stay scalar
  auto uniform_ptr = [](const uint8_t* p) {
    const uint64_t v = (uint64_t)p;
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
    return (const uint8_t*)(((uint64_t)hi << 32) | lo);
  };
  auto tile_scalars = [&](int id) {
    int tp, tq;
    tile_at(g, id, tp, tq);
    P0 = (int64_t)tp * BM;
    Q0 = (int64_t)tq * BN;
    tileL = uniform_ptr(Lp + P0 * g.Kb);
    tileR = uniform_ptr(Rp + Q0 * g.Kb);
    // buffer descriptors over the tile's rows: loads past their end return zero
    const uint64_t bytesL = (uint64_t)min(g.P - P0, (int64_t)BM) * (uint64_t)g.Kb, bytesR = (uint64_t)min(g.Q - Q0, (int64_t)BN) * (uint64_t)g.Kb;
    rsrcL = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(tileL), 0,
        __builtin_amdgcn_readfirstlane((int)(bytesL > 0xffffffffull ? 0xffffffffu : (uint32_t)bytesL)), 0x00020000);
    rsrcR = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint8_t*>(tileR), 0,
        __builtin_amdgcn_readfirstlane((int)(bytesR > 0xffffffffull ? 0xffffffffu : (uint32_t)bytesR)), 0x00020000);
  };
  // The per-lane offsets are recomputed where they are needed (after the main loop for the early
  // fetch of the next tile, and again at the top of that tile) from a copy of the lane id the
  // optimizer cannot see through: kept alive across the epilogue they would cost registers there.
  auto tile_offsets = [&]() {
    int ln = lane;
    asm volatile("" : "+v"(ln));
#pragma unroll
    for (int j = 0; j < NLD; ++j) {
      const int row = 8 * (wave * NLD + j) + (ln >> 3);
      const int chunk = (ln & 7) ^ ((row >> 1) & 7);
      const int64_t rp = min(P0 + row, g.P - 1) - P0;   // rows past the edge re-read the last row
      const int64_t rq = min(Q0 + row, g.Q - 1) - Q0;
      goffL[j] = (uint32_t)(rp * g.Kb + chunk * 16);
      goffR[j] = (uint32_t)(rq * g.Kb + chunk * 16);
    }
  };
  const int KT = (int)((g.Kb + BKB - 1) / BKB);

  f32x16 acc[QI][4];

  // global -> LDS without passing through registers.  Where the last K step overhangs the row (KRAGGED), the chunks
  // behind the row's end take an offset past the descriptor's end and arrive as zeros.  Through registers, with the overhang
  // blanked, such a contraction took twice the time (8192 x 2048, 5504 codes: 100 us, now 51).
  const uint32_t ragged_row = (uint32_t)g.Kb;
  auto load_tile = [&](int kt, int buf, int jb, int je) {
    [[maybe_unused]] const uint32_t room = ragged_row - (uint32_t)(kt * BKB);   // bytes of the row from this step on
    [[maybe_unused]] const int ln = lane;
#pragma unroll
    for (int j = jb; j < je; ++j) {
      uint32_t ol = goffL[j], orr = goffR[j];
      if constexpr (KRAGGED) {
        const int row = 8 * (wave * NLD + j) + (ln >> 3);
        const bool in = (uint32_t)(((ln & 7) ^ ((row >> 1) & 7)) * 16) < room;
        ol = in ? ol : OUT_OF_RANGE;
        orr = in ? orr : OUT_OF_RANGE;
      }
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rsrcL, (__attribute__((address_space(3))) void*)(sL + buf * STAGE_BYTES + (wave * NLD + j) * 1024), 16, ol, kt * BKB, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rsrcR, (__attribute__((address_space(3))) void*)(sR + buf * STAGE_BYTES + (wave * NLD + j) * 1024), 16, orr, kt * BKB, 0, 0);
    }
  };

  // MFMA fragments: lane (l32, lhi) needs, for k-slice ks of a stage, logical chunk 2 ks + lhi
  // of rows l32 + 32 j.  (row >> 1) & 7 only depends on l32 because the row bases are
  // multiples of 32.
  const int key = (l32 >> 1) & 7;
  int frag_l[4], frag_r[4];   // per k-slice byte offsets inside a stage
#pragma unroll
  for (int ks = 0; ks < 4; ++ks) {
    const int slot = (2 * ks + lhi) ^ key;
    frag_l[ks] = (wave_p * 128 + l32) * BKB + slot * 16;
    frag_r[ks] = (wave_q * (QI * 32) + l32) * BKB + slot * 16;
  }
  u32x4 fl[2][4], fr[2][QI];   // fragments of two k-slices
  auto read_frags = [&](int buf, int half) {
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2) {
      const int ks = 2 * half + s2;
#pragma unroll
      for (int j = 0; j < QI; ++j)
        fr[s2][j] = *reinterpret_cast<const u32x4*>(sR + buf * STAGE_BYTES + frag_r[ks] + j * 32 * BKB);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        fl[s2][j] = *reinterpret_cast<const u32x4*>(sL + buf * STAGE_BYTES + frag_l[ks] + j * 32 * BKB);
    }
  };
  const int one = 0x7f7f7f7f;  // E8M0 127 = 2^0 in every byte: hardware block scale off
  auto mfma_pair = [&]() {
#pragma unroll
    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
      for (int qi = 0; qi < QI; ++qi) {
        i32x8 a = {(int)fr[s2][qi].x, (int)fr[s2][qi].y, (int)fr[s2][qi].z, (int)fr[s2][qi].w, 0, 0, 0, 0};
#pragma unroll
        for (int pj = 0; pj < 4; ++pj) {
          i32x8 b = {(int)fl[s2][pj].x, (int)fl[s2][pj].y, (int)fl[s2][pj].z, (int)fl[s2][pj].w, 0, 0, 0, 0};
          acc[qi][pj] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc[qi][pj], 4, 4, 0, one, 0, one);
        }
      }
  };

  // The first stage of a tile is requested before the epilogue of the tile before it (for the
  // first tile: here), the second at the top of the tile; only the first has to have landed when
  // the main loop starts, the second is awaited inside it like every later one.
  tile_scalars(lid);
  tile_offsets();
  load_tile(0, 0, 0, NLD);
  while (true) {
  const int64_t eP0 = P0, eQ0 = Q0;   // this tile's origin, for its epilogue
  tile_offsets();
#pragma unroll
  for (int i = 0; i < QI; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
  load_tile(min(1, KT - 1), 1, 0, NLD);
  {
    // all but the 2 NLD loads just issued: stage 0 and, before it in issue order, whatever the
    // previous epilogue left in flight
    constexpr int n = 2 * NLD;
    static_assert(n < 64, "vmcnt field");
    __builtin_amdgcn_s_waitcnt(0x0f70 | (n & 15) | ((n >> 4) << 14));
  }
  // a bare barrier: the workgroup-wide fence of __syncthreads() would wait for the second stage too
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  read_frags(0, 0);

  // Ping-pong with two k-slices per phase: the two waves of a SIMD (wave w and w + 4) alternate
  // between a compute phase (16 MFMAs) and a memory phase (the 12 fragment reads of the next two
  // slices; once per K step the wave's share of the loads of the tile after next, into the
  // buffer whose last fragments everyone read two phases ago), half a period apart.
  const bool second_group = wave >= NWAVES / 2;
  if (second_group) __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  for (int kt = 0; kt < KT; ++kt) {
    const int cur = kt & 1;
    const int ktn2 = min(kt + 2, KT - 1);
    static_for<2>([&](auto hc) {
      constexpr int h = decltype(hc)::value;
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);
      mfma_pair();
#pragma unroll
      for (int qi = 0; qi < QI; ++qi)
        asm volatile("" : "+v"(acc[qi][0]), "+v"(acc[qi][1]), "+v"(acc[qi][2]), "+v"(acc[qi][3]));
      __builtin_amdgcn_s_setprio(0);
      __builtin_amdgcn_sched_barrier(0);
      // the next tile is first read in the memory phase h = 1; every wave's loads of it (issued
      // a K step ago) must have landed by the barrier before the first group's
      if constexpr (h == 1) {
        if (!second_group) __builtin_amdgcn_s_waitcnt(0x0f70);   // vmcnt(0)
      }
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (h == 0) {
        read_frags(cur, 1);
        if (second_group) __builtin_amdgcn_s_waitcnt(0x0f70);    // vmcnt(0): after the reads are issued
      } else {
        read_frags(cur ^ 1, 0);
        load_tile(ktn2, cur, 0, NLD);
      }
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
    });
  }
  if (!second_group) __builtin_amdgcn_s_barrier();
  __syncthreads();   // every wave is done with the operand buffers

  // the next tile's first stage travels while this tile's epilogue runs
  const int next = lid + wgs_per_xcd;
  const bool has_next = next < run_end;
  if (has_next) {
    tile_scalars(next);
    tile_offsets();
    load_tile(0, 0, 0, NLD);
  }

  // ---- epilogue --------------------------------------------------------------------------
  // Phase A (MFMA layout): scale by 1/gamma_l[p] (edge tiles: and by 1/gamma_r[q]) and park the
  // wave's tile, 32 rows at a time, in its own LDS region (behind the operands' stage 0, which
  // is being filled).  Phase B (row layout): each lane takes 8 consecutive columns of a row
  // (interior tiles: scales them by 1/gamma_r[q] here, the same product in the same order),
  // adds the addend, applies the DGE factor, converts and stores 16 / 32 contiguous bytes.
  float* const stage = reinterpret_cast<float*>(smem + EPI_BASE) + wave * EPI_ROWS * EPI_LD;
  constexpr int WCOLS = QI * 32;        // columns per wave
  constexpr int LPR = WCOLS / 8;        // lanes per row in phase B (8 columns each)
  constexpr int RPP = 64 / LPR;         // rows per pass
  static_assert(EPI_ROWS % RPP == 0, "passes per parked block");
  const bool scaled = gl != nullptr;
  // lane-derived values are rebuilt here from a copy of the lane id the optimizer cannot see
  // through: computed at kernel entry they would sit in registers across the main loop
  int ln = lane;
  asm volatile("" : "+v"(ln));
  const int el32 = ln & 31, elhi = ln >> 5;
  // Tiles that lie wholly inside the matrix take a branch-free epilogue.  What a wave reads from
  // memory here (addend, W for the DGE factor) and what it writes count on the same in-order
  // counter, so a load issued after a store is only usable once that store has completed: pass
  // by pass (load, add, store) the epilogue is a chain of sixteen memory round trips.  Instead
  // the scales are fetched up front and each pass's loads are issued a quarter ahead, before the
  // store of the pass whose registers they take over.
  constexpr bool FAST_OK = !DGE || W_BF16;
  constexpr int NP = EPI_ROWS / RPP;   // passes per parked block
  if (FAST_OK && eP0 + BM <= g.P && eQ0 + BN <= g.Q) {
    const int bcol = (ln % LPR) * 8;
    const int64_t q0 = eQ0 + wave_q * WCOLS + bcol;
    const int64_t prow = eP0 + wave_p * 128 + ln / LPR;
    float il4[4], ir8[8];
    [[maybe_unused]] float gw[8];
#pragma unroll
    for (int pj = 0; pj < 4; ++pj)
      il4[pj] = scaled ? __builtin_amdgcn_rcpf(gl[eP0 + wave_p * 128 + pj * 32 + el32]) : 1.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) ir8[e] = scaled ? __builtin_amdgcn_rcpf(gr[q0 + e]) : 1.0f;
    const float inv_k = DGE ? 1.0f / g.dge_k : 1.0f;
    const float pw = inv_k - 1.0f;
    if constexpr (DGE) {
#pragma unroll
      for (int e = 0; e < 8; ++e) gw[e] = gamma_w[q0 + e];
    }
    {
      // One body for both cases (two copies of it invite the optimizer to hoist what they share,
      // the scaling of all four quarters, above the branch between them).  The loads of a pass
      // are held in one set of registers: as soon as a pass of this quarter has taken its
      // values, the same pass of the next quarter is requested into them, ahead of this pass's
      // store.
      const bool HAS = addend != nullptr;
      [[maybe_unused]] f32x4 ad[NP][2];
      [[maybe_unused]] u32x4 wl[NP];
      auto issue = [&](int pj, int pass) {
        const int64_t p = prow + pj * EPI_ROWS + pass * RPP;
        if (HAS) {
          const float* a = addend + p * g.ldo + q0;
          ad[pass][0] = *reinterpret_cast<const f32x4*>(a);
          ad[pass][1] = *reinterpret_cast<const f32x4*>(a + 4);
        } else {   // defined on every path: an undefined value may be given a register for the whole tile loop
          ad[pass][0] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
          ad[pass][1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        }
        if constexpr (DGE)
          wl[pass] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(Wp) + p * g.ldw + q0);
      };
#pragma unroll
      for (int pass = 0; pass < NP; ++pass) issue(0, pass);
      __builtin_amdgcn_sched_barrier(0);
      static_for<4>([&](auto pc) {
        constexpr int pj = decltype(pc)::value;
        // the scheduler otherwise scales all four quarters up front, next to the raw accumulators
        __builtin_amdgcn_sched_barrier(0);
        static_for<4 * QI>([&](auto ic) {
          constexpr int qi = decltype(ic)::value / 4, g4 = decltype(ic)::value % 4;
          const f32x16& a16 = acc[qi][pj];
          f32x4 y;
          y.x = a16[g4 * 4 + 0] * il4[pj];
          y.y = a16[g4 * 4 + 1] * il4[pj];
          y.z = a16[g4 * 4 + 2] * il4[pj];
          y.w = a16[g4 * 4 + 3] * il4[pj];
          *reinterpret_cast<f32x4*>(stage + el32 * EPI_LD + qi * 32 + g4 * 8 + elhi * 4) = y;
        });
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_sched_barrier(0);
        static_for<NP>([&](auto sc) {
          constexpr int pass = decltype(sc)::value;
          const int rloc = pass * RPP + ln / LPR;
          const int64_t p = prow + pj * EPI_ROWS + pass * RPP;
          const f32x4 v0 = *reinterpret_cast<const f32x4*>(stage + rloc * EPI_LD + bcol);
          const f32x4 v1 = *reinterpret_cast<const f32x4*>(stage + rloc * EPI_LD + bcol + 4);
          float y[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
          for (int e = 0; e < 8; ++e) y[e] = __fmul_rn(y[e], ir8[e]);
          if (HAS) {
            const f32x4 a0 = ad[pass][0], a1 = ad[pass][1];
            y[0] += a0.x; y[1] += a0.y; y[2] += a0.z; y[3] += a0.w;
            y[4] += a1.x; y[5] += a1.y; y[6] += a1.z; y[7] += a1.w;
          }
          [[maybe_unused]] float w[8];
          if constexpr (DGE) {
            const u32x4 r = wl[pass];
            w[0] = u2f(r.x << 16); w[1] = u2f(r.x & 0xffff0000u);
            w[2] = u2f(r.y << 16); w[3] = u2f(r.y & 0xffff0000u);
            w[4] = u2f(r.z << 16); w[5] = u2f(r.z & 0xffff0000u);
            w[6] = u2f(r.w << 16); w[7] = u2f(r.w & 0xffff0000u);
          }
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (pj + 1 < 4) issue(pj + 1, pass);
          __builtin_amdgcn_sched_barrier(0);
          if constexpr (DGE) {
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] *= dge_factor(w[e], gw[e], pw, inv_k, g.dge_cap);
          }
          if constexpr (OUT_BF16) {
            u32x4 pk;
            pk.x = pack_bf16x2(y[0], y[1]);
            pk.y = pack_bf16x2(y[2], y[3]);
            pk.z = pack_bf16x2(y[4], y[5]);
            pk.w = pack_bf16x2(y[6], y[7]);
            *reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(outp) + p * g.ldo + q0) = pk;
          } else {
            float* o = reinterpret_cast<float*>(outp) + p * g.ldo + q0;
            const f32x4 o0 = {y[0], y[1], y[2], y[3]}, o1 = {y[4], y[5], y[6], y[7]};
            *reinterpret_cast<f32x4*>(o) = o0;
            *reinterpret_cast<f32x4*>(o + 4) = o1;
          }
        });
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
      });
    }
  } else {
    float ir[QI][4][4];
    if (scaled) {
#pragma unroll
      for (int qi = 0; qi < QI; ++qi)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int64_t q = min(eQ0 + wave_q * WCOLS + qi * 32 + g4 * 8 + elhi * 4 + e, g.Q - 1);
            ir[qi][g4][e] = __builtin_amdgcn_rcpf(gr[q]);
          }
    } else {
#pragma unroll
      for (int qi = 0; qi < QI; ++qi)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4)
#pragma unroll
          for (int e = 0; e < 4; ++e) ir[qi][g4][e] = 1.0f;
    }
    const int bcol = (ln % LPR) * 8;                    // phase B: this ln's 8 columns
    const int64_t q0 = eQ0 + wave_q * WCOLS + bcol;
    const bool q_full = q0 + 7 < g.Q;
    float gw[8];
    const float inv_k = DGE ? 1.0f / g.dge_k : 1.0f;
    const float pw = inv_k - 1.0f;
    if (DGE) {
#pragma unroll
      for (int e = 0; e < 8; ++e) gw[e] = gamma_w[min(q0 + e, g.Q - 1)];
    }
    static_for<4>([&](auto pc) {
      constexpr int pj = decltype(pc)::value;
      {
        const int64_t p = min(eP0 + wave_p * 128 + pj * 32 + el32, g.P - 1);
        float il = 1.0f;
        if (scaled) il = __builtin_amdgcn_rcpf(gl[p]);
        static_for<4 * QI>([&](auto ic) {
          constexpr int qi = decltype(ic)::value / 4, g4 = decltype(ic)::value % 4;
          f32x4 y;
          const f32x16& a16 = acc[qi][pj];
          y.x = a16[g4 * 4 + 0] * il * ir[qi][g4][0];
          y.y = a16[g4 * 4 + 1] * il * ir[qi][g4][1];
          y.z = a16[g4 * 4 + 2] * il * ir[qi][g4][2];
          y.w = a16[g4 * 4 + 3] * il * ir[qi][g4][3];
          *reinterpret_cast<f32x4*>(stage + el32 * EPI_LD + qi * 32 + g4 * 8 + elhi * 4) = y;
        });
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
#pragma unroll
      for (int pass = 0; pass < EPI_ROWS / RPP; ++pass) {
        const int rloc = pass * RPP + ln / LPR;
        const int64_t p = eP0 + wave_p * 128 + pj * EPI_ROWS + rloc;
        const f32x4 v0 = *reinterpret_cast<const f32x4*>(stage + rloc * EPI_LD + bcol);
        const f32x4 v1 = *reinterpret_cast<const f32x4*>(stage + rloc * EPI_LD + bcol + 4);
        float y[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
        if (p < g.P && q0 < g.Q) {
          if (addend) {
            const float* ad = addend + p * g.ldo + q0;
            if (q_full) {
              const f32x4 a0 = *reinterpret_cast<const f32x4*>(ad), a1 = *reinterpret_cast<const f32x4*>(ad + 4);
              y[0] += a0.x; y[1] += a0.y; y[2] += a0.z; y[3] += a0.w;
              y[4] += a1.x; y[5] += a1.y; y[6] += a1.z; y[7] += a1.w;
            } else {
#pragma unroll
              for (int e = 0; e < 8; ++e)
                if (q0 + e < g.Q) y[e] += ad[e];
            }
          }
          if (DGE) {
            float w[8];
            if (W_BF16) {
              const uint16_t* wp = reinterpret_cast<const uint16_t*>(Wp) + p * g.ldw + q0;
              if (q_full) {
                const u32x4 r = *reinterpret_cast<const u32x4*>(wp);
                w[0] = u2f(r.x << 16); w[1] = u2f(r.x & 0xffff0000u);
                w[2] = u2f(r.y << 16); w[3] = u2f(r.y & 0xffff0000u);
                w[4] = u2f(r.z << 16); w[5] = u2f(r.z & 0xffff0000u);
                w[6] = u2f(r.w << 16); w[7] = u2f(r.w & 0xffff0000u);
              } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) w[e] = q0 + e < g.Q ? bf16_bits_to_f32(wp[e]) : 0.0f;
              }
            } else {
              const float* wp = reinterpret_cast<const float*>(Wp) + p * g.ldw + q0;
#pragma unroll
              for (int e = 0; e < 8; ++e) w[e] = q0 + e < g.Q ? wp[e] : 0.0f;
            }
#pragma unroll
            for (int e = 0; e < 8; ++e) y[e] *= dge_factor(w[e], gw[e], pw, inv_k, g.dge_cap);
          }
          if (OUT_BF16) {
            uint16_t* o = reinterpret_cast<uint16_t*>(outp) + p * g.ldo + q0;
            if (q_full) {
              u32x4 pk;
              pk.x = pack_bf16x2(y[0], y[1]);
              pk.y = pack_bf16x2(y[2], y[3]);
              pk.z = pack_bf16x2(y[4], y[5]);
              pk.w = pack_bf16x2(y[6], y[7]);
              *reinterpret_cast<u32x4*>(o) = pk;
            } else {
#pragma unroll
              for (int e = 0; e < 8; ++e)
                if (q0 + e < g.Q) o[e] = (uint16_t)f32_to_bf16_bits(y[e]);
            }
          } else {
            float* o = reinterpret_cast<float*>(outp) + p * g.ldo + q0;
            if (q_full) {
              const f32x4 o0 = {y[0], y[1], y[2], y[3]}, o1 = {y[4], y[5], y[6], y[7]};
              *reinterpret_cast<f32x4*>(o) = o0;
              *reinterpret_cast<f32x4*>(o + 4) = o1;
            } else {
#pragma unroll
              for (int e = 0; e < 8; ++e)
                if (q0 + e < g.Q) o[e] = y[e];
            }
          }
        }
      }
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
    });
  }  // edge tiles
  __syncthreads();   // the staging regions overlap stage 1 of the operands, which the next tile fills first thing
  if (!has_next) break;
  lid = next;
  }  // tiles
}

// The scales of a thread's eight columns of a T x T tile, requested ahead of the main loop: fetched one by one behind it they were
// a chain of memory round trips.
template <int T, bool DGE>
FP4_D void column_scales(int64_t Q0, const float* gr, const float* gamma_w, const GemmShape& g, float (&ir)[8], float (&gw)[8]) {
  const int64_t q0 = Q0 + (int)(threadIdx.x % (T / 8)) * 8;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    ir[e] = 1.0f;
    gw[e] = 0.0f;
  }
  if (gr != nullptr) {
#pragma unroll
    for (int e = 0; e < 8; ++e) ir[e] = gr[min(q0 + e, g.Q - 1)];
  }
  if constexpr (DGE) {
#pragma unroll
    for (int e = 0; e < 8; ++e) gw[e] = gamma_w[min(q0 + e, g.Q - 1)];
  }
}
// What is left of a T x T tile of sums that lie in LDS scaled by 1/gamma_l: 1/gamma_r, addend, factor, conversion, stores
// along rows.  The same operations in the same order as in fp4_gemm_nt_kernel.  256 threads, the first 128 of them where T is 32.
template <int T, bool OUT_BF16, bool DGE, bool W_BF16>
FP4_D void finish_tile(const float* tile, int64_t P0, int64_t Q0, const float (&ir)[8], const float (&gw)[8], const float* addend,
                       void* outp, const void* Wp, const GemmShape& g) {
  constexpr int LD = T + 4;
  const int tid = threadIdx.x;
  constexpr int UPR = T / 8, RPT = (T == 32 ? 128 : 256) / UPR;   // 8-column units a row, rows a pass
  const int ql = (tid % UPR) * 8;
  const int64_t q0 = Q0 + ql;
  if (q0 >= g.Q) return;
  const bool full = q0 + 7 < g.Q;
  const float inv_k = DGE ? 1.0f / g.dge_k : 1.0f;
  const float pw = inv_k - 1.0f;
  if (full && P0 + T <= g.P) {   // no edge in this thread's part: what it reads is requested four passes at a time
    constexpr int NP = T / RPT, B = NP < 4 ? NP : 4;
#pragma unroll 1
    for (int b = 0; b < NP; b += B) {
      const int pl0 = tid / UPR + b * RPT;
      f32x4 ad[B][2];
      u32x4 w[B][2];
#pragma unroll
      for (int i = 0; i < B; ++i) {
        ad[i][0] = ad[i][1] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        w[i][0] = w[i][1] = u32x4{0u, 0u, 0u, 0u};
      }
      if (addend) {
#pragma unroll
        for (int i = 0; i < B; ++i) {
          const float* a = addend + (P0 + pl0 + i * RPT) * g.ldo + q0;
          ad[i][0] = *reinterpret_cast<const f32x4*>(a);
          ad[i][1] = *reinterpret_cast<const f32x4*>(a + 4);
        }
      }
      if constexpr (DGE) {
#pragma unroll
        for (int i = 0; i < B; ++i) {
          const int64_t off = (P0 + pl0 + i * RPT) * g.ldw + q0;
          if constexpr (W_BF16) {
            w[i][0] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(Wp) + off);
          } else {
            w[i][0] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const float*>(Wp) + off);
            w[i][1] = *reinterpret_cast<const u32x4*>(reinterpret_cast<const float*>(Wp) + off + 4);
          }
        }
      }
#pragma unroll
      for (int i = 0; i < B; ++i) {
        const int pl = pl0 + i * RPT;
        const f32x4 v0 = *reinterpret_cast<const f32x4*>(&tile[pl * LD + ql]), v1 = *reinterpret_cast<const f32x4*>(&tile[pl * LD + ql + 4]);
        float y[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
        for (int e = 0; e < 8; ++e) y[e] = __fmul_rn(y[e], ir[e]);
        if (addend) {
#pragma unroll
          for (int e = 0; e < 8; ++e) y[e] += ad[i][e >> 2][e & 3];
        }
        if constexpr (DGE) {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const uint32_t u = W_BF16 ? ((e & 1) ? w[i][0][e >> 1] & 0xffff0000u : w[i][0][e >> 1] << 16) : w[i][e >> 2][e & 3];
            y[e] *= dge_factor(u2f(u), gw[e], pw, inv_k, g.dge_cap);
          }
        }
        const int64_t off = (P0 + pl) * g.ldo + q0;
        if constexpr (OUT_BF16) {
          *reinterpret_cast<u32x4*>(reinterpret_cast<uint16_t*>(outp) + off) =
              u32x4{pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]), pack_bf16x2(y[4], y[5]), pack_bf16x2(y[6], y[7])};
        } else {
          float* o = reinterpret_cast<float*>(outp) + off;
          *reinterpret_cast<f32x4*>(o) = f32x4{y[0], y[1], y[2], y[3]};
          *reinterpret_cast<f32x4*>(o + 4) = f32x4{y[4], y[5], y[6], y[7]};
        }
      }
    }
    return;
  }
#pragma unroll 2
  for (int pl = tid / UPR; pl < T; pl += RPT) {
    const int64_t p = P0 + pl;
    if (p >= g.P) break;
    const f32x4 v0 = *reinterpret_cast<const f32x4*>(&tile[pl * LD + ql]), v1 = *reinterpret_cast<const f32x4*>(&tile[pl * LD + ql + 4]);
    float y[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = __fmul_rn(y[e], ir[e]);
    if (addend) {
      const float* ad = addend + p * g.ldo + q0;
      if (full) {
        const f32x4 a0 = *reinterpret_cast<const f32x4*>(ad), a1 = *reinterpret_cast<const f32x4*>(ad + 4);
        y[0] += a0.x; y[1] += a0.y; y[2] += a0.z; y[3] += a0.w;
        y[4] += a1.x; y[5] += a1.y; y[6] += a1.z; y[7] += a1.w;
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (q0 + e < g.Q) y[e] += ad[e];
      }
    }
    if constexpr (DGE) {
      float w[8];
      const int64_t off = p * g.ldw + q0;
#pragma unroll
      for (int e = 0; e < 8; ++e) w[e] = 0.0f;
      if (W_BF16 && full) {
        const u32x4 r = *reinterpret_cast<const u32x4*>(reinterpret_cast<const uint16_t*>(Wp) + off);
        w[0] = u2f(r.x << 16); w[1] = u2f(r.x & 0xffff0000u);
        w[2] = u2f(r.y << 16); w[3] = u2f(r.y & 0xffff0000u);
        w[4] = u2f(r.z << 16); w[5] = u2f(r.z & 0xffff0000u);
        w[6] = u2f(r.w << 16); w[7] = u2f(r.w & 0xffff0000u);
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (q0 + e < g.Q)
            w[e] = W_BF16 ? bf16_bits_to_f32(reinterpret_cast<const uint16_t*>(Wp)[off + e]) : reinterpret_cast<const float*>(Wp)[off + e];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) y[e] *= dge_factor(w[e], gw[e], pw, inv_k, g.dge_cap);
    }
    if constexpr (OUT_BF16) {
      uint16_t* o = reinterpret_cast<uint16_t*>(outp) + p * g.ldo + q0;
      if (full) {
        *reinterpret_cast<u32x4*>(o) = u32x4{pack_bf16x2(y[0], y[1]), pack_bf16x2(y[2], y[3]), pack_bf16x2(y[4], y[5]), pack_bf16x2(y[6], y[7])};
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (q0 + e < g.Q) o[e] = (uint16_t)f32_to_bf16_bits(y[e]);
      }
    } else {
      float* o = reinterpret_cast<float*>(outp) + p * g.ldo + q0;
      if (full) {
        *reinterpret_cast<f32x4*>(o) = f32x4{y[0], y[1], y[2], y[3]};
        *reinterpret_cast<f32x4*>(o + 4) = f32x4{y[4], y[5], y[6], y[7]};
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (q0 + e < g.Q) o[e] = y[e];
      }
    }
  }
}

// The same product for outputs with too few 256 x 256 tiles to go round the chip: a workgroup of four waves takes
// 64 x 64 outputs, a wave 32 x 32.  What bounds such a call is the chain of round trips of one tile, not a
// rate, so operands go straight from memory to the matrix core's registers (a lane's 16 bytes of a row are its
// fragment; a 128-byte line serves four steps out of L1), SG_IN steps ahead, and neither barrier nor staging stands
// in between.  The output passes through LDS once so that it is read and written along rows.  Sums, scaling, addend
// and factor are the same operations in the same order as in fp4_gemm_nt_kernel: the same bits.
// 512 x 512 x 256: 4.5 us, 6.3 with 128 x 128 tiles, 10.3 with 256 x 256; 1024 x 2048 x 288: 5.5 / 7.3 / 11.9.
constexpr int SG_IN = 4;   // K steps (32 bytes a row) requested ahead: one 128-byte line of every row
template <bool OUT_BF16, bool DGE, bool W_BF16>
__global__ __launch_bounds__(256) void fp4_gemm_small_kernel(
    const uint8_t* __restrict__ Lp, const uint8_t* __restrict__ Rp, const float* __restrict__ gl,
    const float* __restrict__ gr, const float* addend, void* outp, const void* __restrict__ Wp,
    const float* __restrict__ gamma_w, GemmShape g) {
  constexpr int T = 64, LD = T + 4;
  __shared__ __attribute__((aligned(16))) float tile[T * LD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, lhi = lane >> 5;
  const int wp = (wave & 1) * 32, wq = (wave >> 1) * 32;
  const int64_t P0 = (int64_t)(blockIdx.x % (unsigned)g.tiles_p) * T, Q0 = (int64_t)(blockIdx.x / (unsigned)g.tiles_p) * T;
  // rows past the edge re-read the last row
  const uint8_t* const rowL = Lp + min(P0 + wp + l32, g.P - 1) * g.Kb + lhi * 16;
  const uint8_t* const rowR = Rp + min(Q0 + wq + l32, g.Q - 1) * g.Kb + lhi * 16;
  float ir[8], gw[8], il = 1.0f;
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
  const int one = 127;
  u32x4 a[2][SG_IN], b[2][SG_IN];
  const u32x4 zero = {0u, 0u, 0u, 0u};
  auto request = [&](int set, int64_t k0) {   // steps from byte k0 on; what lies past the row is zero
#pragma unroll
    for (int s = 0; s < SG_IN; ++s) {
      const int64_t k = k0 + 32 * s;
      const bool in = k + lhi * 16 < g.Kb;
      a[set][s] = in ? *reinterpret_cast<const u32x4*>(rowR + k) : zero;
      b[set][s] = in ? *reinterpret_cast<const u32x4*>(rowL + k) : zero;
    }
  };
  auto multiply = [&](int set) {
#pragma unroll
    for (int s = 0; s < SG_IN; ++s) {
      const u32x4 fa = a[set][s], fb = b[set][s];
      const i32x8 va = {(int)fa.x, (int)fa.y, (int)fa.z, (int)fa.w, 0, 0, 0, 0};
      const i32x8 vb = {(int)fb.x, (int)fb.y, (int)fb.z, (int)fb.w, 0, 0, 0, 0};
      acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(va, vb, acc, 4, 4, 0, one, 0, one);
    }
  };
  request(0, 0);
  column_scales<T, DGE>(Q0, gr, gamma_w, g, ir, gw);
  if (gl != nullptr) il = gl[min(P0 + wp + l32, g.P - 1)];
  for (int64_t k0 = 0; k0 < g.Kb; k0 += 64 * SG_IN) {
    request(1, k0 + 32 * SG_IN);
    multiply(0);
    if (k0 + 32 * SG_IN < g.Kb) {
      request(0, k0 + 64 * SG_IN);
      multiply(1);
    }
  }
  il = __builtin_amdgcn_rcpf(il);
#pragma unroll
  for (int e = 0; e < 8; ++e) ir[e] = __builtin_amdgcn_rcpf(ir[e]);
#pragma unroll
  for (int g4 = 0; g4 < 4; ++g4) {
    const f32x4 y = {acc[g4 * 4] * il, acc[g4 * 4 + 1] * il, acc[g4 * 4 + 2] * il, acc[g4 * 4 + 3] * il};
    *reinterpret_cast<f32x4*>(&tile[(wp + l32) * LD + wq + g4 * 8 + lhi * 4]) = y;
  }
  __syncthreads();
  finish_tile<T, OUT_BF16, DGE, W_BF16>(tile, P0, Q0, ir, gw, addend, outp, Wp, g);
}

// The same for outputs in between: 128 x 128 a workgroup of four waves, a wave 64 x 64, one workgroup per CU.  A K step's
// products are over in a fifth of a microsecond, far less than a load takes, so operands go through a ring of four LDS
// stages with three on their way (the layout of fp4_gemm_nt_kernel's); one barrier a step.  A step takes 0.6 us, with 64
// workgroups as with 256: the 32 KiB it brings into a CU bound it (reading a step's fragments while the one before is
// multiplied changed nothing).  Sums, scaling and the rest as above: the same bits.
// 2048 x 2048 x 8192: 25.6 us, 46.9 with 256 x 256 tiles, 119 with 64 x 64; 2048^3 11.2 / 18.9 / 34.7; 1056 x 2080 x 1376
// 9.7 / 17.0 / 12.4; weight gradient with fp32 masters, 2048 x 2048 x 8192, quantizers included: 93 / 140 / 186.
constexpr int MG_T = 128, MG_RING = 4;
constexpr int MG_OP = MG_T * BKB, MG_STAGE = 2 * MG_OP, MG_LD = MG_T * 8 / 256;   // bytes of an operand, of a stage; 16-byte chunks a thread
template <bool OUT_BF16, bool DGE, bool W_BF16>
__global__ __launch_bounds__(256) void fp4_gemm_mid_kernel(
    const uint8_t* __restrict__ Lp, const uint8_t* __restrict__ Rp, const float* __restrict__ gl,
    const float* __restrict__ gr, const float* addend, void* outp, const void* __restrict__ Wp,
    const float* __restrict__ gamma_w, GemmShape g) {
  constexpr int T = MG_T, LD = T + 4;
  static_assert(MG_RING * MG_STAGE >= T * LD * 4, "the sums lie over the ring");
  __shared__ __attribute__((aligned(16))) uint8_t smem[MG_RING * MG_STAGE];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lhi = lane >> 5;
  const int wp = (wave & 1) * 64, wq = (wave >> 1) * 64;
  // each XCD a contiguous run of tiles: of the whole output, or (first > 0) the quarters of the 256 x 256 tiles from `first` on
  const int total = g.count, per_xcd = (total + 7) / 8;
  const int id = (int)(blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8);
  if ((int)(blockIdx.x / 8) >= per_xcd || id >= total) return;
  int tp, tq;
  if (g.first > 0) {
    tile_at(g, g.first + (id >> 2), tp, tq);
    tp = 2 * tp + (id & 1);
    tq = 2 * tq + (id >> 1 & 1);
  } else {
    tile_at(g, id, tp, tq);
  }
  const int64_t P0 = (int64_t)tp * T, Q0 = (int64_t)tq * T;
  if (P0 >= g.P || Q0 >= g.Q) return;   // a quarter behind the edge
  const __amdgpu_buffer_rsrc_t rsrcL = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(Lp) + P0 * g.Kb, 0, (int)(uint32_t)(min(g.P - P0, (int64_t)T) * g.Kb), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrcR = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(Rp) + Q0 * g.Kb, 0, (int)(uint32_t)(min(g.Q - Q0, (int64_t)T) * g.Kb), 0x00020000);
  const uint32_t Kb = (uint32_t)g.Kb;
  uint32_t offL[MG_LD], offR[MG_LD], at[MG_LD];   // a lane's chunk: from the tile's first row, and inside a step
#pragma unroll
  for (int j = 0; j < MG_LD; ++j) {
    const int row = 8 * (wave * MG_LD + j) + (lane >> 3);
    at[j] = (uint32_t)(((lane & 7) ^ ((row >> 1) & 7)) * 16);
    offL[j] = (uint32_t)min((int64_t)row, g.P - 1 - P0) * Kb + at[j];   // rows past the edge re-read the last row
    offR[j] = (uint32_t)min((int64_t)row, g.Q - 1 - Q0) * Kb + at[j];
  }
  auto request = [&](int kt) {   // what lies past the row, and steps past the last, arrive as zeros
    uint8_t* const st = smem + (kt & (MG_RING - 1)) * MG_STAGE + wave * MG_LD * 1024;
    const uint32_t k = (uint32_t)(kt * BKB);
#pragma unroll
    for (int j = 0; j < MG_LD; ++j) {
      const bool in = k + at[j] < Kb;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcL, (__attribute__((address_space(3))) void*)(st + j * 1024), 16,
                                               in ? offL[j] + k : OUT_OF_RANGE, 0, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcR, (__attribute__((address_space(3))) void*)(st + MG_OP + j * 1024), 16,
                                               in ? offR[j] + k : OUT_OF_RANGE, 0, 0, 0);
    }
  };
  float ir[8], gw[8], il[2] = {1.0f, 1.0f};
  const int KT = (int)((g.Kb + BKB - 1) / BKB);
  const int key = (l32 >> 1) & 7;
  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[i >> 1][i & 1][v] = 0.0f;
  const int one = 0x7f7f7f7f;
#pragma unroll
  for (int kt = 0; kt < MG_RING - 1; ++kt) request(kt);
  column_scales<T, DGE>(Q0, gr, gamma_w, g, ir, gw);
  if (gl != nullptr) {
#pragma unroll
    for (int pj = 0; pj < 2; ++pj) il[pj] = gl[min(P0 + wp + pj * 32 + l32, g.P - 1)];
  }
  for (int kt = 0; kt < KT; ++kt) {
    asm volatile("" ::: "memory");
    // this wave's share of step kt is there, and it is done reading step kt - 1; behind the barrier that holds for all
    constexpr int left = (MG_RING - 2) * 2 * MG_LD;
    __builtin_amdgcn_s_waitcnt(0x0070 | (left & 15) | ((left >> 4) << 14));
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    request(kt + MG_RING - 1);
    const uint8_t* const sL = smem + (kt & (MG_RING - 1)) * MG_STAGE + (wp + l32) * BKB;
    const uint8_t* const sR = smem + (kt & (MG_RING - 1)) * MG_STAGE + MG_OP + (wq + l32) * BKB;
    u32x4 fl[4][2], fr[4][2];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int slot = ((2 * ks + lhi) ^ key) * 16;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        fr[ks][j] = *reinterpret_cast<const u32x4*>(sR + slot + j * 32 * BKB);
        fl[ks][j] = *reinterpret_cast<const u32x4*>(sL + slot + j * 32 * BKB);
      }
    }
    __builtin_amdgcn_sched_barrier(0);   // all sixteen requested before the first product
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
#pragma unroll
      for (int qi = 0; qi < 2; ++qi) {
        const i32x8 a = {(int)fr[ks][qi].x, (int)fr[ks][qi].y, (int)fr[ks][qi].z, (int)fr[ks][qi].w, 0, 0, 0, 0};
#pragma unroll
        for (int pj = 0; pj < 2; ++pj) {
          const i32x8 b = {(int)fl[ks][pj].x, (int)fl[ks][pj].y, (int)fl[ks][pj].z, (int)fl[ks][pj].w, 0, 0, 0, 0};
          acc[qi][pj] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc[qi][pj], 4, 4, 0, one, 0, one);
        }
      }
  }
  __builtin_amdgcn_s_waitcnt(0);   // no load may land over the sums
  __syncthreads();
  float* const tile = reinterpret_cast<float*>(smem);
#pragma unroll
  for (int e = 0; e < 8; ++e) ir[e] = __builtin_amdgcn_rcpf(ir[e]);
#pragma unroll
  for (int pj = 0; pj < 2; ++pj) {
    const int p = wp + pj * 32 + l32;
    const float i1 = __builtin_amdgcn_rcpf(il[pj]);
#pragma unroll
    for (int qi = 0; qi < 2; ++qi)
#pragma unroll
      for (int g4 = 0; g4 < 4; ++g4) {
        const f32x16& c = acc[qi][pj];
        *reinterpret_cast<f32x4*>(&tile[p * LD + wq + qi * 32 + g4 * 8 + lhi * 4]) =
            f32x4{c[g4 * 4] * i1, c[g4 * 4 + 1] * i1, c[g4 * 4 + 2] * i1, c[g4 * 4 + 3] * i1};
      }
  }
  __syncthreads();
  finish_tile<T, OUT_BF16, DGE, W_BF16>(tile, P0, Q0, ir, gw, addend, outp, Wp, g);
}

// The same for the smallest outputs (a few tokens): 32 x 32 a workgroup, of which each of the four waves takes every fourth K step.  Such a
// call is one round trip to memory after another, so there are as many workgroups as can be and a wave has SP_RING steps of its own
// under way, which it stages, waits for and multiplies without any other; whole lines at a time (a lane of the 64 x 64 tiles reads 16 bytes
// of its row: 32 lines an instruction).  The waves' sums are multiples of 1/4 below 2^22 (the rule that takes these tiles sees to it), so added
// up they are the same bits as in one chain, and the rest is as above.
constexpr int SP_T = 32, SP_OP = SP_T * BKB, SP_STEP = 2 * SP_OP, SP_LD = SP_T / 8;   // SP_LD: 1 KiB requests an operand and step
static_assert(GEMM_EXACT_CODES / 2 * SP_T <= GEMM_OUT_OF_RANGE, "a tile's rows are within 32-bit offsets");
template <bool OUT_BF16, bool DGE, bool W_BF16, int RING>
__global__ __launch_bounds__(256) void fp4_gemm_split_kernel(
    const uint8_t* __restrict__ Lp, const uint8_t* __restrict__ Rp, const float* __restrict__ gl,
    const float* __restrict__ gr, const float* addend, void* outp, const void* __restrict__ Wp,
    const float* __restrict__ gamma_w, GemmShape g) {
  constexpr int T = SP_T, LD = T + 4, WAVES = 4;
  __shared__ __attribute__((aligned(16))) uint8_t smem[WAVES * RING * SP_STEP];
  static_assert(RING * SP_STEP >= T * LD * 4, "a wave's sums lie over its ring");
  auto part = [&](int w) { return reinterpret_cast<float*>(smem + w * (RING * SP_STEP)); };
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, lhi = lane >> 5;
  // each XCD a contiguous run of tiles, column by column: the rows of Rt are read by one of them
  const int total = g.count, per_xcd = (total + 7) / 8;
  const int id = (int)(blockIdx.x % 8) * per_xcd + (int)(blockIdx.x / 8);
  if ((int)(blockIdx.x / 8) >= per_xcd || id >= total) return;
  const int64_t P0 = (int64_t)(id % g.tiles_p) * T, Q0 = (int64_t)(id / g.tiles_p) * T;
  const __amdgpu_buffer_rsrc_t rsrcL = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(Lp) + P0 * g.Kb, 0, (int)(uint32_t)(min(g.P - P0, (int64_t)T) * g.Kb), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsrcR = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<uint8_t*>(Rp) + Q0 * g.Kb, 0, (int)(uint32_t)(min(g.Q - Q0, (int64_t)T) * g.Kb), 0x00020000);
  const uint32_t Kb = (uint32_t)g.Kb;
  uint32_t offL[SP_LD], offR[SP_LD], at[SP_LD];
#pragma unroll
  for (int j = 0; j < SP_LD; ++j) {
    const int row = 8 * j + (lane >> 3);
    at[j] = (uint32_t)(((lane & 7) ^ ((row >> 1) & 7)) * 16);
    offL[j] = (uint32_t)min((int64_t)row, g.P - 1 - P0) * Kb + at[j];   // rows past the edge re-read the last row
    offR[j] = (uint32_t)min((int64_t)row, g.Q - 1 - Q0) * Kb + at[j];
  }
  uint8_t* const mine = smem + wave * (RING * SP_STEP);
  const int KT = (int)((g.Kb + BKB - 1) / BKB), steps = (KT - wave + WAVES - 1) / WAVES;   // of this wave
  auto request = [&](int i) {   // what lies past the row, and steps past the last, arrive as zeros
    uint8_t* const st = mine + (i % RING) * SP_STEP;
    const uint32_t k = (uint32_t)((wave + WAVES * i) * BKB);
#pragma unroll
    for (int j = 0; j < SP_LD; ++j) {
      const bool in = i < steps && k + at[j] < Kb;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcL, (__attribute__((address_space(3))) void*)(st + j * 1024), 16,
                                               in ? offL[j] + k : OUT_OF_RANGE, 0, 0, 0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrcR, (__attribute__((address_space(3))) void*)(st + SP_OP + j * 1024), 16,
                                               in ? offR[j] + k : OUT_OF_RANGE, 0, 0, 0);
    }
  };
  const int key = (l32 >> 1) & 7;
  f32x16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
  const int one = 0x7f7f7f7f;
#pragma unroll
  for (int i = 0; i < RING; ++i) request(i);
  float ir[8], gw[8], il = 1.0f;
  column_scales<T, DGE>(Q0, gr, gamma_w, g, ir, gw);
  if (gl != nullptr) il = gl[min(P0 + (tid >> 3), g.P - 1)];
  for (int i = 0; i < steps; ++i) {
    asm volatile("" ::: "memory");
    constexpr int left = (RING - 1) * 2 * SP_LD;   // the steps behind this one
    __builtin_amdgcn_s_waitcnt(0x0070 | (left & 15) | ((left >> 4) << 14));
    asm volatile("" ::: "memory");
    const uint8_t* const sL = mine + (i % RING) * SP_STEP + l32 * BKB;
    u32x4 fl[4], fr[4];
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const int slot = ((2 * ks + lhi) ^ key) * 16;
      fr[ks] = *reinterpret_cast<const u32x4*>(sL + SP_OP + slot);
      fl[ks] = *reinterpret_cast<const u32x4*>(sL + slot);
    }
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // read: the slot may be filled again
    request(i + RING);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      const i32x8 a = {(int)fr[ks].x, (int)fr[ks].y, (int)fr[ks].z, (int)fr[ks].w, 0, 0, 0, 0};
      const i32x8 b = {(int)fl[ks].x, (int)fl[ks].y, (int)fl[ks].z, (int)fl[ks].w, 0, 0, 0, 0};
      acc = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, acc, 4, 4, 0, one, 0, one);
    }
  }
  __builtin_amdgcn_s_waitcnt(0);   // no load may land over the sums
#pragma unroll
  for (int g4 = 0; g4 < 4; ++g4)
    *reinterpret_cast<f32x4*>(&part(wave)[l32 * LD + g4 * 8 + lhi * 4]) = f32x4{acc[g4 * 4], acc[g4 * 4 + 1], acc[g4 * 4 + 2], acc[g4 * 4 + 3]};
  __syncthreads();
  {   // four columns of a row a thread
    const int o = (tid >> 3) * LD + (tid & 7) * 4;
    f32x4 sum = *reinterpret_cast<const f32x4*>(&part(0)[o]);
#pragma unroll
    for (int w = 1; w < WAVES; ++w) {
      const f32x4 v = *reinterpret_cast<const f32x4*>(&part(w)[o]);
#pragma unroll
      for (int e = 0; e < 4; ++e) sum[e] += v[e];
    }
    const float i1 = __builtin_amdgcn_rcpf(il);
#pragma unroll
    for (int e = 0; e < 4; ++e) sum[e] = __fmul_rn(sum[e], i1);
    *reinterpret_cast<f32x4*>(&part(0)[o]) = sum;
  }
  __syncthreads();
  if (tid >= 128) return;
#pragma unroll
  for (int e = 0; e < 8; ++e) ir[e] = __builtin_amdgcn_rcpf(ir[e]);
  finish_tile<T, OUT_BF16, DGE, W_BF16>(part(0), P0, Q0, ir, gw, addend, outp, Wp, g);
}

__global__ void fp4_unpack_kernel(const uint8_t* codes, int64_t nbytes, uint8_t* out) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < nbytes) {
    uint8_t b = codes[i];
    out[2 * i] = b & 15;
    out[2 * i + 1] = b >> 4;
  }
}

}  // namespace

// Compute units of the device the launch goes to (here one persistent workgroup each).  Looked up once
// per device; concurrent first calls write the same value.
int fp4_compute_units_of_current_device() {
  static int cached[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  int n = cached[dev];
  if (n == 0) {
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 8) n = 256;
    cached[dev] = n;
  }
  return n;
}

// Internal launcher shared by fp4_gemm and the layer entry points.
int fp4_trace_open(int kind, hipStream_t stream);
void fp4_trace_close(int slot, hipStream_t stream);

int fp4_launch_gemm(const uint8_t* L, const float* gl, const uint8_t* Rt, const float* gr,
                    int64_t P, int64_t Q, int64_t Kc, const float* addend, void* out, int out_bf16,
                    int64_t ldo, const void* W, int w_bf16, int64_t ldw, const float* gamma_w,
                    float dge_k, float dge_cap, hipStream_t stream) {
  if (P == 0 || Q == 0) return FP4_OK;
  GemmShape g;
  g.P = P; g.Q = Q; g.Kb = Kc / 2; g.ldo = ldo; g.ldw = ldw;
  g.dge_k = dge_k; g.dge_cap = dge_cap;
  g.tiles_p = (int)((P + BM - 1) / BM);
  g.tiles_q = (int)((Q + BN - 1) / BN);
  const bool dge = W != nullptr && dge_k > 0.0f;
  const int n_cu = fp4_compute_units_of_current_device();
  const GemmTiling t = gemm_tiling(P, Q, Kc, dge, w_bf16 != 0, addend != nullptr, out_bf16 != 0, n_cu);
  const int trace_slot = fp4_trace_open(FP4_TRACE_GEMM, stream);
  const bool ragged = (g.Kb % BKB) != 0, split = t.tile == 32, small = t.tile == 64, mid = t.tile == 128;
  GemmShape gt = g;
  gt.tiles_p = (int)((P + SP_T - 1) / SP_T);
  gt.tiles_q = (int)((Q + SP_T - 1) / SP_T);
  gt.count = gt.tiles_p * gt.tiles_q;
  const int total = g.tiles_p * g.tiles_q - t.rest;
  g.first = 0;
  g.count = total;
  g.stagger = t.stagger;
  const dim3 grid(std::min((total + 7) / 8 * 8, (n_cu / 8) * 8)), block(NTHREADS);
  GemmShape gs = g, gm = g;
  gs.tiles_p = (int)((P + 63) / 64);
  gm.tiles_p = (int)((P + MG_T - 1) / MG_T);
  gm.tiles_q = (int)((Q + MG_T - 1) / MG_T);
  gm.count = gm.tiles_p * gm.tiles_q;
  if (t.rest) {   // the order of the 256 x 256 tiles
    gm = g;
    gm.first = total;
    gm.count = 4 * t.rest;
  }
#define FP4_GEMM_LAUNCH(OB, DG, WB)                                                                       \
  do {                                                                                                    \
    if (split) {                                                                                          \
      if (gt.count <= n_cu)                                                                               \
        hipLaunchKernelGGL((fp4_gemm_split_kernel<OB, DG, WB, 4>), dim3((unsigned)((gt.count + 7) / 8 * 8)), dim3(256), 0, stream, L, Rt, \
                           gl, gr, addend, out, W, gamma_w, gt);                                          \
      else                                                                                                \
        hipLaunchKernelGGL((fp4_gemm_split_kernel<OB, DG, WB, 2>), dim3((unsigned)((gt.count + 7) / 8 * 8)), dim3(256), 0, stream, L, Rt, \
                         gl, gr, addend, out, W, gamma_w, gt);                                            \
      break;                                                                                              \
    }                                                                                                     \
    if (small)                                                                                            \
      hipLaunchKernelGGL((fp4_gemm_small_kernel<OB, DG, WB>), dim3((unsigned)(((P + 63) / 64) * ((Q + 63) / 64))), dim3(256), 0, stream, L, Rt, gl, gr, \
                         addend, out, W, gamma_w, gs);                                                    \
    else if (mid)                                                                                         \
      ;                                                                                                   \
    else if (ragged)                                                                                      \
      hipLaunchKernelGGL((fp4_gemm_nt_kernel<OB, DG, WB, true>), grid, block, 0, stream, L, Rt, gl, gr,   \
                         addend, out, W, gamma_w, g);                                                     \
    else                                                                                                  \
      hipLaunchKernelGGL((fp4_gemm_nt_kernel<OB, DG, WB, false>), grid, block, 0, stream, L, Rt, gl, gr,  \
                         addend, out, W, gamma_w, g);                                                     \
    if (!small && (mid || t.rest))                                                                        \
      hipLaunchKernelGGL((fp4_gemm_mid_kernel<OB, DG, WB>), dim3((unsigned)((gm.count + 7) / 8 * 8)), dim3(256), 0, stream, L, Rt, \
                         gl, gr, addend, out, W, gamma_w, gm);                                            \
  } while (0)
  if (dge) {
    if (w_bf16) FP4_GEMM_LAUNCH(false, true, true);
    else FP4_GEMM_LAUNCH(false, true, false);
  } else if (out_bf16) {
    FP4_GEMM_LAUNCH(true, false, false);
  } else {
    FP4_GEMM_LAUNCH(false, false, false);
  }
#undef FP4_GEMM_LAUNCH
  fp4_trace_close(trace_slot, stream);
  FP4_CHECK_LAUNCH();
  return FP4_OK;
}

extern "C" int fp4_gemm(const uint8_t* codes_l, const float* gamma_l, const uint8_t* codes_rt,
                        const float* gamma_r, int64_t P, int64_t Q, int64_t Kc, const float* addend,
                        void* out, fp4_dtype out_dt, int64_t ldo, void* stream) {
  if (P < 0 || Q < 0 || Kc < 0 || (Kc % 32) != 0 || ldo < Q) return FP4_ERR_SHAPE;
  if (out_dt != FP4_F32 && out_dt != FP4_BF16) return FP4_ERR_DTYPE;
  if (P == 0 || Q == 0) return FP4_OK;
  if (!out || (Kc > 0 && (!codes_l || !codes_rt))) return FP4_ERR_NULL;
  if ((gamma_l == nullptr) != (gamma_r == nullptr)) return FP4_ERR_NULL;
  if (!gamma_l && out_dt != FP4_F32) return FP4_ERR_DTYPE;
  if (!aligned16(codes_l) || !aligned16(codes_rt) || !aligned16(out) || (ldo % 8) != 0 ||
      (addend && !aligned16(addend)))
    return FP4_ERR_ARG;
  return fp4_launch_gemm(codes_l, gamma_l, codes_rt, gamma_r, P, Q, Kc, addend, out,
                         out_dt == FP4_BF16, ldo, nullptr, 0, 0, nullptr, 0.0f, 0.0f,
                         (hipStream_t)stream);
}

extern "C" int fp4_gemm_tiling(int64_t P, int64_t Q, int64_t Kc, int factor, int w_bf16, int addend, int out_bf16, int compute_units,
                               int* last_round, int* stagger) {
  if (P <= 0 || Q <= 0 || Kc < 0 || (Kc % 32) != 0 || compute_units < 8) return FP4_ERR_SHAPE;
  const GemmTiling t = gemm_tiling(P, Q, Kc, factor != 0, w_bf16 != 0, addend != 0, out_bf16 != 0, compute_units);
  if (last_round) *last_round = t.rest;
  if (stagger) *stagger = t.stagger;
  return t.tile;
}

extern "C" int fp4_gemm_splits(int64_t P, int64_t Q, int64_t Kc, int factor, int compute_units) {
  if (P <= 0 || Q <= 0 || Kc < 0 || (Kc % 32) != 0 || compute_units < 8) return FP4_ERR_SHAPE;
  return gemm_tiling(P, Q, Kc, factor != 0, false, false, false, compute_units).tile == 32;
}

extern "C" int fp4_unpack(const uint8_t* codes, int64_t rows, int64_t cols, uint8_t* one_per_byte,
                          void* stream) {
  if (rows < 0 || cols < 0 || (cols & 1)) return FP4_ERR_SHAPE;
  int64_t nbytes = rows * (cols / 2);
  if (nbytes == 0) return FP4_OK;
  if (!codes || !one_per_byte) return FP4_ERR_NULL;
  hipLaunchKernelGGL(fp4_unpack_kernel, dim3((unsigned)((nbytes + 255) / 256)), dim3(256), 0,
                     (hipStream_t)stream, codes, nbytes, one_per_byte);
  FP4_CHECK_LAUNCH();
  return FP4_OK;
}
