/*
 * fp4_measure.h -- measurement and self-check helpers of libfp4mi.so, kept apart from the
 * product ABI (fp4_linear.h): the library's own rounding routine exposed for exhaustive
 * checks, ceilings of the part the rooflines are read against, and a timer of the
 * GEMM launches and residual products.  Nothing here is on the hot path.  Status codes are fp4_status.
 */
#ifndef FP4_MEASURE_H
#define FP4_MEASURE_H

#include "fp4_linear.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Host-side evaluation of the library's own rounding routine: codes[i] = Q(x[i]) for
 * n fp32 values in HOST memory (the same inline function the kernels use, compiled for
 * the CPU; lets the rounding be checked exhaustively without a GPU). */
int fp4_host_round_codes(const float* x_host, int64_t n, uint8_t* codes_host);
/* The same for the E4M3 rounding of the mixed-format path. */
int fp8_host_round_codes(const float* x_host, int64_t n, uint8_t* codes_host);

/* The rounding as the quantization kernels perform it on the device (App. A's rule carried out
 * by the FP4 convert instruction, eight values per packed word): codes[i] = Q(x[i]), one code per
 * byte, x and codes in DEVICE memory, n a multiple of 8.
 * fp4_device_round_sweep: runs every one of the 2^32 fp32 bit patterns, in each of the eight
 * positions of a packed word, through that routine and through the comparison chain that
 * fp4_host_round_codes exposes, and ADDS the number of disagreements to *mismatches (device
 * memory, 8 bytes, set it to 0 first).  About a second of GPU time. */
int fp4_device_round_codes(const float* x, int64_t n, uint8_t* codes, void* stream);
int fp4_device_round_sweep(unsigned long long* mismatches, void* stream);

/* Output tiles the FP4 GEMM [P x Q], contraction Kc, is cut into on a device with that many compute units, by the rule its launches
 * follow (host arithmetic, no GPU): 32 (whose waves share a contraction), 64, 128 or 256 rows and columns.  With 256, *last_round is the number of tiles of the
 * last round that are cut into 128 x 128 ones and *stagger how much later than the one before each quarter of the workgroups
 * begins, in 512 cycles; otherwise 0 (either may be NULL).  factor: the weight gradient's derivative factor
 * with weights in bf16 (w_bf16) or fp32; addend: whether there is one; out_bf16: the output's type. */
int fp4_gemm_tiling(int64_t P, int64_t Q, int64_t Kc, int factor, int w_bf16, int addend, int out_bf16, int compute_units,
                    int* last_round, int* stagger);

/* Whether those are 32 (1) or not (0): neither types nor an addend matter for it (host arithmetic, no GPU). */
int fp4_gemm_splits(int64_t P, int64_t Q, int64_t Kc, int factor, int compute_units);

/* Whether the tiles of one tensor's column-wise quantization form their scales themselves (1) or a launch before them does (0)
 * (host arithmetic, no GPU). */
int fp4_quantize_cols_folds(int64_t rows, int64_t cols);

/* Which passes find the thresholds of a [rows x cols] tensor and count its rows' outliers (host arithmetic, no GPU). */
#define FP4_SELECT_WINDOWS 1   /* one pass over the elements with bins for the keys around the thresholds, otherwise digit passes alone */
#define FP4_SELECT_SAMPLE 2    /* the windows lie where a sample says, otherwise where a first digit pass does */
#define FP4_SELECT_FOUND 4     /* the thresholds are found in a launch of their own, otherwise by every workgroup that counts */
#define FP4_SELECT_APART 8     /* rows are counted each by itself, without sums of blocks of them */
int fp4_select_route(int64_t rows, int64_t cols, int64_t ld, fp4_dtype dt);

/* What a layer's launches on a device with that many compute units do beside their own work (host arithmetic, no GPU).
 * fp4_select_beside: the first digit pass over A goes with the column-wise codes of W (forward pass, per-tensor thresholds, W not cached);
 * fp4_transpose_beside: the last pass of the residual's transposition with the codes of the weight gradient's operands; both tell how many
 * tiles of 64 columns a workgroup then has (1, 2 or 4), or 0: in launches of their own.  fp4_count_beside: the transposition's first pass, of
 * a residual of at most capacity entries, goes with the launch that begins fp4_linear_bwd (1) or is one of its own (0). */
int fp4_select_beside(int64_t M, int64_t K, int64_t N, fp4_dtype dt, int compute_units);
int fp4_transpose_beside(int64_t M, int64_t K, int64_t N, int compute_units);
int fp4_count_beside(int64_t M, int64_t K, int64_t N, fp4_dtype dt, int cached, int64_t capacity, int compute_units);

/* The transpose that a weight gradient takes of its residual [P x Q]: CSR of [Q x P], indices ascending in every row.  positions: where
 * the entries' places come from, 1: counts of all row blocks, added up where they are needed, 2: a scan of them over the blocks,
 * 3: as 2 and a scan over the columns, or 0: as the sizes have it, which fp4_residual_transpose_positions tells (host arithmetic, no
 * GPU; 0 where there are more than 16384 columns and none of these is used).  1 and 2 need Q % 4 == 0 and P Q < 2^32.  At most
 * fp4_occ_capacity(P, Q, 0.9) entries.  Workspace: fp4_workspace_bytes(FP4_OP_WGRAD, P, Q, 32, FP4_F32). */
int fp4_residual_transpose_positions(int64_t P, int64_t Q);
int fp4_residual_transpose(const int64_t* row_ptr, const int32_t* col_idx, const float* val, const int64_t* nnz, int64_t P, int64_t Q,
                           int64_t capacity, int positions, int64_t* t_ptr, int32_t* t_idx, float* t_val, void* workspace,
                           size_t workspace_bytes, void* stream);

/* Whether a residual product S [P x Q] D [Q x N] of at most so many entries is one launch that gathers rows of D (1) or goes to the
 * kernels of large products (0), by the rule the launches follow (host arithmetic, no GPU). */
int fp4_residual_spmm_gathers(int64_t P, int64_t Q, int64_t N, fp4_dtype dt, int64_t entries);

/* fp4_residual_spmm by the kernels that large products take, whatever the size: same arguments, workspace and result (sums in
 * another order). */
int fp4_residual_spmm_general(const int64_t* row_ptr, const int32_t* col_idx, const float* val, int64_t P, int64_t Q, const void* D,
                              fp4_dtype dt, int64_t N, float* R, void* workspace, size_t workspace_bytes, void* stream);

/* ---- ceilings measured on the part (for reading the rooflines; not part of the method) ----
 * fp4_probe_mfma: `workgroups` workgroups of 8 waves each run `iters` iterations of 8 FP4
 *   32x32x64 MFMAs per wave with operands taken from operand_bytes (device, >= 16 bytes): an
 *   issue loop without memory traffic.  FLOP = workgroups * 8 * iters * 8 * 131072.  The rate
 *   depends on the operand data (random codes draw more power than constant ones).
 *   sink: device, workgroups * 512 floats.
 * fp4_probe_copy: dst[0..nbytes) = src[0..nbytes), 16 bytes per lane (streaming copy). */
int fp4_probe_mfma(const void* operand_bytes, int64_t nbytes, int workgroups, int iters, float* sink,
                   void* stream);
int fp4_probe_copy(const void* src, void* dst, int64_t nbytes, void* stream);

/* ---- measurement helper (host-side state, off by default; not thread-safe) ----
 * Between fp4_trace_begin(n) and fp4_trace_end() every FP4 GEMM launch and every residual product
 * (all of its launches together: packing, multiplication, long rows), from any entry point, is
 * bracketed by a pair of HIP events recorded on the call's own stream (at most n; later ones are
 * not recorded).
 * fp4_trace_end waits for the recorded launches, writes their durations in milliseconds and their
 * kinds, in launch order, to ms_host / kind_host [0..capacity) (HOST memory) and returns the number
 * of launches recorded (>= 0) or a negative fp4_status. */
enum { FP4_TRACE_GEMM = 0, FP4_TRACE_SPMM = 1 };
int fp4_trace_begin(int max_launches);
int fp4_trace_end(float* ms_host, int* kind_host, int capacity);

#ifdef __cplusplus
}
#endif
#endif /* FP4_MEASURE_H */
