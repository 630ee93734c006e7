// Launchers of the gfx950 kernels (defined in ata_kernels.hip).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "ata_plan.h"

namespace atalib {

// Task tables of one plan in device memory.
struct DevTables {
    const DevTask* tasks;
    const DevTerm* terms;
    const int32_t* segs;
};

// Classical tiles (TK_SYRK / TK_GEMM) on FP64 or FP32 MFMA.  out_f64 selects
// a double C for float input.
// Aops: base of the operand-sum buffers read by tasks with src == 1.
hipError_t launch_gemm(bool f32, bool out_f64, const void* A, int64_t lda, const DevTables& tb,
                       const WorkItem* items, int nitems, void* C, double* W, hipStream_t s,
                       const void* Aops = nullptr);

// lower(A^t A) of K rows and n columns (packed C, beta 1 accumulates) on
// tb x tb tiles (64 or 32), the rows in `parts` parts of `rows` rows; more
// than one part writes FP64 partial tiles to `part` (tiles x parts x tb^2
// doubles) and sums them in a second launch.  by_rows: lower(A A^t) of n rows
// of K elements (64 rows below 2^31 bytes).
hipError_t launch_fine(bool f32, bool out_f64, int tb, const void* A, int64_t lda, int K, int n, int parts, int rows,
                       void* C, int beta, double* part, hipStream_t s, bool by_rows = false);

// FP64 tiles on 16-byte direct-to-LDS copies: nt = 1 for classical tiles
// (TK_SYRK / TK_GEMM, and products on operand-sum buffers through Aops),
// nt = 2 for Strassen product tiles with at most two terms per operand (and
// the classical tiles launched with them).  queue (nt = 2): kTileQueues ints
// of device memory, cleared by the launch, which then runs persistent
// workgroups taking the items from per-XCD work queues; null: one workgroup
// per item.
hipError_t launch_tile(int nt, const double* A, int64_t lda, const DevTables& tb, const WorkItem* items, int nitems,
                       double* C, double* W, hipStream_t s, const double* Aops = nullptr, int* queue = nullptr);

// Transposed converted copy of the reduced-precision forms: plane 0 (bfloat16
// hi, or e4m3), plane 1 (bfloat16 lo), row stride in elements, e4m3 scales.
struct LpCopy {
    const void* t0;
    const void* t1;
    int ldt;
    const float* scale;
};
// Reduced-precision classical tiles whose windows lie on 16 bytes of the copy
// (64 rows of it below 2^31 bytes), items of kWideRows x wide_cols(mode) tiles
// (wide) or 128 x 128 ones: nmain whole tiles and ntail parts of K-split tiles
// (slot = tile * nparts + part), whose results go to `part` (one tile of FP64
// values, e4m3 FP32, per slot) and are summed into C by a second launch.
hipError_t launch_lp_tile16(int mode, bool out_f64, bool wide, const LpCopy& cp, const DevTables& tb,
                            const WorkItem* items, int nmain, const WorkItem* tail, int ntail, int nparts, void* part,
                            void* C, double* W, hipStream_t s);

// The same for a launch of k_gemmd tiles (FP32, or FP64 batched/operand-sum
// launches); C of the launch's output type.
hipError_t launch_gemm_split(bool f32, bool out_f64, const void* A, int64_t lda, const DevTables& tb,
                             const WorkItem* tail, int ntail, int nparts, double* part, void* C, double* W,
                             hipStream_t s, const void* Aops = nullptr);

// The same for the reduced-precision classical tiles (partials de-scaled).
hipError_t launch_gemm_lp_split(int mode, bool out_f64, const void* T0, const void* T1, int ldt, const float* scale,
                                const DevTables& tb, const WorkItem* tail, int ntail, int nparts, double* part,
                                void* C, double* W, hipStream_t s, int align);

// A one-term FP64 tile launch with its K-split last round in the same grid
// (the parts run as the whole tiles finish), then the sum of the parts.
hipError_t launch_tile_cat(const double* A, int64_t lda, const DevTables& tb, const WorkItem* items, int nmain,
                           const WorkItem* tail, int ntail, int nparts, double* part, double* C, double* W,
                           hipStream_t s, const double* Aops);

// Operand sums of the product tasks in `recs` (one workgroup per buffer row;
// rows = total rows of the records) into `out`, in the input type.
hipError_t launch_opsum(bool f32, const void* A, int64_t lda, const DevTables& tb, const DevOpSum* recs, int nrec,
                        int64_t rows, void* out, hipStream_t s);

// Strassen product tiles: classical tiles whose operands are signed sums of
// up to tmax terms (column padding reads as zero), written to the workspace.
hipError_t launch_gemm_terms(bool f32, bool out_f64, int tmax, const void* A, int64_t lda, const DevTables& tb,
                             const WorkItem* items, int nitems, void* C, double* W, hipStream_t s);

// Classical tiles of several requests in one launch: work item w uses
// batch[w.slot] for its matrices and tables.
hipError_t launch_gemm_batch(bool f32, bool out_f64, const BatchEntry* batch, const WorkItem* items, int nitems,
                             hipStream_t s);

// Fill count elements with i.i.d. standard normal values drawn from
// (seed, element index) by Philox4x32-10 and the Box-Muller transform.
hipError_t launch_fill_normal(void* p, int64_t count, uint64_t seed, bool f64, hipStream_t s);

// In-tile Strassen tiles (TK_STR).  tmax: most operand terms of any task.
hipError_t launch_str(bool f32, bool out_f64, int variant, int tmax, const void* A, int64_t lda,
                      const DevTables& tb, const WorkItem* items, int nitems, void* C, double* W,
                      hipStream_t s);

// Workspace combinations (FP64 workspace) into packed C.
hipError_t launch_combine(bool out_f64, const DevCombine* cbs, int ncb, int64_t total, const double* W,
                          void* C, hipStream_t s);

hipError_t launch_fill_zero(void* p, int64_t count, int elem_bytes, hipStream_t s);

// Reduced-precision forms.  The prepass writes A^t (columns of A as rows,
// rows of A along the contiguous axis, padded with zeros to ldt) converted
// to bfloat16 hi/lo planes (mode 0) or to scaled OCP e4m3 (mode 1).
// For mode 1 the per-column power-of-two scales are computed first from the
// column maxima (partial maxima per 256-row chunk in `part`).
hipError_t launch_colscale(const float* A, int64_t lda, int m, int n, float* part, float* scale,
                           hipStream_t s);
hipError_t launch_prep_lp(int mode, const float* A, int64_t lda, int m, int n, int ldt, const float* scale,
                          void* out0, void* out1, hipStream_t s);
// Strassen operands of the reduced-precision forms: the operand sums of the
// records (FP32, term order) converted into rows of the operand copy (mode 0
// bfloat16 hi/lo planes, mode 1 scaled e4m3 with per-row scales; colmax holds
// `rows` words of scratch for mode 1).  tiles: 64 x 64 conversion tiles of
// all records.
hipError_t launch_opsum_lp(int mode, const float* A, int64_t lda, const DevTables& tb, const DevOpSum* recs, int nrec,
                           int64_t tiles, int64_t rows, uint32_t* colmax, float* scale, void* out0, void* out1, int ldt,
                           hipStream_t s);
// align: 2 when every segment window of the plan starts and ends on 16
// bytes of the copy (or ends at its last row, past which the copy holds
// zeros), 1 when on dwords, else 0 (see lp_windows_aligned): the tiles stage
// through 16-byte or dword direct-to-LDS copies, or through registers.
hipError_t launch_gemm_lp(int mode, bool out_f64, const void* T0, const void* T1, int ldt,
                          const float* scale, const DevTables& tb, const WorkItem* items, int nitems,
                          void* C, double* W, hipStream_t s, int align);

// Column equilibration (power-of-two column scales into `scale`, the scaled
// copy of A into `out` with row stride n; `part` holds ceil(m/256) x n
// partial maxima) and its inverse on packed lower C.
hipError_t launch_equilibrate(bool f32, const void* A, int64_t lda, int m, int n, void* part, void* scale, void* out,
                              hipStream_t s);
hipError_t launch_descale(bool f32, bool out_f64, void* C, int n, const void* scale, hipStream_t s);

// Element conversions exposed for verification: mode 0 -> bfloat16 hi/lo
// (uint16 pairs), mode 1 -> OCP e4m3 bytes (no scaling).
hipError_t launch_convert(int mode, const float* x, int64_t count, void* out0, void* out1, hipStream_t s);

// Consumers of the packed product (ata_chol.hip), FP64 or FP32 throughout.
// Cholesky factor of packed lower C in place; info (device, may be null)
// receives the first failing column + 1 if it is still 0.  ws holds
// potrf_ws_bytes.  s2: helper stream for the lookahead, with two events e and
// f; the work on s2 is joined back into s before the call returns.
size_t potrf_ws_bytes(int64_t n);
hipError_t launch_potrf(bool f32, void* C, int64_t n, int32_t* info, void* ws, hipStream_t s, hipStream_t s2,
                        hipEvent_t e, hipEvent_t f);
// L L^t X = B in place, B row-major n x nrhs with row stride ldb (n, nrhs >= 1);
// ws holds potrs_ws_bytes (256-byte aligned; none for n <= 64).
size_t potrs_ws_bytes(bool f32, int64_t n, int64_t nrhs);
hipError_t launch_potrs(bool f32, const void* L, int64_t n, void* B, int64_t nrhs, int64_t ldb, void* ws,
                        hipStream_t s);
// out (m x nrhs, row stride ldo) = A X for A m x n (row stride lda) and X
// n x nrhs (row stride ldx, kAxPad readable elements after it), FP64 sums.
constexpr int kAxPad = 16;
hipError_t launch_ax(bool f32, const void* A, int64_t m, int64_t n, int64_t lda, const void* X, int64_t nrhs,
                     int64_t ldx, void* out, int64_t ldo, hipStream_t s);
// out (n x m, row stride m) = A^t for A m x n with row stride lda; elements of
// elem_bytes 4 or 8.
hipError_t launch_transpose(int elem_bytes, const void* A, int64_t m, int64_t n, int64_t lda, void* out,
                            hipStream_t s);
// out = A^t B; part holds atb_chunks(m, n, nrhs) x n x nrhs doubles (null: one chunk).
hipError_t launch_atb(bool f32, const void* A, int64_t m, int64_t n, int64_t lda, const void* B, int64_t nrhs,
                      int64_t ldb, void* out, int64_t ldo, double* part, hipStream_t s);

}  // namespace atalib
