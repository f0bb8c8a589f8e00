/*
 * Symbols libspqr.so exports for the library's own tests and tuning runs.  Not part of the public interface
 * (include/spqr.h): they may change or go away with any build.
 */
#ifndef SPQR_TEST_HOOKS_H_
#define SPQR_TEST_HOOKS_H_

#include <stdint.h>

#ifdef __cplusplus
extern "C" {
#endif

/* Launch plan of a slice of b <= 16 vectors on the matrix-core path of spqr_gemm_smallbatch (count = 1) or of
 * spqr_gemm_fused for matrices m[i] x n[0] of one format (layout 1, 3-bit statistic codes) with nnz[i] outliers and the
 * hint max_row_nnz[i]; host arithmetic only, no device is touched.  plan[0..2] = units of 16 tile columns per split as the plan
 * prices them, splits, workgroups that share a split's outliers beside its dense one (0: none); plan[3..5] = the widths the launch
 * gives them: units of a split, how many of the first have more, how many units more.  Returns the units of the matrix, or
 * an SPQR_ERR_* code (SPQR_ERR_PARAM also for a format without that path). */
int spqr_plan_batch(int count, const int32_t* m, const int32_t* n, const int32_t* max_row_nnz, const int64_t* nnz, int w_bits,
                    int beta1, int beta2, int group_axis, int b, int32_t* plan);

/* Plan of ONE launch of spqr_gemv_grouped for `count` (1..8) matrices of one format (w_bits, beta1, beta2,
 * group_axis, layout_version; 3-bit statistic codes, or 16-bit statistics for layout 3), matrix i being m[i] x n[i]
 * with nnz[i] outliers and the hint max_row_nnz[i]; host arithmetic only, no device is touched.  The matrices of
 * the width n[0] size the launch (the library sorts the width with the most strips to the front before it plans).
 * `max_waves` and `slots` describe the kernel instance: the wavefronts a workgroup may have and the wavefronts a
 * compute unit holds (from the kernel's register count at run time); `row_dots_on_matrix_cores` says whether the
 * instance keeps its row dot products on the matrix cores (3-bit, 8 x 32 tiles, group_axis 1).
 * Returns the number of table entries k (the matrices taken; the others wait for the next launch), in grid order:
 * entries[7 * j + 0..6] = matrix index, strips per workgroup R, wavefronts per strip P, outlier chunks per round,
 * 1 if the outlier products take the place of x, the chunks the LDS behind x holds then, workgroups of the entry.
 * *wavefronts = R * P of every entry, *lds_bytes = the launch's dynamic LDS.  Negative: an SPQR_ERR_* code
 * (SPQR_ERR_PARAM also where no plan exists). */
int spqr_plan_grouped(int count, const int32_t* m, const int32_t* n, const int32_t* max_row_nnz, const int64_t* nnz,
                      int w_bits, int beta1, int beta2, int group_axis, int layout_version, int max_waves, int slots,
                      int row_dots_on_matrix_cores, int32_t* entries, int32_t* wavefronts, int64_t* lds_bytes);

/* Plan of the one-pass kernel for matrices as for spqr_plan_batch and b vectors (1 .. 256), with no more partial results of a
 * row than most_slots (0: the fastest plan's); host arithmetic only.  plan[0..4] = vectors per workgroup, units of 16 tile
 * columns per workgroup, workgroups per block of vectors, partial results of a row at most, workgroups per group of rows
 * of the outlier sort; *us = what its model says of it.  Returns the units of the matrix, or an SPQR_ERR_* code (SPQR_ERR_PARAM
 * also for a format without that kernel). */
int spqr_plan_prompt(int count, const int32_t* m, const int32_t* n, const int32_t* max_row_nnz, const int64_t* nnz, int w_bits,
                     int beta1, int beta2, int group_axis, int b, int most_slots, int32_t* plan, double* us);

/* The way a batch of b vectors (Y 16-byte aligned) goes through a matrix of layout 1 (3-bit statistic codes) with nnz outliers,
 * the hint max_row_nnz and, if has_perm, a permutation: 0 slices of 16 and fewer, 1 a dense copy, 2 the one-pass kernel, or an SPQR_ERR_* code.
 * Its scratch is a workspace of `scratch` bytes, SPQR_SCRATCH_LIBRARY or SPQR_SCRATCH_STATIC (the static array). */
#define SPQR_SCRATCH_LIBRARY (-1)
#define SPQR_SCRATCH_STATIC  (-2)
int spqr_batch_route(int m, int n, int64_t nnz, int max_row_nnz, int has_perm, int w_bits, int beta1, int beta2, int group_axis, int b, int64_t scratch);

/* What the outlier sort of the one-pass product makes of the row pointers (a HOST array of m + 1 entries) of a matrix with
 * nnz outliers in groups of `rows` rows: ranges[3 * g + 0..2] = first entry, end, slot of the group's first chunk of
 * 4096 entries (the others follow).  Returns the number of slots the scratch holds, or an SPQR_ERR_* code. */
int64_t spqr_sort_ranges(const int32_t* row_ptr, int m, int64_t nnz, int rows, int32_t* ranges);

/* Rows per workgroup, 16 or 64, of spqr_quantize's sweep of an m x n layer in blocks of beta1 columns and tiles of beta2 rows, with
 * outlier tests (tau finite) or without. */
int spqr_sweep_rows(int m, int n, int beta1, int beta2, int tests);

#ifdef __cplusplus
}
#endif
#endif  /* SPQR_TEST_HOOKS_H_ */
