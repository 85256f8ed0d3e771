/* Entry points of libdgsp for its own torch binding (not part of the C-ABI in include/dgsp.h). */
#ifndef DGSP_INTERNAL_H
#define DGSP_INTERNAL_H

#include "../../include/dgsp.h"

#ifdef __cplusplus
extern "C" {
#endif

/* What the binding keeps of a matrix: the public statistics, what column blocks half as wide would save
 * (dgsp_internal_saved_share; 0: not measured) and, for products with one to four columns, the share of the entries that reading
 * the hot runs of X from LDS saves the caches (0: nothing, or not measured). */
typedef struct {
    dgsp_features_t features;
    double saved_share, hot_share[4];
} dgsp_internal_stats_t;

/* What a product may know and use beyond the public statistics; NULL: nothing.  hot_columns: the table that
 * dgsp_internal_measure_columns wrote for this matrix, on the product's GPU, or NULL.  workspace(context, bytes): device memory on
 * the product's GPU, aligned to 128 bytes, that is this call's until its launches on the product's stream have run; it may
 * return NULL, and does for a call that has some already, and the product goes without. */
typedef struct {
    double saved_share;
    const uint32_t *hot_columns;
    void *(*workspace)(void *context, size_t bytes);
    void *context;
} dgsp_internal_hints_t;

/* Statistics of a device CSR matrix with `entries` column indices, in one launch, and its arrays in 32-bit form:
 * index_bytes 8: rowptr and colidx are int64 and are written to rowptr32 (M + 1) and colidx32 (entries) as well;
 * index_bytes 4: they are int32 and the last two arguments are not used.  Waits for the result. */
int dgsp_internal_take_csr(int64_t M, int64_t K, int64_t entries, int index_bytes, const void *rowptr, const void *colidx,
                           int32_t *rowptr32, int32_t *colidx32, dgsp_features_t *out, void *stream);

/* Fills stats->saved_share and stats->hot_share from the matrix's device columns (a small launch that the call waits for)
 * where the launch rules would look at them, 0 elsewhere, and writes the hot runs to hot_columns (device memory,
 * dgsp_internal_hot_columns_bytes(stats) bytes; 0: no such table for this matrix, NULL is passed). */
int64_t dgsp_internal_hot_columns_bytes(const dgsp_internal_stats_t *stats);
int dgsp_internal_measure_columns(dgsp_internal_stats_t *stats, const int32_t *colidx, uint32_t *hot_columns, void *stream);
/* Would a product with these statistics look at the table? */
int dgsp_internal_wants_hot_columns(const dgsp_internal_stats_t *stats, int64_t N);
/* Its two halves: distinct columns and columns met once among 16384, 32768, 65536 sampled entries (six counts, of half
 * of the columns; `entries` at least 4096), and the share of entries whose column is not among the last 16384 distinct ones
 * but among the last 32768. */
int dgsp_internal_column_reuse(int64_t entries, const int32_t *colidx, uint64_t *counts, void *stream);
double dgsp_internal_saved_share(const uint64_t *counts);
/* Dense columns per column block of DGSP_NB_SR at width N. */
int dgsp_internal_nb_sr_block(const dgsp_internal_stats_t *stats, int64_t N);

/* The public entry points with hints beside the statistics: dgsp_spmm_csr_auto, dgsp_spmm_csr_phase, and
 * dgsp_spmm_csr_ld / _axpby (alpha_beta NULL / two factors). */
int dgsp_internal_spmm_auto(int64_t M, int64_t K, int64_t N, const dgsp_features_t *features, const dgsp_internal_hints_t *hints,
                            const int32_t *rowptr, const int32_t *colidx, const float *vals, const float *X, float *Y, int *chosen,
                            void *stream);
int dgsp_internal_spmm_phase(int64_t M, int64_t K, int64_t N, int64_t nnz, const int32_t *rowptr, const int32_t *colidx,
                             const float *vals, const float *X, float *Y, int algo, int phase, const dgsp_features_t *features,
                             const dgsp_internal_hints_t *hints, void *stream);
int dgsp_internal_spmm_view(int64_t M, int64_t K, int64_t N, int64_t nnz, const int32_t *rowptr, const int32_t *colidx,
                            const float *vals, const float *X, int64_t ldx, float *Y, int64_t ldy, const float *alpha_beta, int algo,
                            const dgsp_features_t *features, const dgsp_internal_hints_t *hints, void *stream);

/* dgsp_spmm_csr (nnz < 0) and dgsp_spmm_csr_nnz with the length of colidx, which bounds the entry count and sizes the launches. */
int dgsp_internal_spmm_csr(int64_t M, int64_t K, int64_t N, int64_t nnz, int64_t capacity, const int32_t *rowptr,
                           const int32_t *colidx, const float *vals, const float *X, float *Y, int algo,
                           const dgsp_internal_hints_t *hints, void *stream);

#ifdef __cplusplus
}
#endif
#endif
