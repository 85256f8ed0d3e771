/* Entry points of libdgsp for its own torch binding (not part of the C-ABI in include/dgsp.h). */
#ifndef DGSP_INTERNAL_H
#define DGSP_INTERNAL_H

#include "../../include/dgsp.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Statistics of a device CSR matrix with `entries` column indices, in one launch, and its arrays in 32-bit form:
 * index_bytes 8: rowptr and colidx are int64 and are written to rowptr32 (M + 1) and colidx32 (entries) as well;
 * index_bytes 4: they are int32 and the last two arguments are not used.  Waits for the result. */
int dgsp_internal_take_csr(int64_t M, int64_t K, int64_t entries, int index_bytes, const void *rowptr, const void *colidx,
                           int32_t *rowptr32, int32_t *colidx32, dgsp_features_t *out, void *stream);

/* dgsp_spmm_csr with the length of colidx, which bounds the entry count and sizes the launches. */
int dgsp_internal_spmm_csr(int64_t M, int64_t K, int64_t N, int64_t capacity, const int32_t *rowptr, const int32_t *colidx,
                           const float *vals, const float *X, float *Y, int algo, void *stream);

#ifdef __cplusplus
}
#endif
#endif
