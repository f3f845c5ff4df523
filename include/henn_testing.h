/*
 * henn_testing.h -- test-only flags and entry points of libhenn.
 *
 * Not part of the stable interface of henn.h.  Test suites use them to reach
 * alternative code paths that must give results identical to the default
 * ones, and the error paths of the library.  Same conventions as henn.h.
 */
#ifndef HENN_TESTING_H
#define HENN_TESTING_H

#include "henn.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Search flags (henn_search_params.flags) that select an alternative path
 * with the same results: */
#define HENN_SEARCH_NO_ROOT_KERNEL 4u /* scan a complete-graph root inside the search
                                         kernel instead of a separate scan */
#define HENN_SEARCH_ROOT_VALU 8u      /* scan a complete-graph root with the tiled
                                         VALU kernel instead of the matrix-core
                                         shortlist + exact check */
#define HENN_SEARCH_VIS32 16u         /* keep full 32-bit ids in the visited table
                                         even where 8- or 16-bit tags are exact */
#define HENN_SEARCH_VIS16 32u         /* keep 16-bit tags where 8-bit tags would be
                                         exact */

/* Allocation-failure injector for the error paths.  n >= 0: the next n device
 * allocations of the library succeed and every later one fails as out of
 * memory (the calls return HENN_E_NOMEM, and release what they allocated)
 * until the injector is set again; n < 0 turns it off (the default).
 * Process-wide; counts the allocations of every thread. */
henn_status henn_testing_fail_alloc_after(int64_t n);

/* How the kNN build launches one Gram pass (form 0: FP16, 1: split BF16, 2:
 * FP32) over n_rows rows of a layer of n points in d dimensions, for a graph of
 * this degree: splits of the candidates, candidates a split, 128-row blocks a
 * launch, and the blocks of the pilot that decides whether the FP16 form goes
 * on (0: none).
 * Host-only. */
typedef struct {
  int32_t splits;
  int32_t reserved;
  int64_t split_rows, slice_blocks, pilot_blocks;
} henn_testing_gram_plan;
henn_status henn_testing_knn_plan(int32_t form, int64_t n_rows, int64_t n, int32_t d,
                                  int32_t degree, henn_testing_gram_plan *out);

/* The launch shape henn_search_batch takes for nq queries with these params
 * on the current device: the 64-position blocks of the beam's list in
 * registers (0: in LDS), the bytes of LDS a wave uses and how many waves the
 * kernel's registers let a CU hold. */
typedef struct {
  int32_t lanes_per_vec, waves_per_block, vis_bits, persistent;
  int32_t list_blocks, lds_per_wave, register_waves;
  int32_t reserved;
} henn_testing_shape;
henn_status henn_testing_search_shape(const henn_index *idx, int64_t nq,
                                      const henn_search_params *sp, henn_testing_shape *out);

#ifdef __cplusplus
}
#endif

#endif /* HENN_TESTING_H */
