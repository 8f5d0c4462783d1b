/*
 * bbm_mask_index.h -- the whole preprocessing of a mask in one call (see bbm.h for its parts).
 */
#ifndef BBM_MASK_INDEX_H
#define BBM_MASK_INDEX_H

#include "bbm.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Exactly the outputs of bbm_build_block_mask_rect followed by bbm_build_index and, if col_ptr is given, bbm_build_col_index: same
 * arguments, requirements and errors; bin_blk_mat, packed_mask, sched and col_sched may be NULL there and here.  Fewer launches:
 * the indexes of block rows and block columns share one where each would take one, and with `arrivals` a small mask without
 * columns (at most 8 block rows over all planes and 4096 blocks) is served by a single one.
 *   arrivals         one int32 in device memory, zero when it is first used and not written by the caller afterwards (every call
 *                    leaves it zero again); not shared by calls that may run at the same time.  A call that is being recorded
 *                    into a graph leaves it alone.  NULL: not used.
 */
int bbm_build_mask_index(const uint8_t* mask, int64_t Mb, int64_t Nq, int64_t Nk, int64_t row_stride_bytes, int Br, int Bc,
                         uint8_t* blk_class, uint8_t* bin_blk_mat, uint64_t* packed_mask, int32_t* offset,
                         int32_t* total_ones, int32_t* nz_lo, int32_t* nz_hi, int32_t* nz_cnt, int32_t* row_ptr,
                         uint32_t* col_idx, int32_t* sched, int32_t* col_ptr, uint32_t* row_idx, int32_t* col_sched,
                         int32_t* arrivals, void* stream);

#ifdef __cplusplus
}
#endif

#endif /* BBM_MASK_INDEX_H */
