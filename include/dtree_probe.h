/*
 * dtree_probe.h -- measurement helpers of the tree-evaluator library.
 *
 * Not part of the evaluation method.  A plain streaming copy and a plain streaming read
 * whose traffic is known exactly: they calibrate hardware byte counters (FETCH_SIZE /
 * WRITE_SIZE per dispatch) and measure the HBM bandwidth a simple kernel reaches on the
 * same device, next to the datasheet peak.  And which tables and kernels the evaluation
 * calls choose, for tests of the choice.
 */
#ifndef DTREE_PROBE_H
#define DTREE_PROBE_H

#include <stdint.h>

#include "dtree.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * Copy `bytes` bytes from d_src to d_dst (device pointers, 16-byte aligned, bytes a
 * multiple of 16, buffers not overlapping) with one kernel launch on `stream`
 * (a hipStream_t; NULL = null stream).  Asynchronous.  Reads exactly `bytes` and writes
 * exactly `bytes`.
 * Errors: DT_ERR_INVALID_ARG (null pointer with bytes > 0, misalignment, bytes < 0 or not
 * a multiple of 16), DT_ERR_HIP (launch failure).
 */
dt_status dt_probe_copy(const void *d_src, void *d_dst, int64_t bytes, void *stream);

/*
 * Read `bytes` bytes from d_src (device pointer, 16-byte aligned, bytes a multiple of 16)
 * with one kernel launch of waves_per_cu wavefronts per compute unit (1..32), each reading
 * 16 KiB tiles with 16-byte non-temporal loads.  d_sink: a device int32 the kernel may
 * write (in practice it never does; it keeps the reads from being optimised away).
 * Asynchronous on `stream`.  The streaming-read ceiling the tree kernels are compared with.
 * Errors: DT_ERR_INVALID_ARG (null pointer with bytes > 0, misalignment, bytes < 0 or not
 * a multiple of 16, waves_per_cu out of range), DT_ERR_HIP (launch failure).
 */
dt_status dt_probe_read(const void *d_src, int64_t bytes, int32_t *d_sink, int32_t waves_per_cu,
                        void *stream);

/*
 * Which tables the calls that dt_tree_launch_info describes walk: *list is 1 for the node
 * list (the data decomposition of trees that gain from it), 0 for windows.  Only the
 * alignment of d_x is read; nothing is launched.  Errors: as dt_tree_launch_info.
 */
dt_status dt_probe_tree_list(const dt_tree *tree, const void *d_x, dt_dtype x_type, int64_t ld,
                             dt_output out_kind, dt_algo algo, int32_t *list);

/* How a dt_forest_classify call of n > 0 records is spread over kernels. */
typedef struct {
    int32_t list;               /* 1: node lists, 0: windows                              */
    int32_t whole_waves;        /* wavefronts per workgroup of the unsplit kernel, one for
                                   each record tile (0: not launched)                     */
    int32_t split_waves;        /* the same of the kernel with several wavefronts per tile
                                   (0: not launched)                                      */
    int32_t waves_per_tile;     /* of that kernel (0: not launched)                       */
    int32_t whole_blocks_per_cu, split_blocks_per_cu;   /* resident workgroups            */
    int64_t whole_tiles, split_tiles;                   /* tiles of 64 records            */
} dt_forest_spread;

/* Fill *info for dt_forest_classify(forest, d_x, n, ld, ..., algo, ...).  Only the alignment
 * of d_x is read; nothing is launched.  Errors: DT_ERR_INVALID_ARG (null, n < 1, unknown
 * algo), DT_ERR_UNSUPPORTED (more than 256 features). */
dt_status dt_probe_forest_spread(const dt_forest *forest, const float *d_x, int64_t n, int64_t ld,
                                 dt_algo algo, dt_forest_spread *info);

#ifdef __cplusplus
}
#endif

#endif /* DTREE_PROBE_H */
