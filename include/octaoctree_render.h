/*
 * liboctaoctree: the query of octaoctree.h with scratch memory from the
 * caller. Included by octaoctree.h.
 */
#ifndef OCTAOCTREE_RENDER_H
#define OCTAOCTREE_RENDER_H

#include "octaoctree.h"

#ifdef __cplusplus
extern "C" {
#endif

/*
 * oo_query_fwd with a workspace (device memory of the caller, free again
 * when the work on `stream` has passed the call). With a disparity predictor
 * the queries then run as three kernels (predictor, shifted encode into
 * decoder input rows, decoder), in half the time (1280x720 in FP16: 0.59 ms,
 * 1.22 without a workspace); trees without a predictor run the fused kernel
 * and need no workspace. The results are those of oo_query_fwd.
 *  - oo_query_workspace_bytes: the size this needs for B queries (0 without
 *    a predictor; bounded, since large batches run in passes).
 *  - workspace: 16-byte aligned. One that is not, or workspace_bytes smaller
 *    than that: OO_EINVAL, before any launch.
 *  - rgb_out may be the array x or the array dir, as in oo_query_fwd; the
 *    workspace overlaps none of the arrays.
 */
int oo_query_workspace_bytes(const oo_tree* tree, const oo_mlp* mlp, int64_t B, size_t* bytes);
int oo_query_fwd_ws(const oo_tree* tree, const oo_mlp* mlp, const float* x, const float* dir, const float* attr,
                    int64_t B, float* rgb_out, void* workspace, size_t workspace_bytes, hipStream_t stream);

#ifdef __cplusplus
}
#endif
#endif /* OCTAOCTREE_RENDER_H */
