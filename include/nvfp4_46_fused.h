/*
 * nvfp4_46_fused -- pairs of nvfp4_46.h's calls in one (same library, conventions and results).
 */
#ifndef NVFP4_46_FUSED_H
#define NVFP4_46_FUSED_H

#include "nvfp4_46.h"

#ifdef __cplusplus
extern "C" {
#endif

/* nvfp4_46_tensor_scale_ws (nvfp4_46_tensor_scale when `workspace` is NULL) followed by
 * nvfp4_46_quantize with the scale it wrote: the same outputs, bit for bit, and the same
 * requirements and errors as those two calls; nothing is enqueued when either would be refused.
 * A small tensor quantized rowwise, to nearest and without the transform takes one launch, which
 * leaves the workspace alone; any other takes the launches of the two calls.
 *   alpha  out  1 float (device)                                                                */
int nvfp4_46_scale_quantize(const void *x, const nvfp4_46_params *p, float *alpha,
                            void *workspace, size_t workspace_bytes, void *codes_row,
                            void *scales_row, void *codes_col, void *scales_col,
                            void *choice_row, void *choice_col, void *stream);

#ifdef __cplusplus
}
#endif

#endif
