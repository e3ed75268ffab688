/* What the torch conveniences (binding.cpp, __init__.py) lend a call that was given no workspace, for that call alone, or no buffer.  Exported for them by libvq.so;
 * no part of the library's interface. */
#ifndef VQ_LEND_H
#define VQ_LEND_H
#include "../../include/vq.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Of vq_gemv_with_workspace.  0 where no kernel of exactly these rows would use it, and for layers with codebook groups and v = 6 / 12-bit layers in
 * stored order: their kernels without one are good, and those along the rows sum in the same order with vq_gemv_multi (one row, and from three on) or a
 * workspace that is too small.  Of v = 6 rows of an
 * odd width, which those kernels take far more slowly than a copy of them, or than group by group, that order is given up. */
size_t vq_lend_gemv_bytes(const vq_layer_desc *desc, int32_t batch);
/* Of vq_gemm_default, on a card without room for what it asks for: the same route without the sums of a product in parts. */
size_t vq_lend_gemm_least_bytes(const vq_layer_desc *desc, int32_t tokens);

/* vq_assign (down: vq_assign_down) into a buffer as the allocator left it: the rest of every stride is written too, as zeros. */
int vq_lend_assign(const void *W, const void *B, int64_t ld, int32_t rows, int32_t cols, const void *codebook, int32_t v, int32_t k, void *idx,
                   int64_t idx_row_stride, int32_t down, void *hip_stream);

#ifdef __cplusplus
}
#endif
#endif
