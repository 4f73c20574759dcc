/* cg_conv_forward for callers that allocate a workspace call by call: only what the call itself reads of it is asked for. */
#pragma once

#include "cg_conv.h"

#ifdef __cplusplus
extern "C" {
#endif

/* Scratch of a call with or without a bitmap of the caller's, with or without counts: 0 unless fired gates are counted without a bitmap
 * or the layer has a channel-wise gate. */
size_t cg_conv_call_scratch_bytes(const cg_conv* h, int32_t n, int has_bitmap, int has_counts);

/* As cg_conv_forward, with that many bytes of workspace. */
int cg_conv_call(cg_conv* h, int32_t n, const void* x, const void* residual, void* y, uint32_t* bitmap, uint32_t* counts, void* workspace,
                 size_t workspace_bytes, void* hip_stream);

/* As cg_conv_call without residual, bitmap, counts and channel-wise gate, and beside it, of the same x and with the layer's stride, what
 * cg_pointwise_conv computes from w1 [c_out1][c_in], scale1 and shift1 into y1: the first layer of a residual block and its shortcut, in one launch
 * where the layer has few pixels.  bf16 layers whose pixels have no gaps. */
int cg_conv_call_beside(cg_conv* h, int32_t n, const void* x, void* y, const void* w1, const float* scale1, const float* shift1, void* y1,
                        int32_t c_out1, int32_t relu1, void* hip_stream);

#ifdef __cplusplus
}
#endif
