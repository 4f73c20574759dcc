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

#ifdef __cplusplus
}
#endif
