// Runtime entry points shared by the layer runtime and the whole-model
// driver (internal: not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>

#include "hb.h"

namespace hb {

// HB_ERR_HIP when the stream is under graph capture. Calls whose kernels read a
// slot of the metadata ring (or the model's row staging), and the KV append, are
// refused there before anything is enqueued; the capture itself stays valid.
hb_status refuse_capture(hipStream_t s);

// One iteration of a stack of layers that share configuration, pool size
// and stream, over one batch: the batch is validated, planned and its
// metadata uploaded once, and every layer's kernels read that upload.
// Layer l reads x_in[l] and writes x_out[l] (bf16 or fp32 per desc).
hb_status run_layer_stack(hb_layer* const* layers, int n, const hb_batch_desc* desc, const void* const* x_in,
                          void* const* x_out);

}  // namespace hb
