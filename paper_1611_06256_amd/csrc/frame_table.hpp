// Predictions and updates on frames that lie wherever a table of pointers says (the scheduler's agents keep their own
// frames): the first layer's kernels fetch each frame from its place, so the batch is not put together in memory first.
// The table is host memory the GPU can read (pinned) and must stay as it is until the call's GPU work has finished; behind a
// prediction whose values and actions go to coherent host memory, until the last of them has arrived there (each is stored once).
#pragma once
#include <hip/hip_runtime.h>

#include "../../include/ga3c.h"

namespace ga3c {

// Whether the context's first layer can (the shape-specific layer of the small and the larger net); other contexts take
// contiguous frames only.
bool takes_frame_table(const ga3c_ctx *c);
// ga3c_predict, ga3c_train_step (seg_start == nullptr) and ga3c_train_step_ragged (T = 1) from a table.
int predict_from_table(ga3c_ctx *c, const uint8_t *const *table, int B, const float *uniforms, float *values, int32_t *actions, hipStream_t s);
int train_from_table(ga3c_ctx *c, const uint8_t *const *table, const int32_t *actions, const float *rewards, const uint8_t *dones,
                     const float *bootstrap, const int32_t *seg_start, int N, int T, int B, const ga3c_hparams *hp, hipStream_t s);

}  // namespace ga3c
