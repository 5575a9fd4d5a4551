// Host side of the scratch-free attention kernel (attend_items.hip).
#pragma once
#include <hip/hip_runtime.h>

#include "common.hpp"

namespace fsr {

// Runs the attention call *p (already validated; B, N_cap > 0) with one workgroup per (request, KV head, group of
// query rows); needs no workspace.
int attend_items_launch(const void* q, const void* k_cache, const void* v_cache, const int32_t* block_tables,
                        const int32_t* ctx_lens, const int32_t* cu_q, void* out, float* lse, const fsr_attn_params* p,
                        hipStream_t s, const char* who);

}  // namespace fsr
