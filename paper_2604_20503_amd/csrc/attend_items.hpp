// Host side of attend_items.hip, the attention kernel that can do without scratch memory.
#pragma once
#include <hip/hip_runtime.h>

#include "common.hpp"

namespace fsr {

// Runs the attention call *p (already validated; B, N_cap > 0) with one workgroup per (request, KV head, group of
// query rows).  With a workspace of attend_items_workspace_bytes (256-byte aligned) the keys of long items are cut into pieces;
// with less, or none, they are not.
int attend_items_launch(const void* q, const void* k_cache, const void* v_cache, const int32_t* block_tables,
                        const int32_t* ctx_lens, const int32_t* cu_q, void* out, float* lse, const fsr_attn_params* p,
                        void* workspace, size_t ws_bytes, hipStream_t s, const char* who);
size_t attend_items_workspace_bytes(const fsr_attn_params& p);

}  // namespace fsr
