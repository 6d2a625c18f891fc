// The chunk-major key gradients of the attention backward
// (attend_bwd_keys.hip), called by launch_attend_backward.
#pragma once

#include "hga_internal.hpp"

namespace hga {

// Key chunks of a (batch, KV head) the inverted lists cover (one LDS counter
// each while they are built).
constexpr int kBwdIndexChunks = 16384;

// Whether the lists and D_i fit the dq buffer (they do unless a few query
// chunks face a history of hundreds of times their number).
bool bwd_chunks_fit(const hga_plan& plan, int q_chunk0, int n_q_chunks);
size_t bwd_chunks_lds_bytes(const hga_plan& plan);

// dk += .., dv += .. for the query chunks' attention; dq holds the row
// statistics in its leading floats (per 32 query rows, in lse's order: their
// 32 values of -lse in log2 units, then their 32 of -D_i) and is overwritten
// past them with the lists.
hipError_t launch_bwd_chunks(const hga_plan& plan, const void* q_rot, int q_chunk0, int n_q_chunks,
                             const void* k_res, const void* v_res, int64_t res_tokens,
                             const int32_t* group_idx, const void* dout, float* dq, float* dk,
                             float* dv, hipStream_t stream);

}  // namespace hga
