// The chunk-major key gradients of the attention backward
// (attend_bwd_keys.hip), called by launch_attend_backward.
#pragma once

#include "hga_device.hpp"
#include "hga_internal.hpp"

namespace hga {

// Key chunks of a (batch, KV head) whose inverted lists one workgroup builds
// (one LDS counter each).
constexpr int kBwdIndexChunks = 16384;

// Whether the lists and D_i fit the dq buffer (they do unless a few query
// chunks face a history of hundreds of times their number).
bool bwd_chunks_fit(const hga_plan& plan, int q_chunk0, int n_q_chunks);
size_t bwd_chunks_lds_bytes(const hga_plan& plan);

// dk += .., dv += .. for the query chunks' attention (or `write`: = .., and
// zeros in the other rows).  dq is scratch: the row statistics
// (bwd_row_stat), then the lists.
hipError_t launch_bwd_chunks(const hga_plan& plan, const void* q_rot, int q_chunk0, int n_q_chunks,
                             const void* k_res, const void* v_res, int64_t res_tokens,
                             const int32_t* group_idx, const void* out, const float* lse,
                             const void* dout, float* dq, float* dk, float* dv, bool write,
                             hipStream_t stream);

// dk += .., dv += .. unit by unit, from the row statistics; at most `tiles` key
// tiles a unit.
hipError_t launch_bwd_units(const hga_plan& plan, const void* q_rot, int q_chunk0, int n_q_chunks,
                            const void* k_res, const void* v_res, int64_t res_tokens,
                            const int32_t* group_idx, const float* stat, const void* dout,
                            float* dk, float* dv, int tiles, hipStream_t stream);

// Workgroup barrier that orders LDS only: waits for this wave's LDS
// operations, not for its copies or atomics.
__device__ __forceinline__ void lds_barrier() {
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
}

// Value of 16-bit element e of a 16-byte vector of bf16, taken from the 32-bit
// words.
__device__ __forceinline__ float bf16_value(const vec16& v, int e) {
    return __uint_as_float((e & 1) ? (v.w[e >> 1] & 0xffff0000u) : (v.w[e >> 1] << 16));
}

// Row statistics: per 32 query rows (in lse's order), their 32 values of -lse
// in log2 units, then their 32 of -D_i = -dout_i . out_i.  Thread `thread` of
// the launch: eight lanes per row, each over every eighth 16-byte vector.
template <int D>
__device__ __forceinline__ void bwd_row_stat(const bf16_t* __restrict__ out,
                                             const bf16_t* __restrict__ dout,
                                             const float* __restrict__ lse,
                                             float* __restrict__ stat, int64_t rows,
                                             int64_t thread) {
    constexpr int VPR = D / 8;
    const int64_t row = thread >> 3;
    const int part = static_cast<int>(thread & 7);
    float acc = 0.f;
    if (row < rows) {
#pragma unroll
        for (int u = 0; u < VPR / 8; ++u) {
            const vec16 g = load16(dout + row * D + (u * 8 + part) * 8);
            const vec16 o = load16(out + row * D + (u * 8 + part) * 8);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc = fmaf(bf16_value(g, e), bf16_value(o, e), acc);
        }
    }
    acc += __shfl_xor(acc, 1);
    acc += __shfl_xor(acc, 2);
    acc += __shfl_xor(acc, 4);
    if (row < rows && part == 0) {
        float* at = stat + (row >> 5) * 64 + (row & 31);
        at[0] = lse[row] * -1.4426950408889634f;
        at[32] = -acc;
    }
}

}  // namespace hga
