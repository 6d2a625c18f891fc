// The routing query of a query chunk (Sec. 3.3; chunk-shared routing,
// Sec. 1): q_bar = the mean of the r*64 rotated query rows of KV head j over
// the chunk's 64 tokens and the r query heads that share the head.
#pragma once

#include "hga_device.hpp"

namespace hga {

// One wavefront reduces the r*64 rows of one query chunk in a fixed order:
// lane (rs, cv) adds the 16-byte column block cv of rows rs, rs + NRS, ...
// (UNROLL reads in flight), then a butterfly over the row slots adds the
// partial sums; the lanes with rs == 0 write out[0 .. D) (any address
// space).  row_vec(row, cv) returns that 16-byte block of row `row` (row =
// head * 64 + token) from wherever the rows are held.  Each lane adds its
// rows in ascending order whatever kUnroll (the reads in flight) is, so
// q_bar depends only on the shapes: it is bit-identical wherever this runs
// and wherever the rows are read from.
template <typename T, int D, int kUnroll = 16, typename RowVec>
__device__ __forceinline__ void wave_mean_rows(int rows, RowVec row_vec, float* out) {
    constexpr int V = elem<T>::kVec;
    constexpr int VPR = D / V;                               // 16-byte vectors per row
    constexpr int NRS = 64 / VPR;                            // row slots per wave
    constexpr int UNROLL = 64 / NRS < kUnroll ? 64 / NRS : kUnroll;  // NRS * UNROLL divides 64
    static_assert((NRS * UNROLL) <= 64 && 64 % (NRS * UNROLL) == 0, "q_bar row tiling");
    const int lane = threadIdx.x & 63;
    const int cv = lane % VPR, rs = lane / VPR;
    float acc[V];
#pragma unroll
    for (int e = 0; e < V; ++e) acc[e] = 0.f;
    for (int row0 = rs; row0 < rows; row0 += NRS * UNROLL) {
        vec16 x[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) x[u] = row_vec(row0 + u * NRS, cv);
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            float f[V];
            elem<T>::unpack(x[u], f);
#pragma unroll
            for (int e = 0; e < V; ++e) acc[e] += f[e];
        }
    }
#pragma unroll
    for (int m = VPR; m < 64; m <<= 1)
#pragma unroll
        for (int e = 0; e < V; ++e) acc[e] += __shfl_xor(acc[e], m, 64);
    const float inv = 1.0f / static_cast<float>(rows);
    if (rs == 0) {
#pragma unroll
        for (int e = 0; e < V; ++e) out[cv * V + e] = acc[e] * inv;
    }
}

// q_bar of query chunk i of the r query heads from head0 on, rows read from HBM.
template <typename T, int D>
__device__ __forceinline__ void wave_query_mean(const T* __restrict__ q_rot, int head0, int i, int r,
                                                const ChunkMap& map, float* out) {
    constexpr int V = elem<T>::kVec;
    const T* qbase = q_rot + map.at(head0, i) * 64 * D;
    const int64_t head_rows = static_cast<int64_t>(map.head) * 64;
    wave_mean_rows<T, D>(
        r * 64,
        [&](int row, int cv) {
            return load16(qbase + ((row >> 6) * head_rows + (row & 63)) * D + cv * V);
        },
        out);
}

}  // namespace hga
