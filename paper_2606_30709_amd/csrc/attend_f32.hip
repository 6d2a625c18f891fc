// Exact-token attention (Sec. 3.4, Eq. (1)) for fp32 inputs on the gfx950
// matrix cores (v_mfma_f32_32x32x2_f32: fp32 operands and accumulators).
//
// A workgroup of four wavefronts takes one 32-row query tile of one (batch,
// query head, query chunk).  The unit's keys pass in 32-key sub-tiles
// (current chunk, visible chunks, routed rows), dealt to the wavefronts in
// turn; each wavefront keeps its own online softmax and output accumulator
// and the four are merged through LDS at the end, in a fixed order.
//   S^T[key][query] = K.Q^T    (A = K rows from LDS, B = Q in registers)
//   O^T[d][query]  += V^T.P^T  (A = V from LDS, B = P: the lane's own scores)
// A product's contraction index may be permuted when both operands use the
// same permutation.  For S, lane half h holds dimensions h*D/2 + 0 .. D/2-1,
// so a K fragment is a run of 16-byte LDS reads; for P.V, step e takes the
// keys of accumulator element e, so P needs no exchange between lanes at all.
//
// Bound: the fp32 matrix rate (154 TFLOP/s from a large product on this
// card): 2*D MFMAs of 64 cycles per sub-tile and wavefront against about 150
// cycles of softmax and 16 KB (d64) of copies.  Each wavefront copies its own
// sub-tiles into a private LDS region (buffer loads with the LDS
// destination), K(t+1) while P.V(t) runs and V(t+1) while S(t+1) runs, so
// there is no barrier before the merge and one buffer per operand is enough.
// Four-wavefront workgroups leave room for two per CU at d64, whose
// prologues and merges hide behind each other's products.  Measured (whole
// layer, against the same split on the vector ALUs): 6/2 heads x 12,288
// tokens 345 -> 93 us (kernel 341 -> 88 us by rocprofv3, matrix cores 50%
// busy: 4.5 rounds of workgroups, of which the last is half empty), one head
// x 1,024 tokens 52 -> 23 us.  Both 32-row tiles of a head in one workgroup
// (half the copies per product) needs more than the 256 VGPRs that two
// wavefronts per SIMD have: 107 us against 91.
#include <hip/hip_ext.h>
#include <math.h>

#include "attend_common.hpp"
#include "hga_internal.hpp"
#include "lds_copy.hpp"

namespace hga {
namespace {

constexpr int KT = 64;     // tokens per chunk
constexpr int ST = 32;     // keys per sub-tile
constexpr int NW = 4;      // wavefronts per workgroup (key splits)
constexpr int kXcds = 8;

typedef float f32x16_t __attribute__((ext_vector_type(16)));

template <int D>
struct F32Layout {
    static constexpr int kRow = D * 4;                 // bytes per row
    static constexpr int kV = ST * kRow;               // V after K
    static constexpr int kGid = 2 * ST * kRow;         // the unit's group ids
    static constexpr int kWave = kGid + kMaxTopK * 4;  // bytes per wavefront
    static constexpr int kBytes = NW * kWave;
    // the merge reuses the wave's K and V: 32 output rows, then 32 x (m, l)
    static constexpr int kOutRow = D + 4;              // floats, padded against bank conflicts
    static constexpr int kMl = ST * kOutRow * 4;
    static_assert(kMl + ST * 8 <= kGid, "merge area");
};

// K is stored with 16-byte chunk j of row r at j ^ (r & 15) (the 16-byte
// fragment reads of 16 consecutive rows then cover every bank once) and V
// with chunk j at j ^ 8*((r >> 2) & 1), so that the two lane halves of a V
// read, four rows apart, fall in different banks.
__device__ __forceinline__ int swz_k(int row) { return row & 15; }
__device__ __forceinline__ int swz_v(int row) { return ((row >> 2) & 1) << 3; }

__device__ __forceinline__ float xor32_max(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false,
                                                    false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float xor32_add(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false,
                                                    false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

template <int D>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(D == 64 ? 2 : 1)))
void attend_f32_kernel(
    const float* __restrict__ q_rot, int q_chunk0, int n_q_chunks, const float* __restrict__ k_res,
    const float* __restrict__ v_res, int64_t res_tokens, const int32_t* __restrict__ res_slot,
    const float* __restrict__ k_routed, const float* __restrict__ v_routed,
    const int32_t* __restrict__ group_idx, float* __restrict__ out, float* __restrict__ lse, int r,
    FastDiv kv_div, FastDiv chunk_div, FastDiv tile_div, int group_shift, int keep_first,
    int window, int topk_groups, const float* __restrict__ k_src, const float* __restrict__ v_src,
    int64_t src_tokens, int n_items, ChunkMap q_map, ChunkMap unit_map) {
    using Lay = F32Layout<D>;
    constexpr int kRow = Lay::kRow;
    constexpr int CPR = D / 4;               // 16-byte chunks per row
    constexpr int CU = ST * kRow / 1024;     // copies per sub-tile, for K (and V)
    constexpr int NKF = D / 8;               // 16-byte fragments per lane and K row half
    constexpr int NDT = D / 32;
    extern __shared__ __align__(16) unsigned char smem[];

    // consecutive items (the query tiles of one unit, then the next unit) on
    // one XCD, whose L2 then holds the unit's keys
    const int per_xcd = (n_items + kXcds - 1) / kXcds;
    const uint32_t block = linear_block<NW * 64>();
    const int row = static_cast<int>(block / kXcds);  // past per_xcd: beyond the last item
    const int item = static_cast<int>(block % kXcds) * per_xcd + row;
    if (row >= per_xcd || item >= n_items) return;
    const int unit_id = tile_div.div(item);
    const int qtile = item - unit_id * tile_div.d;
    const int bh = chunk_div.div(unit_id);
    const int i = unit_id - bh * n_q_chunks;
    const int64_t unit = unit_map.at(bh, i);
    const int b = kv_div.div(bh), j = bh - b * kv_div.d;
    const int c = q_chunk0 + i;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;
    unsigned char* const mine = smem + wave * Lay::kWave;
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(mine));
    const int* s_gid = reinterpret_cast<const int*>(mine + Lay::kGid);

    const int n_q_heads = r * kv_div.d;
    const int hh = qtile >> 1, tq = qtile & 1;  // head of the group, half of the chunk
    const int64_t row0 = q_map.at(b * n_q_heads + j * r + hh, i) * KT + tq * ST;  // the first query row
    const float scale = 1.4426950408889634f / sqrtf(static_cast<float>(D));  // log2(e)/sqrt(d)
    const int64_t res_chunks = res_tokens / KT;
    const int routed_rows = topk_groups << group_shift;
    const int id_limit = c * (KT >> group_shift);

    const u32x4 rk_res = rsrc_words(k_res + static_cast<int64_t>(bh) * res_tokens * D,
                                    static_cast<uint32_t>(res_tokens * kRow));
    const u32x4 rv_res = rsrc_words(v_res + static_cast<int64_t>(bh) * res_tokens * D,
                                    static_cast<uint32_t>(res_tokens * kRow));
    // routed rows: the unit's routed buffers, or (none given) the source rows
    // of its groups
    const bool from_src = k_routed == nullptr;
    const int64_t rt_off = from_src ? static_cast<int64_t>(bh) * src_tokens * D
                                    : unit * routed_rows * D;
    const uint32_t rt_bytes = from_src ? static_cast<uint32_t>(src_tokens * kRow)
                                       : static_cast<uint32_t>(routed_rows * kRow);
    const u32x4 rk_rt = rsrc_words((from_src ? k_src : k_routed) + rt_off, rt_bytes);
    const u32x4 rv_rt = rsrc_words((from_src ? v_src : v_routed) + rt_off, rt_bytes);

    // the unit's group ids, one copy per wavefront (no barrier needed)
    {
        const u32x4 rg = rsrc_words(group_idx + unit * topk_groups,
                                    topk_groups * 4);
        for (int u = 0; u * 64 < topk_groups; ++u)
            copy4_to_lds(rg, (u * 64 + lane) * 4, lds0 + Lay::kGid + u * 256);
    }
    // B operand of S^T: the lane's query row, dimensions half*D/2 ..
    float q[D / 2];
    {
        const float* qp = q_rot + (row0 + col) * D + half * (D / 2);
#pragma unroll
        for (int u = 0; u < NKF; ++u) {
            const vec16 x = load16(qp + u * 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) q[u * 4 + e] = __uint_as_float(x.w[e]);
        }
    }

    const VisibleChunks vis(c, keep_first, window);
    const int n_fixed = 2 * (1 + vis.count);  // sub-tiles of the current and visible chunks
    const int n_sub = n_fixed + (routed_rows + ST - 1) / ST;
    bool bad = false;
    constexpr int RPC = 64 / CPR;  // rows per copy
    const int crow = lane / CPR;   // row of this lane's slot within a copy

    // Sub-tile `sub`: lane (any half, col) finds where row col of it starts
    // in its source (kAbsent: a row that reads zeros) and whether it counts.
    uint32_t row_at = 0;
    auto locate = [&](int sub) {
        if (sub < n_fixed) {
            const int cc = sub < 2 ? c : vis.chunk((sub >> 1) - 1);
            const int64_t slot = res_slot ? res_slot[cc] : cc;
            const bool ok = slot >= 0 && slot < res_chunks;
            bad |= !ok;
            row_at = ok ? static_cast<uint32_t>(slot * KT + (sub & 1) * ST + col) * kRow : kAbsent;
        } else {
            const int row = (sub - n_fixed) * ST + col;
            const int g = s_gid[min(row >> group_shift, topk_groups - 1)];
            const bool ok = row < routed_rows && g >= 0 && g < id_limit;
            const int at = from_src ? (g << group_shift) + (row & ((1 << group_shift) - 1)) : row;
            row_at = ok ? static_cast<uint32_t>(at) * kRow : kAbsent;
        }
    };
    // Copy u of a sub-tile holds rows u*RPC .. + RPC - 1; the lane's 16-byte
    // slot is chunk lane % CPR of row u*RPC + crow, unswizzled at the source.
    auto copy_rows = [&](const u32x4& rs, bool k_side) {
#pragma unroll
        for (int u = 0; u < CU; ++u) {
            const int row = u * RPC + crow;
            const uint32_t at = __shfl(row_at, row);
            const int sw = k_side ? swz_k(row) : swz_v(row);
            copy16_to_lds(rs, at + ((lane % CPR) ^ sw) * 16,
                          lds0 + (k_side ? 0 : Lay::kV) + u * 1024);
        }
    };
    auto copy_k = [&](int sub) { copy_rows(sub < n_fixed ? rk_res : rk_rt, true); };
    auto copy_v = [&](int sub) { copy_rows(sub < n_fixed ? rv_res : rv_rt, false); };

    f32x16_t oacc[NDT];
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[dt][e] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;  // m_run in log2 units

    int sub = wave;
    if (sub < n_sub) {
        if (sub >= n_fixed) wait_copies<0>();  // locate() reads the group ids
        locate(sub);
        copy_k(sub);
        copy_v(sub);
    }
    for (; sub < n_sub; sub += NW) {
        const int next = sub + NW;
        // keys of this sub-tile that count, one bit each (uniform)
        uint32_t live = static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(row_at < kAbsent));
        if (sub < 2 && sub > tq) live = 0;  // the later half of the current chunk
        wait_copies<CU>();  // K is here; V may be in flight
        // the scores in two chains (even and odd fragments): half the length
        // of the rounding chain, and two independent products in flight
        f32x16_t s, s1;
#pragma unroll
        for (int e = 0; e < 16; ++e) s[e] = s1[e] = 0.f;
        if (live) {
            const unsigned char* kp = mine + col * kRow;
#pragma unroll
            for (int u = 0; u < NKF; u += 2) {
                const vec16 k0 = load16(kp + (((half * NKF + u) ^ swz_k(col)) * 16));
                const vec16 k1 = load16(kp + (((half * NKF + u + 1) ^ swz_k(col)) * 16));
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    s = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(k0.w[e]), q[u * 4 + e],
                                                             s, 0, 0, 0);
                    s1 = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(k1.w[e]),
                                                              q[u * 4 + 4 + e], s1, 0, 0, 0);
                }
            }
        }
        lds_reads_done();  // before the next K lands on this one
        if (next < n_sub) {
            locate(next);
            copy_k(next);
        }
        if (live) {
#pragma unroll
            for (int e = 0; e < 16; ++e) s[e] += s1[e];
            if (live != 0xffffffffu) {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int key = (e >> 2) * 8 + half * 4 + (e & 3);
                    s[e] = (live >> key) & 1 ? s[e] : -INFINITY;
                }
            }
            if (sub < 2 && sub == tq) {  // the diagonal
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int key = (e >> 2) * 8 + half * 4 + (e & 3);
                    s[e] = key > col ? -INFINITY : s[e];
                }
            }
            float mx = s[0];
#pragma unroll
            for (int e = 1; e < 16; ++e) mx = fmaxf(mx, s[e]);
            mx = xor32_max(mx) * scale;
            const bool grow = mx > m_run;
            if (__builtin_amdgcn_ballot_w64(grow)) {
                const float alpha = grow ? __builtin_amdgcn_exp2f(m_run - mx) : 1.0f;
                l_run *= alpha;
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
                    for (int e = 0; e < 16; ++e) oacc[dt][e] *= alpha;
                m_run = grow ? mx : m_run;
            }
            const float m_use = m_run == -INFINITY ? 0.f : m_run;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                s[e] = __builtin_amdgcn_exp2f(fmaf(s[e], scale, -m_use));
                l_run += s[e];
            }
        }
        if (next < n_sub)
            wait_copies<CU>();  // V is here; the next K may be in flight
        else
            wait_copies<0>();
        if (live) {
            // V[key][dt*32 + col], key = (e>>2)*8 + half*4 + (e&3), whose
            // 128-byte block dt sits at dt ^ half (swz_v)
            const unsigned char* vp = mine + Lay::kV + half * 4 * kRow + col * 4;
#pragma unroll
            for (int e = 0; e < 16; ++e)
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt) {
                    const float a = *reinterpret_cast<const float*>(
                        vp + ((e >> 2) * 8 + (e & 3)) * kRow + (dt ^ half) * 128);
                    oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(a, s[e], oacc[dt], 0, 0, 0);
                }
        }
        lds_reads_done();
        if (next < n_sub) copy_v(next);
    }

    // merge of the four partial results, in wavefront order
    float* part = reinterpret_cast<float*>(mine);
    wait_copies<0>();  // (a wavefront without a sub-tile never waited for its ids)
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4)
            *reinterpret_cast<float4*>(part + col * Lay::kOutRow + dt * 32 + g4 * 8 + half * 4) =
                make_float4(oacc[dt][g4 * 4], oacc[dt][g4 * 4 + 1], oacc[dt][g4 * 4 + 2],
                            oacc[dt][g4 * 4 + 3]);
    const float l_tot = xor32_add(l_run);
    if (half == 0)
        *reinterpret_cast<float2*>(mine + Lay::kMl + col * 8) = make_float2(m_run, bad ? NAN : l_tot);
    __syncthreads();
#pragma unroll
    for (int it = 0; it < ST * CPR / (NW * 64); ++it) {
        const int idx = it * (NW * 64) + tid;
        const int row = idx / CPR, cc = idx % CPR;
        float2 ml[NW];
        float m = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            ml[w] = *reinterpret_cast<const float2*>(smem + w * Lay::kWave + Lay::kMl + row * 8);
            m = fmaxf(m, ml[w].x);
        }
        const float mu = m == -INFINITY ? 0.f : m;  // (only where the row's scores are)
        float l = 0.f;
        float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float f = exp2f(ml[w].x - mu);
            const float4 x = *reinterpret_cast<const float4*>(
                smem + w * Lay::kWave + (row * Lay::kOutRow + cc * 4) * 4);
            l = fmaf(ml[w].y, f, l);
            o.x = fmaf(x.x, f, o.x);
            o.y = fmaf(x.y, f, o.y);
            o.z = fmaf(x.z, f, o.z);
            o.w = fmaf(x.w, f, o.w);
        }
        const float inv = 1.0f / l;
        *reinterpret_cast<float4*>(out + (row0 + row) * D + cc * 4) =
            make_float4(o.x * inv, o.y * inv, o.z * inv, o.w * inv);
        if (lse && cc == 0) lse[row0 + row] = (m + log2f(l)) * 0.6931471805599453f;
    }
}

template <int D>
hipError_t launch_f32_t(const hga_plan& plan, const void* q_rot, int q_chunk0, int n_q_chunks,
                        const void* k_res, const void* v_res, int64_t res_tokens,
                        const int32_t* res_slot, const void* k_routed, const void* v_routed,
                        const int32_t* group_idx, void* out, float* lse, hipEvent_t ev_start,
                        hipEvent_t ev_stop, hipStream_t stream, const void* k_src,
                        const void* v_src, int64_t src_tokens, bool block_major) {
    const hga_params& p = plan.p;
    static std::atomic<uint64_t> configured{0};  // per kernel and device
    const hipError_t ce = once_per_device(configured, plan.device, [] {
        return hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_f32_kernel<D>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize,
                                   F32Layout<D>::kBytes);
    });
    if (ce != hipSuccess) return ce;
    const int r = p.n_q_heads / p.n_kv_heads;
    const int64_t items = static_cast<int64_t>(p.batch) * p.n_kv_heads * n_q_chunks * 2 * r;
    if (items > (int64_t(1) << 30)) return hipErrorInvalidConfiguration;
    const dim3 grid = grid_of((items + kXcds - 1) / kXcds * kXcds, NW * 64);
    const int group_shift = p.group == 8 ? 3 : (p.group == 16 ? 4 : 5);
    hipExtLaunchKernelGGL((attend_f32_kernel<D>), grid, dim3(NW * 64), F32Layout<D>::kBytes,
                          stream, ev_start, ev_stop, 0, static_cast<const float*>(q_rot), q_chunk0,
                          n_q_chunks, static_cast<const float*>(k_res),
                          static_cast<const float*>(v_res), res_tokens, res_slot,
                          static_cast<const float*>(k_routed), static_cast<const float*>(v_routed),
                          group_idx, static_cast<float*>(out), lse, r, FastDiv(p.n_kv_heads),
                          FastDiv(n_q_chunks), FastDiv(2 * r), group_shift, p.keep_first,
                          recent_window(p), p.topk_groups, static_cast<const float*>(k_src),
                          static_cast<const float*>(v_src), src_tokens,
                          static_cast<int>(items),
                          chunk_map(p.batch * p.n_q_heads, n_q_chunks, block_major),
                          chunk_map(p.batch * p.n_kv_heads, n_q_chunks, block_major));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_attend_f32(const hga_plan& plan, const void* q_rot, int q_chunk0, int n_q_chunks,
                             const void* k_res, const void* v_res, int64_t res_tokens,
                             const int32_t* res_slot, const void* k_routed, const void* v_routed,
                             const int32_t* group_idx, void* out, float* lse, hipEvent_t ev_start,
                             hipEvent_t ev_stop, hipStream_t stream, const void* k_src,
                             const void* v_src, int64_t src_tokens, bool block_major) {
    return (plan.p.head_dim == 64 ? launch_f32_t<64> : launch_f32_t<128>)(
        plan, q_rot, q_chunk0, n_q_chunks, k_res, v_res, res_tokens, res_slot, k_routed, v_routed,
        group_idx, out, lse, ev_start, ev_stop, stream, k_src, v_src, src_tokens, block_major);
}

}  // namespace hga
