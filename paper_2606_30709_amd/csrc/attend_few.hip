// Exact-token attention (Sec. 3.4, Eq. (1)) for bf16 launches of a few units (a
// decode block, one block of a block-sequential prefill) on the gfx950 matrix
// cores (v_mfma_f32_32x32x16_bf16), without a second launch for the merge.
//
// A workgroup takes one 32-row query tile of one (batch, KV head, query chunk)
// and all of its keys: eight wavefronts deal the 32-key sub-tiles (current
// chunk, visible chunks, routed rows) among themselves, each with its own
// online softmax, output accumulator and LDS staging (no barrier), and their
// partial results meet in LDS at the end, in a fixed order.
//   S^T[key][query] = K.Q^T    (A = K rows, B = Q in registers)
//   O^T[d][query]  += V^T.P^T  (A = transpose reads of V rows, B = the lane's P)
// K(t+1) is copied while P.V(t) runs and V(t+1) while S(t+1) runs.
//
// Bound: latency, then the keys' way into one CU (64 bytes per clock: 5 us for
// the 608 KB of a 64K decode block's 19 tiles).  Dividing each unit's tiles
// among workgroups instead (80 of them for the four units of that block) moves
// less per CU but leaves 10.6 MB of fp32 partial results for a second kernel:
// 19.8 us for that block's attention, against 13.7 here.
#include <hip/hip_runtime.h>
#include <math.h>

#include "attend_common.hpp"
#include "hga_internal.hpp"
#include "lds_copy.hpp"

namespace hga {
namespace {

constexpr int KT = 64;  // tokens per chunk
constexpr int ST = 32;  // keys per sub-tile
constexpr int NW = 8;   // wavefronts per workgroup (key splits)

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;
typedef float f32x16_t __attribute__((ext_vector_type(16)));

template <int D>
struct FewLayout {
    static constexpr int kRow = D * 2;
    static constexpr int kV = ST * kRow;               // V after K
    static constexpr int kGid = 2 * ST * kRow;         // the unit's group ids
    static constexpr int kWave = kGid + kMaxTopK * 4;  // bytes per wavefront
    static constexpr int kBytes = NW * kWave;
    // the merge reuses all of it: 32 output rows, then 32 x (m, l)
    static constexpr int kOutRow = D + 4;              // floats, padded against bank conflicts
    static constexpr int kMl = ST * kOutRow * 4;
    static_assert(kMl + ST * 8 <= kWave, "merge area");
};

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

// kGather: the routed rows come from k_src / v_src by group id and, when
// k_routed / v_routed are given, are written there (the unit's query tiles
// share the writing); otherwise they are read from k_routed / v_routed.
template <int D, bool kGather>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(2)))
void attend_few_kernel(
    const bf16_t* __restrict__ q_rot, int q_chunk0, int n_q_chunks,
    const bf16_t* __restrict__ k_res, const bf16_t* __restrict__ v_res, int64_t res_tokens,
    const int32_t* __restrict__ res_slot, bf16_t* __restrict__ k_routed,
    bf16_t* __restrict__ v_routed, const int32_t* __restrict__ group_idx,
    bf16_t* __restrict__ out, float* __restrict__ lse, int r, FastDiv kv_div, FastDiv chunk_div,
    FastDiv tile_div, int group_shift, int keep_first, int window, int topk_groups,
    const bf16_t* __restrict__ k_src, const bf16_t* __restrict__ v_src, int64_t src_tokens,
    ChunkMap q_map, ChunkMap unit_map) {
    using Lay = FewLayout<D>;
    constexpr int kRow = Lay::kRow;
    constexpr int CPR = D / 8;             // 16-byte chunks per row
    constexpr int RPC = 64 / CPR;          // rows per copy
    constexpr int CU = ST / RPC;           // copies per sub-tile, for K (and V)
    constexpr int NKS = D / 16, NDT = D / 32;
    extern __shared__ __align__(16) unsigned char smem[];

    const int item = tile_div.div(blockIdx.x);
    const int qtile = blockIdx.x - item * tile_div.d;
    const int bh = chunk_div.div(item);
    const int i = item - bh * n_q_chunks;
    const int64_t unit = unit_map.at(bh, i);
    const int b = kv_div.div(bh), j = bh - b * kv_div.d;
    const int c = q_chunk0 + i;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;
    unsigned char* const mine = smem + wave * Lay::kWave;
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(mine));
    const int* s_gid = reinterpret_cast<const int*>(mine + Lay::kGid);

    const int hh = qtile >> 1, tq = qtile & 1;  // head of the group, half of the chunk
    // the tile's first query row
    const int64_t row0 = q_map.at(b * (r * kv_div.d) + j * r + hh, i) * KT + tq * ST;
    const float scale = 1.4426950408889634f / sqrtf(static_cast<float>(D));  // log2(e)/sqrt(d)
    const int64_t res_chunks = res_tokens / KT;
    const int routed_rows = topk_groups << group_shift;
    const int id_limit = c * (KT >> group_shift);

    const u32x4 rk_res = rsrc_words(k_res + static_cast<int64_t>(bh) * res_tokens * D,
                                    static_cast<uint32_t>(res_tokens * kRow));
    const u32x4 rv_res = rsrc_words(v_res + static_cast<int64_t>(bh) * res_tokens * D,
                                    static_cast<uint32_t>(res_tokens * kRow));
    const int64_t rt_off = kGather ? static_cast<int64_t>(bh) * src_tokens * D
                                   : unit * routed_rows * D;
    const uint32_t rt_bytes = static_cast<uint32_t>((kGather ? src_tokens : routed_rows) * kRow);
    const u32x4 rk_rt = rsrc_words((kGather ? k_src : k_routed) + rt_off, rt_bytes);
    const u32x4 rv_rt = rsrc_words((kGather ? v_src : v_routed) + rt_off, rt_bytes);

    // the unit's group ids, one copy per wavefront
    {
        const u32x4 rg = rsrc_words(group_idx + unit * topk_groups,
                                    topk_groups * 4);
        for (int u = 0; u * 64 < topk_groups; ++u)
            copy4_to_lds(rg, (u * 64 + lane) * 4, lds0 + Lay::kGid + u * 256);
    }

    const VisibleChunks vis(c, keep_first, window);
    const int n_fixed = 2 * (1 + vis.count);  // sub-tiles of the current and visible chunks
    const int n_sub = n_fixed + (routed_rows + ST - 1) / ST;
    bool bad = false;
    const int crow = lane / CPR;  // row of this lane's slot within a copy
    uint32_t koff[CU];            // 16-byte chunk it takes of its row, unswizzled at the source
#pragma unroll
    for (int u = 0; u < CU; ++u) koff[u] = ((lane % CPR) ^ swz_rows<D>(u * RPC + crow)) * 16;

    // Sub-tile `sub`: lane (any half, col) finds where row col of it starts
    // in its source (kAbsent: a row that reads zeros).
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
            const int at = kGather ? (g << group_shift) + (row & ((1 << group_shift) - 1)) : row;
            row_at = ok ? static_cast<uint32_t>(at) * kRow : kAbsent;
        }
    };
    auto copy_rows = [&](const u32x4& rs, uint32_t lds) {
#pragma unroll
        for (int u = 0; u < CU; ++u)
            copy16_to_lds(rs, __shfl(row_at, u * RPC + crow) + koff[u], lds + u * 1024);
    };
    auto copy_k = [&](int sub) { copy_rows(sub < n_fixed ? rk_res : rk_rt, lds0); };
    auto copy_v = [&](int sub) { copy_rows(sub < n_fixed ? rv_res : rv_rt, lds0 + Lay::kV); };

    int sub = wave;
    if (sub < n_sub) {
        if (sub >= n_fixed) wait_copies<0>();  // locate() reads the group ids
        locate(sub);
        copy_k(sub);
        copy_v(sub);
    }
    // B operand of S^T: the lane's query row, dimensions kk*16 + half*8 ..
    bf16x8_t qf[NKS];
#pragma unroll
    for (int kk = 0; kk < NKS; ++kk)
        qf[kk] = __builtin_bit_cast(bf16x8_t, load16(q_rot + (row0 + col) * D + half * 8 + kk * 16));

    f32x16_t oacc[NDT];
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) oacc[dt][e] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;  // m_run in log2 units
    // LDS offsets of this lane's reads (rows 16 further on are immediates)
    int aoff[NKS], toff[2][NDT];
#pragma unroll
    for (int kk = 0; kk < NKS; ++kk)
        aoff[kk] = col * kRow + (((2 * kk + half) ^ swz_rows<D>(col)) * 16);
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
            const int row = x * 8 + half * 4 + ((lane & 15) >> 2);
            const int ch = dt * 4 + ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1);
            toff[x][dt] = row * kRow + ((ch ^ swz_rows<D>(row)) * 16) + (lane & 1) * 8;
        }
    // this lane's slots of a staged routed sub-tile to the routed buffer
    auto write_rows = [&](int rs, const unsigned char* staged, bf16_t* dst) {
        unsigned char* at = reinterpret_cast<unsigned char*>(dst) +
                            (unit * routed_rows + rs * ST) * kRow;
#pragma unroll
        for (int u = 0; u < CU; ++u) {
            const int row = u * RPC + crow;
            const vec16 x = *reinterpret_cast<const vec16*>(staged + u * 1024 + lane * 16);
            if (rs * ST + row < routed_rows)
                __builtin_nontemporal_store(__builtin_bit_cast(u32x4, x),
                                            reinterpret_cast<u32x4*>(at + row * kRow + koff[u]));
        }
    };
    const int n_qt = tile_div.d;

    // (the query fragments were requested after the first copies)
    for (bool first = true; sub < n_sub; sub += NW, first = false) {
        const int next = sub + NW;
        // keys of this sub-tile that count, one bit each (uniform)
        uint32_t live = static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(row_at < kAbsent));
        if (sub < 2 && sub > tq) live = 0;  // the later half of the current chunk
        const int rs = sub - n_fixed;
        const bool write = kGather && k_routed != nullptr && rs >= 0 && rs % n_qt == qtile;
        if (first)
            wait_copies<0>();
        else
            wait_copies<CU>();  // K is here; V may be in flight
        if (write) write_rows(rs, mine, k_routed);
        f32x16_t s;
#pragma unroll
        for (int e = 0; e < 16; ++e) s[e] = 0.f;
        if (live) {
#pragma unroll
            for (int kk = 0; kk < NKS; ++kk)
                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    __builtin_bit_cast(bf16x8_t, load16(mine + aoff[kk])), qf[kk], s, 0, 0, 0);
        }
        lds_reads_done();  // before the next K lands on this one
        if (next < n_sub) {
            locate(next);
            copy_k(next);
        }
        bf16x8_t pf[2];
        if (live) {
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
            // the reference point moves only when it is exceeded by more than
            // 8 (log2 units): the weights stay below 2^8
            const bool grow = mx > m_run + 8.0f;
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
                const float p = __builtin_amdgcn_exp2f(fmaf(s[e], scale, -m_use));
                l_run += p;
                pf[e >> 3][e & 7] = static_cast<__bf16>(p);
            }
        }
        // V is here; the next K may be in flight (stores count too: a writing
        // wavefront waits for all)
        if (next < n_sub && !write)
            wait_copies<CU>();
        else
            wait_copies<0>();
        if (write) write_rows(rs, mine + Lay::kV, v_routed);
        if (live) {
            // k-slot half*8 + e of block kap is key kap*16 + (e/4)*8 + half*4 + e%4
#pragma unroll
            for (int kap = 0; kap < 2; ++kap)
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt) {
                    auto tr = [&](int off) {
                        return __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_i16x4_t*)(
                            reinterpret_cast<uintptr_t>(mine + Lay::kV + kap * 16 * kRow + off)));
                    };
                    const bf16x8_t a = __builtin_bit_cast(
                        bf16x8_t, __builtin_shufflevector(tr(toff[0][dt]), tr(toff[1][dt]), 0, 1,
                                                          2, 3, 4, 5, 6, 7));
                    oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pf[kap], oacc[dt], 0, 0, 0);
                }
        }
        lds_reads_done();
        if (next < n_sub) copy_v(next);
    }

    // merge of the partial results, in wavefront order
    wait_copies<0>();  // (a wavefront without a sub-tile never waited for its ids)
    float* part = reinterpret_cast<float*>(mine);
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
    if (tid >= ST * CPR) return;
    const int row = tid / CPR, cc = tid % CPR;  // eight dimensions of one row
    float2 ml[NW];
    float m = -INFINITY;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        ml[w] = *reinterpret_cast<const float2*>(smem + w * Lay::kWave + Lay::kMl + row * 8);
        m = fmaxf(m, ml[w].x);
    }
    const float mu = m == -INFINITY ? 0.f : m;  // (only where the row's scores are)
    float l = 0.f, o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const float f = __builtin_amdgcn_exp2f(ml[w].x - mu);
        l = fmaf(ml[w].y, f, l);
        const float* x = reinterpret_cast<const float*>(smem + w * Lay::kWave) + row * Lay::kOutRow + cc * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = fmaf(x[e], f, o[e]);
    }
    const float inv = 1.0f / l;
    bf16x8_t v;
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = static_cast<__bf16>(o[e] * inv);
    *reinterpret_cast<bf16x8_t*>(out + (row0 + row) * D + cc * 8) = v;
    if (lse && cc == 0) lse[row0 + row] = (m + log2f(l)) * 0.6931471805599453f;
}

template <int D, bool kGather>
hipError_t launch_few_t(const hga_plan& plan, const void* q_rot, int q_chunk0, int n_q_chunks,
                        const void* k_res, const void* v_res, int64_t res_tokens,
                        const int32_t* res_slot, void* k_routed, void* v_routed,
                        const int32_t* group_idx, void* out, float* lse, hipStream_t stream,
                        const void* k_src, const void* v_src, int64_t src_tokens, bool block_major) {
    const hga_params& p = plan.p;
    static std::atomic<uint64_t> configured{0};  // per instantiation and device
    const hipError_t ce = once_per_device(configured, plan.device, [] {
        return hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_few_kernel<D, kGather>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, FewLayout<D>::kBytes);
    });
    if (ce != hipSuccess) return ce;
    const int r = p.n_q_heads / p.n_kv_heads;
    const int group_shift = p.group == 8 ? 3 : (p.group == 16 ? 4 : 5);
    hipLaunchKernelGGL((attend_few_kernel<D, kGather>),
                       dim3(p.batch * p.n_kv_heads * n_q_chunks * 2 * r), dim3(NW * 64),
                       FewLayout<D>::kBytes, stream, static_cast<const bf16_t*>(q_rot), q_chunk0,
                       n_q_chunks, static_cast<const bf16_t*>(k_res),
                       static_cast<const bf16_t*>(v_res), res_tokens, res_slot,
                       static_cast<bf16_t*>(k_routed), static_cast<bf16_t*>(v_routed), group_idx,
                       static_cast<bf16_t*>(out), lse, r, FastDiv(p.n_kv_heads),
                       FastDiv(n_q_chunks), FastDiv(2 * r), group_shift, p.keep_first,
                       recent_window(p), p.topk_groups, static_cast<const bf16_t*>(k_src),
                       static_cast<const bf16_t*>(v_src), src_tokens,
                       chunk_map(p.batch * p.n_q_heads, n_q_chunks, block_major),
                       chunk_map(p.batch * p.n_kv_heads, n_q_chunks, block_major));
    return hipGetLastError();
}

}  // namespace

// One workgroup per CU (the LDS of eight staging regions): launches that fit
// the chip once.
bool attend_few_applies(const hga_plan& plan, int n_q_chunks) {
    const hga_params& p = plan.p;
    const int64_t tiles = 2 * static_cast<int64_t>(p.batch) * p.n_q_heads * n_q_chunks;
    const int lds = p.head_dim == 64 ? FewLayout<64>::kBytes : FewLayout<128>::kBytes;
    return tiles <= plan.n_cu && lds <= plan.max_lds;
}

hipError_t launch_attend_few(const hga_plan& plan, const void* q_rot, int q_chunk0, int n_q_chunks,
                             const void* k_res, const void* v_res, int64_t res_tokens,
                             const int32_t* res_slot, void* k_routed, void* v_routed,
                             const int32_t* group_idx, void* out, float* lse, hipStream_t stream,
                             const void* k_src, const void* v_src, int64_t src_tokens,
                             bool block_major) {
    const bool d64 = plan.p.head_dim == 64, gather = k_src != nullptr;
    return (d64 ? (gather ? launch_few_t<64, true> : launch_few_t<64, false>)
                : (gather ? launch_few_t<128, true> : launch_few_t<128, false>))(
        plan, q_rot, q_chunk0, n_q_chunks, k_res, v_res, res_tokens, res_slot, k_routed, v_routed,
        group_idx, out, lse, stream, k_src, v_src, src_tokens, block_major);
}

}  // namespace hga
