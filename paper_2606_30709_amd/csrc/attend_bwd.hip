// Backward of the exact-token attention (Sec. 3.4, Eq. (1)) for bf16 inputs
// on the gfx950 matrix cores (v_mfma_f32_32x32x16_bf16).  Routing is not
// differentiated: the unit's working set (current chunk under the causal
// mask, visible chunks, routed groups) is the forward's.  For query row i and
// working-set key x, with s = q.k/sqrt(d), p = exp(s - lse_i) (the forward's
// log-sum-exp), D_i = dout_i . out_i:
//   dp = dout_i . v_x,  ds = p (dp - D_i),
//   dq_i = sum_x ds k_x / sqrt(d),  dk_x += sum_i ds q_i / sqrt(d),
//   dv_x += sum_i p dout_i.
// Routed rows are resident rows (group g, row o -> token g*G + o), so their
// key/value gradients land on those rows.
//
// Three kernels: row statistics (D_i, -lse), the key side (dK, dV) and dQ.
// The key side has two forms: chunk by chunk over the whole sequence
// or unit by unit (both in attend_bwd_keys.hip), where a workgroup takes one
// key tile of one unit, streams the unit's r*64 query rows past it and adds
// its gradients with atomics, 64*D*2 of them per tile: cheap when r*64 rows
// share them, the pace of the whole backward when r is small.
//
// A product's contraction index may be permuted as long as both operands use
// the same permutation: dQ's A operand is the lane's own dS^T column (keys in
// the order of the accumulator layout) and its B operand takes K^T in that
// same key order, by transpose reads of the row-major K tile.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>

#include "attend_bwd.hpp"
#include "attend_common.hpp"
#include "hga_internal.hpp"
#include "lds_copy.hpp"

namespace hga {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int KT = 64;    // keys per tile (= chunk)

__device__ __forceinline__ bf16x8_t frag(const bf16_t* p) {
    return __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const vec16*>(p));
}

typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;

__device__ __forceinline__ float add_halves(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false,
                                                    false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

constexpr int kXcds = 8;  // XCDs of the chip; workgroups are dealt to them in turn

// Logical work item of this workgroup: consecutive items on one XCD, so the
// workgroups of one unit (which read the same key tiles or query rows) share
// that XCD's L2.
__device__ __forceinline__ int xcd_item(int n_items) {
    const int per_xcd = (n_items + kXcds - 1) / kXcds;
    return (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
}

// dQ, query-major, on the forward's plan: 32-row query tiles, one wavefront
// each (KS = 1) or two that take one 32-key half of every key tile and add up
// at the end (KS = 2: one query head per KV head); a unit's key tiles (current
// chunk, visible chunks, routed rows gathered by group id) stream through two
// LDS stages, copied without registers.  Per 32-key sub-tile:
//   S^T = K.Q^T, dP^T - D = V.dO^T - D  (A = rows from LDS, B = registers)
//   dS^T = P (dP - D)                   (lane = query, registers = keys)
//   dQ^T += K^T.dS^T                    (A = transpose reads of the K rows)
// The contraction over keys is permuted alike in A and B, so dS goes from
// accumulators to operand in registers.
// Bound: vector work beside twelve (d64) matrix instructions per sub-tile and
// wavefront, like the forward's.  Three wavefronts per SIMD at d64: held to
// four it spills 9 VGPRs (8 x 12 heads x 12,288 tokens: 451 against 371 us; 9/3
// heads x 2,880: 31 against 24).  Staging rows through registers and K a second
// time, transposed by 16-bit writes, took 490 and 36 us there, and 1050
// against 936 us on 32/4 heads of d128 x 32,768 tokens.
template <int D>
struct DqLayout {
    static constexpr int kRow = D * 2;
    static constexpr int kTile = KT * kRow;         // K, then V
    static constexpr int kStage = 2 * kTile;
    static constexpr int kGid = 2 * kStage;
    static constexpr int kBytes = kGid + kMaxTopK * 4;
    static constexpr int kOutRow = 36;              // floats: 32 dimensions, padded
    static constexpr int kOut = 32 * kOutRow * 4;   // one wavefront's staging of the result
};

template <int D, int KS, int NW>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu(D == 64 ? 3 : 2)))
void attend_bwd_dq_kernel(
    const bf16_t* __restrict__ q_rot, int q_chunk0, int n_q_chunks, const bf16_t* __restrict__ k_res,
    const bf16_t* __restrict__ v_res, int64_t res_tokens, const int32_t* __restrict__ group_idx,
    const bf16_t* __restrict__ out, const float* __restrict__ lse,
    const bf16_t* __restrict__ dout, float* __restrict__ dq, int r, FastDiv kv_div, FastDiv wg_div,
    FastDiv chunk_div, int group_shift, int keep_first, int window, int topk_groups, int n_items) {
    using Lay = DqLayout<D>;
    constexpr int kRow = Lay::kRow;
    constexpr int kRowShift = D == 64 ? 7 : 8;
    constexpr int NKS = D / 16, NDT = D / 32;
    constexpr int QT = NW / KS;                   // query tiles per workgroup
    constexpr int KI = Lay::kTile / 1024 / NW;    // copies per wave and tile, for K (and V)
    static_assert(KI >= 1, "copy split");
    static_assert(KS == 1 || QT * (64 * NDT * 16 * 4 + Lay::kOut) <= Lay::kBytes, "merge area");
    static_assert(KS == 2 || QT * Lay::kOut <= Lay::kBytes, "output staging area");
    extern __shared__ __align__(16) unsigned char smem[];
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(smem));
    const int* s_gid = reinterpret_cast<const int*>(smem + Lay::kGid);

    const int item = xcd_item(n_items);
    if (item >= n_items) return;
    const int unit = wg_div.div(item), part = item - unit * wg_div.d;
    const int bh = chunk_div.div(unit), i = unit - bh * n_q_chunks;
    const int b = kv_div.div(bh), j = bh - b * kv_div.d;
    const int c = q_chunk0 + i;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = lane >> 5, col = lane & 31;
    const int qt_local = wave % QT, ksplit = wave / QT;
    const int qtile = part * QT + qt_local;
    const bool qactive = qtile < 2 * r;
    const int routed_rows = topk_groups << group_shift;
    const int lim = c * (KT >> group_shift);  // routed groups must lie in the causal past
    const float scale2 = 1.4426950408889634f / sqrtf(static_cast<float>(D));

    const u32x4 rk = rsrc_words(k_res + static_cast<int64_t>(bh) * res_tokens * D,
                                static_cast<uint32_t>(res_tokens * kRow));
    const u32x4 rv = rsrc_words(v_res + static_cast<int64_t>(bh) * res_tokens * D,
                                static_cast<uint32_t>(res_tokens * kRow));
    {
        const u32x4 rg = rsrc_words(group_idx + static_cast<int64_t>(unit) * topk_groups, topk_groups * 4);
        for (int u = wave; u * 64 < topk_groups; u += NW)
            copy4_to_lds(rg, (u * 64 + lane) * 4, lds0 + Lay::kGid + u * 256);
    }

    // the tile's first query row; B operands: the lane's row of Q and dO,
    // dimensions kk*16 + half*8 .. +7
    const int row_in_unit = (qactive ? qtile : 0) * 32;
    const int64_t row0 = (static_cast<int64_t>(b) * (r * kv_div.d) + j * r + row_in_unit / KT) *
                             (static_cast<int64_t>(n_q_chunks) * KT) +
                         static_cast<int64_t>(i) * KT + row_in_unit % KT;
    const int tq = qtile & 1;  // half of the chunk the tile's tokens lie in
    bf16x8_t qf[NKS], gf[NKS];
    float nd = 0.f, nl = 0.f;  // -D_i, -lse (log2)
    {
        const int64_t at = (row0 + col) * D + half * 8;
#pragma unroll
        for (int kk = 0; kk < NKS; ++kk) {
            const vec16 g = load16(dout + at + kk * 16), o = load16(out + at + kk * 16);
            qf[kk] = frag(q_rot + at + kk * 16);
            gf[kk] = __builtin_bit_cast(bf16x8_t, g);
#pragma unroll
            for (int e = 0; e < 8; ++e) nd = fmaf(-bf16_value(g, e), bf16_value(o, e), nd);
        }
        nd = add_halves(nd);
        nl = lse[row0 + col] * -1.4426950408889634f;
    }

    const VisibleChunks vis(c, keep_first, window);
    const int n_vis = vis.count;
    const int n_tiles = 1 + n_vis + (routed_rows + KT - 1) / KT;
    uint32_t koff[KI];  // this lane's source offset in each copy of a tile
#pragma unroll
    for (int u = 0; u < KI; ++u) {
        const int slot = (u * NW + wave) * 64 + lane, row = slot / (D / 8);
        koff[u] = row * kRow + ((slot % (D / 8)) ^ swz_rows<D>(row)) * 16;
    }
    auto issue = [&](int tile, int stage) {
        uint32_t src[KI];
        if (tile <= n_vis) {
            const uint32_t base = static_cast<uint32_t>((tile == 0 ? c : vis.chunk(tile - 1)) * Lay::kTile);
#pragma unroll
            for (int u = 0; u < KI; ++u) src[u] = base + koff[u];
        } else {
            // row R of the tile is row R % G of the group in slot R / G
            const int slot0 = ((tile - 1 - n_vis) * KT) >> group_shift;
            const int sh = group_shift + kRowShift;
            int g[KI];
#pragma unroll
            for (int u = 0; u < KI; ++u)
                g[u] = s_gid[min(slot0 + static_cast<int>(koff[u] >> sh), topk_groups - 1)];
#pragma unroll
            for (int u = 0; u < KI; ++u) {
                const bool ok = slot0 + static_cast<int>(koff[u] >> sh) < topk_groups &&
                                static_cast<uint32_t>(g[u]) < static_cast<uint32_t>(lim);
                src[u] = ok ? (static_cast<uint32_t>(g[u]) << sh) + (koff[u] & ((1u << sh) - 1)) : kAbsent;
            }
        }
        const uint32_t at = lds0 + stage * Lay::kStage;
#pragma unroll
        for (int u = 0; u < KI; ++u) copy16_to_lds(rk, src[u], at + (u * NW + wave) * 1024);
#pragma unroll
        for (int u = 0; u < KI; ++u) copy16_to_lds(rv, src[u], at + Lay::kTile + (u * NW + wave) * 1024);
    };
    issue(0, 0);

    f32x16_t acc[NDT];  // dQ^T: lane = query, dimension dt*32 + (e/4)*8 + half*4 + e%4
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[dt][e] = 0.f;
    // LDS offsets of this lane's reads; the swizzle repeats every 16 rows, so
    // rows further on are immediates
    int aoff[NKS], toff[2][NDT];
#pragma unroll
    for (int kk = 0; kk < NKS; ++kk) aoff[kk] = col * kRow + (((2 * kk + half) ^ swz_rows<D>(col)) * 16);
#pragma unroll
    for (int x = 0; x < 2; ++x)
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
            const int row = x * 8 + half * 4 + ((lane & 15) >> 2);
            const int ch = dt * 4 + ((lane >> 4) & 1) * 2 + ((lane & 3) >> 1);
            toff[x][dt] = row * kRow + ((ch ^ swz_rows<D>(row)) * 16) + (lane & 1) * 8;
        }

    for (int tile = 0; tile < n_tiles; ++tile) {
        wait_copies<0>();
        lds_barrier();  // the tile is here; everybody has left the other stage
        if (tile + 1 < n_tiles) issue(tile + 1, (tile + 1) & 1);
        if (!qactive) continue;
        const unsigned char* base = smem + (tile & 1) * Lay::kStage;
        // routed rows to leave out: lane g checks the tile's g-th group
        bool partial = false;
        const int rt0 = (tile - 1 - n_vis) * KT;
        if (tile > n_vis) {
            bool bad = false;
            if (lane < (KT >> group_shift)) {
                const int g = (rt0 >> group_shift) + lane;
                bad = g >= topk_groups || static_cast<uint32_t>(s_gid[min(g, topk_groups - 1)]) >=
                                              static_cast<uint32_t>(lim);
            }
            partial = __builtin_amdgcn_ballot_w64(bad) != 0;
        }
#pragma unroll
        for (int x = 0; x < 2 / KS; ++x) {
            const int st = KS == 2 ? ksplit : x;
            if (tile == 0 && st > tq) continue;  // the later half of the current chunk
            const unsigned char* kb = base + st * 32 * kRow;
            f32x16_t s, p;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                s[e] = 0.f;
                p[e] = nd;
            }
#pragma unroll
            for (int kk = 0; kk < NKS; ++kk) {
                s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    __builtin_bit_cast(bf16x8_t, load16(kb + aoff[kk])), qf[kk], s, 0, 0, 0);
                p = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                    __builtin_bit_cast(bf16x8_t, load16(kb + Lay::kTile + aoff[kk])), gf[kk], p, 0, 0, 0);
            }
            if (tile == 0 && st == tq) {
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    s[e] = (e >> 2) * 8 + half * 4 + (e & 3) > col ? -INFINITY : s[e];
            } else if (partial) {
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int g = (rt0 + st * 32 + (e >> 2) * 8 + half * 4 + (e & 3)) >> group_shift;
                    const bool ok = g < topk_groups && static_cast<uint32_t>(s_gid[min(g, topk_groups - 1)]) <
                                                           static_cast<uint32_t>(lim);
                    s[e] = ok ? s[e] : -INFINITY;
                }
            }
            bf16x8_t ds[2];
#pragma unroll
            for (int e = 0; e < 16; ++e)
                ds[e >> 3][e & 7] = static_cast<__bf16>(
                    __builtin_amdgcn_exp2f(fmaf(s[e], scale2, nl)) * p[e]);
            // k-slot half*8 + e of block kap is key kap*16 + (e/4)*8 + half*4 + e%4
#pragma unroll
            for (int kap = 0; kap < 2; ++kap)
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt) {
                    auto tr = [&](int off) {
                        return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                            (lds_i16x4_t*)(reinterpret_cast<uintptr_t>(kb + kap * 16 * kRow + off)));
                    };
                    const bf16x8_t a = __builtin_bit_cast(
                        bf16x8_t, __builtin_shufflevector(tr(toff[0][dt]), tr(toff[1][dt]), 0, 1, 2, 3, 4, 5, 6, 7));
                    acc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, ds[kap], acc[dt], 0, 0, 0);
                }
        }
    }

    lds_barrier();  // the stages are free
    float* stage = reinterpret_cast<float*>(smem + qt_local * Lay::kOut);
    if (KS == 2) {
        float* other = reinterpret_cast<float*>(smem + QT * Lay::kOut) + qt_local * (NDT * 16 * 64) + lane;
        if (ksplit == 1) {
#pragma unroll
            for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
                for (int e = 0; e < 16; ++e) other[(dt * 16 + e) * 64] = acc[dt][e];
        }
        lds_barrier();
        if (ksplit == 1) return;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[dt][e] += other[(dt * 16 + e) * 64];
    }
    if (!qactive) return;
    // 32 dimensions at a time through the wavefront's LDS rows, so that every
    // store instruction writes whole 128-byte pieces of eight rows
    const float inv_sqrt_d = 1.0f / sqrtf(static_cast<float>(D));
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt) {
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *reinterpret_cast<float4*>(stage + col * Lay::kOutRow + g * 8 + half * 4) =
                make_float4(acc[dt][g * 4] * inv_sqrt_d, acc[dt][g * 4 + 1] * inv_sqrt_d,
                            acc[dt][g * 4 + 2] * inv_sqrt_d, acc[dt][g * 4 + 3] * inv_sqrt_d);
        __builtin_amdgcn_wave_barrier();
        lds_reads_done();  // (writes too: the wavefront's own)
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int row = it * 8 + (lane >> 3), cc = lane & 7;
            const vec16 x = *reinterpret_cast<const vec16*>(stage + row * Lay::kOutRow + cc * 4);
            __builtin_nontemporal_store(__builtin_bit_cast(u32x4, x),
                                        reinterpret_cast<u32x4*>(dq + (row0 + row) * D + dt * 32 + cc * 4));
        }
        __builtin_amdgcn_wave_barrier();
        lds_reads_done();
    }
}

// Before the unit-by-unit key side: the row statistics, and (n > 0) zeros over
// n 16-byte vectors of dk and of dv (a kernel, not a memset: the call may be
// captured into a graph).
template <int D>
__global__ __launch_bounds__(256) void attend_bwd_begin_kernel(
    const bf16_t* __restrict__ out, const bf16_t* __restrict__ dout, const float* __restrict__ lse,
    float* __restrict__ stat, int64_t rows, int stat_blocks, float4* __restrict__ dk,
    float4* __restrict__ dv, int64_t n) {
    const int block = blockIdx.x;
    if (block < stat_blocks) {
        bwd_row_stat<D>(out, dout, lse, stat, rows, static_cast<int64_t>(block) * 256 + threadIdx.x);
        return;
    }
    const int64_t at = static_cast<int64_t>(block - stat_blocks) * 1024 + threadIdx.x;
#pragma unroll
    for (int u = 0; u < 4; ++u)
        if (at + u * 256 < n) dk[at + u * 256] = dv[at + u * 256] = make_float4(0.f, 0.f, 0.f, 0.f);
}

// Whether the key side goes chunk by chunk, wherever its lists fit: by the
// pace of each form.  Unit by unit, a tile costs its atomics (8 at d64, 13 at
// d128, in units of 3 and 4 ns of the chip) and one per query head; chunk by
// chunk, a (unit, chunk) entry costs its query rows (1.13 and 1.75 a query
// head), and the lists and their longer launch about 25 us more.  Whole
// backward, unit by unit / chunk by chunk, us, groups of 16 (8), about 0.6
// chunks a group:
//   d64, 2 x 160 chunks, K_g 12: 2 heads 92 / 91, 4 heads 105 / 112, 8 heads
//   130 / 148; K_g 48: 1 head 168 / 104, 4 heads 202 / 191, 8 heads 234 / 297;
//   8 x 192, K_g 12: 4 heads 410 / 290; 4 x 512, K_g 48: 4 heads 1065 / 902, 8
//   heads 1352 / 1756; 2 x 45 (8), K_g 19: 2 heads 36 / 48, 4 heads 39 / 67;
//   6 x 45 (8), K_g 19 of 5 chunks: 3 heads 77 / 66.
//   d128, 2 x 160, K_g 12: 2 heads 171 / 172, 4 heads 198 / 217; K_g 48: 2
//   heads 342 / 232, 4 heads 383 / 356, 6 heads 437 / 527, 8 heads 465 / 604;
//   4 x 512, K_g 48: 4 heads 2157 / 1869, 8 heads 2796 / 3633; 1 x 50, K_g 12:
//   2 heads 42 / 50, 4 heads 47 / 71.
// Every key chunk of the range has a place in the lists, whether anybody
// attends it or not: 0.2 units of the rule for its counter and its workgroup,
// which count where few query chunks follow a long history.  One query head,
// K_g 12, adding: 64 (batch, KV head) pairs x 2 chunks after 3,000 of d128 60 /
// 123, x 8 190 / 230 (d64 100 / 130), x 32 725 / 659 (d64 376 / 347); 12 pairs x
// 16 after 4,000 81 / 78 (d64 46 / 50), x 1 after 2,000 23 / 35.  Longer launch
// (8500): not for one head, where the forms are equal in small launches and
// the lists ahead from there on.
bool by_chunk(const hga_plan& plan, int q_chunk0, int n_q_chunks, int fixed, int tiles) {
    const hga_params& p = plan.p;
    const int r = p.n_q_heads / p.n_kv_heads;
    const double pairs = static_cast<double>(p.batch) * p.n_kv_heads;
    const double units = pairs * n_q_chunks;
    const double entries = units * (fixed + std::min(p.topk_chunks, p.topk_groups));
    const double by_unit = units * tiles * ((p.head_dim == 64 ? 8 : 13) + r);
    const double chunks = entries * r * (p.head_dim == 64 ? 1.13 : 1.75) +
                          pairs * (static_cast<double>(q_chunk0) + n_q_chunks) * 0.2 +
                          (r == 1 ? 0 : 8500);
    return chunks <= by_unit && bwd_chunks_fit(plan, q_chunk0, n_q_chunks);
}

template <int D, int KS, int NW>
hipError_t launch_bwd_t(const hga_plan& plan, const void* q_rot, int q_chunk0, int n_q_chunks,
                        const void* k_res, const void* v_res, int64_t res_tokens,
                        const int32_t* group_idx, const void* out, const float* lse,
                        const void* dout, float* dq, float* dk, float* dv, bool write,
                        hipStream_t stream) {
    const hga_params& p = plan.p;
    static std::atomic<uint64_t> configured{0};  // per instantiation and device
    const hipError_t ce = once_per_device(configured, plan.device, [] {
        return hipFuncSetAttribute(reinterpret_cast<const void*>(&attend_bwd_dq_kernel<D, KS, NW>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize, DqLayout<D>::kBytes);
    });
    if (ce != hipSuccess) return ce;
    const int r = p.n_q_heads / p.n_kv_heads;
    const int group_shift = p.group == 8 ? 3 : (p.group == 16 ? 4 : 5);
    const int window = recent_window(p);
    const int64_t units = static_cast<int64_t>(p.batch) * p.n_kv_heads * n_q_chunks;
    const int wg_per_unit = (2 * r * KS + NW - 1) / NW;
    const int64_t items_dq = units * wg_per_unit;
    if (items_dq > (int64_t(1) << 30)) return hipErrorInvalidConfiguration;
    auto grid = [](int64_t n) { return dim3(static_cast<unsigned>((n + kXcds - 1) / kXcds * kXcds)); };
    // The statistics go to the leading floats of dq, which the dq kernel
    // (last) overwrites: no workspace of its own.
    const int64_t rows = static_cast<int64_t>(p.batch) * p.n_q_heads * n_q_chunks * KT;
    float* stat = dq;
    hipError_t e;
    // tiles of the largest working set: the last chunk's visible chunks
    const int fixed = 1 + VisibleChunks(q_chunk0 + n_q_chunks - 1, p.keep_first, window).count;
    const int tiles = fixed + (p.topk_groups * p.group + KT - 1) / KT;
    if (by_chunk(plan, q_chunk0, n_q_chunks, fixed, tiles)) {
        e = launch_bwd_chunks(plan, q_rot, q_chunk0, n_q_chunks, k_res, v_res, res_tokens,
                              group_idx, out, lse, dout, dq, dk, dv, write, stream);
    } else {
        const int64_t n = write ? static_cast<int64_t>(p.batch) * p.n_kv_heads * res_tokens * (D / 4) : 0;
        const int64_t stat_blocks = (rows * 8 + 255) / 256, zero_blocks = (n + 1023) / 1024;
        if (stat_blocks + zero_blocks > (int64_t(1) << 30)) return hipErrorInvalidConfiguration;
        hipLaunchKernelGGL((attend_bwd_begin_kernel<D>),
                           dim3(static_cast<unsigned>(stat_blocks + zero_blocks)), dim3(256), 0,
                           stream, static_cast<const bf16_t*>(out),
                           static_cast<const bf16_t*>(dout), lse, stat, rows,
                           static_cast<int>(stat_blocks), reinterpret_cast<float4*>(dk),
                           reinterpret_cast<float4*>(dv), n);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
        e = launch_bwd_units(plan, q_rot, q_chunk0, n_q_chunks, k_res, v_res, res_tokens, group_idx,
                             stat, dout, dk, dv, tiles, stream);
    }
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((attend_bwd_dq_kernel<D, KS, NW>), grid(items_dq), dim3(NW * 64),
                       DqLayout<D>::kBytes, stream, static_cast<const bf16_t*>(q_rot), q_chunk0,
                       n_q_chunks, static_cast<const bf16_t*>(k_res), static_cast<const bf16_t*>(v_res),
                       res_tokens, group_idx, static_cast<const bf16_t*>(out), lse,
                       static_cast<const bf16_t*>(dout), dq, r, FastDiv(p.n_kv_heads),
                       FastDiv(wg_per_unit), FastDiv(n_q_chunks), group_shift, p.keep_first,
                       window, p.topk_groups, static_cast<int>(items_dq));
    return hipGetLastError();
}

}  // namespace

size_t attend_backward_lds_bytes(const hga_plan& plan) {
    const size_t dq = plan.p.head_dim == 64 ? DqLayout<64>::kBytes : DqLayout<128>::kBytes;
    return std::max(dq, bwd_chunks_lds_bytes(plan));
}

hipError_t launch_attend_backward(const hga_plan& plan, const void* q_rot, int q_chunk0,
                                  int n_q_chunks, const void* k_res, const void* v_res,
                                  int64_t res_tokens, const int32_t* group_idx, const void* out,
                                  const float* lse, const void* dout, float* dq, float* dk,
                                  float* dv, bool write, hipStream_t stream) {
    const hga_params& p = plan.p;
    const int r = p.n_q_heads / p.n_kv_heads;
#define HGA_BWD(DD, KK, NN)                                                                        \
    return launch_bwd_t<DD, KK, NN>(plan, q_rot, q_chunk0, n_q_chunks, k_res, v_res, res_tokens,  \
                                    group_idx, out, lse, dout, dq, dk, dv, write, stream)
    // The dq kernel's shape: two wavefronts per query tile for one query head
    // per KV head (two tiles a unit), and where one wavefront per tile would
    // leave compute units without a workgroup (whole backward, one KV head: 2
    // heads x 20 chunks of d64 33 -> 30 us, 4 x 50 66 -> 55, 4 x 100 of d128
    // 101 -> 85; at 200 workgroups of d128 equal).
    const int64_t units = static_cast<int64_t>(p.batch) * p.n_kv_heads * n_q_chunks;
    const int tiles = p.head_dim == 64 ? 4 : 8;  // per workgroup, one wavefront each
    if (r == 1 || units * ((2 * r + tiles - 1) / tiles) < plan.n_cu) {
        if (p.head_dim == 64) HGA_BWD(64, 2, 4);
        HGA_BWD(128, 2, 4);
    }
    if (p.head_dim == 64) HGA_BWD(64, 1, 4);
    HGA_BWD(128, 1, 8);
#undef HGA_BWD
}

}  // namespace hga
