// The split form of the exact-token attention (Sec. 3.4, Eq. (1)) for bf16
// launches of a few units (a decode block, one block of a block-sequential
// prefill, all blocks of a prompt) on the gfx950 matrix cores
// (v_mfma_f32_32x32x16_bf16), without partial results in memory and without a
// second launch for the merge.
//
// A workgroup takes one 32-row query tile of one (batch, KV head, query chunk)
// and all of its keys; a wavefront takes one split, the same run of key tiles
// that a workgroup of the split form takes, 32 keys at a time, with its own
// online softmax, output accumulator and LDS staging (no barrier).  The
// partial results meet in LDS, eight at a time, in the order of the splits.
// Every operation on a value is the split form's (attend_mfma.hip: the moving
// reference point, the order of the sums, the merge), so out and lse are the
// split form's bit for bit and the choice between the two is one of speed.
//   S^T[key][query] = K.Q^T    (A = K rows, B = Q in registers)
//   O^T[d][query]  += V^T.P^T  (A = transpose reads of V rows, B = the lane's P)
// K(t+1) is copied while P.V(t) runs and V(t+1) while S(t+1) runs.
//
// Bound: latency, then the keys' way into one CU (64 bytes per clock: 4 us for
// the 608 KB of a 64K decode block's 19 tiles of d128).  For the four units of
// that block (ten splits) the split form's 80 workgroups move less per CU but
// leave 10.6 MB of fp32 partial results for a second kernel: 19.0 us, against
// 15.6 here.
#include <hip/hip_runtime.h>
#include <math.h>

#include "attend_common.hpp"
#include "hga_internal.hpp"
#include "lds_copy.hpp"

namespace hga {
namespace {

constexpr int KT = 64;  // tokens per chunk
constexpr int ST = 32;  // keys per sub-tile
constexpr int kRound = 8;  // partial results in LDS at a time

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;
typedef float f32x16_t __attribute__((ext_vector_type(16)));

template <int D>
struct FewLayout {
    static constexpr int kRow = D * 2;
    static constexpr int kV = ST * kRow;               // V after K
    static constexpr int kWave = 2 * ST * kRow;        // bytes per wavefront
    // the merge reuses all of it: kRound x 32 output rows, then (m, l) of
    // every split and row
    static constexpr int kOutRow = D + 4;              // floats, padded against bank conflicts
    static constexpr int kPart = ST * kOutRow * 4;
    static constexpr int kMl = kRound * kPart;
    static constexpr int kMerge = kMl + kMaxSplit * ST * 8;
    static constexpr int bytes(int waves) {
        return waves * kWave > kMerge ? waves * kWave : kMerge;
    }
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

// NW: most wavefronts of a workgroup; NP: splits a wavefront may take, one
// after the other.  n_split: the call's splits, or (per_unit, a launch of many
// query chunks each standing for a call of its own) the most a unit has, with
// at least two tiles each.
// kGather: the routed rows come from k_src / v_src by group id and, when
// k_routed / v_routed are given, are written there (the unit's query tiles
// share the writing); otherwise they are read from k_routed / v_routed.
template <int D, int NW, int NP, bool kGather>
__global__ __launch_bounds__(NW * 64) __attribute__((amdgpu_waves_per_eu((NW + 3) / 4)))
void attend_few_kernel(
    const bf16_t* __restrict__ q_rot, int q_chunk0, int n_q_chunks,
    const bf16_t* __restrict__ k_res, const bf16_t* __restrict__ v_res, int64_t res_tokens,
    const int32_t* __restrict__ res_slot, bf16_t* __restrict__ k_routed,
    bf16_t* __restrict__ v_routed, const int32_t* __restrict__ group_idx,
    bf16_t* __restrict__ out, float* __restrict__ lse, int r, FastDiv kv_div, FastDiv chunk_div,
    FastDiv tile_div, int group_shift, int keep_first, int window, int topk_groups,
    const bf16_t* __restrict__ k_src, const bf16_t* __restrict__ v_src, int64_t src_tokens,
    ChunkMap q_map, ChunkMap unit_map, int n_split, int per_unit, int n_blocks) {
    using Lay = FewLayout<D>;
    constexpr int kRow = Lay::kRow;
    constexpr int CPR = D / 8;             // 16-byte chunks per row
    constexpr int RPC = 64 / CPR;          // rows per copy
    constexpr int CU = ST / RPC;           // copies per sub-tile, for K (and V)
    constexpr int NKS = D / 16, NDT = D / 32;
    extern __shared__ __align__(16) unsigned char smem[];

    const int block = static_cast<int>(linear_block<NW * 64>());
    if (block >= n_blocks) return;
    const int item = tile_div.div(block);
    const int qtile = block - item * tile_div.d;
    const int bh = chunk_div.div(item);
    const int i = item - bh * n_q_chunks;
    const int64_t unit = unit_map.at(bh, i);
    const int b = kv_div.div(bh), j = bh - b * kv_div.d;
    const int c = q_chunk0 + i;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_waves = blockDim.x >> 6;
    const int half = lane >> 5, col = lane & 31;
    unsigned char* const mine = smem + wave * Lay::kWave;
    const uint32_t lds0 = static_cast<uint32_t>(reinterpret_cast<uintptr_t>(mine));
    // the unit's group ids and the slot map, read by scalar loads (they do not
    // count among the copies that the waits below count)
    typedef const int32_t __attribute__((address_space(4))) * const_ids;
    const const_ids ids = (const_ids)(reinterpret_cast<uintptr_t>(group_idx + unit * topk_groups));
    const const_ids slots = (const_ids)(reinterpret_cast<uintptr_t>(res_slot));

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

    const VisibleChunks vis(c, keep_first, window);
    const int n_fixed = 2 * (1 + vis.count);  // sub-tiles of the current and visible chunks
    const int n_sub = n_fixed + (routed_rows + ST - 1) / ST;
    const int n_tiles = (n_sub + 1) >> 1;
    const int ns = per_unit ? min(n_split, (n_tiles + 1) >> 1) : n_split;
    bool bad = false;
    const int crow = lane / CPR;  // row of this lane's slot within a copy
    // 16-byte chunk it takes of its row, unswizzled at the source: the swizzle
    // is linear over xor, so copy u's differs by a constant (as do the LDS
    // offsets below); `fresh` keeps the compiler from holding one register for
    // each of them across the loop
    const uint32_t koff0 = ((lane % CPR) ^ swz_rows<D>(crow)) * 16;
    auto koff = [&](int u) { return koff0 ^ (swz_rows<D>(u * RPC) * 16); };

    // Sub-tile `sub`: lane (any half, col) finds where row col of it starts
    // in its source (kAbsent: a row that reads zeros).
    uint32_t row_at = 0;
    int gid[4] = {-1, -1, -1, -1};  // the groups of the sub-tile to be located
    auto read_ids = [&](int sub) {
        if (sub < n_fixed) return;
        const int slot = ((sub - n_fixed) * ST) >> group_shift;
#pragma unroll
        for (int x = 0; x < 4; ++x) gid[x] = ids[min(slot + x, topk_groups - 1)];
    };
    auto locate = [&](int sub) {
        if (sub < n_fixed) {
            const int cc = sub < 2 ? c : vis.chunk((sub >> 1) - 1);
            const int64_t slot = res_slot ? slots[cc] : cc;
            const bool ok = slot >= 0 && slot < res_chunks;
            bad |= !ok;
            row_at = ok ? static_cast<uint32_t>(slot * KT + (sub & 1) * ST + col) * kRow : kAbsent;
        } else {
            const int row = (sub - n_fixed) * ST + col;
            const int x = col >> group_shift;
            const int g = x == 0 ? gid[0] : x == 1 ? gid[1] : x == 2 ? gid[2] : gid[3];
            const bool ok = row < routed_rows && g >= 0 && g < id_limit;
            const int at = kGather ? (g << group_shift) + (row & ((1 << group_shift) - 1)) : row;
            row_at = ok ? static_cast<uint32_t>(at) * kRow : kAbsent;
        }
    };
    auto copy_rows = [&](const u32x4& rs, uint32_t lds) {
        asm volatile("" : "+s"(lds));
#pragma unroll
        for (int u = 0; u < CU; ++u)
            copy16_to_lds(rs, __shfl(row_at, u * RPC + crow) + koff(u), lds + u * 1024);
    };
    auto copy_k = [&](int sub) { copy_rows(sub < n_fixed ? rk_res : rk_rt, lds0); };
    auto copy_v = [&](int sub) { copy_rows(sub < n_fixed ? rv_res : rv_rt, lds0 + Lay::kV); };

    // B operand of S^T: the lane's query row, dimensions kk*16 + half*8 ..
    bf16x8_t qf[NKS];
#pragma unroll
    for (int kk = 0; kk < NKS; ++kk)
        qf[kk] = __builtin_bit_cast(bf16x8_t, load16(q_rot + (row0 + col) * D + half * 8 + kk * 16));

    // LDS offsets of this lane's reads: fragment kk of its K row at
    // aoff0 ^ kk*32; V rows x*8 + half*4 + .., dimensions dt*32 + .. at
    // (toff0 ^ dt*64 ^ x*48) + x*8 rows (rows 16 further on are immediates)
    const int aoff0 = col * kRow + ((half ^ swz_rows<D>(col)) * 16);
    const int trow = half * 4 + ((lane & 15) >> 2);
    const int toff0 = trow * kRow +
                      (((((lane >> 4) & 1) * 2 + ((lane & 3) >> 1)) ^ swz_rows<D>(trow)) * 16) +
                      (lane & 1) * 8;
    auto fresh = [](int x) {
        asm volatile("" : "+v"(x));
        return x;
    };
    // this lane's slots of a staged routed sub-tile to the unit's rows of a
    // routed buffer (past its end they are dropped), two at a time (registers)
    auto write_rows = [&](int rs, const unsigned char* staged, bf16_t* dst) {
        const buf_rsrc to = make_rsrc(dst + unit * routed_rows * D, routed_rows * kRow);
#pragma unroll 2
        for (int u = 0; u < CU; ++u) {
            const vec16 x = *reinterpret_cast<const vec16*>(staged + u * 1024 + lane * 16);
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, x), to,
                                                   (rs * ST + u * RPC + crow) * kRow + koff(u), 0,
                                                   2 /* non-temporal */);
        }
    };
    const int n_qt = tile_div.d;

    // the wavefront's splits: sums and statistics of the last one in oacc,
    // m_run, l_run, of an earlier one in held*
    f32x16_t oacc[NDT], held[NP == 2 ? NDT : 1];
    float m_run = -INFINITY, l_run = 0.f, m_held = -INFINITY, l_held = 0.f;  // m in log2 units
#pragma unroll 1
    for (int pass = 0; pass < NP; ++pass) {
        if constexpr (NP == 2) {
            if (pass == 1) {
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt) held[dt] = oacc[dt];
                m_held = m_run;
                l_held = bad ? NAN : xor32_add(l_run);
                m_run = -INFINITY;
                l_run = 0.f;
            }
        }
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
            for (int e = 0; e < 16; ++e) oacc[dt][e] = 0.f;
        const int split = pass * NW + wave;
        int sub = 0, end = 0;
        if (split < ns) {
            sub = 2 * ((split * n_tiles + ns - 1) / ns);
            end = min(2 * (((split + 1) * n_tiles + ns - 1) / ns), n_sub);
        }
        if (sub < end) {
            read_ids(sub);
            locate(sub);
            copy_k(sub);
            copy_v(sub);
        }
        for (; sub < end; ++sub) {
            const int next = sub + 1;
            if (next < end) read_ids(next);
            // keys of this sub-tile that count, one bit each (uniform)
            uint32_t live = static_cast<uint32_t>(__builtin_amdgcn_ballot_w64(row_at < kAbsent));
            if (sub < 2 && sub > tq) live = 0;  // the later half of the current chunk
            const int rs = sub - n_fixed;
            const bool write = kGather && k_routed != nullptr && rs >= 0 && rs % n_qt == qtile;
            wait_copies<CU>();  // K is here; V may be in flight
            if (write) write_rows(rs, mine, k_routed);
            f32x16_t s;
#pragma unroll
            for (int e = 0; e < 16; ++e) s[e] = 0.f;
            if (live) {
                const int aoff = fresh(aoff0);
#pragma unroll
                for (int kk = 0; kk < NKS; ++kk)
                    s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        __builtin_bit_cast(bf16x8_t, load16(mine + (aoff ^ (kk * 32)))), qf[kk], s, 0, 0, 0);
            }
            lds_reads_done();  // before the next K lands on this one
            if (next < end) {
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
            if (next < end && !write)
                wait_copies<CU>();
            else
                wait_copies<0>();
            if (write) write_rows(rs, mine + Lay::kV, v_routed);
            if (live) {
                const int toff = fresh(toff0);
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
                            bf16x8_t, __builtin_shufflevector(tr(toff ^ (dt * 64)),
                                                              tr((toff ^ (dt * 64 + 48)) + 8 * kRow),
                                                              0, 1, 2, 3, 4, 5, 6, 7));
                        oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pf[kap], oacc[dt], 0, 0, 0);
                    }
            }
            lds_reads_done();
            if (next < end) copy_v(next);
        }
    }

    // The merge (the split form's): weights exp2(m_s - M) against the largest
    // reference point, the sums in the order of the splits; kRound partial
    // results in LDS at a time, the others wait in registers.
    wait_copies<0>();
    __syncthreads();  // the staging is free
    auto put = [&](int split, const f32x16_t(&o)[NDT]) {
        float* part = reinterpret_cast<float*>(smem + (split % kRound) * Lay::kPart) + col * Lay::kOutRow + half * 4;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
            for (int g4 = 0; g4 < 4; ++g4)
                *reinterpret_cast<float4*>(part + dt * 32 + g4 * 8) =
                    make_float4(o[dt][g4 * 4], o[dt][g4 * 4 + 1], o[dt][g4 * 4 + 2], o[dt][g4 * 4 + 3]);
    };
    auto put_round = [&](int round) {
        if constexpr (NP == 2) {
            static_assert(NP == 1 || NW == kRound, "a round is a pass");
            if (round == 0)
                put(wave, held);
            else
                put(wave, oacc);
        } else if (wave / kRound == round) {
            put(wave, oacc);
        }
    };
    float2* const s_ml = reinterpret_cast<float2*>(smem + Lay::kMl);
    put_round(0);
    {
        const float l_tot = bad ? NAN : xor32_add(l_run);
        if (half == 0) {
            s_ml[((NP - 1) * NW + wave) * ST + col] = make_float2(m_run, l_tot);
            if (NP == 2) s_ml[wave * ST + col] = make_float2(m_held, l_held);
        }
    }
    __syncthreads();
    // eight dimensions of one row per thread; more than one round only with
    // enough threads for all rows at once
    const int n_threads = n_waves * 64;
    for (int it0 = 0; it0 < ST * CPR; it0 += n_threads) {
        const int it = it0 + tid;
        const bool active = it < ST * CPR;
        const int row = active ? it / CPR : 0, cc = it % CPR;
        // (every slot is read at once; those past the last split are not used)
        float top[kMaxSplit], m = -INFINITY;
#pragma unroll
        for (int w = 0; w < kMaxSplit; ++w) top[w] = s_ml[w * ST + row].x;
#pragma unroll
        for (int w = 0; w < kMaxSplit; ++w) m = w < ns ? fmaxf(m, top[w]) : m;
        float l = 0.f, o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int w0 = 0; w0 < ns; w0 += kRound) {
            if (w0 > 0) {
                __syncthreads();
                put_round(w0 / kRound);
                __syncthreads();
            }
            float2 ml[kRound];
            float4 x[kRound][2];
#pragma unroll
            for (int w = 0; w < kRound; ++w) {
                ml[w] = s_ml[(w0 + w) * ST + row];
                const float4* v = reinterpret_cast<const float4*>(
                    smem + w * Lay::kPart + (row * Lay::kOutRow + cc * 8) * 4);
                x[w][0] = v[0];
                x[w][1] = v[1];
            }
#pragma unroll
            for (int w = 0; w < kRound; ++w) {
                if (w0 + w >= ns) break;
                const float f = __builtin_amdgcn_exp2f(ml[w].x - m);
                l = fmaf(ml[w].y, f, l);
                o[0] = fmaf(x[w][0].x, f, o[0]);
                o[1] = fmaf(x[w][0].y, f, o[1]);
                o[2] = fmaf(x[w][0].z, f, o[2]);
                o[3] = fmaf(x[w][0].w, f, o[3]);
                o[4] = fmaf(x[w][1].x, f, o[4]);
                o[5] = fmaf(x[w][1].y, f, o[5]);
                o[6] = fmaf(x[w][1].z, f, o[6]);
                o[7] = fmaf(x[w][1].w, f, o[7]);
            }
        }
        if (!active) continue;
        const float inv = __builtin_amdgcn_rcpf(l);
        bf16x8_t v;
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = static_cast<__bf16>(o[e] * inv);
        *reinterpret_cast<bf16x8_t*>(out + (row0 + row) * D + cc * 8) = v;
        if (lse && cc == 0) lse[row0 + row] = (m + log2f(l)) * 0.6931471805599453f;
    }
}

// A launch shape: wavefronts of a workgroup at most, and splits of each.
template <int D, int NW, int NP, bool kGather>
hipError_t launch_few_t(const hga_plan& plan, const void* q_rot, int q_chunk0, int n_q_chunks,
                        const void* k_res, const void* v_res, int64_t res_tokens,
                        const int32_t* res_slot, void* k_routed, void* v_routed,
                        const int32_t* group_idx, void* out, float* lse, int n_split,
                        hipStream_t stream, const void* k_src, const void* v_src,
                        int64_t src_tokens, bool block_major) {
    const hga_params& p = plan.p;
    static std::atomic<uint64_t> configured{0};  // per instantiation and device
    const hipError_t ce = once_per_device(configured, plan.device, [] {
        return hipFuncSetAttribute(
            reinterpret_cast<const void*>(&attend_few_kernel<D, NW, NP, kGather>),
            hipFuncAttributeMaxDynamicSharedMemorySize, FewLayout<D>::bytes(NW));
    });
    if (ce != hipSuccess) return ce;
    const int r = p.n_q_heads / p.n_kv_heads;
    const int group_shift = p.group == 8 ? 3 : (p.group == 16 ? 4 : 5);
    const int waves = n_split < NW ? n_split : NW;
    const int64_t blocks = static_cast<int64_t>(p.batch) * p.n_kv_heads * n_q_chunks * 2 * r;
    if (blocks > (int64_t(1) << 30)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((attend_few_kernel<D, NW, NP, kGather>), grid_of(blocks, NW * 64),
                       dim3(waves * 64),
                       FewLayout<D>::bytes(waves), stream, static_cast<const bf16_t*>(q_rot),
                       q_chunk0, n_q_chunks, static_cast<const bf16_t*>(k_res),
                       static_cast<const bf16_t*>(v_res), res_tokens, res_slot,
                       static_cast<bf16_t*>(k_routed), static_cast<bf16_t*>(v_routed), group_idx,
                       static_cast<bf16_t*>(out), lse, r, FastDiv(p.n_kv_heads),
                       FastDiv(n_q_chunks), FastDiv(2 * r), group_shift, p.keep_first,
                       recent_window(p), p.topk_groups, static_cast<const bf16_t*>(k_src),
                       static_cast<const bf16_t*>(v_src), src_tokens,
                       chunk_map(p.batch * p.n_q_heads, n_q_chunks, block_major),
                       chunk_map(p.batch * p.n_kv_heads, n_q_chunks, block_major), n_split,
                       block_major, static_cast<int>(blocks));
    return hipGetLastError();
}

}  // namespace

// Where this form is the faster one: launches whose query tiles fit the chip
// once, up to a number of key tiles.  One CU takes all keys of a query tile, at
// 0.22 us a tile of d64 and 0.46 of d128, while the split form spreads them
// (0.05 to 0.25) but pays a second launch and the partial results' way, the
// more the more query tiles there are.  hga_attend_split, here / split form, us,
// by query tiles and key tiles:
//   d64   4: 10 8.1/8.0, 28 12.7/8.9, 260 63/23;  64: 16 9.1/10.1, 28 13.2/11.9;
//         128: 28 13.6/14.4, 52 21.5/17.4;  256 (4 splits): 16 12.3/14.7, 28 18.8/17.6
//   d128  4: 10 11.1/11.1, 28 21.9/12.0, 260 132/30;  64: 16 13.0/17.6, 28 22.9/21.4;
//         128: 28 23.9/25.7, 52 38.5/28.0;  256 (8 splits): 28 24.1/26.7, 52 38/32;
//         256 (4 splits): 10 16.1/21.3, 16 23.2/20.2
// Few splits are few wavefronts, each with a long run of tiles: two splits of
// 64 query tiles, 10 key tiles 13.1/11.1 (d64) and 17.9/19.0, 16 18.9/14.0 and
// 25.8/23.9; four splits, 16 11.3/10.8 and 15.7/18.6, 28 17.2/13.7 and 24.1/23.4.
bool attend_few_fits(const hga_plan& plan, int n_q_chunks) {
    const hga_params& p = plan.p;
    const int64_t tiles = 2 * static_cast<int64_t>(p.batch) * p.n_q_heads * n_q_chunks;
    const int lds = p.head_dim == 64 ? FewLayout<64>::bytes(16) : FewLayout<128>::bytes(10);
    return tiles <= plan.n_cu && lds <= plan.max_lds;
}

bool attend_few_applies(const hga_plan& plan, int n_q_chunks, int n_tiles, int n_split) {
    const hga_params& p = plan.p;
    if (!attend_few_fits(plan, n_q_chunks)) return false;
    const int q_tiles = 2 * p.batch * p.n_q_heads * n_q_chunks;
    return n_tiles <= 10 + q_tiles * 51 / plan.n_cu &&
           n_tiles <= (p.head_dim == 64 || 2 * q_tiles <= plan.n_cu || n_split >= 8 ? 4 : 3) * n_split;
}

hipError_t launch_attend_few(const hga_plan& plan, const void* q_rot, int q_chunk0, int n_q_chunks,
                             const void* k_res, const void* v_res, int64_t res_tokens,
                             const int32_t* res_slot, void* k_routed, void* v_routed,
                             const int32_t* group_idx, void* out, float* lse, int n_split,
                             hipStream_t stream, const void* k_src, const void* v_src,
                             int64_t src_tokens, bool block_major) {
    // d128: ten staging regions fill the LDS, and one split a wavefront its
    // registers; more splits go two to a wavefront of eight
#define HGA_FEW(DD, WW, PP)                                                                       \
    return (k_src ? launch_few_t<DD, WW, PP, true> : launch_few_t<DD, WW, PP, false>)(            \
        plan, q_rot, q_chunk0, n_q_chunks, k_res, v_res, res_tokens, res_slot, k_routed,          \
        v_routed, group_idx, out, lse, n_split, stream, k_src, v_src, src_tokens, block_major)
    if (plan.p.head_dim == 64) HGA_FEW(64, 16, 1);
    if (n_split <= 10) HGA_FEW(128, 10, 1);
    HGA_FEW(128, 8, 2);
#undef HGA_FEW
}

}  // namespace hga
