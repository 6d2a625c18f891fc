// Key gradients of the exact-token attention (Sec. 3.4, Eq. (1)), chunk by
// chunk: every query unit that attends a key chunk (its own, the recent
// window's, everybody for a sink, and the units that opened some of its
// groups) passes by the chunk's keys, whose dK and dV stay in registers and
// are written or (atomically) added to memory once.
//
// Unit-major accumulation adds 64 x D x 2 floats with atomics for every
// (unit, key tile) pair; with one query head per KV head that is one atomic
// add per 64 products' worth of work, and the L2's atomic rate (about 0.3 T
// adds/s) sets the pace.  Here the pairs are inverted first:
//
//   bwd_index_kernel      one workgroup per (batch, KV head) and 16,384 key
//                         chunks counts, scans and fills, per key chunk, the
//                         list of (query unit, opened groups) entries, and
//                         cuts long lists (sink chunks, chunks everybody looks
//                         up) into segments; the others compute the row
//                         statistics.
//   bwd_chunk_kernel      one workgroup per segment.
//
// Where many query heads share a KV head bwd_unit_kernel passes a unit's rows
// by its own key tiles instead, and adds with atomics.
//
// The lists and their tables stay in the caller's dq buffer, which the dQ kernel
// writes afterwards.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>

#include "attend_bwd.hpp"
#include "bwd_lists.hpp"
#include "attend_common.hpp"
#include "hga_internal.hpp"
#include "lds_copy.hpp"

namespace hga {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef short i16x4_t __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) i16x4_t lds_i16x4_t;
typedef float f32x4_t __attribute__((ext_vector_type(4)));

constexpr int KT = 64;    // tokens per chunk
constexpr int kXcds = 8;
// most 256-thread workgroups of a launch (the runtime takes fewer than 2^32 threads)
constexpr int64_t kMaxGrid = (int64_t(1) << 24) - kXcds;

// The tables of one (batch, KV head), `stride` ints apart.
struct Index {
    int* base;
    int stride, cap_items;
    __device__ int2* items(int bh) const {
        return reinterpret_cast<int2*>(base + static_cast<int64_t>(bh) * stride);
    }
    __device__ uint32_t* entries(int bh) const {
        return reinterpret_cast<uint32_t*>(items(bh) + cap_items);
    }
};

// The lists and the row statistics in one launch (neither needs the other):
// the first workgroups invert one (batch, KV head) each, or a range of its key
// chunks, bound by their two passes over its ids, while the others stream out
// and dout.  A workgroup per range: one head x 20,000 chunks of d64 1991 us
// (whole backward, adding), range after range in one workgroup 2578, unit by
// unit 4330; x 70,000 chunks 7907, 16636.
template <int D, bool kWhole>
__global__ __launch_bounds__(kIndexThreads) void bwd_index_kernel(
    const int32_t* __restrict__ group_idx, int nq, int q_chunk0, int keep_first, int window,
    int topk, int gpc_shift, FastDiv per, int n_chunks, FastDiv ranges, int seg, Index ix, int n_bh,
    int* __restrict__ clear, const bf16_t* __restrict__ out, const bf16_t* __restrict__ dout,
    const float* __restrict__ lse, float* __restrict__ stat, int64_t rows) {
    const int n_lists = n_bh * ranges.d;
    if (blockIdx.x >= n_lists) {
        bwd_row_stat<D>(out, dout, lse, stat, rows,
                        (static_cast<int64_t>(blockIdx.x) - n_lists) * kIndexThreads + threadIdx.x);
        return;
    }
    extern __shared__ int s_cnt[];  // [min(n_chunks, kBwdIndexChunks)]
    __shared__ BwdListsScratch scratch;
    const int bh = kWhole ? blockIdx.x : ranges.div(blockIdx.x);
    const int c0 = kWhole ? 0 : (blockIdx.x - bh * ranges.d) * kBwdIndexChunks;
    struct Workgroup {
        __device__ int thread() const { return threadIdx.x; }
        __device__ void sync() const { __syncthreads(); }
        __device__ int add(int* at, int x) const { return atomicAdd(at, x); }
        __device__ int scan(int x) const { return wave_incl_scan_add(x); }
    };
    build_bwd_lists<kWhole>(
        Workgroup{}, group_idx + static_cast<int64_t>(bh) * nq * topk, nq, q_chunk0, keep_first,
        window, topk, gpc_shift, per, n_chunks, c0, min(n_chunks - c0, kBwdIndexChunks), seg,
        ix.items(bh), ix.cap_items, ix.entries(bh),
        clear ? clear + static_cast<int64_t>(bh) * n_chunks : nullptr, s_cnt, scratch);
}

// For a call that writes dk and dv: zeros in the rows of the chunks that the
// lists mark (cut ones, which add, and those nobody attends) and in the rows
// past the lists' chunks.  A workgroup looks at four chunks of a (batch, KV
// head): most have nothing to clear.
template <int D>
__global__ __launch_bounds__(256) void bwd_clear_kernel(const int* __restrict__ clear, int n_chunks,
                                                        int64_t res_tokens, FastDiv per_bh,
                                                        float4* __restrict__ dk,
                                                        float4* __restrict__ dv) {
    constexpr int VPR = D / 4;  // vectors per row
    const int bh = per_bh.div(blockIdx.x), c0 = (blockIdx.x - bh * per_bh.d) * 4;
    for (int chunk = c0; chunk < c0 + 4; ++chunk) {
        const int64_t row0 = static_cast<int64_t>(chunk) * KT;
        if (row0 >= res_tokens) return;
        if (chunk < n_chunks && !clear[static_cast<int64_t>(bh) * n_chunks + chunk]) continue;
        const int n = static_cast<int>(min(res_tokens - row0, static_cast<int64_t>(KT))) * VPR;
        const int64_t at = (static_cast<int64_t>(bh) * res_tokens + row0) * VPR;
        for (int x = threadIdx.x; x < n; x += 256)
            dk[at + x] = dv[at + x] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
}

// QR query rows per step, NS steps in the LDS ring.
template <int D, int QR, int NS>
struct ChunkLayout {
    static constexpr int kRow = D * 2;
    static constexpr int kG = QR * kRow;           // dO rows after the Q rows
    static constexpr int kStat = 2 * QR * kRow;    // per 32 rows: -lse[32], -D[32]
    static constexpr int kStage = kStat + QR / 32 * 256;
    static constexpr int kBytes = NS * kStage;
    static constexpr int kCopies = QR * D / 8 / 64 / 4;  // 16-byte copies per wavefront, for Q (and dO)
    static_assert(kCopies >= 1, "copy split");
    static constexpr int kLoads = 2 * kCopies + 1;       // loads per wavefront and step
};

// The copies of one step: QR rows of Q and of dO and their statistics, the
// first of them row0 in memory, into a stage.
template <int D, int QR, int NS>
struct StepRows {
    using Lay = ChunkLayout<D, QR, NS>;
    const bf16_t *q, *dout;
    const float* stat;
    uint32_t lds0;
    int lane, wave;
    uint32_t koff[Lay::kCopies];  // source offset of this lane's copies: row * kRow + unswizzled chunk
    __device__ __forceinline__ StepRows(const bf16_t* q_, const bf16_t* dout_, const float* stat_,
                                        const unsigned char* smem)
        : q(q_), dout(dout_), stat(stat_),
          lds0(static_cast<uint32_t>(reinterpret_cast<uintptr_t>(smem))), lane(threadIdx.x & 63),
          wave(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) {
        constexpr int CPR = D / 8;  // 16-byte chunks per row
#pragma unroll
        for (int u = 0; u < Lay::kCopies; ++u) {
            const int row = (u * 4 + wave) * (64 / CPR) + lane / CPR;
            koff[u] = row * Lay::kRow + (((lane % CPR) ^ swz_rows<D>(row)) * 16);
        }
    }
    __device__ __forceinline__ void copy(int64_t row0, int stage) const {
        const u32x4 rq = rsrc_words(q + row0 * D, QR * Lay::kRow);
        const u32x4 rg = rsrc_words(dout + row0 * D, QR * Lay::kRow);
        const uint32_t at = lds0 + stage * Lay::kStage;
#pragma unroll
        for (int u = 0; u < Lay::kCopies; ++u) copy16_to_lds(rq, koff[u], at + (u * 4 + wave) * 1024);
#pragma unroll
        for (int u = 0; u < Lay::kCopies; ++u)
            copy16_to_lds(rg, koff[u], at + Lay::kG + (u * 4 + wave) * 1024);
        // 256 bytes per 32 rows; with fewer blocks than wavefronts several
        // copy the same one, so that all wait for the same count
        const int blk = wave % (QR / 32);
        copy4_to_lds(rsrc_words(stat + 2 * row0 + blk * 64, 256), lane * 4, at + Lay::kStat + blk * 256);
    }
};

// What a wavefront's 16 keys do in one step: whether any counts, whether the
// chunk is the query rows' own, whether only some count (this lane's: bias 0,
// else -inf).
struct StepKeys {
    bool live, causal, some;
    float bias;
};

// The query rows of n_steps steps past a wavefront's 16 keys (`key` is the
// lane's place in the 64 of the workgroup): dK into ak, dV into av.  The first
// NS - 1 steps have been issued.
template <int D, int QR, int NS, typename Issue, typename Keys>
__device__ __forceinline__ void key_steps(const unsigned char* smem, int n_steps,
                                          const bf16x8_t (&kf)[D / 32], const bf16x8_t (&vf)[D / 32],
                                          f32x4_t (&ak)[D / 16], f32x4_t (&av)[D / 16], int key,
                                          float scale2, Issue issue, Keys keys_of) {
    using Lay = ChunkLayout<D, QR, NS>;
    constexpr int kRow = Lay::kRow, NKS = D / 32, NB = D / 16, SPU = KT / QR, LPS = Lay::kLoads;
    const int l16 = threadIdx.x & 15, g4 = (threadIdx.x & 63) >> 4;
    // LDS offsets of this lane's reads: the swizzle repeats every 16 rows, so
    // 16-row blocks are immediates
    int aoff[NKS], toff[NB];
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) aoff[ks] = l16 * kRow + (((ks * 4 + g4) ^ swz_rows<D>(l16)) * 16);
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        const int row = g4 * 4 + (l16 >> 2);  // four queries of one dimension per transpose read
        toff[nb] = row * kRow + (((nb * 2 + ((l16 & 3) >> 1)) ^ swz_rows<D>(row)) * 16) + (l16 & 1) * 8;
    }
    int stage = 0;
    for (int s = 0; s < n_steps; ++s) {
        if (s + NS - 2 < n_steps)  // that many later steps are in flight
            wait_copies<(NS - 2) * LPS>();
        else
            wait_copies<0>();
        lds_barrier();  // the step's rows are here; everybody has left the stage before
        if (s + NS - 1 < n_steps) issue(s + NS - 1, stage == 0 ? NS - 1 : stage - 1);
        const unsigned char* base = smem + stage * Lay::kStage;
        stage = stage == NS - 1 ? 0 : stage + 1;
        const StepKeys e = keys_of(s);
        if (!e.live) continue;
        const unsigned char* sb = base + Lay::kStat + g4 * 16;
#pragma unroll
        for (int pair = 0; pair < QR / 32; ++pair) {
            f32x4_t sa[2], da[2], nl[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int blk = pair * 2 + h;  // 16-row block
                nl[h] = *reinterpret_cast<const f32x4_t*>(sb + pair * 256 + h * 64);
                sa[h] = f32x4_t{0.f, 0.f, 0.f, 0.f};
                da[h] = *reinterpret_cast<const f32x4_t*>(sb + pair * 256 + 128 + h * 64);  // dP - D
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) {
                    const unsigned char* rp = base + aoff[ks] + blk * 16 * kRow;
                    sa[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8_t, load16(rp)), kf[ks], sa[h], 0, 0, 0);
                    da[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                        __builtin_bit_cast(bf16x8_t, load16(rp + Lay::kG)), vf[ks], da[h], 0, 0, 0);
                }
            }
            if (e.some) {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int x = 0; x < 4; ++x) nl[h][x] += e.bias;
            }
            if (e.causal) {
                const int t0 = s % SPU * QR + pair * 32 + g4 * 4;
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int x = 0; x < 4; ++x)
                        nl[h][x] = key <= t0 + h * 16 + x ? nl[h][x] : -INFINITY;
            }
            // A operands: k-slot g4*8 + h*4 + x is query pair*32 + h*16 + g4*4 + x
            bf16x8_t pf, df;
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int x = 0; x < 4; ++x) {
                    const float p = __builtin_amdgcn_exp2f(fmaf(sa[h][x], scale2, nl[h][x]));
                    pf[h * 4 + x] = static_cast<__bf16>(p);
                    df[h * 4 + x] = static_cast<__bf16>(p * da[h][x]);
                }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                const unsigned char* tp = base + toff[nb] + pair * 32 * kRow;
                auto tr = [&](int off) {
                    return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                        (lds_i16x4_t*)(reinterpret_cast<uintptr_t>(tp + off)));
                };
                const bf16x8_t gb = __builtin_bit_cast(
                    bf16x8_t, __builtin_shufflevector(tr(Lay::kG), tr(Lay::kG + 16 * kRow), 0, 1, 2, 3, 4, 5, 6, 7));
                const bf16x8_t qb = __builtin_bit_cast(
                    bf16x8_t, __builtin_shufflevector(tr(0), tr(16 * kRow), 0, 1, 2, 3, 4, 5, 6, 7));
                av[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(pf, gb, av[nb], 0, 0, 0);
                ak[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(df, qb, ak[nb], 0, 0, 0);
            }
        }
    }
}

// One segment: the chunk's 64 keys, 16 to a wavefront (K and V fragments, dK
// and dV in registers), against the segment's (unit, query head) pairs, 64
// query rows staged in LDS at a time and shared by the four wavefronts.  Per
// 32 query rows and wavefront (v_mfma_f32_16x16x32_bf16):
//   S = Q.K^T, dP = dO.V^T     (A = rows from LDS, B = registers)
//   P, dS                      (lane = key, registers = queries)
//   dV += P^T.dO, dK += dS^T.Q (A = the lane's own P, dS; B = transpose reads)
// The contraction over queries is permuted alike in A and B, so P and dS go
// from accumulators to operands without leaving the lane.  A wavefront skips
// the units that opened none of its keys' groups.
// 16-key wavefronts fit the routed groups exactly (no masked products) and
// keep the registers low; several workgroups per CU hide each other's
// barriers and copies.
//
// Bound: the query rows' way to the LDS.  With the products left out the
// kernel takes 400 of its 530-580 us on 8 x 12 heads x 12,288 tokens (3.1 GB
// staged, 61% from the L2; 0.6 GB of dK and dV read and written), matrix
// cores 20% busy, VALU 24%, LDS 25%.  Tried at that size: a three-step ring
// (three workgroups per CU instead of four) 640 us, 32-row steps with three
// or four in the ring 640-650, 32 keys x 32 rows per wavefront (half the LDS
// reads, both blocks always computed) 700.  At d128 a 64-row step leaves room
// for two workgroups per CU and 32 rows for three: 2640 against 2363 us on 32/4
// heads x 32,768 tokens.
template <int D, int QR, int NS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : 2)))
void bwd_chunk_kernel(
    const bf16_t* __restrict__ q_rot, int q_chunk0, int n_q_chunks,
    const bf16_t* __restrict__ k_res, const bf16_t* __restrict__ v_res, int64_t res_tokens,
    const float* __restrict__ stat, const bf16_t* __restrict__ dout,
    float* __restrict__ dk, float* __restrict__ dv, FastDiv r_div,
    FastDiv kv_div, FastDiv item_div, int group_shift, Index ix, int n_blocks, int by_xcd,
    int write) {
    constexpr int NKS = D / 32;            // 32-wide k-steps over d
    constexpr int NB = D / 16;             // 16-wide blocks of d
    constexpr int SPU = KT / QR;           // steps per unit and query head
    extern __shared__ __align__(16) unsigned char smem[];

    int logical = blockIdx.x;
    if (by_xcd) {  // a (batch, KV head)'s segments on one XCD: its Q and dO stay in that L2
        const int per_xcd = (n_blocks + kXcds - 1) / kXcds;
        logical = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
    }
    if (logical >= n_blocks) return;
    const int bh = item_div.div(logical);
    const int it = logical - bh * item_div.d;
    const int2 item = ix.items(bh)[it];
    if (item.x == 0) return;
    const int chunk = item.x & ((1 << kCountShift) - 1);
    const int r = r_div.d;
    const int n_ent = (item.x >> kCountShift) & kCountMask;  // at most 32
    const int n_steps = n_ent * r * SPU;
    const bool shared = (item.x >> 30) & 1;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, g4 = lane >> 4;
    const int b = kv_div.div(bh), j = bh - b * kv_div.d;
    const int64_t qtok = static_cast<int64_t>(n_q_chunks) * KT;
    const int64_t head0 = static_cast<int64_t>(b) * (r * kv_div.d) + static_cast<int64_t>(j) * r;
    const float scale2 = 1.4426950408889634f / sqrtf(static_cast<float>(D));

    // the segment's entries, one per lane
    const uint32_t elist = lane < n_ent ? ix.entries(bh)[item.y + lane] : 0;
    const StepRows<D, QR, NS> rows(q_rot, dout, stat, smem);
    auto issue = [&](int s, int stage) {
        const int x = s / SPU, ent = r_div.div(x), hh = x - ent * r;
        const uint32_t e = __builtin_amdgcn_readlane(elist, ent);
        rows.copy((head0 + hh) * qtok + static_cast<int64_t>(e & ((1u << kUnitBits) - 1)) * KT + s % SPU * QR,
                  stage);
    };

    // B operands: the lane's key row, dimensions ks*32 + g4*8 .. +7
    const int key = wave * 16 + l16;
    const int64_t krow = static_cast<int64_t>(bh) * res_tokens + static_cast<int64_t>(chunk) * KT + key;
    bf16x8_t kf[NKS], vf[NKS];
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
        kf[ks] = __builtin_bit_cast(bf16x8_t, load16(k_res + krow * D + ks * 32 + g4 * 8));
        vf[ks] = __builtin_bit_cast(bf16x8_t, load16(v_res + krow * D + ks * 32 + g4 * 8));
    }
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
        if (s < n_steps) issue(s, s);

    f32x4_t ak[NB], av[NB];  // dK, dV: lane = dimension nb*16 + l16, rows = keys g4*4 + x
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int x = 0; x < 4; ++x) ak[nb][x] = av[nb][x] = 0.f;

    // this wavefront's bits of an entry's mask, and this lane's own
    const uint32_t lane_bit = 1u << (kMaskShift + (key >> group_shift));
    const uint32_t wave_bits =
        (group_shift == 3 ? 3u << (2 * wave) : 1u << ((wave * 16) >> group_shift)) << kMaskShift;

    const bool split_groups = group_shift == 3;  // a wavefront's keys are two groups
    key_steps<D, QR, NS>(smem, n_steps, kf, vf, ak, av, key, scale2, issue, [&](int s) {
        const uint32_t e = __builtin_amdgcn_readlane(elist, r_div.div(s / SPU));
        return StepKeys{(e & wave_bits) != 0, (e & kCausal) != 0, split_groups,
                        e & lane_bit ? 0.f : -INFINITY};
    });

    // Whether anybody opened the group of the lane's rows: a wavefront's keys
    // are one group, or a group in rows 0 .. 7 and another in 8 .. 15.  The
    // others are not added to (a unit that opened one group of sixteen keys
    // costs that many rows of atomics, not 64) and are zeros in a call that
    // writes, whatever their keys hold.
    const uint32_t row_bit = 1u << (kMaskShift + ((wave * 16 + g4 * 4) >> group_shift));
    const bool low = __builtin_amdgcn_ballot_w64((elist & (wave_bits & -wave_bits)) != 0) != 0;
    const bool high = __builtin_amdgcn_ballot_w64((elist & wave_bits & (wave_bits - 1)) != 0) != 0;
    const bool opened = row_bit & wave_bits & -wave_bits ? low : high;

    // In a call that writes, the chunk's only segment writes (nobody else
    // touches its rows in this launch) and the segments of a cut list add to
    // rows that bwd_clear_kernel zeroed.  A call that adds does so atomically
    // throughout: another may be adding to the same rows.
    const float ksc = 1.0f / sqrtf(static_cast<float>(D));
    const int64_t at0 = (static_cast<int64_t>(bh) * res_tokens + static_cast<int64_t>(chunk) * KT +
                         wave * 16 + g4 * 4) * D + l16;
    if (write && !shared) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                __builtin_nontemporal_store(opened ? ak[nb][x] * ksc : 0.f, dk + at0 + x * D + nb * 16);
                __builtin_nontemporal_store(opened ? av[nb][x] : 0.f, dv + at0 + x * D + nb * 16);
            }
    } else if (opened) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int x = 0; x < 4; ++x) {
                unsafeAtomicAdd(dk + at0 + x * D + nb * 16, ak[nb][x] * ksc);
                unsafeAtomicAdd(dv + at0 + x * D + nb * 16, av[nb][x]);
            }
    }
}

// The key side unit by unit: one workgroup per key tile of one query unit
// (current chunk, a visible chunk, or 64 routed rows, 16 keys to a wavefront),
// whose r*64 query rows pass by like a segment's; the tile's gradients are
// added with atomics, once per tile, through LDS so that an instruction adds
// 256 consecutive bytes.
//
// Bound: LDS reads (64 KB per 32 x 32 products and both gradients), then the
// L2's atomic rate: on 32/4 heads of d128 x 32,768 tokens the whole backward
// takes 2800 us, 2390 with plain stores in place of the atomics (timing only);
// 64-row steps 3100, a three-step ring 2820.  A wavefront per role (S twice,
// 32-key sub-tiles, rows staged through registers) took 3070.
template <int D, int QR, int NS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 64 ? 4 : 2)))
void bwd_unit_kernel(
    const bf16_t* __restrict__ q_rot, int q_chunk0, int n_q_chunks,
    const bf16_t* __restrict__ k_res, const bf16_t* __restrict__ v_res, int64_t res_tokens,
    const int32_t* __restrict__ group_idx, const float* __restrict__ stat,
    const bf16_t* __restrict__ dout, float* __restrict__ dk, float* __restrict__ dv, int r,
    FastDiv kv_div, FastDiv chunk_div, FastDiv tile_div, int group_shift, int keep_first,
    int window, int topk_groups, int n_items) {
    using Lay = ChunkLayout<D, QR, NS>;
    constexpr int NKS = D / 32, NB = D / 16, SPU = KT / QR;
    static_assert(Lay::kBytes >= 64 * D * 4, "flush area");
    extern __shared__ __align__(16) unsigned char smem[];

    // consecutive items, which read the same query rows, on one XCD
    const int per_xcd = (n_items + kXcds - 1) / kXcds;
    const int item = (blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
    if (item >= n_items) return;
    const int unit = tile_div.div(item), tile = item - unit * tile_div.d;
    const int bh = chunk_div.div(unit), i = unit - bh * n_q_chunks;
    const int c = q_chunk0 + i;
    const int routed_rows = topk_groups << group_shift;
    const VisibleChunks vis(c, keep_first, window);
    if (tile >= 1 + vis.count + (routed_rows + KT - 1) / KT) return;

    const int lane = threadIdx.x & 63, l16 = lane & 15, g4 = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = kv_div.div(bh), j = bh - b * kv_div.d;
    const int64_t qtok = static_cast<int64_t>(n_q_chunks) * KT;
    const int64_t unit_row = (static_cast<int64_t>(b) * (r * kv_div.d) + static_cast<int64_t>(j) * r) * qtok +
                             static_cast<int64_t>(i) * KT;
    const StepRows<D, QR, NS> rows(q_rot, dout, stat, smem);
    auto issue = [&](int s, int stage) { rows.copy(unit_row + s / SPU * qtok + s % SPU * QR, stage); };
    const int n_steps = r * SPU;

    // the lane's key: its row among the resident ones, -1 for none
    const int key = wave * 16 + l16;
    int tok;
    if (tile <= vis.count) {
        tok = (tile == 0 ? c : vis.chunk(tile - 1)) * KT + key;
    } else {
        const int rr = (tile - 1 - vis.count) * KT + key;
        const int g = rr < routed_rows ? group_idx[static_cast<int64_t>(unit) * topk_groups + (rr >> group_shift)] : -1;
        tok = g >= 0 && g < c * (KT >> group_shift) ? (g << group_shift) + (rr & ((1 << group_shift) - 1)) : -1;
    }
    const uint64_t real = __builtin_amdgcn_ballot_w64(tok >= 0);
    const StepKeys keys{real != 0, tile == 0, ~real != 0, tok >= 0 ? 0.f : -INFINITY};
    const int64_t kv0 = static_cast<int64_t>(bh) * res_tokens * D;
    bf16x8_t kf[NKS], vf[NKS];  // as in bwd_chunk_kernel
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
        const int64_t at = kv0 + static_cast<int64_t>(max(tok, 0)) * D + ks * 32 + g4 * 8;
        kf[ks] = __builtin_bit_cast(bf16x8_t, load16(k_res + at));
        vf[ks] = __builtin_bit_cast(bf16x8_t, load16(v_res + at));
    }
#pragma unroll
    for (int s = 0; s < NS - 1; ++s)
        if (s < n_steps) issue(s, s);

    f32x4_t ak[NB], av[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int x = 0; x < 4; ++x) ak[nb][x] = av[nb][x] = 0.f;
    key_steps<D, QR, NS>(smem, n_steps, kf, vf, ak, av, key,
                         1.4426950408889634f / sqrtf(static_cast<float>(D)), issue,
                         [&](int) { return keys; });

    // 16 rows of D floats per wavefront, row g4*4 + x turned by 16*g4 floats
    // against bank conflicts
    lds_barrier();  // the stages are free
    float* mine = reinterpret_cast<float*>(smem) + wave * 16 * D;
    const float ksc = 1.0f / sqrtf(static_cast<float>(D));
#pragma unroll
    for (int side = 0; side < 2; ++side) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int x = 0; x < 4; ++x)
                mine[(g4 * 4 + x) * D + ((nb * 16 + l16 + g4 * 16) & (D - 1))] =
                    side == 0 ? ak[nb][x] * ksc : av[nb][x];
        lds_reads_done();  // (the wavefront's LDS writes as well)
        float* dst = (side == 0 ? dk : dv) + kv0;
#pragma unroll
        for (int row = 0; row < 16; ++row) {
            const int t = __builtin_amdgcn_readlane(tok, row);
            if (t < 0) continue;
#pragma unroll
            for (int h = 0; h < D / 64; ++h) {
                const int x = h * 64 + lane;
                unsafeAtomicAdd(dst + static_cast<int64_t>(t) * D + x,
                                mine[row * D + ((x + (row >> 2) * 16) & (D - 1))]);
            }
        }
        lds_reads_done();
    }
}

struct IndexShape {
    int per, n_chunks, seg, cap_items, stride;
    bool fits;
};

IndexShape index_shape(const hga_plan& plan, int q_chunk0, int n_q_chunks) {
    const hga_params& p = plan.p;
    const int r = p.n_q_heads / p.n_kv_heads;
    IndexShape s{};
    const int64_t n_chunks = static_cast<int64_t>(q_chunk0) + n_q_chunks;
    const int64_t fixed = 1 + VisibleChunks(static_cast<int>(n_chunks - 1), p.keep_first,
                                            recent_window(p)).count;
    const int64_t per = fixed + p.topk_groups;
    const int64_t entries = per * n_q_chunks;
    // Segments of at most 32 (unit, head) steps, shorter when that leaves
    // fewer than about eight workgroups per compute unit, but of about four:
    // shorter ones only add atomics (one head x 100 chunks, K_g 40: 61 us at
    // four steps, 66 at one; six heads x 20 chunks, 62 at 24 steps, 41 at six).
    const int64_t total = entries * p.batch * p.n_kv_heads;
    int64_t seg = total / (static_cast<int64_t>(plan.n_cu) * 8);
    const int64_t most = r >= 32 ? 1 : 32 / r;
    const int64_t least = r >= 4 ? 1 : 4 / r;
    seg = seg < least ? least : seg;
    seg = seg > most ? most : seg;
    const int64_t cap = n_chunks + entries / seg;
    const int64_t stride = (2 * cap + entries + 3) / 4 * 4;
    const int64_t rows = static_cast<int64_t>(r) * n_q_chunks * KT;  // per (batch, KV head)
    // the row statistics and the tables live in dq
    s.fits = n_chunks <= (1 << kUnitBits) && stride + n_chunks + 2 * rows <= rows * p.head_dim &&
             cap * p.batch * p.n_kv_heads <= kMaxGrid && entries < (int64_t(1) << 30);
    if (!s.fits) return s;
    s.per = static_cast<int>(per);
    s.n_chunks = static_cast<int>(n_chunks);
    s.seg = static_cast<int>(seg);
    s.cap_items = static_cast<int>(cap);
    s.stride = static_cast<int>(stride);
    return s;
}

template <int D, int QR, int NS>
hipError_t launch_chunks_t(const hga_plan& plan, const IndexShape& sh, const void* q_rot,
                           int q_chunk0, int n_q_chunks, const void* k_res, const void* v_res,
                           int64_t res_tokens, const int32_t* group_idx, const void* out,
                           const float* lse, const void* dout, float* dq, float* dk, float* dv,
                           bool write, hipStream_t stream) {
    const hga_params& p = plan.p;
    static std::atomic<uint64_t> configured{0};  // per instantiation and device
    const hipError_t ce = once_per_device(configured, plan.device, [] {
        for (const void* f : {reinterpret_cast<const void*>(&bwd_index_kernel<D, true>),
                              reinterpret_cast<const void*>(&bwd_index_kernel<D, false>)}) {
            const hipError_t e = hipFuncSetAttribute(
                f, hipFuncAttributeMaxDynamicSharedMemorySize, kBwdIndexChunks * 4);
            if (e != hipSuccess) return e;
        }
        return hipFuncSetAttribute(reinterpret_cast<const void*>(&bwd_chunk_kernel<D, QR, NS>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize,
                                   ChunkLayout<D, QR, NS>::kBytes);
    });
    if (ce != hipSuccess) return ce;
    const int r = p.n_q_heads / p.n_kv_heads;
    const int n_bh = p.batch * p.n_kv_heads;
    const int group_shift = p.group == 8 ? 3 : (p.group == 16 ? 4 : 5);
    const int64_t rows = static_cast<int64_t>(p.batch) * p.n_q_heads * n_q_chunks * KT;
    const Index ix{reinterpret_cast<int*>(dq + 2 * rows), sh.stride, sh.cap_items};
    int* clear = write ? ix.base + static_cast<int64_t>(n_bh) * sh.stride : nullptr;
    const unsigned stat_blocks = static_cast<unsigned>((rows * 8 + kIndexThreads - 1) / kIndexThreads);
    const int n_ranges = (sh.n_chunks + kBwdIndexChunks - 1) / kBwdIndexChunks;
    const auto index = n_ranges == 1 ? bwd_index_kernel<D, true> : bwd_index_kernel<D, false>;
    hipLaunchKernelGGL(index, dim3(n_bh * n_ranges + stat_blocks),
                       dim3(kIndexThreads), std::min(sh.n_chunks, kBwdIndexChunks) * 4, stream,
                       group_idx, n_q_chunks, q_chunk0, p.keep_first, recent_window(p),
                       p.topk_groups, 6 - group_shift, FastDiv(sh.per), sh.n_chunks,
                       FastDiv(n_ranges), sh.seg, ix, n_bh, clear, static_cast<const bf16_t*>(out),
                       static_cast<const bf16_t*>(dout), lse, dq, rows);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (write) {
        const int64_t per_bh = (res_tokens + 4 * KT - 1) / (4 * KT);
        if (per_bh * n_bh > (int64_t(1) << 30)) return hipErrorInvalidConfiguration;
        hipLaunchKernelGGL((bwd_clear_kernel<D>), dim3(static_cast<unsigned>(per_bh * n_bh)),
                           dim3(256), 0, stream, clear, sh.n_chunks, res_tokens,
                           FastDiv(static_cast<uint32_t>(per_bh)), reinterpret_cast<float4*>(dk),
                           reinterpret_cast<float4*>(dv));
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    const int n_blocks = n_bh * sh.cap_items;
    const int by_xcd = n_bh >= 2 * kXcds;
    const int grid = by_xcd ? (n_blocks + kXcds - 1) / kXcds * kXcds : n_blocks;
    hipLaunchKernelGGL((bwd_chunk_kernel<D, QR, NS>), dim3(grid), dim3(256), (ChunkLayout<D, QR, NS>::kBytes),
                       stream, static_cast<const bf16_t*>(q_rot), q_chunk0, n_q_chunks,
                       static_cast<const bf16_t*>(k_res), static_cast<const bf16_t*>(v_res),
                       res_tokens, dq, static_cast<const bf16_t*>(dout), dk, dv, FastDiv(r),
                       FastDiv(p.n_kv_heads), FastDiv(sh.cap_items), group_shift, ix, n_blocks,
                       by_xcd, write);
    return hipGetLastError();
}

template <int D, int QR, int NS>
hipError_t launch_units_t(const hga_plan& plan, const void* q_rot, int q_chunk0, int n_q_chunks,
                          const void* k_res, const void* v_res, int64_t res_tokens,
                          const int32_t* group_idx, const float* stat, const void* dout, float* dk,
                          float* dv, int tiles, hipStream_t stream) {
    const hga_params& p = plan.p;
    static std::atomic<uint64_t> configured{0};  // per instantiation and device
    const hipError_t ce = once_per_device(configured, plan.device, [] {
        return hipFuncSetAttribute(reinterpret_cast<const void*>(&bwd_unit_kernel<D, QR, NS>),
                                   hipFuncAttributeMaxDynamicSharedMemorySize,
                                   ChunkLayout<D, QR, NS>::kBytes);
    });
    if (ce != hipSuccess) return ce;
    const int group_shift = p.group == 8 ? 3 : (p.group == 16 ? 4 : 5);
    const int window = recent_window(p);
    const int64_t n = static_cast<int64_t>(p.batch) * p.n_kv_heads * n_q_chunks * tiles;
    if (n > (int64_t(1) << 30)) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((bwd_unit_kernel<D, QR, NS>),
                       dim3(static_cast<unsigned>((n + kXcds - 1) / kXcds * kXcds)), dim3(256),
                       (ChunkLayout<D, QR, NS>::kBytes), stream, static_cast<const bf16_t*>(q_rot),
                       q_chunk0, n_q_chunks, static_cast<const bf16_t*>(k_res),
                       static_cast<const bf16_t*>(v_res), res_tokens, group_idx, stat,
                       static_cast<const bf16_t*>(dout), dk, dv, p.n_q_heads / p.n_kv_heads,
                       FastDiv(p.n_kv_heads), FastDiv(n_q_chunks), FastDiv(tiles), group_shift,
                       p.keep_first, window, p.topk_groups, static_cast<int>(n));
    return hipGetLastError();
}

}  // namespace

hipError_t launch_bwd_units(const hga_plan& plan, const void* q_rot, int q_chunk0, int n_q_chunks,
                            const void* k_res, const void* v_res, int64_t res_tokens,
                            const int32_t* group_idx, const float* stat, const void* dout,
                            float* dk, float* dv, int tiles, hipStream_t stream) {
    return (plan.p.head_dim == 64 ? launch_units_t<64, 64, 2> : launch_units_t<128, 32, 2>)(
        plan, q_rot, q_chunk0, n_q_chunks, k_res, v_res, res_tokens, group_idx, stat, dout, dk, dv,
        tiles, stream);
}

bool bwd_chunks_fit(const hga_plan& plan, int q_chunk0, int n_q_chunks) {
    return index_shape(plan, q_chunk0, n_q_chunks).fits;
}

size_t bwd_chunks_lds_bytes(const hga_plan& plan) {
    const size_t stage = plan.p.head_dim == 64 ? ChunkLayout<64, 64, 2>::kBytes
                                               : ChunkLayout<128, 32, 2>::kBytes;
    return std::max<size_t>(stage, kBwdIndexChunks * 4 + 1024);
}

hipError_t launch_bwd_chunks(const hga_plan& plan, const void* q_rot, int q_chunk0, int n_q_chunks,
                             const void* k_res, const void* v_res, int64_t res_tokens,
                             const int32_t* group_idx, const void* out, const float* lse,
                             const void* dout, float* dq, float* dk, float* dv, bool write,
                             hipStream_t stream) {
    const IndexShape sh = index_shape(plan, q_chunk0, n_q_chunks);
    if (!sh.fits) return hipErrorInvalidConfiguration;
    // d64: 64 query rows a step, four workgroups per CU; d128: 32, so that three fit
    return (plan.p.head_dim == 64 ? launch_chunks_t<64, 64, 2> : launch_chunks_t<128, 32, 2>)(
        plan, sh, q_rot, q_chunk0, n_q_chunks, k_res, v_res, res_tokens, group_idx, out, lse,
        dout, dq, dk, dv, write, stream);
}

}  // namespace hga
