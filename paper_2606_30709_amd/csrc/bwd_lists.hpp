// The inverted lists of the attention backward's chunk-major key gradients
// (attend_bwd_keys.hip): per key chunk of a (batch, KV head), the query units
// that attend it.  The workgroup's thread id, barrier, shared atomic add and
// wavefront scan come from the caller, so that the builder also runs on the
// host, its wavefronts in any order between two barriers.
#pragma once

#include "attend_bwd.hpp"
#include "attend_common.hpp"

namespace hga {

constexpr int kIndexThreads = 1024;

// A list entry: query unit, its opened groups of the chunk (bit per group),
// and whether the chunk is the unit's own (causal mask).
constexpr int kUnitBits = 22, kMaskShift = 22;
constexpr uint32_t kCausal = 1u << 30;
// An item: x = chunk | entries << 24 | (part of a cut list) << 30, y = first
// entry.
constexpr int kCountShift = 24, kCountMask = 63;
static_assert(kUnitBits <= kCountShift, "chunk ids (units are chunks too)");

// Calls f(chunk, entry) for every entry of the (batch, KV head), the work
// spread over the workgroup: slot 0 of unit i is its own chunk, then its
// visible chunks, then its routed groups, where a run of ascending groups of
// one chunk makes one entry (any other order, and repeated ids, make several).
template <typename Wg, typename F>
__host__ __device__ inline void each_entry(const Wg& wg, const int32_t* __restrict__ gid, int nq,
                                           int q_chunk0, int keep_first, int window, int topk,
                                           int gpc_shift, FastDiv per, F f) {
    const int fixed = per.d - topk;
    const int gpc = 1 << gpc_shift;
    for (uint32_t idx = wg.thread(); idx < nq * per.d; idx += kIndexThreads) {
        const int i = per.div(idx), k = idx - i * per.d;
        const int c = q_chunk0 + i;
        const uint32_t all = ((1u << gpc) - 1) << kMaskShift;
        if (k == 0) {
            f(c, static_cast<uint32_t>(i) | all | kCausal);
        } else if (k < fixed) {
            const VisibleChunks vis(c, keep_first, window);
            if (k - 1 < vis.count) f(vis.chunk(k - 1), static_cast<uint32_t>(i) | all);
        } else {
            const int32_t* g = gid + static_cast<int64_t>(i) * topk;
            const int s = k - fixed;
            const int lim = c << gpc_shift;
            auto valid = [&](int x) { return x >= 0 && x < lim; };
            const int g0 = g[s];
            if (!valid(g0)) continue;
            const int chunk = g0 >> gpc_shift;
            const int before = s > 0 ? g[s - 1] : -1;
            if (valid(before) && (before >> gpc_shift) == chunk && before < g0) continue;
            uint32_t mask = 1u << (g0 & (gpc - 1));
            for (int last = g0, t = s + 1; t < topk; ++t) {
                const int gt = g[t];
                if (!valid(gt) || (gt >> gpc_shift) != chunk || gt <= last) break;
                mask |= 1u << (gt & (gpc - 1));
                last = gt;
            }
            f(chunk, static_cast<uint32_t>(i) | mask << kMaskShift);
        }
    }
}

struct BwdListsScratch {
    // per wavefront: entries and segments of the range, entries before it
    int sum[3][kIndexThreads / 64];
    int total[2];  // entries and end of the segments (others still read the sums)
};

// Counts, scans and fills the lists of the key chunks [c0, c0 + n) of one
// (batch, KV head), kIndexThreads threads.  A workgroup per range: it looks at
// all entries, counts those of earlier chunks, and leaves their segments
// c0 + (their entries) / seg items, which holds them however they are cut.
// items: the segments, at most `seg` entries each, the unused ones empty up to
// the next range's first or cap_items; clear (or null): per chunk, whether no
// single segment covers it; cnt: shared, n counters.  kWhole: the one range is
// all chunks.
template <bool kWhole, typename Wg>
__host__ __device__ inline void build_bwd_lists(
    const Wg& wg, const int32_t* __restrict__ gid, int nq, int q_chunk0, int keep_first, int window,
    int topk, int gpc_shift, FastDiv per, int n_chunks, int c0, int n, int seg,
    int2* __restrict__ items, int cap_items, uint32_t* __restrict__ entries,
    int* __restrict__ clear, int* cnt, BwdListsScratch& s) {
    if (kWhole) c0 = 0, n = n_chunks;
    const int tid = wg.thread(), lane = tid & 63, wave = tid >> 6;
    for (int x = tid; x < n; x += kIndexThreads) cnt[x] = 0;
    wg.sync();
    int n_before = 0;
    each_entry(wg, gid, nq, q_chunk0, keep_first, window, topk, gpc_shift, per,
               [&](int chunk, uint32_t) {
                   if (kWhole || static_cast<uint32_t>(chunk - c0) < static_cast<uint32_t>(n))
                       wg.add(&cnt[chunk - c0], 1);
                   else
                       n_before += chunk < c0;
               });
    wg.sync();
    // exclusive sums of the entries and of the segments, a run of chunks per thread
    const int run = (n + kIndexThreads - 1) / kIndexThreads;
    const int lo = tid * run < n ? tid * run : n;
    const int hi = lo + run < n ? lo + run : n;
    int n_ent = 0, n_seg = 0;
    for (int x = lo; x < hi; ++x) {
        n_ent += cnt[x];
        n_seg += (cnt[x] + seg - 1) / seg;
    }
    int at_ent = wg.scan(n_ent), at_seg = wg.scan(n_seg);
    const int before_sum = kWhole ? 0 : wg.scan(n_before);
    if (lane == 63) {
        s.sum[0][wave] = at_ent;
        s.sum[1][wave] = at_seg;
        s.sum[2][wave] = before_sum;
    }
    wg.sync();
    int before = 0;
    if (!kWhole)
        for (int w = 0; w < kIndexThreads / 64; ++w) before += s.sum[2][w];
    at_ent += before - n_ent;
    at_seg += c0 + before / seg - n_seg;
    for (int w = 0; w < wave; ++w) {
        at_ent += s.sum[0][w];
        at_seg += s.sum[1][w];
    }
    for (int x = lo; x < hi; ++x) {
        const int m = cnt[x];
        cnt[x] = at_ent;  // the fill's cursor
        if (clear) clear[c0 + x] = m == 0 || m > seg;
        for (int o = 0; o < m; o += seg)
            items[at_seg++] = make_int2(
                (c0 + x) | (m - o < seg ? m - o : seg) << kCountShift | (m > seg) << 30, at_ent + o);
        at_ent += m;
    }
    if (tid == kIndexThreads - 1) {
        s.total[0] = at_ent;
        s.total[1] = at_seg;
    }
    wg.sync();
    // the unused items have no entries
    const int end = c0 + n < n_chunks ? c0 + n + s.total[0] / seg : cap_items;
    for (int x = s.total[1] + tid; x < end; x += kIndexThreads) items[x] = make_int2(0, 0);
    each_entry(wg, gid, nq, q_chunk0, keep_first, window, topk, gpc_shift, per,
               [&](int chunk, uint32_t e) {
                   if (kWhole || static_cast<uint32_t>(chunk - c0) < static_cast<uint32_t>(n))
                       entries[wg.add(&cnt[chunk - c0], 1)] = e;
               });
}

}  // namespace hga
