// Runs the backward's list builder (csrc/bwd_lists.hpp) on the host, every
// thread of its workgroup a coroutine and the wavefronts of the workgroup in a
// chosen order between two barriers, and compares the lists with a plain
// enumeration.  Exit code 0: all orders gave right lists.
#include <hip/hip_runtime.h>
#include <ucontext.h>

#include <algorithm>
#include <cstdio>
#include <cstring>
#include <functional>
#include <map>
#include <random>
#include <vector>

#include "bwd_lists.hpp"

using namespace hga;

namespace {

constexpr int kThreads = kIndexThreads, kWaves = kThreads / 64;
enum Stop { kBarrier, kScan, kDone };

struct Machine {
    ucontext_t main;
    std::vector<ucontext_t> ctx{kThreads};
    std::vector<char> stacks = std::vector<char>(size_t(kThreads) * 32768);
    Stop stop[kThreads];
    int value[kThreads], current = 0;
    std::function<void()> body;
};
Machine* machine;

struct HostWorkgroup {
    int thread() const { return machine->current; }
    void halt(Stop why) const {
        const int t = machine->current;
        machine->stop[t] = why;
        swapcontext(&machine->ctx[t], &machine->main);
    }
    void sync() const { halt(kBarrier); }
    int add(int* at, int x) const { return (*at += x) - x; }
    int scan(int x) const {
        const int t = machine->current;
        machine->value[t] = x;
        halt(kScan);
        return machine->value[t];
    }
};

void entry() {
    machine->body();
    HostWorkgroup{}.halt(kDone);
}

// All threads from barrier to barrier, the wavefronts in the order given.
void run(Machine& m, const std::vector<int>& order) {
    machine = &m;
    for (int t = 0; t < kThreads; ++t) {
        getcontext(&m.ctx[t]);
        m.ctx[t].uc_stack.ss_sp = &m.stacks[size_t(t) * 32768];
        m.ctx[t].uc_stack.ss_size = 32768;
        m.ctx[t].uc_link = nullptr;
        makecontext(&m.ctx[t], entry, 0);
    }
    for (bool done = false; !done;) {
        for (int w : order) {
            do {
                for (int t = w * 64; t < w * 64 + 64; ++t) {
                    m.current = t;
                    swapcontext(&m.main, &m.ctx[t]);
                }
                if (m.stop[w * 64] == kScan)
                    for (int t = w * 64 + 1; t < w * 64 + 64; ++t) m.value[t] += m.value[t - 1];
            } while (m.stop[w * 64] == kScan);
        }
        done = m.stop[0] == kDone;
    }
}

#define CHECK(x)                                                      \
    do {                                                              \
        if (!(x)) {                                                   \
            std::printf("%s: line %d: %s\n", name, __LINE__, #x);     \
            return false;                                             \
        }                                                             \
    } while (0)

bool check(Machine& m, int nq, int q_chunk0, int first, int window, int group, int topk, int seg,
           int range, int n_bh, const std::vector<int>& order, const char* name) {
    const int gpc = 64 / group, n_chunks = q_chunk0 + nq;
    const int gpc_shift = gpc == 8 ? 3 : gpc == 4 ? 2 : 1;
    const int per = 1 + VisibleChunks(n_chunks - 1, first, window).count + topk;
    const int n_ent = per * nq, cap = n_chunks + n_ent / seg;
    std::mt19937 rng(nq * 131 + topk);
    for (int bh = 0; bh < n_bh; ++bh) {
        std::vector<int32_t> gid(size_t(nq) * topk);
        for (int i = 0; i < nq; ++i)
            for (int s = 0; s < topk; ++s) {
                const int c = q_chunk0 + i, lo = std::max(0, c - 70) * gpc;
                gid[size_t(i) * topk + s] = rng() % 9 == 0 ? -1 : lo + int(rng() % unsigned(c * gpc + 3 - lo));
            }
        const int guard = 64, fill = 0x5a5a5a5a;
        std::vector<int> clear(n_chunks + guard, fill), cnt(std::min(range, n_chunks) + guard, fill);
        std::vector<int2> items(cap + guard, make_int2(fill, fill));
        std::vector<uint32_t> entries(n_ent + guard, fill);
        BwdListsScratch scratch;
        int c0 = 0;
        m.body = [&] {
            const auto build = range < n_chunks ? build_bwd_lists<false, HostWorkgroup>
                                                : build_bwd_lists<true, HostWorkgroup>;
            build(HostWorkgroup{}, gid.data(), nq, q_chunk0, first, window, topk, gpc_shift,
                  FastDiv(per), n_chunks, c0, std::min(range, n_chunks - c0), seg, items.data(), cap,
                  entries.data(), clear.data(), cnt.data(), scratch);
        };
        // the ranges' workgroups in descending order: none waits for an earlier one
        for (c0 = (n_chunks - 1) / range * range; c0 >= 0; c0 -= range) run(m, order);
        // per chunk, how often each unit's groups count, and its causal entries
        using Key = std::pair<int, int>;  // unit, group of the chunk (gpc: causal)
        std::vector<std::map<Key, int>> want(n_chunks), got(n_chunks);
        for (int i = 0; i < nq; ++i) {
            const int c = q_chunk0 + i;
            for (int g = 0; g <= gpc; ++g) ++want[c][{i, g}];
            for (int x = 0; x < c; ++x)
                if (x < first || x >= c - window)
                    for (int g = 0; g < gpc; ++g) ++want[x][{i, g}];
            for (int s = 0; s < topk; ++s) {
                const int g = gid[size_t(i) * topk + s];
                if (g >= 0 && g < c * gpc) ++want[g / gpc][{i, g % gpc}];
            }
        }
        std::vector<int> segments(n_chunks), listed(n_chunks);
        std::vector<char> used(n_ent);
        for (int x = 0; x < cap; ++x) {
            CHECK(items[x].x != fill);
            if (items[x].x == 0) continue;
            const int chunk = items[x].x & ((1 << kCountShift) - 1), n = (items[x].x >> kCountShift) & kCountMask;
            CHECK(chunk < n_chunks && n >= 1 && n <= seg);
            CHECK(items[x].y >= 0 && items[x].y + n <= n_ent);
            ++segments[chunk];
            listed[chunk] += n;
            for (int e = items[x].y; e < items[x].y + n; ++e) {
                CHECK(!used[e]);
                used[e] = 1;
                const int i = int(entries[e] & ((1u << kUnitBits) - 1));
                for (int g = 0; g < gpc; ++g)
                    if (entries[e] >> (kMaskShift + g) & 1) ++got[chunk][{i, g}];
                if (entries[e] & kCausal) ++got[chunk][{i, gpc}];
            }
        }
        for (int x = 0; x < cap; ++x)
            if (items[x].x) {
                const int chunk = items[x].x & ((1 << kCountShift) - 1);
                CHECK((items[x].x >> 30 & 1) == (segments[chunk] > 1));
            }
        for (int x = 0; x < n_chunks; ++x) {
            CHECK(got[x] == want[x]);
            CHECK(segments[x] == (listed[x] + seg - 1) / seg);
            CHECK(clear[x] == (segments[x] != 1));
        }
        for (int x = 0; x < guard; ++x)
            CHECK(clear[n_chunks + x] == fill && cnt[cnt.size() - 1 - x] == fill &&
                  items[cap + x].x == fill && entries[n_ent + x] == uint32_t(fill));
    }
    return true;
}

}  // namespace

int main() {
    Machine m;
    std::vector<int> up(kWaves), down, odd;
    for (int w = 0; w < kWaves; ++w) up[w] = w;
    down.assign(up.rbegin(), up.rend());
    for (int w = 0; w < kWaves; ++w) odd.push_back(w * 7 % kWaves);
    struct {
        const char* name;
        const std::vector<int>& order;
    } orders[] = {{"first wavefront first", up}, {"last wavefront first", down}, {"mixed", odd}};
    for (const auto& o : orders) {
        const bool ok = check(m, 192, 0, 1, 1, 16, 12, 32, 16384, 3, o.order, o.name) &&  // three wavefronts with chunks
                        check(m, 21, 0, 2, 3, 8, 21, 8, 16384, 2, o.order, o.name) &&     // one
                        check(m, 5, 130, 1, 2, 32, 7, 2, 16384, 2, o.order, o.name) &&    // few units, long history
                        check(m, 1100, 300, 1, 1, 16, 4, 4, 16384, 1, o.order, o.name) && // two chunks a thread
                        check(m, 60, 140, 1, 2, 16, 9, 4, 64, 2, o.order, o.name);        // several ranges, the last partly full
        if (!ok) return 1;
        std::printf("%s: right\n", o.name);
    }
    return 0;
}
