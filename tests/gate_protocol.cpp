// The gate of the resident Gram-Schmidt launches (csrc/rok_gate.hpp) run by host threads, one per block.
//
// Every launch must end in one of two ways, on which all its blocks agree: complete (256 blocks in, ranks 0 .. 255) or closed with
// n of them (ranks 0 .. n - 1 in, all others out).  Kinds of launches:
//   0  every block comes                                              -> complete
//   1  some come late, blocks of another launch are stuck meanwhile   -> closed
//   2  as 1, but the late ones enter while the others are closing     -> either
//   3  some come late, nothing else is stuck (a kernel that runs holds their place): they come after five times
//      the looks that make a block stuck                              -> complete
// The counts start where 32 bits end as well, with the mark of the launch before still on the gate.
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <thread>
#include <vector>

#include "rok_gate.hpp"

using namespace rok;

struct HostAtomics {
    template <class T> static T load(const T* p) { return __atomic_load_n(p, __ATOMIC_RELAXED); }
    static unsigned load_first(const unsigned* p) { return __atomic_load_n(p, __ATOMIC_ACQUIRE); }
    template <class T> static T add(T* p, T x) { return __atomic_fetch_add(p, x, __ATOMIC_RELAXED); }
    static bool cas(GateWord* p, GateWord* e, GateWord d) {
        return __atomic_compare_exchange_n(p, e, d, false, __ATOMIC_RELAXED, __ATOMIC_RELAXED);
    }
};

static GateWord gate;
static unsigned waiting;

static void fail(const char* what, int launch, int kind) {
    std::printf("FAILED %s: launch %d of kind %d, gate %llx\n", what, launch, kind, gate);
    std::exit(1);
}

static void run(int launch, int kind, int late, std::mt19937& rng) {
    const GateWord start = gate;
    const GateWord base = gate_base(start);
    if ((start & (kGateBlocks - 1)) != 0) fail("count", launch, kind);
    std::vector<int> rank(kGateBlocks, -2), size(kGateBlocks, -2);
    std::vector<char> is_late(kGateBlocks, 0);
    for (int k = 0; k < late;) {
        const int b = rng() % kGateBlocks;
        if (!is_late[b]) is_late[b] = 1, ++k;
    }
    std::atomic<int> entered{0}, looked{0};
    auto block = [&](int b) {
        if (is_late[b]) {
            Waiting w;
            if (kind != 3) {   // stands for a stuck block of another launch, too
                w.idle = kGateIdle;
                wait_count<HostAtomics>(w, &waiting);
            }
            for (;;) {
                if (kind == 1 && gate_closed(base, HostAtomics::load(&gate))) break;
                if (kind == 2 && looked.load() >= kGateIdle - 1) break;
                if (kind == 3 && looked.load() >= 5 * kGateIdle) break;
                std::this_thread::yield();
            }
            wait_end<HostAtomics>(w, &waiting);
        }
        const Gang q = gate_enter<HostAtomics>(&gate);
        entered.fetch_add(1);
        rank[b] = q.rank;
        if (q.base != base) fail("base", launch, kind);
        if (q.rank < 0) return;
        Waiting w;
        int s = 0;
        for (int n = 1; s == 0; ++n) {
            s = gate_look<HostAtomics>(w, q, &gate, &waiting);
            int seen = looked.load();
            while (n > seen && !looked.compare_exchange_weak(seen, n)) {}
            // kinds 0 and 3: enough looks, the blocks that are not in yet come now
            while ((kind == 0 || kind == 3) && n >= 5 * kGateIdle && entered.load() < kGateBlocks)
                std::this_thread::yield();
            std::this_thread::yield();
        }
        wait_end<HostAtomics>(w, &waiting);
        size[b] = s;
    };
    std::vector<std::thread> t;
    for (int b = 0; b < kGateBlocks; ++b) t.emplace_back(block, b);
    for (auto& x : t) x.join();
    if ((gate & kGateCount) != base + kGateBlocks) fail("count", launch, kind);
    if (waiting != 0) fail("waiting", launch, kind);
    int in = 0, s = 0;
    std::vector<char> taken(kGateBlocks, 0);
    for (int b = 0; b < kGateBlocks; ++b) {
        if (rank[b] < 0) continue;
        if (rank[b] >= kGateBlocks || taken[rank[b]]) fail("rank", launch, kind);
        taken[rank[b]] = 1;
        if (in == 0) s = size[b];
        if (size[b] != s) fail("size differs", launch, kind);
        ++in;
    }
    if (in != s) fail("blocks in", launch, kind);
    for (int r = 0; r < in; ++r)
        if (!taken[r]) fail("a rank is missing", launch, kind);
    if ((kind == 0 || kind == 3) && s != kGateBlocks) fail("closed", launch, kind);
    if (kind == 1 && s >= kGateBlocks) fail("not closed", launch, kind);
}

int main() {
    std::mt19937 rng(12);
    const int kinds[] = {0, 1, 0, 1, 1, 0, 3, 2, 2, 1, 3, 0, 0, 2, 1, 2};
    for (GateWord count : {0ull, 0xfffffc00ull, 0xffffffc00ull, (1ull << 52) - 512}) {
        for (int parity = 0; parity < 2; ++parity) {
            gate = count + 256 * parity;
            if (gate) gate |= gate_mark(gate - kGateBlocks, 77);   // the launch before was closed
            waiting = 0;
            int k = 0;
            for (int kind : kinds) run(k++, kind, kind == 0 ? 0 : 1 + (int)(rng() % 255), rng);
        }
    }
    std::printf("ok\n");
    return 0;
}
