// The gate of a launch of 256 blocks that wait for each other (the resident Gram-Schmidt kernels of rok_mgs.hip).
//
// A plain launch does not promise that all its blocks get onto the chip together: another stream's blocks may hold
// CUs, in the worst case while they wait themselves.  So who takes part is settled by one 64-bit word, the gate:
//   bits 0 .. 53   arrivals: every block adds 1 when it starts, 256 a launch, so the count says which launch it is
//                  in and how many of its blocks have started (it outlasts any number of launches);
//   bits 54 .. 61  size of the closed gang (1 .. 255), 0: none;
//   bit 62         parity of the launch that was closed.
// A block that has waited long with nobody coming, while blocks of another waiting launch are stuck as well (Waiting
// below), closes the gate by a compare-and-swap that keeps the count, unless the count is complete.  A block
// that finds its launch closed when it starts leaves.  With all 256 in, nobody can close any more, and every block
// is running, so the waits end.  A closed launch's mark is taken off by the first arrival of the next one, before
// a launch of the same parity can read it.
//
// Plain C++ over a policy A of relaxed atomics, so that the protocol also runs on the host:
//   A::load(p), A::add(p, x) (returns the value before), A::cas(p, &expected, desired) for the gate's 64-bit word,
//   A::add and A::load_first(p) (ordered before the loads after it) for the 32-bit word of waiting blocks.
#pragma once

#if defined(__HIPCC__)
#define ROK_GATE_FN __device__ __forceinline__
#else
#define ROK_GATE_FN inline
#endif

namespace rok {

constexpr int kGateBlocks = 256;
constexpr int kGateIdle = 20;        // looks without an arrival after which a block counts as stuck (about 1 ms)
constexpr int kGateIdleLong = 400;   // looks after which it closes the gate whatever else waits (about 20 ms)

using GateWord = unsigned long long;
constexpr int kGateSizeShift = 54, kGateParityShift = 62;
constexpr GateWord kGateCount = (1ull << kGateSizeShift) - 1;

struct Gang {
    GateWord base;   // the count before this launch
    int rank;        // this block's order of arrival, or -1: came to a closed gate
    int size;        // blocks that take part (once closed)
};

ROK_GATE_FN GateWord gate_base(GateWord g) { return (g & kGateCount) & ~(GateWord)(kGateBlocks - 1); }

// What the upper bits say where the launch that starts at `base` has been closed with n blocks.
ROK_GATE_FN GateWord gate_mark(GateWord base, int n) {
    return ((base / kGateBlocks & 1) << kGateParityShift) | ((GateWord)n << kGateSizeShift);
}

// Size of the closed gang of the launch that starts at `base`, 0 if it has not been closed.
ROK_GATE_FN int gate_closed(GateWord base, GateWord g) {
    const int n = (int)(g >> kGateSizeShift) & 0xff;
    return n && (g & ~kGateCount) == gate_mark(base, n) ? n : 0;
}

// The launch's state in the gate's value g: 0 open, 256 complete, else the size of the closed gang.
ROK_GATE_FN int gate_state(const Gang& q, GateWord g) {
    const int n = gate_closed(q.base, g);
    if (n) return n;
    return (g & kGateCount) - q.base == (GateWord)kGateBlocks ? kGateBlocks : 0;
}

// Closes the gate unless the count is complete; returns the state (each failed exchange is an arrival or a closure).
template <class A>
ROK_GATE_FN int gate_close(const Gang& q, GateWord* gate) {
    GateWord g = A::load(gate);
    for (;;) {
        const int s = gate_state(q, g);
        if (s) return s;
        const int n = (int)((g & kGateCount) - q.base);
        if (A::cas(gate, &g, (g & kGateCount) | gate_mark(q.base, n))) return n;
    }
}

// This block enters (one thread).
template <class A>
ROK_GATE_FN Gang gate_enter(GateWord* gate) {
    GateWord g = A::add(gate, (GateWord)1);
    Gang q;
    q.base = gate_base(g);
    q.rank = gate_closed(q.base, g) ? -1 : (int)((g & kGateCount) - q.base);
    q.size = 0;
    if (q.rank == 0 && (g & ~kGateCount)) {   // the mark of the launch before
        ++g;
        while ((g & ~kGateCount) && !gate_closed(q.base, g))
            if (A::cas(gate, &g, g & kGateCount)) break;
    }
    return q;
}

// Waiting blocks.  A block whose looks have found nothing new for about 1 ms counts itself in `waiting`, one word
// for all launches of a process on a device.  A gang of n blocks closes only when the word exceeds n: its own
// blocks are all stuck, and so is a block of another launch, which may be waiting for this gang's place.  Where only
// running kernels hold the chip the gang waits for them, as a cooperative launch would (launches of
// another process are not in the word: they are waited for 20 ms).  20 steps at 1000^2, M = 16, beside 20 products of 4096^2
// matrices in 64 bits on another stream: 93.7 ms; closing after 1 ms whatever holds the chip 121.9, cooperative
// launches 108.1.  Two such streams of steps: 95.7 ms for 40 (96.7 and 134.3).
struct Waiting {
    int idle = 0;          // looks without an arrival
    GateWord seen = 0;     // the gate's value at the last look
    bool counted = false;
};

template <class A>
ROK_GATE_FN void wait_count(Waiting& w, unsigned* waiting) {
    if (!w.counted && w.idle >= kGateIdle) {
        A::add(waiting, 1u);
        w.counted = true;
    }
}

// The wait is over (one thread).
template <class A>
ROK_GATE_FN void wait_end(Waiting& w, unsigned* waiting) {
    if (w.counted) A::add(waiting, ~0u);
    w.counted = false;
}

// One look of a waiting block (one thread): the launch's state, after closing it if that is due.
template <class A>
ROK_GATE_FN int gate_look(Waiting& w, const Gang& q, GateWord* gate, unsigned* waiting) {
    // before the count: what the word holds of this gang has arrived by then
    const unsigned stuck = w.idle + 1 >= kGateIdle ? A::load_first(waiting) : 0u;
    const GateWord g = A::load(gate);
    const int s = gate_state(q, g);
    if (s) return s;
    w.idle = g == w.seen ? w.idle + 1 : 0;
    w.seen = g;
    wait_count<A>(w, waiting);
    if (w.idle < kGateIdle) return 0;
    const unsigned n = (unsigned)((g & kGateCount) - q.base);
    if (w.idle >= kGateIdleLong || stuck > n) return gate_close<A>(q, gate);
    return 0;
}

}  // namespace rok
