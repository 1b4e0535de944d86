// Modified Gram-Schmidt for one Arnoldi column with the work vector resident
// on chip (Sec. 2.2.2, modified Arnoldi).
//
// The column's passes h_ij = <v_i, w>, w <- w - h_ij v_i (i = 0..j) and the
// norm h_{j+1,j} = ||w|| are dependent global reductions.  Launched as one
// kernel per pass, each pass streams w in and out (4 vectors of traffic);
// here one kernel keeps w on chip for the whole column, so a pass reads only
// v_i, and its blocks exchange their sums after each pass.
//
// Summation order is the canonical one of the per-pass kernels: 262144 lanes,
// lane t adds the elements t, t + T, t + 2T, ... (T = 262144) in index order,
// each group of 256 consecutive lanes is combined by the halving tree into one
// of 1024 partials, lane t of 256 adds partials t, t + 256, t + 512, t + 768 in
// order, and the halving tree over those 256 lanes gives the sum.  Which block
// holds which group does not enter the result.  A grid of NB blocks (a power
// of two) gives block b the groups g = b (mod NB): their partials are whole
// subtrees of the final tree, so a block hands on ONE value (its 256 / NB
// final lanes, already combined down to lane b) and NB values finish the sum.
//
// Exchange (NB > 1): no counters and no barrier.  Each block stores its value
// into its slot of one of three buffers; wave 0 of every block polls all NB
// slots until none holds the empty mark (a signalling-NaN bit pattern, which no
// sum can produce) and then finishes the tree from the registers it polled
// into: one store and one load across the chip, where arriving at a two-level
// counter barrier and then loading 1024 partials took five dependent ones.
// A buffer has kCopies copies of its slots, written together and polled by
// one block in kCopies each: 256 blocks polling the same 16 cache lines queue
// up at the few memory channels that hold them (a sum over 256 blocks with no
// loads in flight: 3.1 us with one copy, 2.2 with 4, 1.8 with 8, 2.0 with 16,
// 2.2 with 32; over 64 blocks 2.9, 2.2, 1.9, 1.8, 1.8).
// After exchange p every block has finished exchange p - 1, so a block empties its
// slots of buffer (p - 1) mod 3 then; they are written again in exchange p + 2.
// The exchange number continues from launch to launch (kBarPhase; the slots
// of the last exchange of a launch are emptied by the first of the next, which
// between two launch_init has at least as many blocks).
// All of it uses agent-scope atomics (coherent across XCDs without an L2
// write-back); every spin is bounded and reports a status flag instead of
// hanging.
//
// Loads of the next basis vector: in flight, they delay the exchange's store
// and polls, which queue behind them.  Half are issued before the block's
// tree, which they overlap, and the rest when the block's value is out (an extra
// block barrier tells the other waves).  Pass time with 8 elements per thread, 256 blocks: everything
// before the tree 4.0 us, half before and half after the sum 3.7 us, this way 3.3 us.
//
// Grids by size (n elements; a block has 1024 threads):
//   n <= 8192            one block, no exchange: up to 8 elements per thread
//   n <= 32768           eight blocks, up to 4 elements per thread
//   n <= 4194304         256 blocks, up to 16 elements per thread
// An exchange needs all blocks of its grid running.  Eight blocks get there: one process
// has at most one kernel per hardware queue on the device at a time (streams on one queue
// are serialised; 4 queues by default, 32 at most), so at most 32 x 8 = 256 of its
// blocks wait in exchanges of eight, one per CU, every other kernel drains, and a gang of 256 that holds their place
// closes when they are stuck.  (Several processes on one device could exceed that; the wait is
// bounded and sets ROK_FLAG_BARRIER.)  256
// blocks fill the chip, and settle first who takes part (rok_gate.hpp).  Launched
// cooperatively instead, which drains the stream around the kernel, a column cost 12 to 15 us more:
// 611 x 389 step 909 us, now 710; 1024^2 step 2867, 2632; gradient at 512^2 9892, 8166;
// adaptive 512^2 5649, 4552; 24 columns at 64^3 2386, 2072.
//
// The same machinery runs the reverse of a column for the discrete adjoint
// of the step (k_mgs_rev_resident below): the normalisation and the passes
// in reverse order, with the forward iterate and its adjoint resident.
#include "rok.h"
#include "rok_device.hpp"
#include "rok_gate.hpp"
#include "rok_kernels.hpp"

namespace rok {

constexpr int kPT = 1024;                       // threads per block
constexpr int kLanes = kRedBlocks * kRedThreads;     // canonical lanes (262144)
constexpr int kBigGrid = kLanes / kPT;               // 256 blocks: the grid that holds every canonical lane
constexpr int kMidGrid = 8;                          // the plain grid (see above)
constexpr int kCopies = kExchangeCopies;             // copies of the exchange slots
constexpr double kBreakdownTolR = 1e-13;
constexpr long kSpinLimit = 1L << 22;
// s_waitcnt operand with vmcnt = 0 and the other counters at their maximum
// (gfx9 encoding: vmcnt[3:0] and [15:14], expcnt[6:4], lgkmcnt[11:8]).
constexpr int kWaitVmcnt0 = 0x0F70;

#define AGENT __HIP_MEMORY_SCOPE_AGENT

// exchange words in Work::bar (unsigned): the number of the next exchange modulo 3 (and that of the next exchange
// of a closed gang), the error word, and the 64-bit gate
constexpr int kBarPhase = 0;
constexpr int kBarGangPhase = 1;
constexpr int kBarErr = 32;
constexpr int kBarGate = 64;

// The lanes of a block: thread tid of block b holds, for k < K and c < C, the
// element of lane (g * 256 + (tid & 255)), chunk c, of group
// g = b + NB (tid / 256 + 4 k).  E = K C elements per thread.
template <int NB_, int K_, int C_>
struct Lanes {
    static constexpr int NB = NB_, K = K_, C = C_, E = K_ * C_;
    static_assert(NB * 4 * K <= kRedBlocks, "groups past the canonical 1024");
    static_assert(C == 1 || 4 * K * NB == kRedBlocks, "chunks only where every lane of the grid is held");
    static __device__ __forceinline__ int base(int b) {
        return (b + NB * (threadIdx.x >> 8)) * kRedThreads + (threadIdx.x & (kRedThreads - 1));
    }
    static __device__ __forceinline__ int base() { return base(blockIdx.x); }
    static constexpr __device__ int step(int x) { return (x / C) * (NB * kPT) + (x % C) * kLanes; }
};

// In-wave halving of K values at once: value k's six levels s_i + s_{i+h}, h = 32,
// 16, 8, 4, 2, 1.  While several values are left, a level leaves one value in the
// lanes without bit h and another in the lanes with it (one exchange and one
// addition for both); the additions are those of each value's own tree.
// Afterwards the sum of value k is in lane tree_lane(k) (K <= 8).
__host__ __device__ constexpr int tree_lane(int k) { return 32 * (k & 1) + 16 * ((k >> 1) & 1) + 8 * ((k >> 2) & 1); }

template <int K>
__device__ __forceinline__ double wave_tree(double (&v)[K]) {
    static_assert(K == 1 || K == 2 || K == 4 || K == 8, "a power of two up to 8");
    double a[(K + 1) / 2], b[(K + 3) / 4], r;
#pragma unroll
    for (int k = 0; k < (K + 1) / 2; ++k) {
        if constexpr (K >= 2) a[k] = swap_add<32>(v[2 * k], v[2 * k + 1]);
        else a[0] = v[0] + lane_down<32>(v[0]);
    }
#pragma unroll
    for (int k = 0; k < (K + 3) / 4; ++k) {
        if constexpr (K >= 4) b[k] = swap_add<16>(a[2 * k], a[2 * k + 1]);
        else b[0] = a[0] + lane_down<16>(a[0]);
    }
    if constexpr (K == 8) r = swap_add<8>(b[0], b[1]);
    else r = b[0] + lane_down<8>(b[0]);
    r = r + lane_down<4>(r);
    r = r + lane_down<2>(r);
    r = r + lane_down<1>(r);
    return r;
}

// The gang of a launch of 256 blocks: who takes part is settled by the gate (rok_gate.hpp).  The blocks of a closed
// gang do the whole column by themselves (gang_column, gang_reverse), dealing the 256 blocks' work out among them: the same bits,
// slower.  Nothing of this costs a launch but one atomic, under the first loads.
static_assert(kBigGrid == kGateBlocks, "the gate counts these");
constexpr int kGateSpins = 64;    // polls between two looks at the gate (about 50 us)
constexpr int kGateHold = 1 << 16;

struct DeviceAtomics {
    static __device__ __forceinline__ GateWord load(const GateWord* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, AGENT); }
    static __device__ __forceinline__ unsigned load_first(const unsigned* p) { return __hip_atomic_load(p, __ATOMIC_ACQUIRE, AGENT); }
    static __device__ __forceinline__ GateWord add(GateWord* p, GateWord x) { return __hip_atomic_fetch_add(p, x, __ATOMIC_RELAXED, AGENT); }
    static __device__ __forceinline__ unsigned add(unsigned* p, unsigned x) { return __hip_atomic_fetch_add(p, x, __ATOMIC_RELAXED, AGENT); }
    static __device__ __forceinline__ bool cas(GateWord* p, GateWord* e, GateWord d) {
        return __hip_atomic_compare_exchange_strong(p, e, d, __ATOMIC_RELAXED, __ATOMIC_RELAXED, AGENT);
    }
};

// blocks of all launches on this device that are stuck in their first exchange (Waiting)
static __device__ unsigned g_waiting;

__device__ __forceinline__ GateWord* gate_word(unsigned* bar) { return (GateWord*)(bar + kBarGate); }

// This block enters (one thread).  hold > 0 (tests): the blocks from `hold` on come late, counted as stuck meanwhile.
__device__ __forceinline__ Gang enter(unsigned* bar, int hold) {
    if (hold > 0 && (int)blockIdx.x >= hold) {
        Waiting w;
        w.idle = kGateIdle;
        wait_count<DeviceAtomics>(w, &g_waiting);
        for (int i = 0; i < kGateHold; ++i) {
            const GateWord g = DeviceAtomics::load(gate_word(bar));
            if (gate_closed(gate_base(g), g)) break;
        }
        wait_end<DeviceAtomics>(w, &g_waiting);
    }
    return gate_enter<DeviceAtomics>(gate_word(bar));
}

// LDS of one exchange: the block trees' cross-wave levels (SK values per thread), the group sums, the result
template <int K>
struct ExLds {
    static constexpr int SK = K;
    static_assert(K <= 8, "the block trees' LDS");
    double s[SK][kPT];
    double gs[4 * K];
    double out;
    int err;
    Gang gang;
};

// The block's value of one canonical sum: acc[k] is this thread's lane sum of
// its group k.  Returned in wave 0 (every lane); other waves return garbage.
// The cross-wave levels of a 256-lane tree, s_i + s_{i+128} then s_i + s_{i+64}, are
// (x_i + x_{i+128}) + (x_{i+64} + x_{i+192}), taken by one wave after one block barrier.
template <class L>
__device__ __forceinline__ double block_value(double (&acc)[L::K], ExLds<L::K>& X) {
    constexpr int K = L::K, SK = ExLds<K>::SK;
    const int tid = threadIdx.x, lane = tid & 63;
    auto quad = [&](int k, int sub) -> double {
        const double* p = X.s[k] + sub * kRedThreads + lane;
        return (p[0] + p[128]) + (p[64] + p[192]);
    };
    if constexpr (K == 1 && 4 * L::NB == kRedBlocks) {
        // the four sub-blocks' groups are the four partials of one final lane: wave 0 takes all four
        X.s[0][tid] = acc[0];
        __syncthreads();
        double p = 0.0;
        if (tid < 64) {
            double v[4] = {quad(0, 0), quad(0, 1), quad(0, 2), quad(0, 3)};
            const double t = wave_tree<4>(v);
#pragma unroll
            for (int q = 0; q < 4; ++q) p = p + lane_value(t, tree_lane(q));
        }
        return p;
    } else {
        // the 4 K trees are dealt over the 16 waves: wave 4 sub + q takes those of sub-block sub with k = q (mod 4)
#pragma unroll
        for (int k = 0; k < SK; ++k) X.s[k][tid] = acc[k];
        __syncthreads();
        constexpr int P = K < 4 ? 1 : K / 4;   // trees per wave
        const int kw = (tid >> 6) & 3, sub = tid >> 8;
        if (K >= 4 || kw < K) {
            double v[P];
#pragma unroll
            for (int q = 0; q < P; ++q) v[q] = quad(kw + 4 * q, sub);
            const double t = wave_tree<P>(v);
#pragma unroll
            for (int q = 0; q < P; ++q)
                if (lane == tree_lane(q)) X.gs[sub + 4 * (kw + 4 * q)] = t;
        }
        __syncthreads();
        double x = 0.0;
        if (tid < 64) {
            // group m = r + R q of the block is partial q of its final lane r
            constexpr int R = kRedThreads / L::NB, Q = (4 * K + R - 1) / R;
#pragma unroll
            for (int q = 0; q < Q; ++q)
                if (lane < R && lane + R * q < 4 * K) x = x + X.gs[lane + R * q];
            double v[1] = {x};   // lanes past the last hold 0: their levels add +0.0
            x = lane_value(wave_tree<1>(v), 0);
        }
        return x;
    }
}

// An empty slot: a signalling NaN, which arithmetic never returns (a partial of these very bits, which could
// only be passed through from the caller's data, is published as another NaN).
constexpr unsigned long long kEmptySlot = kExchangeEmpty;

constexpr int kBufSlots = kCopies * kRedThreads;       // slots of one buffer
constexpr int kGangSlots = 3 * kBufSlots;              // first slot of a closed gang's three buffers (one copy each)

__device__ __forceinline__ unsigned long long slot_bits(double v) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(v);
    return u == kEmptySlot ? 0x7ff8000000000000ull : u;
}

// wave 0: final lanes t and t + 128, then t and t + 64, then the wave's tree
__device__ __forceinline__ double final_value(const unsigned long long (&u)[4]) {
    double t[1] = {(__longlong_as_double((long long)u[0]) + __longlong_as_double((long long)u[2])) +
                   (__longlong_as_double((long long)u[1]) + __longlong_as_double((long long)u[3]))};
    return lane_value(wave_tree<1>(t), 0);
}

constexpr int kExFailed = 1, kExClosed = 2;   // ways an exchange does not give a sum

// Canonical sum over the grid of the lane sums acc[k]; every thread gets it in
// *out.  phase: the exchange's number modulo 3, advanced.  mid() runs in the
// waves 1-15 once the block's value is out, after() in wave 0 once the other
// blocks' values have arrived (its loads would otherwise delay the polls:
// loads return in order).  One block alone calls neither.  Nonzero (in every thread of the
// block) if the exchange failed, or if it is the launch's first and the gang has been closed.
template <class L, typename Mid, typename After>
__device__ __forceinline__ int grid_sum(double (&acc)[L::K], ExLds<L::K>& X, double* slots, int& phase, unsigned* bar,
                                        bool first, double* out, Mid mid, After after) {
    constexpr int NB = L::NB;
    const int tid = threadIdx.x;
    double v = block_value<L>(acc, X);
    if constexpr (NB == 1) {
        if (tid == 0) X.out = v;
        __syncthreads();
        *out = X.out;
        return 0;
    } else {
        unsigned long long* buf = (unsigned long long*)slots + phase * kBufSlots;
        if (tid < 64) {
            // the slots emptied after the last exchange are seen empty before this value is seen
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
            if (tid < kCopies)
                __hip_atomic_store(buf + tid * kRedThreads + blockIdx.x, slot_bits(v), __ATOMIC_RELAXED, AGENT);
        }
        __syncthreads();
        if (tid >= 64) {
            mid();
        } else {
            const unsigned long long* mine = buf + (blockIdx.x % kCopies) * kRedThreads;
            constexpr int Q = (NB + 63) / 64;
            unsigned long long u[Q];
            long spins = 0;
            int err = 0;
            Waiting wait;
            for (;;) {
                bool miss = false;
#pragma unroll
                for (int q = 0; q < Q; ++q) {
                    const int b = tid + 64 * q;
                    u[q] = (NB >= 64 || b < NB) ? __hip_atomic_load(mine + b, __ATOMIC_RELAXED, AGENT) : 0ull;
                }
#pragma unroll
                for (int q = 0; q < Q; ++q) miss = miss || u[q] == kEmptySlot;
                if (!__any(miss)) break;
                if (++spins > kSpinLimit ||
                    ((spins & 1023) == 0 && __hip_atomic_load(bar + kBarErr, __ATOMIC_RELAXED, AGENT))) {
                    if (tid == 0) __hip_atomic_store(bar + kBarErr, 1u, __ATOMIC_RELAXED, AGENT);
                    err = kExFailed;
                    break;
                }
                if (first && spins % kGateSpins == 0) {
                    int s = 0;
                    if constexpr (NB == kBigGrid) {
                        // (a complete gate stays complete: then only the slots are waited for)
                        if (tid == 0) s = gate_look<DeviceAtomics>(wait, X.gang, gate_word(bar), &g_waiting);
                        s = __builtin_amdgcn_readfirstlane(s);
                    } else if (tid == 0) {
                        ++wait.idle;
                        wait_count<DeviceAtomics>(wait, &g_waiting);
                    }
                    if (s > 0 && s < kBigGrid) {
                        if (tid == 0) X.gang.size = s;
                        err = kExClosed;
                        break;
                    }
                }
            }
            if (tid == 0) wait_end<DeviceAtomics>(wait, &g_waiting);
            after();
            if constexpr (Q == 4) {
                v = final_value(u);
            } else {
                double t[1] = {__longlong_as_double((long long)u[0])};   // lanes past NB hold 0
                v = lane_value(wave_tree<1>(t), 0);
            }
            static_assert(Q == 4 || Q == 1, "256 blocks, or at most 64");
            if (tid < kCopies && err == 0)
                __hip_atomic_store((unsigned long long*)slots + (phase == 0 ? 2 : phase - 1) * kBufSlots +
                                       tid * kRedThreads + blockIdx.x,
                                   kEmptySlot, __ATOMIC_RELAXED, AGENT);
            if (tid == 0) {
                X.out = v;
                X.err = err;
            }
        }
        __syncthreads();
        *out = X.out;
        const int err = X.err;
        if (err == 0) phase = phase == 2 ? 0 : phase + 1;
        return err;
    }
}

// A block of a closed gang, after its first exchange (number `phase`): the slots that a complete launch's next
// exchange would have emptied, and its own of this exchange, which nobody reads.
__device__ __forceinline__ void gang_start(const Gang& q, double* slots, int phase) {
    const int tid = threadIdx.x;
    if (tid >= kCopies) return;
    unsigned long long* prev = (unsigned long long*)slots + (phase == 0 ? 2 : phase - 1) * kBufSlots + tid * kRedThreads;
    for (int b = q.rank; b < kBigGrid; b += q.size) __hip_atomic_store(prev + b, kEmptySlot, __ATOMIC_RELAXED, AGENT);
    __hip_atomic_store((unsigned long long*)slots + phase * kBufSlots + tid * kRedThreads + blockIdx.x, kEmptySlot,
                       __ATOMIC_RELAXED, AGENT);
}

// Canonical sum in a closed gang: its blocks publish the values of all 256 (lanes(b) is this thread's lane sum in
// the place of block b) in slots of their own.  False if the exchange failed.
template <class L, typename Fn>
__device__ __forceinline__ bool gang_sum(const Gang& q, ExLds<L::K>& X, double* slots, int& phase, unsigned* bar,
                                         double* out, Fn lanes) {
    static_assert(L::NB == kBigGrid && L::K == 1, "the grid that needs it");
    const int tid = threadIdx.x;
    unsigned long long* gs = (unsigned long long*)slots + kGangSlots;
    for (int b = q.rank; b < kBigGrid; b += q.size) {
        double acc[1] = {lanes(b)};
        const double v = block_value<L>(acc, X);
        if (tid < 64) {
            // the slots emptied after the last exchange are seen empty before this value is seen
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
            if (tid == 0)
                __hip_atomic_store(gs + phase * kRedThreads + b, slot_bits(v), __ATOMIC_RELAXED, AGENT);
        }
        __syncthreads();   // the block's LDS is free again
    }
    if (tid < 64) {
        unsigned long long u[4];
        long spins = 0;
        int err = 0;
        for (;;) {
            bool miss = false;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                u[k] = __hip_atomic_load(gs + phase * kRedThreads + tid + 64 * k, __ATOMIC_RELAXED, AGENT);
                miss = miss || u[k] == kEmptySlot;
            }
            if (!__any(miss)) break;
            if (++spins > kSpinLimit || ((spins & 1023) == 0 && __hip_atomic_load(bar + kBarErr, __ATOMIC_RELAXED, AGENT))) {
                if (tid == 0) __hip_atomic_store(bar + kBarErr, 1u, __ATOMIC_RELAXED, AGENT);
                err = kExFailed;
                break;
            }
        }
        const double v = final_value(u);
        for (int b = q.rank + q.size * tid; b < kBigGrid; b += q.size * 64)
            __hip_atomic_store(gs + (phase == 0 ? 2 : phase - 1) * kRedThreads + b, kEmptySlot, __ATOMIC_RELAXED, AGENT);
        if (tid == 0) {
            X.out = v;
            X.err = err;
        }
    }
    __syncthreads();
    phase = phase == 2 ? 0 : phase + 1;
    *out = X.out;
    const bool ok = X.err == 0;
    __syncthreads();   // X.out is read before the next exchange writes it
    return ok;
}

// A failed exchange: the results are invalid; later columns do nothing.
__device__ __forceinline__ void exchange_failed(int* ints, bool stop) {
    if (threadIdx.x != 0) return;
    if (stop) __hip_atomic_store(ints + 1, 1, __ATOMIC_RELAXED, AGENT);
    __hip_atomic_fetch_or(ints + 2, (int)ROK_FLAG_BARRIER, __ATOMIC_RELAXED, AGENT);
}

// Buffer descriptor word 3 for raw (untyped, unswizzled) loads on gfx9-class
// devices: data format 32 (a zero format would make every access out of range).
constexpr int kBufWord3 = 0x00020000;

// Loads of the basis vectors: the share (in sixteenths) of the next vector that the waves 1-15 load before
// a pass's block tree, the rest when the block's value is out, and the cache hint (2: non-temporal).  Past 2 M
// elements (16 per thread) the basis is larger than the last-level cache: non-temporal, and a quarter early
// (1024^2 step: 3038 us; half early 3083, none 3075, half early with plain loads 3101).  Below, plain loads, whose
// lines a later column finds again, and half early (64^3 basis of 24: 3327 us; none early 3544, all
// early 3599, half early with the non-temporal hint 3556).
template <class L>
struct Fetch {
    static constexpr bool kLarge = L::E >= 16;
    static constexpr int kHint = kLarge ? 2 : 0;
    static constexpr int kEarly = L::NB == 1 ? 16 : (kLarge ? 4 : 8);
};

// x[i] = the lane's element i of src where it lies below n, +0.0 past the end,
// for X0 <= i < X1 (the rest of x untouched).  Raw buffer loads with the range
// n * 8 bytes: an offset past the
// range reads as zero without touching memory, so the loads need no per-lane
// condition (no exec-masked branches, whose joins would make the compiler
// wait for every outstanding load, prefetches included).  All offsets are in
// the lane's offset register, which is what the range check covers; an opaque
// base offset has the element offsets formed next to each load instead of
// being held in registers across the whole kernel.
template <class L, int X0, int X1, int AUX>
__device__ __forceinline__ void load_range(const double* __restrict__ src, long n, double (&x)[L::E]) {
    const __amdgpu_buffer_rsrc_t r =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<double*>(src), (short)0, (int)(n * 8), kBufWord3);
    int off = L::base() * 8;
    asm volatile("" : "+v"(off));
#pragma unroll
    for (int i = X0; i < X1; ++i)
        x[i] = __builtin_bit_cast(double, __builtin_amdgcn_raw_buffer_load_b64(r, off + L::step(i) * 8, 0, AUX));
}

template <class L, int AUX = 0>
__device__ __forceinline__ void load_lane(const double* __restrict__ src, long n, double (&x)[L::E]) {
    load_range<L, 0, L::E, AUX>(src, n, x);
}

// dst's elements of the lane = x where they lie below n (raw buffer stores
// with the range n * 8 bytes: stores past it are dropped).
template <class L>
__device__ __forceinline__ void store_lane(double* __restrict__ dst, long n, const double (&x)[L::E]) {
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(dst, (short)0, (int)(n * 8), kBufWord3);
    using B64 = decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0, 0, 0));
    int off = L::base() * 8;
    asm volatile("" : "+v"(off));
#pragma unroll
    for (int i = 0; i < L::E; ++i)
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(B64, x[i]), r, off + L::step(i) * 8, 0, 0);
}

// Work vector storage of one lane: registers, or (PER = 16, where three
// register arrays of 16 doubles would exceed the 128 registers a lane has at
// 1024 threads per block) the lane's own LDS slots, used as private storage.
template <int PER, bool LDSW>
struct LaneVec {
    double r[LDSW ? 1 : PER];
    double* l;
    __device__ __forceinline__ double get(int k) const { return LDSW ? l[k * kPT + threadIdx.x] : r[k]; }
    __device__ __forceinline__ void set(int k, double x) {
        if constexpr (LDSW) l[k * kPT + threadIdx.x] = x;
        else r[k] = x;
    }
};

// The end of a column with sum of squares nn: writes h_{j+1,j} (block `lead`), returns it, *brk: breakdown.
__device__ __forceinline__ double column_norm(double nn, const double* hcol, int M, int j, double* H, int* ints, bool lead,
                                              bool* brk) {
    const double hn = sqrt(nn);
    double c = 0.0;
    for (int q = 0; q <= j; ++q) c = c + hcol[q] * hcol[q];
    c = c + hn * hn;
    *brk = hn <= kBreakdownTolR * sqrt(c);
    if (lead && threadIdx.x == 0) {
        H[(j + 1) * M + j] = hn;
        if (*brk) {
            ints[0] = j + 1;
            ints[1] = 1;
            ints[2] |= ROK_FLAG_BREAKDOWN;
        }
        if (!(hn == hn) || hn == __builtin_inf()) ints[2] |= ROK_FLAG_NONFINITE;
    }
    return hn;
}

// The column by a closed gang: w in memory (its buffer is free to change), the passes of k_mgs_resident.  False if an exchange failed.
template <class L>
__device__ __forceinline__ bool gang_column(double* w, const double* V, long n, int M, int j, double* H, double* vnext,
                                            int* ints, double* slots, unsigned* bar, ExLds<L::K>& X, double* hcol) {
    const Gang q = X.gang;
    const bool lead = q.rank == 0;
    int phase = (int)bar[kBarGangPhase];
    double h = 0.0;
    for (int i = 0; i <= j; ++i) {
        const double *prev = V + (long)(i - 1) * n, *cur = V + (long)i * n;
        if (!gang_sum<L>(q, X, slots, phase, bar, &h, [&](int b) {
                double acc = 0.0;
                for (int c = 0; c < L::C; ++c) {
                    const long e = L::base(b) + (long)c * kLanes;
                    if (e >= n) continue;
                    double wk = w[e];
                    if (i > 0) {
                        wk = wk - h * prev[e];
                        w[e] = wk;
                    }
                    acc = acc + cur[e] * wk;
                }
                return acc;
            }))
            return false;
        if (threadIdx.x == 0) {
            hcol[i] = h;
            if (lead) H[i * M + j] = h;
        }
    }
    double nn = 0.0;
    if (j + 1 < M) {
        const double* last = V + (long)j * n;
        if (!gang_sum<L>(q, X, slots, phase, bar, &nn, [&](int b) {
                double acc = 0.0;
                for (int c = 0; c < L::C; ++c) {
                    const long e = L::base(b) + (long)c * kLanes;
                    if (e >= n) continue;
                    const double wk = w[e] - h * last[e];
                    w[e] = wk;
                    acc = acc + wk * wk;
                }
                return acc;
            }))
            return false;
    }
    // every block has read the word: all have taken part in an exchange since
    if (lead && threadIdx.x == 0) bar[kBarGangPhase] = (unsigned)phase;
    if (j + 1 >= M) return true;
    bool brk;
    const double hn = column_norm(nn, hcol, M, j, H, ints, lead, &brk);
    if (brk) return true;
    for (int b = q.rank; b < kBigGrid; b += q.size)
        for (int c = 0; c < L::C; ++c) {
            const long e = L::base(b) + (long)c * kLanes;
            if (e < n) vnext[e] = w[e] / hn;
        }
    return true;
}

template <class L>
__global__ __launch_bounds__(kPT) void k_mgs_resident(double* wsrc, const double* V, long n, int M, int j,
                                                     double* H, double* vnext, int* ints, double* slots,
                                                     unsigned* bar, int hold) {
    constexpr int E = L::E, K = L::K, C = L::C;
    constexpr bool LDSW = E >= 16;
    __shared__ ExLds<K> X;
    __shared__ double s_w[LDSW ? E * kPT : 1];
    __shared__ int s_stop, s_phase;
    // w and v_0 are on their way while the gate answers
    double x0[E], A[E], B[E];
    load_lane<L>(wsrc, n, x0);
    load_lane<L, Fetch<L>::kHint>(V, n, A);
    if (threadIdx.x == 0) {
        if constexpr (L::NB == kBigGrid) X.gang = enter(bar, hold);
        s_stop = ints[1];
        s_phase = L::NB > 1 ? (int)bar[kBarPhase] : 0;
    }
    __syncthreads();
    if (s_stop || (L::NB == kBigGrid && X.gang.rank < 0)) return;
    int phase = s_phase;
    // Two basis-vector arrays alternate: at pass i one holds v_{i-1} (for the
    // update w -= h v_{i-1}) and v_{i+1} is loaded into it after use: by the
    // waves 1-15 before and during the exchange, by wave 0, which polls, when
    // its polls are done (one block alone: by every wave at once).
    const bool prefetch = L::NB == 1 || threadIdx.x >= 64;
    // Lanes past the end hold +0.0: their products are +0.0 and adding +0.0
    // to a lane sum that starts at +0.0 leaves it unchanged.
    LaneVec<E, LDSW> w;
    w.l = s_w;
#pragma unroll
    for (int i = 0; i < E; ++i) w.set(i, x0[i]);
    __shared__ double s_hcol[kMaxM + 1];
    double h = 0.0;
    int failed = 0;
    auto none = [] {};
    // Pass i with cur = v_i and prev = v_{i-1}: w -= h_{i-1} prev (i > 0),
    // h_i = <v_i, w>, then prev <- v_{i+1}.
    auto pass = [&](int i, double (&cur)[E], double (&prev)[E]) {
        double acc[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            acc[k] = 0.0;
#pragma unroll
            for (int c = 0; c < C; ++c) {
                const int x = k * C + c;
                double wk = w.get(x);
                if (i > 0) {
                    wk = wk - h * prev[x];
                    w.set(x, wk);
                }
                acc[k] = acc[k] + cur[x] * wk;
            }
        }
        // the sums are complete before the loads are issued: otherwise the
        // products sink past the (conditional) loads and the merge after them
        // waits for every outstanding load, the prefetch included
#pragma unroll
        for (int k = 0; k < K; ++k) asm volatile("" : "+v"(acc[k]) : : "memory");
        const bool more = i < j;
        constexpr int XS = (E * Fetch<L>::kEarly) / 16, kHint = Fetch<L>::kHint;
        const double* next = V + (long)(more ? i + 1 : j) * n;
        if (more && prefetch) load_range<L, 0, XS, kHint>(next, n, prev);
        auto mid = [&] {
            if (more) load_range<L, XS, E, kHint>(next, n, prev);
        };
        // unconditional (v_j again after the last pass, 64 lanes' worth): no branch around the loads
        auto after = [&] { load_lane<L, kHint>(next, n, prev); };
        failed = grid_sum<L>(acc, X, slots, phase, bar, i == 0, &h, mid, after);
        if (failed) return;
        if (threadIdx.x == 0) s_hcol[i] = h;
        if (blockIdx.x == 0 && threadIdx.x == 0) H[i * M + j] = h;
    };
    int i = 0;
    for (;;) {
        pass(i, A, B);
        if (failed || i == j) break;
        ++i;
        pass(i, B, A);
        if (failed || i == j) break;
        ++i;
    }
    if (failed) {
        if constexpr (L::NB == kBigGrid) {
            if (failed == kExClosed) {
                gang_start(X.gang, slots, phase);
                if (gang_column<L>(wsrc, V, n, M, j, H, vnext, ints, slots, bar, X, s_hcol)) return;
            }
        }
        exchange_failed(ints, true);
        return;
    }
    auto keep_phase = [&] {   // every block has read the word: all have taken part in an exchange since
        if (L::NB > 1 && blockIdx.x == 0 && threadIdx.x == 0) bar[kBarPhase] = (unsigned)phase;
    };
    if (j + 1 >= M) {
        keep_phase();
        return;
    }
    // last update w -= h_j v_j (v_j is A after an even number of passes, else B)
    const bool inA = (j % 2) == 0;
    double acc[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        acc[k] = 0.0;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int x = k * C + c;
            const double wk = w.get(x) - h * (inA ? A[x] : B[x]);
            w.set(x, wk);
            acc[k] = acc[k] + wk * wk;
        }
    }
    double nn;
    if (grid_sum<L>(acc, X, slots, phase, bar, false, &nn, none, none)) {
        exchange_failed(ints, true);
        return;
    }
    keep_phase();
    bool brk;
    const double hn = column_norm(nn, s_hcol, M, j, H, ints, blockIdx.x == 0, &brk);
    if (brk) return;
    double v[E];
#pragma unroll
    for (int x = 0; x < E; ++x) v[x] = w.get(x) / hn;
    store_lane<L>(vnext, n, v);
}

// Reverse of one Arnoldi column (the discrete adjoint of its modified
// Gram-Schmidt passes and of the normalisation v_{j+1} = w / h_{j+1,j}),
// resident like the forward kernel: w (the forward iterates, rebuilt pass
// by pass) and wbar stay in registers, so reverse pass i streams only
// v_{i-1} (for the next dot) and reads and writes vbar_i.  Rules, with x'
// the result of a forward operation:
//   v = w / rho, rho = ||w||:  wbar = vbar / rho + (Hbar_rho - <vbar, v> / rho) v
//   w' = w - h v, h = <v, w>:  hb = Hbar_h - <w'bar, v>, w = w' + h v,
//                              vbar += hb w - h w'bar, wbar = w'bar + hb v
// The final forward iterate is h_{j+1,j} v_{j+1} where v_{j+1} exists, else
// (the basis' last column) J v_j - sum_i h_ij v_i with J v_j read from wsrc.
// Every dot product is the canonical sum (the same lane order and finish as
// the per-pass reverse kernels, whose results this reproduces bit for bit).
// Nothing runs for j >= M_eff or after a failed in-kernel barrier.
template <class L>
__device__ __forceinline__ bool gang_reverse(double* w, const double* V, double* Vbar, const double* sh, const double* shb, long n,
                                             int j, bool nrm, double* wbar, double* slots, unsigned* bar, ExLds<L::K>& X) {
    // by a closed gang, w and wbar in memory
    const Gang q = X.gang;
    int phase = (int)bar[kBarGangPhase];
    double d = 0.0, rho = 0.0, coef = 0.0;
    const double *vn = V + (long)(j + 1) * n, *vbn = Vbar + (long)(j + 1) * n, *vj = V + (long)j * n;
    auto sum = [&](auto term) {
        return gang_sum<L>(q, X, slots, phase, bar, &d, [&](int b) {
            double acc = 0.0;
            for (int c = 0; c < L::C; ++c) {
                const long e = L::base(b) + (long)c * kLanes;
                if (e < n) acc = acc + term(e);
            }
            return acc;
        });
    };
    if (nrm) {
        if (!sum([&](long e) { return vbn[e] * vn[e]; })) return false;
        rho = sh[j + 1];
        coef = shb[j + 1] - d / rho;
    }
    if (!sum([&](long e) {
            double wk, b;
            if (nrm) {
                wk = rho * vn[e];
                b = vbn[e] / rho + coef * vn[e];
            } else {
                wk = w[e];
                for (int i = 0; i <= j; ++i) wk = wk - sh[i] * V[(long)i * n + e];
                b = 0.0;
            }
            w[e] = wk;
            wbar[e] = b;
            return b * vj[e];
        }))
        return false;
    for (int i = j; i >= 0; --i) {
        const double h = sh[i], hb = shb[i] - d;
        const double *cur = V + (long)i * n, *prev = V + (long)(i - 1) * n;
        double* vb = Vbar + (long)i * n;
        auto pass = [&](long e) {
            const double v = cur[e];
            const double wo = w[e] + h * v;
            w[e] = wo;
            const double b = wbar[e];
            vb[e] = vb[e] + hb * wo - h * b;
            const double wn = b + hb * v;
            wbar[e] = wn;
            return wn;
        };
        if (i > 0) {
            if (!sum([&](long e) { return pass(e) * prev[e]; })) return false;
        } else {
            for (int b = q.rank; b < kBigGrid; b += q.size)
                for (int c = 0; c < L::C; ++c) {
                    const long e = L::base(b) + (long)c * kLanes;
                    if (e < n) pass(e);
                }
        }
    }
    if (q.rank == 0 && threadIdx.x == 0) bar[kBarGangPhase] = (unsigned)phase;
    return true;
}

template <class L>
__global__ __launch_bounds__(kPT) void k_mgs_rev_resident(double* wsrc, const double* V, double* Vbar,
                                                         const double* H, const double* Hbar, long n, int M, int j,
                                                         double* wbar_out, int* ints, double* slots,
                                                         unsigned* bar, int hold) {
    constexpr int E = L::E, K = L::K, C = L::C;
    __shared__ ExLds<K> X;
    __shared__ int s_m, s_bad, s_phase;
    __shared__ double s_h[kMaxM + 1], s_hb[kMaxM + 1];   // column j of H and Hbar
    if (threadIdx.x == 0) {
        if constexpr (L::NB == kBigGrid) X.gang = enter(bar, hold);
        s_m = ints[0];
        s_bad = (ints[2] & ROK_FLAG_BARRIER) != 0;
        s_phase = L::NB > 1 ? (int)bar[kBarPhase] : 0;
    }
    if (threadIdx.x < M && threadIdx.x <= j + 1) {
        s_h[threadIdx.x] = H[threadIdx.x * M + j];
        s_hb[threadIdx.x] = Hbar[threadIdx.x * M + j];
    }
    __syncthreads();
    const int m = s_m;
    if (j >= m || s_bad || (L::NB == kBigGrid && X.gang.rank < 0)) return;
    const bool nrm = j + 1 < m;
    double w[E], wb[E], A[E], B[E], vb[E];
    int phase = s_phase;
    double d = 0.0;
    int failed = 0;
    // canonical sum of the lane sums acc; the caller's prefetch: early() by the waves 1-15 before the block's tree,
    // late() by them when the block's value is out, both by wave 0 after its polls.  (Gradient at 512^2 on one card: v early and
    // vbar late 7550 us, the other way round 7583, both late 7693, both early 7682; from card to card the first varies from 7550 to 7660.)
    auto exchange = [&](double (&acc)[K], bool first, auto early, auto late) {
#pragma unroll
        for (int k = 0; k < K; ++k) asm volatile("" : "+v"(acc[k]) : : "memory");
        if (L::NB == 1 || threadIdx.x >= 64) early();
        if constexpr (L::NB == 1) late();
        failed = grid_sum<L>(acc, X, slots, phase, bar, first, &d, late, [&] {
            early();
            late();
        });
    };
    if (nrm) {
        load_lane<L>(V + (long)(j + 1) * n, n, A);      // v_{j+1}
        load_lane<L>(Vbar + (long)(j + 1) * n, n, vb);  // vbar_{j+1}
        double acc[K];
#pragma unroll
        for (int x = 0; x < E; ++x) acc[x / C] = (x % C ? acc[x / C] : 0.0) + vb[x] * A[x];
        exchange(acc, true, [&] { load_lane<L>(V + (long)j * n, n, B); }, [] {});
        if (failed) goto fail;
        const double rho = s_h[j + 1];
        const double coef = s_hb[j + 1] - d / rho;
#pragma unroll
        for (int k = 0; k < E; ++k) {
            w[k] = rho * A[k];
            wb[k] = vb[k] / rho + coef * A[k];
        }
    } else {
        load_lane<L>(wsrc, n, w);
        for (int i = 0; i <= j; ++i) {
            load_lane<L>(V + (long)i * n, n, B);
            const double hij = s_h[i];
#pragma unroll
            for (int k = 0; k < E; ++k) w[k] = w[k] - hij * B[k];
        }
#pragma unroll
        for (int k = 0; k < E; ++k) wb[k] = 0.0;
    }
    {   // <wbar, v_j>; meanwhile v_{j-1} and vbar_j arrive
        double acc[K];
#pragma unroll
        for (int x = 0; x < E; ++x) acc[x / C] = (x % C ? acc[x / C] : 0.0) + wb[x] * B[x];
        exchange(acc, !nrm, [&] { load_lane<L>(V + (long)(j > 0 ? j - 1 : 0) * n, n, A); },
                 [&] { load_lane<L>(Vbar + (long)j * n, n, vb); });
        if (failed) goto fail;
    }
    {
        // reverse pass i with cur = v_i, prev = v_{i-1}, vb = vbar_i, d = <wbar, v_i>
        auto rpass = [&](int i, double (&cur)[E], double (&prev)[E]) {
            const double h = s_h[i];
            const double hb = s_hb[i] - d;
            double acc[K];
#pragma unroll
            for (int k = 0; k < E; ++k) {
                const double v = cur[k];
                const double wo = w[k] + h * v;
                w[k] = wo;
                const double b = wb[k];
                vb[k] = vb[k] + hb * wo - h * b;
                const double wn = b + hb * v;
                wb[k] = wn;
                acc[k / C] = (k % C ? acc[k / C] : 0.0) + wn * prev[k];
            }
            store_lane<L>(Vbar + (long)i * n, n, vb);
            if (i == 0) return;
            exchange(acc, false, [&] { load_lane<L>(V + (long)(i > 1 ? i - 2 : 0) * n, n, cur); },
                     [&] { load_lane<L>(Vbar + (long)(i - 1) * n, n, vb); });
        };
        int i = j;
        for (;;) {
            rpass(i, B, A);
            if (failed || i == 0) break;
            --i;
            rpass(i, A, B);
            if (failed || i == 0) break;
            --i;
        }
        if (failed) goto fail;
    }
    store_lane<L>(wbar_out, n, wb);
    // every block has read the word: all have taken part in an exchange since
    if (L::NB > 1 && blockIdx.x == 0 && threadIdx.x == 0) bar[kBarPhase] = (unsigned)phase;
    return;
fail:
    if constexpr (L::NB == kBigGrid) {
        if (failed == kExClosed) {
            gang_start(X.gang, slots, phase);
            if (gang_reverse<L>(wsrc, V, Vbar, s_h, s_hb, n, j, nrm, wbar_out, slots, bar, X)) return;
        }
    }
    exchange_failed(ints, false);
}

// The shape of a vector of n elements (n <= 16 * 262144): fn(Lanes<...>{}).  MAXE: most elements per thread
// the kernel holds.  The lines, in us a column of a basis of 24 columns: one block 25.4 at 8192 and eight blocks 26.7 at
// 16384; eight blocks 28.1 at 32768 (256: 32.6) and 35.1 at 65536 (256: 32.7).
template <int MAXE, typename Fn>
static hipError_t with_shape(long n, Fn fn) {
    if (n <= 1024) return fn(Lanes<1, 1, 1>{});
    if (n <= 2048) return fn(Lanes<1, 2, 1>{});
    if (n <= 4096) return fn(Lanes<1, 4, 1>{});
    if (n <= 8192) return fn(Lanes<1, 8, 1>{});
    if (n <= 16384) return fn(Lanes<kMidGrid, 2, 1>{});
    if (n <= 32768) return fn(Lanes<kMidGrid, 4, 1>{});
    if (n <= kLanes) return fn(Lanes<kBigGrid, 1, 1>{});
    if (n <= 2L * kLanes) return fn(Lanes<kBigGrid, 1, 2>{});
    if (n <= 4L * kLanes) return fn(Lanes<kBigGrid, 1, 4>{});
    if (n <= 8L * kLanes) return fn(Lanes<kBigGrid, 1, 8>{});
    if constexpr (MAXE >= 16)
        if (n <= 16L * kLanes) return fn(Lanes<kBigGrid, 1, 16>{});
    return hipErrorInvalidValue;
}

// Whether the resident kernel takes vectors of n elements.
bool mgs_resident_fits(long n) { return n <= 16L * kLanes; }

// True if the device holds kernel f's 256 blocks at once.
static bool grid_resident(const void* f) {
    int dev = 0, cus = 0, nb = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, f, kPT, 0) != hipSuccess)
        return false;
    return (long)nb * cus >= kBigGrid;
}

static int g_fwd_ok = -1;

// True if the device can host the forward kernels' grid (checked once).
bool mgs_resident_available() {
    if (g_fwd_ok < 0) g_fwd_ok = grid_resident((const void*)k_mgs_resident<Lanes<kBigGrid, 1, 16>>) ? 1 : 0;
    return g_fwd_ok == 1;
}

hipError_t launch_mgs_resident(const Work& W, double* w, const double* V, long n, int M, int j, double* vnext,
                               hipStream_t st, int hold) {
    double* H = W.H;
    int* ints = W.ints;
    double* slots = W.gpart;
    unsigned* bar = W.bar;
    void* args[] = {(void*)&w, (void*)&V, (void*)&n, (void*)&M, (void*)&j, (void*)&H, (void*)&vnext,
                    (void*)&ints, (void*)&slots, (void*)&bar, (void*)&hold};
    return with_shape<16>(n, [&](auto shape) {
        using L = decltype(shape);
        return hipLaunchKernel((const void*)k_mgs_resident<L>, dim3(L::NB), dim3(kPT), args, 0, st);
    });
}

static int g_rev_ok = -1;

// The resident reverse keeps five lane vectors in registers: up to 8 elements per lane.
bool mgs_rev_resident_available(long n) {
    if (n > 8L * kLanes) return false;
    if (g_rev_ok < 0) g_rev_ok = grid_resident((const void*)k_mgs_rev_resident<Lanes<kBigGrid, 1, 8>>) ? 1 : 0;
    return g_rev_ok == 1;
}

hipError_t launch_mgs_rev_resident(const Work& W, const AdjWork& A, int M, int j, long n, hipStream_t st, int hold) {
    double* wsrc = W.w;
    const double* V = W.V;
    double* Vbar = A.Vbar;
    const double* H = W.H;
    const double* Hbar = A.Hbar;
    double* wbar = A.wbar;
    int* ints = W.ints;
    double* slots = W.gpart;
    unsigned* bar = W.bar;
    void* args[] = {(void*)&wsrc, (void*)&V,  (void*)&Vbar, (void*)&H,    (void*)&Hbar,  (void*)&n,
                    (void*)&M,    (void*)&j,  (void*)&wbar, (void*)&ints, (void*)&slots, (void*)&bar, (void*)&hold};
    return with_shape<8>(n, [&](auto shape) {
        using L = decltype(shape);
        return hipLaunchKernel((const void*)k_mgs_rev_resident<L>, dim3(L::NB), dim3(kPT), args, 0, st);
    });
}

}  // namespace rok
