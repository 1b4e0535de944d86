// Krylov and stage kernels of the ROK step (Sec. 2.2.2, eq. 9): canonical
// reductions, modified Gram-Schmidt Arnoldi passes, the reduced (M x M) LU
// solve, projections V^T F, recoveries k = V lambda + h (F - V phi) and the
// state update.
//
// Reductions follow one canonical order (the same order the CPU oracle
// writes out): a fixed grid of kRedBlocks x kRedThreads lanes, lane t adds
// the elements t, t + T, t + 2T, ... (T = kRedBlocks * kRedThreads) in index
// order, each block combines its lanes by a pairwise halving tree into one
// partial, and the consumer finishes the sum (lane t adds partials t, t+256,
// t+512, t+768, then the tree).  There is no inter-block communication
// inside a kernel: the kernel boundary publishes the partials, so no memory
// fence or atomic is needed, and every block that finishes a sum obtains the
// same bits.
#include "rok.h"
#include "rok_device.hpp"
#include "rok_kernels.hpp"

namespace rok {

constexpr double kBreakdownTol = 1e-13;
constexpr double kEpsMach = 2.220446049250313e-16;   // 2^-52

// Block of kRedThreads threads: the halving tree; every thread gets the sum.
__device__ __forceinline__ double block_sum(double acc, double* s) {
    __shared__ double s_r;
    double r = tree256(acc, s);
    if (threadIdx.x == 0) s_r = r;
    __syncthreads();
    r = s_r;
    __syncthreads();
    return r;
}

// Final stage of the canonical sum (every thread of a kRedThreads block calls it).
__device__ __forceinline__ double final_sum(const double* partials, double* s) {
    double acc = 0.0;
    for (int b = threadIdx.x; b < kRedBlocks; b += kRedThreads) acc = acc + partials[b];
    return block_sum(acc, s);
}

__device__ __forceinline__ bool nonfinite(double x) { return !(x == x) || fabs(x) == __builtin_inf(); }

// Per-lane sums in index order, block tree, one partial per block.
//   UPD:  first w <- w - h vprev, h = finished sum of hpart (block 0 stores
//         it to *hstore); w is written back
//   SELF: sum of w.w, else of vcur.w
template <bool UPD, bool SELF>
__global__ __launch_bounds__(kRedThreads) void k_red(double* w, const double* vprev, const double* hpart,
                                                    double* hstore, const double* vcur, long n,
                                                    const int* ints, double* partials) {
    __shared__ double s[kRedThreads];
    if (ints && ints[1]) return;
    double h = 0.0;
    if constexpr (UPD) {
        h = final_sum(hpart, s);
        if (blockIdx.x == 0 && threadIdx.x == 0) *hstore = h;
    }
    double acc = 0.0;
    const long stride = (long)kRedBlocks * kRedThreads;
    long e = (long)blockIdx.x * kRedThreads + threadIdx.x;
    for (; e + stride < n; e += 2 * stride) {
        double w0 = ld_stream(w + e), w1 = ld_stream(w + e + stride);
        if constexpr (UPD) {
            double a0 = ld_stream(vprev + e), a1 = ld_stream(vprev + e + stride);
            w0 = w0 - h * a0;
            w1 = w1 - h * a1;
            w[e] = w0;
            w[e + stride] = w1;
        }
        double b0, b1;
        if constexpr (SELF) {
            b0 = w0;
            b1 = w1;
        } else {
            b0 = ld_stream(vcur + e);
            b1 = ld_stream(vcur + e + stride);
        }
        acc = acc + b0 * w0;
        acc = acc + b1 * w1;
    }
    if (e < n) {
        double we = ld_stream(w + e);
        if constexpr (UPD) {
            we = we - h * ld_stream(vprev + e);
            w[e] = we;
        }
        if constexpr (SELF) acc = acc + we * we;
        else acc = acc + ld_stream(vcur + e) * we;
    }
    double bs = block_sum(acc, s);
    if (threadIdx.x == 0) partials[blockIdx.x] = bs;
}

enum { FIN_SQRT_TO = 0, FIN_STORE = 1, FIN_EPS = 2 };

// One block: finishes a sum and applies the bookkeeping of `op`.
__global__ __launch_bounds__(kRedThreads) void k_finish(const double* partials, int op, double* out, double* scal,
                                                       int* ints) {
    __shared__ double s[kRedThreads];
    if (op == FIN_STORE && ints[1]) return;
    double tot = final_sum(partials, s);
    if (threadIdx.x != 0) return;
    if (op == FIN_SQRT_TO) {
        *out = sqrt(tot);
    } else if (op == FIN_STORE) {
        *out = tot;
        if (nonfinite(tot)) ints[2] |= ROK_FLAG_NONFINITE;
    } else {  // FIN_EPS: eps = sqrt((1 + ||y||) u) / ||v||
        double ny = sqrt(tot);
        scal[0] = ny;
        double e = sqrt((1.0 + ny) * kEpsMach);
        scal[1] = e / scal[3];
    }
}

// v_{j+1} = w / h_{j+1,j}, h_{j+1,j} = sqrt(w.w) finished from `partials`,
// after the breakdown test h_{j+1,j} <= tol ||(h_1j, ..., h_{j+1,j})||.
__global__ __launch_bounds__(kRedThreads) void k_normalize(const double* w, const double* partials, double* H, int M,
                                                          int j, double* v, long n, int* ints) {
    __shared__ double s[kRedThreads];
    if (ints[1]) return;
    const double hn = sqrt(final_sum(partials, s));
    double c = 0.0;
    for (int i = 0; i <= j; ++i) c = c + H[i * M + j] * H[i * M + j];
    c = c + hn * hn;
    const bool brk = hn <= kBreakdownTol * sqrt(c);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        H[(j + 1) * M + j] = hn;
        if (brk) {
            ints[0] = j + 1;
            ints[1] = 1;
            ints[2] |= ROK_FLAG_BREAKDOWN;
        }
        if (nonfinite(hn)) ints[2] |= ROK_FLAG_NONFINITE;
    }
    if (brk) return;
    const long stride = (long)gridDim.x * blockDim.x;
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) v[e] = ld_stream(w + e) / hn;
}

// Partials of f.f and, with y, of y.y (the two norms a basis starts from), by the
// first nb blocks' lanes.
__global__ __launch_bounds__(kRedThreads) void k_norms(const double* y, const double* f, long n, const int* ints,
                                                      double* pf, double* py) {
    __shared__ double s[kRedThreads];
    if (ints[1]) return;
    const long stride = (long)kRedBlocks * kRedThreads;
    double af = 0.0, ay = 0.0;
    for (long e = (long)blockIdx.x * kRedThreads + threadIdx.x; e < n; e += stride) {
        const double fe = f[e], ye = y ? y[e] : 0.0;
        af = af + fe * fe;
        ay = ay + ye * ye;
    }
    const double bf = block_sum(af, s);
    if (threadIdx.x == 0) pf[blockIdx.x] = bf;
    if (y) {
        const double by = block_sum(ay, s);
        if (threadIdx.x == 0) py[blockIdx.x] = by;
    }
}

// v_0 = f / beta, beta = ||f|| finished from pf by every block; the first block also keeps beta and, with py,
// ||y|| and eps = sqrt((1 + ||y||) u).  A zero f ends the basis (M_eff = 0).
__global__ __launch_bounds__(kRedThreads) void k_start(const double* f, const double* pf, const double* py, int nb,
                                                      double* v, long n, int* ints, double* scal) {
    __shared__ double s_beta;
    if (ints[1]) return;
    if (threadIdx.x < 64) {
        const double b = sqrt(wave_final(pf, nb));
        if (threadIdx.x == 0) s_beta = b;
    } else if (py && blockIdx.x == 0 && threadIdx.x < 128) {
        const double ny = sqrt(wave_final(py, nb));
        if (threadIdx.x == 64) {
            scal[0] = ny;
            scal[1] = sqrt((1.0 + ny) * kEpsMach);
        }
    }
    __syncthreads();
    const double beta = s_beta;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        scal[2] = beta;
        if (beta == 0.0) {
            ints[0] = 0;
            ints[1] = 1;
            ints[2] |= ROK_FLAG_ZERO_RHS;
        }
        if (nonfinite(beta)) ints[2] |= ROK_FLAG_NONFINITE;
    }
    if (beta == 0.0) return;
    const long stride = (long)gridDim.x * blockDim.x;
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) v[e] = f[e] / beta;
}

// The normalisation's bookkeeping without the division: h_{j+1,j} = sqrt(w.w)
// from `partials`, the breakdown test of k_normalize, and sig[j+1] =
// 1 / h_{j+1,j}, the scale of the unnormalised column (one block).
__global__ __launch_bounds__(kRedThreads) void k_norm_scale(const double* partials, double* H, int M, int j,
                                                           int* ints, double* sig) {
    __shared__ double s[kRedThreads];
    if (ints[1]) return;
    const double hn = sqrt(final_sum(partials, s));
    if (threadIdx.x != 0) return;
    double c = 0.0;
    for (int i = 0; i <= j; ++i) c = c + H[i * M + j] * H[i * M + j];
    c = c + hn * hn;
    H[(j + 1) * M + j] = hn;
    if (hn <= kBreakdownTol * sqrt(c)) {
        ints[0] = j + 1;
        ints[1] = 1;
        ints[2] |= ROK_FLAG_BREAKDOWN;
    } else {
        sig[j + 1] = 1.0 / hn;
    }
    if (nonfinite(hn)) ints[2] |= ROK_FLAG_NONFINITE;
}

__global__ void k_init(double* H, int nh, double* phi, double* lam, int nsm, double* scal, int* ints, int meff0,
                       unsigned* bar, int nbar, unsigned long long* slots, int nslot, double* sig, int nsig) {
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    for (int e = t; e < nslot; e += gridDim.x * blockDim.x) slots[e] = kExchangeEmpty;
    for (int e = t; e < nbar; e += gridDim.x * blockDim.x) bar[e] = 0u;
    for (int e = t; e < nsig; e += gridDim.x * blockDim.x) sig[e] = 1.0;
    for (int e = t; e < nh; e += gridDim.x * blockDim.x) H[e] = 0.0;
    for (int e = t; e < nsm; e += gridDim.x * blockDim.x) {
        phi[e] = 0.0;
        lam[e] = 0.0;
    }
    if (t < 16) scal[t] = 0.0;
    if (t < 32) ints[t] = (t == 0) ? meff0 : 0;   // M_eff, stop, flags, barrier words
}

__global__ void k_copy_h(const double* H, int M, double* Hout, const int* ints, int* meff_out) {
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    int m = ints[0];
    for (int e = t; e < M * M; e += gridDim.x * blockDim.x) {
        int i = e / M, j = e % M;
        Hout[e] = (i < m && j < m) ? H[i * M + j] : 0.0;
    }
    if (t == 0 && meff_out) *meff_out = m;
}

// LU with partial pivoting of A = I - hg H (M_eff x M_eff) by one wave, lane r
// holding row r in registers.  Each entry sees the same sequence of
// operations as the textbook right-looking elimination: the first largest |entry| of the column is the pivot, and
// rows keep their lanes, a swap exchanging their positions only.  After step k
// a lane's registers hold columns k + 1, ..., so that every step reads register 0
// for its column; the multipliers go to L (kMaxM x 64 doubles of LDS).  Bound by its
// chain of pivot searches and divisions.  (A block of four waves on an LDS matrix, five
// barriers per step: 15.8 us at M = 16, 7 us at M = 8.)
template <int MB>
__device__ __forceinline__ void lu_wave(const double* H, int M, double hg, double* LU, int* perm, int m, double* L) {
    const int lane = threadIdx.x & 63;
    double a[MB];
#pragma unroll
    for (int c = 0; c < MB; ++c)
        a[c] = (lane < m && c < m) ? (lane == c ? 1.0 : 0.0) - hg * H[lane * M + c] : 0.0;
    int pos = lane;           // the row's position: final once it has been the pivot row
    bool alive = lane < m;
    for (int k = 0; k < m; ++k) {
        const double v = alive ? fabs(a[0]) : -1.0;
        double mx = (v == v) ? v : -1.0;   // a NaN is never larger
        mx = fmax(mx, lane_down<32>(mx));
        mx = fmax(mx, lane_down<16>(mx));
        mx = fmax(mx, lane_down<8>(mx));
        mx = fmax(mx, lane_down<4>(mx));
        mx = fmax(mx, lane_down<2>(mx));
        mx = lane_value(fmax(mx, lane_down<1>(mx)), 0);
        const unsigned long long at_k = __ballot(alive && pos == k);
        const int row_k = __ffsll((long long)at_k) - 1;
        unsigned long long cand = __ballot(alive && v == mx);
        int p = row_k;
        const double vk = lane_value(v, row_k);
        if (vk == vk && cand) {   // (a NaN in place is kept: nothing compares larger)
            p = __ffsll((long long)cand) - 1;
            int best = __builtin_amdgcn_readlane(pos, p);
            for (cand &= cand - 1; cand; cand &= cand - 1) {   // equal entries: the first position
                const int q = __ffsll((long long)cand) - 1;
                const int pq = __builtin_amdgcn_readlane(pos, q);
                if (pq < best) {
                    best = pq;
                    p = q;
                }
            }
        }
        const int pos_p = __builtin_amdgcn_readlane(pos, p);
        if (lane == row_k) pos = pos_p;
        if (lane == p) {
            pos = k;
            alive = false;
        }
        const double l = a[0] / lane_value(a[0], p);
        if (alive) L[k * 64 + lane] = l;
#pragma unroll
        for (int c = 1; c < MB; ++c) {
            const double u = lane_value(a[c], p);
            if (alive) a[c - 1] = a[c] - l * u;
        }
    }
    if (lane < m) {
        for (int c = 0; c < pos; ++c) LU[pos * M + c] = L[c * 64 + lane];
#pragma unroll
        for (int c = 0; c < MB; ++c)
            if (pos + c < m) LU[pos * M + pos + c] = a[c];
        perm[pos] = lane;
    }
}

template <int MB>
__global__ __launch_bounds__(64) void k_lu(const double* H, int M, double hg, double* LU, int* perm, const int* ints) {
    __shared__ double L[MB * 64];
    lu_wave<MB>(H, M, hg, LU, perm, ints[0], L);
}

struct GamRow {
    double g[kMaxStages];
};

constexpr int kSmallThreads = 1024;   // the reduced solve's block
constexpr int kLd = kMaxM + 1;        // leading dimension of its LDS matrices: rows and columns without bank conflicts

// phi_i = V^T F_i finished from the projection partials (one column per wave,
// canonical order), then
// lambda_i = LU^{-1} (h phi_i + h H sum_{j<i} gamma_ij lambda_j) on wave 0.
// Bound by latency: one memory round trip, the sums, then about M^2 / 2
// dependent subtractions.  Every load is issued before the first wait, for the
// compiled size M (entries past M_eff are loaded and never used).  In the back
// substitution all products of a row are formed at once (one per lane) and
// only their subtraction, in increasing column order, is serial.  At M = 16: 16.1 us
// with 256 threads summing 16 columns through LDS trees and the products in
// the chain.
__global__ __launch_bounds__(kSmallThreads) void k_lambda(const double* H, const double* LU, const int* perm, int M,
                                                         int i, GamRow gr, double h, const double* partials, int nb,
                                                         double* phi, double* lam, int* ints, const double* sig) {
    __shared__ double sphi[kMaxM], g[kMaxM];
    __shared__ double sLU[kMaxM * kLd], sH[kMaxM * kLd];
    const int tid = threadIdx.x, lane = tid & 63;
    const int m = ints[0];
    for (int e = tid; e < M * M; e += kSmallThreads) {
        const int r = e / M, c = e - r * M;
        sLU[r * kLd + c] = LU[e];
        sH[r * kLd + c] = H[e];
    }
    if (tid < M) {
        double a = 0.0;
        for (int j = 0; j < i; ++j)
            if (gr.g[j] != 0.0) a = a + gr.g[j] * lam[j * M + tid];
        g[tid] = a;
    }
    const int row = (tid < M) ? perm[tid] : tid;
    for (int c = tid >> 6; c < M; c += kSmallThreads / 64) {
        const double t = wave_final(partials + (long)c * kRedBlocks, nb);
        // a column stored unnormalised: <v_c, F> = sig_c <V_c, F>
        if (lane == 0) sphi[c] = sig ? t * sig[c] : t;
    }
    __syncthreads();
    if (tid >= 64) return;   // m <= kMaxM = 64: row r on lane r
    if (tid < m) phi[i * M + tid] = sphi[tid];
    double x = 0.0;
    if (tid < m) {   // x_r = h phi_r + h (H g)_r
        double hg = 0.0;
        for (int c = 0; c < m; ++c) hg = hg + sH[tid * kLd + c] * g[c];
        x = h * sphi[tid] + h * hg;
    }
    double yr = __shfl(x, tid < m ? row : tid, 64);   // placed at its pivoted position
    // forward substitution with the unit lower factor, column by column (each entry's updates in column order)
    double col = sLU[tid * kLd];
    for (int c = 0; c + 1 < m; ++c) {
        const double next = sLU[tid * kLd + c + 1];
        const double yc = lane_value(yr, c);
        if (tid > c && tid < m) yr = yr - col * yc;
        col = next;
    }
    // back substitution, row by row: a_r = y_r - sum_c U_rc y_c in increasing column order
    double u = m > 0 ? sLU[(m - 1) * kLd + tid] : 0.0;
    for (int r = m - 1; r >= 0; --r) {
        const double next = r > 0 ? sLU[(r - 1) * kLd + tid] : 0.0;
        const double pr = u * yr;
        double a = lane_value(yr, r);
#pragma unroll 4
        for (int c = r + 1; c < m; ++c) a = a - lane_value(pr, c);
        a = a / lane_value(u, r);
        if (tid == r) yr = a;
        u = next;
    }
    if (tid < m) lam[i * M + tid] = yr;
    const bool bad = __any(tid < m && nonfinite(yr));
    if (tid == 0 && bad) ints[2] |= ROK_FLAG_NONFINITE;
}

// Projection partials: for c < M_eff, canonical per-block partial sums of
// V[:, c] . F (finished by k_lambda).  MB >= M; the common case M_eff == MB
// runs a branch-free loop so all loads of an element are in flight together.
// With lu.LU the grid has one block more, the first, which factorises the
// step's reduced matrix meanwhile (nothing before the solve after this kernel needs it).
struct LuArgs {
    const double* H;
    double* LU;
    int* perm;
    int M;
    double hg;
};

template <int MB>
__global__ __launch_bounds__(kRedThreads) void k_project(const double* V, const double* F, long n, const int* ints,
                                                        double* partials, LuArgs lu) {
    __shared__ double sm[16][kRedThreads];
    const int m = ints[0];
    int block = blockIdx.x;
    if (lu.LU) {
        if (block == 0) {
            static_assert(sizeof(sm) >= sizeof(double) * 64 * kMaxM, "the multipliers");
            if (threadIdx.x < 64) lu_wave<MB>(lu.H, lu.M, lu.hg, lu.LU, lu.perm, m, &sm[0][0]);
            return;
        }
        --block;
    }
    double acc[MB];
#pragma unroll
    for (int c = 0; c < MB; ++c) acc[c] = 0.0;
    const long stride = (long)kRedBlocks * kRedThreads;
    if (m == MB) {
        for (long e = (long)block * kRedThreads + threadIdx.x; e < n; e += stride) {
            double fe = ld_stream(F + e);
            double vc[MB];
#pragma unroll
            for (int c = 0; c < MB; ++c) vc[c] = ld_stream(V + (long)c * n + e);
#pragma unroll
            for (int c = 0; c < MB; ++c) acc[c] = acc[c] + vc[c] * fe;
        }
    } else {
        for (long e = (long)block * kRedThreads + threadIdx.x; e < n; e += stride) {
            double fe = ld_stream(F + e);
#pragma unroll
            for (int c = 0; c < MB; ++c)
                if (c < m) acc[c] = acc[c] + ld_stream(V + (long)c * n + e) * fe;
        }
    }
    tree256_chunks<0, MB>(acc, m, sm, [&](int c, double b) { partials[(long)c * kRedBlocks + block] = b; });
}

struct BRow {
    double b[kMaxStages];
};

// k = V lambda + h (F - V phi), column sums in order from zero.  FINAL: the
// last stage, which writes y_{n+1} = y + sum_i b_i k_i instead of k.  Other
// stages i with ynext: also the next stage's input Y_{i+1} = y + sum_{q<=i}
// a_q k_q (a = row i + 1 of alpha; terms with a_q = 0 skipped, k_i from
// registers), in the order the residual forms it from y and the k_q
// (sum in stage order, terms with b_i = 0 skipped).
// Element e from its column sums a = (V lambda)_e and b = (V phi)_e: returns the value of `k`; *next: that of ynext.
template <bool FINAL>
__device__ __forceinline__ double recover_one(double a, double b, double fe, double ye, double h, const double* K, long n, long e, int s,
                                              const BRow& br, bool with_next, int stage, const BRow& ar, double* next) {
    const double ke = a + h * (fe - b);
    if constexpr (FINAL) {
        double acc = ye;
        for (int i = 0; i < s - 1; ++i)
            if (br.b[i] != 0.0) acc = acc + br.b[i] * ld_stream(K + (long)i * n + e);
        if (br.b[s - 1] != 0.0) acc = acc + br.b[s - 1] * ke;
        return acc;
    } else {
        if (with_next) {
            double acc = ye;
            for (int q = 0; q < stage; ++q)
                if (ar.b[q] != 0.0) acc = acc + ar.b[q] * ld_stream(K + (long)q * n + e);
            if (ar.b[stage] != 0.0) acc = acc + ar.b[stage] * ke;
            *next = acc;
        }
        return ke;
    }
}

template <int MB, bool FINAL>
__global__ __launch_bounds__(256) void k_recover(const double* __restrict__ V, const double* __restrict__ F, long n,
                                                const int* ints, const double* lam, const double* phi, double h,
                                                double* __restrict__ k, const double* __restrict__ y,
                                                const double* __restrict__ K, int s, BRow br, const double* sig,
                                                double* __restrict__ ynext, int stage, BRow ar) {
    const int m = ints[0];
    // columns stored unnormalised (v_c = sig_c V_c): the scales go into the coefficients
    auto lamc = [&](int c) { return sig ? lam[c] * sig[c] : lam[c]; };
    auto phic = [&](int c) { return sig ? phi[c] * sig[c] : phi[c]; };
    double lm[MB], ph[MB];
    if (m == MB) {
#pragma unroll
        for (int c = 0; c < MB; ++c) {
            lm[c] = lamc(c);
            ph[c] = phic(c);
        }
    }
    const long stride = (long)gridDim.x * blockDim.x;
    for (long e = (long)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += stride) {
        double a = 0.0, b = 0.0;
        if (m == MB) {
            double vc[MB];
#pragma unroll
            for (int c = 0; c < MB; ++c) vc[c] = ld_stream(V + (long)c * n + e);
#pragma unroll
            for (int c = 0; c < MB; ++c) {
                a = a + vc[c] * lm[c];
                b = b + vc[c] * ph[c];
            }
        } else {
            for (int c = 0; c < m; ++c) {
                double vc = ld_stream(V + (long)c * n + e);
                a = a + vc * lamc(c);
                b = b + vc * phic(c);
            }
        }
        double next = 0.0;
        k[e] = recover_one<FINAL>(a, b, ld_stream(F + e), FINAL || ynext ? ld_stream(y + e) : 0.0, h, K, n, e, s, br,
                                  ynext, stage, ar, &next);
        if (!FINAL && ynext) ynext[e] = next;
    }
}

// k_recover for vectors of many elements per lane: bound by HBM, which loses a fifth of its rate to switching between
// the loads of 19 vectors and two streams of stores.  As in the one-reduce form's update sweep, a block of
// 1024 threads holds its results in LDS and stores kRecHeld of each stream per lane at a
// time: 16 columns of 256^3 2674 us, now 2329, the last stage 2893, now 2338; 20 columns of 2048^2 587, now 560, and 629,
// now 554.
constexpr int kRecThreads = 1024;
constexpr int kRecHeld = 8;

template <int MB, bool FINAL>
__global__ __launch_bounds__(kRecThreads) void k_recover_held(const double* __restrict__ V, const double* __restrict__ F,
                                                             long n, const int* ints, const double* lam, const double* phi,
                                                             double h, double* __restrict__ k,
                                                             const double* __restrict__ y, const double* __restrict__ K,
                                                             int s, BRow br, const double* sig,
                                                             double* __restrict__ ynext, int stage, BRow ar) {
    constexpr int U = FINAL ? 2 * kRecHeld : kRecHeld;
    __shared__ double held[2 * kRecHeld][kRecThreads];
    const int m = ints[0], tid = threadIdx.x;
    double lm[MB], ph[MB];   // uniform: kept in scalar registers
#pragma unroll
    for (int c = 0; c < MB; ++c) {
        lm[c] = lane_value(c < m ? (sig ? lam[c] * sig[c] : lam[c]) : 0.0, 0);
        ph[c] = lane_value(c < m ? (sig ? phi[c] * sig[c] : phi[c]) : 0.0, 0);
    }
    auto one = [&](long e, double* next) {
        double vc[MB];
        const double fe = ld_stream(F + e), ye = FINAL || ynext ? ld_stream(y + e) : 0.0;
#pragma unroll
        for (int c = 0; c < MB; ++c) vc[c] = c < m ? ld_stream(V + (long)c * n + e) : 0.0;
        double a = 0.0, b = 0.0;
#pragma unroll
        for (int c = 0; c < MB; ++c)
            if (c < m) {
                a = a + vc[c] * lm[c];
                b = b + vc[c] * ph[c];
            }
        return recover_one<FINAL>(a, b, fe, ye, h, K, n, e, s, br, ynext, stage, ar, next);
    };
    const long stride = (long)gridDim.x * kRecThreads;
    long e = (long)blockIdx.x * kRecThreads + tid;
    for (; e - tid + kRecThreads + (U - 1) * stride <= n; e += U * stride) {
#pragma unroll 1
        for (int u = 0; u < U; ++u) {
            double next = 0.0;
            held[u][tid] = one(e + u * stride, &next);
            if (!FINAL && ynext) held[U + u][tid] = next;
        }
        __syncthreads();   // the stores of a block's waves together
#pragma unroll
        for (int u = 0; u < U; ++u) __builtin_nontemporal_store(held[u][tid], k + e + u * stride);
        if (!FINAL && ynext) {
#pragma unroll
            for (int u = 0; u < U; ++u) __builtin_nontemporal_store(held[U + u][tid], ynext + e + u * stride);
        }
    }
    for (; e < n; e += stride) {
        double next = 0.0;
        k[e] = one(e, &next);
        if (!FINAL && ynext) ynext[e] = next;
    }
}

// ---------------------------------------------------------------------------
// Workspace: a 256-byte header (status ints, scalars) at offset 0 for every M
// and s, then the small matrices, the reduction partials and the vectors.
// ---------------------------------------------------------------------------

static size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

// Partial columns: the projections (M) and three rotating MGS buffers, or the one-reduce Gram-Schmidt's
// r and s columns (twice the compiled width of its widest column) and its norm column, whichever is more.
static int npart(int M) {
    const int Mm = M > 0 ? M : 1;
    int ls = 0;
    if (lowsync_supported(Mm)) {
        static const int b[] = {1, 2, 4, 8, 12, 16, 20, 24};
        for (int x : b)
            if (Mm <= x) {
                ls = 2 * x + 1;
                break;
            }
    }
    return Mm + 3 > ls ? Mm + 3 : ls;
}

size_t work_small_bytes(int M, int s) {
    int Mm = M > 0 ? M : 1;
    int ss = s > 0 ? s : 1;
    size_t b = 256;
    b += al256(sizeof(double) * (Mm + 1) * Mm);                  // H
    b += al256(sizeof(double) * Mm * Mm);                        // LU
    b += al256(sizeof(double) * ss * Mm);                        // phi
    b += al256(sizeof(double) * ss * Mm);                        // lam
    b += al256(sizeof(int) * Mm);                                // perm
    b += al256(sizeof(double) * Mm * Mm);                        // L
    b += al256(sizeof(double) * (Mm + 1));                       // sig
    b += al256(sizeof(double) * (size_t)npart(M) * kRedBlocks);  // partials
    b += al256(sizeof(double) * (M > 0 ? kExchangeSlots : 0));   // gpart
    b += al256(sizeof(unsigned) * kBarWords);                    // barrier
    return b;
}

size_t work_bytes(long N, int M, int s, bool step) {
    size_t b = work_small_bytes(M, s);
    size_t vec = al256(sizeof(double) * (size_t)N);
    b += vec;                                          // w
    if (step) b += vec * ((size_t)M + 2 * (size_t)s);  // V, F, K
    return b;
}

Work carve(void* base, long N, int M, int s, bool step) {
    int Mm = M > 0 ? M : 1;
    int ss = s > 0 ? s : 1;
    char* p = (char*)base;
    Work W{};
    W.ints = (int*)p;
    W.scal = (double*)(p + 128);
    p += 256;
    W.H = (double*)p;        p += al256(sizeof(double) * (Mm + 1) * Mm);
    W.LU = (double*)p;       p += al256(sizeof(double) * Mm * Mm);
    W.phi = (double*)p;      p += al256(sizeof(double) * ss * Mm);
    W.lam = (double*)p;      p += al256(sizeof(double) * ss * Mm);
    W.perm = (int*)p;        p += al256(sizeof(int) * Mm);
    W.L = (double*)p;        p += al256(sizeof(double) * Mm * Mm);
    W.sig = (double*)p;      p += al256(sizeof(double) * (Mm + 1));
    W.partials = (double*)p; p += al256(sizeof(double) * (size_t)npart(M) * kRedBlocks);
    W.npart = npart(M);
    W.gpart = (double*)p;    p += al256(sizeof(double) * (M > 0 ? kExchangeSlots : 0));
    W.bar = (unsigned*)p;    p += al256(sizeof(unsigned) * kBarWords);
    size_t vec = al256(sizeof(double) * (size_t)N);
    W.w = (double*)p;        p += vec;
    if (step) {
        W.V = (double*)p;    p += vec * (size_t)M;
        W.F = (double*)p;    p += vec * (size_t)s;
        W.K = (double*)p;    p += vec * (size_t)s;
    }
    return W;
}

// Partial buffers: [0, Mm) projection columns, then three rotating MGS buffers.
static double* mgs_part(const Work& W, int k) { return W.partials + (size_t)(W.npart - 3 + (k % 3)) * kRedBlocks; }

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

static inline unsigned grid_for(long n, int threads) {
    long g = (n + threads - 1) / threads;
    if (g > 8192) g = 8192;
    if (g < 1) g = 1;
    return (unsigned)g;
}

// Weighted RMS norm of a step-doubling error estimate: lane sums of q_i^2 in
// the canonical order, q_i = (a_i - b_i) / (c (atol + rtol max(|y_i|, |a_i|))).
// The maximum propagates a NaN of either operand.
__global__ __launch_bounds__(kRedThreads) void k_err_partials(const double* y, const double* a, const double* b,
                                                             long n, double rtol, double atol, double c,
                                                             double* partials) {
    __shared__ double s[kRedThreads];
    double acc = 0.0;
    const long stride = (long)kRedBlocks * kRedThreads;
    for (long e = (long)blockIdx.x * kRedThreads + threadIdx.x; e < n; e += stride) {
        const double ay = fabs(y[e]), aa = fabs(a[e]);
        const double m = (ay != ay || ay > aa) ? ay : aa;
        const double sc = atol + rtol * m;
        const double q = (a[e] - b[e]) / (c * sc);
        acc = acc + q * q;
    }
    double bs = block_sum(acc, s);
    if (threadIdx.x == 0) partials[blockIdx.x] = bs;
}

// *out = sqrt(sum / n) from the partials.
__global__ __launch_bounds__(kRedThreads) void k_err_finish(const double* partials, double n, double* out) {
    __shared__ double s[kRedThreads];
    double tot = final_sum(partials, s);
    if (threadIdx.x == 0) *out = sqrt(tot / n);
}

#define ROK_RED(UPD, SELF, ...) \
    hipLaunchKernelGGL((k_red<UPD, SELF>), dim3(kRedBlocks), dim3(kRedThreads), 0, st, __VA_ARGS__)

hipError_t launch_init(const Work& W, int M, int s, hipStream_t st) {
    int Mm = M > 0 ? M : 1;
    int ss = s > 0 ? s : 1;
    // without a basis nothing is exchanged, and the words' place may hold the slots of a larger layout (rok_jvp's
    // default increment in a workspace that rok_mgs_column uses)
    hipLaunchKernelGGL(k_init, dim3(16), dim3(256), 0, st, W.H, (Mm + 1) * Mm, W.phi, W.lam, ss * Mm, W.scal, W.ints,
                       M, W.bar, M > 0 ? kBarWords : 0, (unsigned long long*)W.gpart, M > 0 ? kExchangeSlots : 0, W.sig,
                       Mm + 1);
    return hipGetLastError();
}

hipError_t launch_norm_eps(const Work& W, const double* y, const double* v, long n, hipStream_t st) {
    ROK_RED(false, true, (double*)v, nullptr, nullptr, nullptr, nullptr, n, nullptr, mgs_part(W, 1));
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(kRedThreads), 0, st, mgs_part(W, 1), (int)FIN_SQRT_TO, W.scal + 3,
                       W.scal, W.ints);
    ROK_RED(false, true, (double*)y, nullptr, nullptr, nullptr, nullptr, n, nullptr, mgs_part(W, 0));
    hipLaunchKernelGGL(k_finish, dim3(1), dim3(kRedThreads), 0, st, mgs_part(W, 0), (int)FIN_EPS, nullptr, W.scal,
                       W.ints);
    return hipGetLastError();
}

hipError_t launch_error_norm(const Work& W, const double* y, const double* a, const double* b, long n, double rtol,
                             double atol, double c, double* out, hipStream_t st) {
    hipLaunchKernelGGL(k_err_partials, dim3(kRedBlocks), dim3(kRedThreads), 0, st, y, a, b, n, rtol, atol, c,
                       mgs_part(W, 0));
    hipLaunchKernelGGL(k_err_finish, dim3(1), dim3(kRedThreads), 0, st, mgs_part(W, 0), (double)n, out);
    return hipGetLastError();
}

// Blocks of a reduction grid that hold elements of an n-vector.
static inline int red_blocks(long n) {
    const long g = (n + kRedThreads - 1) / kRedThreads;
    return (int)(g < 1 ? 1 : (g > kRedBlocks ? kRedBlocks : g));
}

hipError_t launch_start_basis(const Work& W, const double* f, long n, double* v0, hipStream_t st, const double* y) {
    double *pf = mgs_part(W, 0), *py = mgs_part(W, 1);
    const int nb = red_blocks(n);
    hipLaunchKernelGGL(k_norms, dim3((unsigned)nb), dim3(kRedThreads), 0, st, y, f, n, W.ints, pf, py);
    unsigned g = grid_for(n, kRedThreads);
    if (g > 2048) g = 2048;   // every block finishes the sum from 1024 partials
    hipLaunchKernelGGL(k_start, dim3(g), dim3(kRedThreads), 0, st, f, pf, y ? py : nullptr, nb, v0, n, W.ints, W.scal);
    return hipGetLastError();
}

// Orthogonalise w (= J v_j) against V[:, 0..j] by modified Gram-Schmidt;
// writes H[0..j, j] and, if j + 1 < M, H[j+1, j] and v_{j+1}.
hipError_t launch_mgs_column(const Work& W, double* w, const double* V, long n, int M, int j, double* vnext,
                             hipStream_t st) {
    for (int i = 0; i <= j; ++i) {
        const double* vcur = V + (long)i * n;
        if (i == 0) {
            ROK_RED(false, false, w, nullptr, nullptr, nullptr, vcur, n, W.ints, mgs_part(W, 0));
        } else {
            ROK_RED(true, false, w, V + (long)(i - 1) * n, mgs_part(W, i - 1), W.H + (long)(i - 1) * M + j, vcur, n,
                    W.ints, mgs_part(W, i));
        }
    }
    if (j + 1 < M) {
        ROK_RED(true, true, w, V + (long)j * n, mgs_part(W, j), W.H + (long)j * M + j, nullptr, n, W.ints,
                mgs_part(W, j + 1));
        hipLaunchKernelGGL(k_normalize, dim3(grid_for(n, kRedThreads)), dim3(kRedThreads), 0, st, w,
                           mgs_part(W, j + 1), W.H, M, j, vnext, n, W.ints);
    } else {
        hipLaunchKernelGGL(k_finish, dim3(1), dim3(kRedThreads), 0, st, mgs_part(W, j), (int)FIN_STORE,
                           W.H + (long)j * M + j, W.scal, W.ints);
    }
    return hipGetLastError();
}

hipError_t launch_normalize(const Work& W, const double* w, const double* partials, int M, int j, double* v, long n,
                            hipStream_t st) {
    hipLaunchKernelGGL(k_normalize, dim3(grid_for(n, kRedThreads)), dim3(kRedThreads), 0, st, w, partials, W.H, M, j,
                       v, n, W.ints);
    return hipGetLastError();
}

hipError_t launch_norm_scale(const Work& W, const double* partials, int M, int j, hipStream_t st) {
    hipLaunchKernelGGL(k_norm_scale, dim3(1), dim3(kRedThreads), 0, st, partials, W.H, M, j, W.ints, W.sig);
    return hipGetLastError();
}

hipError_t launch_copy_h(const Work& W, int M, double* Hout, int* meff_out, hipStream_t st) {
    hipLaunchKernelGGL(k_copy_h, dim3(grid_for((long)M * M, 256)), dim3(256), 0, st, W.H, M, Hout, W.ints, meff_out);
    return hipGetLastError();
}

// Smallest compiled column count >= M.
static int mbucket(int M) {
    static const int b[] = {1, 2, 4, 8, 12, 16, 20, 24, 32, 48, 64};
    for (int x : b)
        if (M <= x) return x;
    return 64;
}

#define ROK_MB_SWITCH(MBV, CALL)       \
    switch (MBV) {                     \
        case 1: CALL(1); break;        \
        case 2: CALL(2); break;        \
        case 4: CALL(4); break;        \
        case 8: CALL(8); break;        \
        case 12: CALL(12); break;      \
        case 16: CALL(16); break;      \
        case 20: CALL(20); break;      \
        case 24: CALL(24); break;      \
        case 32: CALL(32); break;      \
        case 48: CALL(48); break;      \
        default: CALL(64); break;      \
    }

hipError_t launch_lu(const Work& W, int M, double hg, hipStream_t st) {
#define ROK_LU(MB) hipLaunchKernelGGL((k_lu<MB>), dim3(1), dim3(64), 0, st, W.H, M, hg, W.LU, W.perm, W.ints)
    ROK_MB_SWITCH(mbucket(M), ROK_LU)
#undef ROK_LU
    return hipGetLastError();
}

// The first stage's projection without a pass over the basis: F_1 = f(y_n) =
// beta v_0 (the basis starts from it), so phi_1 = V^T F_1 = beta e_1 in exact
// arithmetic.  Leaves partials that k_lambda finishes to exactly that:
// column 0 holds beta in its first partial, every other partial is zero.
__global__ __launch_bounds__(kRedThreads) void k_project_first(int M, const double* scal, double* partials) {
    const long t = (long)blockIdx.x * kRedThreads + threadIdx.x;
    if (t < (long)M * kRedBlocks) partials[t] = (t == 0) ? scal[2] : 0.0;
}

hipError_t launch_project_first(const Work& W, int M, hipStream_t st) {
    const long n = (long)(M > 0 ? M : 1) * kRedBlocks;
    hipLaunchKernelGGL(k_project_first, dim3((unsigned)((n + kRedThreads - 1) / kRedThreads)), dim3(kRedThreads), 0,
                       st, M, W.scal, W.partials);
    return hipGetLastError();
}

hipError_t launch_project(const Work& W, const double* V, const double* F, long n, int M, hipStream_t st,
                          const double* lu_hg) {
    const LuArgs lu = lu_hg ? LuArgs{W.H, W.LU, W.perm, M, *lu_hg} : LuArgs{};
    const unsigned g = (unsigned)red_blocks(n) + (lu_hg ? 1u : 0u);
#define ROK_PROJ(MB) \
    hipLaunchKernelGGL((k_project<MB>), dim3(g), dim3(kRedThreads), 0, st, V, F, n, W.ints, W.partials, lu)
    ROK_MB_SWITCH(mbucket(M), ROK_PROJ)
#undef ROK_PROJ
    return hipGetLastError();
}

hipError_t launch_lambda(const Work& W, int M, int i, const double* gam_row, double h, long n, hipStream_t st,
                         const double* sig) {
    GamRow gr{};
    for (int j = 0; j < kMaxStages; ++j) gr.g[j] = (j < i) ? gam_row[j] : 0.0;
    hipLaunchKernelGGL(k_lambda, dim3(1), dim3(kSmallThreads), 0, st, W.H, W.LU, W.perm, M, i, gr, h, W.partials,
                       red_blocks(n), W.phi, W.lam, W.ints, sig);
    return hipGetLastError();
}

hipError_t launch_recover(const Work& W, const double* V, const double* F, long n, int M, int i, double h, double* k,
                          const double* y, const double* K, int s, const double* b, hipStream_t st,
                          const double* sig, double* ynext, const double* arow) {
    int Mm = M > 0 ? M : 1;
    BRow br{}, ar{};
    for (int q = 0; q < kMaxStages; ++q) br.b[q] = (b && q < s) ? b[q] : 0.0;
    for (int q = 0; q < kMaxStages; ++q) ar.b[q] = (arow && q <= i) ? arow[q] : 0.0;
    if (ynext && (!y || !K)) return hipErrorInvalidValue;
    const bool fin = y && !ynext;   // the last stage: y_{n+1} into k
    const double* lam = W.lam + (long)i * Mm;
    const double* phi = W.phi + (long)i * Mm;
    const unsigned g = grid_for(n, 256);
    // at 4194304 elements a lane holds 16, two bursts, and most of the basis is in the last-level cache, where the
    // plain form runs at 5.9 TB/s already; the next size of vectors up is out of it.  With a basis of few columns the
    // held form's 16 waves per CU have too few loads in flight: steps at 1300^2 with 0, 1, 2, 4, 8 and 10 columns take
    // 313, 536, 670, 1042, 2058 and 2841 us held, 273, 490, 642, 1016, 2032 and 2945 plain; at 2048^2 the last four 1611,
    // 2546, 4978 and 6875 against 1582, 2537, 5112 and 7215
    const long kHeldFrom = 16L * kRedBlocks * kRedThreads;
#define ROK_REC_ARGS V, F, n, W.ints, lam, phi, h, k, y, K, s, br, sig
#define ROK_REC(MB)                                                                                                  \
    if (MB <= 24 && M > 4 && n > kHeldFrom) {                                                                                 \
        constexpr int B = MB <= 24 ? MB : 24;                                                                        \
        if (fin) hipLaunchKernelGGL((k_recover_held<B, true>), dim3(256), dim3(kRecThreads), 0, st, ROK_REC_ARGS,    \
                                    nullptr, 0, ar);                                                                 \
        else hipLaunchKernelGGL((k_recover_held<B, false>), dim3(256), dim3(kRecThreads), 0, st, ROK_REC_ARGS,       \
                                ynext, i, ar);                                                                       \
    } else if (fin) {                                                                                                \
        hipLaunchKernelGGL((k_recover<MB, true>), dim3(g), dim3(256), 0, st, ROK_REC_ARGS, nullptr, 0, ar);          \
    } else {                                                                                                         \
        hipLaunchKernelGGL((k_recover<MB, false>), dim3(g), dim3(256), 0, st, ROK_REC_ARGS, ynext, i, ar);           \
    }
    ROK_MB_SWITCH(mbucket(M > 0 ? M : 1), ROK_REC)
#undef ROK_REC_ARGS
#undef ROK_REC
    return hipGetLastError();
}

}  // namespace rok
