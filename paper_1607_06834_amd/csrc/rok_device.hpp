// Device-side building blocks shared by the librok kernels: kernel parameter
// blocks, the dual-number type used for exact Jacobian-vector products and
// the periodic index helpers.
//
// Floating-point contract: every file is compiled with -ffp-contract=off and
// evaluates each formula in one fixed, left-to-right operation order, so a
// double-precision result is reproducible bit for bit (FP64 division and
// square root are correctly rounded on gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace rok {

constexpr int kMaxStages = 8;
constexpr int kMaxM = 64;

// Geometry and physics constants of one problem (host-computed, passed by value).
struct Geom {
    int D;          // 2 or 3
    int n[3];       // cells per direction (n[2] = 1 in 2-D)
    int nvar;       // D + 2
    long ncell;     // n0 * n1 * n2
    long N;         // nvar * ncell
    double invdx[3];  // 1 / dx, rounded once
    double hinv[3];   // 0.5 / dx (central differences)
    double g, gm1;    // gamma, gamma - 1
    double gm1_inv;   // 1 / (gamma - 1), 1 / T_ref and 1 / ((gamma - 1) Pr), rounded once (see over)
    double t_ref_inv, kden_inv;
    double mu, c23mu, kappa;  // mu, (2/3) mu, mu gamma / ((gamma-1) Pr)
    int flux;                 // inviscid flux: 0 Rusanov, 1 Roe
    int suth;                 // Sutherland's law (else constant mu)
    double suth_s, suth_one_s, t_ref, kden;   // S / T_ref, 1 + S / T_ref, T_ref, (gamma - 1) Pr
    const double* metric;     // 2-D curvilinear grid: Sx_e, Sy_e, Sx_n, Sy_n, 1/A (ncell each), else null
    int ogrid;                // the curvilinear grid is an O-grid (wall at j = 0, far field past j = n1 - 1):
    double uinf[4];           //   then metric also holds the wall face vectors, and uinf is the free stream
    double t_wall;            //   and (Navier-Stokes) t_wall the isothermal wall's temperature
};

// Residual-kernel inputs: the state y (PLAIN), or y + eps v (FD), or the pair
// (y, v) (TANGENT).
struct ResArgs {
    const double* y;
    const double* v;
    const double* f0;          // FD: f(y)
    const double* eps_dev;     // FD: if non-null, eps is read from here
    double eps;
    void* out;
    // optional: skip the launch unless gate_col + 1 >= *gate (gate: a
    // device-side basis size, e.g. M_eff of the Arnoldi process)
    const int* gate;
    int gate_col;
    // Navier-Stokes kernels: assemble the viscous part of f only
    int viscous_only;
    // optional status word: ROK_FLAG_NONPHYSICAL is or-ed in when a staged
    // cell has rho <= 0 or p <= 0, ROK_FLAG_NONFINITE when an output is NaN or Inf
    int* status;
    // optional: do nothing once *stop is set (a finished Arnoldi process: the
    // basis column this product would read was never written)
    const int* stop;
    // optional (products): the direction is (*vscale) v, for a basis column
    // stored before its normalisation (FD: the increment eps (*vscale) is
    // applied to v; tangent: the tangent is v (*vscale))
    const double* vscale;
};

// ---------------------------------------------------------------------------
// Quotients and roots.  The residual is bound by FP64 issue, and a correctly
// rounded division is about eleven instructions (two of them scalings, one a
// quarter-rate reciprocal).  over(b) takes the reciprocal y of b once, by two Newton
// steps on the hardware's estimate, and a / over(b) is then q = a y corrected by the exact remainder,
// q + (a - b q) y (Markstein 1990), with the hardware's fixup for zeros,
// infinities and NaN: four instructions for every further quotient.
// The same correctly rounded bits as a / b for operands and quotients between
// 2^-900 and 2^900 (FP32: 2^-100 and 2^100): only the scalings for exponents outside are left
// out.  over(b, y): y = RN(1 / b) from the host.
// ---------------------------------------------------------------------------
template <typename S> struct Quot;
template <> struct Quot<double> { double b, y; };
template <> struct Quot<float> { float b, y; };

__device__ __forceinline__ Quot<double> over(double b) {
    double y = __builtin_amdgcn_rcp(b);
    y = __builtin_fma(__builtin_fma(-b, y, 1.0), y, y);
    y = __builtin_fma(__builtin_fma(-b, y, 1.0), y, y);
    return {b, y};
}
__device__ __forceinline__ Quot<double> over(double b, double y) { return {b, y}; }
__device__ __forceinline__ double operator/(double a, Quot<double> r) {
    double q = a * r.y;
    q = __builtin_fma(__builtin_fma(-r.b, q, a), r.y, q);
    return __builtin_amdgcn_div_fixup(q, r.b, a);
}
__device__ __forceinline__ Quot<float> over(float b) {
    float y = __builtin_amdgcn_rcpf(b);
    y = __builtin_fmaf(__builtin_fmaf(-b, y, 1.0f), y, y);
    return {b, y};
}
__device__ __forceinline__ Quot<float> over(float b, double) { return over(b); }
__device__ __forceinline__ float operator/(float a, Quot<float> r) {
    float q = a * r.y;
    q = __builtin_fmaf(__builtin_fmaf(-r.b, q, a), r.y, q);
    return __builtin_amdgcn_div_fixupf(q, r.b, a);
}

// Square root s with h = 1 / (2 s): Goldschmidt's coupled iteration from the hardware's reciprocal root, the last
// two steps correcting by the exact remainder (the correctly rounded root of x above 2^-767: the scaling of smaller
// arguments is left out), then a Newton step of h on s.
__device__ __forceinline__ double root(double x, double& h) {
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y;
    h = 0.5 * y;
    const double r = __builtin_fma(-h, g, 0.5);
    g = __builtin_fma(g, r, g);
    h = __builtin_fma(h, r, h);
    g = __builtin_fma(__builtin_fma(-g, g, x), h, g);
    g = __builtin_fma(__builtin_fma(-g, g, x), h, g);
    h = __builtin_fma(h, __builtin_fma(-(g + g), h, 1.0), h);
    return (x == 0.0 || x == __builtin_inf()) ? x : g;
}
__device__ __forceinline__ float root(float x, float& h) {
    const float y = __builtin_amdgcn_rsqf(x);
    float g = x * y;
    h = 0.5f * y;
    const float r = __builtin_fmaf(-h, g, 0.5f);
    g = __builtin_fmaf(g, r, g);
    h = __builtin_fmaf(h, r, h);
    g = __builtin_fmaf(__builtin_fmaf(-g, g, x), h, g);
    h = __builtin_fmaf(h, __builtin_fmaf(-(g + g), h, 1.0f), h);
    return (x == 0.0f || x == __builtin_inff()) ? x : g;
}

// x y + z with one rounding, y + x / 2 and y - x / 2 (halving is exact, so
// these round once like the separate operations)
__device__ __forceinline__ double mad(double x, double y, double z) { return __builtin_fma(x, y, z); }
__device__ __forceinline__ float mad(float x, float y, float z) { return __builtin_fmaf(x, y, z); }
__device__ __forceinline__ double plus_half(double y, double x) { return __builtin_fma(0.5, x, y); }
__device__ __forceinline__ float plus_half(float y, float x) { return __builtin_fmaf(0.5f, x, y); }
__device__ __forceinline__ double minus_half(double y, double x) { return __builtin_fma(-0.5, x, y); }
__device__ __forceinline__ float minus_half(float y, float x) { return __builtin_fmaf(-0.5f, x, y); }

// ---------------------------------------------------------------------------
// Dual numbers (value, tangent): exact forward-mode derivative of f.  Every
// operation rounds as written, like the plain arithmetic; a quotient's value
// and tangent share the divisor's reciprocal.
// ---------------------------------------------------------------------------
template <typename T>
struct Dual {
    T v, d;
};

template <typename T> __device__ __forceinline__ Dual<T> operator+(Dual<T> a, Dual<T> b) { return {a.v + b.v, a.d + b.d}; }
template <typename T> __device__ __forceinline__ Dual<T> operator-(Dual<T> a, Dual<T> b) { return {a.v - b.v, a.d - b.d}; }
template <typename T> __device__ __forceinline__ Dual<T> operator-(Dual<T> a) { return {-a.v, -a.d}; }
template <typename T> __device__ __forceinline__ Dual<T> operator*(Dual<T> a, Dual<T> b) { return {a.v * b.v, a.d * b.v + a.v * b.d}; }
template <typename T> __device__ __forceinline__ Dual<T> plus_half(Dual<T> y, Dual<T> x) { return {plus_half(y.v, x.v), plus_half(y.d, x.d)}; }
template <typename T> __device__ __forceinline__ Dual<T> minus_half(Dual<T> y, Dual<T> x) { return {minus_half(y.v, x.v), minus_half(y.d, x.d)}; }

// divisor of dual numbers: the value's reciprocal serves value and tangent
template <typename T> struct Quot<Dual<T>> {
    Dual<T> b;
    Quot<T> r;
};
template <typename T> __device__ __forceinline__ Quot<Dual<T>> over(Dual<T> b) { return {b, over(b.v)}; }
template <typename T> __device__ __forceinline__ Dual<T> operator/(Dual<T> a, Quot<Dual<T>> q) {
    const T v = a.v / q.r;
    return {v, (a.d - v * q.b.d) / q.r};
}
template <typename T> __device__ __forceinline__ Dual<T> operator/(Dual<T> a, Dual<T> b) { return a / over(b); }
// a constant divisor (any nesting depth)
template <typename T, typename R, typename = typename std::enable_if<std::is_floating_point<R>::value>::type>
__device__ __forceinline__ Dual<T> operator/(Dual<T> a, Quot<R> r) { return {a.v / r, a.d / r}; }
// products and quotients with a plain floating-point constant (any nesting depth)
template <typename T, typename R, typename = typename std::enable_if<std::is_floating_point<R>::value>::type>
__device__ __forceinline__ Dual<T> operator*(R a, Dual<T> b) { return {a * b.v, a * b.d}; }
template <typename T, typename R, typename = typename std::enable_if<std::is_floating_point<R>::value>::type>
__device__ __forceinline__ Dual<T> operator*(Dual<T> a, R b) { return {a.v * b, a.d * b}; }
template <typename T, typename R, typename = typename std::enable_if<std::is_floating_point<R>::value>::type>
__device__ __forceinline__ Dual<T> operator/(Dual<T> a, R b) { return {a.v / b, a.d / b}; }
template <typename T, typename R, typename = typename std::enable_if<std::is_floating_point<R>::value>::type>
__device__ __forceinline__ Dual<T> operator+(R a, Dual<T> b) { return {a + b.v, b.d}; }
template <typename T, typename R, typename = typename std::enable_if<std::is_floating_point<R>::value>::type>
__device__ __forceinline__ Dual<T> operator+(Dual<T> a, R b) { return {a.v + b, a.d}; }
template <typename T, typename R, typename = typename std::enable_if<std::is_floating_point<R>::value>::type>
__device__ __forceinline__ Dual<T> operator-(Dual<T> a, R b) { return {a.v - b, a.d}; }

// Scalar traits: value part (for branch decisions), construction, sqrt.
template <typename S> struct Sc;
template <> struct Sc<double> {
    using R = double;
    static __device__ __forceinline__ double val(double x) { return x; }
    static __device__ __forceinline__ double make(double x) { return x; }
    static __device__ __forceinline__ double sqrt_(double x, double& h) { return root(x, h); }
    static __device__ __forceinline__ double sqrt_(double x) { double h; return root(x, h); }
};
template <> struct Sc<float> {
    using R = float;
    static __device__ __forceinline__ float val(float x) { return x; }
    static __device__ __forceinline__ float make(double x) { return (float)x; }
    static __device__ __forceinline__ float sqrt_(float x, float& h) { return root(x, h); }
    static __device__ __forceinline__ float sqrt_(float x) { float h; return root(x, h); }
};
template <typename T> struct Sc<Dual<T>> {
    using R = typename Sc<T>::R;
    static __device__ __forceinline__ R val(Dual<T> x) { return Sc<T>::val(x.v); }
    static __device__ __forceinline__ Dual<T> make(double x) { return {Sc<T>::make(x), Sc<T>::make(0.0)}; }
    // sqrt(x) and h = 1 / (2 sqrt(x)), whose tangent is -(s' / s) h
    static __device__ __forceinline__ Dual<T> sqrt_(Dual<T> x, Dual<T>& h) {
        T hv;
        const T s = Sc<T>::sqrt_(x.v, hv);
        const T sd = root_tangent(x.d, s, hv);
        h = {hv, -(sd * hv) * (hv + hv)};
        return {s, sd};
    }
    static __device__ __forceinline__ Dual<T> sqrt_(Dual<T> x) {
        T hv;
        const T s = Sc<T>::sqrt_(x.v, hv);
        return {s, root_tangent(x.d, s, hv)};
    }
    // d / (2 s), h being 1 / (2 s)
    static __device__ __forceinline__ double root_tangent(double d, double s, double h) {
        return d / over(s + s, h);
    }
    static __device__ __forceinline__ float root_tangent(float d, float s, float h) {
        return d / Quot<float>{s + s, h};
    }
    template <typename U> static __device__ __forceinline__ Dual<U> root_tangent(Dual<U> d, Dual<U> s, Dual<U>) { return d / over(s + s); }
};

// 1 / b, correctly rounded (the dual number's tangent by the chain rule)
__device__ __forceinline__ double recip(double b) { return 1.0 / over(b); }
__device__ __forceinline__ Dual<double> recip(Dual<double> b) {
    const double y = 1.0 / over(b.v);
    return {y, -(b.d * y) * y};
}

// The FP64 counterpart of a scalar type (double for float, Dual<double> for
// Dual<float>) and rounding from it.
template <typename S> struct Wide { using type = S; };
template <> struct Wide<float> { using type = double; };
template <typename T> struct Wide<Dual<T>> { using type = Dual<typename Wide<T>::type>; };
template <typename S> __device__ __forceinline__ S narrow(typename Wide<S>::type x) {
    if constexpr (std::is_floating_point<S>::value) return (S)x;
    else return S{narrow<decltype(S{}.v)>(x.v), narrow<decltype(S{}.d)>(x.d)};
}

// Streaming load: for the vector sweeps of the Krylov kernels, which read each
// element of vectors far larger than L2 and the last-level cache once per
// sweep.  The non-temporal hint keeps these lines from displacing reusable
// ones and raises the sweep rate (about 6.3 to 7.1 TB/s for a pure read sweep
// of 17 vectors of 84 M doubles).  Not for stencil staging, whose halos hit in L2.
__device__ __forceinline__ double ld_stream(const double* p) { return __builtin_nontemporal_load(p); }

// The value of v held by lane `lane` (uniform across the wave) of the calling wave.
__device__ __forceinline__ double lane_value(double v, int lane) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffLL), lane);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// Lane i's register moved down by H lanes without going through LDS (a wave
// shuffle by ds_bpermute takes about 60 cycles, these a few): the value of lane
// i + H for the lanes i with i mod 2H < H, which is all a halving tree uses
// (the other lanes get some value of the wave, or zero).  H = 32, 16: swaps of
// wave halves and row pairs; 8 to 1: data-parallel moves within a row of 16.
template <int H>
__device__ __forceinline__ int lane_down_word(int x) {
    static_assert(H == 32 || H == 16 || H == 8 || H == 4 || H == 2 || H == 1, "a power of two below 64");
    if constexpr (H == 32) return (int)__builtin_amdgcn_permlane32_swap(x, x, false, false)[1];
    else if constexpr (H == 16) return (int)__builtin_amdgcn_permlane16_swap(x, x, false, false)[1];
    else return __builtin_amdgcn_update_dpp(0, x, 0x100 + H, 0xf, 0xf, true);   // row_shl:H
}

template <int H>
__device__ __forceinline__ double lane_down(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = lane_down_word<H>((int)(b & 0xffffffffLL)), hi = lane_down_word<H>((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// The value of the lane before, within rows of 16 lanes (the first lane of a row gets zero).
__device__ __forceinline__ double lane_up1(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffLL), 0x111, 0xf, 0xf, true);   // row_shr:1
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x111, 0xf, 0xf, true);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// One level of two halving trees at once: a_i + a_{i+H} in the lanes i with
// i mod 2H < H, b_{i-H} + b_i in the others.
template <int H>
__device__ __forceinline__ double swap_add(double a, double b) {
    const long long x = __double_as_longlong(a), y = __double_as_longlong(b);
    const int xl = (int)(x & 0xffffffffLL), xh = (int)(x >> 32), yl = (int)(y & 0xffffffffLL), yh = (int)(y >> 32);
    int pl, ph, ql, qh;
    if constexpr (H == 32 || H == 16) {
        // the upper part of the first register changes places with the lower part of the second
        const auto l = (H == 32) ? __builtin_amdgcn_permlane32_swap(xl, yl, false, false)
                                 : __builtin_amdgcn_permlane16_swap(xl, yl, false, false);
        const auto h = (H == 32) ? __builtin_amdgcn_permlane32_swap(xh, yh, false, false)
                                 : __builtin_amdgcn_permlane16_swap(xh, yh, false, false);
        pl = (int)l[0]; ql = (int)l[1];
        ph = (int)h[0]; qh = (int)h[1];
    } else {
        static_assert(H == 8 || H == 16 || H == 32, "the levels that rotate by half a row or more");
        const bool up = (threadIdx.x & 8) != 0;
        pl = up ? yl : xl;
        ph = up ? yh : xh;
        // row_ror:8: the lane 8 away in the row of 16
        ql = __builtin_amdgcn_update_dpp(0, up ? xl : yl, 0x128, 0xf, 0xf, true);
        qh = __builtin_amdgcn_update_dpp(0, up ? xh : yh, 0x128, 0xf, 0xf, true);
    }
    return __longlong_as_double(((long long)ph << 32) | (long long)(unsigned)pl) +
           __longlong_as_double(((long long)qh << 32) | (long long)(unsigned)ql);
}

// The in-wave levels h = 32 .. 1 of a halving tree; the sum is in lane 0.
__device__ __forceinline__ double wave_sum(double v) {
    v = v + lane_down<32>(v);
    v = v + lane_down<16>(v);
    v = v + lane_down<8>(v);
    v = v + lane_down<4>(v);
    v = v + lane_down<2>(v);
    return v + lane_down<1>(v);
}

// Final stage of the canonical sum by one wave: the blocks' partials p[0 .. nb)
// (of 1024; those past nb are zero and not read).  Final lane t of 256 adds
// partials t, t + 256, t + 512, t + 768 in order; lane l holds t = l + 64 m, so the
// tree's first two levels are additions within the lane and the rest wave_sum.
// Every lane gets the sum.
__device__ __forceinline__ double wave_final(const double* p, int nb) {
    const int l = threadIdx.x & 63;
    double v[4][4], a[4];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int r = 0; r < 4; ++r) v[m][r] = (l + 64 * m + 256 * r < nb) ? p[l + 64 * m + 256 * r] : 0.0;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        a[m] = 0.0;
#pragma unroll
        for (int r = 0; r < 4; ++r) a[m] = a[m] + v[m][r];
    }
    return lane_value(wave_sum((a[0] + a[2]) + (a[1] + a[3])), 0);
}

// Pairwise halving tree over groups of 256 consecutive threads of a block:
// with x_i the value of lane i of a group, computes s_i <- s_i + s_{i+h} for
// h = 128, 64, ..., 1 (i < h) and returns s_0 in lane 0 of each group (other
// lanes return partial values).  The two cross-wave levels go through LDS
// (`s`, one double per thread), the six in-wave levels through lane
// shuffles; the additions and their order are those of the LDS tree.
__device__ __forceinline__ double tree256(double v, double* s) {
    const int tid = threadIdx.x;
    const int lane = tid & 255;
    s[tid] = v;
    __syncthreads();
    if (lane < 128) {
        v = v + s[tid + 128];
        s[tid] = v;
    }
    __syncthreads();
    if (lane < 64) {
        v = wave_sum(v + s[tid + 64]);
    }
    return v;
}

// tree256 for many values of every thread of a 256-thread block at once:
// values v[C0 .. C0 + 16) (those below nact) go through the tree of tree256
// together, the two LDS levels shared by all of them (three block barriers
// per 16 values, the last before `s` is reused), with the same additions in
// the same order for each; thread 0 passes each sum to store(index, sum).
// `s` holds 16 x 256 doubles of LDS.  nact must be the same in every thread.
template <int C0, int N, typename F>
__device__ __forceinline__ void tree256_chunks(const double (&v)[N], int nact, double (*s)[256], F store) {
    if constexpr (C0 < N) {
        if (C0 >= nact) return;
        const int tid = threadIdx.x;
        constexpr int K = (N - C0) < 16 ? (N - C0) : 16;
        double x[K];
#pragma unroll
        for (int c = 0; c < K; ++c) s[c][tid] = v[C0 + c];
        __syncthreads();
        if (tid < 128) {
#pragma unroll
            for (int c = 0; c < K; ++c) {
                x[c] = v[C0 + c] + s[c][tid + 128];
                s[c][tid] = x[c];
            }
        }
        __syncthreads();
        if (tid < 64) {
#pragma unroll
            for (int c = 0; c < K; ++c) {
                x[c] = wave_sum(x[c] + s[c][tid + 64]);
            }
        }
        if (tid == 0) {
#pragma unroll
            for (int c = 0; c < K; ++c)
                if (C0 + c < nact) store(C0 + c, x[c]);
        }
        __syncthreads();
        tree256_chunks<C0 + 16, N>(v, nact, s, store);
    }
}

// Periodic wrap of an index that may lie anywhere in [-n, 2n) (fast path) or
// beyond (small grids).
__device__ __forceinline__ int wrap(int i, int n) {
    if (i >= 0 && i < n) return i;
    int r = i % n;
    return r < 0 ? r + n : r;
}

// XCD-aware block order: workgroups are dispatched round-robin over the 8
// XCDs; give each XCD a contiguous range of tiles so halos hit in its L2.
__device__ __forceinline__ int xcd_remap(int b, int nb) {
    int q = nb >> 3, r = nb & 7, x = b & 7, i = b >> 3;
    return x < r ? x * (q + 1) + i : r * (q + 1) + (x - r) * q + i;
}

}  // namespace rok
