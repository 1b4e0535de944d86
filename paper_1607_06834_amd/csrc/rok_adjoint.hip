// Adjoint (transposed) Jacobian products of the finite-volume residual:
//   ybar (+)= J(y)^T wbar                          (first-order adjoint)
//   ybar2 (+)= d/dt [J(y + t v)^T wbar] at t = 0   (second-order adjoint)
// for the right-hand side f of Sec. 3.2, eq. (11) (Euler or Navier-Stokes
// physics, first-order or MUSCL-minmod reconstruction, Rusanov or Roe flux,
// periodic Cartesian or 2-D curvilinear grid; on the latter f_c divides by
// the cell area, each inviscid face flux is the rotated one and the viscous
// one follows the chain rule through the face vector).
//
// f_c = sum_d (Fhat_{c-1/2} - Fhat_{c+1/2}) / dx_d, so the adjoint of the face
// a+1/2 (between cells a and a+1) is Fbar = (wbar_{a+1} - wbar_a) / dx_d, and
// cell c collects Fbar^T dFhat/dU_c from every face whose stencil contains c
// (first order: faces c-1/2, c+1/2; MUSCL: the four faces c-3/2 .. c+3/2).
// Each thread owns one cell and gathers its own contributions, so the result
// is deterministic without atomics.
//   most 2-D Cartesian grids (k_vjp_tile): a tile's face fluxes are reversed once
//   each, down to the adjoints of the two reconstructed states, and its cells
//   gather those from LDS;
//   3-D and curvilinear grids, and 2-D ones where that is the faster (k_vjp):
//   each cell reverses the faces whose stencil holds it.
// A face's reverse is one sweep back through Rusanov's flux (the transpose of the tangent of the
// residual's flux code); Roe's takes forward-mode evaluations.
// With a dual scalar (y + t v) the same kernels return
// the second-order adjoint in the tangent part.
#include "rok.h"
#include "rok_device.hpp"
#include "rok_flux.hpp"
#include "rok_kernels.hpp"

namespace rok {

// Transpose of the viscous fluxes of a Cartesian grid (Sec. 3.2: stress row and
// energy term of the face a | b = a + e_d) at one cell c: adds to vb and Tb the adjoints of c's
// velocity and temperature, sum over the faces whose stencil holds c of
// Fbar^T dFv/d(vel_c, T_c).  With Gr[e][t] the face gradient of velocity e along t
// (across the face the difference; along it the mean of a's and b's central
// differences), tau_e = mu (Gr[e][d] + Gr[d][e]) - [e = d] (2/3) mu div and
// tb_e = Fbar_e + uf_e Fbar_E the adjoint of tau_e:
//   Gr[e][d] gets mu tb_e, Gr[d][e] the same, Gr[e][e] gets -(2/3) mu tb_d, uf_e gets Fbar_E tau_e,
//   (T_b - T_a) / dx gets kappa Fbar_E, and the viscosity (Sutherland's law) its own.
// The faces on either side of c along d take the whole stencil; where c is only
// a tangential neighbour of a face, its derivative needs that face's two velocities alone.
//   q(o, r, vel, p): primitives of the cell at offset o from c;  w(o, m): wbar there.
template <int D, typename T, typename Q, typename WB>
__device__ __forceinline__ void visc_vjp_cell(const Geom& G, Q q, WB w, T* vb, T& Tb) {
    const double half = 0.5;
    auto viscosity = [&](T Tf, T& mu, T& c23mu, T& kappa) {
        if (G.suth) {
            const T th = Tf / G.t_ref;
            mu = G.mu * th * Sc<T>::sqrt_(th) * G.suth_one_s / (th + G.suth_s);
            c23mu = (2.0 / 3.0) * mu;
            kappa = mu * G.g / G.kden;
        } else {
            mu = Sc<T>::make(G.mu);
            c23mu = Sc<T>::make(G.c23mu);
            kappa = Sc<T>::make(G.kappa);
        }
    };
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const double inv = G.invdx[d];
        // c = a (side 0) and c = b (side 1)
#pragma nounroll
        for (int side = 0; side < 2; ++side) {
            int oa[3] = {0, 0, 0}, ob[3] = {0, 0, 0};
            oa[d] = -side;
            ob[d] = 1 - side;
            T ra, pa, va[D], rb, pb, vc[D];
            q(oa, ra, va, pa);
            q(ob, rb, vc, pb);
            const T Ta = pa / ra, Tc = pb / rb;
            T Gr[D][D];   // the entries tau and div read: Gr[e][d], Gr[d][t], Gr[t][t]
#pragma unroll
            for (int e = 0; e < D; ++e) Gr[e][d] = (vc[e] - va[e]) * inv;
#pragma unroll
            for (int t = 0; t < D; ++t) {
                if (t == d) continue;
                T rr, pp, vv[4][D];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    int o[3] = {0, 0, 0};
                    o[d] = (k < 2 ? 0 : 1) - side;
                    o[t] = (k & 1) ? 1 : -1;
                    q(o, rr, vv[k], pp);
                }
                const double h = G.hinv[t];
                Gr[d][t] = half * ((vv[1][d] - vv[0][d]) * h + (vv[3][d] - vv[2][d]) * h);
                Gr[t][t] = half * ((vv[1][t] - vv[0][t]) * h + (vv[3][t] - vv[2][t]) * h);
            }
            T div = Gr[0][0];
#pragma unroll
            for (int e = 1; e < D; ++e) div = div + Gr[e][e];
            T mu, c23mu, kappa;
            const T Tf = half * (Ta + Tc);
            viscosity(Tf, mu, c23mu, kappa);
            const double Fe = (w(ob, D + 1) - w(oa, D + 1)) * inv;
            const double sgn = side ? 1.0 : -1.0;
            T mub = Sc<T>::make(0.0);
#pragma unroll
            for (int e = 0; e < D; ++e) {
                const T tb = (w(ob, 1 + e) - w(oa, 1 + e)) * inv + (half * (va[e] + vc[e])) * Fe;
                const T S = Gr[e][d] + Gr[d][e];
                const T tau = (e == d) ? mu * S - c23mu * div : mu * S;
                const T gd = (e == d) ? mu * (tb + tb) - c23mu * tb : mu * tb;   // adjoint of Gr[e][d]
                vb[e] = vb[e] + gd * (sgn * inv) + tau * (half * Fe);
                mub = mub + ((e == d) ? tb * (S - (2.0 / 3.0) * div) : tb * S);
            }
            Tb = Tb + kappa * (sgn * inv * Fe);
            if (G.suth) {
                mub = mub + ((Tc - Ta) * inv) * (Fe * G.g / G.kden);
                const T th = Tf / G.t_ref;
                // d mu / d T_f = mu (3 / (2 theta) - 1 / (theta + s)) / t_ref, and T_f = (T_a + T_b) / 2
                const T ths = th + G.suth_s;
                Tb = Tb + (half / G.t_ref) * (mub * mu * ((1.5 * ths - th) / (th * ths)));
            }
        }
        // c = a -+ e_t or b -+ e_t of a face along d
#pragma unroll
        for (int t = 0; t < D; ++t) {
            if (t == d) continue;
#pragma nounroll
            for (int k = 0; k < 4; ++k) {
                int oa[3] = {0, 0, 0}, ob[3] = {0, 0, 0};
                const int at = (k & 1) ? -1 : 1;
                oa[t] = ob[t] = at;
                oa[d] = k < 2 ? 0 : -1;
                ob[d] = oa[d] + 1;
                T ra, pa, va[D], rb, pb, vc[D];
                q(oa, ra, va, pa);
                q(ob, rb, vc, pb);
                T mu, c23mu, kappa;
                if (G.suth) viscosity(half * (pa / ra + pb / rb), mu, c23mu, kappa);
                else viscosity(Sc<T>::make(0.0), mu, c23mu, kappa);
                const double Fe = (w(ob, D + 1) - w(oa, D + 1)) * inv;
                const T tbt = (w(ob, 1 + t) - w(oa, 1 + t)) * inv + (half * (va[t] + vc[t])) * Fe;
                const T tbd = (w(ob, 1 + d) - w(oa, 1 + d)) * inv + (half * (va[d] + vc[d])) * Fe;
                const double h = (at > 0 ? -half : half) * G.hinv[t];   // c is the lower neighbour where at = 1
                vb[d] = vb[d] + (mu * tbt) * h;
                vb[t] = vb[t] - (c23mu * tbd) * h;
            }
        }
    }
}

// The conserved adjoint of a cell from the adjoints (rb, vb, pb) of its
// primitives (r, vel, p): vel = m / r, p = (gamma - 1)(E - r |vel|^2 / 2).
template <int D, typename T>
__device__ __forceinline__ void prim_adjoint(const Geom& G, T r, const T* vel, T rb, const T* vb, T pb, T* Ub) {
    const double half = 0.5;
    T ke = vel[0] * vel[0];
#pragma unroll
    for (int e = 1; e < D; ++e) ke = ke + vel[e] * vel[e];
    const T tb = -(G.gm1 * pb);
    const T keb = half * r * tb;
    const auto qr = over(r);
    rb = rb + half * ke * tb;
#pragma unroll
    for (int e = 0; e < D; ++e) {
        const T m = (vb[e] + (vel[e] + vel[e]) * keb) / qr;
        Ub[1 + e] = m;
        rb = rb - m * vel[e];
    }
    Ub[0] = rb;
    Ub[D + 1] = G.gm1 * pb;
}

// Viscous flux through a face of a 2-D curvilinear grid (Sec. 3.2) from
// index-space derivatives across the face (nu, nv, nT) and along it (tu, tv,
// tT), turned into Cartesian gradients by the chain rule through the face
// vector S = (sx, sy) and the centroid difference (dcx, dcy) across the face
// (d: 0 across i, 1 across j); the stress, work and conduction terms dotted
// with S.  uf: face velocity; Tf: face temperature (Sutherland's law).
template <typename S>
__device__ __forceinline__ void curv_visc_core(const Geom& G, int d, double sx, double sy, double dcx, double dcy,
                                               S nu, S nv, S nT, S tu, S tv, S tT, S ufx, S ufy, S Tf, S* Fv) {
    const double J = dcx * sx + dcy * sy;
    S ux, uy, vx, vy, Tx, Ty;
    if (d == 0) {
        ux = (nu * sx - tu * dcy) / J;
        uy = (nu * sy + tu * dcx) / J;
        vx = (nv * sx - tv * dcy) / J;
        vy = (nv * sy + tv * dcx) / J;
        Tx = (nT * sx - tT * dcy) / J;
        Ty = (nT * sy + tT * dcx) / J;
    } else {
        ux = (nu * sx + tu * dcy) / J;
        uy = (nu * sy - tu * dcx) / J;
        vx = (nv * sx + tv * dcy) / J;
        vy = (nv * sy - tv * dcx) / J;
        Tx = (nT * sx + tT * dcy) / J;
        Ty = (nT * sy - tT * dcx) / J;
    }
    S mu, c23, kap;
    if (G.suth) {
        const S th = Tf / G.t_ref;
        mu = G.mu * th * Sc<S>::sqrt_(th) * G.suth_one_s / (th + G.suth_s);
        c23 = (2.0 / 3.0) * mu;
        kap = mu * G.g / G.kden;
    } else {
        mu = Sc<S>::make(G.mu);
        c23 = Sc<S>::make(G.c23mu);
        kap = Sc<S>::make(G.kappa);
    }
    const S div = ux + vy;
    const S txx = mu * (ux + ux) - c23 * div;
    const S tyy = mu * (vy + vy) - c23 * div;
    const S txy = mu * (uy + vx);
    Fv[0] = Sc<S>::make(0.0);
    Fv[1] = txx * sx + txy * sy;
    Fv[2] = txy * sx + tyy * sy;
    Fv[3] = (ufx * txx + ufy * txy + kap * Tx) * sx + (ufx * txy + ufy * tyy + kap * Ty) * sy;
}

// The same from the stencil of a periodic curvilinear face (U[0] = a, U[1] = b, U[2..5] = a - e_t, a + e_t, b - e_t, b + e_t with t
// the grid direction along the face): differences across the face and means
// of the two cells' central differences along it.
template <typename S>
__device__ __forceinline__ void curv_visc_face(const Geom& G, const S (*U)[4], int d, double sx, double sy,
                                               double dcx, double dcy, S* Fv) {
    const double half = 0.5;
    S u[6], v[6], Tq[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        S r, vel[2], p;
        primitives<2>(G, U[q], r, vel, p);
        u[q] = vel[0];
        v[q] = vel[1];
        Tq[q] = p / r;
    }
    auto along = [&](const S* f) { return half * ((f[3] - f[2]) * half + (f[5] - f[4]) * half); };
    curv_visc_core<S>(G, d, sx, sy, dcx, dcy, u[1] - u[0], v[1] - v[0], Tq[1] - Tq[0], along(u), along(v),
                      along(Tq), half * (u[0] + u[1]), half * (v[0] + v[1]), half * (Tq[0] + Tq[1]), Fv);
}

template <int FLUX, typename S>
__device__ __forceinline__ void rotated_flux(const Geom& G, const S* UL, S rL, const S* vL, S pL, const S* UR, S rR,
                                             const S* vR, S pR, double sx, double sy, S* Fh);

// Inviscid flux through a face of a 2-D curvilinear grid with face vector
// (sx, sy): the stencil's states reconstructed in index space (first order
// U[0] = a, U[1] = b; MUSCL U[0..3] = a-1, a, b, b+1), rotated into the face
// frame n = S / |S|, the one-dimensional numerical flux there, rotated back
// and scaled by |S|.
template <int RECON, int FLUX, typename S>
__device__ __forceinline__ void curv_face_flux(const Geom& G, const S (*U)[4], double sx, double sy, S* Fh) {
    S UL[4], UR[4], vL[2], vR[2], rL, rR, pL, pR;
    if constexpr (RECON == 0) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            UL[m] = U[0][m];
            UR[m] = U[1][m];
        }
        primitives<2>(G, UL, rL, vL, pL);
        primitives<2>(G, UR, rR, vR, pR);
    } else {
        S q[4][4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            S rr, vv[2], pp;
            primitives<2>(G, U[k], rr, vv, pp);
            q[k][0] = rr;
            q[k][1] = vv[0];
            q[k][2] = vv[1];
            q[k][3] = pp;
        }
        S qL[4], qR[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            qL[m] = q[1][m] + 0.5 * minmod(q[1][m] - q[0][m], q[2][m] - q[1][m]);
            qR[m] = q[2][m] - 0.5 * minmod(q[2][m] - q[1][m], q[3][m] - q[2][m]);
        }
        rL = qL[0];
        rR = qR[0];
        vL[0] = qL[1];
        vL[1] = qL[2];
        vR[0] = qR[1];
        vR[1] = qR[2];
        pL = qL[3];
        pR = qR[3];
        to_conserved<2>(G, rL, vL, pL, UL);
        to_conserved<2>(G, rR, vR, pR, UR);
    }
    rotated_flux<FLUX, S>(G, UL, rL, vL, pL, UR, rR, vR, pR, sx, sy, Fh);
}

// Numerical flux through a face with vector (sx, sy) between reconstructed
// states: rotated into the face frame n = S / |S|, the one-dimensional flux,
// rotated back and scaled by |S|.
template <int FLUX, typename S>
__device__ __forceinline__ void rotated_flux(const Geom& G, const S* UL, S rL, const S* vL, S pL, const S* UR, S rR,
                                             const S* vR, S pR, double sx, double sy, S* Fh) {
    const double ln = sqrt(sx * sx + sy * sy);
    const double nx = sx / ln, ny = sy / ln;
    S vLr[2], vRr[2], ULr[4], URr[4], Fr[4];
    vLr[0] = vL[0] * nx + vL[1] * ny;
    vLr[1] = vL[1] * nx - vL[0] * ny;
    vRr[0] = vR[0] * nx + vR[1] * ny;
    vRr[1] = vR[1] * nx - vR[0] * ny;
    ULr[0] = UL[0];
    ULr[1] = UL[1] * nx + UL[2] * ny;
    ULr[2] = UL[2] * nx - UL[1] * ny;
    ULr[3] = UL[3];
    URr[0] = UR[0];
    URr[1] = UR[1] * nx + UR[2] * ny;
    URr[2] = UR[2] * nx - UR[1] * ny;
    URr[3] = UR[3];
    num_flux<2, FLUX>(G, 0, ULr, rL, vLr, pL, URr, rR, vRr, pR, Fr);
    Fh[0] = Fr[0] * ln;
    Fh[1] = (Fr[1] * nx - Fr[2] * ny) * ln;
    Fh[2] = (Fr[1] * ny + Fr[2] * nx) * ln;
    Fh[3] = Fr[3] * ln;
}

template <int D, int RECON, bool SECOND, int FLUX, bool NSV, int GEO>
__global__ __launch_bounds__(256) void k_vjp(Geom G, const double* y, const double* v, const double* wbar,
                                            double* ybar, double* ybar2, int accumulate, const int* gate, int col) {
    if (gate && col >= gate[0]) return;   // Krylov column beyond M_eff: nothing to add
    constexpr int NV = D + 2;
    constexpr int NS = (RECON == 0) ? 2 : 4;   // stencil cells of a face
    constexpr int NF = (RECON == 0) ? 2 : 4;   // faces per direction whose stencil contains a cell
    using T = typename std::conditional<SECOND, Dual<double>, double>::type;   // value (+ t-derivative)
    const int n0 = G.n[0], n1 = G.n[1], n2 = G.n[2];
    const long ncell = G.ncell;
    const long stride = (long)gridDim.x * blockDim.x;
    for (long c = (long)blockIdx.x * blockDim.x + threadIdx.x; c < ncell; c += stride) {
        const int cx = (int)(c % n0);
        const int cy = (int)((c / n0) % n1);
        const int cz = (int)(c / ((long)n0 * n1));
        T acc[NV];
#pragma unroll
        for (int k = 0; k < NV; ++k) acc[k] = Sc<T>::make(0.0);
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const double inv = G.invdx[d];
#pragma nounroll
            for (int f = 0; f < NF; ++f) {
                // face between cells a and a+1 along d; stencil starts at s0
                const int off_a = (RECON == 0) ? f - 1 : f - 2;      // a - c
                const int off_s0 = (RECON == 0) ? off_a : off_a - 1;  // first stencil cell - c
                const int kc = -off_s0;                               // position of c in the stencil
                long cell[NS];
#pragma unroll
                for (int q = 0; q < NS; ++q) {
                    int o = off_s0 + q;
                    int x = cx, yy = cy, z = cz;
                    if (d == 0) x = wrap(cx + o, n0);
                    else if (d == 1) yy = wrap(cy + o, n1);
                    else z = wrap(cz + o, n2);
                    cell[q] = ((long)z * n1 + yy) * n0 + x;
                }
                const long ca = cell[(RECON == 0) ? 0 : 1];
                const long cb = cell[(RECON == 0) ? 1 : 2];
                T fbar[NV];
                if constexpr (GEO == 0) {
#pragma unroll
                    for (int m = 0; m < NV; ++m)
                        fbar[m] = Sc<T>::make((wbar[m * ncell + cb] - wbar[m * ncell + ca]) * inv);
                } else {
                    // f_c = sum_d (Fhat_{c-1/2} - Fhat_{c+1/2}) / A_c
                    const double ia = G.metric[4 * ncell + ca], ib = G.metric[4 * ncell + cb];
#pragma unroll
                    for (int m = 0; m < NV; ++m)
                        fbar[m] = Sc<T>::make(wbar[m * ncell + cb] * ib - wbar[m * ncell + ca] * ia);
                }
                T base[NS][NV], ub[NS][NV];
#pragma unroll
                for (int q = 0; q < NS; ++q)
#pragma unroll
                    for (int m = 0; m < NV; ++m) {
                        const long i = m * ncell + cell[q];
                        if constexpr (SECOND) base[q][m] = T{y[i], v[i]};
                        else base[q][m] = y[i];
                        ub[q][m] = Sc<T>::make(0.0);
                    }
                if constexpr (GEO == 1) {
                    // rotated face flux: Fbar^T dFhat/dU_c by forward mode, one dual direction per variable of c
                    const double sx = G.metric[(long)(2 * d) * ncell + ca];
                    const double sy = G.metric[(long)(2 * d + 1) * ncell + ca];
                    using TT = Dual<T>;
#pragma unroll 1
                    for (int m = 0; m < NV; ++m) {
                        TT Ud[NS][4], Fd[4];
#pragma unroll
                        for (int q = 0; q < NS; ++q)
#pragma unroll
                            for (int k = 0; k < 4; ++k)
                                Ud[q][k] = TT{base[q][k], Sc<T>::make((q == kc && k == m) ? 1.0 : 0.0)};
                        curv_face_flux<RECON, FLUX, TT>(G, Ud, sx, sy, Fd);
                        T sum = Sc<T>::make(0.0);
#pragma unroll
                        for (int k = 0; k < 4; ++k) sum = sum + fbar[k] * Fd[k].d;
                        ub[kc][m] = sum;
                    }
                } else if constexpr (FLUX == 0) {
                    face_flux_vjp<D, RECON, T>(G, base, d, fbar, ub);
                } else {
                    // Roe: Fbar^T dFhat/dU_c by forward mode, one dual direction per variable of c
                    using TT = Dual<T>;
#pragma unroll 1
                    for (int m = 0; m < NV; ++m) {
                        TT Ud[NS][NV], Fd[NV];
#pragma unroll
                        for (int q = 0; q < NS; ++q)
#pragma unroll
                            for (int k = 0; k < NV; ++k)
                                Ud[q][k] = TT{base[q][k], Sc<T>::make((q == kc && k == m) ? 1.0 : 0.0)};
                        face_flux_cells<D, RECON, TT, 1>(G, Ud, d, Fd);
                        T sum = Sc<T>::make(0.0);
#pragma unroll
                        for (int k = 0; k < NV; ++k) sum = sum + fbar[k] * Fd[k].d;
                        ub[kc][m] = sum;
                    }
                }
#pragma unroll
                for (int q = 0; q < NS; ++q)
                    if (q == kc)
#pragma unroll
                        for (int k = 0; k < NV; ++k) acc[k] = acc[k] + ub[q][k];
            }
            if constexpr (NSV && GEO == 1) {
                // The face flux is Fhat - Fv: cell c collects -Fbar^T dFv/dU_c
                // from every face whose viscous stencil holds it, one face per
                // stencil position (position kv of c), each by forward mode.
                constexpr int NQ = 2 + 4 * (D - 1);
                auto cell_at = [&](int od, int ot, int t) -> long {
                    int o[3] = {0, 0, 0};
                    o[d] += od;
                    if (ot) o[t] += ot;
                    const int x = wrap(cx + o[0], n0), yy = wrap(cy + o[1], n1);
                    const int z = (D == 3) ? wrap(cz + o[2], n2) : 0;
                    return ((long)z * n1 + yy) * n0 + x;
                };
#pragma nounroll
                for (int kv = 0; kv < NQ; ++kv) {
                    // offset of face cell a from c, and of each stencil cell from a
                    int ad = 0, at = 0, tdir = 0;
                    if (kv == 0) ad = 0;
                    else if (kv == 1) ad = -1;
                    else {
                        const int k = (kv - 2) / 4, r = (kv - 2) % 4;
                        tdir = (k < d) ? k : k + 1;
                        ad = (r >= 2) ? -1 : 0;          // c on the b side
                        at = (r % 2 == 0) ? 1 : -1;      // c = a - e_t (r even) or a + e_t
                    }
                    long cell[NQ];
                    cell[0] = cell_at(ad, at, tdir);
                    cell[1] = cell_at(ad + 1, at, tdir);
#pragma unroll
                    for (int k = 0; k < D - 1; ++k) {
                        const int t = (k < d) ? k : k + 1;
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const int od = ad + (r >= 2 ? 1 : 0);
                            int ot = (r % 2 == 0) ? -1 : 1;
                            // offsets along t add up: (a's offset from c) + (stencil cell's from a)
                            if (t == tdir) cell[2 + 4 * k + r] = cell_at(od, at + ot, t);
                            else {
                                int o3[3] = {0, 0, 0};
                                o3[d] += od;
                                o3[tdir] += at;
                                o3[t] += ot;
                                const int x = wrap(cx + o3[0], n0), yy = wrap(cy + o3[1], n1);
                                const int z = (D == 3) ? wrap(cz + o3[2], n2) : 0;
                                cell[2 + 4 * k + r] = ((long)z * n1 + yy) * n0 + x;
                            }
                        }
                    }
                    T fbar[NV];
                    const double ia = G.metric[4 * ncell + cell[0]], ib = G.metric[4 * ncell + cell[1]];
#pragma unroll
                    for (int m = 0; m < NV; ++m)
                        fbar[m] = Sc<T>::make(wbar[m * ncell + cell[1]] * ib - wbar[m * ncell + cell[0]] * ia);
                    T base[NQ][NV];
#pragma unroll
                    for (int q = 0; q < NQ; ++q)
#pragma unroll
                        for (int m = 0; m < NV; ++m) {
                            const long i = m * ncell + cell[q];
                            if constexpr (SECOND) base[q][m] = T{y[i], v[i]};
                            else base[q][m] = y[i];
                        }
                    using TT = Dual<T>;
#pragma unroll 1
                    for (int m = 0; m < NV; ++m) {
                        TT Ud[NQ][NV], Fd[NV];
#pragma unroll
                        for (int q = 0; q < NQ; ++q)
#pragma unroll
                            for (int k = 0; k < NV; ++k)
                                Ud[q][k] = TT{base[q][k], Sc<T>::make((q == kv && k == m) ? 1.0 : 0.0)};
                        const long a0 = cell[0];
                        curv_visc_face<TT>(G, Ud, d, G.metric[(long)(2 * d) * ncell + a0],
                                           G.metric[(long)(2 * d + 1) * ncell + a0],
                                           G.metric[(long)(5 + 2 * d) * ncell + a0],
                                           G.metric[(long)(6 + 2 * d) * ncell + a0], Fd);
                        T sum = Sc<T>::make(0.0);
#pragma unroll
                        for (int k = 1; k < NV; ++k) sum = sum + fbar[k] * Fd[k].d;
                        acc[m] = acc[m] - sum;
                    }
                }
            }
        }
        if constexpr (NSV && GEO == 0) {   // the face flux is Fhat - Fv
            auto index = [&](const int* o) -> long {
                return ((long)((D == 3) ? wrap(cz + o[2], n2) : 0) * n1 + wrap(cy + o[1], n1)) * n0 + wrap(cx + o[0], n0);
            };
            auto q = [&](const int* o, T& r, T* vel, T& p) {
                const long i = index(o);
                T U[NV];
#pragma unroll
                for (int m = 0; m < NV; ++m) {
                    if constexpr (SECOND) U[m] = T{y[m * ncell + i], v[m * ncell + i]};
                    else U[m] = y[m * ncell + i];
                }
                primitives<D>(G, U, r, vel, p);
            };
            auto w = [&](const int* o, int m) -> double { return wbar[m * ncell + index(o)]; };
            T vb[D], Tb = Sc<T>::make(0.0), Uv[NV];
#pragma unroll
            for (int e = 0; e < D; ++e) vb[e] = Sc<T>::make(0.0);
            visc_vjp_cell<D, T>(G, q, w, vb, Tb);
            const int here[3] = {0, 0, 0};
            T r, vel[D], p;
            q(here, r, vel, p);
            prim_adjoint<D, T>(G, r, vel, -(Tb * p / (r * r)), vb, Tb / r, Uv);
#pragma unroll
            for (int k = 0; k < NV; ++k) acc[k] = acc[k] - Uv[k];
        }
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const long o = k * ncell + c;
            if constexpr (SECOND) {
                ybar[o] = accumulate ? ybar[o] + acc[k].v : acc[k].v;
                ybar2[o] = accumulate ? ybar2[o] + acc[k].d : acc[k].d;
            } else {
                ybar[o] = accumulate ? ybar[o] + acc[k] : acc[k];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// 2-D Cartesian grids: one block per tile of 16 x 16 cells.
//   1. primitives of the tile and its halo (3 cells for MUSCL, 1 for first
//      order) staged in LDS;
//   2. per direction, each face flux whose stencil holds a cell of the tile is reversed once:
//      Fbar -> the adjoints (Lb, Rb) of the left and right reconstructed
//      primitive states, into LDS;
//   3. each cell gathers.  q_L of face c + 1/2 is q_c + s_c / 2 and q_R of
//      face c - 1/2 is q_c - s_c / 2, s_c = mm(q_c - q_{c-1}, q_{c+1} - q_c), so
//      qb_c = Lb_{c+1/2} + Rb_{c-1/2} + (the share of sb_{c-1}, sb_c, sb_{c+1} that
//      the branches of mm give c), sb_c = (Lb_{c+1/2} - Rb_{c-1/2}) / 2;
//   4. the viscous fluxes' transpose from the staged primitives, and one
//      transposed conversion to conserved variables per cell.
// Bound by FP64 arithmetic and its latency (the 96 bytes per cell take a tenth of the time).  A face is
// reversed once (1.19 times with the tile's overhang), where a cell on its own
// reverses the 2 (first order) or 4 (MUSCL) faces per direction whose stencil
// holds it; a state's quotients share a reciprocal; the viscous part is a sweep back instead of 4 forward-mode
// evaluations of each of 12 faces.  Measured: Navier-Stokes MUSCL, 700 x 450,
// 312 -> 45.0 us; first-order Euler, 512^2, 22.6 -> 13.4 us.  (vjp_by_cells: where the cells' kernel is faster.)
// ---------------------------------------------------------------------------
constexpr int kVT = 16;

// One side of a face: the primitive state q = (r, u, v, p), its sound speed c and the derivatives
// dc/dr = -c / (2 r), dc/dp = gamma / (2 r c).
template <typename T>
struct Side {
    T q[4], c, cr, cp;
};

// c (the residual's own sequence, so that the two sides' speeds compare as they did there), dc/dr and dc/dp of a state
template <typename T>
__device__ __forceinline__ void sound_speed(const Geom& G, T r, T p, T& c, T& cr, T& cp) {
    const auto qr = over(r);
    c = Sc<T>::sqrt_(G.g * p / qr);
    cr = -0.5 * (c / qr);
    cp = (Sc<T>::make(G.g) / qr) / over(c + c);
}

// Adjoint of one side of Rusanov's flux along d: the physical flux with weight
// 1/2, the jump term's state (ub = +-ha Fbar, its adjoint in conserved variables), and, where this side's wave
// speed |u_d| + c is the maximum (taken), its adjoint ab (c's derivatives are not finite where p <= 0, and do not
// enter from the other side).  Conserved in terms of primitive variables:
// m = r u, E = p / (gamma - 1) + r |u|^2 / 2.
template <typename T>
__device__ __forceinline__ void rusanov_side_vjp(const Geom& G, int d, const Side<T>& s, const T* Fb, T* ub, bool taken, T ab,
                                                 T* qb) {
    const double half = 0.5;
    const auto qg = over(G.gm1, G.gm1_inv);
    const T r = s.q[0], p = s.q[3], un = s.q[1 + d];
    const T ke = s.q[1] * s.q[1] + s.q[2] * s.q[2];
    const T E = p / qg + (half * r) * ke;
    T unb = Sc<T>::make(0.0);
    ub[1 + d] = ub[1 + d] + half * Fb[0];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const T fb = half * Fb[1 + e];
        ub[1 + e] = ub[1 + e] + fb * un;
        unb = unb + fb * (r * s.q[1 + e]);
    }
    const T fe = half * Fb[3];
    ub[3] = ub[3] + fe * un;
    const T none = Sc<T>::make(0.0);
    unb = unb + fe * (E + p) + (taken ? ((Sc<T>::val(un) >= 0) ? ab : -ab) : none);
    const T keb = half * r * ub[3];
    qb[0] = ub[0] + ub[1] * s.q[1] + ub[2] * s.q[2] + half * ke * ub[3] + (taken ? ab * s.cr : none);
    qb[1] = ub[1] * r + (s.q[1] + s.q[1]) * keb;
    qb[2] = ub[2] * r + (s.q[2] + s.q[2]) * keb;
    qb[3] = half * Fb[1 + d] + fe * un + ub[3] / qg + (taken ? ab * s.cp : none);
    qb[1 + d] = qb[1 + d] + unb;
}

// Adjoints of the two states of a face along d from Fbar, handed to store(side, variable, value).
template <int FLUX, typename T, typename Store>
__device__ __forceinline__ void face_states_vjp(const Geom& G, int d, const Side<T>& L, const Side<T>& R, const T* Fb,
                                                Store store) {
    constexpr int NV = 4;
    if constexpr (FLUX == 0) {
        // Fh = half (FL + FR) - ha (UR - UL), ha = half max(|u_L| + c_L, |u_R| + c_R)
        const double half = 0.5;
        const T sL = sabs(L.q[1 + d]) + L.c, sR = sabs(R.q[1 + d]) + R.c;
        const bool left = Sc<T>::val(sL) >= Sc<T>::val(sR);
        const T ha = half * (left ? sL : sR);
        T UL[NV], UR[NV], ul[NV], ur[NV], qb[NV], ab = Sc<T>::make(0.0);
        to_conserved<2>(G, L.q[0], L.q + 1, L.q[3], UL);
        to_conserved<2>(G, R.q[0], R.q + 1, R.q[3], UR);
#pragma unroll
        for (int m = 0; m < NV; ++m) {
            ab = ab - Fb[m] * (UR[m] - UL[m]);
            ul[m] = ha * Fb[m];
            ur[m] = -ul[m];
        }
        ab = half * ab;
        rusanov_side_vjp<T>(G, d, L, Fb, ul, left, ab, qb);
#pragma unroll
        for (int k = 0; k < NV; ++k) store(0, k, qb[k]);
        rusanov_side_vjp<T>(G, d, R, Fb, ur, !left, ab, qb);
#pragma unroll
        for (int k = 0; k < NV; ++k) store(1, k, qb[k]);
    } else {
        // Roe: forward mode, one dual direction per variable of the two states
        using TT = Dual<T>;
#pragma unroll 1
        for (int i = 0; i < 2 * NV; ++i) {
            TT a[NV], b[NV], UL[NV], UR[NV], F[NV];
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                a[k] = TT{L.q[k], Sc<T>::make(i == k ? 1.0 : 0.0)};
                b[k] = TT{R.q[k], Sc<T>::make(i == NV + k ? 1.0 : 0.0)};
            }
            to_conserved<2>(G, a[0], a + 1, a[3], UL);
            to_conserved<2>(G, b[0], b + 1, b[3], UR);
            num_flux<2, 1>(G, d, UL, a[0], a + 1, a[3], UR, b[0], b + 1, b[3], F);
            T sum = Sc<T>::make(0.0);
#pragma unroll
            for (int k = 0; k < NV; ++k) sum = sum + Fb[k] * F[k].d;
            store(i / NV, i % NV, sum);
        }
    }
}

template <int RECON, bool SECOND, int FLUX, bool NSV>
__global__ __launch_bounds__(256) void k_vjp_tile(Geom G, const double* y, const double* v, const double* wbar,
                                                 double* ybar, double* ybar2, int accumulate, const int* gate, int col,
                                                 int nt0) {
    if (gate && col >= gate[0]) return;   // Krylov column beyond M_eff: nothing to add
    using T = typename std::conditional<SECOND, Dual<double>, double>::type;
    constexpr int NV = 4;
    constexpr int H = (RECON == 0) ? 1 : 3, BX = kVT + 2 * H;
    constexpr int FH = (RECON == 0) ? 0 : 1, NL = kVT + 1 + 2 * FH;   // faces past the tile's own, faces per line
    // first order: a face's sides are cells, whose sound speeds are staged (c, dc/dr, dc/dp)
    constexpr bool CS = RECON == 0 && FLUX == 0;
    __shared__ T sq[CS ? NV + 3 : NV][BX * BX];
    __shared__ T sf[2][NV][NL * kVT];
    const int n0 = G.n[0], n1 = G.n[1];
    const long ncell = G.ncell;
    const int b = xcd_remap(blockIdx.x, gridDim.x);
    const int x0 = (b % nt0) * kVT, y0 = (b / nt0) * kVT;
    const int tid = threadIdx.x, tx = tid % kVT, ty = tid / kVT;
    for (int i = tid; i < BX * BX; i += 256) {
        const long c = (long)wrap(y0 - H + i / BX, n1) * n0 + wrap(x0 - H + i % BX, n0);
        T U[NV];
#pragma unroll
        for (int m = 0; m < NV; ++m) {
            if constexpr (SECOND) U[m] = T{y[m * ncell + c], v[m * ncell + c]};
            else U[m] = y[m * ncell + c];
        }
        // the forward's own rounding: limiters and wave speeds take the branches that the residual took
        T r, vel[2], p;
        primitives<2>(G, U, r, vel, p);
        sq[0][i] = r;
        sq[1][i] = vel[0];
        sq[2][i] = vel[1];
        sq[3][i] = p;
        if constexpr (CS) {
            T cc, cr, cp;
            sound_speed(G, r, p, cc, cr, cp);
            sq[4][i] = cc;
            sq[5][i] = cr;
            sq[6][i] = cp;
        }
    }
    __syncthreads();
    const int here = (ty + H) * BX + tx + H;
    const double half = 0.5;
    T qb[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) qb[k] = Sc<T>::make(0.0);
#pragma unroll
    for (int d = 0; d < 2; ++d) {
        const int sd = d == 0 ? 1 : BX;
        const double inv = G.invdx[d];
        for (int f = tid; f < NL * kVT; f += 256) {
            // face f: between a and b = a + e_d, b at (fx, fy) of the tile
            const int fx = d == 0 ? f % NL - FH : f % kVT, fy = d == 0 ? f / NL : f / kVT - FH;
            const int cb = (fy + H) * BX + fx + H, ca = cb - sd;
            const long gb = (long)wrap(y0 + fy, n1) * n0 + wrap(x0 + fx, n0);
            const long ga = (long)wrap(y0 + fy - (d == 1), n1) * n0 + wrap(x0 + fx - (d == 0), n0);
            T Fb[NV];
            Side<T> L, R;
#pragma unroll
            for (int m = 0; m < NV; ++m) Fb[m] = Sc<T>::make((wbar[m * ncell + gb] - wbar[m * ncell + ga]) * inv);
#pragma unroll
            for (int k = 0; k < NV; ++k) {
                const T a0 = sq[k][ca], ap1 = sq[k][cb];
                if constexpr (RECON == 0) {
                    L.q[k] = a0;
                    R.q[k] = ap1;
                } else {
                    L.q[k] = a0 + half * minmod(a0 - sq[k][ca - sd], ap1 - a0);
                    R.q[k] = ap1 - half * minmod(ap1 - a0, sq[k][cb + sd] - ap1);
                }
            }
            if constexpr (CS) {
                L.c = sq[4][ca], L.cr = sq[5][ca], L.cp = sq[6][ca];
                R.c = sq[4][cb], R.cr = sq[5][cb], R.cp = sq[6][cb];
            } else if constexpr (FLUX == 0) {
                sound_speed(G, L.q[0], L.q[3], L.c, L.cr, L.cp);
                sound_speed(G, R.q[0], R.q[3], R.c, R.cr, R.cp);
            }
            face_states_vjp<FLUX, T>(G, d, L, R, Fb, [&](int side, int k, T x) { sf[side][k][f] = x; });
        }
        __syncthreads();
        const int fs = d == 0 ? 1 : kVT;   // from a face to the next along d
        const int lo = d == 0 ? ty * NL + tx + FH : (ty + FH) * kVT + tx, hi = lo + fs;   // faces c - 1/2 and c + 1/2
#pragma unroll
        for (int k = 0; k < NV; ++k) {
            const T Lb = sf[0][k][hi], Rb = sf[1][k][lo];
            qb[k] = qb[k] + Lb + Rb;
            if constexpr (RECON != 0) {
                // the branch of mm(x, y): 0 none, 1 the backward, 2 the forward difference
                auto branch = [](T x, T z) {
                    if (Sc<T>::val(x) * Sc<T>::val(z) <= 0.0) return 0;
                    return Sc<T>::val(sabs(x)) <= Sc<T>::val(sabs(z)) ? 1 : 2;
                };
                const T* q = sq[k] + here;
                const T e0 = q[-sd] - q[-2 * sd], e1 = q[0] - q[-sd], e2 = q[sd] - q[0], e3 = q[2 * sd] - q[sd];
                const int br = branch(e1, e2);
                const T s0 = half * (Lb - Rb);
                if (br == 1) qb[k] = qb[k] + s0;
                if (br == 2) qb[k] = qb[k] - s0;
                if (branch(e0, e1) == 2) qb[k] = qb[k] + half * (sf[0][k][lo] - sf[1][k][lo - fs]);
                if (branch(e2, e3) == 1) qb[k] = qb[k] - half * (sf[0][k][hi + fs] - sf[1][k][hi]);
            }
        }
        if (d == 0) __syncthreads();
    }
    if (x0 + tx >= n0 || y0 + ty >= n1) return;
    const T r = sq[0][here], p = sq[3][here];
    const T vel[2] = {sq[1][here], sq[2][here]};
    T vb[2] = {qb[1], qb[2]}, rb = qb[0], pb = qb[3];
    if constexpr (NSV) {   // the face flux is Fhat - Fv
        auto q = [&](const int* o, T& rr, T* vv, T& pp) {
            const int i = here + o[1] * BX + o[0];
            rr = sq[0][i];
            vv[0] = sq[1][i];
            vv[1] = sq[2][i];
            pp = sq[3][i];
        };
        auto w = [&](const int* o, int m) -> double {
            return wbar[m * ncell + (long)wrap(y0 + ty + o[1], n1) * n0 + wrap(x0 + tx + o[0], n0)];
        };
        T vv[2] = {Sc<T>::make(0.0), Sc<T>::make(0.0)}, Tb = Sc<T>::make(0.0);
        visc_vjp_cell<2, T>(G, q, w, vv, Tb);
        vb[0] = vb[0] - vv[0];
        vb[1] = vb[1] - vv[1];
        Tb = Tb / r;               // T = p / r
        pb = pb - Tb;
        rb = rb + Tb * (p / r);
    }
    T Ub[NV];
    prim_adjoint<2, T>(G, r, vel, rb, vb, pb, Ub);
    const long c = (long)(y0 + ty) * n0 + x0 + tx;
#pragma unroll
    for (int k = 0; k < NV; ++k) {
        const long o = k * ncell + c;
        if constexpr (SECOND) {
            ybar[o] = accumulate ? ybar[o] + Ub[k].v : Ub[k].v;
            ybar2[o] = accumulate ? ybar2[o] + Ub[k].d : Ub[k].d;
        } else {
            ybar[o] = accumulate ? ybar[o] + Ub[k] : Ub[k];
        }
    }
}

// ---------------------------------------------------------------------------
// O-grid (2-D, periodic in i, wall at j = -1/2, far field at j = ny - 1/2).
// A face's flux Fhat - Fv is evaluated from a 4 x 3 patch of cells P[a][b]:
// i-faces (kind 0) between (i, j) and (i + 1, j): P[a][b] = (i + a - 1, j + b - 1);
// j-faces (kind 1) between (i, j) and (i, j + 1): P[a][b] = (i + b - 1, j + a - 1);
// the wall face below (i, 0) (kind 2) and the far-field face above (i, ny - 1)
// (kind 3) read P[1][1] only.  Rows outside the grid hold a copy of P[1][1]
// and are never read: MUSCL slopes and derivatives along j are one-sided
// (or zero) in the first and last rows, as in the residual.
template <int RECON, int FLUX, bool NSV, typename S>
__device__ __forceinline__ void ogrid_face(const Geom& G, int kind, int j, long fc, const S (*P)[3][4], S* F) {
    const long ncell = G.ncell;
    const int ny = G.n[1], n0 = G.n[0];
    const double half = 0.5;
    if (kind >= 2) {
        S r, vel[2], p;
        primitives<2>(G, P[1][1], r, vel, p);
        if (kind == 2) {
            const int i = (int)(fc % n0);
            const double wx = G.metric[9 * ncell + i], wy = G.metric[9 * ncell + n0 + i];
            F[0] = Sc<S>::make(0.0);
            F[1] = p * wx;
            F[2] = p * wy;
            F[3] = Sc<S>::make(0.0);
            if constexpr (NSV) {
                const S zero = Sc<S>::make(0.0);
                const S T0 = p / r;
                S Fv[4];
                curv_visc_core<S>(G, 1, wx, wy, G.metric[9 * ncell + 2 * n0 + i], G.metric[9 * ncell + 3 * n0 + i],
                                  vel[0] - 0.0, vel[1] - 0.0, T0 - G.t_wall, zero, zero, zero, zero, zero,
                                  half * (T0 + G.t_wall), Fv);
#pragma unroll
                for (int m = 1; m < 4; ++m) F[m] = F[m] - Fv[m];
            }
        } else {
            S Ub[4], Uf[4], rf, vf[2], pf;
            to_conserved<2>(G, r, vel, p, Ub);
#pragma unroll
            for (int m = 0; m < 4; ++m) Uf[m] = Sc<S>::make(G.uinf[m]);
            primitives<2>(G, Uf, rf, vf, pf);
            rotated_flux<FLUX, S>(G, Ub, r, vel, p, Uf, rf, vf, pf, G.metric[2 * ncell + fc], G.metric[3 * ncell + fc],
                                  F);
        }
        return;
    }
    const int d = kind;
    constexpr int A0 = (RECON == 0) ? 1 : 0, A1 = (RECON == 0) ? 2 : 3;   // patch slots the flux reads
    constexpr int B0 = NSV ? 0 : 1, B1 = NSV ? 2 : 1;
    S q[4][3][4];   // primitives (r, u, v, p) of the patch
#pragma unroll
    for (int a = A0; a <= A1; ++a)
#pragma unroll
        for (int b = B0; b <= B1; ++b) {
            S vel[2];
            primitives<2>(G, P[a][b], q[a][b][0], vel, q[a][b][3]);
            q[a][b][1] = vel[0];
            q[a][b][2] = vel[1];
        }
    S UL[4], UR[4], vL[2], vR[2], rL, rR, pL, pR;
    if constexpr (RECON == 0) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            UL[m] = P[1][1][m];
            UR[m] = P[2][1][m];
        }
        rL = q[1][1][0], rR = q[2][1][0], pL = q[1][1][3], pR = q[2][1][3];
        vL[0] = q[1][1][1], vL[1] = q[1][1][2], vR[0] = q[2][1][1], vR[1] = q[2][1][2];
    } else {
        const bool flatL = d == 1 && j == 0, flatR = d == 1 && j + 1 == ny - 1;
        S qL[4], qR[4];
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            const S am1 = q[0][1][m], a0 = q[1][1][m], ap1 = q[2][1][m], ap2 = q[3][1][m];
            qL[m] = flatL ? a0 + half * Sc<S>::make(0.0) : a0 + half * minmod(a0 - am1, ap1 - a0);
            qR[m] = flatR ? ap1 - half * Sc<S>::make(0.0) : ap1 - half * minmod(ap1 - a0, ap2 - ap1);
        }
        rL = qL[0], rR = qR[0], pL = qL[3], pR = qR[3];
        vL[0] = qL[1], vL[1] = qL[2], vR[0] = qR[1], vR[1] = qR[2];
        to_conserved<2>(G, rL, vL, pL, UL);
        to_conserved<2>(G, rR, vR, pR, UR);
    }
    rotated_flux<FLUX, S>(G, UL, rL, vL, pL, UR, rR, vR, pR, G.metric[(long)(2 * d) * ncell + fc],
                          G.metric[(long)(2 * d + 1) * ncell + fc], F);
    if constexpr (NSV) {
        // derivatives along the face: central in the periodic i direction; along
        // j one-sided in the first and last rows
        auto T = [&](int a, int b) { return q[a][b][3] / q[a][b][0]; };
        S nf[3], tf[3], uf[2];
        const S Ta = T(1, 1), Tb = T(2, 1);
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            auto val = [&](int a, int b) { return k < 2 ? q[a][b][1 + k] : T(a, b); };
            nf[k] = val(2, 1) - val(1, 1);
            S ga, gb;
            if (d == 1) {
                ga = (val(1, 2) - val(1, 0)) * half;
                gb = (val(2, 2) - val(2, 0)) * half;
            } else if (j == 0) {
                ga = val(1, 2) - val(1, 1);
                gb = val(2, 2) - val(2, 1);
            } else if (j == ny - 1) {
                ga = val(1, 1) - val(1, 0);
                gb = val(2, 1) - val(2, 0);
            } else {
                ga = (val(1, 2) - val(1, 0)) * half;
                gb = (val(2, 2) - val(2, 0)) * half;
            }
            tf[k] = half * (ga + gb);
            if (k < 2) uf[k] = half * (val(1, 1) + val(2, 1));
        }
        S Fv[4];
        curv_visc_core<S>(G, d, G.metric[(long)(2 * d) * ncell + fc], G.metric[(long)(2 * d + 1) * ncell + fc],
                          G.metric[(long)(5 + 2 * d) * ncell + fc], G.metric[(long)(6 + 2 * d) * ncell + fc], nf[0],
                          nf[1], nf[2], tf[0], tf[1], tf[2], uf[0], uf[1], half * (Ta + Tb), Fv);
#pragma unroll
        for (int m = 1; m < 4; ++m) F[m] = F[m] - Fv[m];
    }
}

// Adjoint on an O-grid: cell c gathers Fbar^T d(Fhat - Fv)/dU_c from every
// (face, patch position) pair that places c in the face's patch, each by
// forward mode; Fbar of a face is wbar_b / A_b - wbar_a / A_a (the wall face
// has only b = (i, 0), the far-field face only a = (i, ny - 1)).  One thread
// per (variable m, cell c), c fastest: it seeds the one dual direction U_c[m].
template <int RECON, bool SECOND, int FLUX, bool NSV>
__global__ __launch_bounds__(64) void k_vjp_ogrid(Geom G, const double* y, const double* v, const double* wbar,
                                                  double* ybar, double* ybar2, int accumulate, const int* gate,
                                                  int col) {
    if (gate && col >= gate[0]) return;
    using T = typename std::conditional<SECOND, Dual<double>, double>::type;
    using TT = Dual<T>;
    const int n0 = G.n[0], ny = G.n[1];
    const long ncell = G.ncell;
    const double* ia = G.metric + 4 * ncell;
    constexpr int A0 = (RECON == 0) ? 1 : 0, A1 = (RECON == 0) ? 2 : 3;   // patch rows a the flux reads
    constexpr int B0 = NSV ? 0 : 1, B1 = NSV ? 2 : 1;                     // patch columns b
    const long stride = (long)gridDim.x * blockDim.x;
    for (long idx = (long)blockIdx.x * blockDim.x + threadIdx.x; idx < 4 * ncell; idx += stride) {
        const int m = (int)(idx / ncell);
        const long c = idx - (long)m * ncell;
        const int cx = (int)(c % n0), cy = (int)(c / n0);
        T acc = Sc<T>::make(0.0);
        auto load = [&](long cell, T* u) {
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const long o = m * ncell + cell;
                if constexpr (SECOND) u[m] = T{y[o], v[o]};
                else u[m] = y[o];
            }
        };
        // one (face, position) pair: fi, fj the face's cell a (or the wall /
        // far-field cell), (pa, pb) the position of c in its patch
        auto face = [&](int kind, int fi, int fj, int pa, int pb) {
            const long fc = (long)fj * n0 + fi;
            T base[4][3][4];
            if (kind >= 2) {
                load(fc, base[1][1]);
            } else {
#pragma unroll
                for (int a = 0; a < 4; ++a)
#pragma unroll
                    for (int b = 0; b < 3; ++b) {
                        int ii, jj;
                        if (kind == 0) ii = wrap(fi + a - 1, n0), jj = fj + b - 1;
                        else ii = wrap(fi + b - 1, n0), jj = fj + a - 1;
                        if (a < A0 || a > A1 || b < B0 || b > B1 || jj < 0 || jj >= ny) {
                            ii = fi;
                            jj = fj;
                        }
                        load((long)jj * n0 + ii, base[a][b]);
                    }
            }
            T fbar[4];
            if (kind == 2) {
#pragma unroll
                for (int m = 0; m < 4; ++m) fbar[m] = Sc<T>::make(wbar[m * ncell + fc] * ia[fc]);
            } else if (kind == 3) {
#pragma unroll
                for (int m = 0; m < 4; ++m) fbar[m] = Sc<T>::make(-(wbar[m * ncell + fc] * ia[fc]));
            } else {
                const long fb = (kind == 0) ? (long)fj * n0 + wrap(fi + 1, n0) : fc + n0;
#pragma unroll
                for (int m = 0; m < 4; ++m)
                    fbar[m] = Sc<T>::make(wbar[m * ncell + fb] * ia[fb] - wbar[m * ncell + fc] * ia[fc]);
            }
            TT Ud[4][3][4], Fd[4];
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int b = 0; b < 3; ++b)
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        Ud[a][b][k] = TT{base[a][b][k], Sc<T>::make((a == pa && b == pb && k == m) ? 1.0 : 0.0)};
            ogrid_face<RECON, FLUX, NSV, TT>(G, kind, fj, fc, Ud, Fd);
            T sum = Sc<T>::make(0.0);
#pragma unroll
            for (int k = 0; k < 4; ++k) sum = sum + fbar[k] * Fd[k].d;
            acc = acc + sum;
        };
#pragma nounroll
        for (int a = A0; a <= A1; ++a)
#pragma nounroll
            for (int b = B0; b <= B1; ++b) {
                // i-face with cell a = (cx - a + 1, cy - b + 1)
                const int fj0 = cy - (b - 1);
                if (fj0 >= 0 && fj0 < ny) face(0, wrap(cx - (a - 1), n0), fj0, a, b);
                // j-face with cell a = (cx - b + 1, cy - a + 1), j in [0, ny - 2]
                const int fj1 = cy - (a - 1);
                if (fj1 >= 0 && fj1 <= ny - 2) face(1, wrap(cx - (b - 1), n0), fj1, a, b);
            }
        if (cy == 0) face(2, cx, 0, 1, 1);
        if (cy == ny - 1) face(3, cx, ny - 1, 1, 1);
        if constexpr (SECOND) {
            ybar[idx] = accumulate ? ybar[idx] + acc.v : acc.v;
            ybar2[idx] = accumulate ? ybar2[idx] + acc.d : acc.d;
        } else {
            ybar[idx] = accumulate ? ybar[idx] + acc : acc;
        }
    }
}

template <int RECON, int FLUX, bool NSV>
static hipError_t launch_vjp_og(const Geom& G, const double* y, const double* v, const double* wbar, double* ybar,
                                double* ybar2, int accumulate, const int* gate, int col, hipStream_t st) {
    long g = (4 * G.ncell + 63) / 64;   // small blocks: O-grids have few cells and much work per cell
    if (g > 65536) g = 65536;
    if (v)
        hipLaunchKernelGGL((k_vjp_ogrid<RECON, true, FLUX, NSV>), dim3((unsigned)g), dim3(64), 0, st, G, y, v, wbar,
                           ybar, ybar2, accumulate, gate, col);
    else
        hipLaunchKernelGGL((k_vjp_ogrid<RECON, false, FLUX, NSV>), dim3((unsigned)g), dim3(64), 0, st, G, y, v,
                           wbar, ybar, ybar2, accumulate, gate, col);
    return hipGetLastError();
}

template <int RECON>
static hipError_t launch_vjp_ogrid(const Geom& G, const double* y, const double* v, const double* wbar, double* ybar,
                                   double* ybar2, int accumulate, const int* gate, int col, hipStream_t st) {
    const bool ns = G.mu != 0.0;
    if (G.flux == 1) {
        if (ns) return launch_vjp_og<RECON, 1, true>(G, y, v, wbar, ybar, ybar2, accumulate, gate, col, st);
        return launch_vjp_og<RECON, 1, false>(G, y, v, wbar, ybar, ybar2, accumulate, gate, col, st);
    }
    if (ns) return launch_vjp_og<RECON, 0, true>(G, y, v, wbar, ybar, ybar2, accumulate, gate, col, st);
    return launch_vjp_og<RECON, 0, false>(G, y, v, wbar, ybar, ybar2, accumulate, gate, col, st);
}

// Whether a 2-D Cartesian product is gathered cell by cell (k_vjp) instead of from the faces of tiles (k_vjp_tile).
// A tile's arithmetic is that of its 16 x 16 cells however many of them the grid has, and first order a tile saves
// little: a cell has two faces per direction, which it reverses without the staging.  Measured, tile and cells:
//   first order, Roe: the dual evaluations are the whole time and a tile's second round of faces holds 16 of 272
//     (Euler second-order adjoint 318 and 201 us at 700 x 450, 70 and 40 at 100^2; product 82 and 73, 29 and 20);
//     only the Navier-Stokes product has more to share from 256^2 on (36 and 42 us there, 38 and 31 at 100^2);
//   first order, Euler, Rusanov, second-order adjoint: 36 and 32 us at 700 x 450, 30 and 28 at 512^2, 12 and 10 at 17^2;
//   thin grids of more tiles than CUs: first order the lines cross near five eighths of a tile's cells in the grid
//     (Euler product 20 and 16 us at 30000 x 8, 12 and 11 at 16384 x 12, 13 and 17 at 512^2), with MUSCL near five
//     sixteenths (Euler product 59 and 46 us at 65536 x 4, 22 and 29 at 20000 x 5; Navier-Stokes 84 and 73, 37 and 44),
//     Roe's second-order adjoint nine (533 and 460 at 30000 x 8, 264 and 346 at 16384 x 12).
//     Up to one tile per CU the time is a tile's latency, whatever it holds.
template <int RECON, int FLUX, bool NSV, bool SECOND>
static bool vjp_by_cells(long ncell, long tiles) {
    constexpr int sixteenths = RECON == 0 ? 10 : (FLUX == 1 && SECOND ? 9 : 5);
    const bool thin = tiles > 256 && 16 * ncell < sixteenths * 256 * tiles;
    if (RECON == 0 && FLUX == 1) return thin || SECOND || !NSV || ncell < (1L << 16);
    return thin || (RECON == 0 && !NSV && SECOND);
}

template <int D, int RECON, int FLUX, bool NSV, int GEO, bool SECOND>
static hipError_t launch_vjp_s(const Geom& G, const double* y, const double* v, const double* wbar, double* ybar,
                               double* ybar2, int accumulate, const int* gate, int col, hipStream_t st) {
    if constexpr (D == 2 && GEO == 0) {
        const int nt0 = (G.n[0] + kVT - 1) / kVT, nt1 = (G.n[1] + kVT - 1) / kVT;
        const long nb = (long)nt0 * nt1;
        if (nb <= 0x7fffffffL && !vjp_by_cells<RECON, FLUX, NSV, SECOND>(G.ncell, nb)) {
            hipLaunchKernelGGL((k_vjp_tile<RECON, SECOND, FLUX, NSV>), dim3((unsigned)nb), dim3(256), 0, st, G, y, v, wbar,
                               ybar, ybar2, accumulate, gate, col, nt0);
            return hipGetLastError();
        }
    }
    long g = (G.ncell + 255) / 256;
    if (g > 16384) g = 16384;
    hipLaunchKernelGGL((k_vjp<D, RECON, SECOND, FLUX, NSV, GEO>), dim3((unsigned)g), dim3(256), 0, st, G, y, v, wbar, ybar,
                       ybar2, accumulate, gate, col);
    return hipGetLastError();
}

template <int D, int RECON, int FLUX, bool NSV, int GEO = 0>
static hipError_t launch_vjp_f(const Geom& G, const double* y, const double* v, const double* wbar, double* ybar,
                               double* ybar2, int accumulate, const int* gate, int col, hipStream_t st) {
    if (v) return launch_vjp_s<D, RECON, FLUX, NSV, GEO, true>(G, y, v, wbar, ybar, ybar2, accumulate, gate, col, st);
    return launch_vjp_s<D, RECON, FLUX, NSV, GEO, false>(G, y, v, wbar, ybar, ybar2, accumulate, gate, col, st);
}

template <int D, int RECON, bool NSV>
static hipError_t launch_vjp_n(const Geom& G, const double* y, const double* v, const double* wbar, double* ybar,
                               double* ybar2, int accumulate, const int* gate, int col, hipStream_t st) {
    if (G.flux == 1) return launch_vjp_f<D, RECON, 1, NSV>(G, y, v, wbar, ybar, ybar2, accumulate, gate, col, st);
    return launch_vjp_f<D, RECON, 0, NSV>(G, y, v, wbar, ybar, ybar2, accumulate, gate, col, st);
}

template <int D, int RECON>
static hipError_t launch_vjp_t(const Geom& G, const double* y, const double* v, const double* wbar, double* ybar,
                               double* ybar2, int accumulate, const int* gate, int col, hipStream_t st) {
    if constexpr (D == 2) {
        if (G.metric && G.ogrid)
            return launch_vjp_ogrid<RECON>(G, y, v, wbar, ybar, ybar2, accumulate, gate, col, st);
        // periodic curvilinear grid
        if (G.metric) {
            if (G.mu != 0.0) {
                if (G.flux == 1)
                    return launch_vjp_f<2, RECON, 1, true, 1>(G, y, v, wbar, ybar, ybar2, accumulate, gate, col, st);
                return launch_vjp_f<2, RECON, 0, true, 1>(G, y, v, wbar, ybar, ybar2, accumulate, gate, col, st);
            }
            if (G.flux == 1) return launch_vjp_f<2, RECON, 1, false, 1>(G, y, v, wbar, ybar, ybar2, accumulate, gate, col, st);
            return launch_vjp_f<2, RECON, 0, false, 1>(G, y, v, wbar, ybar, ybar2, accumulate, gate, col, st);
        }
    }
    if (G.mu != 0.0) return launch_vjp_n<D, RECON, true>(G, y, v, wbar, ybar, ybar2, accumulate, gate, col, st);
    return launch_vjp_n<D, RECON, false>(G, y, v, wbar, ybar, ybar2, accumulate, gate, col, st);
}

hipError_t launch_vjp(const Geom& G, int recon, const double* y, const double* v, const double* wbar, double* ybar,
                      double* ybar2, int accumulate, hipStream_t st, const int* gate, int col) {
    if (G.D == 2) return recon == 0 ? launch_vjp_t<2, 0>(G, y, v, wbar, ybar, ybar2, accumulate, gate, col, st)
                                    : launch_vjp_t<2, 1>(G, y, v, wbar, ybar, ybar2, accumulate, gate, col, st);
    return recon == 0 ? launch_vjp_t<3, 0>(G, y, v, wbar, ybar, ybar2, accumulate, gate, col, st)
                      : launch_vjp_t<3, 1>(G, y, v, wbar, ybar, ybar2, accumulate, gate, col, st);
}

}  // namespace rok

