// Per-node pieces of the heated-channel step (collisions and boundary values),
// shared by the one-, two- and many-step kernels so that all of them round
// identically.  Included only by the library's .hip sources.
#pragma once

#include "lbm_device.h"

namespace lbm {
namespace {

// ChanK in the type the kernel computes in: the constants of the collision
// stay in scalar registers over the steps.
template <typename C>
struct ChanKT {
    int nx, ny, batch, bcx, bcy, flow, thermal, flow_mrt, buoy;
    C rho_ref, qdt, Lf[9], Lt[9], Ft[2], Bt[2], Tw[2];
};

template <typename C>
ChanKT<C> chan_kt(const ChanK& k) {
    ChanKT<C> r{};
    r.nx = k.nx; r.ny = k.ny; r.batch = k.batch;
    r.bcx = k.bcx; r.bcy = k.bcy;
    r.flow = k.flow; r.thermal = k.thermal; r.flow_mrt = k.flow_mrt; r.buoy = k.buoy;
    r.rho_ref = C(k.rho_ref);
    r.qdt = C(k.qdt);
    for (int q = 0; q < 9; ++q) {
        r.Lf[q] = C(k.Lf[q]);
        r.Lt[q] = C(k.Lt[q]);
    }
    for (int q = 0; q < 2; ++q) {
        r.Ft[q] = C(k.Ft[q]);
        r.Bt[q] = C(k.Bt[q]);
        r.Tw[q] = C(k.Tw[q]);
    }
    return r;
}

// Thermal lattice of the channel: D2Q5 (QT = 5) or D2Q9 (QT = 9, the set of
// Sec. 3 and App. D).
template <int QT> __device__ __forceinline__ int tex(int i) { return QT == 9 ? EX[i] : EX5[i]; }
template <int QT> __device__ __forceinline__ int tey(int i) { return QT == 9 ? EY[i] : EY5[i]; }
template <int QT> __device__ __forceinline__ int topp(int i) { return QT == 9 ? OPP[i] : OPP5[i]; }
template <int QT> __device__ __forceinline__ int tmir(int i) { return QT == 9 ? MIRY[i] : MIRY5[i]; }
template <int QT, typename C> __device__ __forceinline__ C twt(int i) {
    return QT == 9 ? wgt<C>(i) : wgt5<C>(i);
}

// T - T_ref of a node from its (deviation) thermal populations, with the half
// source (Eq. zero_moment_g)
template <int QT, typename C>
__device__ __forceinline__ C chan_th(const C (&e)[QT], C qdt) {
    if constexpr (QT == 9)
        return ((e[0] + (e[1] + e[3]) + (e[2] + e[4])) + ((e[5] + e[7]) + (e[6] + e[8]))) +
               C(0.5) * qdt;
    else
        return (e[0] + (e[1] + e[3]) + (e[2] + e[4])) + C(0.5) * qdt;
}

// Both collisions of a node: ds from the deviations d (Eq. colisao_MRT or Eq.
// eq_lattice_boltzmann_BGK with Guo forcing; a frozen flow keeps d), es from
// the thermal populations e (Sec. 2.2 and Sec. 3, advective part built on
// T - T_ref, in moment space with the rates Lt).
template <typename C, int QT, typename K>
__device__ __forceinline__ void chan_collide(const K& k, const C (&d)[9], C drho, C rho, C ux,
                                             C uy, C ftx, C fty, const C (&e)[QT], C th, C qdt,
                                             C (&ds)[9], C (&es)[QT]) {
    if (k.flow) {
        const C uu = ux * ux + uy * uy;
        if (k.flow_mrt) {
            // Moment space: the non-equilibrium moments are M d minus the
            // moments of the deviation equilibrium (Eq. feq_geral less
            // w_i rho_ref) in closed form, (drho, -2 drho + 3 rho |u|^2,
            // drho - 3 rho |u|^2, rho u_x, -rho u_x, rho u_y, -rho u_y,
            // rho (u_x^2 - u_y^2), rho u_x u_y); the Guo term of Eq.
            // forcing_term has the moments (0, 6 u.F, -6 u.F, F_x, -F_x, F_y,
            // -F_y, 2 (u_x F_x - u_y F_y), u_x F_y + u_y F_x).
            C md[9], dm[9], dv[9];
            moments9(d, md);
            const C ru2 = rho * uu, rux = rho * ux, ruy = rho * uy;
            const C mn[9] = {md[0] - drho,
                             md[1] - (C(-2) * drho + C(3) * ru2),
                             md[2] - (drho - C(3) * ru2),
                             md[3] - rux,
                             md[4] + rux,
                             md[5] - ruy,
                             md[6] + ruy,
                             md[7] - (rux * ux - ruy * uy),
                             md[8] - rux * uy};
            const C uf = ux * ftx + uy * fty;
            const C mf[9] = {C(0),  C(6) * uf, C(-6) * uf, ftx, -ftx, fty, -fty,
                             C(2) * (ux * ftx - uy * fty), ux * fty + uy * ftx};
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                const C L = C(k.Lf[q]);
                dm[q] = -L * mn[q] + (C(1) - C(0.5) * L) * mf[q];
            }
            inverse9(dm, dv);
#pragma unroll
            for (int i = 0; i < 9; ++i) ds[i] = d[i] + dv[i];
        } else {
            C neq[9], fh[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                const C eu = C(EX[i]) * ux + C(EY[i]) * uy;
                // deviation of Eq. feq_geral from w_i rho_ref
                const C feq =
                    wgt<C>(i) * (drho + rho * (C(3) * eu + C(4.5) * eu * eu - C(1.5) * uu));
                neq[i] = d[i] - feq;
                // dt * Guo term of Eq. forcing_term (without its prefactor)
                fh[i] = wgt<C>(i) * ((C(3) * (C(EX[i]) - ux) + C(9) * eu * C(EX[i])) * ftx +
                                     (C(3) * (C(EY[i]) - uy) + C(9) * eu * C(EY[i])) * fty);
            }
            const C L = C(k.Lf[7]);
#pragma unroll
            for (int i = 0; i < 9; ++i) ds[i] = d[i] - L * neq[i] + (C(1) - C(0.5) * L) * fh[i];
        }
    } else {
#pragma unroll
        for (int i = 0; i < 9; ++i) ds[i] = d[i];
    }
    if (k.thermal) {
        C m[QT], dm[QT], dv[QT];
        if constexpr (QT == 9) {
            C neq[9];
#pragma unroll
            for (int i = 0; i < 9; ++i)
                neq[i] = e[i] - twt<QT, C>(i) * th *
                                    (C(1) + C(3) * (C(tex<QT>(i)) * ux + C(tey<QT>(i)) * uy));
            moments9(neq, m);
            // moments of the source w_i qdot dt: qdt (1, -2, 1, 0, ...)
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                const C L = C(k.Lt[q]);
                const C ms = q == 0 ? qdt : (q == 1 ? C(-2) * qdt : (q == 2 ? qdt : C(0)));
                dm[q] = -L * m[q] + (C(1) - C(0.5) * L) * ms;
            }
            inverse9(dm, dv);
        } else {
            // moments of e less those of the equilibrium w_i th (1 + 3 c_i.u):
            // (th, th u_x, th u_y, -2/3 th, 0)
            C me[5];
            moments5(e, me);
            m[0] = me[0] - th;
            m[1] = me[1] - th * ux;
            m[2] = me[2] - th * uy;
            m[3] = me[3] - C(-2) / C(3) * th;
            m[4] = me[4];
            // moments of the source w_i qdot dt: qdt (1, 0, 0, -2/3, 0)
            const C ms[5] = {qdt, C(0), C(0), C(-2) / C(3) * qdt, C(0)};
#pragma unroll
            for (int q = 0; q < 5; ++q) {
                const C L = C(k.Lt[q]);
                dm[q] = -L * m[q] + (C(1) - C(0.5) * L) * ms[q];
            }
            inverse5(dm, dv);
        }
#pragma unroll
        for (int i = 0; i < QT; ++i) es[i] = e[i] + dv[i];
    }
}

// Values a boundary rule puts into the node's opposite slot OPP[i] for a
// population i that leaves the domain:
// moving-wall bounce-back with the inlet profile u_in (Eq. BB_vel)
template <typename C>
__device__ __forceinline__ C chan_inlet_f(int i, C dsi, C rho_ref, C uin) {
    return dsi - C(6) * wgt<C>(i) * rho_ref * (C(EX[i]) * uin);
}
// anti-bounce-back pressure outlet with the wall velocity u_w (Eq.
// anti_BB_vel, rho_w = rho_ref)
template <typename C>
__device__ __forceinline__ C chan_outlet_f(int i, C dsi, C rho_ref, C uwx, C uwy) {
    const C eu = C(EX[i]) * uwx + C(EY[i]) * uwy;
    return -dsi + C(2) * wgt<C>(i) * rho_ref * (C(4.5) * eu * eu - C(1.5) * (uwx * uwx + uwy * uwy));
}
// prescribed wall flux q (scaled, times the time modulation mod), Eq. BB_T
// with lambda_i = 6 w_i (1 on D2Q5), into slot topp(i)
template <int QT, typename C>
__device__ __forceinline__ C chan_flux_g(int i, C esi, C q, C mod) {
    const C lam = QT == 9 ? C(6) * wgt<C>(i) : C(1);
    return esi + lam * q * mod;
}
// anti-bounce-back fixed temperature tw (deviation form, Eq. anti_BB_T), into
// slot topp(i)
template <int QT, typename C>
__device__ __forceinline__ C chan_antibb_g(int i, C esi, C tw) {
    return -esi + C(2) * twt<QT, C>(i) * tw;
}

}  // namespace
}  // namespace lbm
