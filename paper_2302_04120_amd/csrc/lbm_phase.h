// Per-node pieces of the two-phase D2Q9 step (state layout, stencils, macros and
// both collisions), shared by the one-, two- and many-step kernels so that all
// of them round identically.  Included only by the library's .hip sources.
#pragma once

#include "lbm_device.h"

#include <type_traits>

namespace lbm {
namespace {

// PhaseK in the type the kernel computes in
template <typename C>
struct PhaseKT {
    int nx, ny, batch, bcy, z_mrt, qy_printed, visc_mode;
    C rho_g, drl, nuh_g, dnu, zh_g, dz, w_phi, beta, kap6, fs_scale, Fbt[2], dxW, Geps;
    __device__ __forceinline__ C drho() const { return drl; }
    __device__ __forceinline__ C dnuh() const { return dnu; }
    __device__ __forceinline__ C dzh() const { return dz; }
};
template <typename C>
PhaseKT<C> phase_kt(const PhaseK& k) {
    PhaseKT<C> r{};
    r.nx = k.nx; r.ny = k.ny; r.batch = k.batch; r.bcy = k.bcy;
    r.z_mrt = k.z_mrt; r.qy_printed = k.qy_printed; r.visc_mode = k.visc_mode;
    r.rho_g = C(k.rho_g); r.drl = C(k.drho());
    r.nuh_g = C(k.nuh_g); r.dnu = C(k.dnuh());
    r.zh_g = C(k.zh_g); r.dz = C(k.dzh());
    r.w_phi = C(k.w_phi); r.beta = C(k.beta); r.kap6 = C(k.kap6); r.fs_scale = C(k.fs_scale);
    r.Fbt[0] = C(k.Fbt[0]); r.Fbt[1] = C(k.Fbt[1]);
    r.dxW = C(k.dxW); r.Geps = C(k.Geps);
    return r;
}

// Planes of the two-phase D2Q9 state in the node-block layout (bidx): h_0..h_8,
// z_0..z_8, in FP32 the low part of h_0, then (phi u)_x and (phi u)_y.
template <typename S>
struct PhasePlanes {
    static constexpr bool RMASS = std::is_same<S, float>::value;
    static constexpr int NPL = RMASS ? 21 : 20;
    static constexpr int H = 0, Z = 9, LO = 18, PU = RMASS ? 19 : 18;
};
template <typename S>
__device__ __forceinline__ long long pidx(int i, long long n) {
    return bidx(PhasePlanes<S>::NPL, i, n);
}

// phi of a node from its stored h_i, Eq. zero_moment_h (rest population with
// its low part).  One summation order everywhere, so that every kernel sees
// the same phi for the same populations.
template <typename C>
__device__ __forceinline__ C phi_sum(const C (&h)[9], C hlo) {
    return (h[0] + hlo) + (((h[1] + h[3]) + (h[2] + h[4])) + ((h[5] + h[7]) + (h[6] + h[8])));
}

// Reciprocals of the two-phase collision: the hardware's 1-ulp reciprocal and
// reciprocal square root in FP32 (FP32 storage carries ~1e-7 relative
// rounding anyway), exact division in FP64.
__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double rcp(double x) { return 1.0 / x; }
__device__ __forceinline__ float rsq(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double rsq(double x) { return 1.0 / sqrt(x); }

// Everything a node derives from its phi neighbourhood and its z_i before
// the collision.  pn[i] = phi at x + e_i (pn[0] = phi at the node).
template <typename C>
struct PhaseLocal {
    C phi, Gx, Gy, rho, drl, wn, mu, fsx, fsy, nxv, nyv, ux, uy, uu, ug, ph;
};

template <typename C, typename K>
__device__ __forceinline__ PhaseLocal<C> phase_local(const K& k, const C (&pn)[9],
                                                     const C (&z)[9]) {
    PhaseLocal<C> L;
    // ---- stencils, Eq. gradient and Eq. laplacian in lattice form:
    //      grad phi = 3 G / dx, lap phi = 6 L / dx^2 with G = sum w_i e_i phi_i and
    //      L = sum w_i (phi_i - phi), summed by weight class (1/9 on the axes,
    //      1/36 on the diagonals).  Both are built from differences of
    //      neighbouring values, which are exact in floating point; a sum of the
    //      neighbours minus (5/9) phi would cancel terms of size phi down to the
    //      Laplacian and lose most of its digits in FP32.
    const C phi = pn[0];
    const C dpp = pn[5] - pn[7];  // (+1,+1) - (-1,-1)
    const C dpm = pn[8] - pn[6];  // (+1,-1) - (-1,+1)
    const C Gx = C(1.0 / 9.0) * (pn[1] - pn[3]) + C(1.0 / 36.0) * (dpp + dpm);
    const C Gy = C(1.0 / 9.0) * (pn[2] - pn[4]) + C(1.0 / 36.0) * (dpp - dpm);
    const C sax = ((pn[1] - phi) + (pn[3] - phi)) + ((pn[2] - phi) + (pn[4] - phi));
    const C sdg = ((pn[5] - phi) + (pn[7] - phi)) + ((pn[6] - phi) + (pn[8] - phi));
    const C Lp = C(1.0 / 9.0) * sax + C(1.0 / 36.0) * sdg;
    const C drl = C(k.drho());
    const C rho = C(k.rho_g) + phi * drl;  // linear in phi (Sec. 2.3)
    const C ir = rcp(rho);
    // dt / tau = 1 / (3 nu dt / dx^2 + 1/2), with nu linear in phi or, in the
    // zeta form of Sec. 4.4, nu = zeta / rho
    if (k.visc_mode == 0) {
        L.wn = rcp(C(3) * (C(k.nuh_g) + phi * C(k.dnuh())) + C(0.5));
    } else {
        const C zh = C(k.zh_g) + phi * C(k.dzh());
        L.wn = rho * rcp(C(3) * zh + C(0.5) * rho);
    }
    // chemical potential, Eq. chemical_potential; surface force F_s = mu grad phi
    const C mu = C(4) * C(k.beta) * phi * (phi - C(1)) * (phi - C(0.5)) - C(k.kap6) * Lp;
    L.fsx = mu * Gx * C(k.fs_scale) + C(k.Fbt[0]);
    L.fsy = mu * Gy * C(k.fs_scale) + C(k.Fbt[1]);
    // guarded interface normal (text after Eq. laplacian)
    const C gn2 = Gx * Gx + Gy * Gy;
    L.nxv = C(0);
    L.nyv = C(0);
    if (gn2 > C(k.Geps) * C(k.Geps)) {
        const C ig = rsq(gn2);
        L.nxv = Gx * ig;
        L.nyv = Gy * ig;
    }
    // ---- pressure populations: velocity first (Eq. u_Liang), then pressure
    const C jx = (z[1] - z[3]) + ((z[5] - z[7]) + (z[8] - z[6]));
    const C jy = (z[2] - z[4]) + ((z[5] - z[7]) + (z[6] - z[8]));
    L.ux = (jx + C(0.5) * L.fsx) * ir;
    L.uy = (jy + C(0.5) * L.fsy) * ir;
    L.uu = L.ux * L.ux + L.uy * L.uy;
    L.ug = L.ux * Gx + L.uy * Gy;
    const C zs = ((z[1] + z[3]) + (z[2] + z[4])) + ((z[5] + z[7]) + (z[6] + z[8]));
    // p / c_s^2, Eq. p_Liang: c_s^2/(1 - w_0) [sum_{i>0} z_i + dt/2 u.grad rho + rho s_0(u)]
    L.ph = C(1.8) * (zs + C(1.5) * drl * L.ug - C(1.5) * wgt<C>(0) * rho * L.uu);
    L.phi = phi;
    L.Gx = Gx;
    L.Gy = Gy;
    L.rho = rho;
    L.drl = drl;
    L.mu = mu;
    return L;
}

// The collision of one node.  In: its stored h_i (with the low part of h_0
// for FP32 storage), z_i, (phi u) of the previous step and its PhaseLocal.
// Out: post-collision h_i* (i > 0, in hs), h_0* as a hi/lo pair, z_i*, and
// the node's (phi u).
template <typename S, typename C, typename K>
__device__ __forceinline__ void phase_collide(const K& k, const PhaseLocal<C>& L,
                                              const C (&h)[9], C hlo, const C (&z)[9], C pu0,
                                              C pu1, C (&hs)[9], S& h0hi, S& h0lo, C (&zst)[9],
                                              C& pux, C& puy) {
    constexpr bool RMASS = std::is_same<S, float>::value;
    const C phi = L.phi, ux = L.ux, uy = L.uy;
    // ---- interface populations (Eq. eq_lattice_boltzmann_interface,
    //      source_term_interface, heq_liang); d(phi u)/dt by explicit Euler
    pux = phi * ux;
    puy = phi * uy;
    const C dpx = pux - pu0, dpy = puy - pu1;
    const C wphi = C(k.w_phi);
    const C sfac = C(1) - C(0.5) * wphi;
    const C sharp = C(4) * phi * (C(1) - phi) * C(k.dxW);
    // h_i* = h_i - w (h_i - h_i^eq) + S_i with h_i^eq = phi w_i (1 + 3 e_i.u) and
    // S_i = (1 - w/2) w_i e_i.(3 d(phi u) + sharp n) collects into
    //   h_i* = h_i + (t_i - w h_i),  t_i = w_i (a + e_i.B),
    //   a = w phi,  B = 3 w phi u + (1 - w/2)(3 d(phi u) + sharp n);
    // t_i - w h_i is the step's small change, taken in one fused multiply-add
    // (one rounding of the change, as the non-equilibrium form has).
    const C a = wphi * phi;
    const C a3 = C(3) * a;
    const C Bx = a3 * ux + sfac * (C(3) * dpx + sharp * L.nxv);
    const C By = a3 * uy + sfac * (C(3) * dpy + sharp * L.nyv);
    const C qa = C(1.0 / 9.0) * a, qx = C(1.0 / 9.0) * Bx, qy = C(1.0 / 9.0) * By;
    const C da = C(1.0 / 36.0) * a, ds = C(1.0 / 36.0) * (Bx + By), dd = C(1.0 / 36.0) * (Bx - By);
    const C t[9] = {C(4.0 / 9.0) * a, qa + qx, qa + qy, qa - qx, qa - qy,  // 0, (+1,0) (0,+1) (-1,0) (0,-1)
                    da + ds, da - dd, da - ds, da + dd};                   // (+1,+1) (-1,+1) (-1,-1) (+1,-1)
    hs[0] = C(0);
#pragma unroll
    for (int i = 1; i < 9; ++i) hs[i] = h[i] + (t[i] - wphi * h[i]);
    h0lo = S(0);
    if constexpr (RMASS) {
        // rest population takes the node's exact balance: h0* = phi - sum_{i>0} h_i*
        // with the stored (rounded) h_i*.  The FP32 terms are summed in FP64
        // (each exact there; 18 terms lose at most ~2^-49 of the largest) and
        // the sum is kept as an FP32 hi/lo pair.
        double acc = double(h[0]) + double(hlo);
#pragma unroll
        for (int i = 1; i < 9; ++i) acc += double(h[i]);
#pragma unroll
        for (int i = 1; i < 9; ++i) acc -= double(float(hs[i]));
        h0hi = float(acc);
        h0lo = float(acc - double(h0hi));
    } else {
        h0hi = S(h[0] + (t[0] - wphi * h[0]));  // h_0^eq = (4/9) phi, no source
    }
    // ---- pressure collision in moment space.  The moments of z_i^eq
    //      (Eq. zeq_liang with Eq. s_i_Liang) and of dt F^z_i (Eq.
    //      forcing_term_pressure_evolution) under the integer matrix of
    //      Eq. M_matrix, in closed form:
    //        m^eq = (0, 2 p~ + 3 rho u^2, -3 (p~ + rho u^2), rho u_x, -rho u_x,
    //                rho u_y, -rho u_y, rho (u_x^2 - u_y^2), rho u_x u_y)
    //        m^F  = (3 D, 0, -3 D, F_x, -F_x, F_y, -F_y,
    //                2 drho (G_x u_x - G_y u_y), drho (G_x u_y + G_y u_x))
    //      with p~ = p / c_s^2, D = drho (u . G) and every velocity in units
    //      of c.  BGK is the same update with every rate equal to dt/tau.
    const C rho = L.rho, drl = L.drl, wn = L.wn, Gx = L.Gx, Gy = L.Gy;
    const C ruu = rho * L.uu, D = drl * L.ug;
    const C meq[9] = {C(0), C(2) * L.ph + C(3) * ruu, C(-3) * (L.ph + ruu), rho * ux, -rho * ux,
                      rho * uy, -rho * uy, rho * (ux * ux - uy * uy), rho * ux * uy};
    const C mf[9] = {C(3) * D, C(0), C(-3) * D, L.fsx, -L.fsx, L.fsy, -L.fsy,
                     C(2) * drl * (Gx * ux - Gy * uy), drl * (Gx * uy + Gy * ux)};
    C m[9];
    if (k.z_mrt) {
        // Sec. 3 rates: rho, e, eps, j_x, j_y relax at 1/dt, which leaves
        // m* = m^eq + m^F / 2 whatever the incoming moment; q_x and q_y relax at
        // w_q (q_y at 1/dt in the printed variant), the stresses at w_nu.  Only
        // the moments of those four rows are taken from z.
        const C x13 = z[1] - z[3], y24 = z[2] - z[4];
        const C x58 = (z[5] - z[7]) + (z[8] - z[6]);
        const C y58 = (z[5] - z[7]) + (z[6] - z[8]);
        const C wq = C(3) * (C(2) - wn) * rcp(C(3) - wn);
        const C wqy = k.qy_printed ? C(1) : wq;
        const C mq[4] = {C(-2) * x13 + x58, C(-2) * y24 + y58, (z[1] + z[3]) - (z[2] + z[4]),
                         (z[5] + z[7]) - (z[6] + z[8])};
        const C Lq[4] = {wq, wqy, wn, wn};
        const int row[4] = {4, 6, 7, 8};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int q = row[j];
            m[q] = mq[j] - Lq[j] * (mq[j] - meq[q]) + (C(1) - C(0.5) * Lq[j]) * mf[q];
        }
        m[0] = meq[0] + C(0.5) * mf[0];
        m[1] = meq[1];  // m^F has no e component
        m[2] = meq[2] + C(0.5) * mf[2];
        m[3] = meq[3] + C(0.5) * mf[3];
        m[5] = meq[5] + C(0.5) * mf[5];
    } else {
        // BGK: every row at dt / tau
        moments9(z, m);
#pragma unroll
        for (int q = 0; q < 9; ++q) m[q] += -wn * (m[q] - meq[q]) + (C(1) - C(0.5) * wn) * mf[q];
    }
    inverse9(m, zst);
}

}  // namespace
}  // namespace lbm
