// 3D two-phase step of liblbm for gfx950: the conservative Allen-Cahn h_i and
// the pressure-evolution z_i of Sec. 2.3 on D3Q19, z_i with the dimensional
// MRT of Sec. 3 in the d'Humieres basis, h_i BGK with its source.
//
// One step is one launch of k_p3_march, which sums phi of the planes ahead as it
// marches up z, or two:
//   k_p3_phi   phi = sum_i h_i of the stored state into one plane (Eq.
//              zero_moment_h), so that no node has to re-read the 19 h_i of
//              its 18 neighbours;
//   k_p3_step  tiles of 64 x 4 x 1 nodes (FP32) or 64 x 2 x 2 (FP64); phi of
//              the tile and a one-node halo in LDS for the isotropic
//              stencils, then the node's collision in registers and push
//              streaming.
// All evaluate p3_local and p3_collide per node and agree to the last bit.
// Layout: node blocks (bidx, NPL3 values per node) with h 0-18, z 19-37, the
// low part of h_0 at 38 (FP32 storage: the rest population is an FP32 hi/lo
// pair that carries the node's exact phi balance, as in 2D), then (phi u) of
// the previous step (3 values); phi is one plain array of nodes.
// Arithmetic is lattice-normalised as in the 2D kernels: velocities / c,
// forces F dt^2 / dx, z_i in units of p / c_s^2, rates Lambda dt.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "lbm_d3q19.h"
#include "lbm_device.h"

namespace lbm {
namespace {

// values per node of the 3D two-phase state: 42 in FP32 storage, 41 in FP64
template <typename S>
constexpr int NPL3 = std::is_same<S, float>::value ? 42 : 41;
template <typename S>
__device__ __forceinline__ long long p3idx(int i, long long n) {
    return bidx(NPL3<S>, i, n);
}

// Step tiles, measured on the 256^3 bubble box (ms per step, FP32 / FP64):
// 64 x 4 x 2 1.507 / 2.936, 64 x 2 x 2 1.498 / 2.806, 64 x 4 x 1 1.473 /
// 2.849, 64 x 2 x 4 1.514 / 2.912, 64 x 1 x 4 1.504 / 2.811, 64 x 8 x 1
// 1.568, 1024-thread tiles 1.58-1.62 / 3.59.  The states do not depend on
// the tiling.
template <typename S>
struct P3Tile {
    static constexpr int X = 64, Y = std::is_same<S, float>::value ? 4 : 2,
                         Z = std::is_same<S, float>::value ? 1 : 2;
    static constexpr int HX = X + 2, HY = Y + 2, HZ = Z + 2;
    static constexpr int Halo = HX * HY * HZ;  // phi values in LDS
    static constexpr int Threads = X * Y * Z;
};

__device__ __forceinline__ float rcp3(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double rcp3(double x) { return 1.0 / x; }
__device__ __forceinline__ float rsq3(float x) { return __builtin_amdgcn_rsqf(x); }
__device__ __forceinline__ double rsq3(double x) { return 1.0 / sqrt(x); }

// phi of a node from its h_i (with the low part of h_0): one summation order
// everywhere
template <typename C>
__device__ __forceinline__ C phi_sum19(const C (&h)[19], C hlo) {
    const C ax = (h[1] + h[2]) + ((h[3] + h[4]) + (h[5] + h[6]));
    const C dg = ((h[7] + h[8]) + (h[9] + h[10])) + ((h[11] + h[12]) + (h[13] + h[14])) +
                 ((h[15] + h[16]) + (h[17] + h[18]));
    return (h[0] + hlo) + (ax + dg);
}

// index of a halo coordinate: periodic wrap, or at a wall the first fluid
// node (zero normal gradient of phi, as in 2D).  Halo coordinates of a ragged
// last tile can lie far beyond n (they feed no node but are still loaded),
// hence the full modulo.
__device__ __forceinline__ int ghost(int v, int n, int walls) {
    if (walls) return v < 0 ? 0 : (v >= n ? n - 1 : v);
    return ((v % n) + n) % n;
}

template <typename S>
__global__ __launch_bounds__(256) void k_p3_phi(P3K k, const S* __restrict__ a,
                                                S* __restrict__ phi) {
    constexpr bool RMASS = std::is_same<S, float>::value;
    const long long N = (long long)k.batch * k.nx * k.ny * k.nz;
    for (long long n = blockIdx.x * (long long)blockDim.x + threadIdx.x; n < N;
         n += (long long)gridDim.x * blockDim.x) {
        S h[19];
#pragma unroll
        for (int i = 0; i < 19; ++i) h[i] = a[p3idx<S>(i, n)];
        phi[n] = phi_sum19<S>(h, RMASS ? a[p3idx<S>(38, n)] : S(0));
    }
}

// What one node derives once phi of itself and its 18 neighbours is known
// (pn[i] = phi at x + e_i): stencils and macros.
template <typename C>
struct P3Local {
    C phi, drl, rho, wn, mu, G[3], F[3], nv[3], u[3], uu, ug, ph, m[19];
};

template <typename C, typename K>
__device__ __forceinline__ P3Local<C> p3_local(const K& k, const C (&pn)[19], const C (&zz)[19]) {
    P3Local<C> L;
    C(&G)[3] = L.G;
    C(&F)[3] = L.F;
    C(&nv)[3] = L.nv;
    C(&u)[3] = L.u;
    C(&m)[19] = L.m;
    // ---- stencils (Eq. gradient, Eq. laplacian): grad phi = 3 G / dx,
    //      lap phi = 6 L / dx^2
    const C phi = pn[0];
    C Lp = C(0);
    G[0] = G[1] = G[2] = C(0);
#pragma unroll
    for (int i = 1; i < 19; ++i) {
        const C wp = w19<C>(i) * pn[i];
        G[0] += C(E3X[i]) * wp;
        G[1] += C(E3Y[i]) * wp;
        G[2] += C(E3Z[i]) * wp;
        Lp += w19<C>(i) * (pn[i] - phi);
    }
    const C drl = C(k.drho());
    const C rho = C(k.rho_g) + phi * drl;
    const C ir = rcp3(rho);
    C wn;
    if (k.visc_mode == 0) {
        wn = rcp3(C(3) * (C(k.nuh_g) + phi * C(k.dnuh())) + C(0.5));
    } else {
        const C zh = C(k.zh_g) + phi * C(k.dzh());
        wn = rho * rcp3(C(3) * zh + C(0.5) * rho);
    }
    // chemical potential (Eq. chemical_potential), force mu grad phi + F_b
    const C mu = C(4) * C(k.beta) * phi * (phi - C(1)) * (phi - C(0.5)) - C(k.kap6) * Lp;
#pragma unroll
    for (int c = 0; c < 3; ++c) F[c] = mu * G[c] * C(k.fs_scale) + C(k.Fbt[c]);
    // guarded interface normal
    const C gn2 = (G[0] * G[0] + G[1] * G[1]) + G[2] * G[2];
    nv[0] = nv[1] = nv[2] = C(0);
    if (gn2 > C(k.Geps) * C(k.Geps)) {
        const C ig = rsq3(gn2);
#pragma unroll
        for (int c = 0; c < 3; ++c) nv[c] = G[c] * ig;
    }
    // velocity first (Eq. u_Liang), then pressure (Eq. p_Liang) with w_0 = 1/3:
    // p / c_s^2 = 3/2 [sum_{i>0} z_i + 3/2 drho u.G - rho u^2 / 2]
    moments19(zz, m);
    u[0] = (m[3] + C(0.5) * F[0]) * ir;
    u[1] = (m[5] + C(0.5) * F[1]) * ir;
    u[2] = (m[7] + C(0.5) * F[2]) * ir;
    const C uu = (u[0] * u[0] + u[1] * u[1]) + u[2] * u[2];
    const C ug = (u[0] * G[0] + u[1] * G[1]) + u[2] * G[2];
    const C zsum = ((zz[1] + zz[2]) + ((zz[3] + zz[4]) + (zz[5] + zz[6]))) +
                   (((zz[7] + zz[8]) + (zz[9] + zz[10])) + ((zz[11] + zz[12]) + (zz[13] + zz[14])) +
                    ((zz[15] + zz[16]) + (zz[17] + zz[18])));
    const C ph = C(1.5) * (zsum + C(1.5) * drl * ug - C(0.5) * rho * uu);
    L.phi = phi;
    L.drl = drl;
    L.rho = rho;
    L.wn = wn;
    L.mu = mu;
    L.uu = uu;
    L.ug = ug;
    L.ph = ph;
    return L;
}

// The collisions of one node: post-collision h_i* (i > 0, in hs), h_0* as a
// hi/lo pair, z_i* (zs) and the node's (phi u).  Shared by all step kernels, so
// that they agree to the last bit.
template <typename S, typename K>
__device__ __forceinline__ void p3_collide(const K& k, P3Local<S>& L, const S (&h)[19], S hlo,
                                           const S (&pu)[3], S (&hs)[19], S& h0hi, S& h0lo,
                                           S (&zs)[19], S (&pn3)[3]) {
    using C = S;
    constexpr bool RMASS = std::is_same<S, float>::value;
    const C phi = L.phi, drl = L.drl, rho = L.rho, wn = L.wn, uu = L.uu, ug = L.ug, ph = L.ph;
    const C(&G)[3] = L.G;
    const C(&F)[3] = L.F;
    const C(&nv)[3] = L.nv;
    const C(&u)[3] = L.u;
    C(&m)[19] = L.m;
    // ---- interface populations (Eq. eq_lattice_boltzmann_interface,
    //      source_term_interface, heq_liang); d(phi u)/dt by explicit Euler
    C dp[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        pn3[c] = phi * u[c];
        dp[c] = pn3[c] - pu[c];
    }
    const C wphi = C(k.w_phi);
    const C sfac = C(1) - C(0.5) * wphi;
    const C sharp = C(4) * phi * (C(1) - phi) * C(k.dxW);
    const C A[3] = {C(3) * dp[0] + sharp * nv[0], C(3) * dp[1] + sharp * nv[1],
                    C(3) * dp[2] + sharp * nv[2]};
#pragma unroll
    for (int i = 1; i < 19; ++i) {
        const C eu = (C(E3X[i]) * u[0] + C(E3Y[i]) * u[1]) + C(E3Z[i]) * u[2];
        const C eA = (C(E3X[i]) * A[0] + C(E3Y[i]) * A[1]) + C(E3Z[i]) * A[2];
        const C heq = phi * w19<C>(i) * (C(1) + C(3) * eu);
        hs[i] = h[i] - wphi * (h[i] - heq) + sfac * w19<C>(i) * eA;
    }
    h0lo = S(0);
    if constexpr (RMASS) {
        // rest population: the node's exact balance phi - sum_{i>0} h_i* with
        // the stored (rounded) h_i*, summed in FP64, kept as an FP32 pair
        double acc = double(h[0]) + double(hlo);
#pragma unroll
        for (int i = 1; i < 19; ++i) acc += double(h[i]);
#pragma unroll
        for (int i = 1; i < 19; ++i) acc -= double(float(hs[i]));
        h0hi = float(acc);
        h0lo = float(acc - double(h0hi));
    } else {
        h0hi = S(h[0] - wphi * (h[0] - phi * w19<C>(0)));
    }
    // ---- pressure collision in moment space.  Moments of z^eq (Eq.
    //      zeq_liang) and of dt F^z (Eq. forcing_term_pressure_evolution)
    //      in the D3Q19 basis, with p~ = p / c_s^2, D_ab = drho u_a G_b:
    //        m^eq = (0, 19 p~ + 19 rho u^2, -9 p~ - 11/2 rho u^2, rho u, -2/3 rho u,
    //                rho (2ux^2 - uy^2 - uz^2), -1/2 (.), rho (uy^2 - uz^2), -1/2 (.),
    //                rho ux uy, rho uy uz, rho ux uz, 0, 0, 0)
    //        m^F  = (3 D, 5 D, -2 D, F, -2/3 F, 2 (2Dxx - Dyy - Dzz), -(.),
    //                2 (Dyy - Dzz), -(.), Dxy + Dyx, Dyz + Dzy, Dxz + Dzx, 0, 0, 0)
    //      (j and q interleaved per axis as in the basis order).
    const C ruu = rho * uu;
    const C Dt = drl * ug;
    const C Dxx = drl * u[0] * G[0], Dyy = drl * u[1] * G[1], Dzz = drl * u[2] * G[2];
    const C pxx = rho * (C(2) * u[0] * u[0] - (u[1] * u[1] + u[2] * u[2]));
    const C pww = rho * (u[1] * u[1] - u[2] * u[2]);
    const C fxx = C(2) * Dxx - (Dyy + Dzz), fww = Dyy - Dzz;
    const C c23 = C(2) / C(3);
    const C meq[19] = {C(0), C(19) * (ph + ruu), C(-9) * ph - C(5.5) * ruu,
                       rho * u[0], -c23 * rho * u[0], rho * u[1], -c23 * rho * u[1],
                       rho * u[2], -c23 * rho * u[2], pxx, C(-0.5) * pxx, pww, C(-0.5) * pww,
                       rho * u[0] * u[1], rho * u[1] * u[2], rho * u[0] * u[2],
                       C(0), C(0), C(0)};
    const C mf[19] = {C(3) * Dt, C(5) * Dt, C(-2) * Dt, F[0], -c23 * F[0], F[1], -c23 * F[1],
                      F[2], -c23 * F[2], C(2) * fxx, -fxx, C(2) * fww, -fww,
                      drl * (u[0] * G[1] + u[1] * G[0]), drl * (u[1] * G[2] + u[2] * G[1]),
                      drl * (u[0] * G[2] + u[2] * G[0]), C(0), C(0), C(0)};
    // rates (times dt): 1 on rho, e, eps, j, pi; w_q2 on q and m; dt/tau on
    // the stresses (Sec. 3's two-phase choice row by row); BGK: all dt/tau
    const C wq = C(3) * (C(2) - wn) * rcp3(C(3) - wn);
#pragma unroll
    for (int q = 0; q < 19; ++q) {
        const bool stress = q == 9 || q == 11 || q == 13 || q == 14 || q == 15;
        const bool odd3 = q == 4 || q == 6 || q == 8 || q >= 16;
        const C Lq = !k.z_mrt ? wn : (stress ? wn : (odd3 ? wq : C(1)));
        m[q] += -Lq * (m[q] - meq[q]) + (C(1) - C(0.5) * Lq) * mf[q];
    }
    inverse19(m, zs);
}

// One node of the one-step kernel: its collision and push into b, or, with
// MACROS, its macroscopic fields into mout.
template <typename S, bool MACROS>
__device__ __forceinline__ void p3_node(const P3K& k, const S (&pn)[19], const S (&h)[19], S hlo,
                                        const S (&zz)[19], const S (&pu)[3], long long n, int x,
                                        int y, int z, long long base, S* __restrict__ b,
                                        const MacroOut& mout) {
    constexpr bool RMASS = std::is_same<S, float>::value;
    constexpr int PU = RMASS ? 39 : 38;  // first (phi u) plane
    const int nx = k.nx, ny = k.ny, nz = k.nz;
    const long long plane = (long long)nx * ny;
    P3Local<S> L = p3_local<S>(k, pn, zz);
    if constexpr (MACROS) {
        mout.put(0, n, double(L.rho));
        mout.put(1, n, double(L.ph) * k.cs2);
        mout.put(2, n, double(L.u[0]) * k.c);
        mout.put(3, n, double(L.u[1]) * k.c);
        mout.put(5, n, double(L.phi));
        mout.put(6, n, double(L.mu));
        mout.put(7, n, double(L.u[2]) * k.c);
        return;
    } else {
        S hs[19], zs[19], pn3[3], h0hi, h0lo;
        p3_collide<S>(k, L, h, hlo, pu, hs, h0hi, h0lo, zs, pn3);
        // ---- stores: (phi u), the rest populations, then push streaming with
        //      halfway bounce-back on walled axes
#pragma unroll
        for (int c = 0; c < 3; ++c) st(b + p3idx<S>(PU + c, n), S(pn3[c]));
        st(b + p3idx<S>(0, n), h0hi);
        if constexpr (RMASS) st(b + p3idx<S>(38, n), h0lo);
        st(b + p3idx<S>(19, n), S(zs[0]));
#pragma unroll
        for (int i = 1; i < 19; ++i) {
            const int txd = x + E3X[i], tyd = y + E3Y[i], tzd = z + E3Z[i];
            const bool out = (k.bcx && (txd < 0 || txd >= nx)) || (k.bcy && (tyd < 0 || tyd >= ny)) ||
                             (k.bcz && (tzd < 0 || tzd >= nz));
            if (out) {
                st(b + p3idx<S>(OPP3[i], n), S(hs[i]));
                st(b + p3idx<S>(19 + OPP3[i], n), S(zs[i]));
            } else {
                const long long d = base + (long long)wrap(tzd, nz) * plane +
                                    (long long)wrap(tyd, ny) * nx + wrap(txd, nx);
                st(b + p3idx<S>(i, d), S(hs[i]));
                st(b + p3idx<S>(19 + i, d), S(zs[i]));
            }
        }
    }
}

// One step (or, with MACROS, the macroscopic fields of the stored state).
template <typename S, bool MACROS>
__global__ __launch_bounds__(P3Tile<S>::Threads) void k_p3_step(P3K k, const S* __restrict__ a,
                                                        S* __restrict__ b,
                                                        const S* __restrict__ phig,
                                                        MacroOut mout) {
    using C = S;
    constexpr bool RMASS = std::is_same<S, float>::value;
    constexpr int PU = RMASS ? 39 : 38;  // first (phi u) plane
    using T = P3Tile<S>;
    constexpr int kPX = T::X, kPY = T::Y, kPZ = T::Z, kHX = T::HX, kHY = T::HY;
    __shared__ C sphi[T::HZ][T::HY][T::HX];
    const int nx = k.nx, ny = k.ny, nz = k.nz;
    const int gx = (nx + kPX - 1) / kPX, gy = (ny + kPY - 1) / kPY, gz = (nz + kPZ - 1) / kPZ;
    int tile;
    if (!xcd_tile(gx * gy * gz * k.batch, tile)) return;  // whole workgroup, before the barrier
    const int per = gx * gy * gz;
    const int bb = tile / per, r = tile - bb * per;
    const int x0 = (r % gx) * kPX, y0 = ((r / gx) % gy) * kPY, z0 = (r / (gx * gy)) * kPZ;
    const long long plane = (long long)nx * ny;
    const long long base = (long long)bb * nz * plane;
    const int tx = threadIdx.x, ty = threadIdx.y, tz = threadIdx.z;
    const int x = x0 + tx, y = y0 + ty, z = z0 + tz;
    const bool valid = x < nx && y < ny && z < nz;
    const long long n = base + (long long)z * plane + (long long)y * nx + x;

    // the node's own populations first, then the phi halo, then one barrier
    C h[19], zz[19], hlo = C(0), pu[3] = {C(0), C(0), C(0)};
    if (valid) {
#pragma unroll
        for (int i = 0; i < 19; ++i) h[i] = C(a[p3idx<S>(i, n)]);
#pragma unroll
        for (int i = 0; i < 19; ++i) zz[i] = C(a[p3idx<S>(19 + i, n)]);
        if (RMASS) hlo = C(a[p3idx<S>(38, n)]);
        if constexpr (!MACROS) {
#pragma unroll
            for (int c = 0; c < 3; ++c) pu[c] = C(a[p3idx<S>(PU + c, n)]);
        }
    }
    const int t = (tz * kPY + ty) * kPX + tx;
    for (int j = t; j < T::Halo; j += T::Threads) {
        const int hx = j % kHX, hy = (j / kHX) % kHY, hz = j / (kHX * kHY);
        const int gxx = ghost(x0 + hx - 1, nx, k.bcx);
        const int gyy = ghost(y0 + hy - 1, ny, k.bcy);
        const int gzz = ghost(z0 + hz - 1, nz, k.bcz);
        sphi[hz][hy][hx] = C(phig[base + (long long)gzz * plane + (long long)gyy * nx + gxx]);
    }
    __syncthreads();
    if (!valid) return;
    C pn[19];
#pragma unroll
    for (int i = 0; i < 19; ++i) pn[i] = sphi[tz + 1 + E3Z[i]][ty + 1 + E3Y[i]][tx + 1 + E3X[i]];
    p3_node<S, MACROS>(k, pn, h, hlo, zz, pu, n, x, y, z, base, b, mout);
}

// ---------------------------------------------------------------------------
// The step without the phi pass: a workgroup takes a column of w x h nodes with
// one node of overlap (one per thread, at most NT) and marches up the planes of
// one segment [a, e).  phi of plane v + 1 is summed from the h_i of the column
// and its overlap as they arrive, into an LDS ring of four planes; the column's
// own h_i stay in registers until plane v + 1 takes its step, so that they cross
// HBM once (the phi pass reads them a second time: 84 of 420 bytes per update).
// Threads as in the two-step D3Q19 kernel: the tile's columns row by row, so
// that a wave of a 64-wide row is one node block, then the columns beside it;
// ALIGNED: an access is the plane's block base plus a 32-bit lane offset.
// ---------------------------------------------------------------------------
template <typename C>
struct P3KT {  // P3K in the type the kernel computes in
    int nx, ny, nz, batch, bcx, bcy, bcz, z_mrt, visc_mode;
    C rho_g, drl, nuh_g, dnu, zh_g, dz, w_phi, beta, kap6, fs_scale, Fbt[3], dxW, Geps;
    __device__ __forceinline__ C drho() const { return drl; }
    __device__ __forceinline__ C dnuh() const { return dnu; }
    __device__ __forceinline__ C dzh() const { return dz; }
};
template <typename C>
struct P3MarchArgs {
    P3KT<C> k;
    int ntx, nty, nseg;          // tiles per plane and segments per replica
    int wx, ex, wy, ey, wz, ez;  // tile i spans w nodes, one more for i < e
};

template <typename S, int NT, int NC, bool ALIGNED>
__global__ __launch_bounds__(NT) void k_p3_march(const P3MarchArgs<S> p, const S* __restrict__ A,
                                                 S* __restrict__ B) {
    using C = S;
    constexpr bool RMASS = std::is_same<S, float>::value;
    constexpr int NPL = NPL3<S>, PU = RMASS ? 39 : 38;
    constexpr int NH = RMASS ? 20 : 19;
    __shared__ C sphi[4][NT];
    __shared__ C hb[2][NH][NC];
    const auto& k = p.k;
    const int nx = k.nx, ny = k.ny, nz = k.nz;
    int w, tx, ty, sg, b;
    if (!xcd_tile(p.ntx * p.nty * p.nseg * k.batch, w)) return;  // whole workgroup
    block_divide(w, p.ntx, w, tx);
    block_divide(w, p.nty, w, ty);
    block_divide(w, p.nseg, b, sg);
    const int x0 = tx * p.wx + min(tx, p.ex), x1 = x0 + p.wx + (tx < p.ex);
    const int y0 = ty * p.wy + min(ty, p.ey), y1 = y0 + p.wy + (ty < p.ey);
    const int a = sg * p.wz + min(sg, p.ez), e = a + p.wz + (sg < p.ez);
    const int wc = x1 - x0, rh = y1 - y0 + 2;
    const bool whole = p.ntx == 1;  // rows wrap in LDS
    const int th = threadIdx.x;
    int rx, ry;
    block_divide(th, wc, ry, rx);
    bool in = ry < rh;
    if (!in && !whole) {
        const int q = th - rh * wc;
        ry = q >> 1;
        rx = q & 1 ? wc : -1;
        in = ry < rh;
    }
    const int rw = whole ? wc : wc + 2;  // LDS row
    const bool own = in && rx >= 0 && rx < wc && ry > 0 && ry < rh - 1;
    const int t = in ? ry * rw + rx + (whole ? 0 : 1) : 0;  // LDS position
    // the lane's column: wrapped, or clamped where a wall ends the axis
    const int vx = x0 + rx, vy = y0 - 1 + (in ? ry : 0);
    const int x = vx < 0 ? (k.bcx ? 0 : nx - 1) : vx >= nx ? (k.bcx ? nx - 1 : 0) : vx;
    const int y = vy < 0 ? (k.bcy ? 0 : ny - 1) : vy >= ny ? (k.bcy ? ny - 1 : 0) : vy;
    const bool xlo = k.bcx && x == 0, xhi = k.bcx && x == nx - 1;
    const bool ylo = k.bcy && y == 0, yhi = k.bcy && y == ny - 1;
    const bool plain = !__any(xlo || xhi || ylo || yhi);
    // LDS offsets to the neighbours (0 across a wall: the first fluid node's phi)
    const int om = rx > (whole ? 0 : -1) && !xlo ? -1 : whole && !xlo ? wc - 1 : 0;
    const int op = rx < (whole ? wc - 1 : wc) && !xhi ? 1 : whole && !xhi ? 1 - wc : 0;
    const int od = in && ry > 0 && !ylo ? -rw : 0, ou = ry < rh - 1 && !yhi ? rw : 0;
    const int plane = nx * ny;
    const long long base = (long long)b * nz * plane;
    auto zof = [&](int v) { return v < 0 ? v + nz : (v >= nz ? v - nz : v); };

    // columns of the push: x - 1, x, x + 1 in rows y - 1, y, y + 1 (wrapped)
    unsigned col[9];
#pragma unroll
    for (int c = 0; c < 9; ++c) {
        const int q = wrap(y + c / 3 - 1, ny) * nx + wrap(x + c % 3 - 1, nx);
        col[c] = ALIGNED ? unsigned(((q >> 6) * NPL * kBlk + (q & (kBlk - 1))) * int(sizeof(S)))
                         : unsigned(q);
    }
    auto at = [&](auto* P, int z, int c, int i) {
        const long long po = base + (long long)z * plane;
        if constexpr (ALIGNED) {
            using B8 = std::conditional_t<std::is_const_v<std::remove_pointer_t<decltype(P)>>,
                                          const char, char>;
            auto* row = (B8*)P + (po >> 6) * (long long)(NPL * kBlk * sizeof(S));
            return (decltype(P))(row + col[c]) + i * kBlk;
        } else {
            return P + bidx(NPL, i, po + col[c]);
        }
    };
    auto outxy = [&](int i) {  // whether population i leaves through an x or y wall
        return (E3X[i] < 0 ? xlo : E3X[i] > 0 ? xhi : false) ||
               (E3Y[i] < 0 ? ylo : E3Y[i] > 0 ? yhi : false);
    };
    const int own_at = own ? (ry - 1) * wc + rx : 0;  // place in hb
    C Hn[19], Z[19], pu[3], hnlo = C(0);
    auto load_h = [&](int z) {
#pragma unroll
        for (int i = 0; i < 19; ++i) Hn[i] = C(*at(A, z, 4, i));
        hnlo = RMASS ? C(*at(A, z, 4, 38)) : C(0);
    };
    auto load_z = [&](int z) {
#pragma unroll
        for (int i = 0; i < 19; ++i) Z[i] = C(*at(A, z, 4, 19 + i));
    };
    auto load_pu = [&](int z, C (&q)[3]) {
#pragma unroll
        for (int c = 0; c < 3; ++c) q[c] = C(*at(A, z, 4, PU + c));
    };
    // phi of plane v from the loaded h, which the tile's own lanes keep
    auto take_h = [&](int v) {
        if (in) sphi[v & 3][t] = phi_sum19<C>(Hn, hnlo);
        if (own) {
#pragma unroll
            for (int i = 0; i < 19; ++i) hb[v & 1][i][own_at] = Hn[i];
            if constexpr (RMASS) hb[v & 1][19][own_at] = hnlo;
        }
    };
    // In FP64 the loads of a plane step end here, on every path and before its stores: a
    // wait for them after the stores, which only some lanes make, would wait for those
    // too, and without it the kernel spilled (108 B; 128^3 299 -> 270 us, 64^3 41 -> 36).
    // FP32 gains nothing by it (192^3 496 us either way).
    auto landed = [&] {
        if constexpr (!RMASS) {
#pragma unroll
            for (int i = 0; i < 19; ++i) asm volatile("" : "+v"(Hn[i]), "+v"(Z[i]));
        }
    };
    auto above = [&](int v) { return k.bcz && v + 1 >= nz ? v : zof(v + 1); };
    if (!(k.bcz && a == 0)) {
        load_h(zof(a - 1));
        take_h(a - 1);
    }
    load_h(a);
    load_z(a);
    load_pu(a, pu);
    take_h(a);
    load_h(above(a));

    for (int v = a; v < e; ++v) {
        const bool zlo = k.bcz && v == 0, zhi = k.bcz && v == nz - 1;
        if (!zhi) take_h(v + 1);
        const int vn = min(v + 1, e - 1);  // the last step re-reads an existing plane
        load_h(above(vn));
        __syncthreads();  // the ring's fourth plane was last read a barrier ago
        if (own) {
            P3Local<C> L;
            {
                C pn[19];
#pragma unroll
                for (int i = 0; i < 19; ++i) {
                    const int pl = E3Z[i] < 0 ? (zlo ? v : v - 1) : E3Z[i] > 0 ? (zhi ? v : v + 1) : v;
                    pn[i] = sphi[pl & 3][t + (E3X[i] < 0 ? om : E3X[i] > 0 ? op : 0) +
                                         (E3Y[i] < 0 ? od : E3Y[i] > 0 ? ou : 0)];
                }
                L = p3_local<C>(k, pn, Z);
            }
            C nextpu[3];
            load_z(vn);
            load_pu(vn, nextpu);
            C H[19], hs[19], zs[19], pn3[3];
            S h0hi, h0lo;
#pragma unroll
            for (int i = 0; i < 19; ++i) H[i] = hb[v & 1][i][own_at];
            p3_collide<S>(k, L, H, RMASS ? hb[v & 1][NH - 1][own_at] : C(0), pu, hs, h0hi, h0lo, zs, pn3);
            landed();
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                if constexpr (!RMASS) asm volatile("" : "+v"(nextpu[c]));
                pu[c] = nextpu[c];
            }
            const int zm = zof(v - 1), zp = zof(v + 1);
#pragma unroll
            for (int c = 0; c < 3; ++c) st(at(B, v, 4, PU + c), S(pn3[c]));
            st(at(B, v, 4, 0), h0hi);
            if constexpr (RMASS) st(at(B, v, 4, 38), h0lo);
            st(at(B, v, 4, 19), S(zs[0]));
            if (plain && !zlo && !zhi) {
#pragma unroll
                for (int i = 1; i < 19; ++i) {
                    const int z = E3Z[i] > 0 ? zp : E3Z[i] < 0 ? zm : v, c = 4 + E3X[i] + 3 * E3Y[i];
                    st(at(B, z, c, i), S(hs[i]));
                    st(at(B, z, c, 19 + i), S(zs[i]));
                }
            } else {
#pragma unroll
                for (int i = 1; i < 19; ++i) {
                    const bool outz = E3Z[i] > 0 ? zhi : E3Z[i] < 0 ? zlo : false;
                    if (outz || outxy(i)) {
                        st(at(B, v, 4, OPP3[i]), S(hs[i]));
                        st(at(B, v, 4, 19 + OPP3[i]), S(zs[i]));
                    } else {
                        const int z = E3Z[i] > 0 ? zp : E3Z[i] < 0 ? zm : v, c = 4 + E3X[i] + 3 * E3Y[i];
                        st(at(B, z, c, i), S(hs[i]));
                        st(at(B, z, c, 19 + i), S(zs[i]));
                    }
                }
            }
        } else {
            landed();
        }
    }
}

// equilibria from FP64 fields (staging slots 1 p, 2 ux, 3 uy, 7 uz, 5 phi)
template <typename S>
__global__ void k_p3_init(P3K k, const double* __restrict__ fld, S* __restrict__ a) {
    constexpr bool RMASS = std::is_same<S, float>::value;
    constexpr int PU = RMASS ? 39 : 38;
    const long long N = (long long)k.batch * k.nx * k.ny * k.nz;
    const long long P = k.P;
    for (long long n = blockIdx.x * (long long)blockDim.x + threadIdx.x; n < N;
         n += (long long)gridDim.x * blockDim.x) {
        const double p = fld[P + n], phi = fld[5 * P + n];
        const double u[3] = {fld[2 * P + n] / k.c, fld[3 * P + n] / k.c, fld[7 * P + n] / k.c};
        const double rho = k.rho_g + phi * (k.rho_l - k.rho_g);
        const double ph = p / k.cs2, uu = u[0] * u[0] + u[1] * u[1] + u[2] * u[2];
        double hsum = 0.0;
        for (int i = 1; i < 19; ++i) {
            const double eu = E3X[i] * u[0] + E3Y[i] * u[1] + E3Z[i] * u[2];
            const S hv = S(phi * w19<double>(i) * (1 + 3 * eu));
            a[p3idx<S>(i, n)] = hv;
            hsum += double(hv);
        }
        const double h0 = phi - hsum;  // the rest population closes phi exactly
        const S hi = S(h0);
        a[p3idx<S>(0, n)] = hi;
        if (RMASS) a[p3idx<S>(38, n)] = S(h0 - double(hi));
        for (int i = 0; i < 19; ++i) {
            const double eu = E3X[i] * u[0] + E3Y[i] * u[1] + E3Z[i] * u[2];
            const double w = w19<double>(i);
            a[p3idx<S>(19 + i, n)] =
                S(ph * (i == 0 ? w - 1 : w) + rho * w * (3 * eu + 4.5 * eu * eu - 1.5 * uu));
        }
        for (int c = 0; c < 3; ++c) a[p3idx<S>(PU + c, n)] = S(phi * u[c]);
    }
}

inline unsigned grid_p3(long long N, int bs) {
    long long g = (N + bs - 1) / bs;
    if (g > 65535LL * 16) g = 65535LL * 16;
    return unsigned(g < 1 ? 1 : g);
}

template <typename S>
hipError_t launch_phi(const P3K& k, const S* a, S* phi, hipStream_t s) {
    const long long N = (long long)k.batch * k.nx * k.ny * k.nz;
    hipLaunchKernelGGL(k_p3_phi<S>, dim3(grid_p3(N, 256)), dim3(256), 0, s, k, a, phi);
    return hipGetLastError();
}

template <typename S>
long long p3_tiles(const P3K& k) {
    using T = P3Tile<S>;
    return (long long)((k.nx + T::X - 1) / T::X) * ((k.ny + T::Y - 1) / T::Y) *
           ((k.nz + T::Z - 1) / T::Z) * k.batch;
}

template <typename C>
P3KT<C> p3_kt(const P3K& k) {
    P3KT<C> r{};
    r.nx = k.nx; r.ny = k.ny; r.nz = k.nz; r.batch = k.batch;
    r.bcx = k.bcx; r.bcy = k.bcy; r.bcz = k.bcz;
    r.z_mrt = k.z_mrt; r.visc_mode = k.visc_mode;
    r.rho_g = C(k.rho_g); r.drl = C(k.drho());
    r.nuh_g = C(k.nuh_g); r.dnu = C(k.dnuh());
    r.zh_g = C(k.zh_g); r.dz = C(k.dzh());
    r.w_phi = C(k.w_phi); r.beta = C(k.beta); r.kap6 = C(k.kap6); r.fs_scale = C(k.fs_scale);
    for (int c = 0; c < 3; ++c) r.Fbt[c] = C(k.Fbt[c]);
    r.dxW = C(k.dxW); r.Geps = C(k.Geps);
    return r;
}
template <typename S>
bool p3_aligned(const P3K& k) {
    const long long plane = (long long)k.nx * k.ny;
    return plane % kBlk == 0 && plane * NPL3<S> * (long long)sizeof(S) < (1LL << 31);
}
// Workgroup limits of k_p3_march: threads, and tile nodes whose h it keeps in LDS
// (two planes: 82 KB in FP32, 117 KB in FP64).
template <typename S>
constexpr int p3_max_threads() {
    return sizeof(S) == 4 ? 768 : 512;
}
template <typename S>
constexpr int p3_max_core() {
    return sizeof(S) == 4 ? 512 : 384;
}

}  // namespace

long long p3_march_threads(const P3K& k, const P3MarchPlan& p) {
    return (long long)((k.nx + p.ntx - 1) / p.ntx + (p.ntx > 1 ? 2 : 0)) *
           ((k.ny + p.nty - 1) / p.nty + 2);
}

// Tiles and segments by a cost model fitted to 600 plans on 15 boxes of 0.1 M to
// 7 M nodes (11-15 %; its choice runs within 5 % of the best measured plan on 13
// of them, within 25 % on all).  A plane step takes the cubic mean of
//   l0 + l1 waves   (load, LDS, barrier, collision) and
//   the bytes of all resident workgroups at 12 TB/s, or at 6-7 TB/s where both
//   buffers together outgrow the 256 MB memory-side cache, with lost columns
//   where tiles cut the rows (pad) and more where rows start inside node blocks.
// Measured per step, phi pass + step -> march: FP32 192^3 600 -> 493-515 us
// (4.8 TB/s of 336 B per update), 128^3 179 -> 145, 100 x 120 x 130 162 -> 123,
// 64^3 29 -> 19, 48^3 21.6 -> 13.3; FP64 128^3 356 -> 270 us.  1024-thread
// workgroups (128 registers, 144 B of spills) took 613-740 us on 192^3; keeping
// the next plane's h in registers instead of LDS took 201 registers.
template <typename S>
P3MarchPlan p3_march_plan(const P3K& k) {
    P3MarchPlan best{};
    int dev = 0, cus = 0;
    if (k.nx < 2 || k.ny < 2 || k.nz < 2 || (long long)k.nx * k.ny >= (1LL << 31) ||
        hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        return best;
    constexpr bool F32 = sizeof(S) == 4;
    constexpr int NPL = NPL3<S>;
    const double l0 = F32 ? 2.68 : 2.11, l1 = F32 ? 0.113 : 0.60, pad = F32 ? 22.8 : 12.8;
    const double t0 = F32 ? 0.7 : 3.3;
    const double nodes = double(k.nx) * k.ny * k.nz * k.batch, state = nodes * NPL * sizeof(S);
    const double bw = 2 * state < 3e8 ? 12e6 : F32 ? 7.0e6 : 6.0e6;  // bytes per us
    double least = (12 + nodes * (F32 ? 420 : 816) / 5.0e6) / 1.15;
    P3MarchPlan p{};
    for (p.ntx = 1; p.ntx <= (k.nx + 15) / 16; ++p.ntx) {
        const int w = (k.nx + p.ntx - 1) / p.ntx, across = w + (p.ntx > 1 ? 2 : 0);
        if (p.ntx > 1 && w == (k.nx + p.ntx - 2) / (p.ntx - 1)) continue;
        const int most = std::min({k.ny, p3_max_threads<S>() / across - 2, p3_max_core<S>() / w});
        for (int h = most; h >= 1; --h) {
            p.nty = (k.ny + h - 1) / h;
            if (h > 1 && (k.ny + h - 2) / (h - 1) == p.nty) continue;  // a lower tile of the same count
            const int wv = (across * (h + 2) + 63) / 64;
            const double bytes = double(NPL) * sizeof(S) * (2.0 * w + (p.ntx > 1 ? pad : 0)) * h *
                                 (w % kBlk || k.nx % kBlk ? (F32 ? 1.17 : 1.19) : 1.0);
            const long long column = (long long)p.ntx * p.nty * k.batch, cap = cus;  // LDS holds one a CU
            auto plane = [&](long long n) {
                const double lat = l0 + l1 * wv;
                return std::cbrt(lat * lat * lat + std::pow(bytes * double(n) / bw, 3));
            };
            for (int seg = k.nz; seg >= 1; --seg) {
                p.nseg = (k.nz + seg - 1) / seg;
                if (seg > 1 && (k.nz + seg - 2) / (seg - 1) == p.nseg) continue;
                const long long wgs = column * p.nseg;
                if (wgs >= (1 << 21)) break;
                const double cost = t0 + (seg + 1.6) * (double(wgs / cap) * plane(cap) +
                                                        (wgs % cap ? plane(wgs % cap) : 0.0));
                if (cost < least) {
                    least = cost;
                    best = p;
                }
            }
        }
    }
    return best;
}

namespace {

template <typename S>
hipError_t launch_p3_march(const P3K& k, const P3MarchPlan& plan, const S* a, S* b, hipStream_t s) {
    const long long w = (k.nx + plan.ntx - 1) / plan.ntx, h = (k.ny + plan.nty - 1) / plan.nty;
    const long long threads = p3_march_threads(k, plan);
    const long long wgs = (long long)plan.ntx * plan.nty * plan.nseg * k.batch;
    if (threads > p3_max_threads<S>() || w * h > p3_max_core<S>() || wgs < 1 || wgs >= (1 << 21) ||
        plan.nseg > k.nz || k.nx < 2 || k.ny < 2 || k.nz < 2)
        return hipErrorInvalidValue;
    P3MarchArgs<S> p{};
    p.k = p3_kt<S>(k);
    p.ntx = plan.ntx; p.nty = plan.nty; p.nseg = plan.nseg;
    p.wx = k.nx / plan.ntx; p.ex = k.nx % plan.ntx;
    p.wy = k.ny / plan.nty; p.ey = k.ny % plan.nty;
    p.wz = k.nz / plan.nseg; p.ez = k.nz % plan.nseg;
    const unsigned blk = unsigned((threads + 63) / 64 * 64);
    constexpr int NT = p3_max_threads<S>(), NC = p3_max_core<S>();
    hipLaunchKernelGGL((p3_aligned<S>(k) ? k_p3_march<S, NT, NC, true> : k_p3_march<S, NT, NC, false>),
                       dim3(unsigned((wgs + kXCD - 1) / kXCD * kXCD)), dim3(blk), 0, s, p, a, b);
    return hipGetLastError();
}

}  // namespace

template <typename S>
hipError_t launch_p3_step(const P3K& k, const P3MarchPlan& plan, const S* a, S* b, S* phi,
                          hipStream_t s) {
    if (plan.ntx > 0) return launch_p3_march<S>(k, plan, a, b, s);
    hipError_t e = launch_phi<S>(k, a, phi, s);
    if (e != hipSuccess) return e;
    const long long tiles = p3_tiles<S>(k);
    dim3 blk(P3Tile<S>::X, P3Tile<S>::Y, P3Tile<S>::Z), grd(unsigned((tiles + kXCD - 1) / kXCD * kXCD));
    hipLaunchKernelGGL((k_p3_step<S, false>), grd, blk, 0, s, k, a, b, (const S*)phi,
                       MacroOut{});
    return hipGetLastError();
}

template <typename S>
hipError_t launch_p3_init(const P3K& k, const double* fields, S* a, hipStream_t s) {
    const long long N = (long long)k.batch * k.nx * k.ny * k.nz;
    hipLaunchKernelGGL(k_p3_init<S>, dim3(grid_p3(N, 256)), dim3(256), 0, s, k, fields, a);
    return hipGetLastError();
}

template <typename S>
hipError_t launch_p3_macros(const P3K& k, const S* a, S* phi, const MacroOut& out, hipStream_t s) {
    hipError_t e = launch_phi<S>(k, a, phi, s);
    if (e != hipSuccess) return e;
    const long long tiles = p3_tiles<S>(k);
    dim3 blk(P3Tile<S>::X, P3Tile<S>::Y, P3Tile<S>::Z), grd(unsigned((tiles + kXCD - 1) / kXCD * kXCD));
    hipLaunchKernelGGL((k_p3_step<S, true>), grd, blk, 0, s, k, a, (S*)nullptr, (const S*)phi, out);
    return hipGetLastError();
}

#define LBM_P3_INST(S)                                                                       \
    template P3MarchPlan p3_march_plan<S>(const P3K&);                                       \
    template hipError_t launch_p3_step<S>(const P3K&, const P3MarchPlan&, const S*, S*, S*,  \
                                          hipStream_t);                                      \
    template hipError_t launch_p3_init<S>(const P3K&, const double*, S*, hipStream_t);       \
    template hipError_t launch_p3_macros<S>(const P3K&, const S*, S*, const MacroOut&, hipStream_t);
LBM_P3_INST(float)
LBM_P3_INST(double)

}  // namespace lbm
