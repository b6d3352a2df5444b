// D3Q19 momentum step of liblbm for gfx950: the dimensional MRT of Sec. 3 in
// three dimensions (the extension the paper's conclusions call direct), BGK
// as the case of equal rates, Guo forcing, and per axis periodic or halfway
// bounce-back walls (Eq. BB_vel with u_w = 0).
//
// Layout and streaming follow the two-phase D2Q9 kernels: node n = ((b * nz +
// z) * ny + y) * nx + x, the 19 populations in node blocks (value i of node n
// at bidx(19, i, n); a wave's 64 nodes are one contiguous block), the stored
// state is the pre-collision set, and each node pushes its post-collision
// values to x + e_i (or back into its own opposite slot through a wall).
// FP32 storage keeps f_i - w_i rho_ref.
//
// Moment space.  The basis is the orthogonal set of d'Humieres et al. (2002)
// (rows rho, e, eps, j_x, q_x, j_y, q_y, j_z, q_z, 3p_xx, 3pi_xx, p_ww, pi_ww,
// p_xy, p_yz, p_xz, m_x, m_y, m_z).  The dimensional matrix scales row k by
// c^order(k); a diagonal relaxation commutes with that scaling, so the kernel
// works in lattice-normalised form (u / c, F dt^2 / dx, Lambda dt) and gets
// the populations of the dimensional scheme.  The equilibrium and forcing
// moments are closed forms, so neither feq_i nor the Guo term is built per
// population.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "lbm_d3q19.h"
#include "lbm_device.h"

// Rows of 64 nodes per workgroup.  Measured on the 256^3 box with the state in
// node blocks (ms per FP32 step): 64 x 4 0.489, 64 x 2 0.490, 64 x 1 0.497;
// FP64 0.937-0.942 for all three.  Capping residency at 4 waves per SIMD by
// an LDS reserve, which helped when the state was stored as planes (0.541 ->
// 0.522 ms), now costs time (64 x 4: 0.502-0.504 ms; 64 x 2 0.515, 64 x 1
// 0.505), so every workgroup takes only the LDS it uses (none).
#ifndef LBM_D3_TY
#define LBM_D3_TY 4
#endif

namespace lbm {
namespace {

constexpr int kD3Ty = LBM_D3_TY;  // rows of 64 nodes per workgroup

// Post-collision populations v of one node from its stored deviations d.
// Shared by the one- and two-step kernels, so that both round identically.
template <typename C, typename K>
__device__ __forceinline__ void d3_collide(const K& k, const C (&d)[19], C (&v)[19]) {
    C m[19];
    moments19(d, m);
    // macros: rho = rho_ref + sum d (the deviations carry no momentum of their own)
    const C drho = m[0];
    const C rho = C(k.rho_ref) + drho;
    const C fx = C(k.Ft[0]), fy = C(k.Ft[1]), fz = C(k.Ft[2]);
    const C ir = C(1) / rho;
    const C ux = (m[3] + C(0.5) * fx) * ir;  // Eq. first_moment_f, over c
    const C uy = (m[5] + C(0.5) * fy) * ir;
    const C uz = (m[7] + C(0.5) * fz) * ir;

    // non-equilibrium moments m - m_eq; m_eq in deviation form (minus rho_ref M w)
    const C rxx = rho * ux * ux, ryy = rho * uy * uy, rzz = rho * uz * uz;
    const C ruu = (rxx + ryy) + rzz;
    const C pxx = C(2) * rxx - (ryy + rzz), pww = ryy - rzz;
    C neq[19];
    neq[0] = C(0);
    neq[1] = m[1] - (C(19) * ruu - C(11) * drho);
    neq[2] = m[2] - (C(3) * drho - C(5.5) * ruu);
    neq[3] = C(0);
    neq[4] = m[4] + (C(2) / C(3)) * (rho * ux);
    neq[5] = C(0);
    neq[6] = m[6] + (C(2) / C(3)) * (rho * uy);
    neq[7] = C(0);
    neq[8] = m[8] + (C(2) / C(3)) * (rho * uz);
    neq[9] = m[9] - pxx;
    neq[10] = m[10] + C(0.5) * pxx;
    neq[11] = m[11] - pww;
    neq[12] = m[12] + C(0.5) * pww;
    neq[13] = m[13] - rho * ux * uy;
    neq[14] = m[14] - rho * uy * uz;
    neq[15] = m[15] - rho * ux * uz;
    neq[16] = m[16];
    neq[17] = m[17];
    neq[18] = m[18];
    // moments of the Guo term (Eq. forcing_term): the u-derivative of m_eq along F
    const C uf = (ux * fx + uy * fy) + uz * fz;
    const C fxx = ux * fx, fyy = uy * fy, fzz = uz * fz;
    const C qxx = C(2) * fxx - (fyy + fzz), qww = fyy - fzz;
    C mf[19];
    mf[0] = C(0);
    mf[1] = C(38) * uf;
    mf[2] = C(-11) * uf;
    mf[3] = fx;
    mf[4] = (C(-2) / C(3)) * fx;
    mf[5] = fy;
    mf[6] = (C(-2) / C(3)) * fy;
    mf[7] = fz;
    mf[8] = (C(-2) / C(3)) * fz;
    mf[9] = C(2) * qxx;
    mf[10] = -qxx;
    mf[11] = C(2) * qww;
    mf[12] = -qww;
    mf[13] = ux * fy + uy * fx;
    mf[14] = uy * fz + uz * fy;
    mf[15] = ux * fz + uz * fx;
    mf[16] = C(0);
    mf[17] = C(0);
    mf[18] = C(0);
    // Eq. colisao_MRT: dm = -Lambda (m - m_eq) + (I - Lambda/2) dt F, rates times dt
    C dm[19], dv[19];
#pragma unroll
    for (int q = 0; q < 19; ++q) {
        const C L = C(k.L[q]);
        dm[q] = -L * neq[q] + (C(1) - C(0.5) * L) * mf[q];
    }
    inverse19(dm, dv);
#pragma unroll
    for (int i = 0; i < 19; ++i) v[i] = d[i] + dv[i];
}

// One step: tiles of 64 x kD3Ty nodes in one z plane of one replica, numbered x
// fastest, then y, z and replica, and handed to the XCDs in contiguous bands
// (a tile's z neighbours, into which it pushes, sit gx * gy tiles away in the
// same band).
template <typename S>
__global__ __launch_bounds__(64 * kD3Ty) void k_d3_step(D3K k, const S* __restrict__ fc,
                                                 S* __restrict__ fn) {
    using C = S;
    const int nx = k.nx, ny = k.ny, nz = k.nz;
    const int gx = (nx + 63) / 64, gy = (ny + kD3Ty - 1) / kD3Ty;
    int tile;
    if (!xcd_tile(gx * gy * nz * k.batch, tile)) return;
    const int r = tile % (gx * gy);
    const int bz = tile / (gx * gy);  // b * nz + z
    const int z = bz % nz;
    const int x = (r % gx) * 64 + threadIdx.x;
    const int y = (r / gx) * kD3Ty + threadIdx.y;
    if (x >= nx || y >= ny) return;
    const long long plane = (long long)nx * ny;
    const long long base = (long long)(bz - z) * plane;  // first node of the replica
    const long long n = base + (long long)z * plane + (long long)y * nx + x;

    C d[19];
#pragma unroll
    for (int i = 0; i < 19; ++i) d[i] = C(fc[bidx(19, i, n)]);
    C v[19];
    d3_collide<C>(k, d, v);

    // streaming with halfway bounce-back where a wall closes the axis
#pragma unroll
    for (int i = 0; i < 19; ++i) {
        const int tx = x + E3X[i], ty = y + E3Y[i], tz = z + E3Z[i];
        const bool out = (k.bcx && (tx < 0 || tx >= nx)) || (k.bcy && (ty < 0 || ty >= ny)) ||
                         (k.bcz && (tz < 0 || tz >= nz));
        if (out) {
            st(fn + bidx(19, OPP3[i], n), S(v[i]));
        } else {
            const long long t = base + (long long)wrap(tz, nz) * plane +
                                (long long)wrap(ty, ny) * nx + wrap(tx, nx);
            st(fn + bidx(19, i, t), S(v[i]));
        }
    }
}

// ---------------------------------------------------------------------------
// Two steps per launch (temporal blocking).  The single step moves its bytes
// at the rate of a copy, so the state crosses HBM once per two steps here.  A
// workgroup takes a column of w x h nodes with one node of overlap around it
// (one node per thread, at most NT) and marches up the planes of one segment
// [a, e) of one replica.  At plane v it collides step n at plane v and step
// n + 1 at plane v - 1:
//   - step n's moving values go through LDS; the values that stay in plane v
//     or move up or down are pulled from the neighbour threads into the
//     step-(n + 1) state of planes v, v + 1 and v - 1, of which only that of
//     plane v - 1 (W) and the five values moving into plane v (U) stay in
//     registers from one plane to the next;
//   - step n + 1 at plane v - 1 pushes to memory like the single step, from
//     the tile's own nodes only, so every slot is written by its source.
// The loads of plane v + 1 are issued before step n + 1 collides, so they land
// while it computes (loaded at their own plane step: 148 against 128 us per
// step on 256 x 256 x 128).  Step n runs on planes a - 1 .. e (those that
// exist), so the segments are independent.  A value whose source lies beyond
// a wall is the node's own opposite one, set when the node's plane collides.
//
// ALIGNED: planes a multiple of 64 nodes and under 2 GiB, so an access is the
// plane's block base (uniform) plus a 32-bit lane offset.
// ---------------------------------------------------------------------------
template <typename C>
struct D3KT {  // D3K in the type the kernel computes in
    int nx, ny, nz, batch, bcx, bcy, bcz;
    C rho_ref, L[19], Ft[3];
};
template <typename C>
struct D3Tb2Args {
    D3KT<C> k;
    int ntx, nty, nseg;           // tiles per plane and segments per replica
    int wx, ex, wy, ey, wz, ez;   // tile i spans w nodes, one more for i < e
};

__device__ constexpr int kD3In[8] = {1, 2, 3, 4, 7, 8, 9, 10};  // movers within a plane
__device__ constexpr int kD3Up[4] = {11, 14, 15, 18};           // + (0, 0, 1), i = 5
__device__ constexpr int kD3Dn[4] = {12, 13, 16, 17};           // + (0, 0, -1), i = 6
// LDS plane of mover i (all but 0, 5 and 6, which stay in their column)
__device__ constexpr int d3_plane(int i) { return i < 5 ? i - 1 : i - 3; }

template <typename S, int NT, bool ALIGNED>
__global__ __launch_bounds__(NT) void k_d3_tb2(const D3Tb2Args<S> p, const S* __restrict__ A,
                                               S* __restrict__ B) {
    using C = S;
    __shared__ C buf[2][16][NT];
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
    // Threads: the tile's columns row by row (rows y0 - 1 .. y1), so that a wave
    // of a 64-wide row is one node block, then the columns x0 - 1 and x1.  A
    // tile as wide as the grid has none: its rows wrap in LDS.
    const int wc = x1 - x0, rh = y1 - y0 + 2;
    const bool whole = p.ntx == 1;
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
    // the lane's column: wrapped, or clamped where a wall ends the axis (such
    // a lane feeds nothing: the rule at the wall takes the node's own value)
    const int vx = x0 + rx, vy = y0 - 1 + (in ? ry : 0);
    const int x = vx < 0 ? (k.bcx ? 0 : nx - 1) : vx >= nx ? (k.bcx ? nx - 1 : 0) : vx;
    const int y = vy < 0 ? (k.bcy ? 0 : ny - 1) : vy >= ny ? (k.bcy ? ny - 1 : 0) : vy;
    const bool xlo = k.bcx && x == 0, xhi = k.bcx && x == nx - 1;
    const bool ylo = k.bcy && y == 0, yhi = k.bcy && y == ny - 1;
    const bool edge = xlo || xhi || ylo || yhi;
    const bool plain = !__any(edge);  // no lane of this wave stands at an x or y wall
    const TileOffsets off = tile_offsets(in, whole, rx, ry, wc, rh, xlo, xhi);
    const int plane = nx * ny;
    const long long base = (long long)b * nz * plane;
    auto zof = [&](int v) { return v < 0 ? v + nz : (v >= nz ? v - nz : v); };

    // columns of the push: x - 1, x, x + 1 in rows y - 1, y, y + 1 (wrapped)
    unsigned col[9];
#pragma unroll
    for (int c = 0; c < 9; ++c) {
        const int q = wrap(y + c / 3 - 1, ny) * nx + wrap(x + c % 3 - 1, nx);
        col[c] = ALIGNED ? unsigned(((q >> 6) * 19 * kBlk + (q & (kBlk - 1))) * int(sizeof(S)))
                         : unsigned(q);
    }
    auto at = [&](auto* P, int z, int c, int i) {
        const long long po = base + (long long)z * plane;
        if constexpr (ALIGNED) {
            using B8 = std::conditional_t<std::is_const_v<std::remove_pointer_t<decltype(P)>>,
                                          const char, char>;
            auto* row = (B8*)P + (po >> 6) * (long long)(19 * kBlk * sizeof(S));
            return (decltype(P))(row + col[c]) + i * kBlk;
        } else {
            return P + bidx(19, i, po + col[c]);
        }
    };
    // whether the value in slot j comes through an x or y wall
    auto outxy = [&](int j) {
        return (E3X[j] > 0 ? xlo : E3X[j] < 0 ? xhi : false) ||
               (E3Y[j] > 0 ? ylo : E3Y[j] < 0 ? yhi : false);
    };
    auto pull = [&](const C(&xb)[16][NT], int j) {
        return xb[d3_plane(j)][t + (E3X[j] > 0 ? off.om : E3X[j] < 0 ? off.op : 0) +
                               (E3Y[j] > 0 ? off.od : E3Y[j] < 0 ? off.ou : 0)];
    };

    const int s1 = k.bcz ? max(a - 1, 0) : a - 1;   // first plane of step n
    const int e1 = k.bcz ? min(e + 1, nz) : e + 1;  // end of the step-n planes
    C Ld[19], W[19], U[5];
#pragma unroll
    for (int i = 0; i < 19; ++i) {
        Ld[i] = C(*at(A, zof(s1), 4, i));
        W[i] = C(0);
    }
#pragma unroll
    for (int i = 0; i < 5; ++i) U[i] = C(0);

    for (int v = s1; v <= e; ++v) {
        const bool do_n = v < e1;
        C(&xb)[16][NT] = buf[v & 1];
        C r0 = C(0), rup = C(0), rdn = C(0);  // rest, +z and -z of step n
        if (do_n) {
            C ds[19];
            d3_collide<C>(k, Ld, ds);
            r0 = ds[0];
            rup = ds[5];
            rdn = ds[6];
#pragma unroll
            for (int i = 1; i < 19; ++i)
                if (i != 5 && i != 6 && in) xb[d3_plane(i)][t] = ds[i];
        }
        __syncthreads();  // the other buffer's reads ended a plane ago
        {   // the next plane (the last steps re-read an existing one)
            const int z = zof(min(v + 1, e1 - 1));
#pragma unroll
            for (int i = 0; i < 19; ++i) Ld[i] = C(*at(A, z, 4, i));
        }
        if (do_n && v > s1) {  // plane v - 1 receives the values that move down
            W[6] = rdn;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int j = kD3Dn[q];
                const C pv = pull(xb, j);
                W[j] = outxy(j) ? W[j] : pv;
            }
        }
        // ---- step n + 1 at plane r = v - 1, complete now
        const int r = v - 1;
        if (r >= a && own) {
            C ds[19];
            d3_collide<C>(k, W, ds);
            const bool zlo = k.bcz && r == 0, zhi = k.bcz && r == nz - 1;
            const int zm = zof(r - 1), zp = zof(r + 1);
            if (plain && !zlo && !zhi) {
#pragma unroll
                for (int i = 0; i < 19; ++i)
                    st(at(B, E3Z[i] > 0 ? zp : E3Z[i] < 0 ? zm : r, 4 + E3X[i] + 3 * E3Y[i], i),
                       S(ds[i]));
            } else {
#pragma unroll
                for (int i = 0; i < 19; ++i) {
                    const bool outz = E3Z[i] > 0 ? zhi : E3Z[i] < 0 ? zlo : false;
                    // a mover leaves where the value in the opposite slot comes in
                    if (outz || outxy(OPP3[i]))
                        st(at(B, r, 4, OPP3[i]), S(ds[i]));
                    else
                        st(at(B, E3Z[i] > 0 ? zp : E3Z[i] < 0 ? zm : r,
                              4 + E3X[i] + 3 * E3Y[i], i), S(ds[i]));
                }
            }
        }
        // ---- the state of plane v so far, and what moves up from it
        if (do_n) {
            W[0] = r0;
#pragma unroll
            for (int q = 0; q < 8; ++q) W[kD3In[q]] = pull(xb, kD3In[q]);
            W[5] = U[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                W[kD3Up[q]] = U[q];
                U[q] = pull(xb, kD3Up[q]);
            }
            U[4] = rup;
            const bool zlo = k.bcz && v == 0, zhi = k.bcz && v == nz - 1;
            if (zlo) W[5] = rdn;
            if (zhi) W[6] = rup;
            if (edge || zlo || zhi) {
#pragma unroll
                for (int j = 1; j < 19; ++j) {
                    if (j == 5 || j == 6) continue;
                    const bool outz = E3Z[j] > 0 ? zlo : E3Z[j] < 0 ? zhi : false;
                    if (outz || outxy(j)) W[j] = xb[d3_plane(OPP3[j])][t];
                }
            }
        }
    }
}

// equilibrium populations from FP64 fields (staging slots 0 rho, 2 ux, 3 uy,
// 7 uz; velocities in m/s)
template <typename S>
__global__ void k_d3_init(D3K k, const double* __restrict__ fld, S* __restrict__ f) {
    const long long N = (long long)k.batch * k.nx * k.ny * k.nz;
    const long long P = k.P;
    for (long long n = blockIdx.x * (long long)blockDim.x + threadIdx.x; n < N;
         n += (long long)gridDim.x * blockDim.x) {
        const double rho = fld[n];
        const double ux = fld[2 * P + n] / k.c, uy = fld[3 * P + n] / k.c, uz = fld[7 * P + n] / k.c;
        const double uu = ux * ux + uy * uy + uz * uz;
        for (int i = 0; i < 19; ++i) {
            const double eu = E3X[i] * ux + E3Y[i] * uy + E3Z[i] * uz;
            f[bidx(19, i, n)] = S(w19<double>(i) * ((rho - k.rho_ref) + rho * (3 * eu + 4.5 * eu * eu - 1.5 * uu)));
        }
    }
}

// FP64 macros of the stored state
template <typename S>
__global__ void k_d3_macros(D3K k, const S* __restrict__ f, MacroOut out) {
    const long long N = (long long)k.batch * k.nx * k.ny * k.nz;
    for (long long n = blockIdx.x * (long long)blockDim.x + threadIdx.x; n < N;
         n += (long long)gridDim.x * blockDim.x) {
        double d[19], m[19];
        for (int i = 0; i < 19; ++i) d[i] = double(f[bidx(19, i, n)]);
        moments19(d, m);
        const double rho = k.rho_ref + m[0];
        out.put(0, n, rho);
        out.put(2, n, (m[3] + 0.5 * k.Ft[0]) / rho * k.c);
        out.put(3, n, (m[5] + 0.5 * k.Ft[1]) / rho * k.c);
        out.put(7, n, (m[7] + 0.5 * k.Ft[2]) / rho * k.c);
    }
}

inline unsigned grid_1d(long long N, int bs) {
    long long g = (N + bs - 1) / bs;
    if (g > 65535LL * 16) g = 65535LL * 16;
    return unsigned(g < 1 ? 1 : g);
}

}  // namespace

long long d3_tiles(const D3K& k) {
    return (long long)((k.nx + 63) / 64) * ((k.ny + kD3Ty - 1) / kD3Ty) * k.nz * k.batch;
}

template <typename S>
hipError_t launch_d3_step(const D3K& k, const S* fc, S* fn, hipStream_t s) {
    const long long tiles = d3_tiles(k);
    dim3 blk(64, kD3Ty), grd(unsigned((tiles + kXCD - 1) / kXCD * kXCD));
    hipLaunchKernelGGL(k_d3_step<S>, grd, blk, 0, s, k, fc, fn);
    return hipGetLastError();
}

namespace {

template <typename C>
D3KT<C> d3_kt(const D3K& k) {
    D3KT<C> r{};
    r.nx = k.nx; r.ny = k.ny; r.nz = k.nz; r.batch = k.batch;
    r.bcx = k.bcx; r.bcy = k.bcy; r.bcz = k.bcz;
    r.rho_ref = C(k.rho_ref);
    for (int q = 0; q < 19; ++q) r.L[q] = C(k.L[q]);
    for (int q = 0; q < 3; ++q) r.Ft[q] = C(k.Ft[q]);
    return r;
}

template <typename S>
bool d3_tb2_aligned(const D3K& k) {
    const long long plane = (long long)k.nx * k.ny;
    return plane % kBlk == 0 && plane * 19 * (long long)sizeof(S) < (1LL << 31);
}
template <typename S>
constexpr int d3_max_threads() {
    return sizeof(S) == 4 ? 1024 : 512;
}
template <typename S>
auto d3_tb2_kernel(bool aligned, int threads) {
    if constexpr (sizeof(S) == 4) {
        if (threads > 768) return aligned ? k_d3_tb2<S, 1024, true> : k_d3_tb2<S, 1024, false>;
        if (threads > 512) return aligned ? k_d3_tb2<S, 768, true> : k_d3_tb2<S, 768, false>;
    }
    return aligned ? k_d3_tb2<S, 512, true> : k_d3_tb2<S, 512, false>;
}

}  // namespace

long long d3_tb2_threads(const D3K& k, const D3Tb2Plan& p) {
    return (long long)((k.nx + p.ntx - 1) / p.ntx + (p.ntx > 1 ? 2 : 0)) *
           ((k.ny + p.nty - 1) / p.nty + 2);
}

// Tiles and segments by a cost model fitted to 1200 plans on 30 boxes of 0.1 M
// to 17 M nodes (10 %; its choice runs 3 to 4 % behind the best measured plan on
// average, 12 % at most).  A workgroup takes planes + 2 plane steps, each a
// mean of power 2.7 of
//   l0 + l1 waves   the chain of a plane step: load, two collisions, barrier;
//   the bytes all resident workgroups move in it at 6.8 (FP64: 6.6) TB/s, with
//   lost columns (pad) where tiles cut the rows, a share more (cut) where they
//   cut them inside node blocks, and another (uneven) where tiles differ in
//   height, their workgroups then drifting apart (256 x 256 x 128: tiles of 128 x 4
//   129 us a step, of 64 x 12 and 64 x 13 142),
// in rounds of one workgroup per CU.  Measured per step, single -> two-step:
// FP32 256 x 256 x 128 247 -> 128-133 us (4.98 TB/s of the launch's bytes, the
// rate of a copy), 192^3 227 -> 117, 128^3 73 -> 39, 64^3 13.6 -> 7.0; FP64
// 256 x 256 x 128 473 -> 274-308 us, 64^3 19 -> 12.  Rows of 32 columns, whose
// loads touch twice the lines, take 158 us on the first, rows whose overlap
// columns sit in the same waves (66 lanes a row) 163 us.
// Single steps take 7.5 us plus their bytes at 5.2 TB/s; `fast` asks for 10 %
// less.
template <typename S>
D3Tb2Plan d3_tb2_plan(const D3K& k) {
    D3Tb2Plan best{};
    int dev = 0, cus = 0;
    if (k.nx < 2 || k.ny < 2 || k.nz < 2 || (long long)k.nx * k.ny >= (1LL << 31) ||
        hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        return best;
    constexpr bool F32 = sizeof(S) == 4;
    const double l0 = F32 ? 1.41 : 1.0, l1 = F32 ? 0.15 : 0.38, pad = F32 ? 25 : 8.7;
    const double cut = F32 ? 0.17 : 0.19, uneven = F32 ? 0.10 : 0.05, power = 2.7;
    const double bw = F32 ? 6.8e6 : 6.6e6;  // bytes per us
    const double nodes = double(k.nx) * k.ny * k.nz * k.batch;
    const double single = 7.5 + nodes * 38 * sizeof(S) / 5.2e6;
    double least = 1e300;
    D3Tb2Plan p{};
    for (p.ntx = 1; p.ntx <= (k.nx + 15) / 16; ++p.ntx) {
        const int w = (k.nx + p.ntx - 1) / p.ntx, across = w + (p.ntx > 1 ? 2 : 0);
        if (p.ntx > 1 && w == (k.nx + p.ntx - 2) / (p.ntx - 1)) continue;
        for (int h = std::min(k.ny, d3_max_threads<S>() / across - 2); h >= 1; --h) {
            p.nty = (k.ny + h - 1) / h;
            if (h > 1 && (k.ny + h - 2) / (h - 1) == p.nty) continue;  // a lower tile of the same count
            const double lat = l0 + l1 * ((across * (h + 2) + 63) / 64);
            const double bytes = 19.0 * sizeof(S) * (2.0 * w + (p.ntx > 1 ? pad : 0)) * k.ny / p.nty *
                                 (1 + (w % kBlk && p.ntx > 1 ? cut : 0.0) + (k.ny % p.nty ? uneven : 0.0));
            const long long column = (long long)p.ntx * p.nty * k.batch;
            const double chain = std::pow(lat, power);
            auto plane = [&](long long n) {
                return std::pow(chain + std::pow(bytes * n / bw, power), 1 / power);
            };
            const double full = plane(cus);
            for (int seg = k.nz; seg >= 1; --seg) {
                p.nseg = (k.nz + seg - 1) / seg;
                if (seg > 1 && (k.nz + seg - 2) / (seg - 1) == p.nseg) continue;
                const long long wgs = column * p.nseg;
                if (wgs >= (1 << 21)) break;
                const double planes = F32 ? double(k.nz) / p.nseg : seg;
                const double cost = (planes + 2) * (double(wgs / cus) * full +
                                                 (wgs % cus ? plane(wgs % cus) : 0.0)) / 2;
                if (cost < least) {
                    least = cost;
                    best = p;
                }
            }
        }
    }
    best.fast = least < 0.9 * single;
    return best;
}

template <typename S>
hipError_t launch_d3_tb2(const D3K& k, const D3Tb2Plan& plan, const S* fc, S* fn, hipStream_t s) {
    const long long threads = plan.ntx > 0 && plan.nty > 0 ? d3_tb2_threads(k, plan) : 0;
    const long long wgs = (long long)plan.ntx * plan.nty * plan.nseg * k.batch;
    if (threads < 1 || threads > d3_max_threads<S>() || wgs < 1 || wgs >= (1 << 21) ||
        plan.nseg > k.nz || k.nx < 2 || k.ny < 2 || k.nz < 2)
        return hipErrorInvalidValue;
    D3Tb2Args<S> p{};
    p.k = d3_kt<S>(k);
    p.ntx = plan.ntx; p.nty = plan.nty; p.nseg = plan.nseg;
    p.wx = k.nx / plan.ntx; p.ex = k.nx % plan.ntx;
    p.wy = k.ny / plan.nty; p.ey = k.ny % plan.nty;
    p.wz = k.nz / plan.nseg; p.ez = k.nz % plan.nseg;
    const int blk = int((threads + 63) / 64 * 64);
    hipLaunchKernelGGL(d3_tb2_kernel<S>(d3_tb2_aligned<S>(k), blk),
                       dim3(unsigned((wgs + kXCD - 1) / kXCD * kXCD)), dim3(unsigned(blk)), 0, s, p, fc, fn);
    return hipGetLastError();
}

template <typename S>
hipError_t launch_d3_init(const D3K& k, const double* fields, S* f, hipStream_t s) {
    const long long N = (long long)k.batch * k.nx * k.ny * k.nz;
    hipLaunchKernelGGL(k_d3_init<S>, dim3(grid_1d(N, 256)), dim3(256), 0, s, k, fields, f);
    return hipGetLastError();
}

template <typename S>
hipError_t launch_d3_macros(const D3K& k, const S* f, const MacroOut& out, hipStream_t s) {
    const long long N = (long long)k.batch * k.nx * k.ny * k.nz;
    hipLaunchKernelGGL(k_d3_macros<S>, dim3(grid_1d(N, 256)), dim3(256), 0, s, k, f, out);
    return hipGetLastError();
}

#define LBM_D3_INST(S)                                                                   \
    template hipError_t launch_d3_step<S>(const D3K&, const S*, S*, hipStream_t);        \
    template D3Tb2Plan d3_tb2_plan<S>(const D3K&);                                       \
    template hipError_t launch_d3_tb2<S>(const D3K&, const D3Tb2Plan&, const S*, S*,     \
                                         hipStream_t);                                   \
    template hipError_t launch_d3_init<S>(const D3K&, const double*, S*, hipStream_t);   \
    template hipError_t launch_d3_macros<S>(const D3K&, const S*, const MacroOut&, hipStream_t);
LBM_D3_INST(float)
LBM_D3_INST(double)

}  // namespace lbm
