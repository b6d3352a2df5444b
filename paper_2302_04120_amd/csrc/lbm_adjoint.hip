// Discrete adjoint of the D2Q9 (BGK/MRT) + D2Q5 heated-channel step.
//
// One forward step maps the pre-collision state s(n) = (f, g) to s(n+1) by
// macros -> collision -> push-streaming with the boundary rules.  The reverse
// step applies the transpose of that map's Jacobian to the adjoint state
// lambda(n+1) and returns lambda(n).  It is written in gather form: the node
// reads the adjoint values at the slots its own post-collision populations were
// written to (the transpose of the push, including each boundary rule), applies
// the transposed collision of the thermal and then the momentum populations,
// and writes lambda(n) at its own slots only, so no two threads write the same
// value.  The moment-space relaxation operators M^-1 diag(L) M are symmetric
// (the rows of M are orthogonal), so their transposes are the same transforms.
//
// Parameter gradients accumulate in FP64 with one owner per accumulator: the
// wall-flux gradient per column and wall (the wall-node thread), the
// relaxation-time gradients per tile (thread 0 of the tile's workgroup, the
// tile-to-workgroup map being fixed), then summed in a fixed order.
#include "lbm_channel.h"
#include "lbm_device.h"

#include <cmath>

namespace lbm {
namespace {

__device__ __forceinline__ double wave_sum64(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// The reverse step of one node: lambda(n) into l from its state (d, e) at n and
// lambda(n + 1), read through
//   own(j)    value j of the node itself (lambda_f 0-8, lambda_g 9-13),
//   nb(i)     value i of the node its population i went to (9 + i for g),
//   right(j)  value j of the node at x + 1 (asked for left of the outlet only),
//   side(s, ux, uy)  the velocity of the node at x + s (at and left of the
//             outlet only).
// Adds the node's shares of the gradients to dqb, dqt (flux, bottom and top
// wall), dtn and dtt (tau and tau_T).  Shared by the one- and many-step
// kernels, so that their adjoint states agree to the last bit.
template <bool FORCED, typename C, typename K, typename Own, typename Nb, typename Right, typename Side>
__device__ __forceinline__ void adj_node(const K& k, const AdjK& a, const C (&d)[9],
                                         const C (&e)[5], int x, int y, C mod, Own own, Nb nb,
                                         Right right, Side side, C (&l)[14], double& dqb,
                                         double& dqt, double& dtn, double& dtt) {
    const int nx = k.nx, ny = k.ny;
    const C rho_ref = C(k.rho_ref), ftx = C(k.Ft[0]), fty = C(k.Ft[1]);
    C drho, rho, ux, uy;
    chan_flow_macros_v<C>(d, rho_ref, ftx, fty, drho, rho, ux, uy);
    const C qdt = C(k.qdt);
    const C th = (e[0] + (e[1] + e[3]) + (e[2] + e[4])) + C(0.5) * qdt;

    // ---- transpose of streaming and the momentum boundary rules
    C ubx = C(0), uby = C(0);  // adjoint of the lattice velocity u / c
    C uwx = C(0), uwy = C(0);
    if (k.bcx && x == nx - 1) {
        C ux2, uy2;
        side(-1, ux2, uy2);
        uwx = C(1.5) * ux - C(0.5) * ux2;
        uwy = C(1.5) * uy - C(0.5) * uy2;
    }
    const bool xlo = k.bcx && x == 0, xhi = k.bcx && x == nx - 1;
    const bool ylo = k.bcy && y == 0, yhi = k.bcy && y == ny - 1;
    C ls[9], lsg[5];
#pragma unroll
    for (int i = 0; i < 9; ++i) ls[i] = nb(i);
#pragma unroll
    for (int i = 0; i < 5; ++i) lsg[i] = nb(9 + i);
    if (xlo || xhi || ylo || yhi) {
#pragma unroll
        for (int i = 1; i < 9; ++i) {
            const bool outy = EY[i] < 0 ? ylo : EY[i] > 0 ? yhi : false;
            const bool outx = EX[i] < 0 ? xlo : EX[i] > 0 ? xhi : false;
            if (outy || (outx && EX[i] < 0)) {
                ls[i] = own(OPP[i]);  // bounce-back (wall, moving inlet)
            } else if (outx) {
                // anti-bounce-back outlet: -f_i* + 2 w rho_ref [4.5 (e.u_w)^2 - 1.5 u_w^2]
                const C lam = own(OPP[i]);
                ls[i] = -lam;
                const C eu = C(EX[i]) * uwx + C(EY[i]) * uwy;
                const C k2 = C(2) * wgt<C>(i) * rho_ref;
                // u_w = 1.5 u(x_b) - 0.5 u(x_b - 1): this node's share
                ubx += C(1.5) * lam * k2 * (C(9) * eu * C(EX[i]) - C(3) * uwx);
                uby += C(1.5) * lam * k2 * (C(9) * eu * C(EY[i]) - C(3) * uwy);
            }
        }
        // thermal boundary rules
#pragma unroll
        for (int i = 1; i < 5; ++i) {
            const bool outy = EY5[i] < 0 ? ylo : EY5[i] > 0 ? yhi : false;
            const bool outx = EX5[i] < 0 ? xlo : EX5[i] > 0 ? xhi : false;
            if (outy) {
                // flux wall: + lambda (dt/dx) q'' / rho c_p
                const C lam = own(9 + OPP5[i]);
                lsg[i] = lam;
                const double gq = double(lam) * a.qgrad * double(mod);
                if (EY5[i] < 0) dqb += gq;
                else dqt += gq;
            } else if (outx) {
                // anti-bounce-back inlet; dropped at the extrapolation outlet
                lsg[i] = EX5[i] < 0 ? -own(9 + OPP5[i]) : C(0);
            }
        }
        if (xhi) lsg[3] += own(9 + 3);  // outlet slot took g_3*
    }
    if (k.bcx && nx >= 2 && x == nx - 2) {
        // the outlet node to the right depends on this node's velocity
        C ux2, uy2;
        side(1, ux2, uy2);
        const C vx = C(1.5) * ux2 - C(0.5) * ux, vy = C(1.5) * uy2 - C(0.5) * uy;
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            if (EX[i] != 1) continue;
            const int ty = y + EY[i];
            if (k.bcy && (ty < 0 || ty >= ny)) continue;  // wall rule at the corner
            const C lam = right(OPP[i]);
            const C eu = C(EX[i]) * vx + C(EY[i]) * vy;
            const C k2 = C(2) * wgt<C>(i) * rho_ref;
            ubx += C(-0.5) * lam * k2 * (C(9) * eu * C(EX[i]) - C(3) * vx);
            uby += C(-0.5) * lam * k2 * (C(9) * eu * C(EY[i]) - C(3) * vy);
        }
    }
    // ---- transpose of the thermal collision g* = g - A_T (g - g_eq(T, u)) + B_T S
    {
        C mL[5], mN[5], neq[5], tmp[5], ag[5];
        moments5(lsg, mL);
#pragma unroll
        for (int i = 0; i < 5; ++i)
            neq[i] = e[i] - wgt5<C>(i) * th * (C(1) + C(3) * (C(EX5[i]) * ux + C(EY5[i]) * uy));
        moments5(neq, mN);
        const double ms[5] = {double(qdt), 0.0, 0.0, -2.0 / 3.0 * double(qdt), 0.0};
#pragma unroll
        for (int q = 0; q < 5; ++q) {
            tmp[q] = C(k.Lt[q]) * mL[q];
            if (a.rows_t >> q & 1) dtt += double(mL[q]) * (a.cLt[q] * (double(mN[q]) + 0.5 * ms[q]));
        }
        inverse5(tmp, ag);  // A_T lambda* (A_T is symmetric)
        C tb = C(0);
#pragma unroll
        for (int i = 0; i < 5; ++i) {
            const C eu = C(EX5[i]) * ux + C(EY5[i]) * uy;
            tb += ag[i] * wgt5<C>(i) * (C(1) + C(3) * eu);
            ubx += ag[i] * wgt5<C>(i) * th * C(3) * C(EX5[i]);
            uby += ag[i] * wgt5<C>(i) * th * C(3) * C(EY5[i]);
        }
#pragma unroll
        for (int i = 0; i < 5; ++i) l[9 + i] = lsg[i] - ag[i] + tb;
    }
    // ---- transpose of the momentum collision f* = f - A (f - f_eq(rho, u)) + B F(u)
    //      (without a body force, FORCED false, F and its terms are zero)
    {
        const C uu = ux * ux + uy * uy;
        C neq[9], fh[9], av[9], bv[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const C eu = C(EX[i]) * ux + C(EY[i]) * uy;
            neq[i] = d[i] - wgt<C>(i) * (drho + rho * (C(3) * eu + C(4.5) * eu * eu - C(1.5) * uu));
            if constexpr (FORCED)
                fh[i] = wgt<C>(i) * ((C(3) * (C(EX[i]) - ux) + C(9) * eu * C(EX[i])) * ftx +
                                     (C(3) * (C(EY[i]) - uy) + C(9) * eu * C(EY[i])) * fty);
        }
        if (k.flow_mrt) {
            C mL[9], mN[9], mF[9], t1[9], t2[9];
            moments9(ls, mL);
            moments9(neq, mN);
            if constexpr (FORCED) moments9(fh, mF);
#pragma unroll
            for (int q = 0; q < 9; ++q) {
                const C L = C(k.Lf[q]);
                t1[q] = L * mL[q];
                if constexpr (FORCED) t2[q] = (C(1) - C(0.5) * L) * mL[q];
                if (a.rows_f >> q & 1) {
                    double r = double(mN[q]);
                    if constexpr (FORCED) r += 0.5 * double(mF[q]);
                    dtn += double(mL[q]) * (a.cLf[q] * r);
                }
            }
            inverse9(t1, av);
            if constexpr (FORCED) inverse9(t2, bv);
        } else {
            const C L = C(k.Lf[7]);
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                av[i] = L * ls[i];
                double r = double(neq[i]);
                if constexpr (FORCED) {
                    bv[i] = (C(1) - C(0.5) * L) * ls[i];
                    r += 0.5 * double(fh[i]);
                }
                dtn += double(ls[i]) * (a.cLf[7] * r);
            }
        }
        C rb = C(0);
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const C eu = C(EX[i]) * ux + C(EY[i]) * uy;
            const C w = wgt<C>(i);
            rb += av[i] * w * (C(1) + C(3) * eu + C(4.5) * eu * eu - C(1.5) * uu);
            ubx += av[i] * w * rho * (C(3) * C(EX[i]) + C(9) * eu * C(EX[i]) - C(3) * ux);
            uby += av[i] * w * rho * (C(3) * C(EY[i]) + C(9) * eu * C(EY[i]) - C(3) * uy);
            if constexpr (FORCED) {
                const C eF = C(EX[i]) * ftx + C(EY[i]) * fty;
                ubx += bv[i] * w * (C(-3) * ftx + C(9) * C(EX[i]) * eF);
                uby += bv[i] * w * (C(-3) * fty + C(9) * C(EY[i]) * eF);
            }
        }
        const C ir = C(1) / rho;
#pragma unroll
        for (int i = 0; i < 9; ++i)
            l[i] = ls[i] - av[i] + rb + ((C(EX[i]) - ux) * ubx + (C(EY[i]) - uy) * uby) * ir;
    }
}

template <typename S, bool FORCED>
__global__ __launch_bounds__(256) void k_adj_step(ChanK k, AdjK a, const S* __restrict__ st,
                                                  const S* __restrict__ ln,
                                                  S* __restrict__ l, S mod,
                                                  double* __restrict__ dq_bot,
                                                  double* __restrict__ dq_top,
                                                  double* __restrict__ dtau_acc) {
    using C = S;
    __shared__ double red[2][4];
    const int nx = k.nx, ny = k.ny;
    const int gx = (nx + 63) / 64, gy = (ny + 3) / 4;
    int tile;
    if (!xcd_tile(gx * gy, tile)) return;  // whole workgroup, before the barrier
    const int x = (tile % gx) * 64 + threadIdx.x;
    const int y = (tile / gx) * 4 + threadIdx.y;
    const bool active = x < nx && y < ny;
    const int npl = k.npl;  // node blocks: f 0-8, g 9-13
    double dtn = 0.0, dtt = 0.0;
    if (active) {
        const long long n = (long long)y * nx + x;
        C d[9], e[5], lo[14];
#pragma unroll
        for (int i = 0; i < 9; ++i) d[i] = C(st[bidx(npl, i, n)]);
#pragma unroll
        for (int i = 0; i < 5; ++i) e[i] = C(st[bidx(npl, 9 + i, n)]);
        // node-block positions of the node and its neighbours (wrapped: a value
        // read across a boundary is replaced by that boundary's rule)
        long long at[3][3];
#pragma unroll
        for (int dy = 0; dy < 3; ++dy)
#pragma unroll
            for (int dx = 0; dx < 3; ++dx)
                at[dy][dx] = bidx(npl, 0, (long long)wrap(y + dy - 1, ny) * nx + wrap(x + dx - 1, nx));
        double dqb = 0.0, dqt = 0.0;
        adj_node<FORCED, C>(
            k, a, d, e, x, y, mod, [&](int j) { return C(ln[at[1][1] + j * kBlk]); },
            [&](int i) {
                const int ex = i < 9 ? EX[i] : EX5[i - 9], ey = i < 9 ? EY[i] : EY5[i - 9];
                return C(ln[at[1 + ey][1 + ex] + i * kBlk]);
            },
            [&](int j) { return C(ln[bidx(npl, j, n + 1)]); },
            [&](int s, C& ux2, C& uy2) {
                C d2[9], dr2, r2;
                chan_flow_macros<C, S>(st, npl, n + s, C(k.rho_ref), C(k.Ft[0]), C(k.Ft[1]), d2, dr2, r2,
                                       ux2, uy2);
            },
            lo, dqb, dqt, dtn, dtt);
#pragma unroll
        for (int i = 0; i < 14; ++i) l[bidx(npl, i, n)] = S(lo[i]);
        if (k.bcy && y == 0) dq_bot[x] += dqb;
        if (k.bcy && y == ny - 1) dq_top[x] += dqt;
    }
    // ---- per-tile FP64 sums of the relaxation-time gradients
    const int lane = (threadIdx.y * 64 + threadIdx.x) & 63, wv = threadIdx.y;
    const double sn = wave_sum64(dtn), st_ = wave_sum64(dtt);
    if (lane == 0) {
        red[0][wv] = sn;
        red[1][wv] = st_;
    }
    __syncthreads();
    if (threadIdx.x == 0 && threadIdx.y == 0) {
        dtau_acc[2 * tile] += ((red[0][0] + red[0][1]) + red[0][2]) + red[0][3];
        dtau_acc[2 * tile + 1] += ((red[1][0] + red[1][1]) + red[1][2]) + red[1][3];
    }
}

// Many reverse steps per launch (k_chan_multi's scheme in reverse): a tile with
// an overlap of nsteps nodes, one node per thread, lambda in registers and its
// moving values through LDS; the state of each step is read from the tape a
// step ahead.  st: the state of the first reverse step (the last of the run's
// forward order), stride: from a state to the next one of the tape.  The
// gradients accumulate in registers over the steps: the flux gradient onto the
// column's accumulator in the order of single steps, the relaxation-time
// gradients per node and then per workgroup, tile w's at dtau_acc[2 w].
template <typename S>
struct AdjMultiArgs {
    ChanKT<S> k;
    AdjK a;
    int ntx, nty, wx, ex, wy, ey;  // tile i spans w nodes, one more for i < e
    int nsteps;
    long long stride;
    S mod[kChanMultiMax];  // in the order of the reverse steps
};

template <typename S, bool FORCED, int NT>
__global__ __launch_bounds__(NT) void k_adj_multi(const AdjMultiArgs<S> p, const S* __restrict__ st,
                                                  const S* __restrict__ ln, S* __restrict__ l,
                                                  double* __restrict__ dq_bot,
                                                  double* __restrict__ dq_top,
                                                  double* __restrict__ dtau_acc) {
    using C = S;
    constexpr int NPL = 14;
    __shared__ C buf[2][12][NT];  // lambda_f 1-8, lambda_g 1-4
    __shared__ double red[2][NT / 64];
    const auto& k = p.k;
    const int nx = k.nx, ny = k.ny, h = p.nsteps;
    int w, tx, ty;
    if (!xcd_tile(p.ntx * p.nty, w)) return;  // whole workgroup, before any barrier
    block_divide(w, p.ntx, ty, tx);
    const int x0 = tx * p.wx + min(tx, p.ex), x1 = x0 + p.wx + (tx < p.ex);
    const int y0 = ty * p.wy + min(ty, p.ey), y1 = y0 + p.wy + (ty < p.ey);
    const int rx0 = max(x0 - h, 0), rx1 = min(x1 + h, nx);
    const int ry0 = max(y0 - h, 0), ry1 = min(y1 + h, ny);
    const int rw = rx1 - rx0, rh = ry1 - ry0;
    const int t = threadIdx.x;
    int rx, ry;
    block_divide(t, rw, ry, rx);
    const int x = rx0 + rx, y = ry0 + ry;
    // m: nodes to the nearest edge of the region that cuts through the grid
    int m = 1 << 20;
    if (rx0 > 0) m = min(m, rx);
    if (rx1 < nx) m = min(m, rw - 1 - rx);
    if (ry0 > 0) m = min(m, ry);
    if (ry1 < ny) m = min(m, rh - 1 - ry);
    if (ry >= rh) m = -1;
    const bool own = ry < rh && x >= x0 && x < x1 && y >= y0 && y < y1;
    const long long n = (long long)y * nx + x;
    // LDS offsets to the neighbours (0 across a boundary: its rule replaces the value)
    const int om = x == 0 ? 0 : -1, op = x == nx - 1 ? 0 : 1;
    const int od = y == 0 ? 0 : -rw, ou = y == ny - 1 ? 0 : rw;

    C lam[14], sv[14];
    double dqb = 0.0, dqt = 0.0, dtn = 0.0, dtt = 0.0;
#pragma unroll
    for (int i = 0; i < 14; ++i) {
        lam[i] = m >= 0 ? C(ln[bidx(NPL, i, n)]) : C(0);
        sv[i] = m >= 1 ? C(st[bidx(NPL, i, n)]) : C(0);
    }
    if (own && y == 0) dqb = dq_bot[x];
    if (own && y == ny - 1) dqt = dq_top[x];

    for (int s = 0; s < h; ++s) {
        C(&xb)[12][NT] = buf[s & 1];
        if (m >= s) {
#pragma unroll
            for (int i = 1; i < 9; ++i) xb[i - 1][t] = lam[i];
#pragma unroll
            for (int i = 1; i < 5; ++i) xb[7 + i][t] = lam[9 + i];
        }
        __syncthreads();  // the other buffer's reads ended a step ago
        if (m > s) {
            const S* stc = st + s * p.stride;
            C d[9], e[5], lo[14];
#pragma unroll
            for (int i = 0; i < 9; ++i) d[i] = sv[i];
#pragma unroll
            for (int i = 0; i < 5; ++i) e[i] = sv[9 + i];
            if (s + 1 < h) {
#pragma unroll
                for (int i = 0; i < 14; ++i) sv[i] = C(stc[p.stride + bidx(NPL, i, n)]);
            }
            double b = 0.0, tp = 0.0, an = 0.0, at = 0.0;
            adj_node<FORCED, C>(
                k, p.a, d, e, x, y, p.mod[s], [&](int j) { return lam[j]; },
                [&](int i) {
                    if (i == 0 || i == 9) return lam[i];
                    const int ex = i < 9 ? EX[i] : EX5[i - 9], ey = i < 9 ? EY[i] : EY5[i - 9];
                    return xb[i < 9 ? i - 1 : i - 2][t + (ex < 0 ? om : ex > 0 ? op : 0) +
                                                     (ey < 0 ? od : ey > 0 ? ou : 0)];
                },
                [&](int j) { return xb[j - 1][t + 1]; },
                [&](int sx, C& ux2, C& uy2) {
                    C d2[9], dr2, r2;
                    chan_flow_macros<C, S>(stc, NPL, n + sx, k.rho_ref, k.Ft[0], k.Ft[1], d2, dr2,
                                           r2, ux2, uy2);
                },
                lo, b, tp, an, at);
#pragma unroll
            for (int i = 0; i < 14; ++i) lam[i] = C(S(lo[i]));
            if (own) {
                dqb += b;
                dqt += tp;
                dtn += an;
                dtt += at;
            }
        }
    }
    if (own) {
#pragma unroll
        for (int i = 0; i < 14; ++i) l[bidx(NPL, i, n)] = S(lam[i]);
        if (y == 0) dq_bot[x] = dqb;
        if (y == ny - 1) dq_top[x] = dqt;
    }
    const double sn = wave_sum64(dtn), st_ = wave_sum64(dtt);
    if ((t & 63) == 0) {
        red[0][t >> 6] = sn;
        red[1][t >> 6] = st_;
    }
    __syncthreads();
    if (t < 2) {
        double sum = 0.0;
        for (unsigned i = 0; i < blockDim.x / 64; ++i) sum += red[t][i];
        dtau_acc[2 * w + t] += sum;
    }
}

// Objective J = w_tout T_out + w_nu mean_{x >= x_dev} Nu(x) at the final state
// (definitions as in lbm_nusselt).
// A workgroup takes kSeedCols columns: its threads evaluate the nodes of kSeedRows
// rows at a time into LDS and one thread per column adds them in row order.
constexpr int kSeedCols = 16, kSeedRows = 64;
template <typename S>
__global__ __launch_bounds__(256) void k_adj_seed(
    ChanK k, const S* __restrict__ st, const S* __restrict__ qw, double qsi, double mod, double Dh,
    double kc, double dx, double rho_cp, double cs2, int x_dev, double w_tout, double w_nu,
    S* __restrict__ l, double* __restrict__ dq_direct, double* __restrict__ dtauT_direct) {
    __shared__ double su_[kSeedRows][kSeedCols], sT_[kSeedRows][kSeedCols];
    __shared__ double cb[4][kSeedCols];  // su, T_b, and the adjoints of T_b and T_w
    const int c = threadIdx.x % kSeedCols, r0 = threadIdx.x / kSeedCols;
    const int x = blockIdx.x * kSeedCols + c;
    const int nx = k.nx, ny = k.ny;
    const int npl = k.npl;  // node blocks: f 0-8, g 9-13
    // velocity, density and temperature of a node
    auto node = [&](int y, double& rho, double& ux, double& T) {
        const long long n = (long long)y * nx + x;
        double d[9], drho, uy;
        chan_flow_macros<double, S>(st, npl, n, k.rho_ref, k.Ft[0], k.Ft[1], d, drho, rho, ux,
                                    uy);
        double s = 0;
        for (int i = 0; i < 5; ++i) s += double(st[bidx(npl, 9 + i, n)]);
        T = k.T_ref + s + 0.5 * k.qdt;
    };
    double su = 0, suT = 0, T0 = 0, T1 = 0;
    for (int yb = 0; yb < ny; yb += kSeedRows) {
        const int rows = min(kSeedRows, ny - yb);
        if (x < nx)
            for (int r = r0; r < rows; r += 256 / kSeedCols) {
                double rho;
                node(yb + r, rho, su_[r][c], sT_[r][c]);
            }
        __syncthreads();
        if (r0 == 0)
            for (int r = 0; r < rows; ++r) {
                const double ux = su_[r][c], T = sT_[r][c];
                su += ux * k.c;
                suT += ux * k.c * T;
                if (yb + r == 0) T0 = T;
                if (yb + r == ny - 1) T1 = T;
            }
        __syncthreads();
    }
    if (r0 == 0 && x < nx) {
        const double q = double(qw[x]) * qsi;
        const double tb = suT / su;
        const double dT = 0.5 * (T0 + T1) + q * dx / (2.0 * kc) - tb;
        double bTb = (x == nx - 1) ? w_tout : 0.0, bTw = 0.0, dqd = 0.0, dtd = 0.0;
        if (x >= x_dev) {
            const double nu_x = q * Dh / (kc * dT);
            const double bNu = w_nu / double(nx - x_dev);
            const double bdT = -bNu * nu_x / dT;
            bTw += bdT;
            bTb -= bdT;
            dqd = bNu * mod * Dh / (kc * dT) + bdT * mod * dx / (2.0 * kc);
            dtd = bNu * (-nu_x / kc + (nu_x / dT) * q * dx / (2.0 * kc * kc)) * rho_cp * cs2;
        }
        dq_direct[x] = dqd;
        dtauT_direct[x] = dtd;
        cb[0][c] = su;
        cb[1][c] = tb;
        cb[2][c] = bTb;
        cb[3][c] = bTw;
    }
    __syncthreads();
    if (x >= nx) return;
    su = cb[0][c];
    const double tb = cb[1][c], bTb = cb[2][c], bTw = cb[3][c];
    for (int y = r0; y < ny; y += 256 / kSeedCols) {
        double rho, ux, T;
        node(y, rho, ux, T);
        double Tbar = bTb * ux * k.c / su;
        if (y == 0) Tbar += 0.5 * bTw;
        if (y == ny - 1) Tbar += 0.5 * bTw;
        const double Ubar = bTb * (T - tb) / su * k.c;  // adjoint of u_x / c
        const long long n = (long long)y * nx + x;
        for (int i = 0; i < 5; ++i) l[bidx(npl, 9 + i, n)] = S(Tbar);
        for (int i = 0; i < 9; ++i) l[bidx(npl, i, n)] = S(Ubar * (EX[i] - ux) / rho);
    }
}

// The gradients: the flux gradient per column, and by the last workgroup the
// relaxation-time sums over the tiles and columns (strided partial sums, then a
// tree: a fixed order).
__global__ __launch_bounds__(256) void k_adj_final(
    int nx, int ntiles, double scale, const double* __restrict__ dq_bot,
    const double* __restrict__ dq_top, const double* __restrict__ dq_direct,
    const double* __restrict__ dtauT_direct, const double* __restrict__ dtau_acc,
    double* __restrict__ grad_flux, double* __restrict__ grad_tau) {
    if (blockIdx.x + 1 < gridDim.x) {
        const int t = blockIdx.x * 256 + threadIdx.x;
        if (t < nx) grad_flux[t] = scale * ((dq_bot[t] + dq_top[t]) + dq_direct[t]);
        return;
    }
    __shared__ double part[2][256];
    double sn = 0, st = 0;
    for (int i = threadIdx.x; i < ntiles; i += 256) {
        sn += dtau_acc[2 * i];
        st += dtau_acc[2 * i + 1];
    }
    for (int x = threadIdx.x; x < nx; x += 256) st += dtauT_direct[x];
    part[0][threadIdx.x] = sn;
    part[1][threadIdx.x] = st;
    for (int half = 128; half > 0; half /= 2) {
        __syncthreads();
        if (int(threadIdx.x) < half)
            for (int q = 0; q < 2; ++q) part[q][threadIdx.x] += part[q][threadIdx.x + half];
    }
    if (threadIdx.x < 2) grad_tau[threadIdx.x] = scale * part[threadIdx.x][0];
}

}  // namespace

int chan_tiles(const ChanK& k) { return ((k.nx + 63) / 64) * ((k.ny + 3) / 4); }

template <typename S>
hipError_t launch_adj_seed(const ChanK& k, const S* st, const S* qw, double qsi, double mod,
                           double Dh, double kc, double dx, double rho_cp, double cs2, int x_dev,
                           double w_tout, double w_nu, S* l, double* dq_direct,
                           double* dtauT_direct, hipStream_t s) {
    hipLaunchKernelGGL(k_adj_seed<S>, dim3((k.nx + kSeedCols - 1) / kSeedCols), dim3(256), 0, s, k, st, qw, qsi, mod,
                       Dh, kc, dx, rho_cp, cs2, x_dev, w_tout, w_nu, l, dq_direct, dtauT_direct);
    return hipGetLastError();
}

template <typename S>
hipError_t launch_adj_step(const ChanK& k, const AdjK& a, const S* st, const S* ln, S* l,
                           double mod, double* dq_bot, double* dq_top, double* dtau_acc,
                           hipStream_t s) {
    const int tiles = chan_tiles(k);
    dim3 blk(64, 4), grd(unsigned((tiles + kXCD - 1) / kXCD * kXCD));
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grd, blk, 0, s, k, a, st, ln, l, S(mod), dq_bot, dq_top, dtau_acc);
        return hipGetLastError();
    };
    return k.Ft[0] != 0.0 || k.Ft[1] != 0.0 ? go(k_adj_step<S, true>) : go(k_adj_step<S, false>);
}

template <typename S>
bool adj_multi_fast(const ChanK& k, const ChanMultiPlan& plan) {
    return adj_multi_pays(plan, (chan_multi_region(k, plan, plan.steps) + 63) / 64, sizeof(S));
}

// The many-steps reverse kernel takes the tiles of the channel's plan (the grid
// and its boundaries are the same); up to plan.steps steps per launch.
template <typename S>
hipError_t launch_adj_multi(const ChanK& k, const AdjK& a, const ChanMultiPlan& plan, const S* st,
                            long long stride, const S* ln, S* l, const double* mods, int nsteps,
                            double* dq_bot, double* dq_top, double* dtau_acc, hipStream_t s) {
    const long long nodes = chan_multi_region(k, plan, nsteps);
    if (nsteps < 1 || nsteps > plan.steps || nodes < 1 || nodes > chan_multi_max_nodes(sizeof(S)) ||
        !k.bcx || k.bcy != 1 || k.tq != 5 || k.batch != 1)
        return hipErrorInvalidValue;
    AdjMultiArgs<S> p{};
    p.k = chan_kt<S>(k);
    p.a = a;
    p.ntx = plan.ntx;
    p.nty = plan.nty;
    p.wx = k.nx / plan.ntx;
    p.ex = k.nx % plan.ntx;
    p.wy = k.ny / plan.nty;
    p.ey = k.ny % plan.nty;
    p.nsteps = nsteps;
    p.stride = stride;
    for (int i = 0; i < nsteps; ++i) p.mod[i] = S(mods[i]);
    const unsigned threads = unsigned((nodes + 63) / 64 * 64);
    const int tiles = plan.ntx * plan.nty;
    dim3 grd(unsigned((tiles + kXCD - 1) / kXCD * kXCD)), blk(threads);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, grd, blk, 0, s, p, st, ln, l, dq_bot, dq_top, dtau_acc);
        return hipGetLastError();
    };
    const bool f = k.Ft[0] != 0.0 || k.Ft[1] != 0.0;
    if (threads <= 256) return f ? go(k_adj_multi<S, true, 256>) : go(k_adj_multi<S, false, 256>);
    if (threads <= 512) return f ? go(k_adj_multi<S, true, 512>) : go(k_adj_multi<S, false, 512>);
    if constexpr (sizeof(S) == 4)
        return f ? go(k_adj_multi<S, true, 1024>) : go(k_adj_multi<S, false, 1024>);
    return hipErrorInvalidValue;
}

hipError_t launch_adj_final(int nx, int ntiles, double scale, const double* dq_bot,
                            const double* dq_top, const double* dq_direct,
                            const double* dtauT_direct, const double* dtau_acc, double* grad_flux,
                            double* grad_tau, hipStream_t s) {
    hipLaunchKernelGGL(k_adj_final, dim3((nx + 255) / 256 + 1), dim3(256), 0, s, nx, ntiles, scale,
                       dq_bot, dq_top, dq_direct, dtauT_direct, dtau_acc, grad_flux, grad_tau);
    return hipGetLastError();
}

#define LBM_ADJ_INST(S)                                                                          \
    template hipError_t launch_adj_seed<S>(const ChanK&, const S*, const S*, double, double,     \
                                           double, double, double, double, double, int, double,   \
                                           double, S*, double*, double*, hipStream_t);            \
    template hipError_t launch_adj_step<S>(const ChanK&, const AdjK&, const S*, const S*, S*,    \
                                           double, double*, double*, double*, hipStream_t);     \
    template bool adj_multi_fast<S>(const ChanK&, const ChanMultiPlan&);                          \
    template hipError_t launch_adj_multi<S>(const ChanK&, const AdjK&, const ChanMultiPlan&,      \
                                            const S*, long long, const S*, S*, const double*,     \
                                            int, double*, double*, double*, hipStream_t);
LBM_ADJ_INST(float)
LBM_ADJ_INST(double)

}  // namespace lbm
