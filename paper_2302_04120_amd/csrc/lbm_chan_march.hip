// Several channel steps per launch on grids that fill the GPU (temporal
// blocking): the state crosses HBM once per K steps.
//
// A workgroup of 256 lanes takes one x-tile of one row segment [a, e) of one
// replica: lane l holds column c = (256 - 2 K) t - K + l (modulo nx for periodic
// x; with x ends, lanes whose column lies outside [0, nx) read a clamped column
// and their results are never used).  It marches up the rows; at row step v,
// stage s (0 .. K - 1) collides step n + s at row v - s:
//   - the x-moving values (and u, for the outlet's wall velocity) go to the
//     neighbour lanes through LDS;
//   - each lane pulls the state of step n + s + 1: the values that move down
//     complete row v - s - 1, which the next stage collides at once; the values
//     that stay in row v - s start it (W), those that move up wait for the next
//     row (U).  W and U of every stage stay in registers: 18 values (D2Q5
//     temperature) per stage.
// The last stage's completed row is stored, aligned.  Stage s is exact on lanes
// s .. 255 - s and runs on rows a - (K - s) .. e + (K - s) - 1 (those that
// exist), so tiles and segments are independent.  The boundary rules are those
// of k_chan_step, and so is the arithmetic per node (chan_th, chan_collide and
// the boundary values): K steps here equal K single steps bit for bit.
//
// Every stage has one LDS buffer and one barrier per row: with K >= 2 another
// stage's barrier lies between a buffer's reads and its next writes.
//
// ALIGNED: nx a multiple of 64 and a row's node blocks under 2 GiB, so every
// row starts on a node block and an access is the row's block base (uniform)
// plus a 32-bit lane offset.  ENDS: the code for the cavity's end walls and the
// symmetry plane is compiled in.
#include "lbm_channel.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace lbm {
namespace {

constexpr int kMarchLanes = 256;
constexpr int march_nv(int qt) { return 9 + qt; }
// LDS planes of a stage: flow x movers, thermal x movers 1 and 3, u, thermal diagonals
constexpr int march_x(int qt) { return qt == 9 ? 14 : 10; }

template <typename C, int K>
struct ChanMarchArgs {
    ChanKT<C> k;
    int ntx, nseg, wy, ey;  // tiles per row; segment i spans wy rows, one more for i < ey
    C mod[K];               // wall-flux modulation of each step
};

template <typename S, bool ALIGNED, bool ENDS, int QT, int K>
__global__ __launch_bounds__(kMarchLanes) void k_chan_march(const ChanMarchArgs<S, K> p,
                                                         const S* __restrict__ A,
                                                         S* __restrict__ B,
                                                         const S* __restrict__ qw,
                                                         const S* __restrict__ uin,
                                                         const S* __restrict__ tin) {
    using C = S;
    constexpr int NV = march_nv(QT), G = 9, NU = QT == 9 ? 6 : 4;
    __shared__ C xch[K][march_x(QT)][kMarchLanes];
    const auto& k = p.k;
    const int nx = k.nx, ny = k.ny;
    int w, tx, sg, b;
    if (!xcd_tile(p.ntx * p.nseg * k.batch, w)) return;  // whole workgroup, before any barrier
    block_divide(w, p.ntx, w, tx);  // x fastest
    block_divide(w, p.nseg, b, sg);
    const int a = sg * p.wy + min(sg, p.ey), e = a + p.wy + (sg < p.ey);
    const bool walls = k.bcy != 0;         // y ends: a wall at y-, a wall or the symmetry plane at y+
    const bool symy = ENDS && k.bcy == 2;  // the symmetry plane of Eq. simetria at y+
    const bool xends = k.bcx != 0;         // x not periodic
    const bool io = ENDS ? k.bcx == 1 : xends;  // velocity inlet (left), pressure outlet (right)
    const bool xw = ENDS && k.bcx == 2;    // fixed-temperature no-slip walls at both ends
    const long long base = (long long)b * ny * nx;
    const unsigned lx = threadIdx.x;
    const int col = tx * (kMarchLanes - 2 * K) - K + int(lx);
    int xi = col;
    if (xends) {
        xi = min(max(col, 0), nx - 1);
    } else {
        while (xi < 0) xi += nx;
        while (xi >= nx) xi -= nx;
    }
    const unsigned x = unsigned(xi);
    const bool own = int(lx) >= K && int(lx) < kMarchLanes - K && col < nx;
    const bool x_lo = xends && col == 0, x_hi = xends && col == nx - 1;  // the end columns
    const bool at_in = io && x_lo, at_out = io && x_hi;
    const unsigned lxm = lx == 0 ? 0u : lx - 1, lxp = lx == kMarchLanes - 1 ? lx : lx + 1;
    const C rho_ref = k.rho_ref, qdt = k.qdt, q = C(qw[x]), tw_lo = k.Tw[0], tw_hi = k.Tw[1];

    // memory row of virtual row v: rows of a periodic segment lie in [-K, ny + K)
    auto rowof = [&](int v) {
        while (v < 0) v += ny;
        while (v >= ny) v -= ny;
        return v;
    };
    const unsigned boff =
        ALIGNED ? unsigned(((x >> 6) * NV * kBlk + (x & (kBlk - 1))) * sizeof(S)) : x;
    auto at = [&](auto* P, int row, int i) {
        const long long ro = base + (long long)row * nx;
        if constexpr (ALIGNED) {
            using B8 = std::conditional_t<std::is_const_v<std::remove_pointer_t<decltype(P)>>,
                                          const char, char>;
            auto* r = (B8*)P + (ro >> 6) * (long long)(NV * kBlk * sizeof(S));
            return (decltype(P))(r + boff) + i * kBlk;
        } else {
            return P + bidx(NV, i, ro + boff);
        }
    };

    // W: the state of each stage's last row so far; U: the values that move up from it
    C W[K][NV], U[K][NU];
#pragma unroll
    for (int s = 0; s < K; ++s) {
#pragma unroll
        for (int i = 0; i < NV; ++i) W[s][i] = C(0);
#pragma unroll
        for (int i = 0; i < NU; ++i) U[s][i] = C(0);
    }
    const int first = walls ? max(a - K, 0) : a - K, last = walls ? min(e + K, ny) : e + K;

    C N[NV];  // the next row
    int rn = rowof(first);
    auto load_next = [&] {
#pragma unroll
        for (int i = 0; i < NV; ++i) N[i] = C(*at(A, rn, i));
    };
    // The next row is loaded a row step ahead where that was measured to pay: 8192 x
    // 1024 FP32 K = 4 67.6 -> 65.1 us a step (D2Q9 set 106 -> 96), FP64 D2Q9 K = 3 296
    // -> 259.  At K = 2 the launch runs at HBM's rate either way (FP32 109 -> 112, D2Q9
    // set 137 -> 147), and two K = 3 instances would lose a wave per SIMD to the
    // registers.
    constexpr bool AHEAD = sizeof(S) == 4 ? K == 4 || (K == 3 && QT == 5) : QT == 9;
    if constexpr (AHEAD) load_next();

    for (int v = first; v < e + K; ++v) {
        C T[NV];  // the row the next stage collides
        if constexpr (!AHEAD) load_next();
#pragma unroll
        for (int i = 0; i < NV; ++i) T[i] = N[i];
        if (v + 1 < last) rn = rn + 1 == ny ? 0 : rn + 1;  // else re-reads the last row
        if constexpr (AHEAD) load_next();
#pragma unroll
        for (int s = 0; s < K; ++s) {
            const int r = v - s;
            const int lo = walls ? max(a - (K - s), 0) : a - (K - s);
            const int hi = walls ? min(e + (K - s), ny) : e + (K - s);
            const bool on = r >= lo && r < hi;
            C(&xb)[march_x(QT)][kMarchLanes] = xch[s];
            C ds[9], es[QT], ux = C(0), uy = C(0);
            if (on) {
                C d[9], g[QT], drho, rho, ftx, fty;
#pragma unroll
                for (int i = 0; i < 9; ++i) d[i] = T[i];
#pragma unroll
                for (int i = 0; i < QT; ++i) g[i] = T[G + i];
                const C th = chan_th<QT, C>(g, qdt);
                chan_force(k, th, ftx, fty);
                chan_flow_macros_v<C>(d, rho_ref, ftx, fty, drho, rho, ux, uy);
                chan_collide<C, QT>(k, d, drho, rho, ux, uy, ftx, fty, g, th, qdt, ds, es);
                xb[0][lx] = ds[1];
                xb[1][lx] = ds[3];
                xb[2][lx] = ds[5];
                xb[3][lx] = ds[6];
                xb[4][lx] = ds[7];
                xb[5][lx] = ds[8];
                xb[6][lx] = es[1];
                xb[7][lx] = es[3];
                if (io) {
                    xb[8][lx] = ux;
                    xb[9][lx] = uy;
                }
                if constexpr (QT == 9) {
                    xb[10][lx] = es[5];
                    xb[11][lx] = es[6];
                    xb[12][lx] = es[7];
                    xb[13][lx] = es[8];
                }
            }
            __syncthreads();
            C(&Ws)[NV] = W[s];
            C(&Us)[NU] = U[s];
            if (on) {  // row r - 1 receives the values that move down
                Ws[4] = ds[4];
                Ws[7] = x_hi ? Ws[7] : xb[4][lxp];
                Ws[8] = x_lo ? Ws[8] : xb[5][lxm];
                Ws[G + 4] = es[4];
                if constexpr (QT == 9) {
                    Ws[G + 7] = (x_hi && xw) ? Ws[G + 7] : at_out ? es[7] : xb[12][lxp];
                    Ws[G + 8] = x_lo ? Ws[G + 8] : xb[13][lxm];
                }
            }
#pragma unroll
            for (int i = 0; i < NV; ++i) T[i] = Ws[i];
            if (!on) continue;
            // ---- the state of row r so far
            const bool top = k.bcy == 1 && r == ny - 1, bottom = walls && r == 0;
            const bool stop = symy && r == ny - 1;  // top row under the symmetry plane
            const C mod = p.mod[s];
            Ws[0] = ds[0];
            Ws[1] = xb[0][lxm];
            Ws[3] = xb[1][lxp];
            Ws[2] = Us[0];
            Ws[5] = Us[1];
            Ws[6] = Us[2];
            Us[0] = ds[2];
            Us[1] = xb[2][lxm];
            Us[2] = xb[3][lxp];
            Ws[G + 0] = es[0];
            Ws[G + 1] = xb[6][lxm];
            // outlet extrapolation: the value the left neighbour receives, the node's own
            Ws[G + 3] = at_out ? es[3] : xb[7][lxp];
            Ws[G + 2] = Us[3];
            Us[3] = es[2];
            if constexpr (QT == 9) {
                Ws[G + 5] = Us[4];
                Ws[G + 6] = Us[5];
                Us[4] = xb[10][lxm];
                Us[5] = at_out ? es[6] : xb[11][lxp];
            }
            if (stop) {  // +y movers come back mirrored at x + c_x (Eq. simetria)
                Ws[4] = ds[2];
                Ws[7] = xb[3][lxp];
                Ws[8] = xb[2][lxm];
                Ws[G + 4] = es[2];
                if constexpr (QT == 9) {
                    Ws[G + 7] = at_out ? es[6] : xb[11][lxp];
                    Ws[G + 8] = xb[10][lxm];
                }
            }
            if (x_lo || x_hi) {
                C uwx = C(0), uwy = C(0), u_in = C(0);
                const int y = rowof(r);
                if (io) {
                    u_in = C(uin[y]);
                    uwx = C(1.5) * ux - C(0.5) * xb[8][lxm];
                    uwy = C(1.5) * uy - C(0.5) * xb[9][lxm];
                }
                if (x_lo) {  // an end wall (xw) bounces back like the y walls
                    Ws[1] = io ? chan_inlet_f<C>(3, ds[3], rho_ref, u_in) : ds[3];
                    Ws[5] = io ? chan_inlet_f<C>(7, ds[7], rho_ref, u_in) : ds[7];
                    Ws[8] = io ? chan_inlet_f<C>(6, ds[6], rho_ref, u_in) : ds[6];
                    // the inlet temperature where the link crosses the inlet
                    const C t0 = io ? C(0.5) * (C(tin[y]) + C(tin[y])) : tw_lo;
                    Ws[G + 1] = chan_antibb_g<QT, C>(3, es[3], t0);
                    if constexpr (QT == 9) {
                        const C tp = !io ? tw_lo
                                     : y + 1 < ny ? C(0.5) * (C(tin[y]) + C(tin[y + 1])) : C(tin[y]);
                        const C tm = !io ? tw_lo
                                     : y - 1 >= 0 ? C(0.5) * (C(tin[y]) + C(tin[y - 1])) : C(tin[y]);
                        Ws[G + 8] = chan_antibb_g<QT, C>(6, es[6], tp);
                        Ws[G + 5] = chan_antibb_g<QT, C>(7, es[7], tm);
                    }
                }
                if (x_hi) {
                    Ws[3] = io ? chan_outlet_f<C>(1, ds[1], rho_ref, uwx, uwy) : ds[1];
                    Ws[7] = io ? chan_outlet_f<C>(5, ds[5], rho_ref, uwx, uwy) : ds[5];
                    Ws[6] = io ? chan_outlet_f<C>(8, ds[8], rho_ref, uwx, uwy) : ds[8];
                    if (xw) {
                        Ws[G + 3] = chan_antibb_g<QT, C>(1, es[1], tw_hi);
                        if constexpr (QT == 9) {
                            Ws[G + 7] = chan_antibb_g<QT, C>(5, es[5], tw_hi);
                            Ws[G + 6] = chan_antibb_g<QT, C>(8, es[8], tw_hi);
                        }
                    }
                }
            }
            if (bottom) {
                Ws[2] = ds[4];
                Ws[5] = ds[7];
                Ws[6] = ds[8];
                Ws[G + 2] = chan_flux_g<QT, C>(4, es[4], q, mod);
                if constexpr (QT == 9) {
                    Ws[G + 5] = chan_flux_g<QT, C>(7, es[7], q, mod);
                    Ws[G + 6] = chan_flux_g<QT, C>(8, es[8], q, mod);
                }
            }
            if (top) {
                Ws[4] = ds[2];
                Ws[7] = ds[5];
                Ws[8] = ds[6];
                Ws[G + 4] = chan_flux_g<QT, C>(2, es[2], q, mod);
                if constexpr (QT == 9) {
                    Ws[G + 7] = chan_flux_g<QT, C>(5, es[5], q, mod);
                    Ws[G + 8] = chan_flux_g<QT, C>(6, es[6], q, mod);
                }
            }
        }
        // the loads end here, so that they do not wait for the stores below
#pragma unroll
        for (int i = 0; AHEAD && i < NV; ++i) asm volatile("" : "+v"(N[i]));
        const int r = v - K;
        if (own && r >= a) {  // complete: r < e by the loop's end
#pragma unroll
            for (int i = 0; i < NV; ++i) st(at(B, r, i), S(T[i]));
        }
    }
}

template <typename S>
bool march_aligned(const ChanK& k) {
    return k.nx % kBlk == 0 && (long long)k.nx * march_nv(k.tq) * (long long)sizeof(S) < (1LL << 31);
}

// The instance for a configuration (FP64 up to three steps: four fill the LDS).
template <typename S, int K>
auto march_kernel(const ChanK& k) {
    const bool ends = k.bcx == 2 || k.bcy == 2;
    if (k.tq == 9) {
        if (march_aligned<S>(k))
            return ends ? k_chan_march<S, true, true, 9, K> : k_chan_march<S, true, false, 9, K>;
        return ends ? k_chan_march<S, false, true, 9, K> : k_chan_march<S, false, false, 9, K>;
    }
    if (march_aligned<S>(k))
        return ends ? k_chan_march<S, true, true, 5, K> : k_chan_march<S, true, false, 5, K>;
    return ends ? k_chan_march<S, false, true, 5, K> : k_chan_march<S, false, false, 5, K>;
}

template <typename S, int K>
hipError_t march_launch(const ChanK& k, const S* a, S* b, const S* qw, const S* uin, const S* tin,
                        const double* mods, int nseg, hipStream_t s) {
    const int ntx = chan_march_tiles(k, K);
    const long long wgs = (long long)ntx * nseg * k.batch;
    if (nseg < 1 || nseg > k.ny || wgs >= (1 << 21)) return hipErrorInvalidValue;
    ChanMarchArgs<S, K> p{};
    p.k = chan_kt<S>(k);
    p.ntx = ntx;
    p.nseg = nseg;
    p.wy = k.ny / nseg;
    p.ey = k.ny % nseg;
    for (int i = 0; i < K; ++i) p.mod[i] = S(mods[i]);
    hipLaunchKernelGGL((march_kernel<S, K>(k)), dim3(unsigned((wgs + kXCD - 1) / kXCD * kXCD)),
                       dim3(kMarchLanes), 0, s, p, a, b, qw, uin, tin);
    return hipGetLastError();
}

}  // namespace

int chan_march_tiles(const ChanK& k, int K) {
    return (k.nx + kMarchLanes - 2 * K - 1) / (kMarchLanes - 2 * K);
}

// The marching kernel covers flow with temperature (D2Q5 or the D2Q9 set, with
// or without the Boussinesq force) and every boundary of the channel lattice.
bool chan_march_fits(const ChanK& k) {
    return k.flow && k.thermal && (k.tq == 5 || k.tq == 9) && k.npl == march_nv(k.tq) &&
           k.bcx >= 0 && k.bcx <= 2 && k.bcy >= 0 && k.bcy <= 2 && k.nx >= 2 && k.ny >= 2;
}

// Steps per launch and segments by a cost model fitted to 1300 plans on 15
// channels of 32 k to 17 M nodes (10 %; its choice runs within 15 % of the best
// measured plan).  All workgroups of a round march seg + 2 K rows; a row step is
// the root sum square of
//   the stages' time: row0 + K lam for one workgroup on a CU (the chain of a
//   row), or K beta for each of the w workgroups of a CU (issue), and
//   the bytes of the resident workgroups at 12 to 13 TB/s out of the caches, or 5.7
//   to 7.7 TB/s where both buffers outgrow the 256 MB memory-side cache.
// Measured per step, single step -> K of the plan: 8192 x 1024 FP32 182 -> 65 us
// (K = 4; two steps in the scheme this replaces, which accumulated three rows
// of the next state in registers: 112), with the D2Q9 set 238 -> 97, FP64 325
// -> 145, FP64 with the D2Q9 set 427 -> 260 (2500 x 700 92 -> 63, 3000 x 300 42 ->
// 35); 4000 x 500 FP32 45 -> 21; 1003 x 701 FP64 29 -> 20.  Smaller grids go through the many-steps kernel.
template <typename S>
MarchPlan chan_march_plan(const ChanK& k) {
    MarchPlan best{};
    int dev = 0, cus = 0;
    if (!chan_march_fits(k) || hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        return best;
    constexpr bool F32 = sizeof(S) == 4;
    struct Cost { double t0, lam, row0, beta, near, far; };  // us, and bytes per us
    const Cost c = F32 ? (k.tq == 9 ? Cost{0.5, 0.72, 1.30, 0.225, 12e6, 6.2e6}
                                    : Cost{0.5, 0.55, 1.0, 0.25, 12e6, 5.7e6})
                       : (k.tq == 9 ? Cost{3.7, 1.37, 0.37, 0.82, 13.4e6, 7.7e6}
                                    : Cost{0.5, 0.69, 1.37, 0.43, 12e6, 6.7e6});
    const double row_bytes = 2.0 * kMarchLanes * k.npl * sizeof(S);
    const double state = double(k.nx) * k.ny * k.batch * k.npl * sizeof(S);
    const double bw = 2 * state < 3e8 ? c.near : c.far;
    for (int K = 2; K <= (F32 ? 4 : 3); ++K) {
        const int resident = K == 2   ? resident_workgroups((const void*)march_kernel<S, 2>(k), 4)
                             : K == 3 ? resident_workgroups((const void*)march_kernel<S, 3>(k), 4)
                                      : resident_workgroups((const void*)march_kernel<S, F32 ? 4 : 3>(k), 4);
        if (resident < 1) continue;
        const long long column = (long long)chan_march_tiles(k, K) * k.batch, cap = (long long)cus * resident;
        for (int seg = k.ny; seg >= 1; --seg) {
            const int nseg = (k.ny + seg - 1) / seg;
            if (seg > 1 && (k.ny + seg - 2) / (seg - 1) == nseg) continue;  // shorter, the same count
            const long long wgs = column * nseg;
            if (wgs >= (1 << 21)) break;
            auto row = [&](long long n) {
                const double t = std::max(c.row0 + K * c.lam, K * c.beta * double((n + cus - 1) / cus));
                return std::hypot(t, row_bytes * double(n) / bw);
            };
            const double cost = (c.t0 + (seg + 2 * K) * (double(wgs / cap) * row(cap) +
                                                        (wgs % cap ? row(wgs % cap) : 0.0))) / K;
            if (best.steps == 0 || cost < best.cost) best = MarchPlan{K, nseg, cost};
        }
    }
    return best;
}

template <typename S>
hipError_t launch_chan_march(const ChanK& k, int K, const S* a, S* b, const S* qw, const S* uin,
                             const S* tin, const double* mods, int nseg, hipStream_t s) {
    if (!chan_march_fits(k)) return hipErrorInvalidValue;
    if (K == 2) return march_launch<S, 2>(k, a, b, qw, uin, tin, mods, nseg, s);
    if (K == 3) return march_launch<S, 3>(k, a, b, qw, uin, tin, mods, nseg, s);
    if constexpr (sizeof(S) == 4)
        if (K == 4) return march_launch<S, 4>(k, a, b, qw, uin, tin, mods, nseg, s);
    return hipErrorInvalidValue;
}

#define LBM_MARCH_INST(S)                                                                          \
    template MarchPlan chan_march_plan<S>(const ChanK&);                                       \
    template hipError_t launch_chan_march<S>(const ChanK&, int, const S*, S*, const S*, const S*,  \
                                             const S*, const double*, int, hipStream_t);
LBM_MARCH_INST(float)
LBM_MARCH_INST(double)

}  // namespace lbm
