// Many channel steps per launch for grids that do not fill the GPU.
//
// A paper-sized channel (800 x 40 nodes) holds 125 nodes per CU: a launch of
// the single-step kernel is a chain of one memory round trip, one collision
// and one store behind the gap between two dependent launches, 5 us whatever
// the node count.  Here a workgroup takes a tile of the grid with an overlap
// of K nodes on every side that is not a boundary of the domain, keeps one
// node per thread in registers for K steps, and exchanges only the moving
// post-collision values through LDS, so that the launch, the load and the
// store are paid once per K steps.  The price is the overlap, which several
// tiles collide, and it is free while SIMDs would idle.
//
// Per node the arithmetic is that of k_chan_step (chan_th, chan_collide and
// the boundary values), so the states agree to the last bit.
#include "lbm_channel.h"

#include <algorithm>

namespace lbm {
namespace {

template <typename C>
struct ChanMultiArgs {
    ChanKT<C> k;
    int ntx, nty;         // tiles per replica
    int wx, ex, wy, ey;   // tile i spans w nodes, one more for i < e
    int nsteps;           // steps of this launch = overlap of the tiles
    long long tape;       // 0: store the last state into B; else every step's state, at B + s tape
    C mod[kChanMultiMax];  // wall-flux modulation of each step
};

// LDS planes of one step: flow movers 1-8, thermal movers 1 .. QT - 1, u.
constexpr int cm_planes(int qt) { return 8 + (qt - 1) + 2; }
// Two sets of planes (one barrier per step) where they fit, else one set and
// a second barrier.
template <typename S, int QT, int NT>
constexpr int cm_sets() {
    return 2 * cm_planes(QT) * NT * int(sizeof(S)) <= 160 * 1024 ? 2 : 1;
}

__device__ __forceinline__ int cm_wrap(int v, int n) {
    while (v < 0) v += n;
    while (v >= n) v -= n;
    return v;
}

template <typename S, int QT, int NT>
__global__ __launch_bounds__(NT) void k_chan_multi(const ChanMultiArgs<S> p, const S* __restrict__ A,
                                                   S* __restrict__ B, const S* __restrict__ qw,
                                                   const S* __restrict__ uin,
                                                   const S* __restrict__ tin) {
    using C = S;
    constexpr int NV = 9 + QT, G = 7 /* plane of thermal mover i: G + i */, U = 8 + QT - 1;
    constexpr int SETS = cm_sets<S, QT, NT>();
    __shared__ C buf[SETS][cm_planes(QT)][NT];
    const auto& k = p.k;
    const int nx = k.nx, ny = k.ny, h = p.nsteps;
    int w;
    if (!xcd_tile(p.ntx * p.nty * k.batch, w)) return;  // whole workgroup, before any barrier
    int tx, ty, b;
    block_divide(w, p.ntx, w, tx);
    block_divide(w, p.nty, b, ty);
    const bool xends = k.bcx != 0, yends = k.bcy != 0, io = k.bcx == 1;
    // the tile's own nodes [x0, x1) x [y0, y1) and its region with the overlap
    const int x0 = tx * p.wx + min(tx, p.ex), x1 = x0 + p.wx + (tx < p.ex);
    const int y0 = ty * p.wy + min(ty, p.ey), y1 = y0 + p.wy + (ty < p.ey);
    const int rx0 = xends ? max(x0 - h, 0) : x0 - h, rx1 = xends ? min(x1 + h, nx) : x1 + h;
    const int ry0 = yends ? max(y0 - h, 0) : y0 - h, ry1 = yends ? min(y1 + h, ny) : y1 + h;
    const int rw = rx1 - rx0, rh = ry1 - ry0;
    const int t = threadIdx.x;
    int rx, ry;
    block_divide(t, rw, ry, rx);
    const int vx = rx0 + rx, vy = ry0 + ry;
    const int x = xends ? vx : cm_wrap(vx, nx), y = yends ? vy : cm_wrap(vy, ny);
    // m: nodes between this one and the nearest edge of the region that cuts
    // through the grid.  The node's state is known for the steps s <= m.
    int m = 1 << 20;
    if (!(xends && rx0 == 0)) m = min(m, rx);
    if (!(xends && rx1 == nx)) m = min(m, rw - 1 - rx);
    if (!(yends && ry0 == 0)) m = min(m, ry);
    if (!(yends && ry1 == ny)) m = min(m, rh - 1 - ry);
    if (ry >= rh) m = -1;
    const bool own = ry < rh && vx >= x0 && vx < x1 && vy >= y0 && vy < y1;

    const bool xlo = xends && x == 0, xhi = xends && x == nx - 1;
    const bool ylo = yends && y == 0, yhi = yends && y == ny - 1;
    const bool wtop = yhi && k.bcy == 1, stop = yhi && k.bcy == 2;  // wall, symmetry plane
    const bool edge = xlo || xhi || ylo || wtop;
    // LDS offsets to the neighbours a value comes from (0 across a boundary)
    const int om = xlo ? 0 : -1, op = xhi ? 0 : 1, od = ylo ? 0 : -rw, ou = yhi ? 0 : rw;
    const long long n = ((long long)b * ny + y) * nx + x;
    C f[9], g[QT];
    C q = C(0), u_in = C(0), tw_in[3] = {C(0), C(0), C(0)};
    if (m >= 0) {
#pragma unroll
        for (int i = 0; i < 9; ++i) f[i] = A[bidx(NV, i, n)];
#pragma unroll
        for (int i = 0; i < QT; ++i) g[i] = A[bidx(NV, 9 + i, n)];
        if (edge) {
            q = qw[x];
            if (io && xlo) {
                u_in = uin[y];
#pragma unroll
                for (int c = -1; c <= 1; ++c)  // the inlet temperature of a link with c_y = c
                    tw_in[c + 1] = y + c >= 0 && y + c < ny ? C(0.5) * (C(tin[y]) + C(tin[y + c]))
                                                            : C(tin[y]);
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < 9; ++i) f[i] = C(0);
#pragma unroll
        for (int i = 0; i < QT; ++i) g[i] = C(0);
    }

    for (int s = 0; s < p.nsteps; ++s) {
        C(&xb)[cm_planes(QT)][NT] = buf[SETS == 2 ? (s & 1) : 0];
        C ds[9], es[QT], ux = C(0), uy = C(0);
        if (m >= s) {
            const C th = chan_th<QT, C>(g, k.qdt);
            C ftx, fty, drho, rho;
            chan_force(k, th, ftx, fty);
            chan_flow_macros_v<C>(f, k.rho_ref, ftx, fty, drho, rho, ux, uy);
            chan_collide<C, QT>(k, f, drho, rho, ux, uy, ftx, fty, g, th, k.qdt, ds, es);
#pragma unroll
            for (int i = 1; i < 9; ++i) xb[i - 1][t] = ds[i];
#pragma unroll
            for (int i = 1; i < QT; ++i) xb[G + i][t] = es[i];
            if (io) {
                xb[U][t] = ux;
                xb[U + 1][t] = uy;
            }
        }
        __syncthreads();
        if (m > s) {
            // streaming: each value from the node it leaves, the boundary
            // rules of k_chan_step where that lies outside
            f[0] = ds[0];
            g[0] = es[0];
#pragma unroll
            for (int i = 1; i < 9; ++i)
                f[i] = xb[i - 1][t + (EX[i] > 0 ? om : EX[i] < 0 ? op : 0) +
                                 (EY[i] > 0 ? od : EY[i] < 0 ? ou : 0)];
            // at the outlet column this is also the thermal extrapolation: the
            // offset op is 0 there, the value its left neighbour receives
#pragma unroll
            for (int i = 1; i < QT; ++i)
                g[i] = xb[G + i][t + (tex<QT>(i) > 0 ? om : tex<QT>(i) < 0 ? op : 0) +
                                 (tey<QT>(i) > 0 ? od : tey<QT>(i) < 0 ? ou : 0)];
            if (stop) {  // mirrored +y movers of the top row (Eq. simetria)
#pragma unroll
                for (int i = 1; i < 9; ++i)
                    if (EY[i] < 0)
                        f[i] = xb[MIRY[i] - 1][t + (EX[i] > 0 ? om : EX[i] < 0 ? op : 0)];
#pragma unroll
                for (int i = 1; i < QT; ++i)
                    if (tey<QT>(i) < 0)
                        g[i] = xb[G + tmir<QT>(i)][t + (tex<QT>(i) > 0 ? om : tex<QT>(i) < 0 ? op : 0)];
            }
            if (edge) {
                const C mod = p.mod[s];
                C uwx = C(0), uwy = C(0);
                if (io && xhi) {
                    uwx = C(1.5) * ux - C(0.5) * xb[U][t - 1];
                    uwy = C(1.5) * uy - C(0.5) * xb[U + 1][t - 1];
                }
#pragma unroll
                for (int j = 1; j < 9; ++j) {
                    const int i = OPP[j];  // the population that left, into slot j
                    const bool outy = EY[i] < 0 ? ylo : EY[i] > 0 ? wtop : false;
                    const bool outx = EX[i] < 0 ? xlo : EX[i] > 0 ? xhi : false;
                    if (outy || (outx && !io))
                        f[j] = ds[i];
                    else if (outx && EX[i] < 0)
                        f[j] = chan_inlet_f<C>(i, ds[i], k.rho_ref, u_in);
                    else if (outx)
                        f[j] = chan_outlet_f<C>(i, ds[i], k.rho_ref, uwx, uwy);
                }
#pragma unroll
                for (int j = 1; j < QT; ++j) {
                    const int i = topp<QT>(j);
                    const bool outy = tey<QT>(i) < 0 ? ylo : tey<QT>(i) > 0 ? wtop : false;
                    const bool outx = tex<QT>(i) < 0 ? xlo : tex<QT>(i) > 0 ? xhi : false;
                    if (outy)
                        g[j] = chan_flux_g<QT, C>(i, es[i], q, mod);
                    else if (outx && !io)
                        g[j] = chan_antibb_g<QT, C>(i, es[i], k.Tw[tex<QT>(i) < 0 ? 0 : 1]);
                    else if (outx && tex<QT>(i) < 0)
                        g[j] = chan_antibb_g<QT, C>(i, es[i], tw_in[tey<QT>(i) + 1]);
                }
            }
        }
        if (own && (p.tape != 0 || s == p.nsteps - 1)) {
            S* out = B + (long long)s * p.tape;
#pragma unroll
            for (int i = 0; i < 9; ++i) out[bidx(NV, i, n)] = S(f[i]);
#pragma unroll
            for (int i = 0; i < QT; ++i) out[bidx(NV, 9 + i, n)] = S(g[i]);
        }
        if constexpr (SETS == 1) __syncthreads();  // this step's reads end before the next writes
    }
}

// Largest workgroup (nodes of a region): 1024 threads in FP32, 512 in FP64,
// whose LDS planes take twice the space.
template <typename S>
constexpr int cm_max_nodes() {
    return chan_multi_max_nodes(sizeof(S));
}

}  // namespace

namespace {

// Span of the widest tile's region on an axis: ceil(n / tiles) nodes and the
// overlap, which a boundary of the grid ends on the first and the last tile.
long long cm_span(int n, int tiles, int h, bool ends) {
    const long long w = (n + tiles - 1) / tiles;
    if (!ends) return w + 2 * h;
    return std::min<long long>(n, w + (tiles == 1 ? 0 : tiles == 2 ? h : 2 * h));
}
long long cm_region(const ChanK& k, int ntx, int nty, int h) {
    return cm_span(k.nx, ntx, h, k.bcx != 0) * cm_span(k.ny, nty, h, k.bcy != 0);
}

}  // namespace

long long chan_multi_region(const ChanK& k, const ChanMultiPlan& p, int h) {
    return p.ntx > 0 && p.nty > 0 ? cm_region(k, p.ntx, p.nty, h) : 0;
}

namespace {

// The kernel instance for a workgroup of that many threads.
template <typename S>
auto cm_kernel(int qt, int threads) {
    if constexpr (sizeof(S) == 4)
        if (threads > 512) return qt == 9 ? k_chan_multi<S, 9, 1024> : k_chan_multi<S, 5, 1024>;
    if (threads > 256) return qt == 9 ? k_chan_multi<S, 9, 512> : k_chan_multi<S, 5, 512>;
    return qt == 9 ? k_chan_multi<S, 9, 256> : k_chan_multi<S, 5, 256>;
}

}  // namespace

// Tiles and steps per launch, by a cost model fitted to 1200 plans on 14
// channels of 4 k to 2 M nodes (it predicts them to 9 %, and its choice runs
// within 1-15 % of the best measured plan of each channel):
//   launch = T0 + T1 (rounds - 1) + steps sum over rounds (a + b W)
// in microseconds, W the waves per SIMD of the busiest CU in a round (at
// least 1) and rounds the number of times the workgroups fill the GPU.  T0 is
// the launch gap with the load and the store, b the issue time of one wave's
// step.  More steps per launch share T0 but widen the overlap, so W grows.
// A plan is taken where it saves at least 15 % of the single step
// (chan_single_cost).  Measured per step, single -> plan: 800 x 40
// FP32 5.2 -> 1.7 us, 1600 x 80 6.5 -> 2.6, 2000 x 50 with the D2Q9 thermal
// set 8.0 -> 3.1, 65 x 65 cavity FP64 5.6 -> 2.7, 3000 x 300 22.2 -> 13.8.
template <typename S>
ChanMultiPlan chan_multi_plan(const ChanK& k) {
    ChanMultiPlan best{};
    if (!chan_march_fits(k)) return best;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        return best;
    struct Cost { double t0, t1, a, b; };
    const Cost c = sizeof(S) == 4 ? (k.tq == 9 ? Cost{5.3, 2.0, 0.32, 0.40} : Cost{4.7, 2.0, 0.39, 0.21})
                                  : (k.tq == 9 ? Cost{5.6, 2.5, 0.51, 0.76} : Cost{4.8, 1.8, 0.48, 0.48});
    constexpr int kWaves = cm_max_nodes<S>() / 64;
    int resident[kWaves + 1] = {};  // workgroups of that many waves per CU
    for (int wv = 1; wv <= kWaves; ++wv)
        resident[wv] = resident_workgroups((const void*)cm_kernel<S>(k.tq, wv * 64), wv);
    const double bytes = double(k.nx) * k.ny * k.batch * k.npl * sizeof(S) * 2;
    double best_cost = 0.85 * chan_single_cost(bytes);
    for (int h = 2; h <= 10; ++h)
        for (int nty = 1; nty <= std::min(k.ny, 512); ++nty) {
            // one plan per height of the widest tile: the fewest tiles of it
            if (nty > 1 && (k.ny + nty - 1) / nty == (k.ny + nty - 2) / (nty - 1)) continue;
            const long long rh = cm_span(k.ny, nty, h, k.bcy != 0);
            if (rh > cm_max_nodes<S>()) continue;
            int last = 0;
            for (int wv = 1; wv <= kWaves; ++wv) {
                // the widest tiles whose region fits wv waves
                const long long room = wv * 64 / rh;
                int ntx = 1;
                if (room < cm_span(k.nx, 1, h, k.bcx != 0)) {
                    if (room <= 2 * h) continue;
                    ntx = int((k.nx + room - 2 * h - 1) / (room - 2 * h));
                    if (k.bcx && ntx == 2 && room < cm_span(k.nx, 2, h, true)) ntx = 3;
                }
                if (ntx == last || resident[wv] < 1 || cm_region(k, ntx, nty, h) > wv * 64) continue;
                last = ntx;
                const long long tiles = (long long)ntx * nty * k.batch, cap = (long long)cus * resident[wv];
                if (tiles >= (1 << 21)) continue;
                const long long full = tiles / cap, rem = tiles - full * cap;
                const double rounds = double(full + (rem > 0));
                const double waves = double(full) * std::max(1.0, resident[wv] * wv / 4.0) +
                                     (rem ? std::max<double>(1.0, double(((rem + cus - 1) / cus * wv + 3) / 4)) : 0.0);
                const double cost = (c.t0 + c.t1 * (rounds - 1) + h * (c.a * rounds + c.b * waves)) / h;
                if (cost < best_cost) {
                    best_cost = best.cost = cost;
                    best.steps = h;
                    best.cus = cus;
                    best.ntx = ntx;
                    best.nty = nty;
                }
            }
        }
    return best;
}

template <typename S>
hipError_t launch_chan_multi(const ChanK& k, const ChanMultiPlan& plan, const S* a, S* b,
                             const S* qw, const S* uin, const S* tin, const double* mods,
                             int nsteps, long long tape, hipStream_t s) {
    const long long nodes = chan_multi_region(k, plan, nsteps);
    const long long tiles = (long long)plan.ntx * plan.nty * k.batch;
    if (nsteps < 1 || nsteps > plan.steps || nodes < 1 || nodes > cm_max_nodes<S>() || tiles >= (1 << 21))
        return hipErrorInvalidValue;
    ChanMultiArgs<S> p{};
    p.k = chan_kt<S>(k);
    p.ntx = plan.ntx;
    p.nty = plan.nty;
    p.wx = k.nx / plan.ntx;
    p.ex = k.nx % plan.ntx;
    p.wy = k.ny / plan.nty;
    p.ey = k.ny % plan.nty;
    p.nsteps = nsteps;
    p.tape = tape;
    for (int i = 0; i < nsteps; ++i) p.mod[i] = S(mods[i]);
    const unsigned threads = unsigned((nodes + 63) / 64 * 64);
    dim3 grd(unsigned((tiles + kXCD - 1) / kXCD * kXCD)), blk(threads);
    hipLaunchKernelGGL(cm_kernel<S>(k.tq, int(threads)), grd, blk, 0, s, p, a, b, qw, uin, tin);
    return hipGetLastError();
}

#define LBM_CM_INST(S)                                                                            \
    template ChanMultiPlan chan_multi_plan<S>(const ChanK&);                                      \
    template hipError_t launch_chan_multi<S>(const ChanK&, const ChanMultiPlan&, const S*, S*,    \
                                             const S*, const S*, const S*, const double*, int,    \
                                             long long, hipStream_t);
LBM_CM_INST(float)
LBM_CM_INST(double)

}  // namespace lbm
