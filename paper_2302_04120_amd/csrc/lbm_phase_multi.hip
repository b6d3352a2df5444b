// Many two-phase D2Q9 steps per launch for grids that do not fill the GPU: the
// scheme of k_chan_multi.  A workgroup takes a tile with an overlap of two
// nodes per step on every side that cuts through the grid (one for phi of the
// neighbours, one for their pushes), keeps one node per thread in registers,
// and exchanges phi and the moving post-collision values through LDS.  An axis
// that one tile spans has no overlap: it wraps (or ends at its walls) in LDS.
//
// Per node the arithmetic is phase_local + phase_collide, and values are
// rounded to the storage type between steps, so the states agree with
// single-step launches to the last bit.
#include "lbm_phase.h"

#include <algorithm>

namespace lbm {
namespace {

template <typename C>
struct PhaseMultiArgs {
    PhaseKT<C> k;
    int ntx, nty;         // tiles per replica
    int wx, ex, wy, ey;   // tile i spans w nodes, one more for i < e
    int nsteps;           // steps of this launch; the overlap is 2 nsteps
};

template <typename S, typename C, int NT>
__global__ __launch_bounds__(NT) void k_phase_multi(const PhaseMultiArgs<C> p,
                                                    const S* __restrict__ A, S* __restrict__ B) {
    constexpr bool RMASS = std::is_same<S, float>::value;
    using PL = PhasePlanes<S>;
    __shared__ C sphi[NT];
    __shared__ S buf[16][NT];  // h_1..8, z_1..8 after the collision
    const auto& k = p.k;
    const int nx = k.nx, ny = k.ny, h = 2 * p.nsteps;
    int w, tx, ty, b;
    if (!xcd_tile(p.ntx * p.nty * k.batch, w)) return;  // whole workgroup, before any barrier
    block_divide(w, p.ntx, w, tx);
    block_divide(w, p.nty, b, ty);
    const bool xall = p.ntx == 1, yall = p.nty == 1, walls = k.bcy != 0;
    const int x0 = tx * p.wx + min(tx, p.ex), x1 = x0 + p.wx + (tx < p.ex);
    const int y0 = ty * p.wy + min(ty, p.ey), y1 = y0 + p.wy + (ty < p.ey);
    const int rx0 = xall ? 0 : x0 - h, rx1 = xall ? nx : x1 + h;
    const int ry0 = yall ? 0 : walls ? max(y0 - h, 0) : y0 - h;
    const int ry1 = yall ? ny : walls ? min(y1 + h, ny) : y1 + h;
    const int rw = rx1 - rx0, rh = ry1 - ry0;
    const int t = threadIdx.x;
    int rx, ry;
    block_divide(t, rw, ry, rx);
    const int vx = rx0 + rx, vy = ry0 + ry;
    int x = vx, y = vy;
    while (x < 0) x += nx;
    while (x >= nx) x -= nx;
    if (!walls) {
        while (y < 0) y += ny;
        while (y >= ny) y -= ny;
    }
    // m: nodes to the nearest edge of the region that cuts through the grid.
    // The state is known for the steps s with 2 s <= m.
    int m = 1 << 20;
    if (!xall) m = min(m, min(rx, rw - 1 - rx));
    if (!yall && !(walls && ry0 == 0)) m = min(m, ry);
    if (!yall && !(walls && ry1 == ny)) m = min(m, rh - 1 - ry);
    if (ry >= rh) m = -1;
    const bool own = ry < rh && vx >= x0 && vx < x1 && vy >= y0 && vy < y1;
    const bool ylo = walls && y == 0, yhi = walls && y == ny - 1;
    // LDS offsets to the neighbours: round the axis where the tile spans it, 0
    // across a wall (the mirror ghost of phi)
    const int om = rx > 0 ? -1 : xall ? rw - 1 : 0, op = rx < rw - 1 ? 1 : xall ? 1 - rw : 0;
    const int od = ylo ? 0 : ry > 0 ? -rw : yall ? (rh - 1) * rw : 0;
    const int ou = yhi ? 0 : ry < rh - 1 ? rw : yall ? (1 - rh) * rw : 0;
    auto off = [&](int ex, int ey) {
        return t + (ex < 0 ? om : ex > 0 ? op : 0) + (ey < 0 ? od : ey > 0 ? ou : 0);
    };
    const long long n = ((long long)b * ny + y) * nx + x;
    // every load is issued before the first is converted: with a conversion to
    // FP64 behind each load the 21 round trips came one after another (4.5 us)
    S in[PL::NPL];
    if (m >= 0) {
#pragma unroll
        for (int i = 0; i < PL::NPL; ++i) in[i] = A[pidx<S>(i, n)];
    } else {
#pragma unroll
        for (int i = 0; i < PL::NPL; ++i) in[i] = S(0);
    }
    C hv[9], z[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        hv[i] = C(in[PL::H + i]);
        z[i] = C(in[PL::Z + i]);
    }
    C hlo = RMASS ? C(in[PL::LO]) : C(0), pu0 = C(in[PL::PU]), pu1 = C(in[PL::PU + 1]);
    for (int s = 0; s < p.nsteps; ++s) {
        if (m >= 2 * s) sphi[t] = phi_sum(hv, hlo);
        __syncthreads();
        C hs[9], zst[9], pux = C(0), puy = C(0);
        S h0hi = S(0), h0lo = S(0);
        if (m > 2 * s) {
            C pn[9];
#pragma unroll
            for (int i = 0; i < 9; ++i) pn[i] = sphi[off(EX[i], EY[i])];
            const PhaseLocal<C> L = phase_local<C>(k, pn, z);
            phase_collide<S, C>(k, L, hv, hlo, z, pu0, pu1, hs, h0hi, h0lo, zst, pux, puy);
#pragma unroll
            for (int i = 1; i < 9; ++i) {
                buf[i - 1][t] = S(hs[i]);
                buf[7 + i][t] = S(zst[i]);
            }
        }
        __syncthreads();
        if (m > 2 * s + 1) {
            hv[0] = C(h0hi);
            hlo = C(h0lo);
            z[0] = C(S(zst[0]));
            pu0 = C(S(pux));
            pu1 = C(S(puy));
            // a value comes from the node it leaves, or through a wall from the
            // node itself (halfway bounce-back)
#pragma unroll
            for (int j = 1; j < 9; ++j) {
                const bool wall = EY[j] > 0 ? ylo : EY[j] < 0 ? yhi : false;
                const int from = wall ? t : off(-EX[j], -EY[j]), i = wall ? OPP[j] : j;
                hv[j] = C(buf[i - 1][from]);
                z[j] = C(buf[7 + i][from]);
            }
        }
    }
    if (!own) return;
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        B[pidx<S>(PL::H + i, n)] = S(hv[i]);
        B[pidx<S>(PL::Z + i, n)] = S(z[i]);
    }
    if (RMASS) B[pidx<S>(PL::LO, n)] = S(hlo);
    B[pidx<S>(PL::PU, n)] = S(pu0);
    B[pidx<S>(PL::PU + 1, n)] = S(pu1);
}

// Largest region (threads of a workgroup): FP64 arithmetic takes 160 registers.
template <typename C>
constexpr int pm_max_nodes() {
    return sizeof(C) == 4 ? 1024 : 768;
}
// Span of the widest tile's region on an axis.
long long pm_span(int n, int tiles, int h, bool walls) {
    if (tiles == 1) return n;
    const long long w = (n + tiles - 1) / tiles;
    return walls ? std::min<long long>(n, w + (tiles == 2 ? h : 2 * h)) : w + 2 * h;
}
long long pm_region(const PhaseK& k, int ntx, int nty, int h) {
    return pm_span(k.nx, ntx, h, false) * pm_span(k.ny, nty, h, k.bcy != 0);
}
template <typename S, typename C>
auto pm_kernel(int threads) {
    if (threads > 512) return k_phase_multi<S, C, pm_max_nodes<C>()>;
    return threads > 256 ? k_phase_multi<S, C, 512> : k_phase_multi<S, C, 256>;
}

// Tiles and steps per launch, by a cost model fitted to 1500 plans on 17 grids
// of 2 k to 1.2 M nodes (it predicts those of at most two rounds to 12-16 %, its
// choice runs within 17 % of the best measured plan of each grid):
//   launch = T0 + T1 (rounds - 1) + steps sum over rounds (a + b W)
//            + memory (MB read with the overlap and written)
// in microseconds, W the waves per SIMD of the busiest CU and rounds the number
// of times the workgroups fill the GPU; plans of more than two rounds never
// won.  Single steps take 4.8 us (FP64 6.2, FP64 arithmetic on FP32 5.3) plus
// their bytes at 7.0 (7.4) TB/s, out of the caches at these sizes; a plan is
// taken where it saves 12 %.  Measured per step, single -> plan: 4 x 512 with
// walls FP32 5.4 -> 1.26 us, FP64 6.7 -> 1.6, FP64 arithmetic 5.4 -> 1.55;
// 20 x 8 x 200 5.6 -> 1.6; 128 x 100 FP32 5.2 -> 3.2; 2 x 300 x 280 8.0 -> 7.1;
// 4 x 256 x 256 10.7 -> 9.2 (1024 nodes a CU: four waves a SIMD without any
// overlap).  Pushing from the tile's own nodes in the last step (one node less
// of overlap) and two nodes per thread took 130-255 registers or spilled, and
// were slower (4 x 256 x 256: 10.6 and 12.9 us).
template <typename S, typename C>
PhaseMultiPlan pm_plan(const PhaseK& k) {
    PhaseMultiPlan best{};
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        return best;
    constexpr bool F32 = sizeof(C) == 4, A64 = !F32 && sizeof(S) == 4;
    const double t0 = A64 ? 3.9 : 3.6, t1 = F32 ? 2.5 : A64 ? 4.0 : 0.0, a = F32 ? 0.0 : 0.05;
    const double b = F32 ? 0.50 : A64 ? 0.78 : 0.81, mem = F32 ? 0.071 : A64 ? 0.045 : 0.123;
    constexpr int kWaves = pm_max_nodes<C>() / 64;
    int resident[kWaves + 1] = {};  // workgroups of that many waves per CU
    for (int wv = 1; wv <= kWaves; ++wv)
        resident[wv] = resident_workgroups((const void*)pm_kernel<S, C>(wv * 64), wv);
    const double mb = double(PhasePlanes<S>::NPL) * sizeof(S) / 1e6;
    const double nodes = double(k.nx) * k.ny * k.batch;
    double least = 0.88 * ((F32 ? 4.8 : A64 ? 5.3 : 6.2) + 2 * nodes * mb / (sizeof(S) == 4 ? 7.0 : 7.4));
    for (int steps = 2; steps <= kPhaseMultiMax; ++steps)
        for (int nty = 1; nty <= std::min(k.ny, 512); ++nty) {
            // one plan per height of the widest tile: the fewest tiles of it
            if (nty > 1 && (k.ny + nty - 1) / nty == (k.ny + nty - 2) / (nty - 1)) continue;
            const int h = 2 * steps;
            const long long rh = pm_span(k.ny, nty, h, k.bcy != 0);
            if (rh > pm_max_nodes<C>()) continue;
            int last = 0;
            for (int wv = 1; wv <= kWaves; ++wv) {
                const long long room = wv * 64 / rh;  // the widest tiles whose region fits wv waves
                int ntx = 1;
                if (room < k.nx) {
                    if (room <= 2 * h) continue;
                    ntx = std::max(2, int((k.nx + room - 2 * h - 1) / (room - 2 * h)));
                }
                const long long region = pm_region(k, ntx, nty, h);
                if (ntx == last || resident[wv] < 1 || region > wv * 64) continue;
                last = ntx;
                const long long tiles = (long long)ntx * nty * k.batch, cap = (long long)cus * resident[wv];
                const long long full = tiles / cap, rem = tiles - full * cap;
                const int rounds = int(std::min<long long>(full + (rem > 0), 3));
                if (rounds > 2 || tiles >= (1 << 21)) continue;
                const double waves = double(full) * std::max(1.0, resident[wv] * wv / 4.0) +
                                     (rem ? std::max<double>(1.0, double(((rem + cus - 1) / cus * wv + 3) / 4)) : 0.0);
                const double cost = (t0 + t1 * (rounds - 1) + steps * (a * rounds + b * waves) +
                                     mem * mb * (double(tiles) * region + nodes)) / steps;
                if (cost < least) {
                    least = cost;
                    best.steps = steps;
                    best.cost = cost;
                    best.ntx = ntx;
                    best.nty = nty;
                }
            }
        }
    return best;
}

template <typename S, typename C>
hipError_t pm_launch(const PhaseK& k, const PhaseMultiPlan& plan, const S* a, S* b, int nsteps,
                     hipStream_t s) {
    if (nsteps < 1 || nsteps > plan.steps || plan.ntx < 1 || plan.nty < 1) return hipErrorInvalidValue;
    const long long nodes = pm_region(k, plan.ntx, plan.nty, 2 * nsteps);
    const long long tiles = (long long)plan.ntx * plan.nty * k.batch;
    if (nodes > pm_max_nodes<C>() || tiles >= (1 << 21)) return hipErrorInvalidValue;
    PhaseMultiArgs<C> p{};
    p.k = phase_kt<C>(k);
    p.ntx = plan.ntx;
    p.nty = plan.nty;
    p.wx = k.nx / plan.ntx;
    p.ex = k.nx % plan.ntx;
    p.wy = k.ny / plan.nty;
    p.ey = k.ny % plan.nty;
    p.nsteps = nsteps;
    const int threads = int((nodes + 63) / 64 * 64);
    hipLaunchKernelGGL((pm_kernel<S, C>(threads)), dim3(unsigned((tiles + kXCD - 1) / kXCD * kXCD)),
                       dim3(unsigned(threads)), 0, s, p, a, b);
    return hipGetLastError();
}

}  // namespace

long long phase_multi_region(const PhaseK& k, const PhaseMultiPlan& p, int steps) {
    return p.ntx > 0 && p.nty > 0 ? pm_region(k, p.ntx, p.nty, 2 * steps) : 0;
}

template <typename S>
PhaseMultiPlan phase_multi_plan(const PhaseK& k, bool arith64) {
    return arith64 ? pm_plan<S, double>(k) : pm_plan<S, S>(k);
}

template <typename S>
hipError_t launch_phase_multi(const PhaseK& k, const PhaseMultiPlan& plan, const S* a, S* b,
                              bool arith64, int nsteps, hipStream_t s) {
    return arith64 ? pm_launch<S, double>(k, plan, a, b, nsteps, s)
                   : pm_launch<S, S>(k, plan, a, b, nsteps, s);
}

#define LBM_PM_INST(S)                                                                             \
    template PhaseMultiPlan phase_multi_plan<S>(const PhaseK&, bool);                              \
    template hipError_t launch_phase_multi<S>(const PhaseK&, const PhaseMultiPlan&, const S*, S*,  \
                                              bool, int, hipStream_t);
LBM_PM_INST(float)
LBM_PM_INST(double)

}  // namespace lbm
