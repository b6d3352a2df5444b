// HIP kernels of the dimensional LBM hot path for gfx950 (CDNA4, wave64).
//
// Data layout: node n = (b * ny + y) * nx + x (x fastest); the 2D states in
// node blocks (value i of node n at bidx(npl, i, n): the npl values of 64
// consecutive nodes together), the 1D lattices and the FP64 staging fields in
// planes of stride P.
// The stored state is the pre-collision ("post-streaming") population set;
// each step reads a node's own populations (coalesced), collides in
// registers and pushes the post-collision values to x + e_i in the other
// buffer.  Populations whose destination lies outside the domain are turned
// back into the node by the boundary rule of that side, so every slot of the
// next buffer is written exactly once and no two threads write the same slot.
//
// All arithmetic is in lattice-normalised form (velocities / c, forces
// F dt^2 / dx, rates Lambda dt).  The dimensional MRT of Sec. 3 multiplies
// the rows of the lattice matrix by c^order and its inverse's columns by
// c^-order; a diagonal relaxation commutes with that scaling, so the
// post-collision populations are the same in either form.
#include "lbm_channel.h"
#include "lbm_device.h"
#include "lbm_phase.h"

#include <cmath>
#include <type_traits>

namespace lbm {
namespace {

// One step of the channel model: D2Q9 flow (BGK or dimensional MRT, Guo
// forcing, optional Boussinesq force) + D2Q5 or D2Q9 temperature.  Tiles of
// 64 nodes of one row (one wave each).  y: periodic (bcy 0), halfway walls
// (1), or a wall at y- and the symmetry plane of Eq. simetria at y+ (2).  x:
// periodic (bcx 0), velocity inlet + pressure outlet (1), fixed-temperature
// walls (2).
template <typename S, int QT>
__global__ __launch_bounds__(64) void k_chan_step(ChanK k, const S* __restrict__ A,
                                                        S* __restrict__ B, const S* __restrict__ qw,
                                                        const S* __restrict__ uin,
                                                        const S* __restrict__ tin, S mod) {
    using C = S;
    const int nx = k.nx, ny = k.ny;
    const int gx = (nx + 63) / 64;
    int tile;
    if (!xcd_tile(gx * ny * k.batch, tile)) return;
    const int b = tile / (gx * ny), r = tile - b * gx * ny;
    const int x = (r % gx) * 64 + threadIdx.x;
    const int y = r / gx;
    if (x >= nx) return;
    const int npl = k.npl;  // node blocks: f 0-8, g 9 .. 9 + QT - 1
    const long long base = (long long)b * ny * nx;
    const long long n = base + (long long)y * nx + x;
    const C rho_ref = C(k.rho_ref);
    const C qdt = C(k.qdt);

    // temperature first: the Boussinesq force depends on it
    C e[QT], th = C(0);
    if (k.thermal) {
#pragma unroll
        for (int i = 0; i < QT; ++i) e[i] = C(A[bidx(npl, 9 + i, n)]);
        th = chan_th<QT, C>(e, qdt);
    }
    C ftx, fty;
    chan_force(k, th, ftx, fty);

    C d[9], drho, rho, ux, uy;
    chan_flow_macros<C, S>(A, npl, n, rho_ref, ftx, fty, d, drho, rho, ux, uy);
    C ds[9], es[QT];
    chan_collide<C, QT, ChanK>(k, d, drho, rho, ux, uy, ftx, fty, e, th, qdt, ds, es);

    // ---- outlet wall velocity: 1.5 u(x_b) - 0.5 u(x_b - 1) at time t
    C uwx = C(0), uwy = C(0);
    const bool outlet = k.bcx == 1 && x == nx - 1;
    if (k.flow && outlet) {
        C d2[9], dr2, r2, ux2, uy2, fx2 = ftx, fy2 = fty;
        if (k.buoy) {  // the force of that node, as it computes it itself
            C e2[QT];
#pragma unroll
            for (int i = 0; i < QT; ++i) e2[i] = C(A[bidx(npl, 9 + i, n - 1)]);
            chan_force(k, chan_th<QT, C>(e2, qdt), fx2, fy2);
        }
        chan_flow_macros<C, S>(A, npl, n - 1, rho_ref, fx2, fy2, d2, dr2, r2, ux2, uy2);
        uwx = C(1.5) * ux - C(0.5) * ux2;
        uwy = C(1.5) * uy - C(0.5) * uy2;
    }

    // ---- streaming with boundary substitution (a frozen flow keeps its
    //      populations).  A population leaving through the symmetry plane
    //      re-enters as its mirror image at x + c_x (Eq. simetria); where that
    //      lies outside in x the x rule applies.
    if (!k.flow) {
#pragma unroll
        for (int i = 0; i < 9; ++i) B[bidx(npl, i, n)] = S(d[i]);
    } else {
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            int tx = x + EX[i], ty = y + EY[i], j = i;
            const bool sym = k.bcy == 2 && ty >= ny;
            if (sym) {
                ty = ny - 1;
                j = MIRY[i];
            }
            const bool outy = k.bcy && !sym && (ty < 0 || ty >= ny);
            const bool outx = k.bcx && (tx < 0 || tx >= nx);
            if (!outy && !outx) {
                tx = wrap(tx, nx);
                ty = wrap(ty, ny);
                B[bidx(npl, j, base + (long long)ty * nx + tx)] = S(ds[i]);
            } else {
                C v;
                if (outy || k.bcx == 2)
                    v = ds[i];  // halfway bounce-back, Eq. BB_vel with u_w = 0
                else if (tx < 0)
                    v = chan_inlet_f<C>(i, ds[i], rho_ref, C(uin[y]));
                else
                    v = chan_outlet_f<C>(i, ds[i], rho_ref, uwx, uwy);
                B[bidx(npl, OPP[i], n)] = S(v);
            }
        }
    }
    if (k.thermal) {
        // Thermal outlet, first-order extrapolation g_j(x_b) = g_j(x_b - 1) at
        // t + dt: each value stored into column nx - 2 for a population with
        // c_x < 0 is stored into the outlet column as well, unless a wall rule
        // owns that outlet slot (its source lies beyond a wall in y).
        auto put = [&](int j, int tx, int ty, C v) {
            B[bidx(npl, 9 + j, base + (long long)ty * nx + tx)] = S(v);
            if (k.bcx == 1 && tx == nx - 2 && tex<QT>(j) < 0) {
                const int sy = ty - tey<QT>(j);
                const bool wall_owned = k.bcy && (sy < 0 || (k.bcy == 1 && sy >= ny));
                if (!wall_owned) B[bidx(npl, 9 + j, base + (long long)ty * nx + nx - 1)] = S(v);
            }
        };
#pragma unroll
        for (int i = 0; i < QT; ++i) {
            int tx = x + tex<QT>(i), ty = y + tey<QT>(i), j = i;
            const bool sym = k.bcy == 2 && ty >= ny;
            if (sym) {
                ty = ny - 1;
                j = tmir<QT>(i);
            }
            const bool outy = k.bcy && !sym && (ty < 0 || ty >= ny);
            const bool outx = k.bcx && (tx < 0 || tx >= nx);
            if (!outy && !outx) {
                put(j, wrap(tx, nx), wrap(ty, ny), es[i]);
            } else if (outy) {
                put(topp<QT>(i), x, y, chan_flux_g<QT, C>(i, es[i], C(qw[x]), C(mod)));
            } else if (k.bcx == 2) {
                // fixed-temperature side wall (App. D)
                put(topp<QT>(i), x, y, chan_antibb_g<QT, C>(i, es[i], C(k.Tw[tx < 0 ? 0 : 1])));
            } else if (tx < 0) {
                // anti-bounce-back Dirichlet inlet, T_w where the link crosses
                // the inlet (between rows y and y + c_y)
                const int y2 = y + tey<QT>(i);
                const C tw = (y2 >= 0 && y2 < ny) ? C(0.5) * (C(tin[y]) + C(tin[y2])) : C(tin[y]);
                put(topp<QT>(i), x, y, chan_antibb_g<QT, C>(i, es[i], tw));
            }
            // populations leaving through the outlet: the outlet slots are filled
            // by the extrapolation stores of put()
        }
    }
}

// ---------------------------------------------------------------------------
// Two-phase model: conservative Allen-Cahn h_i (BGK) + pressure z_i (MRT/BGK)
// State planes (node-block layout, PhasePlanes): 0-8 h_i, 9-17 z_i, then
// (FP32 storage only) the low part of h_0, then (phi u) of the previous step
// (2 planes): npop = 19 (FP32) or 18 (FP64) population planes plus 2.
// ---------------------------------------------------------------------------

#ifndef LBM_PHASE_TY
#define LBM_PHASE_TY 8
#endif
constexpr int TX = 64, TY = LBM_PHASE_TY;
// LDS reserved by each FP32 single-step workgroup beyond its own ~1.5 KB: it
// holds residency at four 256-thread workgroups per CU (4 waves per SIMD).
// With more waves resident, more of the 42 population streams per wave are
// open in DRAM at once and the step runs slower (67M-node bubble batch:
// 2.82 ms at 8 waves per SIMD, 2.56 ms at 4).  The FP64 kernel's register
// use already gives 4 waves per SIMD.
constexpr unsigned kPhaseLdsReserve = 36864;
// ---------------------------------------------------------------------------
// Single step.  Tile of TX x TY nodes per block (64 x 8, or nx x 512/nx for
// replicas narrower than 64 nodes, so that no lane idles and a wave still
// covers 64 contiguous nodes); phi of the tile and a one-node ring in LDS.
// MACROS: evaluate the macroscopic fields of the stored state into mout
// instead of stepping.
// ---------------------------------------------------------------------------
// One tile of the single step (every thread of the block calls it; it has
// one barrier).  Returns early for threads without a node, after the barrier.
template <typename S, typename C, bool MACROS, int TX, int TY>
__device__ __forceinline__ void phase_tile(const PhaseK& k, int tile, const S* __restrict__ A,
                                           S* __restrict__ B, const MacroOut& mout,
                                           C (&sphi)[TY + 2][TX + 2]) {
    constexpr bool RMASS = std::is_same<S, float>::value;
    using PL = PhasePlanes<S>;
    const int nx = k.nx, ny = k.ny;
    const int tx = threadIdx.x, ty = threadIdx.y;
    const int gx = (nx + TX - 1) / TX, gy = (ny + TY - 1) / TY;
    const int b = tile / (gx * gy), r = tile - b * gx * gy;
    const int x0 = (r % gx) * TX, y0 = (r / gx) * TY;
    const long long base = (long long)b * ny * nx;
    auto gxw = [&](int gx) { return ((gx % nx) + nx) % nx; };
    auto gyw = [&](int gy) {
        if (k.bcy) return gy < 0 ? 0 : (gy >= ny ? ny - 1 : gy);  // mirror ghost at walls
        return ((gy % ny) + ny) % ny;
    };
    // Every load of the tile is issued before the barrier: the node's own h, z
    // and (phi u) (kept in registers for the collision) and, for 148 threads,
    // the 10 values of one ring node; the barrier then waits for memory once.
    const int x = x0 + tx, y = y0 + ty;
    const bool valid = x < nx && y < ny;
    const long long n = base + (long long)gyw(y) * nx + gxw(x);  // == own node when valid
    C h[9], z[9], hlo = C(0), pu0 = C(0), pu1 = C(0);
#pragma unroll
    for (int i = 0; i < 9; ++i) h[i] = C(A[pidx<S>(PL::H + i, n)]);
    if (RMASS) hlo = C(A[pidx<S>(PL::LO, n)]);
    if (valid) {
#pragma unroll
        for (int i = 0; i < 9; ++i) z[i] = C(A[pidx<S>(PL::Z + i, n)]);
        if constexpr (!MACROS) {
            pu0 = C(A[pidx<S>(PL::PU, n)]);
            pu1 = C(A[pidx<S>(PL::PU + 1, n)]);
        }
    }
    int hx = -2, hy = -2;
    {
        const int t = ty * TX + tx;
        if (t < TX + 2) { hy = -1; hx = t - 1; }
        else if (t < 2 * (TX + 2)) { hy = TY; hx = t - (TX + 2) - 1; }
        else if (t < 2 * (TX + 2) + TY) { hx = -1; hy = t - 2 * (TX + 2); }
        else if (t < 2 * (TX + 2) + 2 * TY) { hx = TX; hy = t - 2 * (TX + 2) - TY; }
    }
    C ring = C(0);
    if (hx > -2) {
        const long long nn = base + (long long)gyw(y0 + hy) * nx + gxw(x0 + hx);
        C hr[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) hr[i] = C(A[pidx<S>(PL::H + i, nn)]);
        ring = phi_sum(hr, RMASS ? C(A[pidx<S>(PL::LO, nn)]) : C(0));
    }
    sphi[ty + 1][tx + 1] = phi_sum(h, hlo);
    if (hx > -2) sphi[hy + 1][hx + 1] = ring;
    __syncthreads();
    if (!valid) return;

    C pn[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) pn[i] = sphi[ty + 1 + EY[i]][tx + 1 + EX[i]];
    const PhaseLocal<C> L = phase_local<C>(k, pn, z);

    if constexpr (MACROS) {
        mout.put(0, n, double(L.rho));
        mout.put(1, n, double(L.ph) * k.cs2);
        mout.put(2, n, double(L.ux) * k.c);
        mout.put(3, n, double(L.uy) * k.c);
        mout.put(5, n, double(L.phi));
        mout.put(6, n, double(L.mu));
        return;
    } else {
        C hs[9], zst[9], pux, puy;
        S h0hi, h0lo;
        phase_collide<S, C>(k, L, h, hlo, z, pu0, pu1, hs, h0hi, h0lo, zst, pux, puy);
        st(B + pidx<S>(PL::PU, n), S(pux));
        st(B + pidx<S>(PL::PU + 1, n), S(puy));
        // ---- streaming of h and z: x periodic; y periodic or halfway
        //      bounce-back walls
        st(B + pidx<S>(PL::H, n), h0hi);
        if constexpr (RMASS) st(B + pidx<S>(PL::LO, n), h0lo);
        st(B + pidx<S>(PL::Z, n), S(zst[0]));
#pragma unroll
        for (int i = 1; i < 9; ++i) {
            const int tyd = y + EY[i];
            if (k.bcy && (tyd < 0 || tyd >= ny)) {
                st(B + pidx<S>(PL::H + OPP[i], n), S(hs[i]));
                st(B + pidx<S>(PL::Z + OPP[i], n), S(zst[i]));
            } else {
                const long long d = base + (long long)wrap(tyd, ny) * nx + wrap(x + EX[i], nx);
                st(B + pidx<S>(PL::H + i, d), S(hs[i]));
                st(B + pidx<S>(PL::Z + i, d), S(zst[i]));
            }
        }
    }
}

template <typename S, typename C, bool MACROS, int TX = lbm::TX, int TY = lbm::TY>
__global__ __launch_bounds__(TX * TY) void k_phase(PhaseK k, const S* __restrict__ A,
                                               S* __restrict__ B, MacroOut mout) {
    static_assert(2 * (TX + 2) + 2 * TY <= TX * TY, "the ring must fit in one pass of the block");
    __shared__ C sphi[TY + 2][TX + 2];
    const int gx = (k.nx + TX - 1) / TX, gy = (k.ny + TY - 1) / TY;
    int tile;
    if (!xcd_tile(gx * gy * k.batch, tile)) return;  // whole workgroup, before any barrier
    phase_tile<S, C, MACROS, TX, TY>(k, tile, A, B, mout, sphi);
}

// ---------------------------------------------------------------------------
// Many steps in one launch for grids of a few tiles (the paper's C4 channel is
// 4 x 512 nodes: sixteen 4 x 32 tiles).  One workgroup per tile, all resident
// at once (cooperative launch).  Between steps a tile waits only for the
// tiles that, in the previous step, pushed into the nodes it reads or read
// the nodes its next pushes overwrite (the tiles around it; every tile of
// its replica when a ragged tail is one node thick), through per-tile step
// counters with device-scope release / acquire; a grid-wide barrier costs
// several times more on this GPU.  Every wait is bounded: past the bound the workgroup
// flags an error and leaves, and so do its neighbours in turn, so the grid
// always drains.  The per-tile work is phase_tile, as in k_phase, so the
// states agree with single-step launches to the last bit.
// ---------------------------------------------------------------------------
constexpr unsigned kPersistSpin = 1u << 22;  // polls before a wait counts as failed

template <typename S, typename C, int TX, int TY>
__global__ __launch_bounds__(TX * TY) void k_phase_persist(PhaseK k, S* __restrict__ A,
                                                           S* __restrict__ B, int nsteps,
                                                           unsigned epoch0,
                                                           unsigned* __restrict__ flags,
                                                           unsigned* __restrict__ err) {
    static_assert(2 * (TX + 2) + 2 * TY <= TX * TY, "the ring of a tile needs a thread per node");
    __shared__ C sphi[TY + 2][TX + 2];
    __shared__ int bad;
    const int gx = (k.nx + TX - 1) / TX, gy = (k.ny + TY - 1) / TY;
    const int tile = blockIdx.x;
    const int b = tile / (gx * gy), r = tile - b * gx * gy;
    const int bx = r % gx, by = r / gx;
    // Tiles whose step s - 1 must be complete before this tile's step s: those
    // that write the tile's nodes or its ring in step s - 1 (data it reads) and
    // those that read, in step s - 1, the nodes it writes in step s.  When
    // every tile spans at least two nodes in x and y these are the tiles of the
    // same replica within one node (x periodic, y periodic or closed by
    // walls); a one-node ragged tail reaches further, and then the tile waits
    // for every tile of its replica.
    const bool thin = (gx > 1 && k.nx - (gx - 1) * TX < 2) || (gy > 1 && k.ny - (gy - 1) * TY < 2);
    const int lin = threadIdx.y * TX + threadIdx.x;
    // Lanes of the first wave watch one tile each: lane j < 8 the j-th of
    // the eight surrounding tiles (x wraps; y wraps unless walls close it),
    // or, for a one-node tail, lane j tile j of the replica (at most 64).
    int wt = -1;
    if (thin) {
        if (lin < gx * gy && lin != r) wt = lin;
    } else if (lin < 8) {
        const int j = lin < 4 ? lin : lin + 1;  // skip the centre of the 3 x 3 block
        const int ox = j % 3 - 1, oy = j / 3 - 1;
        int ty_ = by + oy;
        const bool outside = ty_ < 0 || ty_ >= gy;
        ty_ = (ty_ + gy) % gy;
        const int t = ty_ * gx + (bx + ox + gx) % gx;
        if (!(outside && k.bcy) && t != r) wt = t;
    }
    const bool watch = wt >= 0;
    const unsigned* wflag = flags + b * gx * gy + (watch ? wt : 0);
    if (lin == 0) bad = 0;
    for (int s = 0; s < nsteps; ++s) {
        if (s > 0 && lin < 64) {
            const unsigned want = epoch0 + unsigned(s);
            unsigned spins = 0;
            bool fail = false;
            for (;;) {
                // modular comparison: the counter is behind want
                const bool behind =
                    watch && __hip_atomic_load(wflag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) -
                                     want > 0x7fffffffu;
                if (!__any(behind)) break;
                if (++spins > kPersistSpin ||
                    __any(__hip_atomic_load(err, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != 0)) {
                    fail = true;
                    break;
                }
            }
            if (fail && lin == 0) {
                bad = 1;
                __hip_atomic_fetch_or(err, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
            // one acquire for the workgroup: its waves share this CU's caches
            // and follow the first wave through the barrier below
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        }
        __syncthreads();
        if (bad) return;  // uniform: every thread read it after the barrier
        const S* a = (s & 1) ? B : A;
        S* o = (s & 1) ? A : B;
        phase_tile<S, C, false, TX, TY>(k, tile, a, o, MacroOut{}, sphi);
        // Every wave waits until its stores have reached the L2 (vmcnt counts
        // stores on this GPU), the barrier orders them before the first
        // lane's device-scope release, whose L2 write-back then carries the
        // whole tile: one write-back per workgroup and step instead of one
        // per wave.
        __builtin_amdgcn_s_waitcnt(0);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __syncthreads();
        if (lin == 0)
            __hip_atomic_store(&flags[tile], epoch0 + unsigned(s + 1), __ATOMIC_RELEASE,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
}

// ---------------------------------------------------------------------------
// 1D thermal BGK, whole run in one workgroup of WAVES waves (n <= 64 WAVES M).
// A step is a serial chain of a few FP64 operations, so what it pays for is
// latency: a lane keeps M consecutive nodes in registers, its neighbours'
// values come by a shift across the wave, and only a run of several waves
// exchanges its ends through LDS (one barrier per step).  With one node per
// thread, LDS streaming and two barriers of a 1024-thread workgroup a step took
// 0.59 us whatever n.  One wave then issues what a step costs, so instances spare
// instructions: JE, the last node's place in its lane (its rule in that slot only,
// and the first node's in slot 0), and no velocity factor in the equilibrium (the
// 1D lattices have u = 0: it is one).  42 -> 31 vector instructions for Q = 2,
// M = 2, 97 -> 73 ns a step at 101 nodes.  Q = 2 (D1Q2) or 3 (D1Q3).
// ---------------------------------------------------------------------------
// v of the lane before (shr) or after (shl) in the wave; 0 at its end
__device__ __forceinline__ double wave_shr1(double v) {
    const int lo = __double2loint(v), hi = __double2hiint(v);
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, hi, 0x138, 0xf, 0xf, true),
                            __builtin_amdgcn_update_dpp(0, lo, 0x138, 0xf, 0xf, true));
}
__device__ __forceinline__ double wave_shl1(double v) {
    const int lo = __double2loint(v), hi = __double2hiint(v);
    return __hiloint2double(__builtin_amdgcn_update_dpp(0, hi, 0x130, 0xf, 0xf, true),
                            __builtin_amdgcn_update_dpp(0, lo, 0x130, 0xf, 0xf, true));
}

template <int Q, int M, int WAVES, int JE>
__global__ __launch_bounds__(64 * WAVES) void k_d1(D1K k, double* __restrict__ g, int nsteps) {
    __shared__ double ends[2][WAVES + 2][2];  // per wave: leaving to the right, to the left
    constexpr double w[3] = {Q == 3 ? 4.0 / 6 : 0.5, Q == 3 ? 1.0 / 6 : 0.5, Q == 3 ? 1.0 / 6 : 0.0};
    constexpr int R = Q == 3 ? 1 : 0, L = Q == 3 ? 2 : 1;  // right and left movers
    const int n = k.n, lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int x0 = int(threadIdx.x) * M;
    double v[M][Q];
#pragma unroll
    for (int j = 0; j < M; ++j)
#pragma unroll
        for (int i = 0; i < Q; ++i) v[j][i] = x0 + j < n ? g[i * n + x0 + j] : 0.0;
    for (int s = 0; s < nsteps; ++s) {
        double sg[M][Q];
#pragma unroll
        for (int j = 0; j < M; ++j) {
            double T = 0;
#pragma unroll
            for (int i = 0; i < Q; ++i) T += v[j][i];
            T += 0.5 * k.qdt;
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                const double geq = w[i] * T;
                sg[j][i] = v[j][i] - k.w_tau * (v[j][i] - geq) + (1.0 - 0.5 * k.w_tau) * w[i] * k.qdt;
            }
        }
        double from_left = wave_shr1(sg[M - 1][R]), from_right = wave_shl1(sg[0][L]);
        if constexpr (WAVES > 1) {
            if (lane == 63) ends[s & 1][wv + 1][0] = sg[M - 1][R];
            if (lane == 0) ends[s & 1][wv + 1][1] = sg[0][L];
            __syncthreads();  // the other buffer's reads ended a step ago
            if (lane == 0) from_left = ends[s & 1][wv][0];
            if (lane == 63) from_right = ends[s & 1][wv + 2][1];
        }
#pragma unroll
        for (int j = 0; j < M; ++j) {
            if constexpr (Q == 3) v[j][0] = sg[j][0];
            v[j][R] = j > 0 ? sg[j > 0 ? j - 1 : 0][R] : from_left;
            v[j][L] = j < M - 1 ? sg[j < M - 1 ? j + 1 : 0][L] : from_right;
            // wet-node Dirichlet with the half source: the unknown population
            const int x = x0 + j;
            if (j == 0 && x == 0) v[j][R] = k.T0 - 0.5 * k.qdt - (Q == 3 ? v[j][0] + v[j][L] : v[j][L]);
            if (j == JE && x == n - 1) v[j][L] = k.TL - 0.5 * k.qdt - (Q == 3 ? v[j][0] + v[j][R] : v[j][R]);
        }
    }
#pragma unroll
    for (int j = 0; j < M; ++j)
#pragma unroll
        for (int i = 0; i < Q; ++i)
            if (x0 + j < n) g[i * n + x0 + j] = v[j][i];
}

// ---------------------------------------------------------------------------
// initialisation from macroscopic fields (staging slots: 0 rho|p, 1 ux, 2 uy,
// 3 T, 4 phi; all FP64, velocities in m/s)
// ---------------------------------------------------------------------------
template <typename S>
__global__ void k_chan_init(ChanK k, const double* __restrict__ fld, S* __restrict__ A) {
    const long long N = (long long)k.batch * k.nx * k.ny;
    const long long P = k.P;
    for (long long n = blockIdx.x * (long long)blockDim.x + threadIdx.x; n < N;
         n += (long long)gridDim.x * blockDim.x) {
        const double rho = fld[n], ux = fld[P + n] / k.c, uy = fld[2 * P + n] / k.c;
        const double th = fld[3 * P + n] - k.T_ref;
        const double uu = ux * ux + uy * uy;
        for (int i = 0; i < 9; ++i) {
            const double eu = EX[i] * ux + EY[i] * uy;
            A[bidx(k.npl, i, n)] = S(wgt<double>(i) * ((rho - k.rho_ref) +
                                                       rho * (3 * eu + 4.5 * eu * eu - 1.5 * uu)));
        }
        if (k.thermal && k.tq == 9)
            for (int i = 0; i < 9; ++i)
                A[bidx(k.npl, 9 + i, n)] =
                    S(wgt<double>(i) * th * (1 + 3 * (EX[i] * ux + EY[i] * uy)));
        else if (k.thermal)
            for (int i = 0; i < 5; ++i)
                A[bidx(k.npl, 9 + i, n)] =
                    S(wgt5<double>(i) * th * (1 + 3 * (EX5[i] * ux + EY5[i] * uy)));
    }
}

template <typename S>
__global__ void k_phase_init(PhaseK k, const double* __restrict__ fld, S* __restrict__ A) {
    constexpr bool RMASS = std::is_same<S, float>::value;
    using PL = PhasePlanes<S>;
    const long long N = (long long)k.batch * k.nx * k.ny;
    const long long P = k.P;
    for (long long n = blockIdx.x * (long long)blockDim.x + threadIdx.x; n < N;
         n += (long long)gridDim.x * blockDim.x) {
        const double p = fld[n], ux = fld[P + n] / k.c, uy = fld[2 * P + n] / k.c;
        const double phi = fld[4 * P + n];
        const double rho = k.rho_g + phi * (k.rho_l - k.rho_g);
        const double ph = p / k.cs2, uu = ux * ux + uy * uy;
        double hsum = 0.0;
        for (int i = 1; i < 9; ++i) {
            const double eu = EX[i] * ux + EY[i] * uy;
            const S hv = S(phi * wgt<double>(i) * (1 + 3 * eu));
            A[pidx<S>(PL::H + i, n)] = hv;
            hsum += double(hv);
        }
        const double h0 = phi - hsum;  // rest population closes the node's phi exactly
        const S hi = S(h0);
        A[pidx<S>(PL::H, n)] = hi;
        if (RMASS) A[pidx<S>(PL::LO, n)] = S(h0 - double(hi));
        for (int i = 0; i < 9; ++i) {
            const double eu = EX[i] * ux + EY[i] * uy;
            const double w = wgt<double>(i);
            A[pidx<S>(PL::Z + i, n)] =
                S(ph * (i == 0 ? w - 1 : w) + rho * w * (3 * eu + 4.5 * eu * eu - 1.5 * uu));
        }
        A[pidx<S>(PL::PU, n)] = S(phi * ux);
        A[pidx<S>(PL::PU + 1, n)] = S(phi * uy);
    }
}

__global__ void k_d1_init(D1K k, const double* __restrict__ T, double* __restrict__ g) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= k.n) return;
    if (k.q == 3) {
        const double w[3] = {4.0 / 6, 1.0 / 6, 1.0 / 6};
        for (int i = 0; i < 3; ++i) g[i * k.n + x] = w[i] * T[x];
    } else {
        g[x] = 0.5 * T[x];
        g[k.n + x] = 0.5 * T[x];
    }
}

// ---------------------------------------------------------------------------
// FP64 macros of the stored state
// ---------------------------------------------------------------------------
template <typename S>
__global__ void k_chan_macros(ChanK k, const S* __restrict__ A, MacroOut out) {
    const long long N = (long long)k.batch * k.nx * k.ny;
    for (long long n = blockIdx.x * (long long)blockDim.x + threadIdx.x; n < N;
         n += (long long)gridDim.x * blockDim.x) {
        double th = 0.0;
        if (k.thermal) {
            double s = 0;
            for (int i = 0; i < k.tq; ++i) s += double(A[bidx(k.npl, 9 + i, n)]);
            th = s + 0.5 * k.qdt;
        }
        double fx, fy;
        chan_force(k, th, fx, fy);
        double d[9], drho, rho, ux, uy;
        chan_flow_macros<double, S>(A, k.npl, n, k.rho_ref, fx, fy, d, drho, rho, ux, uy);
        out.put(0, n, rho);
        out.put(2, n, ux * k.c);
        out.put(3, n, uy * k.c);
        out.put(4, n, k.T_ref + th);
    }
}

__global__ void k_d1_macros(D1K k, const double* __restrict__ g, MacroOut out) {
    const int x = blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= k.n) return;
    double s = 0;
    for (int i = 0; i < k.q; ++i) s += g[i * k.n + x];
    out.put(4, x, s + 0.5 * k.qdt);
}

// ---------------------------------------------------------------------------
// deterministic FP64 reductions
// ---------------------------------------------------------------------------
__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

template <int NF>
__device__ void block_sums(double (&v)[NF], double* dst, int stride) {
    __shared__ double red[NF][4];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const double s = wave_sum(v[f]);
        if (lane == 0) red[f][wv] = s;
    }
    __syncthreads();
    if (threadIdx.x == 0)
#pragma unroll
        for (int f = 0; f < NF; ++f) dst[f * stride] = ((red[f][0] + red[f][1]) + red[f][2]) + red[f][3];
}

// pass 1: grid (kRedBlocks, batch), 256 threads; partial[(b*4 + f) * kRedBlocks + blk]
template <typename S>
__global__ __launch_bounds__(256) void k_reduce1(int lattice, ChanK ck, PhaseK pk, D1K dk,
                                                 D3K d3, P3K p3, const S* __restrict__ pops,
                                                 int npop, double* __restrict__ partial) {
    const int b = blockIdx.y;
    long long M, P;
    if (lattice == LBM_D2Q9_PHASE) { M = (long long)pk.nx * pk.ny; P = pk.P; }
    else if (lattice == LBM_D2Q9_D2Q5) { M = (long long)ck.nx * ck.ny; P = ck.P; }
    else if (lattice == LBM_D3Q19) { M = (long long)d3.nx * d3.ny * d3.nz; P = d3.P; }
    else if (lattice == LBM_D3Q19_PHASE) { M = (long long)p3.nx * p3.ny * p3.nz; P = p3.P; }
    else { M = dk.n; P = dk.n; }
    const long long base = b * M;
    double v[4] = {0, 0, 0, 0};
    for (long long j = blockIdx.x * 256LL + threadIdx.x; j < M; j += 256LL * gridDim.x) {
        const long long n = base + j;
        // value i of node n: node blocks for the 2D and 3D lattices, planes
        // of stride P for the 1D ones
        auto at = [&](int i) {
            constexpr int npl3 = std::is_same<S, float>::value ? 42 : 41;
            const long long j = lattice == LBM_D2Q9_PHASE    ? pidx<S>(i, n)
                                : lattice == LBM_D2Q9_D2Q5   ? bidx(ck.npl, i, n)
                                : lattice == LBM_D3Q19       ? bidx(19, i, n)
                                : lattice == LBM_D3Q19_PHASE ? bidx(npl3, i, n)
                                                             : i * P + n;
            return double(pops[j]);
        };
        double cnt = 0;
        for (int i = 0; i < npop; ++i)
            if (!isfinite(at(i))) cnt += 1;
        v[3] += cnt;
        if (lattice == LBM_D2Q9_PHASE) {
            double a = 0;
            for (int i = 0; i < 9; ++i) a += at(PhasePlanes<S>::H + i);
            if (std::is_same<S, float>::value) a += at(PhasePlanes<S>::LO);
            v[1] += a;
            v[0] += pk.rho_g + a * (pk.rho_l - pk.rho_g);
        } else if (lattice == LBM_D3Q19_PHASE) {
            double a = 0;
            for (int i = 0; i < 19; ++i) a += at(i);
            if (std::is_same<S, float>::value) a += at(38);
            v[1] += a;
            v[0] += p3.rho_g + a * (p3.rho_l - p3.rho_g);
        } else if (lattice == LBM_D3Q19) {
            double a = 0;
            for (int i = 0; i < 19; ++i) a += at(i);
            v[0] += d3.rho_ref + a;
        } else if (lattice == LBM_D2Q9_D2Q5) {
            double a = 0;
            for (int i = 0; i < 9; ++i) a += at(i);
            v[0] += ck.rho_ref + a;
            if (ck.thermal) {
                double s = 0;
                for (int i = 0; i < ck.tq; ++i) s += at(9 + i);
                v[2] += ck.T_ref + s + 0.5 * ck.qdt;
            }
        } else {
            double s = 0;
            for (int i = 0; i < dk.q; ++i) s += double(pops[i * dk.n + n]);
            v[2] += s + 0.5 * dk.qdt;
        }
    }
    block_sums<4>(v, partial + (long long)b * 4 * kRedBlocks + blockIdx.x, kRedBlocks);
}

// Non-finite watch: every node value of planes [0, nplanes) (N nodes; plane
// stride P, or the node-block layout of nplanes planes when blocked) that is
// NaN or infinite lowers *first to t.  Grid (blocks, planes).
template <typename S>
__global__ __launch_bounds__(256) void k_nonfinite_watch(const S* __restrict__ pops, long long P,
                                                         long long N, int blocked,
                                                         unsigned long long t,
                                                         unsigned long long* __restrict__ first) {
    const int i = blockIdx.y;
    bool bad = false;
    for (long long n = blockIdx.x * 256LL + threadIdx.x; n < N; n += 256LL * gridDim.x)
        bad |= !isfinite(pops[blocked ? bidx(gridDim.y, i, n) : i * P + n]);
    if (bad) atomicMin(first, t);
}

// pass 2: one thread per (replica, field), fixed-order sum
__global__ void k_reduce2(const double* __restrict__ partial, double* __restrict__ out, int nb) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nb * 4) return;
    const double* p = partial + (long long)t * kRedBlocks;
    double s = 0;
    for (int i = 0; i < kRedBlocks; ++i) s += p[i];
    out[t] = s;
}

// Channel diagnostics of replica 0.  A workgroup takes kNuCols columns: its
// threads evaluate the nodes of kNuRows rows at a time into LDS and one thread
// per column adds them in row order (one thread per column doing both waited
// for memory row after row: 143 us on 1600 x 80).
constexpr int kNuCols = 16, kNuRows = 64;
template <typename S>
__global__ __launch_bounds__(256) void k_nusselt(ChanK k, const S* __restrict__ A,
                                                 const S* __restrict__ qw, double qsi, double Dh,
                                                 double kc, double dx, double* __restrict__ Tb,
                                                 double* __restrict__ Tw, double* __restrict__ Nu) {
    __shared__ double su_[kNuRows][kNuCols], sT_[kNuRows][kNuCols];
    const int c = threadIdx.x % kNuCols, r0 = threadIdx.x / kNuCols;
    const int x = blockIdx.x * kNuCols + c;
    double su = 0, suT = 0, T0 = 0, T1 = 0;
    for (int yb = 0; yb < k.ny; yb += kNuRows) {
        const int rows = min(kNuRows, k.ny - yb);
        if (x < k.nx)
            for (int r = r0; r < rows; r += 256 / kNuCols) {
                const long long n = (long long)(yb + r) * k.nx + x;
                double s = 0;
                for (int i = 0; i < k.tq; ++i) s += double(A[bidx(k.npl, 9 + i, n)]);
                const double T = k.T_ref + s + 0.5 * k.qdt;
                double fx, fy;
                chan_force(k, T - k.T_ref, fx, fy);
                double d[9], drho, rho, ux, uy;
                chan_flow_macros<double, S>(A, k.npl, n, k.rho_ref, fx, fy, d, drho, rho, ux, uy);
                su_[r][c] = ux;
                sT_[r][c] = T;
            }
        __syncthreads();
        if (r0 == 0)
            for (int r = 0; r < rows; ++r) {
                su += su_[r][c];
                suT += su_[r][c] * sT_[r][c];
                if (yb + r == 0) T0 = sT_[r][c];
                if (yb + r == k.ny - 1) T1 = sT_[r][c];
            }
        __syncthreads();
    }
    if (r0 != 0 || x >= k.nx) return;
    const double q = double(qw[x]) * qsi;  // W/m^2 including the time modulation
    const double tb = suT / su;
    // wall temperature: mean of the two wall-adjacent nodes, or the lower one
    // with a symmetry plane on top; plus the half-cell conduction q dx / 2k
    const double tw = (k.bcy == 2 ? T0 : 0.5 * (T0 + T1)) + q * dx / (2.0 * kc);
    Tb[x] = tb;
    Tw[x] = tw;
    Nu[x] = q * Dh / (kc * (tw - tb));
}

// mean of Nu over x >= x_dev (strided partial sums, then a tree) and T_b at the outlet
__global__ __launch_bounds__(256) void k_nusselt_mean(const double* __restrict__ Nu,
                                                      const double* __restrict__ Tb, int nx,
                                                      int x_dev, double* __restrict__ out) {
    __shared__ double part[256];
    double s = 0;
    for (int x = x_dev + int(threadIdx.x); x < nx; x += 256) s += Nu[x];
    part[threadIdx.x] = s;
    for (int half = 128; half > 0; half /= 2) {
        __syncthreads();
        if (int(threadIdx.x) < half) part[threadIdx.x] += part[threadIdx.x + half];
    }
    if (threadIdx.x == 0) {
        out[0] = part[0] / double(nx - x_dev);
        out[1] = Tb[nx - 1];
    }
}

inline unsigned grid1(long long N, int bs) {
    long long g = (N + bs - 1) / bs;
    if (g > 65535LL * 16) g = 65535LL * 16;
    return unsigned(g < 1 ? 1 : g);
}

}  // namespace

// ---------------------------------------------------------------------------
// launch wrappers
// ---------------------------------------------------------------------------
// The channel step runs on one-row tiles (64 x 1, one wave per workgroup) at
// every size.  On the paper-sized channels they spread the grid over more CUs
// than 64 x 4 tiles (C2's 800 x 40 under graph replay 5.37 -> 5.15 us per
// step, C5's 1600 x 80 6.37 -> 6.23 us; two-row tiles 5.27 and 6.15), and on
// the 16384 x 2048 grid the step takes 0.715-0.723 ms against 0.728-0.737 ms
// with 64 x 4 tiles (64 x 2: 0.715-0.722; 64 x 8: 0.771; 64 x 4 capped at
// four or three workgroups per CU by an LDS reserve: 0.793 and 1.236 ms).
// An LDS reserve per one-wave workgroup caps the waves resident per CU: 26
// in FP32 (the register count alone allows 32), 12 in FP64 (20).  With more
// waves, more population streams are open in DRAM at once; on the 16384 x
// 2048 grid: FP32 0.700 ms per step uncapped, 0.666 ms at 26 or 30 waves,
// 0.671 at 22 or 24, 0.699 at 20, 0.737 at 16; FP64 1.420 ms uncapped,
// 1.349 at 16, 1.318 at 12, 1.360 at 10, 1.429 at 8.  The paper-sized grids
// (launch-bound) are unchanged.
constexpr unsigned kChanLdsReserve32 = 6144, kChanLdsReserve64 = 13312;
template <typename S>
hipError_t launch_chan_step(const ChanK& k, const S* a, S* b, const S* qw, const S* uin,
                            const S* tin, double mod, hipStream_t s) {
    const long long tiles = (long long)((k.nx + 63) / 64) * k.ny * k.batch;
    dim3 blk(64), grd(unsigned((tiles + kXCD - 1) / kXCD * kXCD));
    const unsigned lds = sizeof(S) == 4 ? kChanLdsReserve32 : kChanLdsReserve64;
    if (k.tq == 9)
        hipLaunchKernelGGL((k_chan_step<S, 9>), grd, blk, lds, s, k, a, b, qw, uin, tin, S(mod));
    else
        hipLaunchKernelGGL((k_chan_step<S, 5>), grd, blk, lds, s, k, a, b, qw, uin, tin, S(mod));
    return hipGetLastError();
}

// FP32 steps run on 256-node tiles, four resident per CU (kPhaseLdsReserve).
// Measured against 512-node tiles (two per CU): equal on 1024 replicas of
// 256^2, faster on smaller grids (64 replicas 146 -> 141 us per step, C4's
// 4 x 512 replica under graph replay 5.22 -> 4.61 us).  FP64 steps and the
// macro evaluation keep 512-node tiles (FP64: 4 % slower on 256-node tiles).

// One launch of k_phase with the tile shape for the replica width: 64 x TY,
// or, for nx in {4, 8, 16, 32}, nx x (512 / nx); half as many rows for FP32
// steps.
template <typename S, typename C, bool MACROS>
hipError_t launch_phase_kernel(const PhaseK& k, const S* a, S* b, const MacroOut& out, unsigned lds,
                               hipStream_t s) {
    auto ntiles = [&](int tx, int ty) {
        return (long long)((k.nx + tx - 1) / tx) * ((k.ny + ty - 1) / ty) * k.batch;
    };
    const bool half = !MACROS && std::is_same<S, float>::value;
    auto go = [&](auto kern, int tx, int ty) {
        const long long tiles = ntiles(tx, ty);
        dim3 blk(tx, ty), grd(unsigned((tiles + kXCD - 1) / kXCD * kXCD));
        hipLaunchKernelGGL(kern, grd, blk, lds, s, k, a, b, out);
        return hipGetLastError();
    };
    if (half) {
        switch (k.nx) {
            case 4: return go(k_phase<S, C, MACROS, 4, 64>, 4, 64);
            case 8: return go(k_phase<S, C, MACROS, 8, 32>, 8, 32);
            case 16: return go(k_phase<S, C, MACROS, 16, 16>, 16, 16);
            case 32: return go(k_phase<S, C, MACROS, 32, 8>, 32, 8);
            default: return go(k_phase<S, C, MACROS, TX, TY / 2>, TX, TY / 2);
        }
    }
    switch (k.nx) {
        case 4: return go(k_phase<S, C, MACROS, 4, 128>, 4, 128);
        case 8: return go(k_phase<S, C, MACROS, 8, 64>, 8, 64);
        case 16: return go(k_phase<S, C, MACROS, 16, 32>, 16, 32);
        case 32: return go(k_phase<S, C, MACROS, 32, 16>, 32, 16);
        default: return go(k_phase<S, C, MACROS>, TX, TY);
    }
}

#ifndef LBM_PERSIST_MIN_THREADS
#define LBM_PERSIST_MIN_THREADS 128
#endif

// Tile shape of the many-steps kernel for a workgroup of `threads` threads:
// nx x threads/nx for the narrow replicas (nx = 4, 8, 16, 32), else 64 x
// threads/64 (at least 256 threads, so that a thread holds each ring node).
void persist_shape(const PhaseK& k, int threads, int* tx, int* ty) {
    const bool narrow = k.nx == 4 || k.nx == 8 || k.nx == 16 || k.nx == 32;
    if (!narrow && threads < 256) threads = 256;
    *tx = narrow ? k.nx : 64;
    *ty = threads / *tx;
}

long long persist_tiles(const PhaseK& k, int threads) {
    int tx, ty;
    persist_shape(k, threads, &tx, &ty);
    return (long long)((k.nx + tx - 1) / tx) * ((k.ny + ty - 1) / ty) * k.batch;
}

// At most kPersistMaxTiles tiles; with a one-node tail every tile of a
// replica is watched by one wave, so a replica then has at most 64.
bool persist_ok(const PhaseK& k, int threads) {
    int tx, ty;
    persist_shape(k, threads, &tx, &ty);
    const int gx = (k.nx + tx - 1) / tx, gy = (k.ny + ty - 1) / ty;
    const bool thin = (gx > 1 && k.nx - (gx - 1) * tx < 2) || (gy > 1 && k.ny - (gy - 1) * ty < 2);
    return persist_tiles(k, threads) <= kPersistMaxTiles && !(thin && (long long)gx * gy > 64);
}

// The smallest workgroup (most tiles, least work per CU) that fits; 0 if
// none does.
int persist_threads(const PhaseK& k) {
    for (int t = LBM_PERSIST_MIN_THREADS; t <= 512; t *= 2)
        if (persist_ok(k, t)) return t;
    return 0;
}

bool phase_persist_fits(const PhaseK& k) { return persist_threads(k) != 0; }

template <typename S>
hipError_t launch_phase_persist(const PhaseK& k, S* A, S* B, int nsteps, unsigned epoch0,
                                unsigned* flags, unsigned* err, bool arith64, hipStream_t s) {
    if (arith64 && !std::is_same<S, float>::value) return hipErrorInvalidValue;
    const int threads = persist_threads(k);
    if (!threads || nsteps < 1) return hipErrorInvalidValue;
    int tx, ty;
    persist_shape(k, threads, &tx, &ty);
    const unsigned tiles = unsigned(persist_tiles(k, threads));
    void* args[] = {(void*)&k, (void*)&A, (void*)&B, (void*)&nsteps, (void*)&epoch0, (void*)&flags,
                    (void*)&err};
    auto go = [&](const void* kern) {
        return hipLaunchCooperativeKernel(kern, dim3(tiles), dim3(tx, ty), args, 0, s);
    };
#define LBM_PERSIST_CASE(X, Y)                                                                 \
    if (tx == X && ty == Y)                                                                    \
        return go(arith64 ? reinterpret_cast<const void*>(&k_phase_persist<S, double, X, Y>)   \
                          : reinterpret_cast<const void*>(&k_phase_persist<S, S, X, Y>));
    LBM_PERSIST_CASE(4, 32) LBM_PERSIST_CASE(4, 64) LBM_PERSIST_CASE(4, 128)
    LBM_PERSIST_CASE(8, 16) LBM_PERSIST_CASE(8, 32) LBM_PERSIST_CASE(8, 64)
    LBM_PERSIST_CASE(16, 8) LBM_PERSIST_CASE(16, 16) LBM_PERSIST_CASE(16, 32)
    LBM_PERSIST_CASE(32, 4) LBM_PERSIST_CASE(32, 8) LBM_PERSIST_CASE(32, 16)
    LBM_PERSIST_CASE(64, 4) LBM_PERSIST_CASE(64, 8)
#undef LBM_PERSIST_CASE
    return hipErrorInvalidValue;
}

template <typename S>
hipError_t launch_phase_step(const PhaseK& k, const S* a, S* b, bool arith64, hipStream_t s) {
    const unsigned lds = std::is_same<S, float>::value ? kPhaseLdsReserve : 0u;  // half tiles
    if (arith64) {  // FP32 storage, every step evaluated in FP64
        if (!std::is_same<S, float>::value) return hipErrorInvalidValue;
        return launch_phase_kernel<S, double, false>(k, a, b, MacroOut{}, lds, s);
    }
    return launch_phase_kernel<S, S, false>(k, a, b, MacroOut{}, lds, s);
}

// One wave of 1, 2 or 4 nodes a lane up to 256 nodes, then four waves.
hipError_t launch_d1(const D1K& k, double* g, int nsteps, hipStream_t s) {
    if (k.n < 3 || k.n > 1024) return hipErrorInvalidValue;
    auto go = [&](auto kern, int waves) {
        hipLaunchKernelGGL(kern, dim3(1), dim3(64 * waves), 0, s, k, g, nsteps);
        return hipGetLastError();
    };
    auto pick = [&](auto q) {
        constexpr int Q = decltype(q)::value;
        const int two = (k.n - 1) % 2, four = (k.n - 1) % 4;  // the last node's place in its lane
        if (k.n <= 64) return go(k_d1<Q, 1, 1, 0>, 1);
        if (k.n <= 128) return two ? go(k_d1<Q, 2, 1, 1>, 1) : go(k_d1<Q, 2, 1, 0>, 1);
        if (k.n <= 256)
            return four == 0   ? go(k_d1<Q, 4, 1, 0>, 1)
                   : four == 1 ? go(k_d1<Q, 4, 1, 1>, 1)
                   : four == 2 ? go(k_d1<Q, 4, 1, 2>, 1)
                               : go(k_d1<Q, 4, 1, 3>, 1);
        if (k.n <= 512) return two ? go(k_d1<Q, 2, 4, 1>, 4) : go(k_d1<Q, 2, 4, 0>, 4);
        return four == 0   ? go(k_d1<Q, 4, 4, 0>, 4)
               : four == 1 ? go(k_d1<Q, 4, 4, 1>, 4)
               : four == 2 ? go(k_d1<Q, 4, 4, 2>, 4)
                           : go(k_d1<Q, 4, 4, 3>, 4);
    };
    return k.q == 3 ? pick(std::integral_constant<int, 3>{}) : pick(std::integral_constant<int, 2>{});
}

template <typename S>
hipError_t launch_chan_init(const ChanK& k, const double* fields, S* a, hipStream_t s) {
    const long long N = (long long)k.batch * k.nx * k.ny;
    hipLaunchKernelGGL(k_chan_init<S>, dim3(grid1(N, 256)), dim3(256), 0, s, k, fields, a);
    return hipGetLastError();
}

template <typename S>
hipError_t launch_phase_init(const PhaseK& k, const double* fields, S* a, hipStream_t s) {
    const long long N = (long long)k.batch * k.nx * k.ny;
    hipLaunchKernelGGL(k_phase_init<S>, dim3(grid1(N, 256)), dim3(256), 0, s, k, fields, a);
    return hipGetLastError();
}

hipError_t launch_d1_init(const D1K& k, const double* T, double* g, hipStream_t s) {
    hipLaunchKernelGGL(k_d1_init, dim3((k.n + 255) / 256), dim3(256), 0, s, k, T, g);
    return hipGetLastError();
}

template <typename S>
hipError_t launch_chan_macros(const ChanK& k, const S* a, const MacroOut& out, hipStream_t s) {
    const long long N = (long long)k.batch * k.nx * k.ny;
    hipLaunchKernelGGL(k_chan_macros<S>, dim3(grid1(N, 256)), dim3(256), 0, s, k, a, out);
    return hipGetLastError();
}

template <typename S>
hipError_t launch_phase_macros(const PhaseK& k, const S* a, const MacroOut& out, hipStream_t s) {
    return launch_phase_kernel<S, double, true>(k, a, (S*)nullptr, out, 0u, s);
}

hipError_t launch_d1_macros(const D1K& k, const double* g, const MacroOut& out, hipStream_t s) {
    hipLaunchKernelGGL(k_d1_macros, dim3((k.n + 255) / 256), dim3(256), 0, s, k, g, out);
    return hipGetLastError();
}

template <typename S>
hipError_t launch_reduce(int lattice, const ChanK& ck, const PhaseK& pk, const D1K& dk,
                         const D3K& d3, const P3K& p3, const S* pops, int npop, double* partial,
                         double* out, hipStream_t s) {
    const int batch = lattice == LBM_D2Q9_PHASE    ? pk.batch
                      : lattice == LBM_D2Q9_D2Q5    ? ck.batch
                      : lattice == LBM_D3Q19        ? d3.batch
                      : lattice == LBM_D3Q19_PHASE  ? p3.batch
                                                    : 1;
    hipLaunchKernelGGL(k_reduce1<S>, dim3(kRedBlocks, batch), dim3(256), 0, s, lattice, ck, pk,
                       dk, d3, p3, pops, npop, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_reduce2, dim3((batch * 4 + 63) / 64), dim3(64), 0, s, partial, out,
                       batch);
    return hipGetLastError();
}

template <typename S>
hipError_t launch_nonfinite_watch(const S* pops, long long P, long long N, int nplanes,
                                  bool blocked, unsigned long long t, unsigned long long* first,
                                  hipStream_t s) {
    const long long blocks = std::min<long long>((N + 255) / 256, 1024);
    hipLaunchKernelGGL(k_nonfinite_watch<S>, dim3(unsigned(blocks), nplanes), dim3(256), 0, s,
                       pops, P, N, int(blocked), t, first);
    return hipGetLastError();
}

template <typename S>
hipError_t launch_nusselt(const ChanK& k, const S* a, const S* qw, double qsi, double Dh,
                          double kc, double dx, int x_dev, double* Tb, double* Tw, double* Nu,
                          double* small, hipStream_t s) {
    hipLaunchKernelGGL(k_nusselt<S>, dim3((k.nx + kNuCols - 1) / kNuCols), dim3(256), 0, s, k, a, qw, qsi,
                       Dh, kc, dx, Tb, Tw, Nu);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_nusselt_mean, dim3(1), dim3(256), 0, s, Nu, Tb, k.nx, x_dev, small);
    return hipGetLastError();
}

#define LBM_INST(S)                                                                              \
    template hipError_t launch_chan_step<S>(const ChanK&, const S*, S*, const S*, const S*,     \
                                            const S*, double, hipStream_t);                       \
    template hipError_t launch_phase_step<S>(const PhaseK&, const S*, S*, bool, hipStream_t);    \
    template hipError_t launch_phase_persist<S>(const PhaseK&, S*, S*, int, unsigned, unsigned*,  \
                                                unsigned*, bool, hipStream_t);                    \
    template hipError_t launch_chan_init<S>(const ChanK&, const double*, S*, hipStream_t);       \
    template hipError_t launch_phase_init<S>(const PhaseK&, const double*, S*, hipStream_t);    \
    template hipError_t launch_chan_macros<S>(const ChanK&, const S*, const MacroOut&, hipStream_t); \
    template hipError_t launch_phase_macros<S>(const PhaseK&, const S*, const MacroOut&, hipStream_t); \
    template hipError_t launch_reduce<S>(int, const ChanK&, const PhaseK&, const D1K&,           \
                                         const D3K&, const P3K&, const S*, int, double*,          \
                                         double*, hipStream_t);                                   \
    template hipError_t launch_nonfinite_watch<S>(const S*, long long, long long, int, bool,     \
                                                  unsigned long long, unsigned long long*,       \
                                                  hipStream_t);                                   \
    template hipError_t launch_nusselt<S>(const ChanK&, const S*, const S*, double, double,      \
                                          double, double, int, double*, double*, double*, double*, \
                                          hipStream_t);
LBM_INST(float)
LBM_INST(double)

}  // namespace lbm
