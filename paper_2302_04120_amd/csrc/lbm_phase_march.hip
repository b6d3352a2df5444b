// Several two-phase D2Q9 steps per launch on grids that fill the GPU (temporal
// blocking): the state crosses HBM once per K steps.
//
// A workgroup takes one x-tile of one row segment [a, e) of one replica.  Rows of
// up to 256 columns are one tile, a lane per column, that wraps in x (WHOLE);
// longer ones go in tiles of 128 or 256 lanes that store 4 K columns less.  It marches up
// the rows; at row step v, stage s (0 .. K - 1) collides step n + s at row v - 2 s:
//   - phi of the rows around it comes from the stage's ring of four rows in LDS;
//   - the x-moving values go to the neighbour lanes through LDS;
//   - each lane pulls the state of step n + s + 1: the values that move down
//     complete row v - 2 s - 1, whose phi goes into the next stage's ring and which
//     that stage collides a row step later (kept in LDS until then); the values that
//     stay in row v - 2 s start it (W), those that move up wait for the next row (U).
// The last stage's completed row is stored.  A step reaches two nodes (phi of the
// neighbours' populations), so stage s is exact on lanes 2 s + 1 .. LANES - 2 - 2 s of a
// tile and runs on rows a - 2 (K - s) + 1 .. e + 2 (K - s) - 2 (between walls those
// that exist): tiles and segments are independent.  The arithmetic per node is that
// of the single-step kernel (phi_sum, phase_local, phase_collide): K steps here
// equal K single steps bit for bit.  C, the type of the arithmetic, may be wider than
// the state's type S: every stage rounds to S where a single step stores.
//
// The stages share one exchange buffer: the first barrier of the next stage lies
// between a stage's reads and the next writes.  Two row steps per loop iteration let
// the loop-carried rows change registers without copies (6 % of the instructions).
// The prefetched row is waited for before the stores of a row step, since a wait
// after them would wait for the stores too.
//
// Bound: at K = 3 in FP32 the vector ALU (1180 instructions a row step, two waves
// per SIMD at 215 to 220 registers, 79 % of its cycles issue); 2048 x 2048 moves the
// launch's bytes at 3.6 TB/s.  Four stages would need 91 KB of LDS a workgroup, one
// per CU.  FP64 takes two steps: 310 registers, one wave per SIMD (held to 256
// registers it spills and takes 1.9 times as long); FP64 arithmetic on an FP32 state,
// which keeps the rows in FP32, two steps in 252.  The scheme this replaces
// accumulated three rows of the next state in registers (225) for two steps.
//
// ALIGNED: nx a multiple of 64 and a row's node blocks under 2 GiB, so every row
// starts on a node block and an access is the row's block base (uniform) plus a
// 32-bit lane offset.
#include "lbm_phase.h"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace lbm {
namespace {

template <typename C>
struct PhaseMarchArgs {
    PhaseKT<C> k;
    int ntx, nseg, wy, ey;  // tiles per row; segment i spans wy rows, one more for i < ey
};

// The state of a node: h 0-8, z 0-8, (phi u), the low part of h_0 (FP32).
constexpr int mH = 0, mZ = 9, mPU = 18, mLO = 20, mNS = 21;

template <typename S, typename C, bool WHOLE, bool ALIGNED, int LANES, int K>
__global__ __launch_bounds__(LANES) void k_phase_march(const PhaseMarchArgs<C> p,
                                                          const S* __restrict__ A,
                                                          S* __restrict__ B) {
    using PL = PhasePlanes<S>;
    constexpr bool RMASS = std::is_same<S, float>::value;
    constexpr int HALO = 2 * K, OUT = LANES - 2 * HALO;
    __shared__ C ring[K][4][LANES];  // phi of each stage's state, rows mod 4
    __shared__ S xb[12][LANES];      // x-moving post-collision values
    constexpr int NS = PL::NPL;         // LO last: FP64 has none
    __shared__ S next[K > 1 ? K - 1 : 1][NS][LANES];  // the row stages after the first collide next
    const auto& k = p.k;
    const int nx = k.nx, ny = k.ny;
    int w, tx, sg, b;
    if (!xcd_tile(p.ntx * p.nseg * k.batch, w)) return;  // whole workgroup, before any barrier
    block_divide(w, p.ntx, w, tx);
    block_divide(w, p.nseg, b, sg);
    const int a = sg * p.wy + min(sg, p.ey), e = a + p.wy + (sg < p.ey);
    const bool walls = k.bcy != 0;
    const long long base = (long long)b * ny * nx;
    const unsigned lx = threadIdx.x;
    int xi;
    bool own;
    unsigned lxm, lxp;
    if constexpr (WHOLE) {  // the row wraps in LDS; lanes beyond it shadow the last column
        xi = min(int(lx), nx - 1);
        own = int(lx) < nx;
        lxm = xi == 0 ? nx - 1 : xi - 1;
        lxp = xi == nx - 1 ? 0 : xi + 1;
    } else {
        const int col = tx * OUT - HALO + int(lx);
        xi = col;
        while (xi < 0) xi += nx;
        while (xi >= nx) xi -= nx;
        own = int(lx) >= HALO && int(lx) < LANES - HALO && col < nx;
        lxm = lx == 0 ? 0u : lx - 1;
        lxp = lx == LANES - 1 ? lx : lx + 1;
    }
    const unsigned x = unsigned(xi);
    auto rowof = [&](int v) {
        while (v < 0) v += ny;
        while (v >= ny) v -= ny;
        return v;
    };
    const unsigned boff =
        ALIGNED ? unsigned(((x >> 6) * PL::NPL * kBlk + (x & (kBlk - 1))) * sizeof(S)) : x;
    auto at = [&](auto* P, int row, int i) {
        const long long ro = base + (long long)row * nx;
        if constexpr (ALIGNED) {
            using B8 = std::conditional_t<std::is_const_v<std::remove_pointer_t<decltype(P)>>,
                                          const char, char>;
            auto* r = (B8*)P + (ro >> 6) * (long long)(PL::NPL * kBlk * sizeof(S));
            return (decltype(P))(r + boff) + i * kBlk;
        } else {
            return P + pidx<S>(i, ro + boff);
        }
    };
    auto load_h = [&](int row, S (&h)[9], S& lo) {
#pragma unroll
        for (int i = 0; i < 9; ++i) h[i] = *at(A, row, PL::H + i);
        lo = RMASS ? *at(A, row, PL::LO) : S(0);
    };
    auto load_rest = [&](int row, S (&s)[mNS]) {
#pragma unroll
        for (int i = 0; i < 9; ++i) s[mZ + i] = *at(A, row, PL::Z + i);
        s[mPU] = *at(A, row, PL::PU);
        s[mPU + 1] = *at(A, row, PL::PU + 1);
    };
    auto phi_of = [&](const auto& s, S lo) {
        const C hh[9] = {C(s[0]), C(s[1]), C(s[2]), C(s[3]), C(s[4]), C(s[5]), C(s[6]), C(s[7]), C(s[8])};
        return phi_sum(hh, C(lo));
    };
    // first row and end of the collisions of stage s
    auto lo_of = [&](int s) { const int r = a - (2 * (K - s) - 1); return walls ? max(r, 0) : r; };
    auto hi_of = [&](int s) { const int r = e + (2 * (K - s) - 1); return walls ? min(r, ny) : r; };

    // H0: the row stage 0 collides next, N: h of the row after it (its phi is
    // needed a row early); W[s], U[s]: of the state that stage s builds, the started
    // row and the values that move up from it
    S N[9], Nlo, H0[mNS], W[K][mNS], U[K][6];
#pragma unroll
    for (int s = 0; s < K; ++s) {
#pragma unroll
        for (int i = 0; i < mNS; ++i) W[s][i] = S(0);
        if (s > 0) {
#pragma unroll
            for (int i = 0; i < NS; ++i) next[s > 0 ? s - 1 : 0][i][lx] = S(0);
        }
#pragma unroll
        for (int i = 0; i < 6; ++i) U[s][i] = S(0);
    }
    const int rlo = walls ? 0 : -(1 << 30), rhi = walls ? ny - 1 : 1 << 30;  // phi across a wall: the wall row's
    const int first = lo_of(0), lastrow = walls ? min(e + 2 * K, ny) - 1 : e + 2 * K - 1;
    if (!walls || first > 0) {
        load_h(rowof(first - 1), N, Nlo);
        ring[0][(first - 1) & 3][lx] = phi_of(N, Nlo);
    }
    load_h(rowof(first), N, Nlo);
#pragma unroll
    for (int i = 0; i < 9; ++i) H0[mH + i] = N[i];
    H0[mLO] = Nlo;
    load_rest(rowof(first), H0);
    ring[0][first & 3][lx] = phi_of(N, Nlo);
    int rn = rowof(min(first + 1, lastrow));  // the row of N
    load_h(rn, N, Nlo);
    ring[0][(first + 1) & 3][lx] = phi_of(N, Nlo);

    auto row_step = [&](const int v) __attribute__((always_inline)) {
        S T[mNS];
#pragma unroll
        for (int s = 0; s < K; ++s) {
            const int r = v - 2 * s;
            const bool on = r >= lo_of(s) && r < hi_of(s);
            __syncthreads();  // phi of row r + 1 is in this stage's ring
            // post-collision values, rounded to the storage type
            S hs[9], zst[9], pux = S(0), puy = S(0), h0hi = S(0), h0lo = S(0), hc[mNS];
#pragma unroll
            for (int i = 0; i < mNS; ++i) {
                if (s == 0) {
                    hc[i] = H0[i];
                } else if (i < NS) {  // the row below, which stage s - 1 completed an iteration ago
                    hc[i] = next[s > 0 ? s - 1 : 0][i][lx];
                    next[s > 0 ? s - 1 : 0][i][lx] = T[i];
                } else {
                    hc[i] = S(0);
                }
            }
            if (on) {
                const C* rm = ring[s][max(r - 1, rlo) & 3];
                const C* r0 = ring[s][r & 3];
                const C* rp = ring[s][min(r + 1, rhi) & 3];
                const unsigned lc = WHOLE ? unsigned(xi) : lx;
                const C pn[9] = {r0[lc], r0[lxp], rp[lc], r0[lxm], rm[lc], rp[lxp], rp[lxm], rm[lxm], rm[lxp]};
                C h[9], z[9];
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    h[i] = C(hc[mH + i]);
                    z[i] = C(hc[mZ + i]);
                }
                const PhaseLocal<C> L = phase_local<C>(k, pn, z);
                C hw[9], zw[9], pw[2];
                phase_collide<S, C>(k, L, h, C(hc[mLO]), z, C(hc[mPU]), C(hc[mPU + 1]), hw, h0hi, h0lo,
                                    zw, pw[0], pw[1]);
#pragma unroll
                for (int i = 0; i < 9; ++i) {
                    hs[i] = S(hw[i]);
                    zst[i] = S(zw[i]);
                }
                pux = S(pw[0]);
                puy = S(pw[1]);
                const int xm[6] = {1, 3, 5, 6, 7, 8};
#pragma unroll
                for (int j = 0; j < 6; ++j) {
                    xb[j][lx] = hs[xm[j]];
                    xb[6 + j][lx] = zst[xm[j]];
                }
            }
            if (s == 0) {
#pragma unroll
                for (int i = 0; i < 9; ++i) H0[mH + i] = N[i];
                H0[mLO] = Nlo;
                load_rest(rn, H0);
                if (v + 2 <= lastrow) rn = rn + 1 == ny ? 0 : rn + 1;
                load_h(rn, N, Nlo);
            }
            __syncthreads();
            S(&Ws)[mNS] = W[s];
            S(&Us)[6] = U[s];
            if (on) {  // row r - 1 receives the values that move down
                Ws[mH + 4] = hs[4];
                Ws[mH + 7] = xb[4][lxp];
                Ws[mH + 8] = xb[5][lxm];
                Ws[mZ + 4] = zst[4];
                Ws[mZ + 7] = xb[10][lxp];
                Ws[mZ + 8] = xb[11][lxm];
            }
#pragma unroll
            for (int i = 0; i < mNS; ++i) T[i] = Ws[i];
            if (s + 1 < K) ring[s + 1 < K ? s + 1 : 0][(r - 1) & 3][lx] = phi_of(T, T[mLO]);
            if (!on) continue;
            const bool bottom = walls && r == 0, top = walls && r == ny - 1;
            Ws[mH] = h0hi;
            Ws[mLO] = h0lo;
            Ws[mZ] = zst[0];
            Ws[mPU] = pux;
            Ws[mPU + 1] = puy;
            Ws[mH + 1] = xb[0][lxm];
            Ws[mH + 3] = xb[1][lxp];
            Ws[mZ + 1] = xb[6][lxm];
            Ws[mZ + 3] = xb[7][lxp];
            Ws[mH + 2] = bottom ? hs[4] : Us[0];
            Ws[mH + 5] = bottom ? hs[7] : Us[1];
            Ws[mH + 6] = bottom ? hs[8] : Us[2];
            Ws[mZ + 2] = bottom ? zst[4] : Us[3];
            Ws[mZ + 5] = bottom ? zst[7] : Us[4];
            Ws[mZ + 6] = bottom ? zst[8] : Us[5];
            Us[0] = hs[2];
            Us[1] = xb[2][lxm];
            Us[2] = xb[3][lxp];
            Us[3] = zst[2];
            Us[4] = xb[8][lxm];
            Us[5] = xb[9][lxp];
            if (top) {
                Ws[mH + 4] = hs[2];
                Ws[mH + 7] = hs[5];
                Ws[mH + 8] = hs[6];
                Ws[mZ + 4] = zst[2];
                Ws[mZ + 7] = zst[5];
                Ws[mZ + 8] = zst[6];
            }
        }
        // the loads end here, so that they do not wait for the stores below
#pragma unroll
        for (int i = 0; i < 9; ++i) asm volatile("" : "+v"(N[i]), "+v"(H0[mZ + i]));
        asm volatile("" : "+v"(Nlo), "+v"(H0[mPU]), "+v"(H0[mPU + 1]));
        ring[0][(v + 2) & 3][lx] = phi_of(N, Nlo);
        const int r = v - 2 * (K - 1) - 1;
        if (own && r >= a && r < e) {
#pragma unroll
            for (int i = 0; i < 9; ++i) {
                st(at(B, r, PL::H + i), T[mH + i]);
                st(at(B, r, PL::Z + i), T[mZ + i]);
            }
            if constexpr (RMASS) st(at(B, r, PL::LO), T[mLO]);
            st(at(B, r, PL::PU), T[mPU]);
            st(at(B, r, PL::PU + 1), T[mPU + 1]);
        }
    };
    for (int v = first; v <= e + 2 * (K - 1); v += 2) {
        row_step(v);
        row_step(v + 1);
    }
}

template <typename S>
bool phase_march_aligned(const PhaseK& k) {
    return k.nx % kBlk == 0 && (long long)k.nx * PhasePlanes<S>::NPL * (long long)sizeof(S) < (1LL << 31);
}
template <typename S, typename C, int LANES, int K>
auto phase_march_kernel(const PhaseK& k) {
    if (k.nx <= LANES)
        return phase_march_aligned<S>(k) ? k_phase_march<S, C, true, true, LANES, K>
                                         : k_phase_march<S, C, true, false, LANES, K>;
    if constexpr (LANES == 64)  // longer rows go in wider tiles
        return k_phase_march<S, C, true, false, LANES, K>;
    else
        return phase_march_aligned<S>(k) ? k_phase_march<S, C, false, true, LANES, K>
                                         : k_phase_march<S, C, false, false, LANES, K>;
}
template <typename S, typename C, int K>
auto phase_march_kernel(const PhaseK& k, int lanes) {
    using Kernel = decltype(phase_march_kernel<S, C, 64, K>(k));
    return lanes == 64    ? (Kernel)phase_march_kernel<S, C, 64, K>(k)
           : lanes == 128 ? (Kernel)phase_march_kernel<S, C, 128, K>(k)
                          : (Kernel)phase_march_kernel<S, C, 256, K>(k);
}
// waves of a workgroup: those of the row's columns, or all of a tile's lanes
int phase_march_waves(const PhaseK& k, int lanes) { return std::min((k.nx + 63) / 64, lanes / 64); }

template <typename S, typename C, int K>
hipError_t phase_march_launch(const PhaseK& k, int lanes, int nseg, const S* a, S* b, hipStream_t s) {
    if ((lanes != 64 && lanes != 128 && lanes != 256) || (lanes == 64 && k.nx > 64) || nseg < 1 ||
        nseg > k.ny)
        return hipErrorInvalidValue;
    const int ntx = phase_march_tiles(k, lanes, K);
    const long long wgs = (long long)ntx * nseg * k.batch;
    if (wgs >= (1 << 21)) return hipErrorInvalidValue;
    PhaseMarchArgs<C> p{};
    p.k = phase_kt<C>(k);
    p.ntx = ntx;
    p.nseg = nseg;
    p.wy = k.ny / nseg;
    p.ey = k.ny % nseg;
    hipLaunchKernelGGL((phase_march_kernel<S, C, K>(k, lanes)), dim3(unsigned((wgs + kXCD - 1) / kXCD * kXCD)),
                       dim3(unsigned(phase_march_waves(k, lanes) * 64)), 0, s, p, a, b);
    return hipGetLastError();
}

}  // namespace

bool phase_march_fits(const PhaseK& k) { return k.ny >= 4 && k.nx >= 1; }
int phase_march_tiles(const PhaseK& k, int lanes, int K) {
    return k.nx <= lanes ? 1 : (k.nx + lanes - 4 * K - 1) / (lanes - 4 * K);
}
int phase_march_threads(const PhaseK& k, int lanes) { return 64 * phase_march_waves(k, lanes); }

// Lanes per workgroup, steps per launch and segments by a cost model fitted to 1900
// plans on 60 grids of 0.2 M to 12 M nodes (5 %; its choice runs within 4 % of the
// best measured plan on all but the narrowest).  All workgroups of a round march
// seg + 4 K - 2 rows; a row step is the root sum square of
//   the stages' time, the cubic mean of row0 + K lam (the chain of a row: more
//   where four waves meet at the barriers, less in one) and K beta for every four
//   waves of a CU (issue), and
//   the bytes of the resident workgroups at 19.6 (FP64: 14.3; FP64 arithmetic on an
//   FP32 state: 40, where issue hides them) TB/s out of the caches, at 9.2 to 10 TB/s
//   where both buffers outgrow the 256 MB memory-side cache.
// Measured per step, before (the faster of single steps, the two-step scheme above
// and LDS tiles, as automatic mode took them) -> here: FP32 128 replicas of 256^2
// 147 -> 112 us, 32 replicas 73 -> 36, 2048 x 2048 138 -> 66, 4096 x 3000 386 -> 157,
// 4 x 1003 x 701 100 -> 48, 40 x 300 x 280 117 -> 61, 128 x 128^2 73 -> 34, 256 x 64^2
// 32 -> 21; FP64 64 replicas of 256^2 255 -> 151, 2048 x 2048 262 -> 143, 450 x 460 x
// 6 90 -> 49, 1003 x 701 36.7 -> 31.5; FP64 arithmetic on an FP32 state (single steps
// before) 128 x 256^2 303 -> 177, 2048 x 2048 151 -> 94, 4 x 600 x 500 44 -> 35.  128
// lanes instead of 256 waste less of ragged rows, and in FP64, where a SIMD holds one wave, two workgroups fill each other's
// barriers: 2048 x 2048 168 -> 143, 4 x 600 x 500 63 -> 45.  Calls of exactly two or four
// FP32 steps, and captured pairs, go at K = 2 on the segments of K = 3 (others are no
// faster); against the two-step scheme: 2048 x 2048 118 -> 93, 64 x 256^2 87 -> 78, but
// 128 x 256^2 144 -> 150 and 1024 x 256^2 1120 -> 1150.  Rows far narrower than a
// wave (1024 x 4 x 512: single step 72, here 313) stay with the other kernels.
template <typename S, typename C>
MarchPlan march_plan(const PhaseK& k) {
    MarchPlan best{};
    int dev = 0, cus = 0;
    if (!phase_march_fits(k) || hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
        return best;
    constexpr bool F32 = sizeof(C) == 4;
    constexpr bool A64 = !F32 && sizeof(S) == 4;
    const double lam = F32 ? 0.61 : A64 ? 0.76 : 0.915, row0 = F32 ? 0.79 : A64 ? 0.98 : 0.4;
    const double beta = F32 ? 0.417 : A64 ? 0.83 : 1.04, t0 = F32 ? 5.7 : A64 ? 8.9 : 1.9;
    const double one_wave = F32 ? 0.82 : A64 ? 0.6 : 1.0, four_waves = F32 ? 1.14 : A64 ? 0.88 : 1.55;
    const double plane = double(PhasePlanes<S>::NPL) * sizeof(S);
    const double state = double(k.nx) * k.ny * k.batch * plane;
    const double near = F32 ? 19.6e6 : A64 ? 40e6 : 14.3e6, far = F32 ? 9.2e6 : A64 ? 10e6 : 9.7e6;
    const double bw = 2 * state < 3e8 ? near : far;  // bytes per us
    for (int lanes = 64; lanes <= 256; lanes *= 2) {
        // rows in one tile of the fewest lanes, longer ones in tiles of 128 or 256
        if (k.nx <= 256 ? lanes < k.nx || (lanes > 64 && lanes / 2 >= k.nx) : lanes == 64) continue;
        const int waves = phase_march_waves(k, lanes);
        const double row_bytes = 2.0 * std::min(k.nx, lanes) * plane;
        for (int K = 2; K <= (F32 ? 3 : 2); ++K) {
            const int resident = resident_workgroups(
                K == 2 ? (const void*)phase_march_kernel<S, C, 2>(k, lanes)
                       : (const void*)phase_march_kernel<S, C, F32 ? 3 : 2>(k, lanes), waves);
            if (resident < 1) continue;
            const double chain = std::pow(row0 + K * lam * (waves == 1 ? one_wave : waves == 2 ? 1 : four_waves), 3);
            const long long column = (long long)phase_march_tiles(k, lanes, K) * k.batch;
            const long long cap = (long long)cus * resident;
            for (int seg = k.ny; seg >= 1; --seg) {
                const int nseg = (k.ny + seg - 1) / seg;
                if (seg > 1 && (k.ny + seg - 2) / (seg - 1) == nseg) continue;  // shorter, the same count
                const long long wgs = column * nseg;
                if (wgs >= (1 << 21)) break;
                auto row = [&](long long n) {
                    const double issue = K * beta * double((n + cus - 1) / cus) * waves / 4;
                    return std::hypot(std::cbrt(chain + issue * issue * issue), row_bytes * double(n) / bw);
                };
                const double cost = (t0 + (seg + 4 * K - 2) * (double(wgs / cap) * row(cap) +
                                                               (wgs % cap ? row(wgs % cap) : 0.0))) / K;
                if (best.steps == 0 || cost < best.cost) best = MarchPlan{K, nseg, cost, false, lanes};
            }
        }
    }
    return best;
}

template <typename S>
MarchPlan phase_march_plan(const PhaseK& k, bool arith64) {
    return arith64 ? march_plan<S, double>(k) : march_plan<S, S>(k);
}

// K steps in one launch; the whole state (populations and (phi u)) moves from
// buffer a to buffer b.
template <typename S>
hipError_t launch_phase_march(const PhaseK& k, int K, int lanes, int nseg, bool arith64, const S* a, S* b,
                              hipStream_t s) {
    if (!phase_march_fits(k)) return hipErrorInvalidValue;
    if (arith64) return K == 2 ? phase_march_launch<S, double, 2>(k, lanes, nseg, a, b, s) : hipErrorInvalidValue;
    if (K == 2) return phase_march_launch<S, S, 2>(k, lanes, nseg, a, b, s);
    if constexpr (sizeof(S) == 4)
        if (K == 3) return phase_march_launch<S, S, 3>(k, lanes, nseg, a, b, s);
    return hipErrorInvalidValue;
}

#define LBM_PMARCH_INST(S)                                                                         \
    template MarchPlan phase_march_plan<S>(const PhaseK&, bool);                                   \
    template hipError_t launch_phase_march<S>(const PhaseK&, int, int, int, bool, const S*, S*,    \
                                              hipStream_t);
LBM_PMARCH_INST(float)
LBM_PMARCH_INST(double)

}  // namespace lbm
