// Internal declarations of liblbm: context, kernel-argument structs and the
// launch wrappers the C-ABI layer calls.  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <string>

#include "lbm.h"

namespace lbm {

// Node-block layout (every 2D and 3D lattice state): nodes in blocks of 64
// consecutive node indices, each block holding all npl values of its nodes,
// value by value (value i of node n at ((n / 64) npl + i) 64 + n mod 64).  A
// wave that loads 64 consecutive nodes reads one contiguous block of npl x
// 256 bytes (FP32); with one plane array per population the same wave opens
// npl separate streams.  Measured against planes: two-phase D2Q9 single step
// 2.25 -> 2.01 ms (67 M nodes), two-step launch 2.31 -> 2.25 ms, D3Q19 and 3D
// two-phase steps 3-7 % faster.  The padding of the last block is never read
// or written.
constexpr int kBlk = 64;
// the lattices whose state is stored in node blocks (the others keep one
// plane of stride P per population)
inline bool node_blocked(int lattice) {
    return lattice == LBM_D2Q9_PHASE || lattice == LBM_D2Q9_D2Q5 || lattice == LBM_D3Q19 ||
           lattice == LBM_D3Q19_PHASE;
}
__host__ __device__ __forceinline__ long long bidx(int npl, int i, long long n) {
    return ((n >> 6) * npl + i) * kBlk + (n & (kBlk - 1));
}

// Kernel constants of the D2Q9 momentum + D2Q5 temperature step.  Everything
// is pre-scaled by the host into lattice-normalised form (velocities in units
// of c, forces as F dt^2/dx, rates as Lambda dt): the dimensional matrix of
// Sec. 3 is the lattice matrix with rows scaled by c^order, so moment-space
// relaxation gives identical populations in either normalisation.
struct ChanK {
    int nx, ny, batch;
    long long P;          // plane stride of the FP64 staging fields (elements)
    int npl;              // values per node of the state (node blocks): f 9, then g 5 or 9
    int bcx, bcy;         // 0 periodic; bcx 1 inlet/outlet, 2 fixed-T walls;
                          // bcy 1 walls, 2 wall at y- + symmetry plane at y+
    int flow, thermal, flow_mrt, thermal_mrt;
    double rho_ref;
    double Lf[9];         // flow rates * dt in the order rho,e,eps,jx,qx,jy,qy,pxx,pxy
    double Ft[2];         // body force * dt^2 / dx
    int tq;               // thermal lattice: 5 (D2Q5) or 9 (D2Q9)
    double Lt[9];         // thermal rates * dt: D2Q5 T,jx,jy,e,pxx; D2Q9 the flow basis
    double qdt;           // qdot * dt (K)
    double c;             // lattice speed dx/dt (m/s), for outputs
    double T_ref;
    double Tw[2];         // bcx 2: wall temperature - T_ref at x- and x+ (K)
    int buoy;             // Boussinesq force on
    double Bt[2];         // its lattice force per kelvin: -rho_ref beta g dt^2 / dx
};

struct PhaseK {
    int nx, ny, batch;
    long long P;
    int bcy;              // 0 periodic, 1 walls (x periodic)
    int z_mrt, qy_printed, visc_mode;
    double rho_l, rho_g;
    double nuh_l, nuh_g;  // lattice viscosities nu dt/dx^2 (visc_mode 0)
    double zh_l, zh_g;    // zeta dt/dx^2 (visc_mode 1)
    double w_phi;         // dt / tau_phi
    double beta;          // 12 sigma / W        (Pa)
    double kap6;          // 6 kappa / dx^2      (Pa): mu = 4 beta phi(phi-1)(phi-1/2) - kap6 L
    double fs_scale;      // 3 dt^2 / dx^2: F~_s = mu G fs_scale
    double Fbt[2];        // body force * dt^2 / dx
    double dxW;           // dx / W
    double Geps;          // |G| threshold for n = 0 (= normal_eps dx / 3)
    double c, cs2;        // outputs
    __host__ __device__ __forceinline__ double drho() const { return rho_l - rho_g; }
    __host__ __device__ __forceinline__ double dnuh() const { return nuh_l - nuh_g; }
    __host__ __device__ __forceinline__ double dzh() const { return zh_l - zh_g; }
};

// Derivatives of the relaxation rates (times dt) with respect to tau and tau_T,
// in 1/s, and the flux boundary coefficient dt / (dx rho_cp).
struct AdjK {
    double dLf[9];
    double dLt[5];
    double qgrad;
    double cLf[9], cLt[5];  // -dL / squared row norm (MRT); BGK: cLf[7] = -dLf[7]
    int rows_f, rows_t;     // bit q: cLf[q], cLt[q] is not zero
};

// D3Q19 momentum: lattice-normalised like ChanK
struct D3K {
    int nx, ny, nz, batch;
    long long P;
    int bcx, bcy, bcz;    // per axis: 0 periodic, 1 halfway walls on both sides
    double rho_ref;
    double L[19];         // rates * dt in the basis order rho, e, eps, j_x, q_x, j_y, q_y,
                          // j_z, q_z, 3p_xx, 3pi_xx, p_ww, pi_ww, p_xy, p_yz, p_xz, m_x, m_y, m_z
    double Ft[3];         // body force * dt^2 / dx
    double c;             // dx / dt (outputs)
};

// 3D two-phase model (h_i and z_i on D3Q19), lattice-normalised like PhaseK
struct P3K {
    int nx, ny, nz, batch;
    long long P;
    int bcx, bcy, bcz;    // per axis: 0 periodic, 1 halfway walls on both sides
    int z_mrt, visc_mode;
    double rho_l, rho_g;
    double nuh_l, nuh_g;  // nu dt / dx^2 (visc_mode 0)
    double zh_l, zh_g;    // zeta dt / dx^2 (visc_mode 1)
    double w_phi;         // dt / tau_phi
    double beta;          // 12 sigma / W (Pa)
    double kap6;          // 6 kappa / dx^2 (Pa)
    double fs_scale;      // 3 dt^2 / dx^2
    double Fbt[3];        // body force * dt^2 / dx
    double dxW;           // dx / W
    double Geps;          // |G| threshold for n = 0
    double c, cs2;        // outputs
    __host__ __device__ __forceinline__ double drho() const { return rho_l - rho_g; }
    __host__ __device__ __forceinline__ double dnuh() const { return nuh_l - nuh_g; }
    __host__ __device__ __forceinline__ double dzh() const { return zh_l - zh_g; }
};

// Where the macro kernels put the FP64 fields (rho, p, ux, uy, T, phi, mu, uz,
// the bits of the macro mask): null where a field is not wanted.
struct MacroOut {
    double* p[8] = {nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr};
    __device__ __forceinline__ void put(int field, long long n, double v) const {
        if (p[field]) p[field][n] = v;
    }
};

// Whether kernels on GPU `device` may write to memory of these attributes straight
// away: its own device memory.  Another GPU's needs peer access that nobody need have
// enabled, and host memory that is not registered faults; a copy reaches all of them.
inline bool kernel_may_write(const hipPointerAttribute_t& a, int device) {
    return a.type == hipMemoryTypeDevice && a.device == device;
}

// Expected time of a single channel step that reads and writes that many bytes,
// in us (measured: 5.2 us on 800 x 40, 22.2 us on 3000 x 300, 182 us on 8192 x 1024
// in FP32).
inline double chan_single_cost(double bytes) { return 4.6 + bytes / 5.6e6; }

// The same of a single two-phase D2Q9 step (measured: FP32 10.6 us on 4 x 256^2, 22 us
// on 1003 x 701, 260 us on 128 x 256^2; FP64 14.5, 36.5 and 490 us; beyond the
// memory-side cache at the rate of HBM, in FP64 below 100 MB at the caches' 9 TB/s).
// FP64 arithmetic on an FP32 state: 28 us on 1003 x 701, 303 us on 128 x 256^2.
inline double phase_single_cost(double bytes, bool f64, bool arith64) {
    if (arith64) return 5.3 + bytes / (bytes < 3e8 ? 5.1e6 : 4.7e6);
    const double near = f64 ? (bytes < 1e8 ? 9.0e6 : 7.4e6) : 7.0e6;
    return (f64 ? 6.2 : 4.8) + bytes / (bytes < 3e8 ? near : 4.9e6);
}

// Tiles and steps per launch of the many-steps channel kernel (lbm_chan_multi.hip);
// steps 0: not used.
constexpr int kChanMultiMax = 16;
struct ChanMultiPlan {
    int steps = 0, ntx = 0, nty = 0;
    double cost = 0.0;  // expected time of a step (us)
    int cus = 0;        // compute units it was made for
};

// Whether the many-steps reverse kernel beats single reverse steps on a plan's tiles,
// `waves` waves each.  A reverse step is three times the arithmetic of a forward one
// (600 VALU instructions a node in FP32 without a body force), so the overlap weighs
// more: it is taken while the plan puts at most four waves on a SIMD, two in FP64.
// Measured per reverse step with its share of the recomputed tape, single -> many:
// 1600 x 80 FP32 (four waves) 13.8 -> 12.0 us, 300 x 20 10.7 -> 7.8 us; 1600 x 80 FP64
// (eight) 21.2 -> 21.9 us.
inline bool adj_multi_pays(const ChanMultiPlan& p, long long waves, size_t value_bytes) {
    const long long tiles = (long long)p.ntx * p.nty;
    return p.cus > 0 && (tiles + p.cus - 1) / p.cus * waves <= (value_bytes == 4 ? 16 : 8);
}

// Steps per launch (2 to 4) and row segments per replica of a marching 2D kernel,
// with the expected time of a step (us); steps 0: not usable.
struct MarchPlan {
    int steps = 0, nseg = 0;
    double cost = 0.0;
    bool fast = false;  // expected to beat the other kernels (automatic mode takes it)
    int lanes = 256;    // per workgroup
};

// Tiles and steps per launch of the many-steps two-phase kernel
// (lbm_phase_multi.hip); steps 0: not used.
constexpr int kPhaseMultiMax = 8;  // the plan search ends here; longer launches are not measured
struct PhaseMultiPlan {
    int steps = 0, ntx = 0, nty = 0;
    double cost = 0.0;
};

// Tiles per plane and z segments per replica of the 3D two-phase step that
// sums phi as it marches; ntx 0: not used.
struct P3MarchPlan {
    int ntx = 0, nty = 0, nseg = 0;
};

// Tiles per plane and z segments per replica of the two-step D3Q19 kernel;
// ntx 0: not used.
struct D3Tb2Plan {
    int ntx = 0, nty = 0, nseg = 0;
    bool fast = false;  // expected to beat single steps (automatic mode takes it)
};

struct D1K {
    int n, q;
    double w_tau;         // dt / tau
    double qdt;           // qdot * dt
    double ufac;          // always 0; its bytes belong to the parameter hash of saved states
    double T0, TL;
};

}  // namespace lbm

struct lbm_ctx {
    lbm_desc desc;
    int device;
    hipStream_t stream;
    // layout
    long long N;          // nodes per replica * batch
    long long P;          // plane stride
    int npop;             // population planes (non-finite checks, reductions)
    int nplanes;          // planes per state buffer: npop, plus (phi u) for PHASE
    size_t esize;         // bytes per population value
    char* popA;
    char* popB;
    char* aux;            // flux (qw), inlet_u (uin), inlet_T (tin): storage type
    double* staging;      // 8 planes of FP64
    double* partial;      // reduction partials
    double* scratch;      // device address of the static scratch of lbm_reduce_noalloc
    unsigned long long* watch;  // first step with a non-finite state seen (~0: none)
    int watch_every = 4096;     // steps between non-finite checks (0: off)
    double fp32_forcing_share = 0.0;  // per-step share of the slowest forced mode (guard)
    double* small;        // small FP64 results
    int cur;              // 0: A holds the state, 1: B holds it
    long long t;          // steps since init
    bool has_params, has_state;
    lbm_params_si sp;     // SI scalars (array pointers cleared)
    lbm::ChanK ck;
    lbm::PhaseK pk;
    lbm::D1K dk;
    lbm::D3K d3k;
    lbm::P3K p3k;
    char* phi3;           // D3Q19_PHASE: phi of the current state (one plane, storage type)
    double flux_amp, flux_omega, dt;
    double k_cond, Dh, dx, rho_cp;
    std::string err;
    uint64_t hash;
    // adjoint
    lbm::AdjK ak;
    double cs2;
    bool has_record;
    char* rec_work;
    size_t rec_bytes;
    int rec_nsteps, rec_K, rec_nseg;
    long long rec_t0;
    lbm_objective rec_obj;
    // step replay: graph_steps (even) steps captured once per buffer parity
    // on a private stream and replayed on `stream`; 0 disables
    int graph_steps = 64;
    hipStream_t cap_stream = nullptr;
    bool own_capture = false;  // while step graphs are being captured
    hipGraphExec_t step_graph[2] = {nullptr, nullptr};
    int graph_swaps[2] = {0, 0};  // buffer swaps made by each captured graph
    // steps: 0 automatic, 1 single-step kernel only, 2 marching or two-step
    // kernels wherever they apply, 3 many steps per cooperative launch
    int fusion = 0;
    lbm::MarchPlan cmarch;              // channel: several steps per marching launch
    lbm::ChanMultiPlan cmulti;          // channel: many steps per launch (automatic mode)
    bool cplans_made = false;
    lbm::PhaseMultiPlan pmulti;         // two-phase D2Q9: many steps per launch (automatic mode)
    bool pplans_made = false;
    lbm::P3MarchPlan p3march;           // 3D two-phase: one marching launch per step
    bool p3march_made = false;
    lbm::D3Tb2Plan d3tb2;               // D3Q19: two steps per launch (automatic mode)
    lbm::MarchPlan pmarch;              // two-phase D2Q9: several steps per marching launch
    bool capture_pairs = false;         // steps the caller captures go in pairs (automatic mode)
    unsigned* persist_flags = nullptr;  // kPersistMaxTiles step counters, then the error word
    unsigned persist_epoch = 0;         // steps taken by persistent launches since the reset
};

namespace lbm {

// Workgroups of `waves` waves of a kernel that a CU holds at once, from its
// registers (512 per lane and SIMD, at most 8 waves) and LDS (160 KB); 0 on
// error.
inline int resident_workgroups(const void* kernel, int waves) {
    hipFuncAttributes f;
    if (hipFuncGetAttributes(&f, kernel) != hipSuccess || waves < 1) return 0;
    const int regs = f.numRegs > 0 ? (f.numRegs + 7) / 8 * 8 : 8;
    const int slots = 4 * (512 / regs < 8 ? 512 / regs : 8);
    const int lds = f.sharedSizeBytes > 0 ? int(163840 / f.sharedSizeBytes) : slots;
    return slots / waves < lds ? slots / waves : lds;
}

constexpr int kRedBlocks = 256;  // first-pass blocks per replica and field

// launch wrappers (lbm_kernels.hip); all enqueue on s and return hipGetLastError()
// one channel step from state a to state b (node blocks: f 0-8, g from 9)
template <typename S>
hipError_t launch_chan_step(const ChanK& k, const S* a, S* b, const S* qw, const S* uin,
                            const S* tin, double mod, hipStream_t s);
// K (2 to 4, FP64 3) channel steps in one marching launch from state a to state b
// where chan_march_fits; mods: the wall-flux modulation of each step, nseg: row
// segments per replica (chan_march_plan, made with the parameters)
bool chan_march_fits(const ChanK& k);
int chan_march_tiles(const ChanK& k, int K);  // x-tiles per row
template <typename S>
MarchPlan chan_march_plan(const ChanK& k);
template <typename S>
hipError_t launch_chan_march(const ChanK& k, int K, const S* a, S* b, const S* qw, const S* uin,
                             const S* tin, const double* mods, int nseg, hipStream_t s);
// nsteps (at most plan.steps) channel steps in one launch: the last state into
// b (tape 0), or the state after step s into b + s tape.  mods: the wall-flux
// modulation of each step.  chan_multi_plan gives steps 0 where the kernel
// does not cover the configuration or another kernel is faster.
// chan_multi_region: nodes of the largest region of the plan's tiles for
// launches of h steps.
template <typename S>
ChanMultiPlan chan_multi_plan(const ChanK& k);
long long chan_multi_region(const ChanK& k, const ChanMultiPlan& p, int h);
// largest workgroup (nodes of a region): 1024 threads in FP32, 512 in FP64,
// whose LDS planes take twice the space
constexpr int chan_multi_max_nodes(size_t value_bytes) { return value_bytes == 4 ? 1024 : 512; }
template <typename S>
hipError_t launch_chan_multi(const ChanK& k, const ChanMultiPlan& plan, const S* a, S* b,
                             const S* qw, const S* uin, const S* tin, const double* mods,
                             int nsteps, long long tape, hipStream_t s);
// one two-phase step from state a to state b (node-block layout); arith64:
// evaluate the step in FP64 on FP32 storage (S = float)
template <typename S>
hipError_t launch_phase_step(const PhaseK& k, const S* a, S* b, bool arith64, hipStream_t s);
// nsteps (at most plan.steps) two-phase steps in one launch; phase_multi_plan
// gives steps 0 where another kernel is faster
template <typename S>
PhaseMultiPlan phase_multi_plan(const PhaseK& k, bool arith64);
long long phase_multi_region(const PhaseK& k, const PhaseMultiPlan& p, int steps);
template <typename S>
hipError_t launch_phase_multi(const PhaseK& k, const PhaseMultiPlan& plan, const S* a, S* b,
                              bool arith64, int nsteps, hipStream_t s);
// several steps in one launch (plan.steps, in FP64 two): a to b
bool phase_march_fits(const PhaseK& k);
// x-tiles per row and threads of a workgroup
int phase_march_tiles(const PhaseK& k, int lanes, int K);
int phase_march_threads(const PhaseK& k, int lanes);
template <typename S>
MarchPlan phase_march_plan(const PhaseK& k, bool arith64);
template <typename S>
hipError_t launch_phase_march(const PhaseK& k, int K, int lanes, int nseg, bool arith64, const S* a, S* b,
                              hipStream_t s);
// *first = min(*first, t) if any node value of the nplanes planes is not
// finite (plane stride P, or the node-block layout when blocked)
template <typename S>
hipError_t launch_nonfinite_watch(const S* pops, long long P, long long N, int nplanes,
                                  bool blocked, unsigned long long t, unsigned long long* first,
                                  hipStream_t s);
// many steps in one cooperative launch for grids that split into at most
// kPersistMaxTiles tiles of 512 threads (phase_persist_fits); flags: one step
// counter per tile (zeroed with the state, advanced to epoch0 + steps), err:
// set when a bounded wait ran out
#ifndef LBM_PERSIST_MAX_TILES
#define LBM_PERSIST_MAX_TILES 16
#endif
constexpr int kPersistMaxTiles = LBM_PERSIST_MAX_TILES;
constexpr size_t kPersistFlagBytes = 256 * ((kPersistMaxTiles + 1) * 4 / 256 + 1);
bool phase_persist_fits(const PhaseK& k);
template <typename S>
hipError_t launch_phase_persist(const PhaseK& k, S* A, S* B, int nsteps, unsigned epoch0,
                                unsigned* flags, unsigned* err, bool arith64, hipStream_t s);
hipError_t launch_d1(const D1K& k, double* g, int nsteps, hipStream_t s);

template <typename S>
hipError_t launch_chan_init(const ChanK& k, const double* fields, S* a, hipStream_t s);
template <typename S>
hipError_t launch_phase_init(const PhaseK& k, const double* fields, S* a, hipStream_t s);
hipError_t launch_d1_init(const D1K& k, const double* T, double* g, hipStream_t s);

// D3Q19 (lbm_d3q19.hip)
long long d3_tiles(const D3K& k);
template <typename S>
hipError_t launch_d3_step(const D3K& k, const S* fc, S* fn, hipStream_t s);
// two steps in one launch; d3_tb2_plan gives ntx 0 where single steps are faster
template <typename S>
D3Tb2Plan d3_tb2_plan(const D3K& k);
long long d3_tb2_threads(const D3K& k, const D3Tb2Plan& p);  // of a plan's widest tile
template <typename S>
hipError_t launch_d3_tb2(const D3K& k, const D3Tb2Plan& plan, const S* fc, S* fn, hipStream_t s);
template <typename S>
hipError_t launch_d3_init(const D3K& k, const double* fields, S* f, hipStream_t s);
template <typename S>
hipError_t launch_d3_macros(const D3K& k, const S* f, const MacroOut& out, hipStream_t s);

// 3D two-phase (lbm_phase3d.hip).  A step is one launch that sums phi as it
// marches (plan from p3_march_plan), or, with an empty plan, two: phi of the
// stored state into one plane, then the step kernel, which reads phi through an
// LDS tile with a one-node halo.  Buffer planes: h 0-18, z 19-37, the low part
// of h_0 at 38 (FP32 only), then (phi u) of the previous step (3 planes).
template <typename S>
P3MarchPlan p3_march_plan(const P3K& k);
long long p3_march_threads(const P3K& k, const P3MarchPlan& p);  // of a plan's widest tile
template <typename S>
hipError_t launch_p3_step(const P3K& k, const P3MarchPlan& plan, const S* a, S* b, S* phi,
                          hipStream_t s);
template <typename S>
hipError_t launch_p3_init(const P3K& k, const double* fields, S* a, hipStream_t s);
template <typename S>
hipError_t launch_p3_macros(const P3K& k, const S* a, S* phi, const MacroOut& out, hipStream_t s);

// macroscopic fields of the stored state
template <typename S>
hipError_t launch_chan_macros(const ChanK& k, const S* a, const MacroOut& out, hipStream_t s);
template <typename S>
hipError_t launch_phase_macros(const PhaseK& k, const S* a, const MacroOut& out, hipStream_t s);
hipError_t launch_d1_macros(const D1K& k, const double* g, const MacroOut& out, hipStream_t s);

// per-replica FP64 sums: out[b*4 + f], f = mass, phase, energy, nonfinite
template <typename S>
hipError_t launch_reduce(int lattice, const ChanK& ck, const PhaseK& pk, const D1K& dk,
                         const D3K& d3, const P3K& p3, const S* pops, int npop, double* partial,
                         double* out, hipStream_t s);

// qsi converts the stored scaled flux to W/m^2 (including the time modulation);
// small receives (mean Nu over x >= x_dev, Tb[nx-1])
template <typename S>
hipError_t launch_nusselt(const ChanK& k, const S* a, const S* qw, double qsi, double Dh,
                          double kc, double dx, int x_dev, double* Tb, double* Tw, double* Nu,
                          double* small, hipStream_t s);

// ---- discrete adjoint of the heated channel (lbm_adjoint.hip)
// The adjoint state has the layout of the channel state (node blocks: lambda_f
// 0-8, lambda_g 9-13).  Seed at the final state st: lambda into l, and the
// objective's direct derivatives per column (dq_direct[x], dtauT_direct[x])
template <typename S>
hipError_t launch_adj_seed(const ChanK& k, const S* st, const S* qw, double qsi, double mod,
                           double Dh, double kc, double dx, double rho_cp, double cs2, int x_dev,
                           double w_tout, double w_nu, S* l, double* dq_direct,
                           double* dtauT_direct, hipStream_t s);
// one reverse step: lambda(n) into l from lambda(n+1) in ln and the state st at n
template <typename S>
hipError_t launch_adj_step(const ChanK& k, const AdjK& a, const S* st, const S* ln, S* l,
                           double mod, double* dq_bot, double* dq_top, double* dtau_acc,
                           hipStream_t s);
// nsteps reverse steps in one launch on the tiles of a channel plan: st the
// state of the first, stride (in values, negative) to the next; mods in that
// order.  adj_multi_fast: whether that beats single reverse steps.
template <typename S>
bool adj_multi_fast(const ChanK& k, const ChanMultiPlan& plan);
template <typename S>
hipError_t launch_adj_multi(const ChanK& k, const AdjK& a, const ChanMultiPlan& plan, const S* st,
                            long long stride, const S* ln, S* l, const double* mods, int nsteps,
                            double* dq_bot, double* dq_top, double* dtau_acc, hipStream_t s);
// gradient assembly (fixed order): grad_flux[nx], grad_tau[2]
hipError_t launch_adj_final(int nx, int ntiles, double scale, const double* dq_bot,
                            const double* dq_top, const double* dq_direct,
                            const double* dtauT_direct, const double* dtau_acc,
                            double* grad_flux, double* grad_tau, hipStream_t s);
int chan_tiles(const ChanK& k);

}  // namespace lbm
