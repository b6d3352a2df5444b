"""Performance cases of the library: the runs its users make, from the paper-sized grids, where a
step is a few microseconds of latency, to grids that fill the GPU.

A pass advances one lattice by the steps a program takes between two field outputs and reads the
macroscopic fields into a device tensor (``Lattice.step`` then ``Lattice.macros_device``), with the
library's own choice of kernel; the adjoint case evaluates the objective and its gradients
(``ChannelAdjoint``).  Grids, fluids and options are those of ``workloads`` (the paper's cases C1 to
C5, the natural-convection cavity, the paper's half channel and the 3D models) and their neighbours.

``exact`` evaluates the same model in FP64 with plain torch operations, in population space (BGK and
MRT through explicit moment matrices), so that it shares no arithmetic with the kernels.
"""
import math

import numpy as np
import torch

from paper_2302_04120_amd import workloads as WL

# --------------------------------------------------------------------------------------------------
# The cases
# --------------------------------------------------------------------------------------------------


def listed():
    return [
        # C1: the 1D slab with a heat source, FP64, the smallest run of all
        dict(name="slab_c1", kind="slab", n=101, q=2, steps=2000),
        # C2 as the paper sizes it: 800 x 40, FP32, one output every 500 steps
        dict(name="channel_c2", kind="channel", nx=800, ny=40, prec="fp32", mrt=True,
             oscillating=False, steps=500),
        # the paper's own half channel (symmetry plane, D2Q9 temperature), FP32
        dict(name="channel_half", kind="half", case="developed_alternating", H=0.5e-3, L=10e-3,
             prec="fp32", steps=200),
        # a channel that fills the GPU, with an output after a few steps
        dict(name="channel_large", kind="channel", nx=8192, ny=1024, prec="fp32", mrt=True,
             oscillating=False, steps=40),
        # natural convection on the paper's 65 x 65 grid, FP64, frequent output
        dict(name="cavity_ra1e4", kind="cavity", n=65, prec="fp64", steps=25),
        # C3: the four bubble radii as one batch, FP32
        dict(name="bubble_c3", kind="bubble", nx=256, ny=256, batch=4, prec="fp32", steps=200),
        # the bubble cell as a batch that fills the GPU (a parameter sweep), FP32
        dict(name="bubble_batch", kind="bubble", nx=256, ny=256, batch=128, prec="fp32", steps=40),
        # one domain of odd size in FP64
        dict(name="bubble_ragged_fp64", kind="bubble", nx=1003, ny=701, batch=1, prec="fp64",
             steps=40),
        # C4: layered channel flow, 4 x 512, FP32 state with FP64 arithmetic (its long-run mode)
        dict(name="layered_c4", kind="layered", nx=4, ny=512, batch=1, prec="fp32_arith64",
             steps=500),
        # 3D momentum, a periodic box of water
        dict(name="d3q19_box", kind="d3q19", nx=256, ny=256, nz=128, prec="fp32", mrt=True,
             walls=False, steps=20),
        # 3D two-phase, air spheres in water
        dict(name="phase3d_bubbles", kind="phase3d", cell=64, cells=3, prec="fp32", steps=10),
        # C5: objective and gradients of the heated channel, forward and reverse
        dict(name="adjoint_c5", kind="adjoint", nx=1600, ny=80, prec="fp32", steps=500, ckpt=125),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _steps(rng, nodes, most_updates, most=500):
    top = max(4, min(most, int(most_updates / nodes)))
    return _log(rng, max(4, top // 8), top)


def draw(rng):
    kind = rng.choice(["slab", "channel", "channel", "half", "cavity", "bubble", "bubble", "layered",
                       "d3q19", "phase3d", "adjoint"])
    prec = rng.choice(["fp32", "fp32", "fp64"])
    if kind == "slab":
        return dict(kind=kind, n=_log(rng, 33, 1001), q=rng.choice([2, 3]),
                    steps=_log(rng, 200, 2000))
    if kind == "channel":
        nx, ny = _log(rng, 120, 6000), _log(rng, 12, 900)
        return dict(kind=kind, nx=nx, ny=ny, prec=prec, mrt=rng.random() < 0.7,
                    oscillating=rng.random() < 0.3, steps=_steps(rng, nx * ny, 1e8))
    if kind == "half":
        return dict(kind=kind, case=rng.choice(["developed_alternating", "developing_constant",
                                                "developing_alternating"]),
                    H=rng.randrange(20, 200) * 5e-6, L=rng.randrange(200, 2000) * 5e-6, prec=prec,
                    steps=_log(rng, 20, 300))
    if kind == "cavity":
        return dict(kind=kind, n=_log(rng, 33, 500), prec=prec, steps=_log(rng, 10, 300))
    if kind == "bubble":
        nx, ny = _log(rng, 48, 1200), _log(rng, 48, 1200)
        if prec == "fp32" and rng.random() < 0.2:
            prec = "fp32_arith64"
        batch = _log(rng, 1, max(1, min(128, 4000000 // (nx * ny))))
        return dict(kind=kind, nx=nx, ny=ny, batch=batch, prec=prec,
                    steps=_steps(rng, nx * ny * batch, 5e7, 200))
    if kind == "layered":
        return dict(kind=kind, nx=rng.choice([4, 4, 8, 16, 11]), ny=_log(rng, 64, 512),
                    batch=_log(rng, 1, 64), prec=rng.choice(["fp32", "fp32_arith64", "fp64"]),
                    steps=_log(rng, 50, 300))
    if kind == "d3q19":
        nx, ny, nz = (_log(rng, 24, 200) for _ in range(3))
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, prec=prec, mrt=rng.random() < 0.7,
                    walls=rng.random() < 0.4, steps=_steps(rng, nx * ny * nz, 5e7, 100))
    if kind == "phase3d":
        cell, cells = rng.randrange(40, 72), rng.choice([1, 1, 2])
        return dict(kind=kind, cell=cell, cells=cells, prec=prec, steps=_log(rng, 5, 20))
    steps = _log(rng, 80, 400)
    return dict(kind=kind, nx=_log(rng, 150, 1600), ny=_log(rng, 10, 80), prec=prec, steps=steps,
                ckpt=max(1, steps // rng.choice([1, 2, 4])))


# --------------------------------------------------------------------------------------------------
# Inputs (SI values and fields, the same for the library and for exact())
# --------------------------------------------------------------------------------------------------


def _smooth(g, ny, nx, modes=3):
    """A smooth random field of order one on ny x nx, zero at the edges."""
    y, x = (np.arange(ny) + 0.5) / ny, (np.arange(nx) + 0.5) / nx
    out = np.zeros((ny, nx))
    for a in g.uniform(-1, 1, (modes, 3)):
        k, m = int(g.integers(1, 4)), int(g.integers(1, 6))
        out += a[0] * np.outer(np.sin(np.pi * k * y), np.sin(np.pi * m * x))
    return out


def _channel_inputs(prm, ini, seed):
    """Disturb a channel's start and its wall flux: the fields of a run that is under way."""
    ny, nx = ini["T"].shape
    g = WL.rng(seed)
    um = prm["u_m"]
    ini = dict(ini, ux=ini["ux"] + 0.05 * um * _smooth(g, ny, nx),
               uy=0.05 * um * _smooth(g, ny, nx), T=ini["T"] + 2.0 * _smooth(g, ny, nx))
    wave = 1.0 + 0.1 * _smooth(g, 1, nx)[0]
    return dict(prm, flux=prm["flux"] * wave), ini


def _inputs(case, seed):
    """(prm, ini) of a case: SI parameters and initial fields as numpy arrays."""
    kind = case["kind"]
    if kind == "slab":
        prm, T0 = WL.slab_1d(seed=seed, n=case["n"], noise=5.0)
        return prm, dict(T=T0)
    if kind == "channel":
        prm, ini = WL.channel(nx=case["nx"], ny=case["ny"], oscillating=case["oscillating"])
        prm["flow_mrt"] = int(case["mrt"])
        return _channel_inputs(prm, ini, seed)
    if kind == "half":
        prm, ini = WL.paper_channel(case["case"], H=case["H"], L=case["L"])
        return _channel_inputs(prm, ini, seed)
    if kind == "adjoint":
        prm, ini = WL.adjoint_channel(nx=case["nx"], ny=case["ny"])
        return _channel_inputs(prm, ini, seed)
    if kind == "cavity":
        prm, ini = WL.cavity(1e4, n=case["n"])
        g = WL.rng(seed)
        ini = dict(ini, T=ini["T"] + 5.0 * _smooth(g, case["n"], case["n"]))
        return prm, ini
    if kind == "bubble":
        small = min(case["nx"], case["ny"])
        radii = (20, 30, 40, 50) if small >= 120 else (0.2 * small, 0.3 * small)
        prm, ini, _ = WL.bubble(n=case["nx"], ny=case["ny"], radii=radii, batch=case["batch"],
                                seed=seed)
        return prm, ini
    if kind == "layered":
        prm, ini, _ = WL.layered(nx=case["nx"], ny=case["ny"], batch=case["batch"], seed=seed)
        return prm, ini
    if kind == "d3q19":
        nx, ny = case["nx"], case["ny"]
        period = (64, 64) if nx % 64 == 0 and ny % 64 == 0 else None
        prm, ini = WL.box3d(nx, ny, case["nz"], seed=seed, F=(30.0, 20.0, -10.0), period=period,
                            mrt=case["mrt"])
        return prm, ini
    props = {k: v for k, v in WL.TWO_PHASE_SYSTEMS["air_water_25C"].items()
             if k not in ("zeta_l", "zeta_g")}
    prm, ini = WL.bubble3d(n=case["cell"], R_nodes=0.25 * case["cell"], seed=seed, p_laplace=True,
                           **props)
    reps = (1,) + (case["cells"],) * 3
    return prm, {k: np.tile(v, reps) for k, v in ini.items()}


_FIELDS = {"slab": ("T",), "channel": ("rho", "ux", "uy", "T"), "half": ("rho", "ux", "uy", "T"),
           "cavity": ("rho", "ux", "uy", "T"), "bubble": ("p", "ux", "uy", "phi"),
           "layered": ("p", "ux", "phi"), "d3q19": ("rho", "ux", "uy", "uz"),
           "phase3d": ("p", "ux", "uy", "uz", "phi")}


def _tau(prm):
    cs2 = (prm["dx"] / prm["dt"]) ** 2 / 3.0
    return [prm["nu"] / cs2 + 0.5 * prm["dt"], prm["alpha"] / cs2 + 0.5 * prm["dt"]]


# --------------------------------------------------------------------------------------------------
# The pass
# --------------------------------------------------------------------------------------------------


def prepare(case, seed):
    from paper_2302_04120_amd import adjoint, lbm
    kind = case["kind"]
    prm, ini = _inputs(case, seed)
    if kind == "adjoint":
        prob = adjoint.ChannelAdjoint(prm, ini, case["nx"], case["ny"], case["steps"], case["ckpt"],
                                      prec=case["prec"])
        flux = torch.tensor(prm["flux"], dtype=torch.float64, requires_grad=True)
        tau = torch.tensor(_tau(prm), dtype=torch.float64, requires_grad=True)
        return dict(kind=kind, prob=prob, flux=flux, tau=tau)
    walls = lbm.BC_WALL
    if kind == "slab":
        L = lbm.Lattice("d1q%d" % case["q"], case["n"], prec="fp64")
    elif kind in ("channel", "half"):
        ny, nx = ini["T"].shape
        top = lbm.BC_SYMMETRY if kind == "half" else walls
        L = lbm.Lattice("channel", nx, ny, prec=case["prec"],
                        bc=(lbm.BC_VEL_INLET, lbm.BC_P_OUTLET, walls, top), flow=True,
                        thermal="d2q9" if kind == "half" else True)
    elif kind == "cavity":
        L = lbm.Lattice("channel", case["n"], case["n"], prec=case["prec"],
                        bc=(lbm.BC_DIRICHLET, lbm.BC_DIRICHLET, walls, walls), flow=True,
                        thermal="d2q9")
    elif kind in ("bubble", "layered"):
        L = lbm.Lattice("phase", case["nx"], case["ny"], batch=case["batch"], prec=case["prec"],
                        bc=(0, 0, walls, walls) if kind == "layered" else None)
    elif kind == "d3q19":
        w = walls if case["walls"] else 0
        L = lbm.Lattice("d3q19", case["nx"], case["ny"], prec=case["prec"], bc=(0, 0, w, w),
                        nz=case["nz"], bc_z=(w, w))
    else:
        n = case["cell"] * case["cells"]
        L = lbm.Lattice("phase3d", n, n, prec=case["prec"], nz=n)
    L.set_params(prm)
    if kind in ("d3q19", "phase3d"):
        L.init3d(ini.get("rho", ini.get("p")), ini["ux"], ini["uy"], ini["uz"], ini.get("phi"))
    else:
        L.init(ini.get("rho", ini.get("p")), ini.get("ux"), ini.get("uy"), ini.get("T"),
               ini.get("phi"))
    return dict(kind=kind, L=L, steps=case["steps"], fields=_FIELDS[kind])


def run(state):
    if state["kind"] == "adjoint":
        flux, tau = state["flux"], state["tau"]
        flux.grad = tau.grad = None
        J = state["prob"].J(flux, tau)
        J.backward()
        return dict(J=J.detach(), dflux=flux.grad, dtau=tau.grad)
    state["L"].step(state["steps"])
    return state["L"].macros_device(state["fields"])


#: floating-point operations of one node update (moments, relaxation, inverse, boundary-free)
_FLOPS = {"slab": 20, "channel": 230, "half": 330, "cavity": 330, "bubble": 330, "layered": 330,
          "d3q19": 420, "phase3d": 1000, "adjoint": 1100}


def work(case):
    """The state read and written once and the output fields written once; every node update's
    operations.  The adjoint reads and writes its forward states and adjoint states once each."""
    kind = case["kind"]
    size = 8 if kind == "slab" or case["prec"] == "fp64" else 4
    if kind == "slab":
        nodes, vals = case["n"], case["q"]
    elif kind in ("channel", "adjoint"):
        nodes, vals = case["nx"] * case["ny"], 14
    elif kind == "half":
        dx = 5e-6 if case["case"] == "developed_alternating" else 2.5e-6
        nodes, vals = round(case["L"] / dx) * round(0.5 * case["H"] / dx), 18
    elif kind == "cavity":
        nodes, vals = case["n"] ** 2, 18
    elif kind in ("bubble", "layered"):
        nodes, vals = case["nx"] * case["ny"] * case["batch"], 20 if size == 8 else 21
    elif kind == "d3q19":
        nodes, vals = case["nx"] * case["ny"] * case["nz"], 19
    else:
        nodes, vals = (case["cell"] * case["cells"]) ** 3, 41 if size == 8 else 42
    flops = float(nodes) * case["steps"] * _FLOPS[kind]
    if kind == "adjoint":
        return dict(bytes=4.0 * nodes * vals * size, flops=flops)
    return dict(bytes=2.0 * nodes * vals * size + 8.0 * nodes * len(_FIELDS[kind]), flops=flops)


# --------------------------------------------------------------------------------------------------
# The same model in FP64 with plain torch
# --------------------------------------------------------------------------------------------------

_E2 = [(0, 0), (1, 0), (0, 1), (-1, 0), (0, -1), (1, 1), (-1, 1), (-1, -1), (1, -1)]
_E5 = _E2[:5]
_E3 = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1), (1, 1, 0),
       (-1, -1, 0), (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1), (-1, 0, 1),
       (0, 1, 1), (0, -1, -1), (0, 1, -1), (0, -1, 1)]
_W2 = [4 / 9] + [1 / 9] * 4 + [1 / 36] * 4
_W5 = [1 / 3] + [1 / 6] * 4
_W3 = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _t(a):
    return torch.as_tensor(np.asarray(a, dtype=np.float64), device=_device())


def _opp(E):
    return [E.index(tuple(-c for c in e)) for e in E]


def _basis9():
    """rho, e, eps, j_x, q_x, j_y, q_y, p_xx, p_xy of D2Q9."""
    e = np.array(_E2, dtype=float)
    x, y = e[:, 0], e[:, 1]
    s = x * x + y * y
    return np.array([s * 0 + 1, 3 * s - 4, 4.5 * s * s - 10.5 * s + 4, x, (3 * s - 5) * x, y,
                     (3 * s - 5) * y, x * x - y * y, x * y])


def _basis5():
    """T, j_x, j_y, e, p_xx of D2Q5."""
    e = np.array(_E5, dtype=float)
    x, y = e[:, 0], e[:, 1]
    s = x * x + y * y
    return np.array([s * 0 + 1, x, y, 5 * s - 4, x * x - y * y])


def _basis19():
    """The d'Humieres et al. (2002) basis: rho, e, eps, j and q per axis, 3p_xx, 3pi_xx, p_ww,
    pi_ww, p_xy, p_yz, p_xz, m."""
    e = np.array(_E3, dtype=float)
    x, y, z = e.T
    s = x * x + y * y + z * z
    pxx, pww = 3 * x * x - s, y * y - z * z
    return np.array([s * 0 + 1, 19 * s - 30, (21 * s * s - 53 * s + 24) / 2, x, (5 * s - 9) * x, y,
                     (5 * s - 9) * y, z, (5 * s - 9) * z, pxx, (3 * s - 5) * pxx, pww,
                     (3 * s - 5) * pww, x * y, y * z, x * z, (y * y - z * z) * x,
                     (z * z - x * x) * y, (x * x - y * y) * z])


def _mat(A, f):
    """A (q x q) applied to the populations f [q, ...]."""
    return (A @ f.reshape(f.shape[0], -1)).reshape(f.shape)


class _Channel:
    """D2Q9 flow and D2Q5 or D2Q9 temperature on [ny, nx]; f and g are deviations from w rho_ref and
    w T_ref.  flux (scaled), lf, lt may carry autograd graphs."""

    def __init__(self, prm, nx, ny, inlet, sym, qt):
        self.prm, self.nx, self.ny, self.inlet, self.sym = prm, nx, ny, inlet, sym
        dev = _device()
        self.X = torch.arange(nx, device=dev).view(1, nx)
        self.Y = torch.arange(ny, device=dev).view(ny, 1)
        self.Eg, self.Wg = (_E2, _W2) if qt == 9 else (_E5, _W5)
        self.M, self.Mi = _t(_basis9()), _t(np.linalg.inv(_basis9()))
        bg = _basis9() if qt == 9 else _basis5()
        self.Mg, self.Mgi = _t(bg), _t(np.linalg.inv(bg))
        self.dt, self.dx = prm["dt"], prm["dx"]
        self.c = self.dx / self.dt
        self.rr = prm["rho_ref"]
        self.Ft = [prm.get(k, 0.0) * self.dt ** 2 / self.dx for k in ("Fx", "Fy")]
        g = prm.get("gravity", (0.0, 0.0))
        self.Bt = [-self.rr * prm.get("beta_T", 0.0) * gk * self.dt ** 2 / self.dx for gk in g]
        self.buoy = any(b != 0.0 for b in self.Bt)
        self.qdt = prm.get("qvol", 0.0) / prm["rho_cp"] * self.dt
        self.uin = _t(np.broadcast_to(prm["inlet_u"], (ny,))) / self.c
        self.tin = _t(np.broadcast_to(prm["inlet_T"], (ny,))) - prm["T_ref"]
        self.tw = [t - prm["T_ref"] for t in prm.get("T_wall", (0.0, 0.0))]

    def rates(self, tau, tau_T):
        one, zero = torch.ones((), dtype=torch.float64, device=_device()), 0.0
        wn, wt = self.dt / tau * one, self.dt / tau_T * one
        wq = 3 * (2 - wn) / (3 - wn)
        zero = 0 * one
        if self.prm["flow_mrt"]:
            we, wp = self.prm["omega_e"] * self.dt * one, self.prm["omega_eps"] * self.dt * one
            lf = [zero, we, wp, zero, wq, zero, wq, wn, wn]
        else:
            lf = [wn] * 9
        q = len(self.Eg)
        jrows = (3, 5) if q == 9 else (1, 2)
        lt = [wt if k in jrows or not self.prm["thermal_mrt"] else (zero if k == 0 else one)
              for k in range(q)]
        return torch.stack(lf).view(9, 1, 1), torch.stack(lt).view(q, 1, 1)

    def feq(self, drho, rho, u, v):
        uu = u * u + v * v
        out = []
        for (ex, ey), w in zip(_E2, _W2):
            eu = ex * u + ey * v
            out.append(w * (drho + rho * (3 * eu + 4.5 * eu * eu - 1.5 * uu)))
        return torch.stack(out)

    def geq(self, th, u, v):
        return torch.stack([w * th * (1 + 3 * (ex * u + ey * v))
                            for (ex, ey), w in zip(self.Eg, self.Wg)])

    def macros(self, f, g):
        th = g.sum(0) + 0.5 * self.qdt
        Fx = self.Ft[0] + self.Bt[0] * th if self.buoy else self.Ft[0] + 0 * th
        Fy = self.Ft[1] + self.Bt[1] * th if self.buoy else self.Ft[1] + 0 * th
        drho = f.sum(0)
        rho = self.rr + drho
        jx = sum(e[0] * f[i] for i, e in enumerate(_E2) if e[0])
        jy = sum(e[1] * f[i] for i, e in enumerate(_E2) if e[1])
        return th, Fx, Fy, drho, rho, (jx + 0.5 * Fx) / rho, (jy + 0.5 * Fy) / rho

    def outside(self, e):
        """Masks of the nodes whose source x - e lies outside: below, above, left, right."""
        sx, sy = self.X - e[0], self.Y - e[1]
        zero = torch.zeros((self.ny, self.nx), dtype=torch.bool, device=self.X.device)
        return zero | (sy < 0), zero | (sy >= self.ny), zero | (sx < 0), zero | (sx >= self.nx)

    def step(self, f, g, lf, lt, flux, mod):
        th, Fx, Fy, drho, rho, u, v = self.macros(f, g)
        guo = torch.stack([w * ((3 * (ex - u) + 9 * (ex * u + ey * v) * ex) * Fx +
                                (3 * (ey - v) + 9 * (ex * u + ey * v) * ey) * Fy)
                           for (ex, ey), w in zip(_E2, _W2)])
        fs = f + _mat(self.Mi, -lf * _mat(self.M, f - self.feq(drho, rho, u, v)) +
                      (1 - 0.5 * lf) * _mat(self.M, guo))
        src = torch.stack([w * self.qdt * torch.ones_like(th) for w in self.Wg])
        gs = g + _mat(self.Mgi, -lt * _mat(self.Mg, g - self.geq(th, u, v)) +
                      (1 - 0.5 * lt) * _mat(self.Mg, src))
        uw = 1.5 * u[:, -1:] - 0.5 * u[:, -2:-1]
        vw = 1.5 * v[:, -1:] - 0.5 * v[:, -2:-1]

        def pulled(p, j, e, E):
            lo, hi, left, right = self.outside(e)
            new = torch.roll(p[j], (e[1], e[0]), (0, 1))
            if self.sym and e[1] < 0:  # mirrored mover of the top row, at its own x - e_x
                k = E.index((e[0], -e[1]))
                new = torch.where(hi, torch.roll(p[k], e[0], 1), new)
                hi = torch.zeros_like(hi)
            return new, lo | hi, left, right

        fn, gn = [], []
        opp = _opp(_E2)
        for j, e in enumerate(_E2):
            new, wall, left, right = pulled(fs, j, e, _E2)
            i, w, ei = opp[j], _W2[j], _E2[opp[j]]
            if self.inlet:
                inl = fs[i] - 6 * w * self.rr * ei[0] * self.uin.view(-1, 1)
                eu = ei[0] * uw + ei[1] * vw
                out = -fs[i] + 2 * w * self.rr * (4.5 * eu * eu - 1.5 * (uw * uw + vw * vw))
                new = torch.where(left, inl, torch.where(right, out, new))
            else:
                new = torch.where(left | right, fs[i], new)
            fn.append(torch.where(wall, fs[i], new))
        opp = _opp(self.Eg)
        for j, e in enumerate(self.Eg):
            new, wall, left, right = pulled(gs, j, e, self.Eg)
            i, w, ei = opp[j], self.Wg[j], self.Eg[opp[j]]
            lam = 6 * w if len(self.Eg) == 9 else 1.0
            if self.inlet:
                other = torch.arange(self.ny, device=self.X.device) + ei[1]
                tin2 = self.tin[other.clamp(0, self.ny - 1)]  # the row itself beyond the channel
                inl = -gs[i] + 2 * w * (0.5 * (self.tin + tin2)).view(-1, 1)
                new = torch.where(left, inl, new)
                if e[0] < 0:  # outlet: the value of the neighbour column
                    new = torch.cat([new[:, :-1], new[:, -2:-1]], 1)
            else:
                new = torch.where(left, -gs[i] + 2 * w * self.tw[0], new)
                new = torch.where(right, -gs[i] + 2 * w * self.tw[1], new)
            gn.append(torch.where(wall, gs[i] + lam * flux.view(1, -1) * mod, new))
        return torch.stack(fn), torch.stack(gn)

    def start(self, ini):
        u, v = _t(ini["ux"]) / self.c, _t(ini["uy"]) / self.c
        rho, th = _t(ini["rho"]), _t(ini["T"]) - self.prm["T_ref"]
        return self.feq(rho - self.rr, rho, u, v), self.geq(th, u, v)

    def modulation(self, n):
        return 1.0 + self.prm.get("flux_amp", 0.0) * math.sin(
            self.prm.get("flux_omega", 0.0) * n * self.dt)


def _exact_channel(case, prm, ini):
    ny, nx = ini["T"].shape
    m = _Channel(prm, nx, ny, case["kind"] != "cavity", case["kind"] == "half",
                 5 if case["kind"] == "channel" else 9)
    lf, lt = m.rates(*_tau(prm))
    flux = _t(prm["flux"]) * m.dt / (m.dx * prm["rho_cp"])
    f, g = m.start(ini)
    for n in range(case["steps"]):
        f, g = m.step(f, g, lf, lt, flux, m.modulation(n))
    th, _, _, _, rho, u, v = m.macros(f, g)
    out = dict(rho=rho, ux=u * m.c, uy=v * m.c, T=th + prm["T_ref"])
    return {k: a.unsqueeze(0) for k, a in out.items()}


def _exact_adjoint(case, prm, ini):
    from torch.utils.checkpoint import checkpoint
    nx, ny = case["nx"], case["ny"]
    m = _Channel(prm, nx, ny, True, False, 5)
    flux = _t(prm["flux"]).requires_grad_()
    tau = _t(_tau(prm)).requires_grad_()

    def block(f, g, flux, tau, n0, count):
        lf, lt = m.rates(tau[0], tau[1])
        q = flux * m.dt / (m.dx * prm["rho_cp"])
        for n in range(n0, n0 + count):
            f, g = m.step(f, g, lf, lt, q, m.modulation(n))
        return f, g

    f, g = m.start(ini)
    for n in range(0, case["steps"], 16):
        f, g = checkpoint(block, f, g, flux, tau, n, min(16, case["steps"] - n),
                          use_reentrant=False)
    th, _, _, _, _, u, _ = m.macros(f, g)
    T = th + prm["T_ref"]
    kc = prm["rho_cp"] * (tau[1] - 0.5 * m.dt) * m.c ** 2 / 3.0
    q = flux * m.modulation(case["steps"])
    Tb = (u * T).sum(0) / u.sum(0)
    Tw = 0.5 * (T[0] + T[-1]) + q * m.dx / (2 * kc)
    Nu = q * (2.0 * ny * m.dx) / (kc * (Tw - Tb))
    J = Tb[-1] + Nu[nx // 2:].mean()
    J.backward()
    return dict(J=J.detach(), dflux=flux.grad, dtau=tau.grad)


def _stream(p, E, walls):
    """p [q, b, (z,) y, x] streamed along E; walls: per axis (x, y, z), halfway bounce-back."""
    opp, out = _opp(E), []
    for i, e in enumerate(E):
        new = p[i]
        for a, s in enumerate(e):
            if s:
                new = torch.roll(new, s, new.dim() - 1 - a)
        for a, s in enumerate(e):
            if s and walls[a]:
                d = new.dim() - 1 - a
                at = [slice(None)] * new.dim()
                at[d] = slice(0, 1) if s > 0 else slice(new.shape[d] - 1, None)
                new[tuple(at)] = p[opp[i]][tuple(at)]
        out.append(new)
    return torch.stack(out)


def _shift(a, e, walls):
    """a at x + e: periodic, or at a wall the first node inside."""
    for ax, s in enumerate(e):
        d = a.dim() - 1 - ax
        if s:
            r = torch.roll(a, -s, d)
            if walls[ax]:
                at = [slice(None)] * a.dim()
                at[d] = slice(a.shape[d] - 1, None) if s > 0 else slice(0, 1)
                r[tuple(at)] = a[tuple(at)]
            a = r
    return a


def _exact_phase(case, prm, ini, dim):
    """The two-phase model on D2Q9 or D3Q19: h BGK, z MRT (zeq, F^z) in moment space."""
    E, W = (_E2, _W2) if dim == 2 else (_E3, _W3)
    B = _basis9() if dim == 2 else _basis19()
    M, Mi = _t(B), _t(np.linalg.inv(B))
    walls = (False, case["kind"] == "layered", False)[:dim]
    dx, dt = prm["dx"], prm["dt"]
    c, cs2 = dx / dt, (dx / dt) ** 2 / 3.0
    ex = [[e[a] for e in E] for a in range(dim)]
    drho, sc = prm["rho_l"] - prm["rho_g"], dt / dx ** 2
    wphi = dt / (prm["M"] / cs2 + 0.5 * dt)
    beta, kap6 = 12 * prm["sigma"] / prm["W"], 9 * prm["sigma"] * prm["W"] / dx ** 2
    F0 = list(prm["F"]) if dim == 3 else [prm["Fx"], prm["Fy"]]
    F0 = [a * dt * dt / dx for a in F0]
    geps = prm["normal_eps"] * dx / 3.0

    def dot(a, b):
        return sum(p * q for p, q in zip(a, b))

    def s_i(u):
        uu, out = dot(u, u), []
        for e, w in zip(E, W):
            eu = dot(e, u)
            out.append(w * (3 * eu + 4.5 * eu * eu - 1.5 * uu))
        return out

    def local(h, z):
        phi = h.sum(0)
        pn = [_shift(phi, e, walls) for e in E]
        G = [sum(W[i] * ex[a][i] * pn[i] for i in range(len(E)) if ex[a][i]) for a in range(dim)]
        Lp = sum(W[i] * (pn[i] - phi) for i in range(1, len(E)))
        rho = prm["rho_g"] + phi * drho
        mu = 4 * beta * phi * (phi - 1) * (phi - 0.5) - kap6 * Lp
        F = [mu * G[a] * 3 * dt * dt / dx ** 2 + F0[a] for a in range(dim)]
        u = [(sum(ex[a][i] * z[i] for i in range(len(E)) if ex[a][i]) + 0.5 * F[a]) / rho
             for a in range(dim)]
        uu, ug = dot(u, u), dot(u, G)
        ph = (z[1:].sum(0) + 1.5 * drho * ug - 1.5 * W[0] * rho * uu) / (1 - W[0])
        return phi, G, rho, F, u, ph

    u0 = [_t(ini[k]) / c for k in ("ux", "uy", "uz")[:dim]]
    phi, ph = _t(ini["phi"]), _t(ini["p"]) / cs2
    rho, s = prm["rho_g"] + _t(ini["phi"]) * drho, s_i(u0)
    h = torch.stack([phi * w * (1 + 3 * dot(e, u0)) for e, w in zip(E, W)])
    z = torch.stack([ph * (w - 1 if i == 0 else w) + rho * s[i] for i, w in enumerate(W)])
    pu = [phi * a for a in u0]
    for _ in range(case["steps"]):
        phi, G, rho, F, u, ph = local(h, z)
        if prm["visc_mode"] == 0:
            nu = (prm["nu_g"] + phi * (prm["nu_l"] - prm["nu_g"])) * sc
        else:
            nu = (prm["zeta_g"] + phi * (prm["zeta_l"] - prm["zeta_g"])) * sc / rho
        wn = 1 / (3 * nu + 0.5)
        wq = 3 * (2 - wn) / (3 - wn)
        one = torch.ones_like(wn)
        if dim == 2:
            rates = [one, one, one, one, wq, one, wq, wn, wn]
        else:
            rates = [one, one, one, one, wq, one, wq, one, wq, wn, one, wn, one, wn, wn, wn, wq, wq,
                     wq]
        gn = torch.sqrt(dot(G, G))
        n = [torch.where(gn > geps, a / gn.clamp_min(1e-300), 0 * a) for a in G]
        pu1 = [phi * a for a in u]
        dpu = [a - b for a, b in zip(pu1, pu)]
        sharp = 4 * phi * (1 - phi) * dx / prm["W"]
        A = [3 * a + sharp * b for a, b in zip(dpu, n)]
        heq = torch.stack([phi * w * (1 + 3 * dot(e, u)) for e, w in zip(E, W)])
        Sh = torch.stack([w * dot(e, A) + 0 * phi for e, w in zip(E, W)])
        hs = h - wphi * (h - heq) + (1 - 0.5 * wphi) * Sh
        s = s_i(u)
        zeq = torch.stack([ph * (w - 1 if i == 0 else w) + rho * s[i] for i, w in enumerate(W)])
        Fz = []
        for e, w in zip(E, W):
            eu, eG = dot(e, u), dot(e, G) * drho
            Fz.append((dot(e, F), eu, eG, w))
        Fz = torch.stack([w * (3 * eF + 9 * eu * eG) for eF, eu, eG, w in Fz])
        mneq, mF = _mat(M, z - zeq), _mat(M, Fz)
        R = torch.stack(rates)
        z = z + _mat(Mi, -R * mneq + (1 - 0.5 * R) * mF)
        pu = pu1
        h, z = _stream(hs, E, walls), _stream(z, E, walls)
    phi, G, rho, F, u, ph = local(h, z)
    out = dict(p=ph * cs2, ux=u[0] * c, uy=u[1] * c, phi=phi)
    if dim == 3:
        out["uz"] = u[2] * c
    return {k: out[k] for k in _FIELDS[case["kind"]]}


def _exact_d3q19(case, prm, ini):
    B = _basis19()
    M, Mi = _t(B), _t(np.linalg.inv(B))
    dx, dt, rr = prm["dx"], prm["dt"], prm["rho_ref"]
    c = dx / dt
    wn = 1 / (3 * prm["nu"] * dt / dx ** 2 + 0.5)
    wq = 3 * (2 - wn) / (3 - wn)
    rates = ([0, 1, 1, 0, wq, 0, wq, 0, wq, wn, 1, wn, 1, wn, wn, wn, wq, wq, wq] if case["mrt"]
             else [wn] * 19)
    R = _t(rates).view(19, 1, 1, 1, 1)
    walls = (False, case["walls"], case["walls"])
    F = [a * dt * dt / dx for a in prm["F"]]

    def feq(drho, rho, u):
        uu, out = sum(a * a for a in u), []
        for e, w in zip(_E3, _W3):
            eu = sum(p * q for p, q in zip(e, u))
            out.append(w * (drho + rho * (3 * eu + 4.5 * eu * eu - 1.5 * uu)))
        return torch.stack(out)

    def macros(f):
        drho = f.sum(0)
        rho = rr + drho
        return drho, rho, [(sum(e[a] * f[i] for i, e in enumerate(_E3) if e[a]) + 0.5 * F[a]) / rho
                           for a in range(3)]

    u = [_t(ini[k]) / c for k in ("ux", "uy", "uz")]
    rho = _t(ini["rho"])
    f = feq(rho - rr, rho, u)
    for _ in range(case["steps"]):
        drho, rho, u = macros(f)
        guo = []
        for e, w in zip(_E3, _W3):
            eu = sum(p * q for p, q in zip(e, u))
            guo.append(w * sum((3 * (e[a] - u[a]) + 9 * eu * e[a]) * F[a] for a in range(3)))
        f = f + _mat(Mi, -R * _mat(M, f - feq(drho, rho, u)) +
                     (1 - 0.5 * R) * _mat(M, torch.stack(guo)))
        f = _stream(f, _E3, walls)
    _, rho, u = macros(f)
    return dict(rho=rho, ux=u[0] * c, uy=u[1] * c, uz=u[2] * c)


def _exact_slab(case, prm, ini):
    q, n = case["q"], case["n"]
    dx, dt = prm["dx"], prm["dt"]
    cs2 = (dx / dt) ** 2 / (1.0 if q == 2 else 3.0)
    omega = dt / (prm["alpha"] / cs2 + 0.5 * dt)
    qdt = prm["qvol"] / prm["rho_cp"] * dt
    w = np.array([0.5, 0.5] if q == 2 else [4 / 6, 1 / 6, 1 / 6])[:, None]
    ex = [1, -1] if q == 2 else [0, 1, -1]
    g = w * ini["T"][None, :]
    for _ in range(case["steps"]):
        T = g.sum(0) + 0.5 * qdt
        gs = g - omega * (g - w * T) + (1 - 0.5 * omega) * w * qdt
        g = np.stack([np.roll(gs[i], e) for i, e in enumerate(ex)])
        a, b = ex.index(1), ex.index(-1)
        g[a, 0] = prm["T0"] - 0.5 * qdt - (g[:, 0].sum() - g[a, 0])
        g[b, -1] = prm["TL"] - 0.5 * qdt - (g[:, -1].sum() - g[b, -1])
    return dict(T=(g.sum(0) + 0.5 * qdt).reshape(1, 1, n))


def exact(case, seed):
    kind = case["kind"]
    prm, ini = _inputs(case, seed)
    if kind == "slab":
        return _exact_slab(case, prm, ini)
    if kind in ("channel", "half", "cavity"):
        return _exact_channel(case, prm, ini)
    if kind == "adjoint":
        return _exact_adjoint(case, prm, ini)
    if kind == "d3q19":
        return _exact_d3q19(case, prm, ini)
    return _exact_phase(case, prm, ini, 2 if kind in ("bubble", "layered") else 3)
