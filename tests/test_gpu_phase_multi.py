"""The many-steps two-phase kernel (automatic mode on grids that do not fill the
GPU) against the single-step kernel.  Both evaluate phase_local and
phase_collide, so the states must agree to the last bit: periodic and walled y,
axes that one tile spans (they wrap in LDS) and axes cut into tiles, grids
smaller than the overlap, batches, the three precisions, both viscosity and
collision variants, and step counts that leave a remainder."""
import numpy as np
import pytest

from paper_2302_04120_amd import workloads as WL

from gpu_cases import print_case

pytestmark = pytest.mark.gpu

CASES = [
    # name, nx, ny, batch, walls, prec, overrides
    ("c4", 4, 512, 1, True, "fp32", {}),
    ("c4_arith64", 4, 512, 1, True, "fp32_arith64", {}),
    ("c4_fp64", 4, 512, 1, True, "fp64", {}),
    ("narrow_batch", 8, 75, 20, True, "fp32", {"qy_printed": 1}),
    ("one_column", 1, 40, 2, True, "fp32", {}),
    ("one_row", 33, 1, 1, False, "fp32", {}),
    ("two_rows_walls", 30, 2, 1, True, "fp64", {}),
    ("one_tile", 31, 29, 3, False, "fp32", {}),
    ("x_tiles", 211, 9, 1, False, "fp32", {"z_mrt": 0}),
    ("tiles_both", 128, 100, 1, False, "fp32", {"Fx": 2.0, "Fy": -1.0}),
    ("tiles_walls", 101, 143, 1, True, "fp32", {}),
    ("tiles_fp64", 97, 83, 1, False, "fp64", {"visc_mode": 1}),
    ("tiles_arith64", 97, 83, 1, True, "fp32_arith64", {}),
    ("c3", 256, 256, 4, False, "fp32", {}),
]


def _state(case, mode):
    from paper_2302_04120_amd import lbm
    name, nx, ny, batch, walls, prec, over = case
    if walls:
        prm, ini, _ = WL.layered(nx=nx, ny=ny, batch=batch, seed=len(name), W_nodes=4.0)
    else:
        r = 0.25 * max(4, min(nx, ny))
        prm, ini, _ = WL.bubble(n=nx, ny=ny, radii=(r, 1.3 * r), batch=batch, seed=len(name))
    prm = dict(prm, **over)
    g = WL.rng(7)
    u = 1e-4 * prm["dx"] / prm["dt"]
    ini = dict(ini, ux=g.uniform(-u, u, ini["phi"].shape), uy=g.uniform(-u, u, ini["phi"].shape))
    L = lbm.Lattice("phase", nx, ny, batch=batch, prec=prec,
                    bc=(0, 0, lbm.BC_WALL, lbm.BC_WALL) if walls else None)
    L.set_graph_steps(0)
    L.set_params(prm)
    L.set_step_fusion(mode)
    L.init(ini["p"], ini["ux"], ini["uy"], None, ini["phi"])
    for n in (1, 2, 19, 8):
        L.step(n)
    out = L.save_state(), L.reduce(("nonfinite",))["nonfinite"].sum()
    L.close()
    return out


@pytest.mark.filterwarnings("ignore::RuntimeWarning")
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_many_steps_phase_kernel_bit_identical(case):
    print_case(test="phase-multi", case=case[0], nx=case[1], ny=case[2], prec=case[5])
    one, many = _state(case, 1), _state(case, 0)
    assert one[1] == 0 and many[1] == 0
    if one[0] != many[0]:
        a, b = np.frombuffer(one[0], np.uint8), np.frombuffer(many[0], np.uint8)
        pytest.fail("states differ in %d of %d bytes" % (int((a != b).sum()), a.size))
