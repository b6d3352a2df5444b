"""The marching channel kernel (fusion mode 2, and automatic where it is fastest)
against the single-step kernel: the same per-node arithmetic, so the states must
agree to the last bit for every number of steps a launch can take.  Step counts
2, 3 and 4 in one call each are single launches of that many steps where the
plan allows them; the grids put tile edges, segment edges and remainders at and
beside every kind of boundary, down to grids narrower than a tile's overlap."""
import numpy as np
import pytest

from gpu_cases import print_case
from test_gpu_chan_fusion import _bc, _case, _cavity_case, _state

pytestmark = pytest.mark.gpu

STEPS = [2, 3, 4, 1, 5, 11]

CASES = [
    # name, nx, ny, bc, prec, batch, thermal, oscillating, overrides
    ("io_one_past_a_tile", 249, 37, "io_walls", "fp32", 1, True, True, {}),
    ("io_tiles", 992, 60, "io_walls", "fp32", 1, True, False, {}),
    ("io_aligned_d2q9", 768, 41, "io_walls", "fp32", 1, "d2q9", True, {}),
    ("half_d2q9", 500, 50, "io_symmetry", "fp32", 1, "d2q9", False, {}),
    ("half", 251, 3, "io_symmetry", "fp32", 2, True, True, {}),
    ("periodic", 300, 33, "periodic", "fp32", 1, True, False, {"Fx": 50.0}),
    ("px_walls_narrow", 5, 90, "px_walls", "fp32", 3, True, True, {"Fx": 50.0}),
    ("tiny_periodic", 2, 2, "periodic", "fp32", 1, "d2q9", False, {"Fx": 50.0}),
    ("tiny_io", 2, 2, "io_walls", "fp32", 1, "d2q9", True, {}),
    ("io_periodic_y_d2q9", 260, 7, "io_py", "fp32", 1, "d2q9", False, {}),
    ("buoyant_bgk", 513, 20, "io_walls", "fp32", 1, True, False,
     {"flow_mrt": 0, "thermal_mrt": 0, "qvol": 1e6, "beta_T": 3e-4, "gravity": (1.0, -9.81)}),
    ("end_walls_half_d2q9", 70, 44, "xw_symmetry", "fp32", 1, "d2q9", False, {}),
    ("io_fp64", 501, 45, "io_walls", "fp64", 1, True, True, {}),
    ("half_d2q9_fp64", 256, 31, "io_symmetry", "fp64", 1, "d2q9", False, {}),
]


def _compare(one, many):
    assert one[1] == 0 and many[1] == 0
    if one[0] != many[0]:
        a, b = np.frombuffer(one[0], np.uint8), np.frombuffer(many[0], np.uint8)
        pytest.fail("states differ in %d of %d bytes" % (int((a != b).sum()), a.size))


@pytest.mark.parametrize("name,nx,ny,bc,prec,batch,thermal,osc,over", CASES,
                         ids=[c[0] for c in CASES])
def test_marching_channel_kernel_bit_identical(name, nx, ny, bc, prec, batch, thermal, osc, over):
    print_case(test="chan-march", case=name, nx=nx, ny=ny, prec=prec, batch=batch)
    prm, ini = _case(nx, ny, seed=len(name), oscillating=osc, **over)
    args = dict(prec=prec, batch=batch, thermal=thermal)
    _compare(_state(prm, ini, nx, ny, _bc(bc), 1, STEPS, **args),
             _state(prm, ini, nx, ny, _bc(bc), 2, STEPS, **args))


@pytest.mark.parametrize("n,prec,thermal", [(253, "fp32", "d2q9"), (40, "fp64", True)])
def test_marching_cavity_bit_identical(n, prec, thermal):
    print_case(test="chan-march-cavity", n=n, prec=prec)
    prm, ini = _cavity_case(n, seed=n)
    args = dict(prec=prec, thermal=thermal)
    _compare(_state(prm, ini, n, n, _bc("cavity"), 1, STEPS, **args),
             _state(prm, ini, n, n, _bc("cavity"), 2, STEPS, **args))


def test_automatic_choice_on_a_grid_that_fills_the_gpu():
    print_case(test="chan-march-auto", nx=4096, ny=500)
    prm, ini = _case(4096, 500, seed=3, oscillating=True)
    _compare(_state(prm, ini, 4096, 500, _bc("io_walls"), 1, [13]),
             _state(prm, ini, 4096, 500, _bc("io_walls"), 0, [13]))
