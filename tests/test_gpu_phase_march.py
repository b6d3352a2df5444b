"""The marching two-phase kernel (fusion mode 2, and automatic where it is fastest)
against the single-step kernel: the same per-node arithmetic, so the states must
agree to the last bit.  Rows of one tile (a multiple of a wave and beside it),
of several tiles with their edges at and one past a tile, segments down to a few
rows, walls and periodic y, both precisions, and calls of 1, 2 and many steps."""
import numpy as np
import pytest

from paper_2302_04120_amd import workloads as WL

from gpu_cases import print_case
from test_gpu_chan_fusion import _bc, _case
from test_gpu_phase_multi import _state

pytestmark = pytest.mark.gpu

CASES = [
    # name, nx, ny, batch, walls, prec, overrides
    ("one_column", 1, 40, 2, True, "fp32", {}),
    ("shortest", 65, 4, 3, False, "fp32", {}),
    ("shortest_walls", 64, 4, 1, True, "fp32", {}),
    ("few_rows", 192, 7, 2, False, "fp32", {"z_mrt": 0}),
    ("whole_row", 256, 61, 2, True, "fp32", {"qy_printed": 1}),
    ("one_past_a_wave", 193, 50, 1, False, "fp32", {"visc_mode": 1}),
    ("one_past_a_row", 257, 45, 1, True, "fp32", {}),
    ("tiles_of_three_steps", 488, 33, 2, False, "fp32", {"Fx": 2.0, "Fy": -1.0}),
    ("one_past_the_tiles", 497, 90, 1, False, "fp32", {}),
    ("aligned_tiles", 512, 70, 1, True, "fp32", {}),
    ("one_wave", 33, 80, 3, True, "fp32", {}),
    ("tiles_of_128_lanes", 360, 40, 2, False, "fp32", {}),
    ("one_past_128_lane_tiles", 349, 21, 1, True, "fp32", {}),
    ("one_past_128_lane_tiles_fp64", 361, 30, 1, False, "fp64", {}),
    ("whole_row_fp64", 128, 37, 2, False, "fp64", {}),
    ("tiles_fp64", 300, 5, 2, True, "fp64", {}),
    ("aligned_fp64", 320, 64, 1, False, "fp64", {"z_mrt": 0}),
]


def _compare(one, many):
    assert one[1] == 0 and many[1] == 0
    if one[0] != many[0]:
        a, b = np.frombuffer(one[0], np.uint8), np.frombuffer(many[0], np.uint8)
        pytest.fail("states differ in %d of %d bytes" % (int((a != b).sum()), a.size))


@pytest.mark.filterwarnings("ignore::RuntimeWarning")
@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_marching_phase_kernel_bit_identical(case):
    print_case(test="phase-march", case=case[0], nx=case[1], ny=case[2], prec=case[5])
    _compare(_state(case, 1), _state(case, 2))


@pytest.mark.parametrize("nx,ny,batch,walls,prec", [
    (256, 256, 32, False, "fp32"),
    (256, 256, 32, False, "fp64"),
    # FP64 arithmetic on the FP32 state: whole rows of one, two and four waves, tiles
    (256, 256, 32, False, "fp32_arith64"),
    (61, 64, 400, True, "fp32_arith64"),
    (100, 130, 130, True, "fp32_arith64"),
    (601, 500, 5, False, "fp32_arith64"),
    (512, 800, 4, True, "fp32_arith64"),
])
def test_automatic_choice_on_grids_that_fill_the_gpu(nx, ny, batch, walls, prec):
    case = ("auto", nx, ny, batch, walls, prec, {})
    print_case(test="phase-march-auto", nx=nx, ny=ny, batch=batch, prec=prec)
    _compare(_state(case, 1), _state(case, 0))


@pytest.mark.parametrize("kind,nx,ny,batch,prec,steps", [
    ("phase", 256, 256, 32, "fp32", 2),   # single steps: two swaps
    ("phase", 256, 256, 128, "fp32", 4),  # pairs: two swaps
    ("phase", 256, 256, 128, "fp32_arith64", 2),  # always single steps
    ("channel", 4096, 500, 1, "fp64", 2),
])
def test_captured_steps_of_automatic_mode_replay(kind, nx, ny, batch, prec, steps):
    """Steps that the caller captures end in the buffer they started from where
    they always have, whatever launches automatic mode takes outside a capture."""
    import torch
    from paper_2302_04120_amd import lbm
    print_case(test="march-capture", kind=kind, nx=nx, ny=ny, batch=batch, prec=prec)
    if kind == "phase":
        prm, ini, _ = WL.bubble(n=nx, ny=ny, radii=(60.0, 70.0), batch=batch, seed=3)
    else:
        prm, ini = _case(nx, ny, seed=3)
    s = torch.cuda.Stream()

    def make(stream, mode):
        L = lbm.Lattice("phase" if kind == "phase" else "channel", nx, ny, batch=batch, prec=prec,
                        bc=None if kind == "phase" else _bc("io_walls"), stream=stream)
        L.set_params(prm)
        L.set_step_fusion(mode)
        if kind == "phase":
            L.init(ini["p"], ini["ux"], ini["uy"], None, ini["phi"])
        else:
            L.init(ini["rho"], ini["ux"], ini["uy"], ini["T"])
        return L

    cap, ref = make(s, 0), make(None, 1)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        cap.step(steps)
    for rep in range(3):
        g.replay()
        torch.cuda.synchronize()
        ref.step(steps)
        a, b = cap.macros(), ref.macros()
        for k in a:
            assert np.array_equal(a[k], b[k]), (rep, k)
