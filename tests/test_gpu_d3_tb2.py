"""The two-step D3Q19 kernel (fusion mode 2, and automatic where it is faster)
against the single-step kernel.  Both collide with the same function, so the
states must agree to the last bit: periodic and walled axes, planes that are
and are not whole node blocks, boxes from two nodes across (every thread an
overlap of another) to several tiles and segments, batches, BGK and MRT, odd
step counts and graph replay."""
import numpy as np
import pytest

from paper_2302_04120_amd import workloads as WL

from gpu_cases import print_case

pytestmark = pytest.mark.gpu

CASES = [
    # name, nx, ny, nz, walls (x, y, z), prec, batch, mrt
    ("periodic", 70, 37, 29, (0, 0, 0), "fp32", 1, True),
    ("aligned_planes", 64, 32, 40, (0, 0, 0), "fp32", 1, True),
    ("channel_walls", 64, 32, 40, (0, 1, 1), "fp32", 1, True),
    ("closed_box", 41, 33, 30, (1, 1, 1), "fp32", 1, False),
    ("x_walls_tiles", 200, 20, 9, (1, 0, 0), "fp32", 2, True),
    ("wide_rows", 1100, 3, 4, (0, 1, 0), "fp32", 1, True),
    ("two_nodes", 2, 2, 2, (0, 0, 0), "fp32", 1, True),
    ("two_nodes_closed", 2, 2, 2, (1, 1, 1), "fp32", 3, True),
    ("flat_z_walls", 65, 40, 2, (0, 0, 1), "fp32", 1, True),
    ("three_tall", 3, 2, 150, (0, 1, 0), "fp32", 1, True),
    ("periodic_fp64", 70, 37, 29, (0, 0, 0), "fp64", 1, True),
    ("aligned_walls_fp64", 64, 32, 24, (1, 1, 1), "fp64", 1, True),
    ("x_tiles_fp64", 300, 9, 8, (1, 0, 1), "fp64", 1, False),
]


def _state(c, mode, graph_steps=0):
    from paper_2302_04120_amd import lbm
    name, nx, ny, nz, walls, prec, batch, mrt = c
    prm, ini = WL.box3d(nx, ny, nz, batch=batch, seed=len(name), F=(30.0, 20.0, -10.0), mrt=mrt)
    wx, wy, wz = (lbm.BC_WALL if w else 0 for w in walls)
    L = lbm.Lattice("d3q19", nx, ny, batch=batch, prec=prec, bc=(wx, wx, wy, wy), nz=nz,
                    bc_z=(wz, wz))
    L.set_graph_steps(graph_steps)
    L.set_params(prm)
    L.set_step_fusion(mode)
    L.init3d(ini["rho"], ini["ux"], ini["uy"], ini["uz"])
    for n in (1, 2, 7, 16):
        L.step(n)
    blob, bad = L.save_state(), L.reduce(("nonfinite",))["nonfinite"].sum()
    L.close()
    return blob, bad


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_two_step_d3q19_bit_identical(case):
    print_case(test="d3-tb2", case=case[0], nx=case[1], ny=case[2], prec=case[5])
    one, bad = _state(case, 1)
    assert bad == 0
    for mode, graph in ((2, 0), (2, 4), (0, 0)):
        two, bad = _state(case, mode, graph)
        assert bad == 0
        if one != two:
            a, b = np.frombuffer(one, np.uint8), np.frombuffer(two, np.uint8)
            pytest.fail("mode %d: states differ in %d of %d bytes" % (mode, (a != b).sum(), a.size))


def test_captured_d3q19_steps_replay():
    """Two steps captured by the caller end in the buffer they started from."""
    import torch
    from paper_2302_04120_amd import lbm
    nx, ny, nz = 64, 32, 40
    prm, ini = WL.box3d(nx, ny, nz, seed=3)
    print_case(test="d3-tb2-capture", nx=nx)
    s = torch.cuda.Stream()

    def make(stream, mode):
        L = lbm.Lattice("d3q19", nx, ny, nz=nz, stream=stream)
        L.set_params(prm)
        L.set_step_fusion(mode)
        L.init3d(ini["rho"], ini["ux"], ini["uy"], ini["uz"])
        return L

    cap, ref = make(s, 0), make(None, 1)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        cap.step(2)
    for rep in range(3):
        g.replay()
        torch.cuda.synchronize()
        ref.step(2)
        a, b = cap.macros(), ref.macros()
        for k in a:
            assert np.array_equal(a[k], b[k]), (rep, k)
