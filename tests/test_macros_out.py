"""Where lbm_macros writes with out_on_device: kernels write to the context's own GPU
only; every other memory (another GPU's, host memory) is reached by a copy, as a
kernel's store to it could fault."""
import ctypes as C
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_2302_04120_amd import workloads as WL

from gpu_cases import print_case

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_only_the_own_gpu_is_written_directly(tmp_path):
    exe = str(tmp_path / "drv")
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2302_04120_amd", "csrc"),
                    os.path.join(HERE, "pointer_kind_driver.cpp"), "-o", exe], check=True, timeout=300)
    cases = [(t, owner, dev) for t in range(4) for owner in (0, 1, 7) for dev in (0, 1, 7)]
    out = subprocess.run([exe], input="\n".join("%d %d %d" % c for c in cases), text=True,
                         capture_output=True, check=True, timeout=60).stdout.split()
    assert [int(v) for v in out] == [int(t == 0 and owner == dev) for t, owner, dev in cases]


def _lattice(lattice):
    from paper_2302_04120_amd import lbm
    if lattice == "channel":
        prm, ini = WL.channel(nx=75, ny=20)
        L = lbm.Lattice("channel", 75, 20, bc=(lbm.BC_VEL_INLET, lbm.BC_P_OUTLET, lbm.BC_WALL, lbm.BC_WALL))
        L.set_params(prm)
        L.init(ini["rho"], ini["ux"], ini["uy"], ini["T"])
    elif lattice == "phase":
        prm, ini, _ = WL.bubble(n=40, ny=36, radii=(9.0,), batch=2, seed=1)
        L = lbm.Lattice("phase", 40, 36, batch=2)
        L.set_params(prm)
        L.init(ini["p"], ini["ux"], ini["uy"], None, ini["phi"])
    elif lattice == "d3q19":
        prm, ini = WL.box3d(20, 18, 16, seed=2)
        L = lbm.Lattice("d3q19", 20, 18, nz=16)
        L.set_params(prm)
        L.init3d(ini["rho"], ini["ux"], ini["uy"], ini["uz"])
    else:
        props = {k: v for k, v in WL.TWO_PHASE_SYSTEMS["air_water_25C"].items()
                 if k not in ("zeta_l", "zeta_g")}
        prm, ini = WL.bubble3d(n=16, ny=16, nz=16, R_nodes=4.0, seed=3, p_laplace=True, **props)
        L = lbm.Lattice("phase3d", 16, 16, nz=16)
        L.set_params(prm)
        L.init3d(ini["p"], ini["ux"], ini["uy"], ini["uz"], ini["phi"])
    return L


@pytest.mark.gpu
@pytest.mark.parametrize("lattice", ["channel", "phase", "d3q19", "phase3d"])
def test_fields_are_the_same_in_every_memory(lattice):
    import torch
    from paper_2302_04120_amd import lbm
    print_case(test="macros-out", lattice=lattice)
    L = _lattice(lattice)
    L.step(3)
    want = L.macros()
    names = [f for f in lbm.MACRO_BITS if f in want]
    for some in (names, names[1::2], names[-1:]):
        mask = sum(lbm.MACRO_BITS[f] for f in some)
        ref = np.stack([want[f] for f in some])
        dev = torch.zeros(ref.shape, dtype=torch.float64, device="cuda:0")
        pinned = torch.zeros(ref.shape, dtype=torch.float64, pin_memory=True)
        for out in (dev, pinned):
            assert lbm.lib().lbm_macros(L.ctx, mask, C.cast(out.data_ptr(), C.POINTER(C.c_double)), 1) == 0
        torch.cuda.synchronize()
        assert np.array_equal(dev.cpu().numpy(), ref)
        assert np.array_equal(pinned.numpy(), ref)
    L.close()


@pytest.mark.gpu
def test_captured_fields_replay():
    """Steps and fields captured by the caller: every replay writes the fields of its own
    state, into the tensor of the capture."""
    import torch
    from paper_2302_04120_amd import lbm
    print_case(test="macros-capture")
    prm, ini, _ = WL.bubble(n=40, ny=36, radii=(9.0,), batch=2, seed=1)
    s = torch.cuda.Stream()
    L, ref = lbm.Lattice("phase", 40, 36, batch=2, stream=s), lbm.Lattice("phase", 40, 36, batch=2)
    for q in (L, ref):
        q.set_params(prm)
        q.init(ini["p"], ini["ux"], ini["uy"], None, ini["phi"])
    names = [f for f in lbm.MACRO_BITS if f in ref.macros()]
    mask = sum(lbm.MACRO_BITS[f] for f in names)
    out = torch.zeros((len(names), 2, 36, 40), dtype=torch.float64, device="cuda:0")
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        L.step(2)
        assert lbm.lib().lbm_macros(L.ctx, mask, C.cast(out.data_ptr(), C.POINTER(C.c_double)), 1) == 0
    for rep in range(3):
        g.replay()
        torch.cuda.synchronize()
        ref.step(2)
        want = ref.macros()
        assert np.array_equal(out.cpu().numpy(), np.stack([want[f] for f in names])), rep
    L.close()
    ref.close()
