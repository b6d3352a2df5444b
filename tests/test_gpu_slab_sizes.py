"""The 1D kernel at the sizes where its instances change (nodes per lane and
waves: 64, 128, 256, 512 nodes and their neighbours) against the FP64 oracle.
Both run in FP64 with at most ~20 roundings a step, so after s steps of values
near T they differ by at most 20 s 2^-52 T."""
import numpy as np
import pytest

from paper_2302_04120_amd import workloads as WL

from gpu_cases import print_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q", [2, 3])
@pytest.mark.parametrize("n", [3, 4, 63, 64, 65, 128, 129, 256, 257, 512, 513, 1023, 1024])
def test_slab_at_the_instance_edges(q, n):
    import oracle as O
    from paper_2302_04120_amd import lbm
    print_case(test="slab-sizes", q=q, n=n)
    prm, T0 = WL.slab_1d(seed=n + q, n=n, noise=5.0)
    L = lbm.Lattice("d1q%d" % q, n, prec="fp64")
    L.set_params(prm)
    L.init(T=T0)
    steps = 0
    for m in (1, 2, 60):
        L.step(m)
        steps += m
        T = L.macros(("T",))["T"].reshape(-1)
        ref = O.d1_run(q, n, prm["dx"], prm["dt"], prm["alpha"], prm["qvol"] / prm["rho_cp"],
                       prm["T0"], prm["TL"], T0, steps)
        ref = np.asarray(ref[0] if isinstance(ref, tuple) else ref).reshape(-1)
        assert np.abs(T - ref).max() <= 20 * steps * 2.0 ** -52 * 310.0
    L.close()
