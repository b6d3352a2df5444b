"""The many-steps kernels of the adjoint (several recomputed or reverse steps per
launch, automatic mode) against single-step launches (fusion mode 1): the same
per-node function, so the adjoint states agree to the last bit and with them
the flux gradient, which accumulates in the same order.  The relaxation-time
gradients are FP64 sums over all nodes and steps in another order: they agree
to the rounding of those sums (n = nodes x steps terms, sqrt(n) 2^-53 of the
sum of magnitudes, of which the result is taken to be at least 1e-3)."""
import numpy as np
import pytest

from paper_2302_04120_amd import workloads as WL

from gpu_cases import print_case

pytestmark = pytest.mark.gpu

CASES = [
    # name, nx, ny, prec, steps, ckpt, overrides
    ("c5_rows", 400, 80, "fp32", 60, 23, {}),
    ("flat", 150, 10, "fp32", 40, 40, {}),
    ("two_columns", 2, 12, "fp32", 15, 4, {}),
    ("one_row", 40, 1, "fp32", 12, 5, {}),
    ("forced", 120, 16, "fp32", 30, 11, {"Fx": 40.0}),
    ("bgk_osc", 203, 21, "fp32", 30, 7, {"flow_mrt": 0, "thermal_mrt": 0, "osc": True}),
    ("fp64_osc_source", 203, 21, "fp64", 30, 7, {"osc": True, "qvol": 1e6}),
    ("forced_fp64", 64, 12, "fp64", 25, 25, {"Fx": 40.0, "Fy": -5.0}),
]


def _grads(case, mode):
    from paper_2302_04120_amd import lbm
    name, nx, ny, prec, steps, ckpt, over = case
    over = dict(over)
    prm, ini = WL.channel(nx=nx, ny=ny, dx=5e-5, tau_ratio=0.7,
                          oscillating=over.pop("osc", False))
    g = WL.rng(len(name))
    prm = dict(prm, flux=prm["flux"] * g.uniform(0.5, 1.5, nx), **over)
    ini = dict(ini, T=ini["T"] + g.uniform(-0.5, 0.5, ini["T"].shape))
    L = lbm.Lattice("channel", nx, ny, prec=prec,
                    bc=(lbm.BC_VEL_INLET, lbm.BC_P_OUTLET, lbm.BC_WALL, lbm.BC_WALL),
                    thermal=True)
    L.set_step_fusion(mode)
    L.set_params(prm)
    L.init(ini["rho"], ini["ux"], ini["uy"], ini["T"])
    J = L.record(steps, ckpt, nx // 2)
    out = (J,) + L.grad(1.5) + L.grad(1.5)  # a second gradient of the same record
    L.close()
    return out


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_many_steps_adjoint_equals_single_steps(case):
    print_case(test="adj-multi", case=case[0], nx=case[1], ny=case[2], prec=case[3])
    one, many = _grads(case, 1), _grads(case, 0)
    assert one[0] == many[0]
    n = case[1] * case[2] * case[4]
    for k in (1, 3):
        assert np.array_equal(one[k], many[k])
        np.testing.assert_allclose(many[k + 1], one[k + 1], rtol=1e3 * np.sqrt(n) * 2.0 ** -53)
    assert np.array_equal(many[1], many[3]) and np.array_equal(many[2], many[4])
