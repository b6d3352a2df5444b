"""A NaN speed sets the speed warning wherever it stands (include/lbm.h: LBM_W_MACH is
"also set for a NaN speed"): in any component of the initial velocity and in the inlet
profile, before or behind finite values, and it hides no speed above the limit."""
import warnings

import numpy as np
import pytest

from paper_2302_04120_amd import workloads as WL

from gpu_cases import print_case

pytestmark = pytest.mark.gpu


def _warned(call):
    with warnings.catch_warnings(record=True) as w:
        warnings.simplefilter("always")
        call()
    return [str(x.message) for x in w]


def _channel():
    from paper_2302_04120_amd import lbm
    prm, ini = WL.channel(nx=75, ny=20)
    L = lbm.Lattice("channel", 75, 20, bc=(lbm.BC_VEL_INLET, lbm.BC_P_OUTLET, lbm.BC_WALL, lbm.BC_WALL))
    return L, prm, ini


@pytest.mark.parametrize("where", [0, 7, 8, 1016, 1023, 1024, 1498, 1499])
@pytest.mark.parametrize("component", [0, 1])
def test_nan_initial_velocity(where, component):
    print_case(test="speed-nan", where=where, component=component)
    L, prm, ini = _channel()
    L.set_params(prm)
    c = prm["dx"] / prm["dt"]
    u = [np.zeros(1500), np.zeros(1500)]
    u[component][where] = np.nan
    fields = [v.reshape(20, 75) for v in u]
    text = _warned(lambda: L.init(ini["rho"], fields[0], fields[1], ini["T"]))
    assert any("nan" in t.lower() for t in text), text
    # a speed above the limit before or behind the NaN is reported as such
    for at in (where - 1, where + 1):
        if 0 <= at < 1500:
            u[component][:] = 0.0
            u[component][where], u[component][at] = np.nan, 0.5 * c
            text = _warned(lambda: L.init(ini["rho"], fields[0], fields[1], ini["T"]))
            assert any("above" in t for t in text), text
    L.close()


def test_nan_initial_velocity_3d():
    from paper_2302_04120_amd import lbm
    print_case(test="speed-nan-3d")
    prm, ini = WL.box3d(20, 18, 16, seed=2)
    L = lbm.Lattice("d3q19", 20, 18, nz=16)
    L.set_params(prm)
    for component in range(3):
        u = [np.zeros((16, 18, 20)) for _ in range(3)]
        u[component][3, 4, 5] = np.nan
        text = _warned(lambda: L.init3d(ini["rho"], *u))
        assert any("nan" in t.lower() for t in text), (component, text)
    L.close()


@pytest.mark.parametrize("where", [0, 11, 19])
def test_nan_inlet_profile(where):
    print_case(test="speed-nan-inlet", where=where)
    L, prm, _ = _channel()
    profile = np.zeros(20)
    profile[where] = np.nan
    text = _warned(lambda: L.set_params(dict(prm, inlet_u=profile)))
    assert any("nan" in t.lower() for t in text), text
    L.close()


def test_finite_speeds_below_the_limit_do_not_warn():
    print_case(test="speed-quiet")
    L, prm, ini = _channel()
    c = prm["dx"] / prm["dt"]
    prm = dict(prm, inlet_u=np.full(20, 0.1 * c))
    u = np.full((20, 75), 0.29 * c)
    assert _warned(lambda: (L.set_params(prm), L.init(ini["rho"], u, -u, ini["T"]))) == []
    L.close()
