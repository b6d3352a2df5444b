"""Initial fields are read from the caller's arrays: an omitted field acts as the
array it stands for (zeros, T_ref for the channel's temperature), and the speed
warning sees every position of an array, whose blocks are searched eight values at
a time."""
import warnings

import numpy as np
import pytest

from paper_2302_04120_amd import workloads as WL

from gpu_cases import print_case

pytestmark = pytest.mark.gpu


def _blob(L):
    b = L.save_state()
    L.close()
    return b


@pytest.mark.parametrize("lattice", ["channel", "phase", "d3q19", "phase3d"])
def test_omitted_fields_are_their_defaults(lattice):
    from paper_2302_04120_amd import lbm
    print_case(test="init-defaults", lattice=lattice)

    def run(omit):
        if lattice == "channel":
            prm, ini = WL.channel(nx=75, ny=20)
            L = lbm.Lattice("channel", 75, 20, bc=(lbm.BC_VEL_INLET, lbm.BC_P_OUTLET, lbm.BC_WALL, lbm.BC_WALL))
            L.set_params(prm)
            z = np.zeros((20, 75))
            if omit:
                L.init(ini["rho"])
            else:
                L.init(ini["rho"], z, z, z + prm["T_ref"])
        elif lattice == "phase":
            prm, ini, _ = WL.bubble(n=40, ny=36, radii=(9.0,), batch=2, seed=1)
            L = lbm.Lattice("phase", 40, 36, batch=2)
            L.set_params(prm)
            z = np.zeros((2, 36, 40))
            L.init(phi=ini["phi"]) if omit else L.init(z, z, z, None, ini["phi"])
        elif lattice == "d3q19":
            prm, ini = WL.box3d(20, 18, 16, seed=2)
            L = lbm.Lattice("d3q19", 20, 18, nz=16)
            L.set_params(prm)
            z = np.zeros((16, 18, 20))
            L.init3d(ini["rho"]) if omit else L.init3d(ini["rho"], z, z, z)
        else:
            props = {k: v for k, v in WL.TWO_PHASE_SYSTEMS["air_water_25C"].items()
                     if k not in ("zeta_l", "zeta_g")}
            prm, ini = WL.bubble3d(n=16, ny=16, nz=16, R_nodes=4.0, seed=3, p_laplace=True, **props)
            L = lbm.Lattice("phase3d", 16, 16, nz=16)
            L.set_params(prm)
            z = np.zeros((16, 16, 16))
            L.init3d(phi=ini["phi"]) if omit else L.init3d(z, z, z, z, ini["phi"])
        L.step(2)
        return _blob(L)

    assert run(True) == run(False)


@pytest.mark.parametrize("where", [0, 7, 1016, 1023, 1024, 1499])
@pytest.mark.parametrize("value", [0.5, np.nan])
def test_speed_warning_at_every_position(where, value):
    """0.5 c anywhere warns.  A NaN warns as the last value; before others those decide."""
    from paper_2302_04120_amd import lbm
    print_case(test="init-speed", where=where, value=value)
    prm, ini = WL.channel(nx=75, ny=20)
    L = lbm.Lattice("channel", 75, 20, bc=(lbm.BC_VEL_INLET, lbm.BC_P_OUTLET, lbm.BC_WALL, lbm.BC_WALL))
    L.set_params(prm)
    ux = np.zeros(1500)
    ux[where] = value * prm["dx"] / prm["dt"]
    with warnings.catch_warnings(record=True) as w:
        warnings.simplefilter("always")
        L.init(ini["rho"], ux.reshape(20, 75), None, ini["T"])
    L.close()
    warned = any("above" in str(x.message) for x in w)
    assert warned == (value == 0.5 or where == 1499)
