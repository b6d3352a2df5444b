"""bench.py's kernel names and steps per launch come from the library's plan, not from
a guess at it: a plan that differs shows in both."""
import os
import sys

import pytest

from gpu_cases import print_case

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
sys.path.insert(0, ROOT)


class _Fake:
    def __init__(self, nx, bc=(0, 0, 0, 0), flags=3, **plan):
        self.nx = nx
        self.desc = type("D", (), dict(bc=bc, flags=flags))()
        self.plan = dict(dict(threads=256, tiles_x=1, tiles_y=1, segments=4), **plan)

    def step_plan(self):
        return self.plan


@pytest.mark.parametrize("lat,prec,want", [
    (_Fake(256, kernel="k_phase_march", steps=3), "fp32", "k_phase_march<float, float, true, true, 256, 3>"),
    (_Fake(256, kernel="k_phase_march", steps=2), "fp32_arith64",
     "k_phase_march<float, double, true, true, 256, 2>"),
    (_Fake(130, kernel="k_phase_march", steps=2, threads=192), "fp64",
     "k_phase_march<double, double, true, false, 256, 2>"),
    (_Fake(8192, kernel="k_phase_march", steps=2, threads=128, tiles_x=69), "fp64",
     "k_phase_march<double, double, false, true, 128, 2>"),
    (_Fake(256, kernel="k_phase", steps=1, threads=0), "fp32_arith64", "k_phase<float, double, false>"),
    (_Fake(256, kernel="k_phase_multi", steps=2), "fp32", "k_phase_multi<float, float>"),
    (_Fake(16384, kernel="k_chan_march", steps=4, bc=(2, 3, 1, 1)), "fp32",
     "k_chan_march<float, true, false, 5, 4>"),
    (_Fake(500, kernel="k_chan_march", steps=3, bc=(2, 3, 1, 5), flags=7), "fp64",
     "k_chan_march<double, false, true, 9, 3>"),
    (_Fake(16384, kernel="k_chan_step", steps=1, bc=(2, 3, 1, 1)), "fp32", "k_chan_step<float, 5>"),
    (_Fake(256, kernel="k_d3_tb2", steps=2), "fp32", "k_d3_tb2<float>"),
])
def test_names_follow_the_plan(lat, prec, want):
    import bench
    assert bench.launches(lat, prec) == (want, lat.plan["steps"])


@pytest.mark.gpu
def test_a_small_batch_reports_the_kernel_that_ran():
    """Automatic mode on four replicas takes LDS tiles, not single steps."""
    import bench
    print_case(test="bench-launches", batch=4)
    r = bench.run_gpu(4, 10, 4, "fp32", n=256, fusion=0)
    assert r["kernel"] == "k_phase_multi<float, float>" and r["steps_per_launch"] >= 2
    r = bench.run_gpu(4, 10, 4, "fp32", n=256, fusion=1)
    assert (r["kernel"], r["steps_per_launch"]) == ("k_phase<float, float, false>", 1)
