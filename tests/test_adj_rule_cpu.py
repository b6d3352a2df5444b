"""The rule that takes the many-steps reverse kernel counts the waves a compute unit
gets with the device's own number of them (a partition of the GPU has fewer than 256)."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_waves_per_compute_unit_bound_the_rule(tmp_path):
    exe = str(tmp_path / "drv")
    subprocess.run(["g++", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "include"),
                    "-I", os.path.join(ROOT, "paper_2302_04120_amd", "csrc"),
                    os.path.join(HERE, "adj_rule_driver.cpp"), "-o", exe], check=True, timeout=300)
    cases = [(ntx, nty, waves, size, cus) for ntx in (1, 7, 64) for nty in (1, 4, 5)
             for waves in (1, 4, 8, 16) for size in (4, 8) for cus in (32, 64, 128, 256)]
    out = subprocess.run([exe], input="\n".join("%d %d %d %d %d" % c for c in cases), text=True,
                         capture_output=True, check=True, timeout=60).stdout.split()
    for (ntx, nty, waves, size, cus), got in zip(cases, out):
        a_cu = -(-ntx * nty // cus) * waves
        assert int(got) == int(a_cu <= (16 if size == 4 else 8)), (ntx, nty, waves, size, cus)
