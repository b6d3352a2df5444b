"""The lanes of the two-step D3Q19 kernel stay inside their workgroup's LDS planes: on
every tile shape of a range each lane, those of the last wave that hold no node among
them, pulls its moving values from within the region, and lanes with a node from the
neighbour the value leaves.  The kernel's own offsets (lbm_d3q19.h), compiled for the
host."""
import os
import shutil
import subprocess

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.mark.skipif(shutil.which("g++") is None, reason="g++ not available")
def test_lanes_pull_from_within_the_region(tmp_path):
    exe = str(tmp_path / "drv")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I", os.path.join(ROOT, "paper_2302_04120_amd", "csrc"),
                    os.path.join(HERE, "d3_tile_driver.cpp"), "-o", exe], check=True, timeout=300)
    cases = []
    for whole in (0, 1):
        for walls in ((0, 1) if whole else (0,)):
            for wc in (2, 3, 16, 17, 31, 32, 63, 64, 65, 100, 128, 250):
                for h in (1, 2, 3, 4, 5, 7, 12, 30):
                    nodes = (wc + (0 if whole else 2)) * (h + 2)
                    if nodes <= 1024:
                        # the widest tile's workgroup, and a narrower tile's in it
                        for threads in {(nodes + 63) // 64 * 64, min((nodes + 63) // 64 * 64 + 64, 1024)}:
                            cases.append((wc, h + 2, whole, walls, threads))
    out = subprocess.run([exe], input="\n".join(" ".join(map(str, c)) for c in cases), text=True,
                         capture_output=True, check=True, timeout=300).stdout.split("\n")
    for c, line in zip(cases, out):
        lo, hi, wrong = map(int, line.split())
        wc, rh, whole = c[:3]
        assert lo >= 0 and hi < rh * (wc if whole else wc + 2) and wrong == 0, (c, line)
