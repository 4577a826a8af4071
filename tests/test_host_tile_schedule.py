"""The order in which a tiling's tiles go over the XCDs (no GPU): compiled with
g++ from the library's host sources; every tile once, on meshes of fewer tiles
than XCDs, odd grids, and sweeps of one and several bands."""
import os
import subprocess
import tempfile

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_1908_07038_amd", "csrc")


@pytest.fixture(scope="module")
def checker():
    exe = os.path.join(tempfile.mkdtemp(prefix="schedule_check_"), "tile_schedule_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, "-o", exe,
                    os.path.join(HERE, "host", "tile_schedule_check.cpp"), os.path.join(CSRC, "mesh_build.cpp")],
                   check=True)
    return exe


@pytest.mark.parametrize("geom", [(1, 1, 4, 1, 65536), (5, 2, 4, 1, 65536), (33, 1, 3, 1, 65536), (33, 2, 4, 8, 81920),
                                  (64, 2, 6, 1, 163840), (32, 2, 4, 8, 14000)])
def test_schedule_lists_every_tile_once(checker, geom):
    r = subprocess.run([checker] + [str(v) for v in geom], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout + r.stderr
