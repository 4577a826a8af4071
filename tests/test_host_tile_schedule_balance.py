"""How a tiling's tiles are shared among the XCDs (no GPU): bands of few tiles,
odd ones and of one or two more than a multiple of eight."""
import os
import subprocess
import tempfile

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_1908_07038_amd", "csrc")


@pytest.fixture(scope="module")
def checker():
    exe = os.path.join(tempfile.mkdtemp(prefix="balance_check_"), "tile_schedule_balance_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, "-o", exe,
                    os.path.join(HERE, "host", "tile_schedule_balance_check.cpp"), os.path.join(CSRC, "mesh_build.cpp")],
                   check=True)
    return exe


@pytest.mark.parametrize("N", [32, 33, 64, 100, 160, 200])
@pytest.mark.parametrize("shape", [(1, 4, 1, 65536), (1, 3, 1, 40960), (2, 4, 1, 81920), (2, 6, 1, 163840),
                                   (1, 4, 8, 65536)])
def test_xcds_take_the_same(checker, N, shape):
    r = subprocess.run([checker, str(N)] + [str(v) for v in shape], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout + r.stderr
