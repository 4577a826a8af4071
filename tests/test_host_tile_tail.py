"""The LDS a one-tile launch asks for holds every level its steps read (no
GPU): the geometry functions come from the built library, the tilings from its
host sources.  Level counts around one, two and three 64-level slices, with and
without a remainder of 1..32 levels, and the chunk sizes of long columns."""
import os
import subprocess
import tempfile

import pytest

import paper_1908_07038_amd as pa
from paper_1908_07038_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def checker():
    pa.lib()
    exe = os.path.join(tempfile.mkdtemp(prefix="tail_check_"), "tile_tail_check")
    libdir = os.path.dirname(pa.LIB_PATH)
    subprocess.run(["g++", "-O2", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", build.CSRC,
                    "-I", os.path.join(build.ROCM, "include"), "-o", exe,
                    os.path.join(HERE, "host", "tile_tail_check.cpp"), "-L", libdir, "-latlas_nabla",
                    "-Wl,-rpath," + libdir, "-Wl,--allow-shlib-undefined"], check=True)
    return exe


@pytest.mark.parametrize("form", ["one", "batched"])
@pytest.mark.parametrize("L", [33, 63, 64, 96, 97, 127, 128, 137, 160, 161, 180, 191, 192, 193, 224, 225, 256, 320,
                               384, 545, 576, 700])
def test_reads_end_inside_the_request(checker, L, form):
    r = subprocess.run([checker, "33", str(L), form], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout + r.stderr
