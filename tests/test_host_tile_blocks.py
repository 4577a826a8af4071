"""Blocks of a tiling (no GPU): compiled with g++ from the library's host
sources and checked on several meshes, rings and block sizes, tiles of a few
nodes and odd grids included."""
import os
import subprocess
import tempfile

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "..", "paper_1908_07038_amd", "csrc")


@pytest.fixture(scope="module")
def checker():
    exe = os.path.join(tempfile.mkdtemp(prefix="blocks_check_"), "tile_blocks_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I", CSRC, "-o", exe,
                    os.path.join(HERE, "host", "tile_blocks_check.cpp"), os.path.join(CSRC, "mesh_build.cpp")],
                   check=True)
    return exe


# N, ring, tile rows, bands of a sweep, nodes of a block, budget
GEOMS = [(1, 1, 4, 8, 2, 65536), (5, 2, 4, 1, 3, 65536), (32, 1, 4, 1, 3, 40960), (33, 1, 3, 8, 2, 65536),
         (33, 2, 4, 1, 4, 81920), (64, 2, 6, 1, 3, 163840), (40, 1, 4, 1, 0, 65536), (32, 2, 4, 8, 3, 14000)]


@pytest.mark.parametrize("geom", GEOMS, ids=[f"O{g[0]}-r{g[1]}-b{g[4]}" for g in GEOMS])
def test_tile_blocks(checker, geom):
    r = subprocess.run([checker] + [str(v) for v in geom], capture_output=True, text=True, timeout=300)
    print(r.stdout)
    assert r.returncode == 0 and r.stdout.strip().endswith("OK"), r.stdout + r.stderr
