"""Short columns (8 to 32 levels) of large fields on the LDS tiles against the
gather path, bit for bit up to the sign of zero: the sums of both run in slot
order with the same fused multiply-adds.  Level counts around the edges of the
rule (8 levels; 5 x 2^19 values) and where the lanes of a wave divide into
whole and partial groups (8, 9, 16, 19, 31, 32)."""
import pytest
import torch

import paper_1908_07038_amd as pa
import workloads as W
from test_gpu_tile_blocks import CODES, DEV, OPS

pytestmark = pytest.mark.gpu
CASES = [("O288", 7, False), ("O288", 8, True), ("O288", 9, True), ("O200", 15, False), ("O200", 16, True),
         ("O201", 19, True), ("O200", 31, True), ("O201", 32, True)]


def set_all(M, bit, dtype, shape):
    for b in (bit, pa.OP_GRADIENT, pa.OP_CURL, pa.OP_GRADIENT_ADJOINT):
        pa.set_tune(M, b, CODES[dtype], shape)


@pytest.mark.parametrize("dtype", list(CODES), ids=["f64", "f32", "bf16"])
@pytest.mark.parametrize("grid,L,tiles", CASES, ids=[f"{g}x{n}" for g, n, _ in CASES])
def test_short_columns_equal_the_gather(grid, L, tiles, dtype):
    M = pa.Mesh(grid, radius=6371220.0, device=0)
    x1 = torch.from_numpy(W.normal((M.nnodes, L), 63)).to(DEV).to(dtype)
    x2 = torch.from_numpy(W.normal((M.nnodes, L, 2), 64)).to(DEV).to(dtype)
    for name, (comps, bit) in OPS.items():
        print(f"case {name} {grid} x {L} {dtype}", flush=True)
        assert (pa.describe(M, bit, CODES[dtype], L)[1].startswith("k_tile<")) == tiles
        f, x = getattr(pa, name), (x1 if comps == 1 else x2)
        got = f(M, x)
        set_all(M, bit, dtype, dict(lds_tiles=2))
        ref = f(M, x)
        torch.cuda.synchronize()
        set_all(M, bit, dtype, None)
        for y, r in zip(got if isinstance(got, tuple) else (got,), ref if isinstance(ref, tuple) else (ref,)):
            assert torch.equal(y + 0.0, r + 0.0), (name, L)


def test_first_call_of_a_level_count_under_capture():
    # no tiles of 20 levels are there and none can be built while the stream
    # is captured: the gather records instead, and later calls take the tiles
    M = pa.Mesh("O200", radius=6371220.0, device=0)
    warm = torch.from_numpy(W.normal((M.nnodes, 4), 65)).to(DEV)
    pa.gradient_laplacian(M, warm)
    x = torch.from_numpy(W.normal((M.nnodes, 20), 66)).to(DEV)
    g, d = torch.zeros((M.nnodes, 20, 2), device=DEV, dtype=x.dtype), torch.zeros_like(x)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        pa.gradient_laplacian(M, x, g, d)
    ref = pa.gradient_laplacian(M, x)
    for _ in range(3):
        g.zero_(), d.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(g + 0.0, ref[0] + 0.0) and torch.equal(d + 0.0, ref[1] + 0.0)
