"""Infinities, NaN and the types' largest values at single nodes: blocks, lone
nodes and short columns on the LDS tiles give what the gather gives, and the
conservation sums keep them to their own levels."""
import pytest
import torch

import paper_1908_07038_amd as pa
import workloads as W
from test_gpu_tile_blocks import CODES, DEV, OPS

pytestmark = pytest.mark.gpu


def spoiled(M, L, comps, dtype, seed):
    x = torch.from_numpy(W.normal((M.nnodes, L) + ((2,) if comps == 2 else ()), seed)).to(DEV).to(dtype)
    big = torch.finfo(dtype).max
    for k, v in enumerate((float("inf"), float("-inf"), float("nan"), big, -big)):
        nodes = torch.arange(37 + 100 * k, M.nnodes, 997, device=DEV)   # all over the rows, poles' neighbours too
        x[nodes, (5 * k + 3) % L] = v
    return x


def same(y, r):
    return torch.equal(torch.nan_to_num(y + 0.0, nan=7.0), torch.nan_to_num(r + 0.0, nan=7.0)) and \
        torch.equal(torch.isnan(y), torch.isnan(r))


@pytest.mark.parametrize("dtype", list(CODES), ids=["f64", "f32", "bf16"])
@pytest.mark.parametrize("grid,L", [("O33", 60), ("O33", 137), ("O200", 19)])
def test_nonfinite_values(grid, L, dtype):
    M = pa.Mesh(grid, radius=6371220.0, device=0)
    for name, (comps, bit) in OPS.items():
        print(f"case {name} {grid} x {L} {dtype}", flush=True)
        f, x = getattr(pa, name), spoiled(M, L, comps, dtype, 68 + comps)
        got = f(M, x)
        for b in (bit, pa.OP_GRADIENT, pa.OP_CURL, pa.OP_GRADIENT_ADJOINT):
            pa.set_tune(M, b, CODES[dtype], dict(lds_tiles=2, row_window=2))
        ref = f(M, x)
        torch.cuda.synchronize()
        for b in (bit, pa.OP_GRADIENT, pa.OP_CURL, pa.OP_GRADIENT_ADJOINT):
            pa.set_tune(M, b, CODES[dtype], None)
        for y, r in zip(got if isinstance(got, tuple) else (got,), ref if isinstance(ref, tuple) else (ref,)):
            assert same(y, r), (name, L, int((torch.isnan(y) != torch.isnan(r)).sum()))


@pytest.mark.parametrize("dtype", list(CODES), ids=["f64", "f32", "bf16"])
@pytest.mark.parametrize("L", [3, 19, 137])
def test_nonfinite_sums(L, dtype):
    M = pa.Mesh("O33", radius=6371220.0, device=0)
    x = torch.from_numpy(W.normal((M.nnodes, L), 70)).to(DEV).to(dtype)
    y = x.clone()
    y[11, 0], y[M.nnodes - 1, 1], y[M.nnodes // 2, 2] = float("inf"), float("-inf"), float("nan")
    (s, a), (t, b) = pa.conservation(M, x), pa.conservation(M, y)
    assert torch.equal(s[3:], t[3:]) and torch.equal(a[3:], b[3:])
    inf = float("inf")
    assert t[:2].tolist() == [inf, -inf] and b[:2].tolist() == [inf, inf] and bool(t[2].isnan() & b[2].isnan())
