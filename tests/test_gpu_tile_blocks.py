"""Blocks of regular nodes in the LDS tiles against the gather path (one node
at a time from the neighbour tables), bit for bit up to the sign of zero: the
sums of every path run in slot order with the same fused multiply-adds.  Level
counts at the edges: one level past 32, just under, at and past one and two
64-level slices, remainders of 1, 27 and 32 levels in the packed pass, and of
33 (no packed pass); an odd grid, whose rows end in partial blocks."""
import pytest
import torch

import paper_1908_07038_amd as pa
import workloads as W

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)
CODES = {torch.float64: pa.F64, torch.float32: pa.F32, torch.bfloat16: pa.BF16}
OPS = {"gradient": (1, pa.OP_GRADIENT), "divergence": (2, pa.OP_DIVERGENCE), "laplacian": (1, pa.OP_LAPLACIAN),
       "gradient_adjoint": (2, pa.OP_GRADIENT_ADJOINT), "divergence_adjoint": (1, pa.OP_DIVERGENCE_ADJOINT),
       "gradient_laplacian": (1, pa.OP_LAPLACIAN), "divergence_curl": (2, pa.OP_DIVERGENCE),
       "divergence_gradient_adjoint": (2, pa.OP_DIVERGENCE)}


@pytest.mark.parametrize("dtype", list(CODES), ids=["f64", "f32", "bf16"])
@pytest.mark.parametrize("L", [33, 60, 64, 65, 91, 96, 97, 128, 137, 160, 200])
def test_tiles_equal_the_gather(L, dtype):
    M = pa.Mesh("O33", radius=6371220.0, device=0)
    gather = dict(lds_tiles=2, row_window=2)
    x1 = torch.from_numpy(W.normal((M.nnodes, L), 61)).to(DEV).to(dtype)
    x2 = torch.from_numpy(W.normal((M.nnodes, L, 2), 62)).to(DEV).to(dtype)
    for name, (comps, bit) in OPS.items():
        print(f"case {name} O33 x {L} {dtype}", flush=True)
        f, x = getattr(pa, name), (x1 if comps == 1 else x2)
        got = f(M, x)
        # the pairs' two calls: every operator they fall back to on the gather
        for b in (bit, pa.OP_GRADIENT, pa.OP_CURL, pa.OP_GRADIENT_ADJOINT):
            pa.set_tune(M, b, CODES[dtype], gather)
        ref = f(M, x)
        torch.cuda.synchronize()
        for b in (bit, pa.OP_GRADIENT, pa.OP_CURL, pa.OP_GRADIENT_ADJOINT):
            pa.set_tune(M, b, CODES[dtype], None)
        for y, r in zip(got if isinstance(got, tuple) else (got,), ref if isinstance(ref, tuple) else (ref,)):
            assert torch.equal(y + 0.0, r + 0.0), (name, L)
