"""The divergence adjoint added to a field in one pass, bit for bit the sum of
the two (D^T d rounded to the dtype, then one rounded addition): on the LDS
tiles with whole, packed and short columns, and on the gather; and the
differentiable one-pass forms, whose backward it serves, against the same sums
written out - with a gradient of one output only, and with one that is not
aligned to its pairs."""
import pytest
import torch

import paper_1908_07038_amd as pa
import workloads as W

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)
DTYPES = [torch.float64, torch.float32, torch.bfloat16]


def field(M, shape, seed, dtype):
    return torch.from_numpy(W.normal((M.nnodes,) + shape, seed)).to(DEV).to(dtype)


@pytest.mark.parametrize("dtype", DTYPES, ids=["f64", "f32", "bf16"])
@pytest.mark.parametrize("grid,L", [("O33", 1), ("O33", 19), ("O33", 33), ("O33", 60), ("O33", 64), ("O33", 91),
                                    ("O33", 137), ("O33", 200), ("O200", 19), ("O200", 32)])
def test_add_equals_the_sum(grid, L, dtype):
    M = pa.Mesh(grid, radius=6371220.0, device=0)
    d, w = field(M, (L,), 101, dtype), field(M, (L, 2), 102, dtype)
    got = pa._divergence_adjoint_add(M, d, w)
    assert torch.equal(got, w + pa.divergence_adjoint(M, d))


@pytest.mark.parametrize("dtype", DTYPES, ids=["f64", "f32", "bf16"])
def test_backward_of_the_one_pass_forms(dtype):
    M, L = pa.Mesh("O33", radius=6371220.0, device=0), 91
    f, uv = field(M, (L,), 103, dtype).requires_grad_(), field(M, (L, 2), 104, dtype).requires_grad_()
    g2, g1, h1 = field(M, (L, 2), 105, dtype), field(M, (L,), 106, dtype), field(M, (L,), 107, dtype)
    odd = torch.empty(g2.numel() + 1, device=DEV, dtype=dtype)[1:].view_as(g2).copy_(g2)
    want = pa.gradient_adjoint(M, g2 + pa.divergence_adjoint(M, g1))
    for gbar in (g2, odd):
        assert torch.equal(torch.autograd.grad(pa.grad_lap(M, f), f, (gbar, g1))[0], want)
    assert torch.equal(torch.autograd.grad(pa.grad_lap(M, f)[1], f, g1)[0],
                       pa.gradient_adjoint(M, pa.divergence_adjoint(M, g1)))
    assert torch.equal(torch.autograd.grad(pa.div_rot(M, uv), uv, (g1, h1))[0],
                       pa.divergence_adjoint(M, g1) + pa.curl_adjoint(M, h1))
    assert torch.equal(torch.autograd.grad(pa.div_gradt(M, uv), uv, (g1, h1))[0],
                       pa.divergence_adjoint(M, g1) + pa.gradient(M, h1))
