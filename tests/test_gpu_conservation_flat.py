"""Conservation sums at the edges of the flat form: columns shorter than a
16-byte vector, around 64 and 256 levels, the longest it takes and one more
(64-level slices), meshes of one workgroup, of partial steps and of many; and a
field that is not 16-byte aligned, whose sums must be the same bits.

Bound: a sum of V rounded products in any order is off by at most
(V + 1) u sum |V_i div_ik| (u = 2^-53), to first order; the oracle's volumes
agree with the library's to 1e-13 relative, the tolerance its sums are
compared with elsewhere."""
import pytest
import torch

import paper_1908_07038_amd as pa
import workloads as W
from _oracle_cache import mesh_and_dual

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)
LEVELS = [1, 2, 3, 5, 7, 8, 9, 31, 63, 64, 65, 137, 255, 257, 513, 1000, 1023, 1024, 1025]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32, torch.bfloat16], ids=["f64", "f32", "bf16"])
@pytest.mark.parametrize("N", [1, 5, 33, 48])
def test_conservation_edges(N, dtype):
    grid = f"O{N}"
    M = pa.Mesh(grid, radius=6371220.0, device=0)
    V = M.nnodes
    _, g = mesh_and_dual(N)
    vol = torch.from_numpy(g.V).to(DEV)
    for L in LEVELS:
        print(f"case {grid} x {L} {dtype}", flush=True)
        raw = torch.empty(V * L + 8, device=DEV, dtype=dtype)
        x = torch.from_numpy(W.normal((V, L), 71)).to(DEV).to(dtype)
        s, a = pa.conservation(M, x)
        p = vol[:, None] * x.double()
        ref, mag = p.cpu().numpy().astype("longdouble").sum(0), p.abs().cpu().numpy().astype("longdouble").sum(0)
        tol = (1e-13 + (V + 1) * 2.0 ** -53) * mag
        assert (abs(s.cpu().numpy() - ref) <= tol).all() and (abs(a.cpu().numpy() - mag) <= tol).all(), L
        y = raw[1:1 + V * L].view(V, L)
        y.copy_(x)
        s2, a2 = pa.conservation(M, y)
        assert torch.equal(s, s2) and torch.equal(a, a2), L
