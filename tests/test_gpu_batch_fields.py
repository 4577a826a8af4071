"""Plans of large fields left at the library's defaults, which run the tracers'
field launches: eager and replayed as a graph, the same bits as the
single-field calls, with the divergence and gradient adjoint as one pass and,
where one's output is also the other's, one after the other."""
import pytest
import torch

import paper_1908_07038_amd as pa
import workloads as W

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)


@pytest.mark.parametrize("shared", [False, True])
@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
def test_field_form_equals_single_calls(dtype, shared):
    M = pa.Mesh("O200", radius=6371220.0, device=0)
    tracers, refs = [], []
    for t, L in enumerate((137, 140, 1, 180, 200, 137)):
        f = torch.from_numpy(W.normal((M.nnodes, L), 80 + t)).to(DEV).to(dtype)
        uv = torch.from_numpy(W.normal((M.nnodes, L, 2), 90 + t)).to(DEV).to(dtype)
        d = torch.empty_like(f)
        tracers.append({"gradient": (f, torch.empty_like(uv)), "divergence": (uv, d),
                        "gradient_adjoint": (uv, d if shared else torch.empty_like(f)),
                        "divergence_adjoint": (f, torch.empty_like(uv))})
        refs.append({"gradient": pa.gradient(M, f), "divergence": pa.divergence(M, uv),
                     "gradient_adjoint": pa.gradient_adjoint(M, uv), "divergence_adjoint": pa.divergence_adjoint(M, f)})
    plan = pa.Batch(M, tracers)
    # the mesh's own shapes do not reach a plan of defaults
    pa.set_tune(M, pa.OP_GRADIENT, pa.F64 if dtype == torch.float64 else pa.F32, dict(lds_tiles=2, band_rows=7))
    for launch in (plan.run, plan.graph_launch, plan.graph_launch):
        for tr in tracers:
            for _, y in tr.values():
                y.fill_(float("nan"))
        launch()
        torch.cuda.synchronize()
        for t, (tr, ref) in enumerate(zip(tracers, refs)):
            for n in tr:
                if shared and n == "divergence":
                    continue   # overwritten by the gradient adjoint
                assert torch.equal(tr[n][1] + 0.0, ref[n] + 0.0), (t, n)
    plan.close()
