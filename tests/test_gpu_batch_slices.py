"""Persistent plans whose tracers take one, two and three slices a step (161 to
256 levels in one chunk), whose kernels have blocks for some of them only: bit
for bit the single-field calls, each operator alone and with the pair."""
import pytest
import torch

import paper_1908_07038_amd as pa
import workloads as W

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)
LEVELS = [180, 60, 256, 137, 10, 192]


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32], ids=["f64", "f32"])
@pytest.mark.parametrize("tile_kb", [0, 160])
@pytest.mark.parametrize("paired", [False, True])
def test_slices_of_a_persistent_plan(dtype, tile_kb, paired):
    M = pa.Mesh("O33", radius=6371220.0, device=0)
    tracers = []
    for t, L in enumerate(LEVELS):
        f = torch.from_numpy(W.normal((M.nnodes, L), 110 + t)).to(DEV).to(dtype)
        uv = torch.from_numpy(W.normal((M.nnodes, L, 2), 120 + t)).to(DEV).to(dtype)
        w = uv if paired else uv.clone()
        tracers.append({"gradient": (f, torch.empty_like(uv)), "divergence": (uv, torch.empty_like(f)),
                        "gradient_adjoint": (w, torch.empty_like(f)), "divergence_adjoint": (f, torch.empty_like(uv))})
    plan = pa.Batch(M, tracers, tune=dict(batch_mode=1, tile_kb=tile_kb, waves_per_block=8))
    plan.run()
    torch.cuda.synchronize()
    for t, tr in enumerate(tracers):
        for name, (x, y) in tr.items():
            assert torch.equal(y + 0.0, getattr(pa, name)(M, x) + 0.0), (name, LEVELS[t])
    plan.close()
