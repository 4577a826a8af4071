"""The first call of a short level count while another thread captures a
stream: it builds its tiles, the capture is not disturbed, and both results
are those of the gather."""
import threading

import pytest
import torch

import paper_1908_07038_amd as pa
import workloads as W

pytestmark = pytest.mark.gpu
DEV = torch.device("cuda", 0)


def test_first_short_call_beside_a_capture():
    M = pa.Mesh("O200", radius=6371220.0, device=0)
    x = torch.from_numpy(W.normal((M.nnodes, 18), 67)).to(DEV)
    warm = x[:, :3].contiguous()
    outs = [torch.empty((M.nnodes, n, 2), device=DEV, dtype=x.dtype) for n in (18, 3)]
    pa.gradient(M, warm, outs[1])
    beside, errors = torch.cuda.Stream(), []
    torch.cuda.synchronize()

    def call():
        try:
            with torch.cuda.stream(beside):
                pa.gradient(M, x, outs[0])
        except Exception as ex:   # shown by the main thread
            errors.append(ex)

    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="global"):
        t = threading.Thread(target=call)
        t.start()
        t.join(60)
        pa.gradient(M, warm, outs[1])
    assert not t.is_alive() and not errors, errors
    torch.cuda.synchronize()
    assert pa.describe(M, pa.OP_GRADIENT, pa.F64, 18)[1].startswith("k_tile<")
    pa.set_tune(M, pa.OP_GRADIENT, pa.F64, dict(lds_tiles=2))
    refs = [pa.gradient(M, x), pa.gradient(M, warm)]
    for _ in range(3):
        outs[1].zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(outs[1] + 0.0, refs[1] + 0.0)
    assert torch.equal(outs[0] + 0.0, refs[0] + 0.0)
