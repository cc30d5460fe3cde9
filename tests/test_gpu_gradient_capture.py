"""The gradients hold no workspace: a context's first call can be captured, on any
stream, and f may be left out."""
import pytest
import torch

import paper_2302_13524_amd as tm

from gpu_util import c64, dev, f32, problem

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n1,n2,P", [(8, 8, 32), (64, 32, 40), (64, 32, 1500), (64, 128, 9)])
@pytest.mark.parametrize("grad", ["tm_gradient", "tm_amp_gradient"])
def test_first_call_in_a_graph(n1, n2, P, grad):
    masks, T, I, _ = problem(n1, n2, 3, P, cfg=957, noise=1e4)
    mk, Id, t = c64(masks), f32(I), c64(T + 0.1)
    eager = tm.Context(0)
    call = getattr(tm, grad)
    g0, f0 = call(eager, mk, Id, t, n1, n2)
    ctx = tm.Context(0)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        g, f = call(ctx, mk, Id, t, n1, n2)
    for k in range(3):
        g.zero_(), f.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(g, g0) and torch.equal(f, f0), k
        call(eager, mk, Id, t, n1, n2)  # eager work between the replays
    del graph
    # without f
    gn = torch.zeros_like(g0)
    fn = getattr(ctx.lib, grad)
    rc = fn(ctx.h, tm.tm_dims(n1, n2, 3, P), mk.data_ptr(), Id.data_ptr(), tm.TM_F32, t.data_ptr(), gn.data_ptr(), None,
            torch.cuda.current_stream(dev()).cuda_stream)
    assert rc == tm.TM_OK and torch.equal(gn, g0)
    ctx.close()
    eager.close()
