"""Batches on either side of one work item per CU (the kernels for few items hold
more registers): rows equal single-problem runs."""
import pytest
import torch

import paper_2302_13524_amd as tm

from gpu_util import dev
from test_gpu_batch import opts

pytestmark = pytest.mark.gpu


def _problem(n1, n2, P, seed):
    K, N = 3, n1 * n2
    g = torch.Generator().manual_seed(seed)
    masks = torch.polar(torch.ones(K, N), 6.28 * torch.rand(K, N, generator=g)).to(dev())
    T = torch.randn(P, N, dtype=torch.complex64, generator=g).to(dev())
    return masks, T, torch.randn(P, N, dtype=torch.complex64, generator=g).to(dev())


# items: 1 row of 128 x 64, 2 of 64 x 64, 4 of 64 x 32, 8 of 32 x 32
@pytest.mark.parametrize("extra", [0, 1])
@pytest.mark.parametrize("method,start,mom", [("er", "spectral", 0.0), ("er", "given", 0.7), ("er_cyclic", "lanczos", 0.0)])
def test_batch_around_one_item_per_cu(extra, method, start, mom):
    ctx = tm.Context(0)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    shapes = [(32, 32, 21), (64, 32, 9), (64, 64, 7), (128, 64, cus - 3 - 3 - 4 + extra)]
    probs, ref = [], []
    for i, (n1, n2, P) in enumerate(shapes):
        masks, T, seed = _problem(n1, n2, P, 40 + i)
        I = tm.tm_forward(ctx, masks, T, n1, n2, True, True)
        o = opts(mom, 3, 2, method, start)
        t = seed.clone()
        raw = tm.tm_retrieve(ctx, masks, I, t, n1, n2, o)
        ref.append((t, raw))
        probs.append({"n1": n1, "n2": n2, "masks": masks, "I": I, "t": seed.clone(),
                      "stats": torch.empty((P, tm.ROW_STATS_BYTES), dtype=torch.uint8, device=dev())})
    b = tm.Batch(ctx, probs, opts(mom, 3, 2, method, start), use_graph=True)
    b.run()
    torch.cuda.synchronize()
    for p, (t, raw) in zip(probs, ref):
        assert torch.equal(p["t"], t), (p["n1"], p["n2"])
        assert torch.equal(p["stats"], raw), (p["n1"], p["n2"])
    b.close()
    ctx.close()
