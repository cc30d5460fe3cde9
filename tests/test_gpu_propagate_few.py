"""Propagation of few and of many TM columns: the same bits."""
import pytest
import torch

import paper_2302_13524_amd as tm
import tm_synth

from gpu_util import dev

pytestmark = pytest.mark.gpu


# waves: columns x grid points / 1024, few up to 2048
@pytest.mark.parametrize("g1,g2,many", [(32, 32, 2049), (64, 32, 1025), (64, 64, 513)])
def test_few_columns_have_the_same_bits(g1, g2, many):
    ctx = tm.Context(0)
    P = min(g1, g2) ** 2 // 4
    pix = torch.from_numpy(tm_synth.nearest_pixels(min(g1, g2), P).astype("int32")).to(dev())
    T = torch.randn(P, many, dtype=torch.complex64, generator=torch.Generator().manual_seed(many)).to(dev())
    optics = (1.0, 0.5, 0.22, 20.0)
    whole = tm.tm_propagate_tm(ctx, T, pix, g1, g2, optics)
    for n in (1, many - 1):
        part = tm.tm_propagate_tm(ctx, T[:, :n].contiguous(), pix, g1, g2, optics)
        assert torch.equal(part, whole[..., :n])
    ctx.close()
