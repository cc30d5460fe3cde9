"""The learned weighting's training kernels in the forms that the sizes choose:
many waves (the row partly read again per mask, its loads in groups) or few,
masks in parts of unequal size or all in one, against the reference."""
import numpy as np
import pytest
import torch

import paper_2302_13524_amd as tm
from oracle import learned_weights as lw
from oracle import operators as ops

from gpu_util import c64, dev, device_intensities, f32, relerr
from test_gpu_wnet import data

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = tm.Context(0)
    yield c
    c.close()


# waves of a launch: rows x parts x N / 1024, few up to 2048; parts: 512 / rows up to K
@pytest.mark.parametrize("n1,n2,P,K", [
    (128, 64, 128, 4),   # 4 parts, 4096 waves
    (128, 64, 112, 6),   # 4 parts of 1 and 2 masks
    (128, 64, 260, 3),   # one part, 2080 waves
    (64, 64, 520, 3),    # one part, 2080 waves
    (64, 64, 100, 6),    # 5 parts of 1 and 2 masks, 2000 waves
    (64, 32, 1030, 2),   # one part, 2060 waves
    (32, 32, 2100, 2),   # one part, 2100 waves
])
@pytest.mark.parametrize("bf16", [False, True])
def test_table_gradient(ctx, n1, n2, P, K, bf16):
    nt, steps = 64, 2
    masks, T, I64, v0 = data(n1, n2, P, 41, K)
    I, Iv = device_intensities(I64, bf16)
    vals = np.minimum(np.linspace(0.0, 16.0, nt), 4.0).astype(np.float32)
    tab = np.stack([vals, np.append(np.diff(vals), 0.0).astype(np.float32)], 1)
    m = masks.astype(np.complex64).astype(np.complex128)
    Lref, gref = lw.power_loss(ops.FFTOp(m, n1, n2), Iv, T.astype(np.complex128), v0.astype(np.complex128),
                               vals.astype(np.float64), steps)
    for _ in range(2):  # the second call on workspaces that hold the first one's sums
        loss, dtab = tm.tm_wtab_power_grad(ctx, c64(masks), I, c64(T), c64(v0), n1, n2, f32(tab), steps)
        # the bounds of the gradient's test at the default table
        assert abs(float(loss.item()) - Lref) < 1e-5 * max(1.0, abs(Lref))
        assert relerr(dtab.cpu().numpy(), gref) < 1e-3


@pytest.mark.parametrize("n1,n2,P,K", [(128, 64, 112, 6), (64, 64, 100, 6), (32, 32, 90, 7), (64, 128, 200, 5)])
def test_forward_in_uneven_parts(ctx, n1, n2, P, K):
    # more rows than two workgroups per CU: one part
    g = torch.Generator().manual_seed(K)
    N = n1 * n2
    masks = torch.polar(torch.ones(K, N), 6.28 * torch.rand(K, N, generator=g)).to(dev())
    t = torch.randn(600, N, dtype=torch.complex64, generator=g).to(dev())
    for intensity in (False, True):
        all_rows = tm.tm_forward(ctx, masks, t, n1, n2, intensity)
        assert torch.equal(tm.tm_forward(ctx, masks, t[:P].contiguous(), n1, n2, intensity), all_rows[:P])
