"""Few rows: the masks of a row shared out over several workgroups. The forward
operator computes each mask as before, so its values equal those of the same
rows among many; the training gradient of the learned weighting adds up the
parts (and its histogram of any table size), against the reference."""
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


@pytest.mark.parametrize("n1,n2,many", [(8, 8, 16500), (16, 16, 4200), (32, 32, 1100), (64, 32, 520), (128, 64, 520)])
@pytest.mark.parametrize("K", [1, 3, 6])
def test_forward_of_few_rows(ctx, n1, n2, many, K):
    g = torch.Generator().manual_seed(n1 * K)
    N = n1 * n2
    masks = torch.polar(torch.ones(K, N), 6.28 * torch.rand(K, N, generator=g)).to(dev())
    t = torch.randn(many, N, dtype=torch.complex64, generator=g).to(dev())
    for intensity in (False, True):
        all_rows = tm.tm_forward(ctx, masks, t, n1, n2, intensity)
        for P in (1, 37, 150):
            few = tm.tm_forward(ctx, masks, t[:P].contiguous(), n1, n2, intensity)
            assert torch.equal(few, all_rows[:P]), (intensity, P)


@pytest.mark.parametrize("n1,n2,P,nt", [(8, 8, 5, 2), (32, 32, 3, 257), (64, 32, 2, 4096), (16, 16, 300, 64)])
@pytest.mark.parametrize("bf16", [False, True])
def test_table_gradient_of_parts(ctx, n1, n2, P, nt, bf16):
    masks, T, I64, v0 = data(n1, n2, P, 31 + nt)
    I, Iv = device_intensities(I64)
    if bf16:
        I = I.to(torch.bfloat16)
        Iv = I.float().cpu().numpy().astype(np.float64)
    vals = np.minimum(np.linspace(0.0, 16.0, nt), 4.0).astype(np.float32)
    tab = np.stack([vals, np.append(np.diff(vals), 0.0).astype(np.float32)], 1)
    m = masks.astype(np.complex64).astype(np.complex128)
    Lref, gref = lw.power_loss(ops.FFTOp(m, n1, n2), Iv, T.astype(np.complex128), v0.astype(np.complex128),
                               vals.astype(np.float64), 3)
    loss, dtab = tm.tm_wtab_power_grad(ctx, c64(masks), I, c64(T), c64(v0), n1, n2, f32(tab), 3)
    # the bounds of the gradient's test at the default table
    assert abs(float(loss.item()) - Lref) < 1e-5 * max(1.0, abs(Lref))
    assert relerr(dtab.cpu().numpy(), gref) < 1e-3


@pytest.mark.parametrize("n1,n2,many", [(32, 32, 2049), (64, 32, 1025), (64, 64, 513), (128, 64, 257)])
@pytest.mark.parametrize("bf16", [False, True])
def test_few_row_kernels_have_the_same_bits(ctx, n1, n2, many, bf16):
    # the kernels for few rows (up to many - 1) and for many differ in when they load only
    g = torch.Generator().manual_seed(many)
    K, N = 3, n1 * n2
    masks = torch.polar(torch.ones(K, N), 6.28 * torch.rand(K, N, generator=g)).to(dev())
    t = torch.randn(many, N, dtype=torch.complex64, generator=g).to(dev())
    I = tm.tm_forward(ctx, masks, t, n1, n2, True, bf16)
    s = torch.randn(many, N, dtype=torch.complex64, generator=g).to(dev())

    def run(P):
        Ip, sp = I[:P].contiguous(), s[:P].contiguous()
        out = list(tm.tm_gradient(ctx, masks, Ip, sp, n1, n2)) + list(tm.tm_amp_gradient(ctx, masks, Ip, sp, n1, n2))
        y = tm.tm_forward(ctx, masks, sp, n1, n2)
        out.append(tm.tm_adjoint(ctx, masks, y, n1, n2))
        for method in ("lbfgs", "lbfgs_amp"):
            x = sp.clone()
            tm.tm_retrieve(ctx, masks, Ip, x, n1, n2, opts=tm.retrieve_opts(method=method, iters=3, bf16=bf16))
            out.append(x)
        for start in ("lanczos", "spectral"):
            x = sp.clone()
            tm.tm_retrieve(ctx, masks, Ip, x, n1, n2,
                           opts=tm.retrieve_opts(method="er", iters=0, start=start, spectral_iters=5, bf16=bf16))
            out.append(x)
        return out

    for P in (1, many - 1):
        for few, all_rows in zip(run(P), run(many)):
            assert torch.equal(few, all_rows[:P]), P
