"""Grids that keep one FFT axis per pass: the kernels whose loads, LDS layout and
barriers depend on the size of the row, against the FP64 oracle. Tolerances are
those of the per-step operators: 1e-5 relative per transform pair in FP32."""
import pytest
import torch

import paper_2302_13524_amd as tm
import tm_synth
from oracle import operators as ops
from oracle import retrieval as rt

from gpu_util import c64, dev, device_intensities, problem, relerr, rounded

pytestmark = pytest.mark.gpu

OPTOL = 1e-5


@pytest.fixture(scope="module")
def ctx():
    c = tm.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("bf16", [False, True])
def test_steps_of_8192_points(ctx, bf16):
    # 64 x 128: error reduction and both gradients, whose loads go out in groups
    n1, n2, K, P = 64, 128, 3, 5
    masks, T, I, _ = problem(n1, n2, K, P, cfg=953, noise=1e4)
    t0 = T + 0.3 * tm_synth.tm_iid(P, n1 * n2, tm_synth.rng(953, 3))
    m, t, _ = rounded(masks, t0, I)
    op = ops.FFTOp(m, n1, n2)
    Id, Iv = device_intensities(I, bf16)
    mk, td = c64(masks), c64(t0)
    for kw, ref in ((dict(), rt.er_step(op, Iv, rt.er_step(op, Iv, t))),
                    (dict(er_momentum=0.6), rt.er_accelerated(op, Iv, t, 2, 0.6))):
        tt = td.clone()  # sums only after the last step: both forms of the kernel
        tm.tm_retrieve(ctx, mk, Id, tt, n1, n2, tm.retrieve_opts("er", iters=2, bf16=bf16, **kw))
        assert relerr(tt.cpu().numpy(), ref) < 2 * K * OPTOL, kw
    for grad, ref in ((tm.tm_gradient, rt.intensity_grad), (tm.tm_amp_gradient, rt.amplitude_grad)):
        g, f = grad(ctx, mk, Id, td, n1, n2)
        fo, go, _ = ref(op, Iv, t)
        assert relerr(g.cpu().numpy(), go) < OPTOL and relerr(f.cpu().numpy(), fo) < OPTOL


@pytest.mark.parametrize("n1,n2", [(1, 16), (4, 4), (4, 16), (16, 4), (8, 8), (1, 64), (16, 16), (8, 32), (1, 1024),
                                   (32, 64), (128, 32), (64, 128)])
@pytest.mark.parametrize("P", [1, 70])
def test_masks_in_sequence(ctx, n1, n2, P):
    # rows from one lane (1 x 16, 4 x 4) to eight waves; every mask's transform follows
    # another in the same LDS copy: two of a kind (operator), alternating (cyclic sweep)
    K = 3
    masks, T, I, _ = problem(n1, n2, K, P, cfg=954, noise=1e4)
    m, t, Ir = rounded(masks, T, I)
    op = ops.FFTOp(m, n1, n2)
    mk, td = c64(masks), c64(T)
    y = tm.tm_forward(ctx, mk, td, n1, n2)
    assert relerr(y.cpu().numpy(), op.forward(t)) < OPTOL
    x = tm.tm_adjoint(ctx, mk, y, n1, n2).cpu().numpy()
    assert relerr(x, op.adjoint(y.cpu().numpy().astype("complex128"))) < OPTOL
    rho = tm.tm_residual_f64(ctx, mk, c64(I).real.contiguous(), td, n1, n2).cpu().numpy()
    # FP64 throughout, of residuals around 1e-2
    assert relerr(rho, rt.acceptance_residual(op, Ir, t)) < 1e-10
    tt = td.clone()
    tm.tm_retrieve(ctx, mk, c64(I).real.contiguous(), tt, n1, n2, tm.retrieve_opts("er_cyclic", iters=1))
    # K projections, each near the row: those of few points can divide by small fields
    assert relerr(tt.cpu().numpy(), rt.er_cyclic(m, n1, n2, Ir, t, 1)) < 4 * K * OPTOL


@pytest.mark.parametrize("bf16", [False, True])
def test_few_rows_of_8192_points_have_the_same_bits(ctx, bf16):
    # 64 x 128: up to one row per CU the adjoint and the cyclic sweep run with two LDS copies
    n1, n2, K = 64, 128, 3
    few = torch.cuda.get_device_properties(0).multi_processor_count
    g = torch.Generator().manual_seed(955)
    masks = torch.polar(torch.ones(K, n1 * n2), 6.28 * torch.rand(K, n1 * n2, generator=g)).to(dev())
    T = torch.randn(few + 1, n1 * n2, dtype=torch.complex64, generator=g).to(dev())
    y = tm.tm_forward(ctx, masks, T, n1, n2)
    Id = (y.abs() ** 2).to(torch.bfloat16 if bf16 else torch.float32)
    x = tm.tm_adjoint(ctx, masks, y, n1, n2)
    assert torch.equal(tm.tm_adjoint(ctx, masks, y[:few].contiguous(), n1, n2), x[:few])
    o = tm.retrieve_opts("er_cyclic", iters=2, bf16=bf16)
    many, t = T + 0.1, (T + 0.1)[:few].contiguous()
    tm.tm_retrieve(ctx, masks, Id, many, n1, n2, o)
    tm.tm_retrieve(ctx, masks, Id[:few].contiguous(), t, n1, n2, o)
    assert torch.equal(t, many[:few])
