"""FFT digit orders where they are two kernels (one axis per pass), and launch
configurations beside a batch, which runs the kernels of configuration 0."""
import pytest
import torch

import paper_2302_13524_amd as tm
import tm_synth
from oracle import operators as ops
from oracle import retrieval as rt

from gpu_util import c64, f32, problem, relerr, rounded
from test_gpu_batch import SHAPES, make_problems, opts, singles

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = tm.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n1,n2", [(8, 32), (32, 64), (32, 128), (128, 32), (64, 128)])
def test_both_digit_orders(ctx, n1, n2):
    assert tm.tm_config_kernel(n1, n2, 1)[0] == 1
    K, P = 4, 7
    masks, T, I, _ = problem(n1, n2, K, P, cfg=956, noise=1e4)
    t0 = T + 0.5 * tm_synth.tm_iid(P, n1 * n2, tm_synth.rng(956, 3))
    m, t, Ir = rounded(masks, t0, I)
    op = ops.FFTOp(m, n1, n2)
    mk, td = c64(masks), c64(t0)
    ref = rt.er_step(op, Ir, t)
    try:
        for v in (0, 1):
            tm.tm_set_variant(ctx, n1, n2, v)
            y = tm.tm_forward(ctx, mk, td, n1, n2)
            assert relerr(y.cpu().numpy(), op.forward(t)) < 1e-5, v
            x = tm.tm_adjoint(ctx, mk, y, n1, n2).cpu().numpy()
            assert relerr(x, op.adjoint(y.cpu().numpy().astype("complex128"))) < 1e-5, v
            tt = td.clone()
            tm.tm_retrieve(ctx, mk, f32(I), tt, n1, n2, tm.retrieve_opts("er", iters=1))
            assert relerr(tt.cpu().numpy(), ref) < 1e-5, v
    finally:
        tm.tm_set_variant(ctx, n1, n2, 0)


@pytest.mark.parametrize("cfg", range(8))
def test_batch_beside_any_configuration(ctx, cfg):
    shapes = [s for s in SHAPES if tm.tm_config_info(s[0], s[1], cfg) is not None]
    probs = make_problems(ctx, shapes, cfg=985)
    ref = singles(ctx, probs, 0.0, 3, 2, "er_cyclic", "lanczos")
    try:
        for p in probs:
            tm.tm_set_config(ctx, p["n1"], p["n2"], cfg)
        b = tm.Batch(ctx, probs, opts(0.0, 3, 2, "er_cyclic", "lanczos"), use_graph=True)
        b.run()
        torch.cuda.synchronize()
        for p, r in zip(probs, ref):
            assert torch.equal(p["t"], r), (p["n1"], p["n2"])
        b.close()
    finally:
        for p in probs:
            tm.tm_set_config(ctx, p["n1"], p["n2"], 0)
