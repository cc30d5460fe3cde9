"""Mixed-axis FFT plans (32x32, 64x32, 64x64, 128x64) in every row kernel that
runs them, from one row up and with one mask (one transform pair, so that each
pass's twiddles and exchanges count alone), against the FP64 oracle. Tolerances
are those of the per-step operators: 1e-5 relative per transform pair in FP32."""
import numpy as np
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


@pytest.mark.parametrize("n1,n2", [(32, 32), (64, 32), (64, 64), (128, 64)])
@pytest.mark.parametrize("K,P", [(1, 1), (3, 11)])
def test_every_mode(ctx, n1, n2, K, P):
    N = n1 * n2
    masks, T, I, _ = problem(n1, n2, K, P, cfg=951, noise=1e4)
    t0 = T + 0.3 * tm_synth.tm_iid(P, N, tm_synth.rng(951, 3))
    m, t, Ir = rounded(masks, t0, I)
    op = ops.FFTOp(m, n1, n2)
    mk, td = c64(masks), c64(t0)
    # single values at every place of the grid's edges: a misplaced slot shows at once
    e = np.zeros((P, N), dtype=np.complex64)
    e[np.arange(P), (np.arange(P) * (N - 1)) // max(P - 1, 1)] = 1.0
    assert relerr(tm.tm_forward(ctx, mk, c64(e), n1, n2).cpu().numpy(), op.forward(e.astype(np.complex128))) < OPTOL
    y = op.forward(t).astype(np.complex64)
    x = tm.tm_adjoint(ctx, mk, c64(y), n1, n2).cpu().numpy()
    assert relerr(x, op.adjoint(y.astype(np.complex128))) < OPTOL
    for bf in (False, True):
        Id, Iv = device_intensities(I, bf)
        g, f = tm.tm_gradient(ctx, mk, Id, td, n1, n2)
        fo, go, _ = rt.intensity_grad(op, Iv.reshape(P, K, N), t)
        assert relerr(g.cpu().numpy(), go) < OPTOL and relerr(f.cpu().numpy(), fo) < OPTOL, bf
        g, f = tm.tm_amp_gradient(ctx, mk, Id, td, n1, n2)
        fo, go, _ = rt.amplitude_grad(op, Iv.reshape(P, K, N), t)
        assert relerr(g.cpu().numpy(), go) < OPTOL and relerr(f.cpu().numpy(), fo) < OPTOL, bf
        for method, iters, kw, ref in (
                ("er", 2, {}, lambda s: rt.er_step(op, Iv, rt.er_step(op, Iv, s))),
                ("er", 2, dict(er_momentum=0.6), lambda s: rt.er_accelerated(op, Iv, s, 2, 0.6)),
                ("er_cyclic", 2, {}, lambda s: rt.er_cyclic(m, n1, n2, Iv, s, 2)),
                ("er", 0, dict(start="lanczos", spectral_iters=2, spectral_tau=3.0),
                 lambda s: rt.spectral_lanczos(op, Iv, s, 2, tau=3.0)),
                ("er", 0, dict(start="spectral", spectral_iters=2, spectral_momentum=0.5),
                 lambda s: rt.spectral_start(op, Iv, s, 2, tau=3.0, momentum=0.5)),
                ("er", 0, dict(start="backprop"), lambda s: rt.backprop_start(op, Iv))):
            tt = td.clone()
            tm.tm_retrieve(ctx, mk, Id, tt, n1, n2, tm.retrieve_opts(method, iters=iters, bf16=bf, **kw))
            err = relerr(tt.cpu().numpy(), ref(t))
            print(f"{n1}x{n2} K={K} P={P} bf16={bf} {method} {kw}: {err:.2e}", flush=True)
            # two steps of K pairs each; the heavy-ball start's normalisations as in its own test
            assert err < (2e-4 if kw.get("start") == "spectral" else 2 * K * OPTOL), (method, kw)


def test_rows_around_a_round_of_workgroups(ctx):
    # one row fewer and one more than two workgroups on each of 256 CUs hold: the
    # same rows come out whatever the launch holds beside them
    n1, n2, K = 64, 64, 1
    N = n1 * n2
    masks = c64(tm_synth.mask_phases(K, N, tm_synth.rng(952, 0)))
    T = c64(tm_synth.tm_iid(513, N, tm_synth.rng(952, 1)))
    y = tm.tm_forward(ctx, masks, T, n1, n2)
    for P in (511, 512):
        assert torch.equal(tm.tm_forward(ctx, masks, T[:P].contiguous(), n1, n2), y[:P])
    assert y.device == dev()
