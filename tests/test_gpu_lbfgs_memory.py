"""The L-BFGS direction solve (a pair per lane) at the ends of the memory's range,
with the ring full and wrapping, against the FP64 oracle."""
import numpy as np
import pytest

import paper_2302_13524_amd as tm
import tm_synth
from oracle import operators as ops
from oracle import retrieval as rt

from gpu_util import c64, f32, problem, relerr, rounded

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n1,n2,P", [(32, 32, 13), (16, 16, 7)])
@pytest.mark.parametrize("mem,iters,other", [(1, 6, 2), (12, 14, 11), (16, 20, 15)])
def test_memory(n1, n2, P, mem, iters, other):
    ctx = tm.Context(0)
    masks, T, I, _ = problem(n1, n2, 4, P, cfg=933, noise=1e4)
    t0 = T + 0.5 * tm_synth.tm_iid(P, n1 * n2, tm_synth.rng(933, 3))
    m, t, Ir = rounded(masks, t0, I)
    op = ops.FFTOp(m, n1, n2)
    ref, _ = rt.lbfgs(op, Ir, t, iters, m=mem)
    tt = c64(t0)
    tm.tm_retrieve(ctx, c64(masks), f32(I), tt, n1, n2, tm.retrieve_opts("lbfgs", iters=iters, lbfgs_m=mem))
    err = relerr(tt.cpu().numpy().astype(np.complex128), ref)
    # near the minimum, where the steps shrink: the operators' tolerance
    assert err < 1e-5
    # the same rows with another memory differ by more, so the pairs count
    assert relerr(rt.lbfgs(op, Ir, t, iters, m=other)[0], ref) > 10 * err
    ctx.close()
