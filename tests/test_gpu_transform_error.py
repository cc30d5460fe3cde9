"""Error of the mixed-axis FFT plans against 64 bits: no larger than that of the
plans with one axis per pass, which run where no mixed-axis plan is compiled. The
bounds are those plans' rms errors for normal inputs (their FP32 arithmetic redone
on the CPU); over this many values the rms of another sample is within 0.2 %."""
import numpy as np
import pytest
import torch

import paper_2302_13524_amd as tm

from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n1,n2,rms", [(32, 32, 1.062e-7), (64, 32, 1.125e-7), (64, 64, 1.186e-7),
                                       (128, 64, 1.234e-7)])
@pytest.mark.parametrize("P", [50, 4100])
def test_transform_error(n1, n2, rms, P):
    # masks of ones: their product is exact, so that one transform's error is left
    ctx = tm.Context(0)
    N = n1 * n2
    g = torch.Generator(device=dev()).manual_seed(N)
    ones = torch.ones((1, N), dtype=torch.complex64, device=dev())
    x = torch.randn((P, N), generator=g, device=dev(), dtype=torch.complex64)
    for inverse in (False, True):
        if inverse:
            got = tm.tm_adjoint(ctx, ones, x[:, None].contiguous(), n1, n2)
        else:
            got = tm.tm_forward(ctx, ones, x, n1, n2)[:, 0]
        v = x[:512].cpu().numpy().astype(np.complex128).reshape(-1, n1, n2)
        ref = (np.fft.ifft2(v) * N if inverse else np.fft.fft2(v)).reshape(-1, N)
        err = np.sqrt(np.mean(np.abs(got[:512].cpu().numpy() - ref) ** 2) / np.mean(np.abs(ref) ** 2))
        print(f"{n1}x{n2} P={P} {'inverse' if inverse else 'forward'}: rms error {err:.4e}", flush=True)
        assert err < 1.002 * rms
    ctx.close()
