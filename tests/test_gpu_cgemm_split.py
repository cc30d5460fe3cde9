"""The complex GEMM on split operands (64 and more complex k): edges of its
tiles, remainders of its K steps and operands that do not split, against the
product of the same FP32 inputs in 64 bits."""
import numpy as np
import pytest
import torch

import paper_2302_13524_amd as tm

from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = tm.Context(0)
    yield c
    c.close()


def _parts(A, B):
    """Re and Im of A B^T in 64 bits, and the sum of the products' magnitudes."""
    a, b = A.astype(np.complex128), B.astype(np.complex128)
    ar, ai, br, bi = a.real[:, None], a.imag[:, None], b.real[None], b.imag[None]
    with np.errstate(invalid="ignore"):
        re = (ar * br).sum(-1) - (ai * bi).sum(-1)
        im = (ar * bi).sum(-1) + (ai * br).sum(-1)
    return re, im, np.abs(a) @ np.abs(b).T


def _check(C, A, B):
    re, im, mag = _parts(A, B)
    # K / 8 sums of 8 k, each of six MFMAs, or 2 K FP32 products: at most 2 K + 64
    # roundings of one unit in the last place of what is at most mag
    tol = (2 * A.shape[1] + 64) * 2.0**-23 * mag
    for got, ref in ((C.real, re), (C.imag, im)):
        fin = np.isfinite(ref)
        assert np.array_equal(np.isnan(got), np.isnan(ref))
        assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
        assert np.all(np.abs(got[fin] - ref[fin]) <= tol[fin])


@pytest.mark.parametrize("kind", ["plain", "one sign", "not finite", "tiny", "huge"])
@pytest.mark.parametrize("M,N,K", [(1, 1, 64), (127, 63, 65), (128, 64, 79), (129, 65, 80), (257, 130, 97)])
@pytest.mark.parametrize("trans_b", [False, True])
def test_split_product(ctx, M, N, K, trans_b, kind):
    g = np.random.default_rng(M + N + K)

    def rnd(*s):
        return (g.standard_normal(s) + 1j * g.standard_normal(s)).astype(np.complex64)

    A, B = rnd(M, K), rnd(N, K)
    if kind == "one sign":
        A = (np.abs(A.real) + 0j).astype(np.complex64)
        B = (np.abs(B.real) + 0j).astype(np.complex64)
    elif kind == "not finite":
        A[M - 1, K - 1] = np.inf
        B[0, K // 2] = np.nan
    elif kind == "tiny":  # the last row tile alone holds values that do not split
        A[M - 1, K - 1] = 1e-30
        B[N - 1] *= np.float32(1e-25)
    elif kind == "huge":
        A[0, 0] = 1e25
    Bd = B if trans_b else np.ascontiguousarray(B.T)
    C = tm.tm_cgemm_f32(ctx, torch.from_numpy(A).to(dev()), torch.from_numpy(Bd).to(dev()), trans_b)
    _check(C.cpu().numpy(), A, B)


def test_split_product_on_offset_views(ctx):
    # operands that start 8 bytes off a 16-byte boundary
    g = np.random.default_rng(5)
    M, N, K = 130, 66, 101
    buf = torch.from_numpy((g.standard_normal(1 + M * K + N * K) + 1j * g.standard_normal(1 + M * K + N * K))
                           .astype(np.complex64)).to(dev())
    A, B = buf[1:1 + M * K].view(M, K), buf[1 + M * K:].view(N, K)
    C = tm.tm_cgemm_f32(ctx, A, B, True)
    _check(C.cpu().numpy(), A.cpu().numpy(), B.cpu().numpy())
