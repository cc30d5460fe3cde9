"""Error of the complex GEMM on split operands (64 and more complex k): what FP32
products and sums give, so that each part and each partial product counts."""
import numpy as np
import pytest
import torch

import paper_2302_13524_amd as tm

from gpu_util import dev
from test_gpu_cgemm_split import _parts

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = tm.Context(0)
    yield c
    c.close()


def _product(ctx, A, B, trans_b=True):
    Bd = B if trans_b else np.ascontiguousarray(B.T)
    return tm.tm_cgemm_f32(ctx, torch.from_numpy(A).to(dev()), torch.from_numpy(Bd).to(dev()), trans_b).cpu().numpy()


@pytest.mark.parametrize("trans_b", [False, True])
@pytest.mark.parametrize("M,N,K", [(64, 64, 64), (200, 130, 97)])
@pytest.mark.parametrize("imag", [False, True])
def test_single_products(ctx, M, N, K, trans_b, imag):
    # one nonzero (real or imaginary) value in each row of A: every component of C is one
    # product of two full mantissas, which FP32 rounds to within 2^-24. The parts' own
    # product of lowest order (2^-33 and less) is left out.
    g = np.random.default_rng(M + K)
    A = np.zeros((M, K), np.complex64)
    v = (g.choice([-1.0, 1.0], M) * np.exp(3 * g.standard_normal(M))).astype(np.float32)
    A[np.arange(M), g.integers(0, K, M)] = v * (1j if imag else 1)
    B = (g.standard_normal((N, K)) + 1j * g.standard_normal((N, K))).astype(np.complex64)
    B[:, :8] = 1 + 2.0**-23 * g.integers(0, 2**12, (N, 8)) + 1j * (1 - 2.0**-24 * g.integers(0, 2**12, (N, 8)))
    C = _product(ctx, A, B, trans_b)
    re, im, _ = _parts(A, B)
    for got, ref in ((C.real, re), (C.imag, im)):
        assert np.all(np.abs(got - ref) <= 2.0**-24 * (1 + 2.0**-8) * np.abs(ref))


@pytest.mark.parametrize("M,N,K", [(127, 63, 65), (128, 64, 79), (257, 130, 97), (64, 64, 101)])
@pytest.mark.parametrize("one_sign", [False, True])
def test_short_sums(ctx, M, N, K, one_sign):
    # sums of up to 13 groups of 8 k: a group's products come out within about a unit in the
    # last place (2^-23) of their magnitudes, the groups' sum within half a unit of each partial
    # sum: 2.5e-7 of the magnitudes is four times the expected largest. Without the third
    # parts the error is 4e-7 to 4e-6.
    g = np.random.default_rng(K)

    def rnd(*s):
        x = g.standard_normal(s) + 1j * g.standard_normal(s)
        return (np.abs(x.real) + 0j if one_sign else x).astype(np.complex64)

    A, B = rnd(M, K), rnd(N, K)
    C = _product(ctx, A, B)
    re, im, mag = _parts(A, B)
    err = max(np.max(np.abs(C.real - re) / mag), np.max(np.abs(C.imag - im) / mag))
    print(f"{M}x{N}x{K} one sign {one_sign}: {err:.2e} of the magnitudes", flush=True)
    assert err < 2.5e-7


def test_long_sum_of_one_sign_is_not_short(ctx):
    # the matrix cores cut off below the accumulator's last place: over 1024 groups that must
    # not add up. The rounding of the groups' sum averages out over the outputs; what is left
    # is a group's own cut, less than a unit in the last place.
    g = np.random.default_rng(9)
    A = np.abs(g.standard_normal((130, 8192))).astype(np.complex64)
    B = np.abs(g.standard_normal((66, 8192))).astype(np.complex64)
    C = _product(ctx, A, B)
    ref = A.real.astype(np.float64) @ B.real.astype(np.float64).T
    short = np.mean((ref - C.real) / ref)
    print(f"mean shortfall {short:.2e}, largest {np.max(np.abs(C.real - ref) / ref):.2e}", flush=True)
    assert abs(short) < 2.0**-23


@pytest.mark.parametrize("value", [1e-15, 1e-30, 1e-42, 2.0**27, np.nan])
def test_other_rows_do_not_see_a_value_out_of_range(ctx, value):
    # values far below the others (a sine of pi, subnormal ones), or large, or NaN, keep the
    # tile on its path: the bits of every other row and column stay
    g = np.random.default_rng(11)

    def rnd(*s):
        return (g.standard_normal(s) + 1j * g.standard_normal(s)).astype(np.complex64)

    A, B = rnd(100, 90), rnd(60, 90)
    C = _product(ctx, A, B)
    A[7, 88] = value
    B[9, 3] = value * 1j
    got = _product(ctx, A, B)
    keep = np.ones(C.shape, bool)
    keep[7] = keep[:, 9] = False
    assert np.array_equal(got[keep], C[keep])


@pytest.mark.parametrize("ea,eb", [(-40, -40), (-100, 10), (10, -100), (-60, -64), (-140, 60), (60, -140), (-70, -75),
                                   (30, 30), (90, -50), (60, 50)])
def test_single_products_of_any_scale(ctx, ea, eb):
    # A's and B's values around 2^ea and 2^eb, subnormal ones among them, beside others near
    # one; products down to FP32's subnormal numbers (steps of 2^-149)
    g = np.random.default_rng(12)
    M, N, K = 130, 70, 64
    A = np.zeros((M, K), np.complex64)
    A[np.arange(M), np.arange(M) % K] = np.ldexp((1 + g.random(M)).astype(np.float32), ea)
    B = np.ldexp((1 + g.random((N, K))).astype(np.float32), eb).astype(np.complex64)
    A[::3, :] = A[::3, :] != 0
    C = _product(ctx, A, B).real.astype(np.float64)
    ref = A.real.astype(np.float64) @ B.real.astype(np.float64).T
    assert np.all(np.abs(C - ref) <= 2.0**-24 * (1 + 2.0**-8) * np.abs(ref) + 2.0**-149)


@pytest.mark.parametrize("trans_b", [False, True])
@pytest.mark.parametrize("M,N,K,pad", [(130, 70, 81, 1), (129, 65, 64, 3), (5, 200, 97, 10)])
def test_padded_rows(ctx, M, N, K, pad, trans_b):
    # leading dimensions beyond the operands' rows (NaN between them), and a result with room
    # between its rows, which stays
    g = np.random.default_rng(pad)
    A = (g.standard_normal((M, K)) + 1j * g.standard_normal((M, K))).astype(np.complex64)
    B = (g.standard_normal((N, K)) + 1j * g.standard_normal((N, K))).astype(np.complex64)
    Bd = B if trans_b else B.T

    def padded(x):
        out = torch.full((x.shape[0], x.shape[1] + pad), float("nan"), dtype=torch.complex64)
        out[:, :x.shape[1]] = torch.from_numpy(np.ascontiguousarray(x))
        return out.to(dev())

    Ap, Bp = padded(A), padded(Bd)
    C = torch.full((M, N + pad), 7.0, dtype=torch.complex64, device=dev())
    rc = ctx.lib.tm_cgemm_f32(ctx.h, M, N, K, Ap.data_ptr(), K + pad, Bp.data_ptr(), Bp.shape[1], int(trans_b),
                              C.data_ptr(), N + pad, 0, torch.cuda.current_stream(dev()).cuda_stream)
    assert rc == tm.TM_OK
    C = C.cpu().numpy()
    assert np.array_equal(C[:, :N], _product(ctx, A, B, trans_b)) and np.all(C[:, N:] == 7.0)
