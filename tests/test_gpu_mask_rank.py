"""The fiber mask by counted ranks at the sizes where its pieces change (one
pixel, one wave, the 1024 sorted places of a round, the largest), with ties,
and the row gather at the edges of its 64-image tiles, against the oracle."""
import numpy as np
import pytest
import torch

import paper_2302_13524_amd as tm
from oracle import preprocess as pp

from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = tm.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("npix", [1, 2, 15, 17, 64, 1023, 1024, 1025, 3000, 8191, 8192])
@pytest.mark.parametrize("kind", ["whole numbers", "ties", "one value"])
def test_mask(ctx, npix, kind):
    # sums of whole numbers are exact in any order, so the masks are equal
    g = np.random.default_rng(npix)
    E = np.ones(npix) if kind == "one value" else g.integers(0, 4 if kind == "ties" else 1 << 30, npix).astype(float)
    E[0] += 1.0
    for frac in (0.25, 0.999, 1.0):
        pix = tm.tm_pre_fiber_mask(ctx, torch.from_numpy(E).to(dev()), frac).cpu().numpy()
        assert np.array_equal(pix, pp.fiber_mask(E, frac)), frac


def test_mask_of_energies_that_are_not_numbers(ctx):
    E = np.arange(1.0, 2001.0)
    E[[3, 700, 1999]] = np.nan  # no total, no mask
    assert tm.tm_pre_fiber_mask(ctx, torch.from_numpy(E).to(dev()), 0.9).numel() == 0
    E[[3, 700, 1999]] = [np.inf, 0.0, -5.0]
    assert tm.tm_pre_fiber_mask(ctx, torch.from_numpy(E).to(dev()), 0.9).cpu().tolist() == [3]


@pytest.mark.parametrize("n", [1, 63, 64, 65, 130])
@pytest.mark.parametrize("P", [1, 255, 257])
@pytest.mark.parametrize("dtype", [np.uint16, np.float32])
@pytest.mark.parametrize("bf16", [False, True])
def test_gather(ctx, n, P, dtype, bf16):
    g = np.random.default_rng(n + P)
    stack = g.integers(0, 65536, (n, 48, 50)).astype(dtype)
    pix = np.sort(g.permutation(24 * 25)[:P]).astype(np.int32)
    rows = tm.tm_pre_gather(ctx, torch.from_numpy(stack).to(dev()), torch.from_numpy(pix).to(dev()), bf16=bf16)
    ref = torch.from_numpy(pp.gather_rows(stack, pix).astype(np.float32))
    assert torch.equal(rows.cpu(), ref.to(torch.bfloat16) if bf16 else ref)
