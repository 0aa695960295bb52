"""The benchmark's count of Legendre units against 80-bit values of lambda_lm."""
import numpy as np
import pytest

import bench
from oracle import healpix
from tests.test_gpu_few_rings import lambda_tables


@pytest.mark.parametrize("nside,lmax", [(1, 3), (8, 31), (32, 95), (64, 200)])
def test_summed_units(nside, lmax):
    z = healpix.ring_info(nside)["z"][:2 * nside]
    first = np.full((2 * nside, lmax + 1), lmax + 1)
    for l, lam in lambda_tables(z, lmax):
        m = np.arange(l + 1)
        new = (np.abs(lam) > np.longdouble(2) ** -128) & (first[:, :l + 1] > lmax)
        first[:, :l + 1] = np.where(new, l - m, first[:, :l + 1])
    want = int(np.maximum(lmax + 1 - np.arange(lmax + 1) - first, 0).sum())
    assert bench.summed_units(nside, lmax) == want
