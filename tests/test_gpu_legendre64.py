"""FP64 Legendre kernels at the edges of their blocks, forms and work lists, against the oracle.

The sizes take every block size of the analysis (64, 128, 256 ring pairs) and of the synthesis,
one to several items per (m, block), rows that end inside a step pair or a chunk, and the three
forms of the recurrence (equatorial, plain and cap blocks; the plain one from Nside 512 on).
Bar: 1e-12 relative L2, the bar of the FP64 transforms (rounding of the sums is far below it).
"""
import numpy as np
import pytest

from oracle import sht
from tests.helpers import alm_rel_l2, rel_l2

pytestmark = pytest.mark.gpu

SIZES = [(1, 0), (1, 3), (2, 1), (8, 15), (8, 16), (32, 33), (64, 65), (128, 200), (256, 301), (512, 129)]


@pytest.mark.parametrize("nside,lmax", SIZES)
def test_pair_vs_oracle(nside, lmax):
    import torch
    from paper_1211_0585_amd import mwf
    rng = np.random.default_rng(nside * 4096 + lmax)
    npix = 12 * nside * nside
    maps = rng.standard_normal((2, npix))
    alm = rng.standard_normal((2, mwf.n_alm(lmax))) + 1j * rng.standard_normal((2, mwf.n_alm(lmax)))
    alm[:, :lmax + 1] = alm[:, :lmax + 1].real
    with mwf.Plan(nside, lmax, np.ones(lmax + 1), np.ones(npix), max_batch=2) as p:
        for _ in range(2):                       # the second pass reuses the plan's buffers
            a = p.map2alm(torch.from_numpy(maps).cuda())
            f = p.alm2map(torch.from_numpy(alm).cuda())
        p.sync()
        a, f = a.cpu().numpy(), f.cpu().numpy()
    for i in range(2):
        ea = alm_rel_l2(a[i], sht.map2alm(maps[i], nside, lmax), lmax)
        ef = rel_l2(f[i], sht.alm2map(alm[i], nside, lmax))
        print(f"Nside {nside} lmax {lmax} map {i}: analysis {ea:.2e} synthesis {ef:.2e}", flush=True)
        assert ea <= 1e-12 and ef <= 1e-12
