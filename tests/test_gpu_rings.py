"""Ring transforms at every Bluestein length and launch shape, against the oracle.

Nside 8 to 512 covers Bluestein transforms of 128 to 4096 points, the largest Nside
8192; 1 and 3 maps take the launches of few maps, 4 and more the batched ones; 3, 5 and 11
maps leave ragged blocks in the ring-major map order. Bars: 1e-12 in FP64, the bar of the FP64
transforms; 1e-5 in FP32, the bar of the reduced-precision ones. The first and the last map of the
batch are compared: they sit in different blocks.
"""
import numpy as np
import pytest

from oracle import sht
from tests.helpers import alm_rel_l2, random_alm, rel_l2

pytestmark = pytest.mark.gpu

SHAPES = [(1, 2, 5), (8, 15, 1), (16, 47, 4), (32, 33, 11), (64, 70, 5), (128, 130, 3), (128, 130, 4),
          (256, 64, 5), (512, 40, 1), (512, 40, 4), (1024, 24, 1), (1024, 24, 4)]


@pytest.mark.parametrize("dtype,bar", [(0, 1e-12), (1, 1e-5)], ids=["f64", "f32"])
@pytest.mark.parametrize("nside,lmax,nmaps", SHAPES)
def test_ring_transforms_vs_oracle(nside, lmax, nmaps, dtype, bar):
    import torch
    from paper_1211_0585_amd import mwf
    rng = np.random.default_rng(nside * 64 + nmaps)
    npix = 12 * nside * nside
    maps = rng.standard_normal((nmaps, npix))
    alm = np.stack([random_alm(lmax, nside + i) for i in range(nmaps)])
    if dtype:
        maps, alm = maps.astype(np.float32), alm.astype(np.complex64)
    with mwf.Plan(nside, lmax, np.ones(lmax + 1), np.ones(npix), dtype=dtype, max_batch=nmaps) as p:
        a = p.map2alm(torch.from_numpy(maps).cuda())
        f = p.alm2map(torch.from_numpy(alm).cuda())
        p.sync()
        a, f = a.cpu().numpy(), f.cpu().numpy()
    for i in sorted({0, nmaps - 1}):
        ea = alm_rel_l2(a[i], sht.map2alm(maps[i].astype(np.float64), nside, lmax), lmax)
        ef = rel_l2(f[i], sht.alm2map(alm[i].astype(np.complex128), nside, lmax))
        print(f"Nside {nside} lmax {lmax} map {i} of {nmaps}: analysis {ea:.2e} synthesis {ef:.2e}", flush=True)
        assert ea <= bar and ef <= bar
