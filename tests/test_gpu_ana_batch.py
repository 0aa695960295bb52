"""FP64 analysis of a batch against its maps one at a time.

From a number of maps on (80 l a wave of a full launch) shapes with short items take other work
items, split elsewhere in l and dealt to other workgroups. Every (l, m) still adds the same products in the
same order, so the coefficients agree bit for bit where both calls run the same ring kernels; where the batch
takes other ring kernels (more than 8 maps below Nside 256), to 1e-13, the transforms' errors being below 1e-14.
"""
import numpy as np
import pytest

from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nside,lmax,nmaps,tol", [
    (256, 300, 2, 0), (256, 300, 3, 0), (256, 301, 17, 0), (256, 512, 2, 0), (256, 700, 3, 0), (256, 150, 24, 0),
    (128, 256, 8, 0), (128, 383, 5, 0), (512, 300, 2, 0), (1024, 256, 2, 0), (64, 191, 30, 1e-13), (32, 64, 160, 1e-13)])
def test_batch_analysis_equals_single_maps(nside, lmax, nmaps, tol):
    import torch
    from paper_1211_0585_amd import mwf
    npix = 12 * nside * nside
    gen = torch.Generator(device="cuda").manual_seed(nside + nmaps)
    x = torch.randn(nmaps, npix, dtype=torch.float64, device="cuda", generator=gen)
    with mwf.Plan(nside, lmax, np.ones(lmax + 1), np.ones(npix), max_batch=nmaps) as p:
        whole = p.map2alm(x).cpu().numpy().reshape(nmaps, -1)
        for i in sorted({0, nmaps // 2, nmaps - 1}):
            one = p.map2alm(x[i].contiguous()).cpu().numpy().reshape(-1)
            err = rel_l2(whole[i], one)
            print(f"Nside {nside} lmax {lmax} map {i} of {nmaps}: {err:.2e}", flush=True)
            assert np.array_equal(whole[i], one) if tol == 0 else err <= tol
        p.sync()


def test_polarised_batch_analysis_equals_single_maps():
    """The spin-0 part of a polarised batch takes the same lists; its ring kernels do not depend on the count."""
    import torch
    from paper_1211_0585_amd import mwf
    nside, lmax, nmaps = 128, 383, 6
    npix = 12 * nside * nside
    cl4 = np.zeros((4, lmax + 1))
    cl4[:3, 2:] = 1.0
    ninv6 = np.zeros((6, npix))
    ninv6[:3] = 1.0
    x = torch.randn(nmaps, 3, npix, dtype=torch.float64, device="cuda", generator=torch.Generator("cuda").manual_seed(7))
    with mwf.PolPlan(nside, lmax, cl4, ninv6, max_batch=nmaps) as p:
        whole = p.map2alm(x).cpu().numpy().reshape(nmaps, 3, -1)
        for i in (0, nmaps - 1):
            one = p.map2alm(x[i].contiguous()).cpu().numpy().reshape(3, -1)
            assert np.array_equal(whole[i], one)
        p.sync()
