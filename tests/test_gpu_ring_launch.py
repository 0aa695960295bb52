"""One ring launch against the launches per transform kind, at the map counts where the choice turns.

A batch beyond the bound of the single launch and the same maps in smaller calls run different ring
kernels (threads per ring, order of the rings). Both use the same radices and sums, so the results
agree to rounding: 1e-13 relative in FP64 (the transforms' errors are below 1e-14), 1e-6 in FP32.
"""
import numpy as np
import pytest

from tests.helpers import rel_l2

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,tol", [(0, 1e-13), (1, 1e-6)], ids=["f64", "f32"])
@pytest.mark.parametrize("nside,nmaps", [(1, 9), (16, 9), (64, 9), (128, 9), (256, 25), (512, 9)])
def test_batch_beyond_one_launch_equals_parts(nside, nmaps, dtype, tol):
    import torch
    from paper_1211_0585_amd import mwf
    lmax, npix = min(2 * nside, 96), 12 * nside * nside
    ell = np.arange(lmax + 1)
    d = np.random.default_rng(nside).standard_normal((nmaps, npix))
    x = torch.from_numpy(d if dtype == 0 else d.astype(np.float32)).cuda()
    lams = np.geomspace(50.0, 1.0, 3)
    part = 8 if nside != 256 else 24
    with mwf.Plan(nside, lmax, 1.0 / (1.0 + ell) ** 2, np.ones(npix), dtype=dtype, max_batch=nmaps) as p:
        whole = p.solve(x, lams)[0].clone()
        parts = torch.cat([p.solve(x[i:i + part].contiguous(), lams)[0].clone().reshape(-1, npix)
                           for i in range(0, nmaps, part)])
        p.sync()
    err = rel_l2(whole.double().cpu().numpy().reshape(-1), parts.double().cpu().numpy().reshape(-1))
    print(f"Nside {nside} maps {nmaps}: {err:.2e}", flush=True)
    assert err <= tol
