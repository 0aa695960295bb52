"""The ring launches of batches, at the first map count that takes them, against the oracle.

Few maps run all ring pairs in one launch; from some count on, which depends on Nside, a batch runs one launch
per transform kind and length, the short transforms one wave (64 threads) per ring pair. The count is looked for here by
the kernels that run, so these tests stay on the batched launches wherever the bound lies: long and
short Bluestein rings, long mixed-radix rings, long power-of-two rings, and the one-wave class.
Bars: 1e-12 in FP64 and 1e-5 in FP32, those of the transforms; static workspace against plan buffers
1e-13 and 1e-6, the same radices and sums in other workgroup sizes.
"""
import re

import numpy as np
import pytest

from oracle import sht
from tests.helpers import alm_rel_l2, random_alm, rel_l2

pytestmark = pytest.mark.gpu

COUNTS = (4, 6, 9, 13, 17, 25, 33, 49, 65)
# batched launches of one ring phase: the one-wave class alone up to Nside 128 (transforms of at most 1024
# points); with the longest Bluestein rings and the long mixed-radix rings at 256; with long powers of two beyond
LAUNCHES = {16: 1, 32: 1, 64: 1, 128: 1, 256: 3, 512: 4, 1024: 4}


def ring_threads(call):
    """Threads per workgroup of the ring launches of call()."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    found = [re.search(r"phase_b_kernel<\w+, \w+, (\d+),", e.name) for e in prof.events()]
    return [int(f.group(1)) for f in found if f]


def batched_plan(nside, lmax, dtype):
    """Plan and maps of the first batch that takes the batched ring launches."""
    import torch
    from paper_1211_0585_amd import mwf
    npix = 12 * nside * nside
    tt = torch.float32 if dtype else torch.float64
    for n in COUNTS:
        p = mwf.Plan(nside, lmax, np.ones(lmax + 1), np.ones(npix), dtype=dtype, max_batch=n)
        x = torch.randn(n, npix, dtype=tt, device="cuda", generator=torch.Generator("cuda").manual_seed(nside + n))
        threads = ring_threads(lambda: p.map2alm(x))
        assert threads, "no ring kernel seen"
        if 64 in threads:
            print(f"Nside {nside}: {n} maps, ring launches of {threads} threads", flush=True)
            assert len(threads) == LAUNCHES[nside]
            return p, x
        p.close()
    raise AssertionError("no map count takes the batched ring launches")


@pytest.mark.parametrize("dtype,bar", [(0, 1e-12), (1, 1e-5)], ids=["f64", "f32"])
@pytest.mark.parametrize("nside,lmax", [(16, 47), (32, 48), (64, 70), (128, 130), (256, 64), (512, 40), (1024, 24)])
def test_batched_ring_launches_vs_oracle(nside, lmax, dtype, bar):
    import torch
    p, x = batched_plan(nside, lmax, dtype)
    nmaps = x.shape[0]
    alm = np.stack([random_alm(lmax, nside + i) for i in range(nmaps)])
    if dtype:
        alm = alm.astype(np.complex64)
    with p:
        b = torch.from_numpy(alm).cuda()
        assert 64 in ring_threads(lambda: p.alm2map(b))
        a, f = p.map2alm(x).cpu().numpy(), p.alm2map(b).cpu().numpy()
        p.sync()
    for i in (0, nmaps - 1):
        ea = alm_rel_l2(a[i], sht.map2alm(x[i].double().cpu().numpy(), nside, lmax), lmax)
        ef = rel_l2(f[i], sht.alm2map(alm[i].astype(np.complex128), nside, lmax))
        print(f"Nside {nside} lmax {lmax} map {i} of {nmaps}: analysis {ea:.2e} synthesis {ef:.2e}", flush=True)
        assert ea <= bar and ef <= bar


@pytest.mark.parametrize("dtype,tol", [(0, 1e-13), (1, 1e-6)], ids=["f64", "f32"])
@pytest.mark.parametrize("nside,lmax", [(64, 40), (256, 24), (512, 10)])
def test_batched_static_solve_equals_plan_solve(nside, lmax, dtype, tol):
    p, x = batched_plan(nside, lmax, dtype)
    lams = [20.0, 4.0, 1.0]
    with p:
        assert 64 in ring_threads(lambda: p.solve(x, lams, static=True))
        whole = p.solve(x, lams)[0].clone()
        static = p.solve(x, lams, static=True)[0].clone()
        p.sync()
    err = rel_l2(static.double().cpu().numpy(), whole.double().cpu().numpy())
    print(f"Nside {nside} lmax {lmax} maps {x.shape[0]}: {err:.2e}", flush=True)
    assert err <= tol
