"""wf_footprint against the device memory that a first plan of a shape takes.

The allocator rounds: up to 2 MiB for each of the larger buffers of a plan and its tables, of which there
are fewer than eight; and the footprint is an upper estimate where the polar skip leaves work items out, by
less than a quarter. (An estimate several times too high refuses plans that fit.)
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

MIB = 1 << 20


@pytest.mark.parametrize("nside,lmax,dtype,nmaps", [
    (16, 33, 0, 1), (64, 190, 0, 1), (64, 254, 0, 4), (128, 255, 0, 1), (256, 301, 0, 2), (256, 511, 0, 1), (256, 701, 0, 1),
    (512, 301, 0, 1), (512, 1020, 0, 1), (1024, 255, 0, 1), (128, 255, 1, 1), (256, 509, 1, 4)])
def test_footprint_is_what_a_plan_takes(nside, lmax, dtype, nmaps):
    import torch
    from paper_1211_0585_amd import mwf
    torch.cuda.synchronize()
    with mwf.Plan(4, 7, np.ones(8), np.ones(192), dtype=dtype):
        before = torch.cuda.mem_get_info()[0]
        with mwf.Plan(nside, lmax, np.ones(lmax + 1), np.ones(12 * nside * nside), dtype=dtype, max_batch=nmaps):
            used = before - torch.cuda.mem_get_info()[0]
    est = mwf.footprint(nside, lmax, dtype, nmaps)
    print(f"Nside {nside} lmax {lmax} dtype {dtype} maps {nmaps}: footprint {est / MIB:.1f} MiB, used {used / MIB:.1f} MiB", flush=True)
    assert used <= est + 16 * MIB
    assert est <= 1.25 * used + 2 * MIB
