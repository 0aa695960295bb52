"""Device work of plan building, counted by the profiler: what a plan does not need is not done."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def events(call):
    """Names of the kernels and runtime calls of call()."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
        call()
        torch.cuda.synchronize()
    return [e.name for e in prof.events()]


def test_one_reach_pass_per_new_shape():
    """The polar reach of a shape is found in one pass, FP64 or not; a later FP64 plan of a shape that a
    reduced-precision plan made adds one, a further plan none."""
    from paper_1211_0585_amd import mwf

    def made(nside, lmax, dtype, keep):
        def call():
            keep.append(mwf.Plan(nside, lmax, np.ones(lmax + 1), np.ones(12 * nside * nside), dtype=dtype))
        names = events(call)
        return sum("reach_kernel" in n for n in names), sum("start_state_kernel" in n for n in names)

    keep = []
    assert made(32, 41, 1, keep)[0] == 1          # the profiler sees this library's kernels
    reach, states = made(32, 43, 0, keep)
    assert states >= 2
    assert reach == 1
    assert made(32, 41, 0, keep)[0] == 1
    assert made(32, 43, 0, keep) == (0, 0)
    for p in keep:
        p.close()


@pytest.mark.parametrize("nside,streams", [(16, 0), (256, 0), (1024, 1)])
def test_truncated_solve_makes_a_stream_only_where_used(nside, streams):
    """The ring phase of one map forks onto a second stream only where its transforms do not go in one
    launch (beyond 4096 points); a truncated solve makes no stream anywhere else."""
    import torch
    from paper_1211_0585_amd import mwf
    lmax, npix = 24, 12 * nside * nside
    x = torch.randn(npix, dtype=torch.float64, device="cuda")
    with mwf.Plan(nside, lmax, np.ones(lmax + 1), np.ones(npix)) as p:
        names = events(lambda: p.solve_banded(x, [3.0, 2.0, 1.0], [8, 16, 24]))
        p.sync()
    assert sum("phase_b_kernel" in n for n in names) >= 4
    assert sum("hipStreamCreate" in n for n in names) == streams
