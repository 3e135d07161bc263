"""Load profile of variables that arrive in the order in which they are allocated: neighbouring lanes meet the same
step, and the scatter kernels add runs of equal steps as one.  All kernels (small traces in one launch, short and long time
lines), run lengths on either side of where runs are merged, and list lengths at the edges of waves, groups and
workgroups."""
import numpy as np
import pytest

from gpu_util import u64
from helpers import mk_trace

pytestmark = pytest.mark.gpu


# a wave's 256 variables form 256 / run runs: 1 to 64 of its lanes, and 32 and 33
@pytest.mark.parametrize("long_line", [False, True])
@pytest.mark.parametrize("n,run", [(1, 1), (3, 2), (63, 64), (64, 64), (65, 2), (257, 8), (1023, 3), (1025, 1), (4095, 7),
                                   (4096, 8), (4097, 9), (8193, 345), (20011, 16), (12288, 100000),
                                   (16384, 5), (16385, 5)])
def test_load_profile_sorted_runs(oracle_mod, long_line, n, run):
    import paper_1903_06631_amd as lap
    rng = np.random.default_rng(n * 7 + run)
    alloc = np.arange(n) // run
    top = int(alloc[-1]) + 600
    T = max(top, 8192 + 57) if long_line else min(top, 8191)
    alloc = np.minimum(alloc, T - 1)
    free = alloc + 1
    far = rng.random(n) < 0.03                                     # a few live longer: they break the runs of releases
    free[far] = np.minimum(T, free[far] + rng.integers(1, 580, int(far.sum())))
    size = rng.integers(1, 1 << 40, n)
    size[rng.random(n) < 0.1] = (1 << 46) + 1                      # sums of a run pass 2^53
    tr = mk_trace(size, alloc, free, T=T)
    got = lap.load_profile(lap.DeviceTrace(tr))
    load, peak, at = oracle_mod.load_profile(tr)
    assert np.array_equal(u64(got["load"]), load)
    assert int(u64(got["peak"])[0]) == peak and int(got["t_peak"].item()) == at


@pytest.mark.parametrize("n,T", [(257, 30), (20000, 500), (20000, 20000)])
@pytest.mark.parametrize("off", [(1, 0, 0), (0, 1, 0), (0, 0, 3), (1, 2, 2)])
def test_load_profile_unaligned_arrays(oracle_mod, n, T, off):
    """arrays that are aligned to their elements only: no 16-byte loads"""
    import torch
    import paper_1903_06631_amd as lap
    from traces import random_trace
    tr = random_trace(n + T, n, T)
    dt = lap.DeviceTrace(tr, use_gaps=False)

    def moved(t, by):
        big = torch.empty(t.numel() + by, dtype=t.dtype, device=t.device)
        big[by:] = t
        return big[by:]

    dt.size, dt.alloc, dt.free = moved(dt.size, off[0]), moved(dt.alloc, off[1]), moved(dt.free, off[2])
    got = lap.load_profile(dt)
    load, peak, at = oracle_mod.load_profile(tr)
    assert np.array_equal(u64(got["load"]), load)
    assert int(u64(got["peak"])[0]) == peak and int(got["t_peak"].item()) == at


# on both sides of the number of steps whose bins lie in LDS together; variables for one and for several workgroups, for
# less and more than a turn of each; with events at the first and at the last step
@pytest.mark.parametrize("in_order", [False, True])
@pytest.mark.parametrize("n,T", [(16385, 1), (16385, 8191), (16385, 8192), (20000, 4095), (20000, 4096), (65537, 8191),
                                 (1_048_577, 4094), (2_100_003, 8191), (2_100_003, 3)])
def test_load_profile_short_lines(oracle_mod, n, T, in_order):
    import paper_1903_06631_amd as lap
    rng = np.random.default_rng(n + T)
    alloc = rng.integers(0, T, n)
    alloc[:2], alloc[-2:] = 0, T - 1
    free = np.minimum(T, alloc + rng.integers(1, 40, n))
    free[::997] = T
    if in_order:
        o = np.argsort(alloc, kind="stable")
        alloc, free = alloc[o], free[o]
    tr = mk_trace(rng.integers(1, 1 << 40, n), alloc, free, T=T)
    got = lap.load_profile(lap.DeviceTrace(tr, use_gaps=False))
    load, peak, at = oracle_mod.load_profile(tr)
    assert np.array_equal(u64(got["load"]), load)
    assert int(u64(got["peak"])[0]) == peak and int(got["t_peak"].item()) == at


def test_load_profile_unordered_time():
    """On a time line whose bins all lie in LDS the order of the variables costs next to nothing (1.1 times the time of
    variables in order; 3.1 times when a workgroup flushed its bins after every 4096 variables)."""
    import torch
    import paper_1903_06631_amd as lap
    n, T = 16 << 20, 8191
    rng = np.random.default_rng(1)
    alloc = rng.integers(0, T, n)
    best = []
    lap.profile_enable(True)
    try:
        for a in (np.sort(alloc), alloc):
            dt = lap.DeviceTrace(mk_trace(np.full(n, 512), a, a + 1, T=T), use_gaps=False)
            times = []
            for _ in range(8):
                lap.load_profile(dt, sync=False)
                torch.cuda.synchronize()
                times.append(lap.profile_last_ms(lap.K_LOAD_SCATTER))
            best.append(min(times[1:]))
    finally:
        lap.profile_enable(False)
    assert best[1] < 1.8 * best[0], best
