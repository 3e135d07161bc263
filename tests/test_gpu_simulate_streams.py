"""GPU parity of lap_simulate_swaps where the replay goes from one stream at work to the other and to both: swap-outs that end
before the first swap-in, that go on beside the swap-ins, that the next swap-in waits for, and none at all."""
import numpy as np
import pytest

from helpers import mk_trace
from test_gpu_simulate import _check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lap():
    import paper_1903_06631_amd as lap
    lap.load_library()
    return lap


# T on both sides of a window of 64 and of 256 entries
@pytest.mark.parametrize("T", [5, 63, 64, 65, 128, 255, 257, 700])
@pytest.mark.parametrize("shape", ["nested", "queue", "late", "mixed"])
def test_streams(lap, oracle_mod, shape, T):
    rng = np.random.default_rng(T)
    k = np.arange(T // 2 if shape != "mixed" else T)
    if shape == "nested":                      # the first one out is the last one back
        lo, hi = k, T - 1 - k
    elif shape == "queue":                     # the first one out is the first one back, with others still leaving
        lo, hi = k, k + T // 2
    elif shape == "late":                      # back at the last step: swap-outs to the end
        lo, hi = k, np.full(len(k), T - 1)
    else:
        lo = rng.integers(0, T, len(k))
        hi = np.minimum(T - 1, lo + rng.integers(0, T, len(k)))
    keep = lo <= hi
    lo, hi = lo[keep], hi[keep]
    size = rng.integers(1, 60, len(lo)) * 1000
    # a one-step variable per step, so that steps ask for memory
    sizes = np.concatenate([size, rng.integers(1, 30, T) * 1000])
    al = np.concatenate([lo, np.arange(T)])
    fr = np.concatenate([hi + 1, np.arange(T) + 1])
    glo, ghi = np.concatenate([lo, np.arange(T)]), np.concatenate([hi, np.arange(T)])
    tr = mk_trace([int(x) for x in sizes], [int(x) for x in al], [int(x) for x in fr], T=T, gap_lo=[int(x) for x in glo],
                  gap_hi=[int(x) for x in ghi], step_ns=[int(x) for x in rng.integers(50, 400, T)])
    peak = max(sum(int(s) for s, a, f in zip(sizes, al, fr) if a <= t < f) for t in range(T))
    order = [int(x) for x in rng.permutation(len(lo))]
    runs = [(n, peak * q // 8) for n in (0, 1, len(lo) // 2, len(lo)) for q in range(9)]
    for link in (0.05, 0.5, 20.0):             # the streams are far behind, level, and ahead of the steps
        _check(lap, oracle_mod, tr, link, order, runs)
