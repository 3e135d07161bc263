"""GPU parity of lap_plan_pool in every form of its per-step-list and sweep kernel: four or eight waves per ordering
(more than 512 orderings or not), the per-step words in LDS or not (up to 800 steps or more), one launch for one policy
or for both, multi-step blocks in registers (up to 256 per wave) or in lists; and the same without per-step lists, on
traces too large for the register kernel.  Offsets and footprints against the oracle's."""
import numpy as np
import pytest

from gpu_util import oracle_all_orderings, u64
from traces import make_orderings, random_trace

pytestmark = pytest.mark.gpu

FITS = {"first": [0], "best": [1], "both": [0, 1]}


@pytest.fixture(scope="module")
def lap():
    import paper_1903_06631_amd as lap
    lap.load_library()
    return lap


def _check(lap, oracle, tr, B, fits):
    kinds, seeds = make_orderings(B)
    fits = [FITS[fits][b % len(FITS[fits])] for b in range(B)]
    got = lap.plan_pool(lap.DeviceTrace(tr), kinds, seeds, fits=fits)
    all_off, fps = u64(got["all_offsets"]), u64(got["footprints"])
    which = sorted({b for b in (0, 1, 2, 3, 4, 5, 255, 256, B - 2, B - 1) if b < B})
    for b, (_, off, fp) in oracle_all_orderings(oracle, tr, kinds, seeds, None, which, fits).items():
        assert np.array_equal(all_off[b], off), f"ordering {b}"
        assert fps[b] == fp, f"ordering {b}"
    assert np.array_equal(fps, (all_off + tr.size[None, :]).max(axis=1))
    best = int(got["best_ordering"].item())
    assert best == int(np.argmin(fps)) and np.array_equal(u64(got["best_offsets"]), all_off[best])


def _per_step(n, T, n_multi, max_life):
    """n_multi variables of 2 to max_life steps, one-step variables otherwise"""
    tr = random_trace(9500 + n_multi, n, T, size_choices=[1, 1, 2, 3, 5, 8, 13, 64], one_step_frac=1.0)
    rng = np.random.default_rng(n_multi)
    a = np.minimum(tr.alloc, T - max_life).astype(np.uint32)
    f = a + 1
    f[rng.permutation(n)[:n_multi]] += rng.integers(1, max_life, n_multi).astype(np.uint32)
    tr.alloc, tr.free, tr.gap_lo, tr.gap_hi = a, f, a.copy(), (f - 1).astype(np.uint32)
    assert int((f - a).sum()) + T <= 6 * n                   # per-step lists apply
    return tr


@pytest.mark.parametrize("fits", ["first", "best", "both"])
@pytest.mark.parametrize("B,n,T,n_multi", [(513, 4600, 800, 1024), (513, 4600, 800, 1025), (513, 4600, 801, 1024),
                                           (513, 4600, 801, 1025), (8, 6000, 800, 2048), (8, 6000, 800, 2049),
                                           (8, 6000, 801, 2048), (8, 6000, 801, 2049), (512, 4600, 800, 1025)])
def test_per_step_lists(lap, oracle_mod, B, n, T, n_multi, fits):
    _check(lap, oracle_mod, _per_step(n, T, n_multi, 14), B, fits)


# eight and four waves, the step words (which such traces do not have) with room in LDS and without, every policy
@pytest.mark.parametrize("B,T,fits", [(8, 3000, "best"), (8, 3000, "both"), (8, 700, "best"), (8, 700, "both"), (513, 3000, "first"),
                                      (513, 3000, "best"), (513, 3000, "both"), (513, 700, "both"), (513, 66000, "first")])
def test_sweep(lap, oracle_mod, B, T, fits):
    """one variable more than fits the registers, lifetimes that sum to more than per-step lists take, and no segment
    lists: the sweep's forms (first-fit orderings alone go to the batches up to 65 535 steps, and are swept beyond)"""
    tr = random_trace(9601, 32769, T, size_choices=[1, 2, 3, 7, 20, 50], max_life=40)
    assert int((tr.free - tr.alloc).sum()) > 6 * tr.n_vars
    lap.set_option(lap.OPT_SEG_MIN_VARS, 1 << 30)
    try:
        _check(lap, oracle_mod, tr, B, fits)
    finally:
        lap.set_option(lap.OPT_SEG_MIN_VARS, lap.SEG_MIN_VARS_DEFAULT)
