"""GPU parity of lap_plan_pool around the sizes where a plan's orders and its preparation change kernels: orders of up to
640 variables are found by counting, preparation of up to 4096 variables and 4096 steps is one launch.  Offsets,
footprints and orders are compared element by element with the oracle's."""
import numpy as np
import pytest

from gpu_util import oracle_all_orderings, u64
from traces import random_trace

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lap():
    import paper_1903_06631_amd as lap
    lap.load_library()
    return lap


def _check(lap, oracle, tr, B, want_all):
    rng = np.random.default_rng(B)
    kinds = rng.permutation(np.resize([lap.ORD_SIZE_DESC, lap.ORD_LIFE_DESC, lap.ORD_AREA_DESC, lap.ORD_ALLOC_ASC,
                                       lap.ORD_SEEDED, lap.ORD_CLASS_SEEDED], B)).astype(np.uint32)
    seeds = rng.integers(0, 1 << 62, B).astype(np.uint64)
    got = lap.plan_pool(lap.DeviceTrace(tr), kinds, seeds, want_all=want_all)
    fps, best = u64(got["footprints"]), int(got["best_ordering"].item())
    which = range(B) if B <= 16 else sorted({0, 1, 2, 3, B // 2, B - 1, best})
    ref = oracle_all_orderings(oracle, tr, kinds, seeds, None, which)
    for b, (_, off, fp) in ref.items():
        assert fps[b] == fp, f"ordering {b}"
        if want_all:
            assert np.array_equal(u64(got["all_offsets"])[b], off), f"ordering {b}"
    assert best == int(np.argmin(fps)) and int(u64(got["best_footprint"])[0]) == fps[best]
    if best in ref:
        assert np.array_equal(u64(got["best_offsets"]), ref[best][1])


# many equal sizes and lifetimes: ties are decided by the index
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 511, 512, 513, 639, 640, 641])
def test_orders_by_counting(lap, oracle_mod, n):
    _check(lap, oracle_mod, random_trace(9500 + n, n, 30, size_choices=[1, 2, 3, 7]), 12, True)


@pytest.mark.parametrize("n,T", [(40, 1), (300, 4096), (300, 4097), (4096, 50), (4097, 50), (4096, 4096)])
def test_preparation(lap, oracle_mod, n, T):
    _check(lap, oracle_mod, random_trace(9600 + n + T, n, T, size_choices=[1, 2, 3, 7, 20]), 6, True)


# 64-bit sizes leave the packed records out; one launch carries the descriptors of up to about a hundred orderings
@pytest.mark.parametrize("B,all_", [(1, False), (63, True), (64, False), (65, True), (112, False), (113, False), (300, True)])
def test_orderings(lap, oracle_mod, B, all_):
    _check(lap, oracle_mod, random_trace(9700, 90, 25), B, all_)
    _check(lap, oracle_mod, random_trace(9701, 90, 25, size_choices=[1, 3 << 31, 5 << 33]), B, all_)
