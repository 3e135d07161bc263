"""GPU parity: lap_simulate_swaps against the oracle's discrete-event run, value by value."""
import numpy as np
import pytest

from gpu_util import u64
from helpers import mk_trace, read_golden
from traces import make_config, random_trace

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lap():
    import paper_1903_06631_amd as lap
    lap.load_library()
    return lap


def _check(lap, oracle, tr, link, sl, runs, use_gaps=True):
    """runs: list of (prefix length, limit)"""
    import torch
    dt = lap.DeviceTrace(tr, use_gaps=use_gaps)
    lst = torch.from_numpy(np.asarray(sl, dtype=np.uint32).view(np.int32)).to(dt.device)
    got = lap.simulate_swaps(dt, link, lst, [r[0] for r in runs], [r[1] for r in runs])
    tot, ovh, pk = u64(got["total_ns"]), u64(got["overhead_ns"]), u64(got["peak_resident"])
    forced = got["forced"].cpu().numpy().view(np.uint32)
    refs = []
    for q, (k, lim) in enumerate(runs):
        ref = oracle.simulate_swaps(tr, link, list(sl[:k]), lim, use_gaps=use_gaps)
        mine = (int(tot[q]), int(ovh[q]), int(pk[q]), int(forced[q]))
        assert mine == (ref["total_ns"], ref["overhead_ns"], ref["peak_resident"], ref["forced"]), (q, k, lim)
        refs.append(ref)
    return refs


def test_simulate_golden(lap, oracle_mod):
    g = read_golden("e5_schedule.txt")
    ints = lambda r: [int(x) for x in r]
    tr = mk_trace(g["size"][0], g["alloc"][0], g["free"][0], T=10, gap_lo=ints(g["gap_lo"][0]),
                  gap_hi=ints(g["gap_hi"][0]), step_ns=[100] * 10)
    sl = ints(g["swap_list"][0])
    refs = _check(lap, oracle_mod, tr, 1.0, sl, [(3, 10 ** 9), (3, 620), (3, 560), (3, 520), (3, 499), (3, 100),
                                                 (0, 829), (0, 830), (1, 560), (2, 520)])
    assert [r["total_ns"] for r in refs[:4]] == [1000, 1000, 1030, 1060]


def test_simulate_golden_listed_variable_without_idle_gap(lap, oracle_mod):
    g = read_golden("e6_simulate.txt")
    ints = lambda key: [int(x) for x in g[key][0]]
    tr = mk_trace(ints("nogap_size"), ints("nogap_alloc"), ints("nogap_free"), T=10, gap_lo=ints("nogap_gap_lo"),
                  gap_hi=ints("nogap_gap_hi"), step_ns=[100] * 10)
    refs = _check(lap, oracle_mod, tr, 1.0, ints("nogap_swap_list"), [(4, lim) for lim in ints("nogap_limits")])
    assert [r["total_ns"] for r in refs] == ints("nogap_total_ns")
    assert [r["peak_resident"] for r in refs] == ints("nogap_peak_resident")


@pytest.mark.parametrize("seed,n,T", [(0, 1, 1), (1, 30, 9), (2, 400, 25), (3, 3000, 120), (4, 12000, 700)])
def test_simulate_random(lap, oracle_mod, seed, n, T):
    tr = random_trace(1900 + seed, n, T, with_step_ns=(seed % 2 == 0))
    rng = np.random.default_rng(seed)
    cand = np.nonzero(tr.gap_hi > tr.gap_lo)[0]
    sl = rng.permutation(n)[: max(1, n * 2 // 3)].astype(np.uint32)      # includes variables without a gap
    _, peak, _ = oracle_mod.load_profile(tr)
    for link in (0.004, 1.0, 64.0):
        runs = [(len(sl), 10 ** 15), (len(sl), peak), (len(sl), peak * 3 // 4), (len(sl) // 2, peak // 2),
                (len(sl) // 3, peak * 9 // 10), (0, peak), (0, peak - 1), (len(sl), 0), (1, peak // 3)]
        _check(lap, oracle_mod, tr, link, sl, runs)
    _check(lap, oracle_mod, tr, 1.0, sl, [(len(sl), peak * 2 // 3)], use_gaps=False)


@pytest.mark.parametrize("n,T", [(12, 20), (300, 40), (1500, 100)])
def test_simulate_transfers_whose_times_do_not_fit_64_bits(lap, oracle_mod, n, T):
    """sizes near the largest legal ones over the slowest links: the planned starts wrap around, as the oracle's do"""
    rng = np.random.default_rng(n)
    a = rng.integers(0, T - 4, n)
    f = a + 3 + rng.integers(0, T - a - 2)
    size = rng.integers(1 << 49, 1 << 52, n).astype(np.uint64)
    tr = mk_trace(size, a, f, T=T, step_ns=rng.integers(1, 1 << 40, T))
    assert oracle_mod.validate_trace(tr) == 0
    _, peak, _ = oracle_mod.load_profile(tr)
    sl = rng.permutation(n).astype(np.uint32)
    for link in (0.001, 0.002, 0.05, 64.0):
        _check(lap, oracle_mod, tr, link, sl, [(k, lim) for k in (n, n // 2, 9, 1) for lim in (peak, peak * 3 // 5, peak // 4)])


@pytest.mark.parametrize("wide", [False, True])
@pytest.mark.parametrize("n,T", [(600, 255), (600, 256), (601, 257), (4000, 513), (8193, 40)])
def test_simulate_window_edges(lap, oracle_mod, n, T, wide):
    """steps and transfers are fetched 256 at a time, swap-in starts scanned 512 at a time, job lists built 8192 at a time;
    by the machine of 31-bit numbers, and by the one of 64-bit numbers that a step of 2^31 ns and more needs"""
    tr = random_trace(2300 + n + T, n, T, with_step_ns=True)
    assert int(tr.step_ns.max()) < 1 << 31
    if wide:
        tr.step_ns[T // 2] = (1 << 31) + 12345
    _, peak, _ = oracle_mod.load_profile(tr)
    with_gap = np.nonzero(tr.gap_hi > tr.gap_lo)[0]
    sl = np.random.default_rng(n).permutation(with_gap).astype(np.uint32)
    ks = sorted({min(k, len(sl)) for k in (1, 255, 256, 257, 511, 512, 513, len(sl) - 1, len(sl))})
    _check(lap, oracle_mod, tr, 2.0, sl, [(k, lim) for k in ks for lim in (peak, peak * 3 // 5, 0)])


@pytest.mark.parametrize("k", [63, 65, 1025, 16384, 16385])
def test_simulate_list_lengths(lap, oracle_mod, k):
    """ordered by counting up to 16 384 variables, beyond by the sort of all variables"""
    tr = random_trace(4200, 16500, 200, with_step_ns=True)
    _, peak, _ = oracle_mod.load_profile(tr)
    sl = np.random.default_rng(k).permutation(16500)[:k].astype(np.uint32)
    _check(lap, oracle_mod, tr, 3.0, sl, [(k, peak), (k, peak // 2), (k * 2 // 3, peak // 3), (k, 0), (0, peak)])


EDGE = (1 << 31) - 1


@pytest.mark.parametrize("what", ["step", "transfer", "resident"])
@pytest.mark.parametrize("edge", [EDGE - 1, EDGE, EDGE + 1, EDGE + 2])
@pytest.mark.parametrize("granule", [1, 512])
def test_simulate_on_both_sides_of_31_bits(lap, oracle_mod, what, edge, granule):
    """the longest step, the longest transfer and the bytes resident (in granules) where 31 bits end, each with 70
    transfers, steps that allocate nothing and limits that block every step"""
    rng = np.random.default_rng(edge * 3 + granule)
    n, T, link = 100, 90, 1.0                                   # 1 GB/s: a byte takes 1 ns
    a = np.sort(rng.integers(0, T // 3, n) * 2)
    f = a + 8 + rng.integers(0, T - a - 8)
    size = rng.integers(1, 1 << 20, n).astype(np.uint64) * granule
    step_ns = rng.integers(1, 1 << 21, T).astype(np.uint64)
    if what == "step":
        step_ns[T // 2] = edge
    else:
        # variable 0: alone beyond the edge as a transfer, or up to the peak; its granule is the trace's
        a[0], f[0] = 0, T
        size[0] = edge if what == "transfer" else granule
        if what == "resident":
            peak = oracle_mod.load_profile(mk_trace(size, a, f, T=T))[1]
            size[0] = granule * edge - (peak - granule)
    tr = mk_trace(size, a, f, T=T, gap_lo=a, gap_hi=f - 1, step_ns=step_ns)
    peak = oracle_mod.load_profile(tr)[1]
    assert what != "resident" or peak == granule * edge
    sl = np.concatenate([[0], 1 + rng.permutation(n - 1)[:70]]).astype(np.uint32)
    _check(lap, oracle_mod, tr, link, sl, [(71, 0), (71, peak // 2), (71, peak - 1), (71, peak), (64, peak * 3 // 4), (1, peak // 3),
                                           (0, 0), (71, (1 << 64) - 1)])


@pytest.mark.parametrize("cfg", [2, 3, 5])
def test_simulate_limit_sweep_on_configs(lap, oracle_mod, cfg):
    """what the planner is for: the selection's prefixes for a sweep of limits, each replayed under its limit"""
    tr = make_config(cfg)
    link, mb = tr.meta["link_GBps"], tr.meta["min_bytes"]
    _, peak, _ = oracle_mod.load_profile(tr)
    limits = [peak * q // 10 for q in range(3, 11)]
    sel = oracle_mod.select_swaps(tr, link, mb, 3, limits)
    runs = [(int(sel["n_selected"][q]), limits[q]) for q in range(len(limits))]
    refs = _check(lap, oracle_mod, tr, link, sel["order"], runs)
    assert refs[-1]["overhead_ns"] == 0 and refs[-1]["forced"] == 0          # limit = peak, nothing swapped


def test_simulate_argument_errors(lap):
    import torch
    tr = random_trace(1, 100, 10)
    dt = lap.DeviceTrace(tr)
    lst = torch.arange(4, dtype=torch.int32, device="cuda")
    with pytest.raises(lap.LapError) as e:
        lap.simulate_swaps(dt, 1.0, lst, [5], [100])
    assert e.value.status == -2
    with pytest.raises(lap.LapError) as e:
        lap.simulate_swaps(dt, float("nan"), lst, [4], [100])
    assert e.value.status == -5
