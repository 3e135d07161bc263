"""GPU parity of lap_detect_iteration on lists whose end is found again at many distances: short repeats, runs of one token that
are shorter than the iteration asked for, layers, and repeats that differ in their first token only; around the list size that
one workgroup takes and around the tokens that are compared before all of a distance is."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lap():
    import paper_1903_06631_amd as lap
    lap.load_library()
    return lap


def _tail(rng, m, tail):
    head = rng.integers(0, 300, max(m - len(tail), 0)).astype(np.uint64)
    return np.concatenate([head, np.asarray(tail, np.uint64)])[-m:]


def _lists(rng, m):
    word = lambda n: rng.integers(0, 300, n)
    run = m // 2
    yield "one token", np.full(m, 7, np.uint64), (1, 64, m // 3, m // 2, m // 2 + 1)
    yield "run", _tail(rng, m, np.full(run, 7)), (1, run // 2, run // 2 + 1, run - 40, run)
    yield "short period", _tail(rng, m, np.tile(word(12), run // 12)), (5, 64, 1057, run // 2 - 6, run // 2 + 12)
    block = word(max(m // 40, 3))
    yield "layers", _tail(rng, m, np.tile(np.concatenate([word(m // 30)] + [block] * 9), 2)), (1, 64, m // 30, m // 5, m // 3)
    for p in (31, 32, 33, 1055, 1056, 1057, m // 2):         # equal but for one token: the first, one in the middle, none
        half = word(p)
        for at in (0, p // 2, None):
            other = half.copy()
            if at is not None:
                other[at] += 1000
            if 2 * p <= m:
                yield f"two halves of {p}", _tail(rng, m, np.concatenate([other, half])), (1, p, p + 1)


@pytest.mark.parametrize("m", [2000, 6144, 6145, 9000, 33001])
def test_many_distances(lap, oracle_mod, m):
    import torch
    rng = np.random.default_rng(m)
    for what, s, periods in _lists(rng, m):
        t = torch.from_numpy(s.view(np.int64)).cuda()
        for mp in periods:
            if mp >= 1:
                assert int(lap.detect_iteration(t, mp).item()) == oracle_mod.detect_iteration(s, mp), (what, mp)


def test_scratch_of_an_earlier_call_does_not_matter(lap, oracle_mod):
    """the same scratch for a list that comes to the hashes and for one that does not, in turn"""
    import torch
    rng = np.random.default_rng(1)
    m = 20000
    run = _tail(rng, m, np.full(m // 2, 7))
    it = rng.integers(0, 300, m // 3).astype(np.uint64)
    plain = _tail(rng, m, np.concatenate([it, it]))
    for s, mp in [(run, m // 4 + 1), (plain, 64), (run, m // 4 + 1), (run, 3), (plain, 64), (plain, m // 3 + 1)]:
        t = torch.from_numpy(s.view(np.int64)).cuda()
        assert int(lap.detect_iteration(t, mp).item()) == oracle_mod.detect_iteration(s, mp)


def _marked(rng, m, period, at, again):
    """a list of a short period but for one token `at` places from the end, and another one like it `again` places before that:
    every multiple of the period above at / 2 differs in that one token, `again` excepted"""
    s = np.tile(rng.integers(0, 300, period), m // period + 1)[:m].astype(np.uint64)
    s[m - at] += 1000
    if again:
        s[m - at - again] += 1000
    return s


def _check(lap, s, min_period, want, cut):
    import torch
    t = torch.empty(len(s) + cut, dtype=torch.int64, device="cuda")[cut:]
    t.copy_(torch.from_numpy(s.astype(np.int64)))
    assert t.data_ptr() % 16 == 8 * cut
    for _ in range(3):
        assert int(lap.detect_iteration(t, min_period).item()) == want


# more distances remain than are compared directly, and where these differ the others do, one excepted or none; in the one
# workgroup and in all, and where the list starts between two 16-byte words.  The answers are known by construction: the oracle
# compares every multiple.
@pytest.mark.parametrize("m", [2000, 6000, 6144, 6145, 70001, 2000003])
@pytest.mark.parametrize("cut", [0, 1])
def test_lists_with_odd_tokens(lap, oracle_mod, m, cut):
    rng = np.random.default_rng(m)
    period, at = 7, m // 8 if m > 9000 else 1100 if m > 6144 else 100
    again = m // 3 // period * period
    for second, want in ((0, 0), (again, again)):
        s = _marked(rng, m, period, at, second)
        if m < 9000:
            assert oracle_mod.detect_iteration(s, at // 2 + 1) == want
        _check(lap, s, at // 2 + 1, want, cut)


def _fibonacci(m):
    a, b = [1], [1, 2]
    while len(b) < m:
        a, b = b, b + a
    return np.asarray(b[-m:])


def _reference(s, min_period):
    """every distance that is left out was shown to differ somewhere, and what is returned was compared in full"""
    m = len(s)
    p = np.arange(min_period, m // 2 + 1)
    while len(p):
        c = int(p[0])
        differs = np.nonzero(s[m - 2 * c:m - c] != s[m - c:])[0]
        if len(differs) == 0:
            return c
        p = p[1:]
        for w in (m - c + int(differs[-1]), m - 2 * c + int(differs[-1])):
            last, first = w >= m - p, (w < m - p) & (w >= m - 2 * p)
            p = p[~((last & (s[w] != s[np.maximum(w - p, 0)])) | (first & (s[w] != s[np.minimum(w + p, m - 1)])))]
    return 0


# a word in which distances differ in few places, other ones every time, so that it comes to the hashes: with tiles of 1024
# tokens and the first larger ones (beyond 1024 * 1024 tokens), with as many workgroups as there are compute units
@pytest.mark.parametrize("m,min_period", [(6144, 1200), (70001, 17500), (1 << 20, 262144), ((1 << 20) + 1, 262144), (2000003, 666667)])
@pytest.mark.parametrize("cut", [0, 1])
def test_lists_that_come_to_the_hashes(lap, oracle_mod, m, min_period, cut):
    s = _fibonacci(m)
    want = _reference(s, min_period)
    if m < 9000:
        assert oracle_mod.detect_iteration(s.astype(np.uint64), min_period) == want
    _check(lap, s, min_period, want, cut)


def test_time_of_lists_that_end_in_a_run(lap):
    """iterations that end in a run shorter than themselves take no longer than others (measured: 1.0 times; 5.7 times where every
    distance inside the run went on to the hashes)"""
    import time
    import torch
    rng = np.random.default_rng(5)
    m = 200000
    word = lambda n: rng.integers(0, 300, n)
    plain, run = word(m // 3), np.concatenate([word(m // 3 - m // 10), np.full(m // 10, 7)])

    def us(it):
        t = torch.from_numpy(_tail(rng, m, np.concatenate([it, it])).view(np.int64)).cuda()
        assert int(lap.detect_iteration(t, m // 15).item()) == len(it)
        best = float("inf")
        for _ in range(8):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(100):
                lap.detect_iteration(t, m // 15, sync=False)
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - t0) * 1e4)
        return best

    a, b = us(plain), us(run)
    print(f"plain {a:.1f} us, ending in a run {b:.1f} us")
    assert b < 2 * a
