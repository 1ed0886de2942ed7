"""The 8-bit copy gives way: searches and loads that run out of memory take it back and
return what they return without it.  SIEVE_COPY_ALLOC_CAP refuses allocations while there is
a copy to take, SIEVE_ALLOC_CAP every one above it."""
import pytest

torch = pytest.importorskip("torch")

from test_gpu_screen import SIZES, _index, _same, _screened, knobs  # noqa: E402

pytestmark = pytest.mark.gpu


def _queries(v, ids, step):
    sel = torch.arange(0, len(v), step).cuda()
    return v[sel].contiguous(), ids[sel].contiguous()


def _exact(ix, q, ex, **kw):
    with knobs(SIEVE_SCREEN=0):
        return ix.search(q, ex, 4, kw.pop("tau", 0.9), kw.pop("W", 2), len(SIZES), **kw)


def _screens(ix, q, ex):
    with knobs(SIEVE_SCREEN=2):
        ix.search(q, ex, 4, 0.9, 2, len(SIZES), with_stats=True)
    return all(_screened(ix))


def test_copy_lost_before_the_first_round():
    ix, v, ids = _index(128, torch.float16, 1)
    q, ex = _queries(v, ids, 3)
    with knobs(SIEVE_SCREEN=2, SIEVE_COPY_ALLOC_CAP=1):
        got = ix.search(q, ex, 4, 0.9, 2, len(SIZES), with_stats=True)
    assert not any(_screened(ix))
    _same(got[:3], _exact(ix, q, ex))
    assert not _screens(ix, q, ex)  # it does not come back
    fx = ix.search_fixed(q, ex, 4, 0.9, len(SIZES))
    with knobs(SIEVE_SCREEN=0):
        _same(fx, ix.search_fixed(q, ex, 4, 0.9, len(SIZES)))


@pytest.mark.parametrize("lookahead", [True, False])
def test_copy_lost_between_rounds(lookahead):
    # two ranks ordered up front: queries whose stop line passes them need the rank
    # extension's buffers after a round, and those take the copy
    ix, v, ids = _index(128, torch.float16, 2)
    q, ex = _queries(v, ids, 3)
    kw = dict(lookahead=lookahead, with_stats=True)
    n = len(SIZES)
    with knobs(SIEVE_SCREEN=2, SIEVE_RANK_PREFIX=2):
        ix.search(q, ex, 4, float("inf"), 1, n, **kw)  # no hits, no extension
        assert all(_screened(ix))
        with knobs(SIEVE_COPY_ALLOC_CAP=1):
            got = ix.search(q, ex, 4, -2.0, 1, n, **kw)
    rounds = _screened(ix)
    assert rounds[0] and not rounds[-1] and rounds == sorted(rounds, reverse=True)
    _same(got[:3], _exact(ix, q, ex, tau=-2.0, W=1, lookahead=lookahead))


def test_queries_copy_does_not_fit():
    # 15 MB of 8-bit queries above a cap that every other buffer of the call stays below
    ix, v, ids = _index(768, torch.float16, 3)
    sel = torch.randint(len(v), (20000,), generator=torch.Generator().manual_seed(1)).cuda()
    q, ex = v[sel].contiguous(), ids[sel].contiguous()
    few = q[:50].contiguous(), ex[:50].contiguous()
    assert _screens(ix, *few)
    with knobs(SIEVE_SCREEN=2, SIEVE_ALLOC_CAP=4 << 20):
        got = ix.search(q, ex, 4, 0.9, 2, len(SIZES), with_stats=True)
    assert not any(_screened(ix))
    _same(got[:3], _exact(ix, q, ex))
    assert _screens(ix, *few)  # the index keeps its copy for searches that fit


def test_load_and_search_take_idle_copies():
    import paper_2608_03199_amd as ps
    a, va, ia = _index(128, torch.float16, 4)
    qa, ea = _queries(va, ia, 5)
    assert _screens(a, qa, ea)
    with knobs(SIEVE_COPY_ALLOC_CAP=1):
        b, vb, ib = _index(96, torch.float32, 5)  # the load takes a's copy
    assert not _screens(a, qa, ea)
    qb, eb = _queries(vb, ib, 5)
    c, vc, ic = _index(64, torch.float16, 6)
    assert _screens(c, *_queries(vc, ic, 50))
    with knobs(SIEVE_SCREEN=2, SIEVE_COPY_ALLOC_CAP=1):
        got = b.search(qb, eb, 4, 0.9, 2, len(SIZES))  # b's workspace takes b's, then c's
    _same(got, _exact(b, qb, eb))
    assert not _screens(b, qb, eb) and not _screens(c, *_queries(vc, ic, 50))
    # shards of one call: the second's workspace takes the first's copy
    d, vd, idd = _index(128, torch.float16, 7)
    e, _, _ = _index(128, torch.float16, 8)
    q, ex = _queries(vd, idd, 5)
    with knobs(SIEVE_SCREEN=0):
        want = ps.search_multi([d, e], q, ex, 4, 0.9, 2, len(SIZES))
    f, vf, idf = _index(128, torch.float16, 7)
    g, _, _ = _index(128, torch.float16, 8)
    with knobs(SIEVE_SCREEN=2, SIEVE_COPY_ALLOC_CAP=1):
        _same(ps.search_multi([f, g], q, ex, 4, 0.9, 2, len(SIZES)), want)


def test_copy_declined_at_load():
    with knobs(SIEVE_SCREEN=0):
        ix, v, ids = _index(128, torch.float16, 9)
    q, ex = _queries(v, ids, 5)
    assert not _screens(ix, q, ex)
    ref, _, _ = _index(128, torch.float16, 9)
    assert _screens(ref, q, ex)
    _same(ix.search(q, ex, 4, 0.9, 2, len(SIZES)), ref.search(q, ex, 4, 0.9, 2, len(SIZES)))


def test_calibrated_call_loses_the_copy():
    ix, v, ids = _index(128, torch.float16, 10)
    q, ex = _queries(v, ids, 3)
    smp = torch.arange(0, len(q), 9, dtype=torch.int32).cuda()
    with knobs(SIEVE_SCREEN=0):
        ref, _, _ = _index(128, torch.float16, 10)
    want = ref.search_calibrated(q, ex, 4, 0.9, len(SIZES), smp, 0.01)
    with knobs(SIEVE_SCREEN=2, SIEVE_COPY_ALLOC_CAP=1):
        got = ix.search_calibrated(q, ex, 4, 0.9, len(SIZES), smp, 0.01)
    _same(got[:3], want[:3])
    assert got[3] == want[3]
