"""The ranking's selection from materialised scores (prefixes of few centroids, long prefixes of
many) against the fp64 order (exact, no tolerance), where its bound on the n-th score is loose."""
import contextlib
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


@contextlib.contextmanager
def screen_path():
    os.environ["SIEVE_RANK_PATH"] = "1"
    try:
        yield
    finally:
        del os.environ["SIEVE_RANK_PATH"]


def _index(C):
    import paper_2608_03199_amd as ps
    nlist = len(C)
    cu = lambda x: torch.tensor(x).cuda()  # noqa: E731
    return ps.Index(cu(C[:1]), cu(np.append(np.zeros(nlist, np.int64), 1)),
                    cu(np.zeros(1, np.int64)), cu(C))


def _order(Q, C, n):
    s = np.zeros((len(Q), len(C)))
    for t in range(C.shape[1]):  # the dimension-ordered fp64 sum
        s += Q[:, t:t + 1].astype(np.float64) * C[:, t].astype(np.float64)
    return np.argsort(-s, axis=1, kind="stable")[:, :n]


# the wave kernel's register counts (4, 8 and 16 keys a lane, at their edges) and the block
# kernel's (16, 32); n up to and past the ranks that the lane maxima bound
@pytest.mark.parametrize("dtype", [np.float32, np.float16])
@pytest.mark.parametrize("n", [1, 40, 41, 63])
@pytest.mark.parametrize("nlist", [63, 64, 256, 257, 300, 512, 513, 1024, 1025, 4097])
def test_selection_sizes(nlist, n, dtype):
    d = 72
    g = np.random.default_rng(nlist + n)
    C = g.standard_normal((nlist, d))
    C = (C / np.linalg.norm(C, axis=1, keepdims=True)).astype(dtype)
    C[nlist // 2:nlist // 2 + 9] = C[1]  # ties to the lower index
    Q = C[g.integers(0, nlist, 9)]
    with screen_path():
        P = _index(C).rank(torch.tensor(Q).cuda(), n).cpu().numpy()
    assert np.array_equal(P, _order(Q, C, n))


def _scored(scores, d=64):
    """One query and centroids whose products with it are `scores` (exact in fp32)."""
    C = np.zeros((len(scores), d), np.float32)
    C[:, 0] = scores
    Q = np.zeros((1, d), np.float32)
    Q[0, 0] = 1.0
    return Q, C


# large scores on few lanes (centroid c is held by lane c % 64): the n-th lane maximum lies
# under far more than n scores
@pytest.mark.parametrize("nlist", [300, 500, 1000])
def test_large_scores_on_few_lanes(nlist):
    g = np.random.default_rng(7)
    s = g.uniform(-0.5, 0.4, nlist)
    crowd = np.arange(nlist)[np.arange(nlist) % 64 < nlist // 100 + 4]
    s[crowd] = g.uniform(0.5, 1.0, len(crowd))
    Q, C = _scored(s.astype(np.float32))
    with screen_path():
        P = _index(C).rank(torch.tensor(Q).cuda(), 32).cpu().numpy()
    assert np.array_equal(P, _order(Q, C, 32))


# near-ties under a loose bound, fewer and more than the candidate buffer holds (n + 141 places
# of a wave, n + 525 of a block): 0.75 is where the search by bits stops, the ties lie just under
@pytest.mark.parametrize("nlist,ties,n", [(300, 120, 44), (300, 160, 44), (1000, 160, 44),
                                          (3000, 490, 44), (3000, 560, 44)])
def test_near_ties_under_the_loose_bound(nlist, ties, n):
    g = np.random.default_rng(11)
    s = g.uniform(-0.5, 0.4, nlist)
    at = g.permutation(nlist)
    s[at[:n]] = g.uniform(0.8, 0.99, n)
    s[at[n:n + ties]] = 0.75 - 1e-6 * g.integers(1, 5, ties)
    Q, C = _scored(s.astype(np.float32))
    ix = _index(C)
    with screen_path():
        P = ix.rank(torch.tensor(Q).cuda(), n).cpu().numpy()
        assert np.array_equal(P, _order(Q, C, n))
        P = ix.rank(torch.tensor(Q).cuda(), n + 4).cpu().numpy()  # the boundary among the ties
        assert np.array_equal(P, _order(Q, C, n + 4))


# a query with inf or NaN: the order of the scores as they are (+inf before -inf), ties and NaN
# by index, as the wide selection gives it
@pytest.mark.parametrize("nlist", [100, 500, 2000])
@pytest.mark.parametrize("value", [np.inf, np.nan])
def test_queries_that_are_not_finite(value, nlist):
    pos = np.arange(nlist) % 10 < 6
    Q, C = _scored(np.where(pos, 0.5, -0.5).astype(np.float32))
    Q[0, 0] = value
    want = np.argsort(~pos, kind="stable") if value == np.inf else np.arange(nlist)
    ix = _index(C)
    for n in (10, 41, nlist * 56 // 100, nlist * 61 // 100, nlist):
        with screen_path():
            P = ix.rank(torch.tensor(Q).cuda(), n).cpu().numpy()
        assert np.array_equal(P[0], want[:n])
