"""The screened scan (8-bit bound, exact scores of what passes) against the exact scan.

SIEVE_SCREEN=2 takes every scan through the screen, 0 none; the round log shows which copy
each round read.  Both score a pair with the same MFMA sequence, so ids, probe counts and
scores agree bit for bit (no tolerance)."""
import contextlib
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

SIZES = [0, 1, 15, 16, 17, 300, 2100, 64, 33, 5, 1025, 48]  # ragged partitions


@contextlib.contextmanager
def knobs(**kv):
    old = {k: os.environ.get(k) for k in kv}
    os.environ.update({k: str(v) for k, v in kv.items()})
    try:
        yield
    finally:
        for k, v in old.items():
            os.environ.pop(k, None)
            if v is not None:
                os.environ[k] = v


def _index(d, dtype, seed, edit=None):
    import paper_2608_03199_amd as ps
    g = np.random.default_rng(seed)
    cent = g.standard_normal((len(SIZES), d))
    cent /= np.linalg.norm(cent, axis=1, keepdims=True)
    rows = []
    for c, m in zip(cent, SIZES):
        x = c + 0.5 * g.standard_normal((m, d)) / np.sqrt(d)
        for i in range(1, m, 3):  # near duplicates of the row before
            x[i] = x[i - 1] + 0.2 * g.standard_normal(d) / np.sqrt(d)
        rows.append(x / np.linalg.norm(x, axis=1, keepdims=True))
    v = np.concatenate(rows)
    if edit is not None:
        v = edit(v)
    v = torch.tensor(v).to(dtype).cuda()
    off = torch.tensor(np.concatenate([[0], np.cumsum(SIZES)]), dtype=torch.int64).cuda()
    ids = torch.tensor(g.permutation(len(v)).astype(np.int64)).cuda()
    return ps.Index(v, off, ids, torch.tensor(cent).to(dtype).cuda()), v, ids


def _calls(ix, q, ex, k, tau):
    n = len(SIZES)
    yield "search", lambda **s: ix.search(q, ex, k, tau, 2, n, **s)
    yield "basic", lambda **s: ix.search(q, ex, k, tau, 2, n, lookahead=False, **s)
    yield "speculative", lambda **s: ix.search(q, ex, k, tau, 2, n, speculative=True, **s)
    yield "fixed", lambda **s: ix.search_fixed(q, ex, k, tau, n, **s)


def _same(a, b, name=""):
    for x, y in zip(a, b):
        assert torch.equal(x.view(torch.int32) if x.dtype == torch.float32 else x,
                           y.view(torch.int32) if y.dtype == torch.float32 else y), name


def _screened(ix):
    """For each round of the last call with statistics, whether it read the 8-bit rows: a
    round's bytes are list_rows rows, and per item one row and an 8-byte record, and 16 bytes
    per candidate."""
    out = []
    for r in ix.round_log():
        row = (r.scan_bytes - 8 * r.items - 16 * r.candidates) / (r.list_rows + r.items)
        exact = ix.d * (2 if ix.dtype == torch.float16 else 4)
        out.append(row != exact)
        assert row == exact or row in [64 * c for c in (1, 2, 3, 4, 6, 8, 12, 16)]
    return out


def _check(ix, q, ex, k, tau, **env):
    for name, call in _calls(ix, q, ex, k, tau):
        with knobs(SIEVE_SCREEN=0, **env):
            a = call()
            call(with_stats=True)
        assert not any(_screened(ix)), name
        with knobs(SIEVE_SCREEN=2, **env):
            b = call()
            c = call(with_stats=True)
        assert all(x == (ix.d <= 1024) for x in _screened(ix)), name
        torch.cuda.synchronize()
        _same(a, b, name)
        _same(a, c, name)


# chunk edges of the 8-bit rows (64 dimensions), each compiled chunk count, partial 16- and
# 32-dimension segments, and a dimension past the screen's largest (1,024: the exact scan)
@pytest.mark.parametrize("dtype", ["f32", "f16"])
@pytest.mark.parametrize("d", [8, 64, 72, 96, 128, 136, 192, 256, 264, 384, 512, 520, 768, 776,
                               1024, 1032])
def test_screen_equals_exact_scan(d, dtype):
    ix, v, ids = _index(d, torch.float32 if dtype == "f32" else torch.float16, d)
    sel = torch.randperm(len(v), generator=torch.Generator().manual_seed(d))[:333].cuda()
    _check(ix, v[sel].contiguous(), ids[sel].contiguous(), 4, 0.9)
    _check(ix, v[sel[:1]].contiguous(), None, 64, 0.5)  # one query, no exclusion, largest k


# every pair passes the screen: its LDS arena fills inside a tile (the stream resumes), moves
# to the global part, and past that the exact top-k pass takes the queries
@pytest.mark.parametrize("spill", [16384, 512, 0])
@pytest.mark.parametrize("d,dtype", [(128, "f16"), (64, "f32"), (200, "f16"), (768, "f16")])
def test_screen_flood(d, dtype, spill):
    ix, v, ids = _index(d, torch.float32 if dtype == "f32" else torch.float16, 3)
    sel = torch.arange(0, len(v), 13).cuda()
    _check(ix, v[sel].contiguous(), ids[sel].contiguous(), 3, -2.0, SIEVE_SPILL_CAP=spill)


def _non_finite(v):
    v = v.copy()
    v[40, 3], v[500, 0], v[501, 5], v[2600, 1] = np.nan, np.inf, -np.inf, np.inf
    return v


def _scaled(v):  # norms over many powers of ten, zero rows
    v = v * np.logspace(-20, 17, len(v))[:, None]
    v[::97] = 0
    return v


def _outlier(v):  # one large coordinate coarsens its list's scale
    v = v.copy()
    v[700, 2] = 60.0
    return v


@pytest.mark.parametrize("edit,dtype,tau", [
    (_non_finite, "f32", 0.9), (_non_finite, "f16", 0.9), (_scaled, "f32", 1e-3),
    (_scaled, "f32", 1e25), (_scaled, "f32", 0.0), (_outlier, "f16", 0.9),
    (_outlier, "f32", float("inf")), (_outlier, "f32", float("-inf"))])
def test_screen_unusual_values(edit, dtype, tau):
    ix, v, ids = _index(96, torch.float32 if dtype == "f32" else torch.float16, 5, edit)
    sel = torch.arange(0, len(v), 7).cuda()
    _check(ix, v[sel].contiguous(), ids[sel].contiguous(), 5, tau)


# Norms whose products leave fp32: a pair with a small negative product scores 0 (or -0) and
# reaches tau = 0, whatever its integer product says.
@pytest.mark.parametrize("scale", [1e-24, 1e-21, 1e-19])
def test_screen_underflowing_products(scale):
    ix, v, ids = _index(96, torch.float32, 5, lambda x: x * scale)
    sel = torch.arange(0, len(v), 11).cuda()
    q = torch.cat([v[sel], -v[sel], v[sel].flip(1)]).contiguous()
    _check(ix, q, ids[sel].repeat(3).contiguous(), 5, 0.0)
    _check(ix, q, ids[sel].repeat(3).contiguous(), 64, scale * scale / 2)


# The default setting: which rounds are screened is a rule on the data, the outputs are not.
def _grouped(n_lists, per, d, group, seed):
    """Lists of `per` rows, the first `group` of each near duplicates of one another."""
    import paper_2608_03199_amd as ps
    g = torch.Generator().manual_seed(seed)
    c = torch.nn.functional.normalize(torch.randn(n_lists, d, generator=g), dim=1)
    v = torch.nn.functional.normalize(
        c[:, None] + 2.0 * torch.randn(n_lists, per, d, generator=g) / d ** 0.5, dim=2)
    if group > 1:
        v[:, 1:group] = torch.nn.functional.normalize(
            v[:, :1] + 0.05 * torch.randn(n_lists, group - 1, d, generator=g) / d ** 0.5, dim=2)
        v = torch.stack([x[torch.randperm(per, generator=g)] for x in v])
    v = v.reshape(-1, d).half().cuda()
    off = torch.arange(0, n_lists * per + 1, per).cuda()
    ids = torch.arange(len(v)).cuda()
    return ps.Index(v, off, ids, c.half().cuda()), v, ids


def test_default_screens_no_crowded_first_round():
    # 1/9 of a list's row pairs are near duplicates: exact; 1/40: the first round exact, the
    # rest screened (rows from memory); none: all rounds screened
    seen = {}
    for group in (100, 40, 1):
        ix, v, ids = _grouped(1024, 300, 128, group, group)
        sel = torch.arange(0, len(v), 37).cuda()
        q, ex = v[sel].contiguous(), ids[sel].contiguous()
        got = ix.search(q, ex, 10, 0.9, 2, 64, with_stats=True)
        seen[group] = _screened(ix)
        with knobs(SIEVE_SCREEN=0):
            _same(got[:3], ix.search(q, ex, 10, 0.9, 2, 64))
        ix.close()
    assert not any(seen[100])
    assert not seen[40][0] and all(seen[40][1:]) and len(seen[40]) > 1
    assert all(seen[1])


def test_default_stops_screening_between_rounds():
    # queries unlike the rows sampled at load: all their pairs pass from the first round on,
    # and the rounds after it are exact
    ix, v, ids = _grouped(256, 300, 128, 1, 5)
    q = (8.0 * v[::300]).contiguous()
    got = ix.search(q, None, 10, 0.9, 2, 64, with_stats=True)
    rounds = _screened(ix)
    assert rounds[0] and len(rounds) > 1 and not any(rounds[1:])
    with knobs(SIEVE_SCREEN=0):
        _same(got[:3], ix.search(q, None, 10, 0.9, 2, 64))


def test_default_stops_screening_between_fixed_chunks():
    ix, v, ids = _grouped(256, 300, 128, 1, 5)
    few = (8.0 * v[::300]).contiguous()
    with knobs(SIEVE_FIX_CHUNK=100):
        got = ix.search_fixed(few, None, 10, 0.9, 64, with_stats=True)
        rounds = _screened(ix)
        assert rounds == [True, False, False]
        ix.search_fixed(v[::300].contiguous(), None, 10, 0.9, 64, with_stats=True)
        assert all(_screened(ix)) and len(_screened(ix)) == 3
    with knobs(SIEVE_SCREEN=0):
        _same(got[:3], ix.search_fixed(few, None, 10, 0.9, 64))


# The item scatter by groups of 4,096 (at least 32,768 items on at most 2,048 lists), against
# the exact search with one item at a time (fewer than 32,768 in a round)
@pytest.mark.parametrize("n_lists,nq,W", [(16, 4100, 8), (2048, 4097, 8), (1, 33000, 1),
                                          (2049, 4097, 8), (700, 4096, 8), (700, 4095, 8)])
def test_grouped_item_scatter(n_lists, nq, W):
    ix, v, ids = _grouped(n_lists, 20, 64, 3, nq)
    sel = (torch.arange(nq) * 7919 % len(v)).cuda()
    q, ex = v[sel].contiguous(), ids[sel].contiguous()
    got = ix.search(q, ex, 5, 0.8, W, 32)
    for a in range(0, nq, 1000):
        part = ix.search(q[a:a + 1000].contiguous(), ex[a:a + 1000].contiguous(), 5, 0.8, W, 32)
        _same([x[a:a + 1000] for x in got], part)
