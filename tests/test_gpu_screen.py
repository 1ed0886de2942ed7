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
