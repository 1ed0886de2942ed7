"""The fused ranking's compile-time fp16 dimensions against the fp64 order (exact, no tolerance)."""
import os

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


# 96: the run-time kernel; 256: LDS-staged queries (64 a work-group); 384 / 512: the wide
# configuration (96).  131 queries: a second, ragged work-group in each; 1,041
# centroids: a last row block of one; R = 64: the longest fused prefix.
@pytest.mark.parametrize("nq", [1, 131])
@pytest.mark.parametrize("R", [1, 32, 64])
@pytest.mark.parametrize("d", [96, 256, 384, 512])
def test_prefix_order_of_compile_time_dimensions(d, R, nq):
    import paper_2608_03199_amd as ps
    g = np.random.default_rng(d + R)
    nlist = 1041
    C = g.standard_normal((nlist, d))
    C = (C / np.linalg.norm(C, axis=1, keepdims=True)).astype(np.float16)
    C[700:720] = C[3]  # ties to the lower index
    Q = g.standard_normal((nq, d))
    Q = (Q / np.linalg.norm(Q, axis=1, keepdims=True)).astype(np.float16)
    Q[0] = C[3]
    off = np.zeros(nlist + 1, np.int64)
    off[1:] = 4
    cu = lambda x: torch.tensor(x).cuda()  # noqa: E731
    ix = ps.Index(cu(C[:4]), cu(off), cu(np.arange(4)), cu(C))
    os.environ["SIEVE_RANK_PATH"] = "2"
    try:
        P = ix.rank(cu(Q), R).cpu().numpy()
    finally:
        del os.environ["SIEVE_RANK_PATH"]
    s = np.zeros((nq, nlist))
    for t in range(d):  # the dimension-ordered fp64 sum
        s += Q[:, t:t + 1].astype(np.float64) * C[:, t].astype(np.float64)
    assert np.array_equal(P, np.argsort(-s, axis=1, kind="stable")[:, :R])
