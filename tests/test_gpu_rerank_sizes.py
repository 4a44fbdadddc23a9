"""GPU: re-ranking at every number of coordinates a lane can hold and at the edges of its candidate counts (one wavefront's load,
256 that are placed by counting, and more, which are sorted), with repeated, missing and foreign labels, against float64.

Tolerance: <q, x> / (|q| |x|) from float32 sums of at most 4 products a lane and 6 additions across lanes: below
16 * 2^-24 = 1e-6 of a score of at most 1."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,r,k", [(1, 1, 1), (7, 2, 2), (63, 3, 1), (64, 5, 5), (65, 63, 10), (96, 64, 64), (128, 65, 20), (129, 255, 100),
                                   (192, 256, 256), (193, 257, 30), (255, 300, 300), (256, 256, 10), (256, 1000, 17)])
def test_sizes(d, r, k):
    import paper_2605_17415_amd as pkg
    rs = np.random.default_rng(1000 * d + r)
    n, nq = 700, 9
    X = rs.standard_normal((n, d)).astype(np.float32)
    X[11] = 0.0                                                       # a row without a norm is never a result
    Q = rs.standard_normal((nq, d)).astype(np.float32)
    cand = rs.integers(0, n, (nq, r))
    cand[0] = -1
    cand[1, ::2] = rs.integers(0, 3, len(cand[1, ::2]))               # the same few labels again and again
    cand[2, r // 2:] = -1
    cand[3, ::3] = n + rs.integers(0, 5, len(cand[3, ::3]))
    cand[4, ::2] = 11
    cand[5, 0] = 2 ** 40
    print(f"[rerank sizes] d={d} r={r} k={k}", flush=True)
    s, i = (t.cpu().numpy() for t in pkg.ivftq_rerank(torch.from_numpy(Q).cuda(), torch.from_numpy(X).cuda(), torch.from_numpy(cand).cuda(), k))
    Xd, Qd = X.astype(np.float64), Q.astype(np.float64)
    for q in range(nq):
        ids = np.unique(cand[q][(cand[q] >= 0) & (cand[q] < n) & (cand[q] != 11)])
        want = Xd[ids] @ Qd[q] / (np.linalg.norm(Xd[ids], axis=1) * np.linalg.norm(Qd[q]))
        m = min(k, len(ids))
        got = i[q, :m]
        assert np.all(i[q, m:] == -1) and np.all(np.isneginf(s[q, m:])) and len(set(got.tolist())) == m and np.isin(got, ids).all()
        np.testing.assert_allclose(s[q, :m], want[np.searchsorted(ids, got)], rtol=0, atol=1e-6)
        np.testing.assert_allclose(s[q, :m], np.sort(want)[::-1][:m], rtol=0, atol=1e-6)
        assert np.all(np.diff(s[q, :m]) <= 0)
        tied = np.flatnonzero(np.diff(s[q, :m]) == 0)                 # (d = 1: every score is 1 or -1)
        assert np.all(got[tied] < got[tied + 1])
