"""Selection of search results: of a streaming search from its scores, around lists that are empty, near whole blocks of 64 and long, or
through the block maxima that the scan leaves for few, long rows; 1 to 193 results (192 is the most the workgroup kernel's short cut
takes, 24 / 25 the line between its two bounds); many equal scores; more probes than are staged in LDS; many queries, from either
scan; queries and scores that are no numbers.  Against float64 scores of every candidate.  A score is coarse + gamma * (a float32 sum of d products), so it is within
gamma |z| |C| d 2^-24 < 1e-5 of float64 for the gamma <= 1.2, |C| <= 2 and d = 48 used here, plus the 2e-7 of the coarse term."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TOL = 1e-5
D, B = 48, 4


def _index(sizes, rng, tied, same_cells=False):
    import paper_2605_17415_amd as pkg
    L, n = len(sizes), int(sum(sizes))
    cell = rng.permutation(np.repeat(np.arange(L), sizes)).astype(np.int32)
    cent = rng.standard_normal((L, D)).astype(np.float32)
    cent /= np.linalg.norm(cent, axis=1, keepdims=True)
    if same_cells:                                   # the same coarse term everywhere
        cent[:] = cent[0]
    codes = rng.integers(0, 1 << B, (n, D)).astype(np.uint8)
    gamma = rng.uniform(0.2, 1.2, n).astype(np.float16)
    if tied:                                         # a handful of different vectors, over and over
        codes, gamma = codes[rng.integers(0, 5, n)], np.full(n, 0.5, np.float16)
    ix = pkg.Index(D, B, L, rotation_seed=5)
    ix.set_coarse(cent)
    ix.add_encoded(*[torch.from_numpy(v).to("cuda:0") for v in (cell, codes, gamma)])
    return ix, cell, cent, codes, gamma


def _scores(ix, q, cell, cent, codes, gamma):
    q = q.astype(np.float64) / np.linalg.norm(q.astype(np.float64), axis=1, keepdims=True)
    level = ix.get_codebook()[0].astype(np.float64)[codes]
    z = q @ ix.get_rotation().astype(np.float64).T
    return (q @ cent.astype(np.float64).T)[:, cell] + gamma.astype(np.float64) * (z @ level.T)


@pytest.mark.parametrize("shape,nprobe,tied", [("edges", 9, False), ("edges", 20, False), ("edges", 20, True), ("long", 4, False), ("long", 4, True),
                                               ("few", 3, False), ("many", 300, False)])
@pytest.mark.parametrize("k", [1, 10, 24, 25, 100, 192, 193])
def test_streaming_results(shape, nprobe, tied, k):
    rng = np.random.default_rng(len(shape) + 10 * nprobe + k)
    sizes = {"edges": [0, 1, 63, 64, 65, 0, 127, 128, 129, 0, 0, 191, 255, 256, 257, 300, 511, 512, 513, 64],
             "long": [6000, 1, 0, 70, 4097, 3000], "few": [40, 0, 3], "many": rng.integers(0, 200, 320).tolist()}[shape]
    print(f"[selection] {shape} nprobe={nprobe} tied={tied} k={k}", flush=True)
    ix, cell, cent, codes, gamma = _index(sizes, rng, tied)
    ix.set_search_mode(1)
    for nq in (1, 66):
        q = rng.standard_normal((nq, D)).astype(np.float32)
        qd = torch.from_numpy(q).to("cuda:0")
        probe = ix.coarse_probe(qd, nprobe)[0].cpu().numpy()
        got_s, got_i = [t.cpu().numpy() for t in ix.search(qd, nprobe, k)]
        true = _scores(ix, q, cell, cent, codes, gamma)
        for r in range(nq):
            cand = np.flatnonzero(np.isin(cell, probe[r]))
            take = min(k, len(cand))
            ids = got_i[r, :take]
            assert len(set(ids.tolist())) == take and set(ids.tolist()) <= set(cand.tolist())
            assert (got_i[r, take:] == -1).all() and np.isneginf(got_s[r, take:]).all()
            np.testing.assert_allclose(got_s[r, :take], true[r, ids], rtol=0, atol=TOL)
            np.testing.assert_allclose(got_s[r, :take], np.sort(true[r, cand])[::-1][:take], rtol=0, atol=TOL)
            same = got_s[r, :take][:-1] == got_s[r, :take][1:]
            assert (np.diff(got_s[r, :take]) <= 0).all() and (np.diff(ids)[same] > 0).all()
    ix.close()


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("nq", [5, 300])
def test_a_query_without_a_norm_leaves_the_others_alone(mode, nq):
    """infinite and zero queries: no results for the first, coarse term 0 for the second, and nobody else's change"""
    rng = np.random.default_rng(nq)
    ix, *_ = _index([300] * 16, rng, False)
    ix.set_search_mode(mode)
    q = rng.standard_normal((nq, D)).astype(np.float32)
    want = [t.cpu().numpy() for t in ix.search(torch.from_numpy(q).to("cuda:0"), 4, 10)]
    q[1, 3] = np.inf
    q[nq - 2] = 0.0
    got = [t.cpu().numpy() for t in ix.search(torch.from_numpy(q).to("cuda:0"), 4, 10)]
    others = np.setdiff1d(np.arange(nq), [1, nq - 2])
    np.testing.assert_array_equal(got[0][others], want[0][others])
    np.testing.assert_array_equal(got[1][others], want[1][others])
    assert (got[1][1] == -1).all() and np.isneginf(got[0][1]).all()
    assert (got[0][nq - 2] == 0.0).all()
    ix.close()


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("metric", ["ip", "l2"])
@pytest.mark.parametrize("k", [10, 1300])
def test_missing_results_of_raw_metrics(mode, metric, k):
    """Places without a result hold -inf (inner product) or +inf (distance), never what is no number, also where the query has no usable
    norm: an infinite query has no results at all, a zero one the same values for all, and 1300 are more than four lists of 300 hold."""
    import paper_2605_17415_amd as pkg
    rng = np.random.default_rng(mode + k)
    L, n, nq = 16, 4800, 70
    cent = rng.standard_normal((L, D)).astype(np.float32)
    cent /= np.linalg.norm(cent, axis=1, keepdims=True)
    ix = pkg.Index(D, B, L, rotation_seed=5)
    ix.set_metric(pkg.binding.METRIC_IP if metric == "ip" else pkg.binding.METRIC_L2)
    ix.set_coarse(cent)
    xnorm = rng.uniform(0.5, 2.0, n).astype(np.float32)
    ix.add_encoded_raw(*[torch.from_numpy(v).to("cuda:0") for v in ((np.arange(n) % L).astype(np.int32), rng.integers(0, 1 << B, (n, D)).astype(np.uint8),
                                                                  rng.uniform(0.2, 1.2, n).astype(np.float16), xnorm)])
    ix.set_search_mode(mode)
    q = rng.standard_normal((nq, D)).astype(np.float32)
    q[1, 3] = np.inf
    q[2] = 0.0
    print(f"[missing results] mode={mode} {metric} k={k}", flush=True)
    s, i = (t.cpu().numpy() for t in ix.search(torch.from_numpy(q).to("cuda:0"), 4, k))
    real = min(k, 1200)
    for r in range(nq):
        have = 0 if r == 1 else real
        assert (i[r, :have] >= 0).all() and (i[r, have:] == -1).all()
        assert np.isfinite(s[r, :have]).all() and (s[r, have:] == (-np.inf if metric == "ip" else np.inf)).all()
    np.testing.assert_allclose(s[2, :real], 0.0 if metric == "ip" else xnorm[i[2, :real]] ** 2, rtol=1e-6, atol=0)
    ix.close()


@pytest.mark.parametrize("nprobe", [10, 70])
@pytest.mark.parametrize("nq", [64, 65, 3000])
def test_a_query_that_is_no_number_has_no_cells_and_no_results(nprobe, nq):
    """whichever kernels a call's size leads to: 10 or 70 probes, 10 to 100 results, rows of up to 28,000 candidates, few queries or many"""
    rng = np.random.default_rng(nq + nprobe)
    ix, *_ = _index([400] * 100, rng, False)
    q = rng.standard_normal((nq, D)).astype(np.float32)
    q[7, 5], q[nq - 1, 0] = np.inf, np.nan
    bad = [7, nq - 1]
    qd = torch.from_numpy(q).to("cuda:0")
    print(f"[no number] nprobe={nprobe} nq={nq}", flush=True)
    probe, coarse = (t.cpu().numpy() for t in ix.coarse_probe(qd, nprobe))
    assert (probe[bad] == -1).all() and np.isneginf(coarse[bad]).all()
    good = np.delete(np.arange(nq), bad)
    assert (probe[good] >= 0).all()
    for mode in (1, 2):
        ix.set_search_mode(mode)
        for k in (10, 64, 100):
            s, i = (t.cpu().numpy() for t in ix.search(qd, nprobe, k))
            assert (i[bad] == -1).all() and np.isneginf(s[bad]).all()
            assert (i[good] >= 0).all() and np.isfinite(s[good]).all()
    s, i = (t.cpu().numpy() for t in ix.search_cascade(qd, nprobe, 10, 2, 100))
    assert (i[bad] == -1).all() and np.isneginf(s[bad]).all() and (i[good] >= 0).all()
    ix.close()


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("k", [10, 100, 300])
def test_a_distance_that_is_no_number_is_no_result(mode, k):
    """Squared distance to a stored length of +inf: its ranking key is inf - inf for some of the queries and comes last, so the results are
    those of the finite vectors, for any number of results and from either scan."""
    import paper_2605_17415_amd as pkg
    rng = np.random.default_rng(k)
    L, n, nq = 4, 4000, 40
    cent = rng.standard_normal((L, D)).astype(np.float32)
    cent /= np.linalg.norm(cent, axis=1, keepdims=True)
    ix = pkg.Index(D, B, L, rotation_seed=1)
    ix.set_metric(pkg.binding.METRIC_L2)
    ix.set_coarse(cent)
    xnorm = rng.uniform(0.5, 2.0, n).astype(np.float32)
    far = rng.choice(n, 20, replace=False)
    xnorm[far] = np.inf
    ix.add_encoded_raw(*[torch.from_numpy(v).to("cuda:0") for v in (rng.integers(0, L, n).astype(np.int32), rng.integers(0, 1 << B, (n, D)).astype(np.uint8),
                                                                  rng.uniform(0.2, 1.2, n).astype(np.float16), xnorm)])
    ix.set_search_mode(mode)
    print(f"[infinite length] mode={mode} k={k}", flush=True)
    s, i = (t.cpu().numpy() for t in ix.search(torch.from_numpy(rng.standard_normal((nq, D)).astype(np.float32)).to("cuda:0"), L, k))
    assert np.isfinite(s).all() and (i >= 0).all() and not np.isin(i, far).any()
    ix.close()


def _check_results(got_s, got_i, true, cell, probe, k, rows):
    for r in rows:
        cand = np.flatnonzero(np.isin(cell, probe[r]))
        take = min(k, len(cand))
        ids = got_i[r, :take]
        assert len(set(ids.tolist())) == take and np.isin(ids, cand).all()
        assert (got_i[r, take:] == -1).all() and np.isneginf(got_s[r, take:]).all()
        np.testing.assert_allclose(got_s[r, :take], true[r, ids], rtol=0, atol=TOL)
        np.testing.assert_allclose(got_s[r, :take], np.sort(true[r, cand])[::-1][:take], rtol=0, atol=TOL)
        same = got_s[r, :take][:-1] == got_s[r, :take][1:]
        assert (np.diff(got_s[r, :take]) <= 0).all() and (np.diff(ids)[same] > 0).all()


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("tied", [False, True])
@pytest.mark.parametrize("k", [1, 10, 32, 33, 64, 65, 200, 256])
def test_results_of_many_queries(mode, tied, k):
    """Above 1024 rows of up to 2048 candidates, and above 2048 longer ones, up to 64 results are selected by one wavefront a row; more,
    and smaller calls, by a workgroup a row (from 193 on by its radix search).  One query is infinite."""
    rng = np.random.default_rng(k + 7 * mode + tied)
    ix, cell, cent, codes, gamma = _index([0, 1, 63, 64, 65, 0, 127, 128, 129, 0, 0, 191, 255, 256, 257, 300, 511, 512, 513, 64], rng, tied)
    ix.set_search_mode(mode)
    print(f"[many queries] mode={mode} tied={tied} k={k}", flush=True)
    for nq, nprobe in ((1025, 4), (2049, 20)):
        q = rng.standard_normal((nq, D)).astype(np.float32)
        q[5, 2] = np.inf
        qd = torch.from_numpy(q).to("cuda:0")
        probe = ix.coarse_probe(qd, nprobe)[0].cpu().numpy()
        s, i = (t.cpu().numpy() for t in ix.search(qd, nprobe, k))
        assert (i[5] == -1).all() and np.isneginf(s[5]).all()
        q[5, 2] = 0.0
        some = np.setdiff1d(rng.integers(0, nq, 60), [5])
        true = np.zeros((nq, len(cell)))
        true[some] = _scores(ix, q[some], cell, cent, codes, gamma)
        _check_results(s, i, true, cell, probe, k, some)
    ix.close()


@pytest.mark.parametrize("shape,tied", [("edges", False), ("edges", True), ("equal", True), ("longest", False), ("longest", True)])
@pytest.mark.parametrize("k", [1, 10, 24, 25, 100, 192, 193])
def test_results_of_long_rows(shape, tied, k):
    """Rows whose results are selected through block maxima (up to 192 results, from 8192 candidates and the square of the number of results on): lists around whole blocks;
    more than 512 blocks whose best scores are equal, where the selection goes back to the whole row; more than 262,144 candidates,
    whose block maxima no longer fit a thread's registers."""
    rng = np.random.default_rng(len(shape) + k + 3 * tied)
    sizes = {"edges": [0, 1, 63, 64, 65, 0, 127, 128, 129, 0, 0, 191, 255, 256, 257, 300, 511, 512, 513, 64] * 8,
             "equal": [6000] * 8, "longest": [6000] * 50}[shape]
    ix, cell, cent, codes, gamma = _index(sizes, rng, tied, same_cells=shape == "equal")       # (equal: some 9600 vectors share a score)
    ix.set_search_mode(1)
    print(f"[long rows] {shape} tied={tied} k={k}", flush=True)
    for nq in (1, 3) if shape == "longest" else (1, 66):
        q = rng.standard_normal((nq, D)).astype(np.float32)
        qd = torch.from_numpy(q).to("cuda:0")
        nprobe = len(sizes)
        probe = ix.coarse_probe(qd, nprobe)[0].cpu().numpy()
        s, i = (t.cpu().numpy() for t in ix.search(qd, nprobe, k))
        some = np.arange(nq) if nq < 4 else rng.integers(0, nq, 10)
        true = np.zeros((nq, len(cell)))
        true[some] = _scores(ix, q[some], cell, cent, codes, gamma)
        _check_results(s, i, true, cell, probe, k, some)
    ix.close()
