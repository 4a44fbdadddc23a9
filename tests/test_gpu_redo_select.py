"""Queries redone exactly because their candidate list overflowed: the selection among what they keep, for numbers of winners
at its edges (1, one wavefront's, kRedoFew - 1 / + 0 / + 1 = 127 ... 129, many) and for numbers of kept entries around kRedoFew,
below and beyond the 2048 that its LDS holds, with distinct scores and with all scores of a cell equal.  Against the
streaming scan of the same index; every case is one in which the query really is redone.

Tolerance: as in the other comparisons of two float32 evaluations of coarse + gamma * (d products), 1e-4 for gamma <= 1.2."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


# (seven lists of 120 overflow a candidate list of 512, i.e. k up to 32, but not the 1024 to 2048 of larger k)
@pytest.mark.parametrize("per_list,equal,k", [(120, False, k) for k in (1, 10, 32)] +
                         [(n, equal, k) for n, equal in ((400, False), (2000, False), (2000, True)) for k in (1, 10, 64, 127, 128, 129, 300)])
def test_selection_of_a_redone_query(per_list, equal, k):
    import paper_2605_17415_amd as pkg
    print(f"[redo select] per_list={per_list} equal={equal} k={k}", flush=True)
    rng = np.random.default_rng(per_list + k)
    d, L, b = 64, 16, 4
    cent = rng.standard_normal((L, d)).astype(np.float32)
    cent /= np.linalg.norm(cent, axis=1, keepdims=True)
    q = torch.from_numpy(rng.standard_normal((2, d)).astype(np.float32)).to("cuda:0")
    order = np.argsort(-(q[0].cpu().numpy() @ cent.T))
    pi = np.linalg.qr(rng.standard_normal((d, d)))[0].astype(np.float32)
    # the nearest cell, whose vectors the threshold comes from, holds those furthest from the first query (the lowest code
    # where its rotated coordinate is positive, else the highest); what the other cells hold beats it
    near = 1500 if k < 300 else 4000                 # the whole dense prefix: more than k * (candidates) / capacity
    cell = np.concatenate([np.full(near, order[0])] + [np.full(per_list, l) for l in order[1:8]]).astype(np.int32)
    codes = rng.integers(0, 1 << b, (len(cell), d)).astype(np.uint8)
    codes[:near] = np.where(pi @ q[0].cpu().numpy() > 0, 0, (1 << b) - 1)
    gamma = rng.uniform(0.2, 1.2, len(cell)).astype(np.float16)
    gamma[:near] = 1.2
    if equal:
        gamma[near:] = 0.0
    ix = pkg.Index(d, b, L)
    ix.set_coarse(cent)
    ix.set_rotation(pi)
    ix.add_encoded(*[torch.from_numpy(v).to("cuda:0") for v in (cell, codes, gamma)])
    got = []
    for mode in (1, 2):
        ix.set_search_mode(mode)
        got.append([t.cpu().numpy() for t in ix.search(q, 8, k)])
    assert ix.scan_stats()["redone_exactly"] >= 1
    (s1, i1), (s2, i2) = got
    np.testing.assert_array_equal(s1 == -np.inf, s2 == -np.inf)
    real = np.isfinite(s1)
    np.testing.assert_allclose(s2[real], s1[real], rtol=0, atol=1e-4)
    for a, c, sa in zip(i1, i2, s1):
        assert len(set(c[c >= 0].tolist())) == (c >= 0).sum()
        odd = np.isin(a, c, invert=True) & (a >= 0)
        assert np.all(np.abs(sa[odd] - sa[a >= 0][-1]) <= 2e-4)
    ix.close()


@pytest.mark.parametrize("metric,norm,q_len,x_len", [("cosine", 1.0, 1.0, 1.0), ("cosine", 1e4, 1.0, 1.0), ("cosine", 6e4, 1.0, 1.0), ("ip", 1e4, 1.0, 3.0),
                                                     ("l2", 1e4, 0.5, 2.0), ("l2", 1.0, 1e-3, 1.0), ("l2", 1.0, 1e-4, 1.0)])
def test_threshold_survives_the_redo_at_any_norm(metric, norm, q_len, x_len):
    """Stored norms far beyond the quantiser's own (a caller's codes may have any float16) and distances of queries much
    shorter than the rows: the k best all sit in the nearest list, whose k-th is the threshold, and the other lists hold
    900 copies of it per query one float16 step of the norm below, which overflow the candidate list.  The redo has to
    find the k-th again although it sums in another order.

    Tolerance: the sums differ by at most |z||C| (2 d 2^-24 + 2^-20) <= 2.7 * 8.6e-6 = 2.4e-5 per unit of the norm
    (d = 64, |C| <= 8 * 0.33), a quarter of the copies' distance (2^-11 of a score of at least 0.2); rounding of the value itself
    2^-22 of its terms."""
    import paper_2605_17415_amd as pkg
    print(f"[redo norms] {metric} norm={norm} q_len={q_len}", flush=True)
    rng = np.random.default_rng(11)
    d, L, b, nq, k = 64, 16, 4, 16, 10
    cent = np.repeat(rng.standard_normal((1, d)).astype(np.float32), L, axis=0)
    cent /= np.linalg.norm(cent, axis=1, keepdims=True)
    pi = np.linalg.qr(rng.standard_normal((d, d)))[0].astype(np.float32)
    ix = pkg.Index(d, b, L)
    ix.set_coarse(cent)                              # equal cells: probed in ascending order, list 0 is the nearest
    ix.set_rotation(pi)
    levels, _ = ix.get_codebook()
    q = rng.standard_normal((nq, d)).astype(np.float32)
    q /= np.linalg.norm(q, axis=1, keepdims=True)
    near = rng.integers(0, 1 << b, (3000, d)).astype(np.uint8)
    est = (q.astype(np.float64) @ pi.T) @ levels[near].astype(np.float64).T
    copies = np.repeat(near[np.argsort(-est, axis=1)[:, k - 1]], 900, axis=0)
    codes = np.concatenate([near, copies])
    full = np.float16(norm)
    gamma = np.concatenate([np.full(len(near), full), np.full(len(copies), np.nextafter(full, np.float16(0)))])
    cell = np.concatenate([np.zeros(len(near)), 1 + np.arange(len(copies)) % (L - 1)]).astype(np.int32)
    on = [torch.from_numpy(v).to("cuda:0") for v in (cell, codes, gamma)]
    if metric == "cosine":
        ix.add_encoded(*on)
    else:
        ix.set_metric(pkg.binding.METRIC_IP if metric == "ip" else pkg.binding.METRIC_L2)
        ix.add_encoded_raw(*on, torch.full((len(cell),), x_len, dtype=torch.float32, device="cuda:0"))
    qd = torch.from_numpy(q * np.float32(q_len)).to("cuda:0")
    got = []
    for mode in (1, 2):
        ix.set_search_mode(mode)
        got.append([t.cpu().numpy() for t in ix.search(qd, L, k)])
    assert ix.scan_stats()["redone_exactly"] == nq
    (s1, i1), (s2, i2) = got
    assert (i1 >= 0).all() and (i2 >= 0).all()
    scale = {"cosine": 1.0, "ip": q_len * x_len, "l2": 2 * q_len * x_len}[metric]
    offset = q_len ** 2 + x_len ** 2 if metric == "l2" else 0.0
    tol = scale * 2.4e-5 * norm + 2.0 ** -22 * (offset + np.abs(s1).max())
    np.testing.assert_allclose(s2, s1, rtol=0, atol=tol)
    for a, c, sa in zip(i1, i2, s1):
        assert len(set(c.tolist())) == k
        odd = np.isin(a, c, invert=True)
        assert np.all(np.abs(sa[odd] - sa[-1]) <= 2 * tol)
    ix.close()


@pytest.mark.parametrize("above", [0, 116, 117, 118, 119, 120, 300])
def test_few_kept_entries(above):
    """About above + 10 entries reach the threshold (the 10 best of the nearest list and what other lists hold above it), around
    the 128 from which on a radix search narrows them down; 900 copies a float16 step of the norm below it overflow the
    candidate list."""
    import paper_2605_17415_amd as pkg
    print(f"[redo few] above={above}", flush=True)
    rng = np.random.default_rng(above)
    d, L, b, k = 64, 8, 4, 10
    cent = np.repeat(rng.standard_normal((1, d)).astype(np.float32), L, axis=0)
    cent /= np.linalg.norm(cent, axis=1, keepdims=True)
    ix = pkg.Index(d, b, L, rotation_seed=3)
    ix.set_coarse(cent)
    levels, _ = ix.get_codebook()
    q = rng.standard_normal((1, d)).astype(np.float32)
    q /= np.linalg.norm(q)
    pool = rng.integers(0, 1 << b, (4000, d)).astype(np.uint8)
    est = levels[pool].astype(np.float64) @ (ix.get_rotation().astype(np.float64) @ q[0])
    pool = pool[np.argsort(-est)]
    near = pool[above:]
    codes = np.concatenate([near, pool[:above], np.repeat(near[k - 1:k], 900, axis=0)])
    gamma = np.ones(len(codes), np.float16)
    gamma[len(pool):] = np.nextafter(np.float16(1), np.float16(0))
    cell = np.zeros(len(codes), np.int32)
    cell[len(near):] = 1 + np.arange(len(codes) - len(near)) % (L - 1)
    ix.add_encoded(*[torch.from_numpy(v).to("cuda:0") for v in (cell, codes, gamma)])
    got = []
    for mode in (1, 2):
        ix.set_search_mode(mode)
        got.append([t.cpu().numpy() for t in ix.search(torch.from_numpy(q).to("cuda:0"), L, k)])
    assert ix.scan_stats()["redone_exactly"] == 1
    (s1, i1), (s2, i2) = got
    assert (i2 >= 0).all() and len(set(i2[0].tolist())) == k
    np.testing.assert_allclose(s2, s1, rtol=0, atol=1e-4)
    odd = np.isin(i1[0], i2[0], invert=True)
    assert np.all(np.abs(s1[0][odd] - s1[0][-1]) <= 2e-4)
    ix.close()


@pytest.mark.parametrize("nq,limit", [(1200, 4 << 30), (1025, 4 << 30), (1024, 4 << 30), (513, 4 << 30), (300, 1 << 20), (600, 3 << 20), (1200, 36 << 20)])
def test_more_redone_queries_than_rows_or_workgroups(nq, limit):
    """Every query of the call is redone: in one launch, with as many score rows as queries or workgroups (1024), or in launches for as
    many queries as a small workspace has rows for (30, 91 and 1097 rows; the last is one launch again).

    Tolerance: as above."""
    import paper_2605_17415_amd as pkg
    print(f"[redo many] nq={nq} limit={limit}", flush=True)
    rng = np.random.default_rng(nq)
    d, L, b, k, near, per_list = 64, 16, 4, 10, 1500, 400
    cent = rng.standard_normal((L, d)).astype(np.float32)
    cent /= np.linalg.norm(cent, axis=1, keepdims=True)
    base = rng.standard_normal(d)
    q = torch.from_numpy((base + 0.02 * rng.standard_normal((nq, d))).astype(np.float32)).to("cuda:0")
    order = np.argsort(-(cent @ base))
    pi = np.linalg.qr(rng.standard_normal((d, d)))[0].astype(np.float32)
    cell = np.concatenate([np.full(near, order[0])] + [np.full(per_list, l) for l in order[1:8]]).astype(np.int32)
    codes = rng.integers(0, 1 << b, (len(cell), d)).astype(np.uint8)
    codes[:near] = np.where(pi @ base > 0, 0, (1 << b) - 1)          # the nearest cell's are the furthest from the queries
    gamma = rng.uniform(0.2, 1.2, len(cell)).astype(np.float16)
    gamma[:near] = 1.2
    ix = pkg.Index(d, b, L)
    ix.set_coarse(cent)
    ix.set_rotation(pi)
    ix.add_encoded(*[torch.from_numpy(v).to("cuda:0") for v in (cell, codes, gamma)])
    ix.set_search_mode(1)
    s1, i1 = [t.cpu().numpy() for t in ix.search(q, 8, k)]
    ix.set_search_mode(2)
    ix.set_workspace_limit(limit)
    for _ in range(2):
        s2, i2 = [t.cpu().numpy() for t in ix.search(q, 8, k)]
        stats = ix.scan_stats()
        assert stats["redone_exactly"] == stats["queries"] > 0
        assert (i1 >= 0).all() and (i2 >= 0).all()
        np.testing.assert_allclose(s2, s1, rtol=0, atol=1e-4)
        for a, c, sa in zip(i1, i2, s1):
            assert len(set(c.tolist())) == k
            assert np.all(np.abs(sa[np.isin(a, c, invert=True)] - sa[-1]) <= 2e-4)
    ix.close()
