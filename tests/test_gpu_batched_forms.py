"""The batched list scan (search mode 2) over the forms it takes: every bit count it has, dimensions that end inside and at
the end of a block of 16, cosine and raw metrics, lists that are empty, shorter than one tile of vectors, at its edges, and
long enough to be cut into several parts (lists of more than 512 vectors are cut into nearly equal parts of at most that
many), and with more than 256 results, which the merge sorts instead of counting.  Against the streaming scan (mode 1) of
the same index, which sums float32 products in another order.

Tolerance: a score is coarse + gamma * (d products, both split float16 operands), its two evaluations apart by at most
gamma |z| |C| (2 * 2^-21 + d 2^-24) <= 1e-4 for gamma <= 1.2, |z| = 1, |C| <= 2 and d <= 256; a raw metric scales that by |q||x|
(twice that for a distance).  Labels may differ only where the values are that close to the k-th."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = [0, 1, 31, 64, 65, 0, 127, 511, 512, 513, 577, 1025, 2500, 64 * 33, 900, 3]
FORMS = [(32, 4, "cosine", 1), (50, 2, "l2", 10), (64, 3, "ip", 33), (96, 4, "l2", 10), (100, 5, "cosine", 100), (128, 8, "cosine", 10),
         (129, 4, "ip", 7), (161, 5, "l2", 20), (200, 3, "cosine", 64), (208, 8, "ip", 10), (224, 2, "cosine", 100), (255, 8, "l2", 65), (256, 5, "ip", 20),
         (96, 4, "l2", 300), (100, 4, "ip", 500), (64, 8, "cosine", 300),
         # (a tile holds candidates back in LDS: at most 4096 at d = 64, about 900 at d = 256 with 5 bits, and these have more)
         (64, 4, "l2", 600), (256, 5, "ip", 600)]


def _index(d, b, metric, rng):
    import paper_2605_17415_amd as pkg
    L, n = len(SIZES), sum(SIZES)
    cell = rng.permutation(np.repeat(np.arange(L), SIZES)).astype(np.int32)
    cent = rng.standard_normal((L, d)).astype(np.float32)
    cent /= np.linalg.norm(cent, axis=1, keepdims=True)
    ix = pkg.Index(d, b, L, rotation_seed=d)
    ix.set_coarse(cent)
    on = [torch.from_numpy(v).to("cuda:0") for v in (cell, rng.integers(0, 1 << b, (n, d)).astype(np.uint8), rng.uniform(0.2, 1.2, n).astype(np.float16))]
    length = rng.uniform(0.5, 2.0, n).astype(np.float32)
    if metric == "cosine":
        ix.add_encoded(*on)
    else:
        ix.set_metric(pkg.binding.METRIC_IP if metric == "ip" else pkg.binding.METRIC_L2)
        ix.add_encoded_raw(*on, torch.from_numpy(length).to("cuda:0"))
    return ix


@pytest.mark.parametrize("d,b,metric,k", FORMS)
def test_batched_equals_streaming(d, b, metric, k):
    print(f"[batched forms] d={d} b={b} {metric} k={k}", flush=True)
    rng = np.random.default_rng(1000 * d + b)
    ix = _index(d, b, metric, rng)
    scale = 1.0 if metric == "cosine" else 2.0 * 2.0 if metric == "ip" else 2.0 * 2.0 * 2.0
    for nq in (1, 33, 300):                          # 300: some list meets more than one tile of 128 queries
        q = rng.standard_normal((nq, d)).astype(np.float32)
        q /= np.linalg.norm(q, axis=1, keepdims=True)
        q *= rng.uniform(0.5, 2.0, (nq, 1)).astype(np.float32)
        qd = torch.from_numpy(q).to("cuda:0")
        got = []
        for mode in (1, 2):
            ix.set_search_mode(mode)
            s, i = ix.search(qd, 9, k)
            torch.cuda.synchronize()
            got.append((s.cpu().numpy(), i.cpu().numpy()))
        stats = ix.scan_stats()
        assert stats["queries"] == nq                # mode 2 took the batched scan
        if k >= 300 and nq == 300:                   # and the merge had more than k entries to order
            assert stats["mean_candidates"] > 0 and stats["redone_exactly"] < nq
        (s1, i1), (s2, i2) = got
        real = i1 >= 0
        np.testing.assert_array_equal(real, i2 >= 0)
        np.testing.assert_array_equal(s1[~real], s2[~real])
        tol = 1e-4 * scale + 1e-6
        assert np.all(np.abs(s1[real] - s2[real]) <= tol)
        for a, c, sa in zip(i1, i2, s1):             # a label that only one side has sits at the k-th value
            odd = np.isin(a, c, invert=True) & (a >= 0)
            last = sa[a >= 0][-1] if (a >= 0).any() else 0.0
            assert np.all(np.abs(sa[odd] - last) <= 2 * tol)
    ix.close()


def test_infinite_norm_in_a_partial_query_tile():
    """A stored norm of +inf (only a caller's own codes can hold one) is best for every query whose sum is positive; queries
    beyond a tile's last one get nothing appended, and the finite results of the streaming scan come back."""
    import paper_2605_17415_amd as pkg
    rng = np.random.default_rng(3)
    d, L, n = 64, 4, 4000
    cent = rng.standard_normal((L, d)).astype(np.float32)
    cent /= np.linalg.norm(cent, axis=1, keepdims=True)
    gamma = rng.uniform(0.2, 1.2, n).astype(np.float16)
    gamma[rng.integers(0, n, 5)] = np.inf
    ix = pkg.Index(d, 4, L, rotation_seed=1)
    ix.set_coarse(cent)
    ix.add_encoded(*[torch.from_numpy(v).to("cuda:0") for v in (rng.integers(0, L, n).astype(np.int32), rng.integers(0, 16, (n, d)).astype(np.uint8), gamma)])
    q = torch.from_numpy(rng.standard_normal((5, d)).astype(np.float32)).to("cuda:0")
    got = []
    for mode in (1, 2):
        ix.set_search_mode(mode)
        s, i = ix.search(q, L, 20)
        torch.cuda.synchronize()
        got.append((s.cpu().numpy(), i.cpu().numpy()))
    (s1, i1), (s2, i2) = got
    for a, c in zip(i1, i2):
        assert len(set(c.tolist())) == 20
        assert len(set(a.tolist()) ^ set(c.tolist())) <= 2       # (a tie at the last place)
    fin = np.isfinite(s1) & np.isfinite(s2)
    np.testing.assert_array_equal(np.isposinf(s1), np.isposinf(s2))
    np.testing.assert_allclose(s2[fin], s1[fin], rtol=0, atol=1e-4)
    ix.close()


@pytest.mark.parametrize("d,b", [(8, 4), (10, 2), (12, 3), (16, 4), (32, 2), (32, 4), (64, 8)])
def test_scores_no_further_off_than_streamed(d, b):
    """Returned scores against float64: mode 2 (which streams the shapes whose split operands would be further off) is at most
    1.5 % above the streaming scan, three times the scatter of a root mean square over 60,000 scores."""
    import paper_2605_17415_amd as pkg
    print(f"[score error] d={d} b={b}", flush=True)
    rng = np.random.default_rng(d + b)
    L, n, nq, k = 64, 20000, 6000, 10
    ix = pkg.Index(d, b, L, rotation_seed=7)
    cent = rng.standard_normal((L, d)).astype(np.float32)
    cent /= np.linalg.norm(cent, axis=1, keepdims=True)
    ix.set_coarse(cent)
    levels, tau = ix.get_codebook()
    codes = np.searchsorted(tau, rng.standard_normal((n, d)) / np.sqrt(d), side="right").astype(np.uint8)
    gamma, cell = rng.uniform(0.3, 0.8, n).astype(np.float16), rng.integers(0, L, n).astype(np.int32)
    ix.add_encoded(*[torch.from_numpy(v).to("cuda:0") for v in (cell, codes, gamma)])
    q = rng.standard_normal((nq, d)).astype(np.float32)
    unit = q / np.linalg.norm(q.astype(np.float64), axis=1, keepdims=True)
    z = unit @ ix.get_rotation().astype(np.float64).T
    rms = []
    for mode in (1, 2):
        ix.set_search_mode(mode)
        s, i = (t.cpu().numpy() for t in ix.search(torch.from_numpy(q).to("cuda:0"), 8, k))
        want = np.einsum("qd,qkd->qk", unit, cent[cell[i]].astype(np.float64)) + gamma[i] * np.einsum("qd,qkd->qk", z, levels[codes[i]].astype(np.float64))
        rms.append(np.sqrt(np.mean((s - want) ** 2)))
    assert rms[1] <= 1.015 * rms[0]
    ix.close()


@pytest.mark.parametrize("d", [33, 64, 96, 100, 128, 150, 192, 200, 224, 256])
def test_long_passes_give_the_bits_of_short_ones(d):
    """From 400 million looked-up coordinates on, a threshold pass of 4-bit codes keeps its table in sixteen copies (at every width but
    256, where they do not fit): 4000 queries of 128 lists in one call, and the first 70 and last 33 in calls of their own, on codes without
    clusters, so that there are candidates to hold back and append."""
    import paper_2605_17415_amd as pkg
    rng = np.random.default_rng(d)
    L, nq, nprobe, k = 256, 4000, 128, 10
    panel = min(p for p in (64, 96, 128, 160, 192, 208, 224, 256) if p >= d)
    typical = int(4.2e8 / ((L + nq * nprobe // 128) * d)) + 1
    n = typical * L
    print(f"[long pass] d={d} panel={panel} n={n}", flush=True)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(d)
    ix = pkg.Index(d, 4, L, rotation_seed=3)
    cent = rng.standard_normal((L, d)).astype(np.float32)
    ix.set_coarse(cent / np.linalg.norm(cent, axis=1, keepdims=True))
    ix.add_encoded(torch.randint(0, L, (n,), generator=g, device="cuda:0", dtype=torch.int32), torch.randint(0, 16, (n, d), generator=g, device="cuda:0", dtype=torch.uint8),
                   (0.3 + 0.5 * torch.rand(n, generator=g, device="cuda:0")).to(torch.float16))
    ix.set_search_mode(2)
    q = torch.randn((nq, d), generator=g, device="cuda:0")
    whole = [t.cpu().numpy() for t in ix.search(q, nprobe, k)]
    stats = ix.scan_stats()
    assert stats["queries"] == nq and stats["mean_candidates"] >= 1      # (that is 4000 held back and more; a few a query in the first widths)
    for lo, hi in ((0, 70), (nq - 33, nq)):
        part = [t.cpu().numpy() for t in ix.search(q[lo:hi].contiguous(), nprobe, k)]
        np.testing.assert_array_equal(part[0], whole[0][lo:hi])
        np.testing.assert_array_equal(part[1], whole[1][lo:hi])
    ix.close()
