"""The batched scan where a list meets as many queries as fill a row tile, one fewer, and one more: the dense pass takes 16 queries to a row
tile and 32 to a tile, the threshold pass 32 to a row tile and two to four row tiles to a tile, by the width.  Every query probes all
six lists, whose sizes lie around the edges of a slab of 32 vectors and of a part.  Against the streaming scan of the same index.

Tolerance: two evaluations of a score lie at most gamma |z| |C| (2 * 2^-21 + d 2^-24) <= 1e-4 apart for gamma <= 1.2, |C| <= 2, d <= 256."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = [33, 256, 257, 1000, 31, 64]


@pytest.mark.parametrize("d,b", [(64, 4), (96, 4), (97, 2), (128, 3), (128, 4), (193, 8), (200, 4), (209, 4), (225, 5), (256, 4)])
def test_query_counts_at_tile_edges(d, b):
    import paper_2605_17415_amd as pkg
    print(f"[batch tiles] d={d} b={b}", flush=True)
    rng = np.random.default_rng(1000 * d + b)
    L, n = len(SIZES), sum(SIZES)
    cent = rng.standard_normal((L, d)).astype(np.float32)
    ix = pkg.Index(d, b, L, rotation_seed=d)
    ix.set_coarse(cent / np.linalg.norm(cent, axis=1, keepdims=True))
    cell = rng.permutation(np.repeat(np.arange(L), SIZES)).astype(np.int32)
    ix.add_encoded(*[torch.from_numpy(v).to("cuda:0") for v in (cell, rng.integers(0, 1 << b, (n, d)).astype(np.uint8), rng.uniform(0.2, 1.2, n).astype(np.float16))])
    for nq in (3, 4, 5, 15, 16, 17, 32, 33, 64, 65, 96, 97, 128, 129, 193):
        q = torch.from_numpy(rng.standard_normal((nq, d)).astype(np.float32)).to("cuda:0")
        got = []
        for mode in (1, 2):
            ix.set_search_mode(mode)
            got.append([t.cpu().numpy() for t in ix.search(q, L, 10)])
        assert ix.scan_stats()["queries"] == nq      # mode 2 took the batched scan
        (s1, i1), (s2, i2) = got
        assert np.all(np.abs(s1 - s2) <= 1e-4) and (i1 >= 0).all() and (i2 >= 0).all()
        for a, c, sa in zip(i1, i2, s1):             # a label that only one side has sits at the k-th value
            assert np.all(np.abs(sa[np.isin(a, c, invert=True)] - sa[-1]) <= 2e-4)
    ix.close()


@pytest.mark.parametrize("nq", [255, 600, 2000])
def test_lists_with_many_tiles(nq):
    """Few lists that every query probes: a list has up to 20 parts for each of 63 tiles of queries, more tiles than a thread writes by itself (64),
    and other lists fewer."""
    import paper_2605_17415_amd as pkg
    print(f"[many tiles] nq={nq}", flush=True)
    rng = np.random.default_rng(nq)
    d, b, sizes = 64, 4, [3000, 257, 64, 31, 5000, 1, 1024]
    L, n = len(sizes), sum(sizes)
    cent = rng.standard_normal((L, d)).astype(np.float32)
    ix = pkg.Index(d, b, L, rotation_seed=1)
    ix.set_coarse(cent / np.linalg.norm(cent, axis=1, keepdims=True))
    cell = rng.permutation(np.repeat(np.arange(L), sizes)).astype(np.int32)
    ix.add_encoded(*[torch.from_numpy(v).to("cuda:0") for v in (cell, rng.integers(0, 1 << b, (n, d)).astype(np.uint8), rng.uniform(0.2, 1.2, n).astype(np.float16))])
    q = torch.from_numpy(rng.standard_normal((nq, d)).astype(np.float32)).to("cuda:0")
    got = []
    for mode in (1, 2):
        ix.set_search_mode(mode)
        got.append([t.cpu().numpy() for t in ix.search(q, L, 10)])
    assert ix.scan_stats()["queries"] == nq
    (s1, i1), (s2, i2) = got
    assert np.all(np.abs(s1 - s2) <= 1e-4) and (i1 >= 0).all() and (i2 >= 0).all()
    for a, c, sa in zip(i1, i2, s1):
        assert np.all(np.abs(sa[np.isin(a, c, invert=True)] - sa[-1]) <= 2e-4)
    ix.close()
