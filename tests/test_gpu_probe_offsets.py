"""Candidate offsets for every number of probes: up to 64 they are written by the wavefront that selects the probes, beyond
that (or over more than 8192 cells) by a launch of their own.  A search over P probes must return what a search over all
cells gives once the vectors of other cells are left out (the same sums in the same order when streamed: equal bits; the
batched scan within 1e-4: coarse + gamma * (d products of split float16 operands), gamma <= 1.2, d = 48)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nprobe", [1, 2, 31, 32, 33, 63, 64, 65, 90])
@pytest.mark.parametrize("mode,nq,k", [(1, 3, 10), (1, 70, 10), (2, 7, 5), (2, 70, 40)])
def test_any_number_of_probes(nprobe, mode, nq, k):
    import paper_2605_17415_amd as pkg
    print(f"[probe offsets] nprobe={nprobe} mode={mode} nq={nq} k={k}", flush=True)
    rng = np.random.default_rng(nprobe)
    d, L = 48, 90
    sizes = rng.integers(0, 20, L)
    sizes[rng.integers(0, L, 8)] = 0
    n = int(sizes.sum())
    cell = rng.permutation(np.repeat(np.arange(L), sizes)).astype(np.int32)
    cent = rng.standard_normal((L, d)).astype(np.float32)
    cent /= np.linalg.norm(cent, axis=1, keepdims=True)
    ix = pkg.Index(d, 4, L, rotation_seed=5)
    ix.set_coarse(cent)
    ix.add_encoded(*[torch.from_numpy(v).to("cuda:0") for v in (cell, rng.integers(0, 16, (n, d)).astype(np.uint8),
                                                                  rng.uniform(0.2, 1.2, n).astype(np.float16))])
    q = torch.from_numpy(rng.standard_normal((nq, d)).astype(np.float32)).to("cuda:0")
    ix.set_search_mode(1)
    all_s, all_i = [t.cpu().numpy() for t in ix.search(q, L, n)]
    probes = np.argsort(-(q.cpu().numpy().astype(np.float64) @ cent.T.astype(np.float64)), axis=1)[:, :nprobe]
    ix.set_search_mode(mode)
    for _ in range(2):                               # (the second call finds the first one's counters)
        got_s, got_i = [t.cpu().numpy() for t in ix.search(q, nprobe, k)]
        for a in range(nq):
            keep = np.isin(cell[all_i[a]], probes[a])
            want_s, want_i = all_s[a][keep][:k], all_i[a][keep][:k]
            m = len(want_s)
            assert np.all(got_i[a, m:] == -1)
            if mode == 1:
                np.testing.assert_array_equal(got_i[a, :m], want_i)
                np.testing.assert_array_equal(got_s[a, :m], want_s)
            else:
                np.testing.assert_allclose(got_s[a, :m], want_s, rtol=0, atol=1e-4)
    ix.close()
