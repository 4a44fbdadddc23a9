"""Queries redone exactly because their candidate list overflowed: the selection among what they keep, for numbers of winners
at its edges (1, one wavefront's, kRedoFew - 1 / + 0 / + 1 = 127 ... 129, many) and for numbers of kept entries below and
beyond the 2048 that its LDS holds, with distinct scores and with all scores of a cell equal.  Against the streaming scan
of the same index.

Tolerance: as in the other comparisons of two float32 evaluations of coarse + gamma * (d products), 1e-4 for gamma <= 1.2."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 10, 64, 127, 128, 129, 300])
@pytest.mark.parametrize("per_list,equal", [(120, False), (400, False), (2000, False), (2000, True)])
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
    cell = np.concatenate([np.full(1500, order[0])] + [np.full(per_list, l) for l in order[1:8]]).astype(np.int32)
    codes = rng.integers(0, 1 << b, (len(cell), d)).astype(np.uint8)
    codes[:1500] = np.where(pi @ q[0].cpu().numpy() > 0, 0, (1 << b) - 1)
    gamma = rng.uniform(0.2, 1.2, len(cell)).astype(np.float16)
    gamma[:1500] = 1.2
    if equal:
        gamma[1500:] = 0.0
    ix = pkg.Index(d, b, L)
    ix.set_coarse(cent)
    ix.set_rotation(pi)
    ix.add_encoded(*[torch.from_numpy(v).to("cuda:0") for v in (cell, codes, gamma)])
    got = []
    for mode in (1, 2):
        ix.set_search_mode(mode)
        got.append([t.cpu().numpy() for t in ix.search(q, 8, k)])
    (s1, i1), (s2, i2) = got
    np.testing.assert_array_equal(s1 == -np.inf, s2 == -np.inf)
    real = np.isfinite(s1)
    np.testing.assert_allclose(s2[real], s1[real], rtol=0, atol=1e-4)
    for a, c, sa in zip(i1, i2, s1):
        assert len(set(c[c >= 0].tolist())) == (c >= 0).sum()
        odd = np.isin(a, c, invert=True) & (a >= 0)
        assert np.all(np.abs(sa[odd] - sa[a >= 0][-1]) <= 2e-4)
    ix.close()
