"""GPU: coarse scores and rotated queries have the same bits whichever operand the queries are (small calls: the column one, from 8M scores
on: the row one), at every panel width, with queries that end inside a tile and a number of cells that is no
multiple of anything; and the scores agree with float64.

Tolerance: a dot product of unit vectors in split float16 form is within 2e-6 of float64."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,L,nq", [(20, 67, 1025), (64, 70, 1026), (96, 133, 1300), (100, 1000, 1055), (128, 65, 1057), (150, 70, 1025), (192, 64, 1060), (200, 333, 1281),
                                    (208, 70, 1025), (224, 66, 1100), (255, 70, 1027), (256, 129, 1536),
                                    (20, 4033, 2110), (64, 2050, 4070), (96, 4096, 2049), (100, 4095, 2081), (128, 1025, 7720), (150, 4040, 2075),
                                    (192, 4097, 2056), (200, 3333, 2501), (208, 4000, 2101), (224, 1026, 7720), (255, 4010, 2091), (256, 2049, 3999)])
def test_same_bits_in_large_and_small_calls(d, L, nq):
    import paper_2605_17415_amd as pkg
    rng = np.random.default_rng(d + L)
    cent = rng.standard_normal((L, d)).astype(np.float32)
    cent /= np.linalg.norm(cent, axis=1, keepdims=True)
    n = 5000
    ix = pkg.Index(d, 4, L, rotation_seed=3)
    ix.set_coarse(cent)
    ix.add_encoded(*[torch.from_numpy(v).cuda() for v in (rng.integers(0, L, n).astype(np.int32), rng.integers(0, 16, (n, d)).astype(np.uint8),
                                                          rng.uniform(0.2, 1.2, n).astype(np.float16))])
    q = torch.from_numpy(rng.standard_normal((nq, d)).astype(np.float32)).cuda()
    print(f"[coarse layouts] d={d} L={L} nq={nq}", flush=True)
    ix.set_search_mode(1)
    probe, coarse = (t.cpu().numpy() for t in ix.coarse_probe(q, 16))
    scores, ids = (t.cpu().numpy() for t in ix.search(q, 16, 10))
    for lo in range(0, nq, 500):
        part = q[lo:lo + 500].contiguous()
        p, c = (t.cpu().numpy() for t in ix.coarse_probe(part, 16))
        s, i = (t.cpu().numpy() for t in ix.search(part, 16, 10))
        np.testing.assert_array_equal(p, probe[lo:lo + 500])
        np.testing.assert_array_equal(c, coarse[lo:lo + 500])
        np.testing.assert_array_equal(s, scores[lo:lo + 500])
        np.testing.assert_array_equal(i, ids[lo:lo + 500])
    unit = q.cpu().numpy().astype(np.float64)
    unit /= np.linalg.norm(unit, axis=1, keepdims=True)
    want = np.take_along_axis(unit @ cent.astype(np.float64).T, probe.astype(np.int64), axis=1)
    np.testing.assert_allclose(coarse, want, rtol=0, atol=2e-6)
    ix.close()
