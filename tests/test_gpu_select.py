"""Probe selection over thousands of cells with large nprobe (figure "Architecture", Search: the nprobe
cells with the largest coarse scores), through `ivftq_coarse_probe`: the workgroup-per-row selection kernel
with and without its short cut, against a float64 sort.  Half of the centroids are exact copies of others,
so scores tie exactly across the cut and the rule "smallest cell number wins" is visible."""
import numpy as np
import pytest

from oracle import ivftq_oracle as orc

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
TOL = 1e-5


@pytest.mark.parametrize("L,nprobe", [(4096, 33), (4096, 40), (4096, 64), (2500, 50), (8000, 64), (1200, 48), (4096, 100), (4096, 128), (4096, 192), (4096, 200), (4096, 256), (2500, 150), (9000, 96)])
def test_probe_selection_with_exact_ties(L, nprobe):
    import paper_2605_17415_amd as pkg
    d, nq = 32, 300
    rs = np.random.Generator(np.random.Philox(key=[L, nprobe]))
    base = rs.standard_normal((L // 2, d))
    C = np.concatenate([base, base[: L - L // 2]])              # cell i + L/2 is a copy of cell i
    C = (C / np.linalg.norm(C, axis=1, keepdims=True)).astype(np.float32)
    Q = rs.standard_normal((nq, d)).astype(np.float32)
    ix = pkg.Index(d, 4, L)
    ix.set_coarse(C)
    print(f"[select] L={L} nprobe={nprobe}", flush=True)
    probe, coarse = ix.coarse_probe(torch.from_numpy(Q).to(DEV), nprobe)
    torch.cuda.synchronize()
    probe, coarse = probe.cpu().numpy(), coarse.cpu().numpy()
    S = orc.normalize_rows(Q) @ orc.normalize_rows(C).T           # float64
    rows = np.arange(nq)[:, None]
    np.testing.assert_allclose(coarse, S[rows, probe], rtol=1e-5, atol=1e-6)
    assert np.all(np.diff(coarse, axis=1) <= 0), "scores not descending"
    half = L // 2
    swaps = 0
    for qi in range(nq):
        got = probe[qi]
        assert len(set(got.tolist())) == nprobe, "a cell is listed twice"
        order = np.argsort(-S[qi], kind="stable")                 # score descending, cell number ascending
        want = order[:nprobe]
        kth = S[qi, want[-1]]
        if set(got.tolist()) != set(want.tolist()):
            # only cells whose score is within the tolerance of the cut may differ
            for cell in set(got.tolist()) ^ set(want.tolist()):
                assert abs(S[qi, cell] - kth) < TOL, f"query {qi}: cell {cell} differs away from the cut"
            swaps += 1
        # exact ties: a copy is never chosen without its original (the smaller number)
        chosen = set(got.tolist())
        for cell in got:
            if cell >= half:
                assert int(cell) - half in chosen, f"query {qi}: copy {cell} chosen without cell {cell - half}"
        # equal scores are listed by ascending cell number
        for a, b, ca, cb in zip(coarse[qi][:-1], coarse[qi][1:], got[:-1], got[1:]):
            if a == b:
                assert ca < cb, f"query {qi}: tied cells {ca}, {cb} out of order"
    print(f"  rows whose set differs within the tolerance of the cut: {swaps} of {nq}", flush=True)
    ix.close()


@pytest.mark.parametrize("L,nprobe,nq,different", [
    (4096, 8, 2049, 2048), (4096, 32, 2049, 2048), (4096, 33, 2049, 2048), (4096, 64, 2049, 2048), (8000, 64, 2050, 4000), (2500, 50, 2051, 1250),
    (1200, 10, 1025, 600), (1200, 48, 1027, 600), (100, 10, 1025, 50), (2048, 20, 1025, 1024), (2049, 20, 2048, 1025),
    (4096, 10, 2049, 5), (4096, 50, 2049, 5), (1000, 64, 1030, 3),                         # (hundreds of equal scores at the cut)
    (8193, 193, 70, 4000), (8193, 300, 70, 9), (8192, 193, 70, 9),          # (the radix search alone: more than 192 of more than 8192)
    (127, 20, 300, 64), (128, 64, 300, 7), (129, 64, 300, 7), (129, 100, 300, 65), (300, 8, 300, 3), (512, 200, 300, 256), (513, 30, 300, 5)])
def test_probes_of_every_kernel_with_exact_ties(L, nprobe, nq, different):
    """The one-wavefront kernel, which takes over above 1024 rows of up to 2048 cells and above 2048 longer ones, with its short cuts for up to
    32 and 64 winners and its radix search (hundreds of equal scores); the workgroup kernel around the 128 cells that it orders
    whole.  Cell i is a copy of cell i - different: a copy is never listed without, nor before, the cell that it copies."""
    import paper_2605_17415_amd as pkg
    d = 32
    rs = np.random.Generator(np.random.Philox(key=[L + nq, nprobe]))
    base = rs.standard_normal((different, d))
    base = (base / np.linalg.norm(base, axis=1, keepdims=True)).astype(np.float32)
    of = np.arange(L) % different
    Q = rs.standard_normal((nq, d)).astype(np.float32)
    Q[nq // 2, 3] = np.inf
    ix = pkg.Index(d, 4, L)
    ix.set_coarse(base[of])
    print(f"[select] L={L} nprobe={nprobe} nq={nq} different={different}", flush=True)
    probe, coarse = (t.cpu().numpy() for t in ix.coarse_probe(torch.from_numpy(Q).to(DEV), nprobe))
    assert (probe[nq // 2] == -1).all() and np.isneginf(coarse[nq // 2]).all()
    keep = np.arange(nq) != nq // 2
    probe, coarse, Q = probe[keep], coarse[keep], Q[keep]
    S = (orc.normalize_rows(Q) @ orc.normalize_rows(base).T)[:, of]
    rows = np.arange(nq - 1)[:, None]
    want = np.sort(S, axis=1)[:, ::-1][:, :nprobe]
    np.testing.assert_allclose(coarse, want, rtol=0, atol=TOL)
    np.testing.assert_allclose(S[rows, probe], want, rtol=0, atol=TOL)
    assert np.all(np.diff(coarse, axis=1) <= 0)
    assert np.all((np.diff(coarse, axis=1) < 0) | (np.diff(probe, axis=1) > 0)), "tied cells out of order"
    listed = np.zeros((nq - 1, L), bool)
    listed[rows, probe] = True
    assert np.all(listed.sum(1) == nprobe), "a cell is listed twice"
    assert np.all(listed[:, :-different] | ~listed[:, different:]), "a copy is listed without the cell that it copies"
    ix.close()


@pytest.mark.parametrize("L,nprobe,nq", [
    (1535, 10, 1025), (1536, 40, 1025), (1537, 10, 1025), (2559, 32, 2049), (2560, 10, 2049), (2561, 40, 2049),      # 8 groups of 64 after 1024 or 2048
    (2047, 10, 300), (2049, 100, 300), (4097, 10, 300), (6143, 100, 70), (6144, 10, 70), (6145, 100, 70)])           # 8 groups of 256
def test_probes_at_the_edges_of_full_rounds(L, nprobe, nq):
    """One column fewer than fills a round of loads, which then tests every column's range, exactly as many, and one more."""
    test_probes_of_every_kernel_with_exact_ties(L, nprobe, nq, L // 2 + 1)
