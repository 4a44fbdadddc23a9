"""Raw-metric search (inner product and squared L2 of un-normalised vectors) through the C ABI against the
oracle: the norms encode_add stores, and the search over identical stored codes and norms.  Tolerances:
values within 1e-4 of the size of their terms (|q||x| for the inner product, |q|^2 + |x|^2 for the
distance, whose three terms cancel for near neighbours), top-k sets identical up to ties within that."""
import numpy as np
import pytest

import gpu_cases
import parity
from oracle import ivftq_oracle as orc

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

DEV = "cuda:0"
RTOL = 1e-4


def _pkg():
    import paper_2605_17415_amd as pkg
    return pkg


def _scaled_inputs(cs, seed):
    """The case's rows and queries at lengths spread over a factor of 40 (directions unchanged, so the
    case's oracle encode still applies)."""
    rs = np.random.Generator(np.random.Philox(key=[seed, 55]))
    xs = rs.uniform(0.1, 4.0, size=(len(cs.X), 1)).astype(np.float32)
    qs = rs.uniform(0.3, 3.0, size=(len(cs.Q), 1)).astype(np.float32)
    return cs.X / np.linalg.norm(cs.X, axis=1, keepdims=True) * xs, cs.Q * qs


def _compare(metric, g_vals, g_ids, o_vals, o_ids, o_all, xnorm, qnorm, probe_gap, k):
    """Every returned (label, value) against the oracle's value for that candidate; sets up to ties."""
    swaps = 0
    for q in range(len(o_ids)):
        cid, val = o_all[q]
        lookup = dict(zip(cid.tolist(), val.tolist()))
        n_real = min(k, len(cid))
        gi, gv = g_ids[q], g_vals[q]
        worst = -np.inf if metric == "ip" else np.inf
        assert np.all(gi[n_real:] == -1) and np.all(gv[n_real:] == worst), f"query {q}: bad padding"
        d = np.diff(gv[:n_real])
        assert np.all(d <= 0) if metric == "ip" else np.all(d >= 0), f"query {q}: not best-first"
        assert len(set(gi[:n_real].tolist())) == n_real
        near_probe_tie = probe_gap[q] < parity.BOUNDARY_TOL
        tol_of = (lambda lab: RTOL * qnorm[q] * xnorm[lab] + 1e-6) if metric == "ip" else \
                 (lambda lab: RTOL * (qnorm[q] ** 2 + xnorm[lab] ** 2) + 1e-6)
        for lab, v in zip(gi[:n_real].tolist(), gv[:n_real].tolist()):
            if lab not in lookup:
                assert near_probe_tie, f"query {q}: label {lab} is outside the oracle's probed lists"
                continue
            assert abs(v - lookup[lab]) <= tol_of(lab), f"query {q} label {lab}: {v} vs oracle {lookup[lab]}"
        gset, oset = set(gi[:n_real].tolist()), set(o_ids[q, :n_real].tolist())
        if gset != oset and not near_probe_tie:
            kth = o_vals[q, n_real - 1]
            for lab in (gset - oset) | (oset - gset):
                assert abs(lookup[lab] - kth) <= 2 * tol_of(lab), f"query {q}: label {lab} is no tie of the k-th value"
            swaps += 1
    return swaps


@pytest.mark.parametrize("name", ["d96_b4", "d128", "d70_b6", "d96_b3s"])
@pytest.mark.parametrize("metric", ["ip", "l2"])
def test_raw_metric_search_matches_oracle(name, metric):
    pkg = _pkg()
    cs = gpu_cases.get_case(name)
    X, Q = _scaled_inputs(cs, 7)
    enc = orc.encode(X, cs.cent, cs.Pi, cs.tau)
    xnorm = orc.raw_norms_fp32(X)
    qnorm = np.linalg.norm(Q.astype(np.float64), axis=1)
    n = len(X)
    print(f"[raw metric {metric} {name}] n={n} d={cs.d} b={cs.b}", flush=True)
    code = pkg.binding.METRIC_IP if metric == "ip" else pkg.binding.METRIC_L2

    # the whole path: encode_add stores the norms; codes and float16 residual norms as in the cosine index
    ix = pkg.Index(cs.d, cs.b_stage1, cs.nlist, sign_bit=cs.sign_bit)
    ix.set_coarse(cs.cent)
    ix.set_rotation(cs.Pi)
    ix.set_metric(code)
    ix.encode_add(torch.from_numpy(X).to(DEV))
    assert ix.index_bytes() == n * (4 * ((cs.b * cs.d + 31) // 32) + 2 + 8 + 4)
    g_assign = np.full(n, -1, np.int32)
    g_codes = np.zeros((n, cs.d), np.uint8)
    g_gamma = np.zeros(n, np.float16)
    g_norm = np.zeros(n, np.float32)
    for l in range(cs.nlist):
        ids, lc, lg = ix.export_list(l)
        g_assign[ids], g_codes[ids], g_gamma[ids], g_norm[ids] = l, lc, lg, ix.export_norms(l)
    print("  encode:", parity.compare_encode(enc, g_assign, g_codes, g_gamma), flush=True)
    np.testing.assert_allclose(g_norm, xnorm, rtol=2.5e-7, atol=0)          # float32 sum of squares against the rounded double
    ix.close()

    # search over the oracle's codes and norms
    ref = orc.ListIndex(cs.cent, cs.Pi, cs.c, cs.tau)
    ref.add_encoded(enc["assign"], np.arange(n, dtype=np.int64), enc["codes"], enc["gamma16"])
    ix = pkg.Index(cs.d, cs.b_stage1, cs.nlist, sign_bit=cs.sign_bit)
    ix.set_coarse(cs.cent)
    ix.set_rotation(cs.Pi)
    ix.set_metric(code)
    with pytest.raises(pkg.IvftqError):
        ix.add_encoded(torch.from_numpy(enc["assign"]).to(DEV), torch.from_numpy(enc["codes"]).to(DEV),
                       torch.from_numpy(enc["gamma16"]).to(DEV))              # norms are required
    half = n // 2                                                             # two appends: the norms follow the pool's growth
    for lo, hi in ((0, half), (half, n)):
        ix.add_encoded_raw(torch.from_numpy(enc["assign"][lo:hi]).to(DEV), torch.from_numpy(enc["codes"][lo:hi]).to(DEV),
                           torch.from_numpy(enc["gamma16"][lo:hi]).to(DEV), torch.from_numpy(xnorm[lo:hi]).to(DEV))
    o_vals, o_ids, _, S, o_all = orc.search_raw(ref, xnorm, Q, cs.nprobe, cs.k, metric, return_all=True)
    gap = parity.probe_cut_gap(S, cs.nprobe)
    vals, ids = ix.search(torch.from_numpy(Q).to(DEV), cs.nprobe, cs.k)
    torch.cuda.synchronize()
    swaps = _compare(metric, vals.cpu().numpy(), ids.cpu().numpy(), o_vals, o_ids, o_all, xnorm.astype(np.float64), qnorm, gap, cs.k)
    print(f"  search: {len(Q)} queries, {swaps} with a tie swapped at the k-th place", flush=True)
    # the other raw metric on the same index: free to switch; cosine is not
    other = pkg.binding.METRIC_L2 if metric == "ip" else pkg.binding.METRIC_IP
    ix.set_metric(other)
    o2 = orc.search_raw(ref, xnorm, Q, cs.nprobe, cs.k, "l2" if metric == "ip" else "ip", return_all=True)
    vals2, ids2 = ix.search(torch.from_numpy(Q).to(DEV), cs.nprobe, cs.k)
    torch.cuda.synchronize()
    _compare("l2" if metric == "ip" else "ip", vals2.cpu().numpy(), ids2.cpu().numpy(), o2[0], o2[1], o2[4],
             xnorm.astype(np.float64), qnorm, gap, cs.k)
    with pytest.raises(pkg.IvftqError) as e:
        ix.set_metric(pkg.binding.METRIC_COSINE)
    assert e.value.status == pkg.binding.BAD_STATE
    with pytest.raises(pkg.IvftqError) as e:
        ix.search_cascade(torch.from_numpy(Q).to(DEV), cs.nprobe, cs.k, 1, 2 * cs.k)
    assert e.value.status == pkg.binding.UNSUPPORTED
    ix.close()


def test_raw_metric_on_unit_inputs_is_the_cosine_search():
    """With unit rows and unit queries the inner-product values are the cosine scores and the ranking is the same."""
    pkg = _pkg()
    cs = gpu_cases.get_case("d96_b4")
    X = (cs.X / np.linalg.norm(cs.X, axis=1, keepdims=True)).astype(np.float32)
    Q = (cs.Q / np.linalg.norm(cs.Q, axis=1, keepdims=True)).astype(np.float32)
    out = []
    for metric in (pkg.binding.METRIC_COSINE, pkg.binding.METRIC_IP):
        ix = pkg.Index(cs.d, cs.b_stage1, cs.nlist)
        ix.set_coarse(cs.cent)
        ix.set_rotation(cs.Pi)
        ix.set_metric(metric)
        ix.set_search_mode(1)
        ix.encode_add(torch.from_numpy(X).to(DEV))
        s, i = ix.search(torch.from_numpy(Q).to(DEV), cs.nprobe, cs.k)
        torch.cuda.synchronize()
        out.append((s.cpu().numpy(), i.cpu().numpy()))
        ix.close()
    assert (out[0][1] == out[1][1]).mean() > 0.995
    np.testing.assert_allclose(out[1][0], out[0][0], rtol=2e-6, atol=1e-6)


@pytest.mark.parametrize("metric", ["ip", "l2"])
@pytest.mark.parametrize("d,b", [(40, 4), (96, 4), (128, 3), (200, 4), (256, 8)])
def test_a_length_that_is_no_number_hides_no_other_vector(metric, d, b):
    """One vector of every 32 has a NaN for a length, with either sign: it is no result itself, and the others are found by the
    batched scan, which looks at the range of the lengths of 32 vectors at a time, as by the streaming scan.

    Tolerance: two evaluations of a score lie at most gamma |z| |C| (2 * 2^-21 + d 2^-24) <= 1e-4 apart for gamma <= 1.2, |C| <= 2, d <= 256;
    times |q| |x| <= 3 for an inner product, twice that for a distance."""
    pkg = _pkg()
    print(f"[NaN lengths] {metric} d={d} b={b}", flush=True)
    rng = np.random.default_rng(d + b)
    sizes = [33, 256, 257, 1000, 31, 640]
    L, n, k, nq = len(sizes), sum(sizes), 10, 40
    cent = rng.standard_normal((L, d)).astype(np.float32)
    ix = pkg.Index(d, b, L, rotation_seed=d)
    ix.set_metric(pkg.binding.METRIC_IP if metric == "ip" else pkg.binding.METRIC_L2)
    ix.set_coarse(cent / np.linalg.norm(cent, axis=1, keepdims=True))
    cell = np.repeat(np.arange(L), sizes).astype(np.int32)          # (list order is input order: every slab of a list has one)
    length = rng.uniform(0.5, 2.0, n).astype(np.float32)
    none = np.concatenate([np.arange(int(rng.integers(0, min(32, s))), s, 32) + at for s, at in zip(sizes, np.cumsum([0] + sizes))])
    length[none] = np.array([np.nan, -np.nan], np.float32)[np.arange(len(none)) % 2]
    rows = (cell, rng.integers(0, 1 << b, (n, d)).astype(np.uint8), rng.uniform(0.2, 1.2, n).astype(np.float16), length)
    ix.add_encoded_raw(*[torch.from_numpy(v).to(DEV) for v in rows])
    q = rng.standard_normal((nq, d)).astype(np.float32)
    q *= 1.5 / np.linalg.norm(q, axis=1, keepdims=True)
    got = []
    for mode in (1, 2):
        ix.set_search_mode(mode)
        got.append([t.cpu().numpy() for t in ix.search(torch.from_numpy(q).to(DEV), L, k)])
    assert ix.scan_stats()["queries"] == nq
    (s1, i1), (s2, i2) = got
    tol = 3e-4 if metric == "ip" else 6e-4
    assert (i1 >= 0).all() and not np.isin(i1, none).any() and not np.isin(i2, none).any()
    np.testing.assert_allclose(s2, s1, rtol=0, atol=tol)
    for a, c, sa in zip(i1, i2, s1):                                 # a label that only one side has sits at the k-th value
        assert np.all(np.abs(sa[np.isin(a, c, invert=True)] - sa[-1]) <= 2 * tol)
    ix.close()
