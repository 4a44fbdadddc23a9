"""ivftq_reconstruct on lists whose lengths sit around the kernel's tiles of 32, 64 and 128 vectors (empty ones and runs
of empty ones among them), for every padded width and every number of stored bits, against the definition
x^ = c~_l + gamma * Pi^T C[code] in float64, with guard rows behind both outputs.

Tolerance: every product carries a relative error of at most 2^-21 (two split float16 operands), and d of them are
added in float32; Cauchy-Schwarz bounds the sum of their magnitudes by |C[code]| <= sqrt(d) max|C|, the rows of Pi being
unit vectors.  So |error| <= gamma * sqrt(d) * max|C| * (2^-21 + d 2^-24), plus the rounding of the result."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = [0, 1, 31, 0, 0, 32, 33, 63, 64, 65, 127, 128, 129, 0, 300, 1, 0]


@pytest.mark.parametrize("d,b", [(8, 1), (32, 4), (33, 3), (60, 7), (61, 5), (64, 2), (70, 7), (96, 4), (100, 5), (128, 8), (129, 6), (160, 4), (192, 3),
                                 (200, 7), (224, 4), (255, 5), (256, 8)])
def test_tiles_and_widths(d, b):
    import paper_2605_17415_amd as pkg
    print(f"[reconstruct tiles] d={d} b={b}", flush=True)
    rng = np.random.default_rng(1000 * d + b)
    L, n = len(SIZES), sum(SIZES)
    cell = rng.permutation(np.repeat(np.arange(L), SIZES)).astype(np.int32)
    codes = rng.integers(0, 1 << b, (n, d)).astype(np.uint8)
    gamma = rng.uniform(0.0, 1.2, n).astype(np.float16)
    labels = rng.permutation(10 * n)[:n].astype(np.int64)
    cent = rng.standard_normal((L, d)).astype(np.float32)
    cent /= np.linalg.norm(cent, axis=1, keepdims=True)
    dev = torch.device("cuda:0")
    ix = pkg.Index(d, b, L, rotation_seed=d)
    ix.set_coarse(cent)
    ix.add_encoded(torch.from_numpy(cell).to(dev), torch.from_numpy(codes).to(dev), torch.from_numpy(gamma).to(dev),
                   torch.from_numpy(labels).to(dev))
    # guard rows behind the outputs: stores of a tile past its list's end are dropped, and nothing goes past the last list's
    guard = 64
    x, ids = torch.full((n + guard, d), -7.0, device=dev), torch.full((n + guard,), -7, dtype=torch.int64, device=dev)
    pkg.binding._check(ix._lib.ivftq_reconstruct(ix._h, x.data_ptr(), ids.data_ptr(), None))
    torch.cuda.synchronize()
    assert (x[n:] == -7.0).all() and (ids[n:] == -7).all()
    x, ids = x[:n], ids[:n]
    order = np.argsort(cell, kind="stable")
    levels, _ = ix.get_codebook()
    pi = ix.get_rotation().astype(np.float64)
    want = cent[cell[order]] + gamma[order].astype(np.float64)[:, None] * (levels[codes[order]].astype(np.float64) @ pi)
    bound = gamma[order].astype(np.float64)[:, None] * np.sqrt(d) * np.abs(levels).max() * (2.0 ** -21 + d * 2.0 ** -24) + 2.0 ** -24 * (np.abs(want) + 1)
    np.testing.assert_array_equal(ids.cpu().numpy(), labels[order])
    assert np.all(np.abs(x.cpu().numpy() - want) <= bound)
    ix.close()


@pytest.mark.parametrize("d,b", [(8, 4), (12, 1), (12, 3), (25, 2), (32, 2), (33, 1), (49, 3), (60, 4), (64, 2), (65, 1), (96, 4)])
def test_no_further_off_than_float32_multiply_adds(d, b):
    """The error against float64 over many vectors, next to that of float32 fused multiply-adds in ascending order, which
    hold every operand in full.  Both are root mean squares over 4000 d values, so 5 % is far outside their scatter."""
    import paper_2605_17415_amd as pkg
    print(f"[reconstruct error] d={d} b={b}", flush=True)
    rng = np.random.default_rng(100 * d + b)
    L, n = 16, 4000
    cell = rng.integers(0, L, n).astype(np.int32)
    gamma = rng.uniform(0.3, 0.8, n).astype(np.float16)
    cent = rng.standard_normal((L, d)).astype(np.float32)
    cent /= np.linalg.norm(cent, axis=1, keepdims=True)
    ix = pkg.Index(d, b, L, rotation_seed=7)
    ix.set_coarse(cent)
    levels, tau = ix.get_codebook()
    codes = np.searchsorted(tau, rng.standard_normal((n, d)) / np.sqrt(d), side="right").astype(np.uint8)
    ix.add_encoded(*[torch.from_numpy(v).to("cuda:0") for v in (cell, codes, gamma)])
    x, ids = (t.cpu().numpy() for t in ix.reconstruct())
    g, c, val, pi = gamma[ids].astype(np.float64)[:, None], cent[cell[ids]], levels[codes[ids]].astype(np.float64), ix.get_rotation().astype(np.float64)
    want = c + g * (val @ pi)
    acc = np.zeros((n, d), np.float32)
    for k in range(d):
        acc = (acc + val[:, k:k + 1] * pi[k]).astype(np.float32)
    plain = (c + g * acc).astype(np.float32)
    rms = lambda e: np.sqrt(np.mean(e ** 2))
    assert rms(x - want) <= 1.05 * rms(plain - want)
    ix.close()
