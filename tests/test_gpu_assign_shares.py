"""GPU: the coarse assignment where the row blocks of the screening pass's last round, or of a short batch, are shared by
several workgroups: sizes one row, one block and a few blocks past whole rounds, and between, against float64.

A whole round is 512 row blocks of 256 rows at 200 coordinates and 768 at 96, so n = 131,072 + 1 and the like have a
last block that nothing else shares the chip with.
"""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,L,n", [
    (200, 512, 131_072), (200, 512, 131_073), (200, 512, 131_072 + 256), (200, 1000, 131_072 + 3 * 256 + 5),
    (200, 512, 262_147), (96, 1024, 196_608 + 77), (96, 700, 196_608 + 30 * 256 - 1),
    (96, 256, 1), (33, 4096, 255), (128, 520, 257), (128, 2048, 64_999),
])
def test_assignment_of_shared_blocks(d, L, n):
    import paper_2605_17415_amd as pkg
    g = torch.Generator(device="cuda:0")
    g.manual_seed(n + d)
    cent = torch.nn.functional.normalize(torch.randn((L, d), generator=g, device="cuda:0"), dim=1)
    ix = pkg.Index(d, 4, L)
    ix.set_coarse(cent.cpu().numpy())
    x = torch.randn((n, d), generator=g, device="cuda:0")
    x += 0.5 * x.norm(dim=1, keepdim=True) * cent[torch.randint(0, L, (n,), generator=g, device="cuda:0")]
    print(f"[shares] d={d} L={L} n={n}", flush=True)
    for rows in (n, min(n, 1000)):               # and a short batch on the workspace of the long one
        assign, _, _ = ix.encode_only(x[:rows], want_codes=False)
        wrong = 0
        for lo in range(0, rows, 32768):
            part = torch.nn.functional.normalize(x[lo:min(lo + 32768, rows)].double(), dim=1)
            s = part @ cent.double().T
            got = s.gather(1, assign[lo:lo + 32768].long()[:, None])[:, 0]
            # a cell other than the best is right where the two are within the stated near-tie of 1e-5
            wrong += int((got < s.max(1).values - 1e-5).sum())
        assert wrong == 0
