"""GPU: rows enter their lists in arrival order at the sizes where the counting sort changes shape: around one wavefront (64), one
round of a workgroup (1024), and 512 segments of one round (524,288), from which a segment has two; one cell that takes
everything, cells that few rows reach, and the most cells an index may have.  Against numpy's stable sort."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,L", [
    (1, 1), (63, 1), (65, 3), (1023, 16), (1024, 1000), (1025, 17), (4097, 16384), (70_001, 4096),
    (524_287, 64), (524_288, 1), (524_289, 1000), (1_200_007, 300),
])
def test_lists_hold_rows_in_arrival_order(n, L):
    import paper_2605_17415_amd as pkg
    rs = np.random.default_rng(n + L)
    cell = np.where(rs.random(n) < 0.3, L // 2, rs.integers(0, L, n)).astype(np.int32)
    cell[-1] = L - 1
    ix = pkg.Index(16, 4, L)
    ix.set_coarse(np.eye(16, dtype=np.float32)[np.arange(L) % 16])
    codes = torch.zeros((n, 16), dtype=torch.uint8, device="cuda:0")
    gamma = torch.ones(n, dtype=torch.float16, device="cuda:0")
    print(f"[stable order] n={n} L={L}", flush=True)
    for batch in range(2):                       # the second behind the first
        ix.add_encoded(torch.from_numpy(cell).cuda(), codes, gamma)
    order = np.argsort(np.concatenate([cell, cell]), kind="stable")
    size = np.bincount(cell, minlength=L) * 2
    first = np.cumsum(size) - size
    for l in {0, L // 2, L // 3, L - 1}:
        ids = ix.export_list(l)[0]
        assert np.array_equal(np.asarray(ids), order[first[l]:first[l] + size[l]])
    ix.close()
