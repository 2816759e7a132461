"""The k-vector product between the sizes of test_gpu_spmm: matrices beyond
the L2s (rounds of eight entries) that a cache keeps (ordinary loads of the
stream), Y below and above the size from which it is stored past L2.  Every
column equals the single-vector product of that column bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
spmv = pytest.importorskip("paper_2107_12371_amd")

pytestmark = pytest.mark.gpu


SIZES = [(9_000, 40), (30_000, 250), (200_001, 40)]


@pytest.mark.parametrize("rows,most,k", [(*s, k) for s in SIZES for k in (2, 3, 8)] + [(100_000, 20, 32)])
def test_columns_equal_single_products(rows, most, k):
    # 2 MB of matrix and at k = 2 a small Y; 45 MB with a small Y (0.5 MB at
    # k = 2) and a larger one; 48 MB with a larger one; 12 MB that would stay in
    # the L2s but for an X of 26 MB
    rng = np.random.default_rng(rows)
    lens = rng.integers(0, most + 1, rows)
    ptr = np.zeros(rows + 1, np.int32)
    np.cumsum(lens, out=ptr[1:])
    at = np.arange(ptr[-1]) - np.repeat(ptr[:-1].astype(np.int64), lens)
    col = np.minimum(np.repeat(np.arange(rows), lens) + at, rows - 1).astype(np.int32)
    with spmv.Matrix(rows, rows, ptr, col, rng.uniform(-1, 1, int(ptr[-1]))) as A:
        X = torch.as_tensor(rng.uniform(-1, 1, (rows, k)), device="cuda")
        Y = A.spmm(X)
        for j in range(k):
            assert torch.equal(Y[:, j], A.apply(X[:, j].contiguous())), j
