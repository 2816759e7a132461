"""The k-vector product's tiles: every column equals the single-vector product
of that column bit for bit (both add a row's rounded products in ascending
order), at the edges of rounds (4 and 8 entries), tiles (1,024 and 2,048
entries, 512 rows), column groups, alignments and 32-bit offsets."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
spmv = pytest.importorskip("paper_2107_12371_amd")

pytestmark = pytest.mark.gpu
EDGES = [0, 1, 3, 4, 5, 7, 8, 9, 11, 12, 13, 15, 16, 17, 1023, 1024, 1025, 2047, 2048, 2049, 0, 0]


def _csr(lens, n_cols, seed):
    rng = np.random.default_rng(seed)
    lens = np.asarray(lens, dtype=np.int64)
    ptr = np.zeros(lens.size + 1, dtype=np.int32)
    np.cumsum(lens, out=ptr[1:])
    # ascending columns at a row's own stride, from the row's own start
    stride = np.maximum(1, (n_cols - 1) // np.maximum(lens, 1))
    at = np.arange(ptr[-1], dtype=np.int64) - np.repeat(ptr[:-1].astype(np.int64), lens)
    near = np.repeat((np.arange(lens.size) * n_cols) // max(lens.size, 1), lens)
    col = np.where(np.repeat(lens > 64, lens), at * np.repeat(stride, lens), np.minimum(near, n_cols - 65) + 3 * (at % 22))
    return ptr, col.astype(np.int32), rng.uniform(-1, 1, int(ptr[-1]))


def _lens(kind):
    if kind == "edges":
        return EDGES
    if kind == "empty":
        return [0] * 1500 + EDGES + [0] * 700 + [1] * 1025
    if kind == "one":
        return [5]
    return EDGES + [17] * 1_400_000 + EDGES  # streams from HBM, rounds of 8


@pytest.mark.parametrize("kind", ["edges", "empty", "one", "large"])
@pytest.mark.parametrize("k", [2, 3, 4, 5, 8, 17])
def test_columns_equal_single_products(kind, k):
    lens = _lens(kind)
    n_cols = max(len(lens), 2200)
    ptr, col, val = _csr(lens, n_cols, 7)
    A = spmv.Matrix(len(lens), n_cols, ptr, col, val)
    buf = torch.rand(n_cols * k + 1, dtype=torch.float64, device="cuda") - 0.5
    for shift_x, shift_y in ((0, 0), (1, 0), (0, 1)):  # 16-byte aligned or not
        X = buf[shift_x:shift_x + n_cols * k].view(n_cols, k)
        Y = torch.full((len(lens) * k + 2,), 7.0, dtype=torch.float64, device="cuda")
        A.spmm(X, Y[shift_y:shift_y + len(lens) * k].view(len(lens), k))
        got = Y[shift_y:shift_y + len(lens) * k].view(len(lens), k)
        assert all(v == 7.0 for v in Y[shift_y + len(lens) * k:].tolist() + Y[:shift_y].tolist())
        for j in range(k):
            assert torch.equal(got[:, j], A.apply(X[:, j].contiguous()))


def test_x_of_more_than_4_gb():
    n_cols, k = (1 << 28) + 1000, 2  # X: 4 GiB and 16 KB
    rng = np.random.default_rng(3)
    ptr = np.arange(0, 300 * 9 + 1, 9, dtype=np.int32)
    col = np.sort(rng.integers(0, n_cols, (300, 9)), axis=1).astype(np.int32)
    col[:, -1] = n_cols - 1 - np.arange(300)  # beyond 32 bits of byte offset
    val = rng.uniform(-1, 1, 2700)
    A = spmv.Matrix(300, n_cols, ptr, np.sort(col, axis=1).ravel(), val)
    X = torch.rand((n_cols, k), dtype=torch.float64, device="cuda")
    Y = torch.empty((300, k), dtype=torch.float64, device="cuda")
    A.spmm(X, Y)
    for j in range(k):
        assert torch.equal(Y[:, j], A.apply(X[:, j].contiguous()))
