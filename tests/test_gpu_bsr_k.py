"""The 3x3 block product with k columns: every column equals the one-column
product of that column bit for bit (both add a block row's products in
ascending order), at the edges of tiles (84 block rows, 510 blocks, a longer
row in a tile of its own), for k below, at and above the width whose Y rows
are stored non-temporally (16 bytes), aligned and not."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
spmv = pytest.importorskip("paper_2107_12371_amd")

pytestmark = pytest.mark.gpu
ROWS = {"one": [3], "empty": [0] * 85, "edges": [0, 1, 2, 5, 6, 7, 509, 510, 511, 0, 700, 1],
        "many": [0, 3, 7] + [6] * 83 + [7] * 84 + [5] * 85 + [1] * 400 + [0]}


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("k", [2, 3, 4, 6, 8, 12])
@pytest.mark.parametrize("kind", sorted(ROWS) + ["large"])  # large: streams from HBM
def test_columns_equal_one_column_products(kind, k, fp32):
    rng = np.random.default_rng(k)
    n_cols = 800
    lens = np.asarray(ROWS[kind] if kind != "large" else [0, 1, 509, 700] + [8] * 480_000 + [511, 0])
    ptr = np.zeros(lens.size + 1, np.int32)
    np.cumsum(lens, out=ptr[1:])
    # a row's columns ascend at a stride of its own
    at = np.arange(ptr[-1]) - np.repeat(ptr[:-1].astype(np.int64), lens)
    col = (at * np.repeat(n_cols // np.maximum(lens, 1), lens)).astype(np.int32)
    val = rng.uniform(-1, 1, (int(ptr[-1]), 3, 3))
    dt = torch.float32 if fp32 else torch.float64
    with spmv.Matrix.from_bsr3(lens.size, n_cols, ptr, col, val, fp32=fp32) as M:
        mm = M.spmm_f32 if fp32 else M.spmm
        for off in (0, 1):
            X = torch.empty(3 * n_cols * k + 1, dtype=dt, device="cuda")[off:off + 3 * n_cols * k].view(-1, k)
            X.copy_(torch.as_tensor(rng.uniform(-1, 1, (3 * n_cols, k))))
            Y = torch.full((3 * lens.size * k + 1,), float("nan"), dtype=dt, device="cuda")
            Yk = Y[off:off + 3 * lens.size * k].view(-1, k)
            mm(X, Yk)
            for j in range(k):
                one = mm(X[:, j:j + 1].contiguous())
                assert torch.equal(Yk[:, j], one[:, 0]), (off, j)
            assert torch.isnan(Y[-1 if off == 0 else 0])
