"""3x3 blocks with FP32 values that stream from HBM: Y rows of 16 bytes (k = 4)
leave non-temporally; every column equals the one-column product of that
column bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
spmv = pytest.importorskip("paper_2107_12371_amd")

pytestmark = pytest.mark.gpu


def test_columns_equal_one_column_products():
    # 6.9M blocks of 40 bytes: 275 MB
    rng = np.random.default_rng(3)
    lens = np.r_[0, 1, 509, 700, np.full(860_000, 8), 511, 0]
    ptr = np.r_[0, np.cumsum(lens)].astype(np.int32)
    at = np.arange(ptr[-1]) - np.repeat(ptr[:-1].astype(np.int64), lens)
    col = (at * np.repeat(800 // np.maximum(lens, 1), lens)).astype(np.int32)
    with spmv.Matrix.from_bsr3(lens.size, 800, ptr, col, rng.random((int(ptr[-1]), 3, 3)), fp32=True) as M:
        X = torch.as_tensor(rng.uniform(-1, 1, (2400, 4)), dtype=torch.float32, device="cuda")
        Y = M.spmm_f32(X)
        for j in range(4):
            assert torch.equal(Y[:, j], M.spmm_f32(X[:, j:j + 1].contiguous())[:, 0]), j
