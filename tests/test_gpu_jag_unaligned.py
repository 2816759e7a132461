"""Solves whose jagged products read vectors that are not 16-byte aligned:
cg_noalloc's p lies an odd number of words into its scratch array, and its x
is the caller's, here one word off.  Same kernels and partials as cg, whose
vectors are aligned: the same iterates bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
spmv = pytest.importorskip("paper_2107_12371_amd")

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [60_001, 60_002])
def test_solves_on_unaligned_vectors(n):
    # a symmetric band of half-width 9 with a dominant diagonal; 2^20 entries
    # and more, so that the handle has jagged tiles
    rng = np.random.default_rng(n)
    w = [rng.uniform(0.5, 1.5, n - d) for d in range(1, 10)]
    cols = np.arange(n)[:, None] + np.arange(-9, 10)
    vals = np.zeros((n, 19))
    for d in range(1, 10):
        vals[d:, 9 - d] = -w[d - 1]
        vals[:n - d, 9 + d] = -w[d - 1]
    vals[:, 9] = 0.5 - vals.sum(1)
    keep = (cols >= 0) & (cols < n)
    ptr = np.concatenate([[0], np.cumsum(keep.sum(1))]).astype(np.int32)
    b = torch.as_tensor(rng.uniform(-1, 1, n), device="cuda")
    with spmv.Matrix(n, n, ptr, cols[keep].astype(np.int32), vals[keep]) as A:
        assert A.nnz >= 1 << 20
        x, info = A.cg(b, tol=1e-9)
        buf = torch.zeros(n + 1, dtype=torch.float64, device="cuda")
        for off in (0, 1):
            buf.zero_()
            y, got = A.cg_noalloc(b, x=buf[off:off + n], tol=1e-9)
            assert got.iterations == info.iterations
            assert torch.equal(y, x)
