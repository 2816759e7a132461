"""Jagged window tiles (the default product of matrices of 2^20 entries and
more without compact windows, and of FP32 / BF16 values): the same bits as
the direct-gather row tiles, whose kernel choice is spmv_params.kernel = 1,
at the edges of tiles, slices, groups of entries and windows."""
import numpy as np
import pytest

import meshgen as mg
import oracle

torch = pytest.importorskip("torch")
spmv = pytest.importorskip("paper_2107_12371_amd")

pytestmark = pytest.mark.gpu
DEV = "cuda"
ROW_TILES = {"kernel": 1}


def banded(lens, n_cols, seed, spread=300):
    """Rows of the given lengths, distinct sorted columns near the diagonal."""
    rng = np.random.default_rng(seed)
    n = len(lens)
    rp = np.zeros(n + 1, np.int64)
    rp[1:] = np.cumsum(lens)
    row = np.repeat(np.arange(n), lens)
    j = np.arange(rp[-1]) - rp[row]
    step = np.maximum(1, (2 * spread) // np.maximum(lens, 1))[row]
    start = np.clip(row * n_cols // n - spread, 0, max(0, n_cols - 2 * spread - 32))
    col = start + j * step + rng.integers(0, step)
    ci = np.clip(col, 0, n_cols - 1).astype(np.int32)
    return mg.CSR(n, n_cols, rp.astype(np.int32), ci, rng.uniform(-1, 1, rp[-1]), 1)


def check(A, x, expect_jag=True):
    """All products bitwise against the row tiles, x aligned and 8 bytes off."""
    n = A.n_cols
    with spmv.Matrix.from_csr(A, fp32=True, bf16=True) as M, \
            spmv.Matrix.from_csr(A, fp32=True, bf16=True, params=ROW_TILES) as R:
        assert (M.info["device_bytes"] > 1.3 * R.info["device_bytes"]) == expect_jag
        for off in (0, 1):
            xd = torch.empty(n + 1, dtype=torch.float64, device=DEV)[off:off + n]
            xd.copy_(torch.as_tensor(x))
            xf = torch.empty(n + 1, dtype=torch.float32, device=DEV)[off:off + n]
            xf.copy_(xd)
            for f, v in (("apply", xd), ("apply_f32v", xd), ("apply_f32", xf), ("apply_bf16", xf)):
                a, b = getattr(M, f)(v).cpu().numpy(), getattr(R, f)(v).cpu().numpy()
                assert np.array_equal(a, b, equal_nan=True), (f, off)
        return M.apply(torch.as_tensor(x, device=DEV)).cpu().numpy()


@pytest.mark.parametrize("longest", [1, 4, 8, 9, 16, 17, 27, 28])
@pytest.mark.parametrize("extra_rows,extra_cols", [(0, 0), (1, 3), (63, 5), (255, 7)])
def test_row_lengths_and_ragged_sizes(longest, extra_rows, extra_cols):
    rng = np.random.default_rng(longest * 1000 + extra_rows)
    n = 256 * (1 + (1 << 20) // (128 * max(2, longest))) + 256 * 24 + extra_rows
    lens = rng.integers(0 if longest > 1 else 1, longest + 1, n)
    lens[rng.integers(0, n, 8)] = longest
    lens[:256] = 0          # a tile of empty rows
    lens[256:512] = longest  # and one of equal rows
    A = banded(lens, n + extra_cols, longest, spread=40)
    assert A.nnz >= 1 << 20
    x = rng.uniform(-1, 1, A.n_cols)
    # rows of one entry would stage more words than they have entries: those
    # keep the row tiles
    y = check(A, x, longest > 1)
    y_ref, bound = oracle.spmv(A, x)
    assert oracle.spmv_accept(y, y_ref, bound).all()


@pytest.mark.parametrize("sectors", [511, 512, 513])
def test_window_limit(sectors):
    # one tile whose rows touch exactly `sectors` sectors of 8 words
    n = 90_000
    lens = np.full(n, 14)
    A = banded(lens, n, 3)
    col = (np.arange(256 * 14) % sectors) * 8 + np.arange(256 * 14) // sectors
    A.col_idx[512 * 14:768 * 14] = np.sort(col.reshape(256, 14), 1).reshape(-1).astype(np.int32)
    check(A, np.random.default_rng(1).uniform(-1, 1, n))


def test_long_and_rejected_rows():
    # rows of 29 to 40 entries in no jagged tile, rows longer than a tile, and
    # one in several pieces
    rng = np.random.default_rng(5)
    n = 120_000
    lens = rng.integers(5, 20, n)
    lens[rng.integers(0, n, 60)] = rng.integers(29, 41, 60)
    lens[[1000, 70_000]] = [5000, 40_000]
    A = banded(lens, n, 6)
    x = rng.uniform(-1, 1, n)
    y = check(A, x)
    y_ref, bound = oracle.spmv(A, x)
    assert oracle.spmv_accept(y, y_ref, bound).all()


def test_unsorted_duplicates_and_non_finite_x():
    rng = np.random.default_rng(8)
    n = 100_000
    A = banded(rng.integers(6, 20, n), n, 9)
    A.col_idx[:] = A.col_idx[np.arange(A.nnz) ^ 1] if A.nnz % 2 == 0 else A.col_idx
    A.col_idx[5000:5004] = 17
    x = rng.uniform(-1, 1, n)
    x[[3, 5000, 99_990]] = [np.nan, np.inf, -np.inf]
    check(A, x)


def test_scattered_columns_keep_the_row_tiles():
    rng = np.random.default_rng(10)
    n = 160_000
    A = banded(np.full(n, 7), n, 11)
    A.col_idx[:] = rng.integers(0, n, A.nnz)
    check(A, rng.uniform(-1, 1, n), expect_jag=False)


@pytest.mark.parametrize("mode", [spmv.CG_FP64, spmv.CG_MIXED_FP32, spmv.CG_MIXED_FP32V, spmv.CG_PCG_JACOBI,
                                  spmv.CG_PCG_BF16])
def test_solves_on_jagged_products(mode):
    # products with the p.q and residual epilogues; more than 2^20 rows, so
    # that FP64 solves take them too
    A = mg.config1("rcm", m=102)
    assert A.n_rows > 1 << 20
    b = mg.uniform(A.n_rows, 12, 0)
    with spmv.Matrix.from_csr(A, fp32=True, bf16=True) as M, \
            spmv.Matrix.from_csr(A, fp32=True, bf16=True, params=ROW_TILES) as R:
        bd = torch.as_tensor(b, device=DEV)
        x, info = M.cg(bd, tol=1e-9, mode=mode)
        xr, ref = R.cg(bd, tol=1e-9, mode=mode)
    Ax, _ = oracle.spmv(A, x.cpu().numpy())
    assert np.linalg.norm(b - Ax) <= 1.05e-9 * np.linalg.norm(b)
    # both solutions lie within kappa * tol of the exact one (Gershgorin
    # bound: the diagonal exceeds the off-diagonals by 1e-3)
    kappa = 2 * A.values.max() / 1e-3
    assert float((x - xr).norm() / xr.norm()) <= 2 * kappa * 1e-9
    assert abs(info.iterations - ref.iterations) <= 0.1 * ref.iterations
