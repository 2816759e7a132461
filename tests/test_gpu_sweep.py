"""Sweep tiles (the default plain product of scattered orderings with 2^22
entries and more over an x beyond an XCD's L2): the same bits as the
direct-gather row tiles (spmv_params.kernel = 1) in every precision."""
import numpy as np
import pytest

import meshgen as mg
import oracle

torch = pytest.importorskip("torch")
spmv = pytest.importorskip("paper_2107_12371_amd")

pytestmark = pytest.mark.gpu
DEV = "cuda"
ROW_TILES = {"kernel": 1}


def scattered(lens, n_cols, seed):
    """Rows of the given lengths over uniformly random columns (unsorted,
    duplicates possible)."""
    rng = np.random.default_rng(seed)
    rp = np.zeros(len(lens) + 1, np.int64)
    rp[1:] = np.cumsum(lens)
    return mg.CSR(len(lens), n_cols, rp.astype(np.int32), rng.integers(0, n_cols, rp[-1]).astype(np.int32),
                  rng.uniform(-1, 1, rp[-1]), 1)


def check(A, x, expect_sweep=True):
    with spmv.Matrix.from_csr(A, fp32=True, bf16=True) as M, \
            spmv.Matrix.from_csr(A, fp32=True, bf16=True, params=ROW_TILES) as R:
        assert (M.info["device_bytes"] > 1.3 * R.info["device_bytes"]) == expect_sweep
        for off in (0, 1):
            xd = torch.empty(A.n_cols + 1, dtype=torch.float64, device=DEV)[off:off + A.n_cols]
            xd.copy_(torch.as_tensor(x))
            xf = torch.empty(A.n_cols + 1, dtype=torch.float32, device=DEV)[off:off + A.n_cols]
            xf.copy_(xd)
            for f, v in (("apply", xd), ("apply_f32v", xd), ("apply_f32", xf), ("apply_bf16", xf)):
                a, b = getattr(M, f)(v).cpu().numpy(), getattr(R, f)(v).cpu().numpy()
                assert np.array_equal(a, b, equal_nan=True), (f, off)
        return M.apply(torch.as_tensor(x, device=DEV)).cpu().numpy()


@pytest.mark.parametrize("n,mean", [(1_000_003, 5), (500_001, 11), (1_700_000, 4)])
def test_random_columns(n, mean):
    # binary64 x of 8, 16 (n_cols > n) and 13.6 MB; FP32 x below, above and
    # above the limit; tiles of full rounds and their remainders
    rng = np.random.default_rng(n)
    lens = rng.integers(0, 2 * mean + 1, n)
    lens[1000:60_000] = 0  # more empty rows than a tile has lanes
    A = scattered(lens, max(n, 2_000_003 if mean == 11 else n), n)
    assert A.nnz >= 1 << 22
    x = rng.uniform(-1, 1, A.n_cols)
    y = check(A, x)
    y_ref, bound = oracle.spmv(A, x)
    assert oracle.spmv_accept(y, y_ref, bound).all()


def test_long_rows_and_non_finite_x():
    # rows near the row tiles' limit, long rows of one and several pieces, and
    # NaN / Inf in x
    rng = np.random.default_rng(2)
    n = 900_000
    lens = rng.integers(1, 10, n)
    lens[[0, 5, 400_000, n - 1]] = [2045, 2000, 60_000, 4096]
    A = scattered(lens, n, 3)
    x = rng.uniform(-1, 1, n)
    x[[7, 500_000, n - 1]] = [np.nan, np.inf, -np.inf]
    check(A, x)


@pytest.mark.parametrize("n,lens", [(600_000, 8), (1_000_000, 4)])
def test_small_x_or_few_entries_keep_the_row_tiles(n, lens):
    # x of 4.8 MB, and 4,000,000 entries
    A = scattered(np.full(n, lens), n, 4)
    check(A, np.random.default_rng(1).uniform(-1, 1, n), expect_sweep=False)


def test_solve_on_a_scattered_ordering():
    # the solvers' epilogues keep the row tiles; the polynomial's plain
    # products take the sweep tiles where their x is large enough
    A = mg.config1("random", m=118)
    b = mg.uniform(A.n_rows, 12, 0)
    with spmv.Matrix.from_csr(A, bf16=True) as M, spmv.Matrix.from_csr(A, bf16=True, params=ROW_TILES) as R:
        bd = torch.as_tensor(b, device=DEV)
        for mode in (spmv.CG_FP64, spmv.CG_PCG_BF16):
            x, info = M.cg(bd, tol=1e-9, mode=mode)
            xr, ref = R.cg(bd, tol=1e-9, mode=mode)
            # same partials, same products: same iterates
            assert info.iterations == ref.iterations and torch.equal(x, xr)
