"""The Jacobi-preconditioned solve takes one z = D^-1 r, rounded, for r.z and
for p = z + beta p: the iterates equal the recurrence with a stored z bit for
bit.  Systems of two unknowns, so that every dot product is one addition of
two rounded products and its order cannot matter; the recurrence is formed
here in exact arithmetic rounded where the solver rounds."""
from fractions import Fraction

import numpy as np
import pytest

torch = pytest.importorskip("torch")
spmv = pytest.importorskip("paper_2107_12371_amd")

pytestmark = pytest.mark.gpu


def fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))


def stored_z(A, b, iterations):
    """x after so many iterations from x = 0."""
    dinv = [1.0 / A[0][0], 1.0 / A[1][1]]
    x, r = [0.0, 0.0], list(b)
    z = [dinv[i] * r[i] for i in range(2)]
    rho = r[0] * z[0] + r[1] * z[1]
    p = list(z)
    for _ in range(iterations):
        q = [A[i][0] * p[0] + A[i][1] * p[1] for i in range(2)]
        alpha = rho / (p[0] * q[0] + p[1] * q[1])
        x = [fma(alpha, p[i], x[i]) for i in range(2)]
        r = [fma(-alpha, q[i], r[i]) for i in range(2)]
        z = [dinv[i] * r[i] for i in range(2)]
        rz = r[0] * z[0] + r[1] * z[1]
        p = [fma(rz / rho, p[i], z[i]) for i in range(2)]
        rho = rz
    return x


def test_iterates_equal_the_stored_z_recurrence():
    rng = np.random.default_rng(5)
    ptr, col = np.array([0, 2, 4], np.int32), np.array([0, 1, 0, 1], np.int32)
    for trial in range(40):
        off = -rng.uniform(0.5, 1.5)
        A = [[2.0 + rng.uniform(), off], [off, 2.0 + rng.uniform()]]
        b = rng.uniform(-1, 1, 2)
        with spmv.Matrix(2, 2, ptr, col, np.array(A).reshape(-1)) as M:
            for iterations in (1, 2):
                x, info = M.cg(torch.as_tensor(b, device="cuda"), tol=0.0, max_iter=iterations,
                               mode=spmv.CG_PCG_JACOBI, raise_on_error=False)
                want = stored_z(A, [float(v) for v in b], iterations)
                assert info.iterations == iterations
                assert x.cpu().tolist() == want, (trial, iterations)
