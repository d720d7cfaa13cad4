"""GPU rational (partial-fraction) projected-matrix step of the sign calls.

c = sgn(T) e_1 of tridiagonal matrices with a known gap to the imaginary axis against the
Schur sign, at the smallest sizes, around a wavefront and at the largest size; the gap
decides the route: one pole set, the larger one, or the Newton iteration.  The matrices
are real symmetric plus a multiple of i (normal), so the sign's condition number is at
most 2 |T| / gap and a backward error of 10 k u gives the tolerance.
"""
import numpy as np
import pytest

from gpu_util import host, rel, say
from oracle.sign import sign_schur

pytestmark = pytest.mark.gpu


def _tridiagonal(k, gap, rng):
    """Jacobi matrix with eigenvalues in +-[gap, 2], one of them at gap (Lanczos on a
    diagonal matrix, orthogonalised twice)."""
    lam = rng.uniform(gap, 2.0, k) * rng.choice([-1.0, 1.0], k)
    lam[0] = gap
    Q = np.zeros((k, k))
    q = rng.uniform(0.5, 1.5, k)
    q /= np.linalg.norm(q)
    a, b = np.zeros(k), np.zeros(max(k - 1, 0))
    for j in range(k):
        Q[:, j] = q
        r = lam * q
        a[j] = q @ r
        for _ in range(2):
            r -= Q[:, :j + 1] @ (Q[:, :j + 1].T @ r)
        if j + 1 < k:
            b[j] = np.linalg.norm(r)
            q = r / b[j]
    return a, b


@pytest.mark.parametrize("k,gap,route", [(1, 0.1, 1), (2, 0.1, 1), (3, 0.1, 1), (64, 0.1, 1), (65, 0.1, 1),
                                         (400, 0.1, 1), (1024, 0.2, 1), (65, 0.006, 2), (65, 1e-5, 3)])
def test_rational_sign_step(k, gap, route):
    from paper_1604_08057_amd import Context
    a, b = _tridiagonal(k, gap, np.random.default_rng(k))
    T = np.diag(a + 0.3j) + np.diag(b, -1) + np.diag(b, 1)
    ctx = Context((2, 2, 2, 2), -2.0, 0.0)
    c, info = ctx.tridiag_sign(a + 0.3j, b, b)
    ctx.close()
    e = rel(host(c), sign_schur(T)[:, 0])
    tol = 10 * k * 2.2e-16 * 2 * np.linalg.norm(T, 2) / gap
    say(f"rational sign k={k} gap={gap}: err {e:.2e} (tol {tol:.1e}), steps {info.newton_iters}")
    assert e < tol
    assert min(info.newton_iters, 3) == route
