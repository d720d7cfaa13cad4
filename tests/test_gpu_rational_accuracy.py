"""GPU rational projected-matrix step: what its acceptance lets through.

An eigenvalue next to the imaginary axis with a tiny weight in e_1 hides behind a small
difference of the two members: the first matrices couple such a row to the first one by
2e-11, so that 1024 poles leave 2e-13 to 1.3e-12 of c while their members differ by 3e-12 to
7e-12, and only the larger set resolves it.  The others are the block process's own
matrices, whose eigenvalues nearly coincide in pairs.  Against the Schur sign; k steps of
rounding on entries whose relative changes c amplifies by at most `sens` (measured on the
oracle, at least 1) give the tolerance.
"""
import numpy as np
import pytest

from gpu_util import host, rel, say
from oracle.blockderiv import BlockOperator, block_tsl, link_direction_field
from oracle.sign import sign_schur
from oracle.wilson import WilsonOperator
from synthetic import random_links, z2_complex_source

pytestmark = pytest.mark.gpu

U = 2.2e-16


def _dense(a, b, g):
    return np.diag(a) + np.diag(b, -1) + np.diag(g, 1)


def _gpu_sign(a, b, g):
    from paper_1604_08057_amd import Context
    ctx = Context((2, 2, 2, 2), -2.0, 0.0)
    c, info = ctx.tridiag_sign(a, b, g)
    ctx.close()
    return host(c), info


def _sensitivity(a, b, g, want):
    rng = np.random.default_rng(0)
    h = 1e-9
    sens = 1.0
    for _ in range(4):
        n = [rng.normal(size=len(x)) for x in (a, b, g)]
        c = sign_schur(_dense(a * (1 + h * n[0]), b * (1 + h * n[1]), g * (1 + h * n[2])))[:, 0]
        sens = max(sens, rel(c, want) / h)
    return sens


@pytest.mark.parametrize("k", [2, 12, 40, 64])
def test_light_eigenvalue_next_to_the_axis(k):
    rng = np.random.default_rng(0)
    a = np.where(np.arange(k) < 1, rng.uniform(0.8, 1.2, k), rng.uniform(-1.2, -0.8, k)).astype(complex)
    a[1] = -1.5e-3 + 0.3j
    b, g = np.full(k - 1, 0.1), np.full(k - 1, 0.1 + 0j)
    if k > 2:
        b[1] = g[1] = 0.02
    b[0], g[0] = 2e-11, 0.1
    c, info = _gpu_sign(a, b, g)
    e = rel(c, sign_schur(_dense(a, b, g))[:, 0])
    say(f"rational sign, light eigenvalue k={k}: err {e:.2e}, steps {info.newton_iters}")
    assert e < 10 * k * U
    assert info.newton_iters == 2


@pytest.mark.parametrize("mu,k", [(0.0, 40), (0.2, 100), (0.4, 100)])
def test_block_process_matrix(mu, k):
    dims, V = (4, 4, 4, 4), 256
    rng = np.random.default_rng(7)
    links, psi = random_links(dims, 0.4, rng), z2_complex_source(V, rng)
    X = rng.normal(size=(3, 3)) + 1j * rng.normal(size=(3, 3))
    X = X + X.conj().T
    X -= np.trace(X) / 3 * np.eye(3)
    bop = BlockOperator(WilsonOperator(dims, -2.0, mu), links, link_direction_field(links, 3, 17, X), (V, 4, 3))
    T = block_tsl(bop, np.zeros(12 * V), psi, k)["T"]
    a, b, g = np.diag(T).copy(), np.diag(T, -1).real.copy(), np.diag(T, 1).copy()
    want = sign_schur(T)[:, 0]
    c, info = _gpu_sign(a, b, g)
    e = rel(c, want)
    tol = 10 * k * U * _sensitivity(a, b, g, want)
    say(f"rational sign, block process mu={mu} k={k}: err {e:.2e} (tol {tol:.1e}), steps {info.newton_iters}")
    assert e < tol
