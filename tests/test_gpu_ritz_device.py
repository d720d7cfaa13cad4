"""GPU Ritz summary of the sign calls (min |Re theta|, |T|_inf) against LAPACK.

Sizes around the leaf of the divide and conquer, its first splits, a wavefront, the longest
block one workgroup sweeps (64) and sizes whose rows a thread loads in one, two and three
parts; Krylov spaces longer than the lattice has components, whose close copies of one
eigenvalue settle slowly, so that the first sixteen sweeps at the full size do not do; T_k is the call's own projected matrix.
The eigenvalues of these matrices have condition numbers below 1e4, so 1e-10 relative to
|T| separates a wrong root from rounding.
"""
import numpy as np
import pytest

from gpu_util import dev, say
from synthetic import random_links, z2_complex_source

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [1, 2, 23, 24, 25, 26, 49, 63, 64, 65, 129, 300, 512, 513])
def test_ritz_summary_of_sign_call(k):
    from paper_1604_08057_amd import Context
    dims = (6, 6, 5, 6)
    rng = np.random.default_rng(k)
    ctx = Context(dims, -2.0, 0.2)
    ctx.set_links(dev(random_links(dims, 0.4, rng)))
    psi = dev(z2_complex_source(1080, rng))
    _, info = ctx.sign(psi, k)
    T, _ = ctx.lanczos_matrix(psi, k)
    ctx.close()
    assert info.k_used == k
    lam = np.linalg.eigvals(T)
    nrm = np.abs(T).sum(1).max()
    say(f"ritz k={k}: min |Re| {info.min_abs_re_ritz:.12e} (LAPACK {np.abs(lam.real).min():.12e}) flags {info.flags}")
    assert abs(info.min_abs_re_ritz - np.abs(lam.real).min()) < 1e-10 * nrm
    assert abs(info.norm_T - nrm) < 1e-13 * nrm
    assert not info.flags & 4


@pytest.mark.parametrize("dims,k", [((2, 2, 2, 2), 250), ((2, 2, 2, 2), 330), ((2, 2, 2, 4), 500)])
def test_ritz_summary_of_clustered_values(dims, k):
    from paper_1604_08057_amd import Context
    rng = np.random.default_rng(k)
    V = int(np.prod(dims))
    ctx = Context(dims, -2.0, 0.2)
    ctx.set_links(dev(random_links(dims, 0.4, rng)))
    psi = dev(z2_complex_source(V, rng))
    _, info = ctx.sign(psi, k)
    T, _ = ctx.lanczos_matrix(psi, k)
    ctx.close()
    T = T[:info.k_used, :info.k_used]
    lam = np.linalg.eigvals(T)
    nrm = np.abs(T).sum(1).max()
    say(f"ritz {dims} k={k}: min |Re| {info.min_abs_re_ritz:.12e} (LAPACK {np.abs(lam.real).min():.12e})")
    assert abs(info.min_abs_re_ritz - np.abs(lam.real).min()) < 1e-10 * nrm
    assert not info.flags & 4
