"""GPU Ritz summary of the sign calls (min |Re theta|, |T|_inf) at the sizes whose rows a
thread loads in three and in four parts, up to the largest, against LAPACK on the call's own
projected matrix.  An eigenvalue of condition number c is good to k u c |T| in either, so ten
times that (the worst c of the matrix) separates a wrong root from rounding.
"""
import numpy as np
import pytest
import scipy.linalg

from gpu_util import dev, say
from synthetic import random_links, z2_complex_source

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [768, 769, 1023, 1024])
def test_ritz_summary_of_long_sign_call(k):
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
    lam, vl, vr = scipy.linalg.eig(T, left=True, right=True)
    cond = (1.0 / np.abs((vl.conj() * vr).sum(0))).max()
    nrm = np.abs(T).sum(1).max()
    err = abs(info.min_abs_re_ritz - np.abs(lam.real).min()) / nrm
    tol = 10 * k * 2.2e-16 * cond
    say(f"ritz k={k}: err {err:.1e} (tol {tol:.1e}) flags {info.flags}")
    assert err < tol
    assert abs(info.norm_T - nrm) < 1e-13 * nrm
    assert not info.flags & 4
