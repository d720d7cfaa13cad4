"""GPU Ritz summary of the sign calls where the two lanes that share a root once parted.

At large mu the last correction of a root is cancellation, and a pair of lanes that did not
form it with the same bits could settle in one lane and go on in the other, on half the
matrix: roots that never settle or are no eigenvalues.  The named cases raised the unsettled
flag in that way; the others sweep sizes whose blocks one workgroup settles, alone (k <= 64)
and as starting points of the larger ones.  Against LAPACK on the call's own projected
matrix: an eigenvalue of condition number c is good to k u c |T| in either, so ten times that
(the worst c of the matrix, at least 1e-13 |T|) separates a wrong root from rounding.
"""
import numpy as np
import pytest
import scipy.linalg

from gpu_util import dev, say
from synthetic import random_links, z2_complex_source

pytestmark = pytest.mark.gpu

DIMS = (2, 2, 2, 4)


def _check(mu, seed, ks):
    from paper_1604_08057_amd import Context
    rng = np.random.default_rng(seed)
    ctx = Context(DIMS, -2.0, mu)
    ctx.set_links(dev(random_links(DIMS, 0.4, rng)))
    psi = dev(z2_complex_source(32, rng))
    for k in ks:
        _, info = ctx.sign(psi, k)
        T, _ = ctx.lanczos_matrix(psi, k)
        T = T[:info.k_used, :info.k_used]
        lam, vl, vr = scipy.linalg.eig(T, left=True, right=True)
        cond = (1.0 / np.abs((vl.conj() * vr).sum(0))).max()
        nrm = np.abs(T).sum(1).max()
        err = abs(info.min_abs_re_ritz - np.abs(lam.real).min()) / nrm
        tol = max(1e-13, 10 * k * 2.2e-16 * cond)
        say(f"ritz pair mu={mu} seed={seed} k={k}: err {err:.1e} (tol {tol:.1e}) flags {info.flags}")
        assert err < tol
        assert not info.flags & 4
    ctx.close()


@pytest.mark.parametrize("mu,seed,k", [(0.8, 18, 16), (1.0, 27, 64), (1.4, 8, 30), (1.4, 15, 64), (1.4, 30, 41),
                                       (1.6, 35, 64)])
def test_lanes_of_a_root_agree(mu, seed, k):
    _check(mu, seed, [k])


@pytest.mark.parametrize("mu", [0.8, 1.2, 1.6])
def test_ritz_summary_at_large_mu(mu):
    for seed in range(60, 70):
        _check(mu, seed, [16, 30, 50, 64, 90])
