"""The link currents of a batch, summed over its sources, against the gradients they project.

j(x, nu) = mean over sources of -Im tr(G_s^H U_nu(x)) with G_s = dS_s/dU of
S_s = Re <g5 xi_s|sgn(H)|xi_s>: the batched derivative gives the G_s, torch the projection.
The contraction takes four sources at a time and 64 sites per block: one source, a part of a
group, a whole one, a group and a rest, more groups; whole and ragged last blocks.  Both sides
use the same partial sums in double precision, so 1e-12 of the largest current separates a
misplaced term from rounding.
"""
import numpy as np
import pytest
import torch

from gpu_util import dev, say
from synthetic import random_links, z2_complex_source

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 3, 4, 5, 9])
@pytest.mark.parametrize("dims", [(3, 3, 3, 4), (4, 4, 4, 4)])
def test_current_is_projected_gradient(dims, n):
    from paper_1604_08057_amd import Context
    r = np.random.default_rng(10 * n + dims[0])
    V = int(np.prod(dims))
    U = dev(random_links(dims, 0.4, r))
    xi = dev(np.stack([z2_complex_source(V, r) for _ in range(n)]))
    ks = [10 + (i % 3) for i in range(n)]
    ctx = Context(dims, -2.0, 0.3)
    ctx.set_links(U)
    j = ctx.current_estimate(xi, ks)[0]
    g5xi = xi.clone()
    g5xi[:, :, 2:] *= -1
    _, dU, *_ = ctx.sign_grad_batched(g5xi, xi, ks)
    ctx.close()
    u = U.reshape(4, V, 3, 3)
    ref = -(dU.reshape(n, 4, V, 3, 3).conj() * u).sum((-1, -2)).imag.mean(0)
    err = float((j - ref).abs().max() / ref.abs().max())
    say(f"current of {n} sources on {dims}: {err:.2e}")
    assert err < 1e-12
