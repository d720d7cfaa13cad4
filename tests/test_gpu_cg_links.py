"""The link-resident operator form of the shifted solves at the edges of its blocks and chunks.

A block of it serves 64 sites and, once the chip is full, several systems: whole and
ragged site blocks, chunks of one, of a few and of more systems than a block takes at
once, systems that freeze at different iterations.  Reference: the colour split, which
the small lattices of test_gpu_deflated_grad check against the dense oracle.  The
shifts lie outside the spectrum (|H| <= 1 + 8 kappa cosh(mu) < 3.2, |lambda| >= 6:
condition below 4), so two solutions to a relative residual of 1e-13 agree to
2 * 4 * 1e-13, and S, dS/dU and dS/dpsi, linear in them, to 1e-11 with room for the
norms of the factors.
"""
import numpy as np
import pytest
import torch

from gpu_util import dev, host, rel, say
from synthetic import random_links, z2_complex_source

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,l", [((2, 2, 2, 2), 1), ((8, 8, 8, 8), 20), ((9, 9, 9, 9), 17), ((4, 4, 4, 2), 33),
                                    ((16, 16, 16, 8), 33)])
def test_link_resident_solves(dims, l):
    from paper_1604_08057_amd import Context
    mass, mu, k = -2.0, 0.3, 8
    r = np.random.default_rng(sum(dims) + l)
    V = int(np.prod(dims))
    U = random_links(dims, 0.4, r)
    psi, eta = dev(z2_complex_source(V, r)), dev(z2_complex_source(V, r))
    g = torch.Generator().manual_seed(l)
    R = torch.randn((l, V, 4, 3), dtype=torch.complex128, generator=g).to("cuda") / np.sqrt(12.0 * V)
    L = torch.randn((l, V, 4, 3), dtype=torch.complex128, generator=g).to("cuda") / np.sqrt(12.0 * V)
    lam = np.array([(-1) ** i * (6.0 + 40.0 * i / l) + 0.5j for i in range(l)])
    out = {}
    ctx = Context(dims, mass, mu)
    ctx.set_links(dev(U))
    defl = ctx.deflation(R, L, lam)
    for form in (1, 3):
        ctx.set_cg_operator(form)
        S, dU, dpsi, info = ctx.sign_grad(eta, psi, k, want_dpsi=True, defl=defl)
        out[form] = S, host(dU), host(dpsi), info.cg_iters
    ctx.close()
    a, b = out[1], out[3]
    eS, eG, eP = abs(b[0] - a[0]) / abs(a[0]), rel(b[1], a[1]), rel(b[2], a[2])
    say(f"link-resident solves {dims} l={l}: S {eS:.2e} G {eG:.2e} dpsi {eP:.2e}, iterations {a[3]} {b[3]}")
    assert eS < 1e-11 and eG < 1e-11 and eP < 1e-11
