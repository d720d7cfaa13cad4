"""The direction-split pair kernels give the bits of the colour split.

Three sources of uneven Krylov size on lattices whose site blocks go out in one round of
workgroups, so that a launch with one entry per workgroup takes the direction split; two
entries per workgroup (forced) take the colour split.  Whole and ragged last site blocks,
odd extents, a lattice whose last steps (one source left) take the colour split, but for the
reverse pair with float32 links, float64 and float32 links, stored and regenerated Krylov vectors.  Both add the
same products in the same order, so every output is compared bit for bit, but for the
link gradient of the regenerated run, whose sum over 15 steps is cut elsewhere (1e-13).
"""
import numpy as np
import pytest
import torch

from gpu_util import dev, host, rel
from synthetic import random_links, z2_complex_source

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32links"])
@pytest.mark.parametrize("dims", [(9, 10, 10, 10), (8, 8, 8, 17), (13, 11, 7, 9), (14, 14, 14, 14)])
def test_direction_split_bits(dims, precision):
    from paper_1604_08057_amd import Context
    r = np.random.default_rng(sum(dims))
    V = int(np.prod(dims))
    U = dev(random_links(dims, 0.4, r))
    psi = dev(np.stack([z2_complex_source(V, r) for _ in range(3)]))
    eta = dev(np.stack([z2_complex_source(V, r) for _ in range(3)]))
    out = {}
    for ns in (1, 2):
        ctx = Context(dims, -2.0, 0.3, precision=precision)
        ctx.set_links(U)
        ctx.set_pair_ns(ns)
        S, dU, dpsi, _, y = ctx.sign_grad_batched(eta, psi, [18, 15, 17], want_dpsi=True, want_y=True)
        out[ns] = np.asarray(S), dU, dpsi, y
        if ns == 1:   # one source, vectors regenerated in segments of seven steps
            S1, dU1, dpsi1, _ = ctx.sign_grad(eta[1], psi[1], 15, want_dpsi=True, recompute=7)
        ctx.close()
    a, b = out[1], out[2]
    assert np.array_equal(a[0], b[0])
    for x, z in zip(a[1:], b[1:]):
        assert torch.isfinite(torch.view_as_real(x)).all() and torch.equal(x, z)
    assert S1 == b[0][1] and torch.equal(dpsi1, b[2][1])
    assert rel(host(dU1), host(b[1][1])) < 1e-13
