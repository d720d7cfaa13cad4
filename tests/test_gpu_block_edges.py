"""GPU block-matrix process at the edges of its two kernels' layouts.

Less than a site block, a ragged last block, both stencil layouts around 8192 sites, an
extent of 2 (where the link's two sites are neighbours twice over), each direction, links
that wrap in space and across the antiperiodic boundary, and k = 1 (no recurrence), from a
general source (x1, x2) against the oracle's block process; a zero source.  At these sizes
the recursion amplifies rounding by less than 1e3, so 1e-12 separates it from a wrong term.
"""
import numpy as np
import pytest
import torch

from gpu_util import dev, host, rel, say
from oracle import blockderiv as BD
from oracle import grad as GR
from oracle.wilson import WilsonOperator
from synthetic import random_links, z2_complex_source

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,k", [((2, 2, 2, 2), 6), ((3, 2, 5, 2), 12), ((5, 3, 4, 7), 1), ((16, 8, 8, 8), 10),
                                    ((11, 9, 9, 10), 10), ((16, 8, 8, 9), 8)])
def test_block_process_edges(dims, k):
    from paper_1604_08057_amd import Context
    rng = np.random.default_rng(sum(dims) + k)
    V = int(np.prod(dims))
    U = random_links(dims, 0.4, rng)
    x1, x2 = z2_complex_source(V, rng), z2_complex_source(V, rng)
    op = WilsonOperator(dims, -2.0, 0.3)
    ctx = Context(dims, -2.0, 0.3)
    ctx.set_links(dev(U))
    for nu in range(4) if V < 1000 else (int(rng.integers(0, 4)), 3):
        site = V - 1 if nu % 2 else int(rng.integers(0, V))   # the last site wraps in every direction
        X = GR.su3_direction(rng)
        bop = BD.BlockOperator(op, U, BD.link_direction_field(U, nu, site, X), x2.shape)
        ref = BD.block_tsl(bop, x1, x2, k)
        y1, y2, info = ctx.block_sign(nu, site, X, dev(x2), k, x1=dev(x1))
        e1, e2 = rel(host(y1), ref["y1"]), rel(host(y2), ref["y2"])
        say(f"block process {dims} k={k} link ({nu}, {site}): errs {e1:.1e} {e2:.1e} k_used {info.k_used}")
        assert info.k_used == k and e1 < 1e-12 and e2 < 1e-12
    y1, y2, info = ctx.block_sign(0, 0, np.eye(3), torch.zeros_like(dev(x2)), k)
    ctx.close()
    assert info.k_used == 0 and not host(y1).any() and not host(y2).any()
