"""GPU block-matrix process from sources far from unit size, in both stencil layouts.

Scaling the source by a power of two scales every sum of the process exactly, so the result
is the unscaled one's, bit for bit, times that power.
"""
import numpy as np
import pytest
import torch

from gpu_util import dev, say
from synthetic import random_links, z2_complex_source

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(4, 3, 4, 5), (16, 8, 8, 9)])
@pytest.mark.parametrize("power", [-332, -270, 270, 332])
def test_block_process_scales_with_the_source(dims, power):
    from paper_1604_08057_amd import Context
    rng = np.random.default_rng(3)
    V = int(np.prod(dims))
    ctx = Context(dims, -2.0, 0.3)
    ctx.set_links(dev(random_links(dims, 0.4, rng)))
    x1, x2 = dev(z2_complex_source(V, rng)), dev(z2_complex_source(V, rng))
    X = rng.normal(size=(3, 3)) + 1j * rng.normal(size=(3, 3))
    X = X + X.conj().T
    scale = 2.0 ** power
    for a in (None, x1):
        want = ctx.block_sign(2, V // 3, X, x2, 12, x1=a)
        got = ctx.block_sign(2, V // 3, X, x2 * scale, 12, x1=None if a is None else a * scale)
        assert got[2].k_used == 12
        for g, w in zip(got[:2], want[:2]):
            assert torch.equal(g, w * scale)
    ctx.close()
    say(f"block process scaled by 2^{power} on {dims}")
