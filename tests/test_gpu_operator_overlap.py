"""Operator calls whose output shares bytes with the input: the bits of the call on arrays
apart, for both directions of the shift, one site, half a field and all but one site, on a
lattice of one launch round, a ragged one and a marching one.
"""
import ctypes

import numpy as np
import pytest
import torch

from gpu_util import dev, say
from synthetic import random_links, z2_complex_source

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32links", "mixed"])
@pytest.mark.parametrize("dims", [(6, 4, 8, 10), (9, 7, 10, 11), (16, 16, 16, 16)])
@pytest.mark.parametrize("entry", ["tslov_apply_dw", "tslov_apply_h", "tslov_apply_h_noalloc"])
def test_overlapping_output(dims, precision, entry):
    from paper_1604_08057_amd import Context
    rng = np.random.default_rng(5)
    V = int(np.prod(dims))
    ctx = Context(dims, -2.0, 0.3, precision=precision)
    ctx.set_links(dev(random_links(dims, 0.4, rng)))
    x = dev(z2_complex_source(V, rng))
    call = getattr(ctx.lib, entry)
    ptr = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    want = torch.empty_like(x)
    assert call(ctx.handle, ptr(x), ptr(want), 0) == 0
    buf = torch.empty((2 * V, 4, 3), dtype=torch.complex128, device="cuda")
    for shift in (1, V // 2, V - 1):
        for lo, hi in ((0, shift), (shift, 0)):
            src, out = buf[lo:lo + V], buf[hi:hi + V]
            src.copy_(x)
            assert call(ctx.handle, ptr(src), ptr(out), 0) == 0
            torch.cuda.synchronize()
            assert torch.equal(out, want), (shift, lo)
    src.copy_(x)
    assert call(ctx.handle, ptr(src), ptr(src), 0) != 0   # the same array stays refused
    ctx.close()
    say(f"overlapping output {entry} {dims} {precision}")
