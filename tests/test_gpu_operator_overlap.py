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


def test_overlapping_output_captured():
    """The allocation-free entry as a graph, its copy of the input included, replayed on new inputs."""
    from paper_1604_08057_amd import Context
    dims, V = (16, 8, 8, 8), 8192
    rng = np.random.default_rng(6)
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        ctx = Context(dims, -2.0, 0.3)
        ctx.set_links(dev(random_links(dims, 0.4, rng)))
        xs = [dev(z2_complex_source(V, rng)) for _ in range(3)]
        wants = [ctx.apply_h(x) for x in xs]
        buf = torch.zeros((V + 1, 4, 3), dtype=torch.complex128, device="cuda")
    st.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=st):
        rc = ctx.lib.tslov_apply_h_noalloc(ctx.handle, ctypes.c_void_p(buf.data_ptr()),
                                           ctypes.c_void_p(buf[1:].data_ptr()), 0)
    assert rc == 0
    for x, want in zip(xs, wants):
        buf[:V].copy_(x)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(buf[1:], want)
    del graph
    ctx.close()
