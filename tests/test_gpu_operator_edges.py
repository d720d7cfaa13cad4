"""GPU operator on canonical spinors at the edges of its tiles and of its dispatch.

One site block and less, ragged last blocks, both sides of the colour grid's range (8192
sites), and marching lattices (x, y, z volumes in multiples of 1024 sites) with every
chunk length of an odd and an even time extent, in the three precisions, D_w, D_w^dag, H
and H^dag, against the oracle.  Each output component is a sum of 8 hops of 3 complex
products, so the error relative to the largest component is a few tens of roundings:
1e-14 in float64 and 100 * 2^-24 in float32; float32 links are compared with the oracle on
the rounded links.
"""
import numpy as np
import pytest
import torch

from gpu_util import dev, host, rel_max, say
from oracle.wilson import WilsonOperator
from synthetic import random_links

pytestmark = pytest.mark.gpu

DIMS = [(2, 2, 2, 2), (3, 3, 3, 3), (4, 4, 4, 4), (5, 13, 2, 3), (16, 8, 8, 8), (13, 10, 9, 7), (11, 9, 9, 10),
        (16, 8, 8, 9), (16, 16, 8, 6)]


@pytest.mark.parametrize("precision", ["fp64", "fp32links", "mixed"])
@pytest.mark.parametrize("dims", DIMS)
def test_operator_edges(dims, precision):
    from paper_1604_08057_amd import Context
    rng = np.random.default_rng(sum(dims))
    V = int(np.prod(dims))
    U = random_links(dims, 0.5, rng)
    x = rng.standard_normal((V, 4, 3)) + 1j * rng.standard_normal((V, 4, 3))
    ctx = Context(dims, -2.0, 0.3, precision=precision)
    ctx.set_links(dev(U))
    op = WilsonOperator(dims, -2.0, 0.3)
    Ut = torch.from_numpy(U if precision == "fp64" else U.astype(np.complex64).astype(np.complex128))
    xt = torch.from_numpy(x)
    want = {"dw": op.dw(Ut, xt), "dw_dag": op.dw_dag(Ut, xt), "h": op.h(Ut, xt), "h_dag": op.h_dag(Ut, xt)}
    xd = dev(x)
    chunks = [T for T in range(1, dims[3] + 1) if dims[3] % T == 0] if dims[0] * dims[1] * dims[2] % 1024 == 0 else [0]
    tol = 100 * 2.0 ** -24 if precision == "mixed" else 1e-14
    worst = 0.0
    first = {}
    for T in chunks:
        ctx.set_apply_chunk(T)
        got = {"dw": ctx.apply_dw(xd), "dw_dag": ctx.apply_dw(xd, dagger=True), "h": ctx.apply_h(xd),
               "h_dag": ctx.apply_h(xd, dagger=True)}
        for name, y in got.items():
            worst = max(worst, rel_max(host(y), want[name].numpy()))
            assert torch.equal(y, first.setdefault(name, y)), (T, name)   # no chunk length changes a bit
    ctx.close()
    say(f"operator edges {dims} {precision} chunks {chunks}: rel max err {worst:.1e}")
    assert worst < tol
