"""Performance cases of the public entry points, over the range a user runs them.

The library is used in four ways, and the cases cover each of them: the Wilson operator
on its own (a solver or an eigensolver calls it thousands of times on one field), the
overlap sign of a vector, the derivative with respect to every link (one source, many
noise sources in one call, with regenerated Krylov vectors, through torch's autograd,
projected on the link current, deflated by eigenpairs), and the block-matrix derivative
of one link parameter.  Lattices run from 4^4, where a call is a handful of launches,
over the ragged ones of the tests, to 16^4 (whole derivatives) and 32^4 (the operator).

Links are random SU(3) matrices exp(i s sum_a c_a lambda_a), sources are Z2-complex
noise, mass -2, kappa = 1/4: what the benchmark and the tests run.  Krylov sizes of the
derivatives stop at 180: beyond that the unreorthogonalised recursion amplifies the
last bit of any inner product to more than 1e-9 of the derivative, and two correct
programs can no longer be told from a wrong one by their outputs.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1604_08057_amd import Context, SignGrad

MASS = -2.0


def listed():
    return [
        # the operator as an eigensolver calls it on a small field: launches and latency
        dict(name="apply_h 8^4", kind="apply_h", nx=8, ny=8, nz=8, nt=8, precision="fp64", mu=0.2, dagger=False),
        # the adjoint operator on the ragged batching lattice in the float32 mode
        dict(name="apply_dw_dag 18^3x6 fp32", kind="apply_dw", nx=18, ny=18, nz=18, nt=6, precision="mixed", mu=0.5,
             dagger=True),
        # the operator on a production-size field, bound by memory
        dict(name="apply_h 32^4", kind="apply_h", nx=32, ny=32, nz=32, nt=32, precision="fp64", mu=0.3, dagger=False),
        # D_ov psi on a small field: a chain of several hundred dependent launches
        dict(name="overlap 8^4 k200", kind="overlap", nx=8, ny=8, nz=8, nt=8, precision="fp64", mu=0.2, k=200),
        # sgn(H) psi at the paper's lattice and full Krylov size
        dict(name="sign 14^4 k400", kind="sign", nx=14, ny=14, nz=14, nt=14, precision="fp64", mu=0.3, k=400),
        # one optimisation step through torch.autograd on a tiny field
        dict(name="autograd 4^4 k64", kind="autograd", nx=4, ny=4, nz=4, nt=4, precision="fp64", mu=0.3, k=64),
        # the derivative of one source on a small field, with its output and source gradient
        dict(name="grad 8^4 k150", kind="grad", nx=8, ny=8, nz=8, nt=8, precision="fp64", mu=0.2, k=150),
        # many noise sources with uneven Krylov sizes in one call: the benchmark's workload,
        # with fewer sources and smaller sizes (memory for several states, and see above)
        dict(name="batch 18^3x6", kind="batch", nx=18, ny=18, nz=18, nt=6, precision="fp64", mu=0.5, nsrc=6, klo=80,
             khi=180),
        # the overlap derivative at 16^4 with regenerated Krylov vectors and float32 links
        dict(name="overlap_grad 16^4 recompute", kind="overlap_grad", nx=16, ny=16, nz=16, nt=16,
             precision="fp32links", mu=0.3, k=100, recompute=20),
        # the stochastic link current with its divergence and Ward check
        dict(name="current 10^4", kind="current", nx=10, ny=10, nz=10, nt=10, precision="fp64", mu=0.3, nsrc=8, klo=40,
             khi=100),
        # the derivative deflated by eigenpairs, whose motion needs 2l shifted solves
        dict(name="deflated grad 16^3x4 l8", kind="deflated", nx=16, ny=16, nz=16, nt=4, precision="fp64", mu=0.3,
             k=60, l=8),
        # the block-matrix derivative of one link parameter
        dict(name="block_sign 8^4 k100", kind="block", nx=8, ny=8, nz=8, nt=8, precision="fp64", mu=0.2, k=100),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _dims(rng, lo, hi, most):
    """Four extents in [lo, hi], even and odd, with at most `most` sites."""
    while True:
        d = [_log_int(rng, lo, hi) for _ in range(4)]
        if d[0] * d[1] * d[2] * d[3] <= most:
            return dict(zip(("nx", "ny", "nz", "nt"), d))


def draw(rng):
    kind = rng.choice(["apply_h", "apply_dw", "apply_h", "overlap", "sign", "autograd", "grad", "batch",
                       "overlap_grad", "current", "deflated", "block"])
    mu = rng.choice([0.0, 0.2, 0.3, 0.5])
    if kind in ("apply_h", "apply_dw"):
        big = rng.random() < 0.5
        return dict(kind=kind, **(_dims(rng, 12, 40, 32 ** 4) if big else _dims(rng, 3, 16, 16 ** 4)),
                    precision=rng.choice(["fp64", "fp32links", "mixed"]), mu=mu, dagger=rng.random() < 0.5)
    if kind in ("overlap", "sign"):
        d = _dims(rng, 4, 20, 14 ** 4)
        return dict(kind=kind, **d, precision=rng.choice(["fp64", "fp64", "fp32links", "mixed"]), mu=mu,
                    k=_log_int(rng, 16, 400))
    if kind == "autograd":
        return dict(kind=kind, **_dims(rng, 3, 8, 8 ** 4), precision="fp64", mu=mu, k=_log_int(rng, 16, 100))
    if kind == "grad":
        return dict(kind=kind, **_dims(rng, 4, 18, 14 ** 4), precision=rng.choice(["fp64", "fp32links"]), mu=mu,
                    k=_log_int(rng, 16, 150))
    if kind == "batch":
        klo = _log_int(rng, 16, 80)
        return dict(kind=kind, **_dims(rng, 6, 18, 18 ** 3 * 6), precision=rng.choice(["fp64", "fp32links"]), mu=mu,
                    nsrc=rng.randint(2, 6), klo=klo, khi=_log_int(rng, klo, 160))
    if kind == "overlap_grad":
        return dict(kind=kind, **_dims(rng, 6, 16, 16 ** 4), precision=rng.choice(["fp64", "fp32links"]), mu=mu,
                    k=_log_int(rng, 24, 100), recompute=rng.choice([0, 5, 10, 20]))
    if kind == "current":
        klo = _log_int(rng, 16, 60)
        return dict(kind=kind, **_dims(rng, 4, 12, 10 ** 4), precision="fp64", mu=mu, nsrc=rng.randint(2, 8), klo=klo,
                    khi=_log_int(rng, klo, 100))
    if kind == "deflated":
        d = dict(zip(("nx", "ny", "nz", "nt"), rng.choice([(8, 8, 8, 8), (16, 16, 8, 4), (16, 8, 8, 8), (6, 10, 8, 9),
                                                           (12, 11, 6, 5), (16, 16, 16, 4)])))
        return dict(kind=kind, **d, precision="fp64", mu=rng.choice([0.2, 0.3, 0.5]), k=_log_int(rng, 16, 60),
                    l=rng.randint(2, 8))
    return dict(kind="block", **_dims(rng, 4, 10, 8 ** 4), precision="fp64", mu=mu, k=_log_int(rng, 16, 100))


# ------------------------------------------------------------------ inputs
def _device():
    return torch.device("cuda", torch.cuda.current_device()) if torch.cuda.is_available() else torch.device("cpu")


def _geometry(case):
    d = (case["nx"], case["ny"], case["nz"], case["nt"])
    return d, d[0] * d[1] * d[2] * d[3]


def _mm(a, b):
    """Product of 3x3 matrices (any batch), elementwise."""
    return (a[..., :, :, None] * b[..., None, :, :]).sum(-2)


def _su3(n, spread, gen, dev):
    """n SU(3) matrices exp(i spread sum_a c_a lambda_a), c_a ~ N(0, 1)."""
    z = spread * torch.randn(n, 8, generator=gen, dtype=torch.float64, device=dev)
    h = torch.zeros(n, 3, 3, dtype=torch.complex128, device=dev)
    s3 = z[:, 7] / math.sqrt(3.0)
    h[:, 0, 0], h[:, 1, 1], h[:, 2, 2] = (z[:, 2] + s3).to(h.dtype), (s3 - z[:, 2]).to(h.dtype), (-2 * s3).to(h.dtype)
    for (a, b), (p, q) in (((0, 1), (0, 1)), ((0, 2), (3, 4)), ((1, 2), (5, 6))):
        h[:, a, b] = torch.complex(z[:, p], -z[:, q])
        h[:, b, a] = torch.complex(z[:, p], z[:, q])
    x = 1j * h / 16.0
    u = torch.eye(3, dtype=h.dtype, device=dev).expand(n, 3, 3)
    for i in range(9, 0, -1):                      # Taylor by Horner, then four squarings
        u = torch.eye(3, dtype=h.dtype, device=dev) + _mm(x, u) / i
    for _ in range(4):
        u = _mm(u, u)
    a = u[:, 0] / u[:, 0].abs().square().sum(-1, keepdim=True).sqrt()
    b = u[:, 1] - a * (a.conj() * u[:, 1]).sum(-1, keepdim=True)
    b = b / b.abs().square().sum(-1, keepdim=True).sqrt()
    return torch.stack([a, b, torch.linalg.cross(a, b).conj()], 1)


def _z2(shape, gen, dev):
    s = torch.randint(0, 2, tuple(shape) + (2,), generator=gen, device=dev).to(torch.float64) * 2 - 1
    return torch.view_as_complex(s / math.sqrt(2.0))


def _spread(case):
    return 0.5 if case["nx"] * case["ny"] * case["nz"] * case["nt"] <= 512 else 0.35


def _shift(f, nu, dims, step):
    """f(x + step nu) for a field of shape (V, ...)."""
    g = f.reshape(dims[::-1] + tuple(f.shape[1:]))
    return torch.roll(g, -step, 3 - nu).reshape(f.shape)


# chiral basis: (gamma_nu psi)_s = phase_s psi_{perm(s)}
_PERM = ((3, 2, 1, 0), (3, 2, 1, 0), (2, 3, 0, 1), (2, 3, 0, 1))
_PHASE = ((-1j, -1j, 1j, 1j), (-1.0, 1.0, 1.0, -1.0), (-1j, 1j, 1j, -1j), (1.0, 1.0, 1.0, 1.0))


def _gamma(nu, p):
    ph = torch.tensor(_PHASE[nu], dtype=p.dtype, device=p.device)
    return ph[:, None] * p[:, list(_PERM[nu])]


def _eigenpairs(case, gen, dev):
    """Links of a constant field seen through a random gauge rotation, and l of its
    eigenpairs near zero: U_nu(x) = g(x) C_nu g(x + nu)^dag has the plane waves of the
    constant field, rotated, as eigenvectors, one 12 x 12 problem per momentum.  Of the
    lowest eigenvalues the l best separated ones are taken."""
    dims, V = _geometry(case)
    l, mu, kap = case["l"], case["mu"], 1.0 / (2 * MASS + 8.0)
    C = _su3(4, 0.35, gen, dev)
    g = _su3(V, 1.0, gen, dev)
    U = torch.stack([_mm(_mm(g, C[nu].expand(V, 3, 3)), _shift(g, nu, dims, 1).mH) for nu in range(4)])
    n = np.indices(dims[::-1]).reshape(4, V)[::-1]
    p = 2 * np.pi * n / np.array(dims)[:, None]
    p[3] += np.pi / dims[3]
    gam = [np.array([[(_PHASE[nu][s] if _PERM[nu][s] == r else 0) for r in range(4)] for s in range(4)]) for nu in range(4)]
    Ch = C.cpu().numpy()
    M = np.broadcast_to(np.eye(12, dtype=complex), (V, 12, 12)).copy()
    for nu in range(4):
        e = math.exp(mu) if nu == 3 else 1.0
        M -= kap * (e * np.exp(1j * p[nu])[:, None, None] * np.kron(np.eye(4) + gam[nu], Ch[nu])
                    + np.exp(-1j * p[nu])[:, None, None] / e * np.kron(np.eye(4) - gam[nu], Ch[nu].conj().T))
    M[:, 6:] *= -1                                  # gamma_5
    lam, R = np.linalg.eig(M)
    flat = lam.ravel()
    low = np.argsort(np.abs(flat))[:64]
    low = low[np.abs(flat[low].real) > 0.02]
    gap = np.array([np.partition(np.abs(flat - flat[i]), 1)[1] for i in low])
    pick = low[np.argsort(-gap)[:l]]
    mom, idx = pick // 12, pick % 12
    Lt = np.linalg.inv(R[mom]).conj().transpose(0, 2, 1)
    wave = torch.from_numpy(np.exp(1j * (p[:, mom].T @ n)) / math.sqrt(V)).to(dev)

    def field(chi):
        c = torch.from_numpy(np.ascontiguousarray(chi)).to(dev).reshape(l, 1, 4, 1, 3)
        return (wave[:, :, None, None] * (g[None, :, None] * c).sum(-1)).contiguous()

    every = np.arange(l)
    return U, field(R[mom, :, idx]), field(Lt[every, :, idx]), [complex(z) for z in flat[pick]]


def _inputs(case, seed):
    dims, V = _geometry(case)
    dev = _device()
    gen = torch.Generator(device=dev)
    gen.manual_seed(1604 + 7919 * int(seed))
    s = dict(case=case)
    if case["kind"] == "deflated":
        s["U"], s["R"], s["L"], s["lam"] = _eigenpairs(case, gen, dev)
    else:
        s["U"] = _su3(4 * V, _spread(case), gen, dev).reshape(4, V, 3, 3)
    n = (case["nsrc"],) if "nsrc" in case else ()
    s["psi"] = _z2(n + (V, 4, 3), gen, dev)
    s["eta"] = _z2(n + (V, 4, 3), gen, dev)
    if "klo" in case:
        r = np.random.default_rng(int(seed))
        s["ks"] = [int(v) for v in r.integers(case["klo"], case["khi"] + 1, case["nsrc"])]
        s["ks"][0] = case["khi"]                    # the largest size is the same for every seed
    if case["kind"] == "block":
        x = torch.randn(3, 3, generator=torch.Generator().manual_seed(int(seed)), dtype=torch.complex128).numpy()
        x = x + x.conj().T
        s["X"] = x - np.trace(x) / 3 * np.eye(3)
        s["nu"], s["site"] = int(seed) % 4, int(seed) * 31 % V
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    dims, _ = _geometry(case)
    s["ctx"] = Context(dims, MASS, case["mu"], precision=case["precision"])
    s["ctx"].set_links(s["U"])
    if case["kind"] == "deflated":
        s["defl"] = s["ctx"].deflation(s["R"], s["L"], s["lam"])
    if case["kind"] == "autograd":
        for n in ("U", "psi", "eta"):
            s[n].requires_grad_(True)
    return s


def run(s):
    c, ctx, kind = s["case"], s["ctx"], s["case"]["kind"]
    if kind == "apply_h":
        return ctx.apply_h(s["psi"], c["dagger"])
    if kind == "apply_dw":
        return ctx.apply_dw(s["psi"], c["dagger"])
    if kind == "overlap":
        return ctx.overlap(s["psi"], c["k"])[0]
    if kind == "sign":
        return ctx.sign(s["psi"], c["k"])[0]
    if kind == "autograd":
        S = SignGrad.apply(s["U"], s["psi"], s["eta"], ctx, c["k"])
        return (S.detach(),) + torch.autograd.grad(S, (s["U"], s["psi"], s["eta"]))
    if kind == "grad":
        S, dU, dpsi, _, y = ctx.sign_grad(s["eta"], s["psi"], c["k"], want_dpsi=True, want_y=True)
        return S, dU, dpsi, y
    if kind == "batch":
        S, dU, dpsi, _ = ctx.sign_grad_batched(s["eta"], s["psi"], s["ks"], want_dpsi=True)
        return S, dU, dpsi
    if kind == "overlap_grad":
        S, dU, dpsi, dov, _ = ctx.overlap_grad(s["eta"], s["psi"], c["k"], recompute=c["recompute"])
        return S, dU, dpsi, dov
    if kind == "current":
        return ctx.current_estimate(s["psi"], s["ks"], ward=False)[:3]
    if kind == "deflated":
        S, dU, dpsi, _ = ctx.sign_grad(s["eta"], s["psi"], c["k"], want_dpsi=True, defl=s["defl"])
        return S, dU, dpsi
    y1, y2, _ = ctx.block_sign(s["nu"], s["site"], s["X"], s["psi"], c["k"])
    return y1, y2


# ------------------------------------------------------------------ work
def work(case):
    """One pass without which the path does not get by.  A Wilson application is 1392
    flops per site; a step of the two-sided process applies it twice, reads and writes
    both Krylov vectors and reads the links (once for all sources); the derivative's
    reverse step is two more applications, the step's vectors and two adjoint vectors;
    the shifted solves are counted as 500 iterations of two applications each."""
    _, V = _geometry(case)
    kind = case["kind"]
    zl = 16 if case["precision"] == "fp64" else 8
    z = 8 if case["precision"] == "mixed" else 16
    links, canon, field, app = 36 * zl * V, 12 * 16 * V, 12 * z * V, 1392 * V
    if kind in ("apply_h", "apply_dw"):
        return dict(bytes=links + 2 * canon, flops=app)
    if kind in ("sign", "overlap"):
        return dict(bytes=case["k"] * (links + 5 * field) + 2 * canon, flops=case["k"] * (2 * app + 16 * 12 * V))
    if kind == "block":
        return dict(bytes=case["k"] * (links + 10 * field) + 3 * canon, flops=case["k"] * (4 * app + 32 * 12 * V))
    n = case.get("nsrc", 1)
    kmax = case.get("khi", case.get("k"))
    ksum = n * (case["klo"] + case["khi"]) / 2 if "klo" in case else case["k"]
    extra = 2 if case.get("recompute") else 1
    b = kmax * (1 + extra) * links + ksum * (4 * extra + 8) * field + n * (36 * 16 * V + 3 * canon)
    f = ksum * ((2 + 2 * extra) * app + 2 * 1152 * V)
    if kind == "deflated":
        b += 500 * (2 * links + 2 * case["l"] * 8 * field)
        f += 500 * 2 * case["l"] * 2 * app
    return dict(bytes=b, flops=f)


# ------------------------------------------------------------------ 64-bit reference
def _hop(U, p, dims, mu):
    """Hopping sum of D_w(mu) (the temporal boundary sign folded into U)."""
    out = torch.zeros_like(p)
    for nu in range(4):
        e = math.exp(mu) if nu == 3 else 1.0
        f = _shift(p, nu, dims, 1)
        f = e * (U[nu][:, None] * f[:, :, None, :]).sum(-1)
        b = (U[nu].conj().transpose(-1, -2)[:, None] * p[:, :, None, :]).sum(-1)
        b = _shift(b, nu, dims, -1) / e
        out = out + f + _gamma(nu, f) + b - _gamma(nu, b)
    return out


def _g5(p):
    return torch.cat([p[:, :2], -p[:, 2:]], 1)


def _signed(U, dims):
    s = torch.ones(U.shape[:2] + (1, 1), dtype=torch.float64, device=U.device)
    s[3, -(dims[0] * dims[1] * dims[2]):] = -1.0
    return U * s


def _h(U, p, dims, mu):
    return _g5(p - _hop(U, p, dims, mu) / (2 * MASS + 8.0))


class _SignColumn(torch.autograd.Function):
    """sgn(T) e_1 by the eigendecomposition, and its derivative by divided differences."""

    @staticmethod
    def forward(ctx, T):
        lam, R = np.linalg.eig(T.detach().cpu().numpy())
        Ri = np.linalg.inv(R)
        ctx.eig = lam, R, Ri
        return torch.from_numpy((R * np.sign(lam.real)) @ Ri[:, 0]).to(T.device)

    @staticmethod
    def backward(ctx, grad):
        lam, R, Ri = ctx.eig
        s = np.sign(lam.real)
        d = lam[:, None] - lam[None, :]
        same = s[:, None] == s[None, :]
        F = np.where(same, 0.0, (s[:, None] - s[None, :]) / np.where(same, 1.0, d))
        G = np.zeros_like(R)
        G[0] = grad.cpu().numpy().conj()            # E = e_1 g^dag
        return torch.from_numpy((R @ (F * (Ri @ G @ R)) @ Ri).conj().T.copy()).to(grad.device)


def _tsl(A, Ad, x, k):
    nx = x.abs().square().sum().sqrt()
    v = w = x / nx
    V, al, be, ga = [v], [], [], []
    vp = wp = None
    for j in range(k):
        a = A(v)
        alpha = (w.conj() * a).sum()
        al.append(alpha)
        if j == k - 1:
            break
        r = a - alpha * v
        s = Ad(w) - alpha.conj() * w
        if j:
            r = r - ga[-1] * vp
            s = s - be[-1] * wp
        om = (s.conj() * r).sum()
        b = om.abs().sqrt()
        g = om / b
        vp, wp, v, w = v, w, r / b, s / g.conj()
        be.append(b)
        ga.append(g)
        V.append(v)
    T = torch.diag(torch.stack(al))
    if k > 1:
        T = T + torch.diag(torch.stack(be).to(T.dtype), -1) + torch.diag(torch.stack(ga), 1)
    c = _SignColumn.apply(T)
    y = torch.zeros_like(x)
    for cj, v in zip(c, V):
        y = y + cj * v
    return nx * y


def _sign_and_grad(U, psi, eta, k, dims, mu):
    """S, dU, dpsi, y of S = Re <eta|TSL_k(psi)>."""
    from torch.utils.checkpoint import checkpoint
    U = U.detach().requires_grad_(True)
    psi = psi.detach().requires_grad_(True)

    def op(m):
        return lambda v: checkpoint(lambda u, p: _h(_signed(u, dims), p, dims, m), U, v, use_reentrant=False)

    y = _tsl(op(mu), op(-mu), psi, k)
    S = (eta.conj() * y).sum().real
    S.backward()
    return S.detach(), U.grad, psi.grad, y.detach()


def exact(case, seed):
    kind = case["kind"]
    if kind == "deflated":
        return None
    s = _inputs(case, seed)
    dims, V = _geometry(case)
    mu, psi, eta, U = case["mu"], s["psi"], s["eta"], s["U"]
    Us = _signed(U, dims)
    if kind == "apply_h":
        return _h(Us, psi, dims, -mu if case["dagger"] else mu)
    if kind == "apply_dw":
        return _h(Us, _g5(psi), dims, -mu) if case["dagger"] else _g5(_h(Us, psi, dims, mu))
    if kind in ("sign", "overlap"):
        y = _tsl(lambda v: _h(Us, v, dims, mu), lambda v: _h(Us, v, dims, -mu), psi, case["k"])
        return psi + _g5(y) if kind == "overlap" else y
    if kind == "block":
        dU = torch.zeros_like(Us)
        nu, site = s["nu"], s["site"]
        dU[nu, site] = 1j * _mm(torch.from_numpy(s["X"]).to(U.device), Us[nu, site])

        def two(m, adjoint):
            def f(v):
                a, b = v[:V], v[V:]
                ha, hb = _h(Us, a, dims, m), _h(Us, b, dims, m)
                d = -_g5(_hop(dU, a if adjoint else b, dims, m)) / (2 * MASS + 8.0)
                return torch.cat([ha, hb + d] if adjoint else [ha + d, hb])
            return f

        y = _tsl(two(mu, False), two(-mu, True), torch.cat([torch.zeros_like(psi), psi]), case["k"])
        return y[:V], y[V:]
    if V * case.get("khi", case.get("k")) > 4_000_000:     # too long: the first source of a batch does
        if kind != "batch":
            return None
    if kind in ("grad", "autograd"):
        S, dU, dp, y = _sign_and_grad(U, psi, eta, case["k"], dims, mu)
        return (S, dU, dp, y)
    if kind == "overlap_grad":
        S, dU, dp, y = _sign_and_grad(U, psi, _g5(eta), case["k"], dims, mu)
        return S + (eta.conj() * psi).sum().real, dU, dp + eta, psi + _g5(y)
    if kind == "current":
        j = 0.0
        for x, k in zip(psi, s["ks"]):
            _, dU, _, _ = _sign_and_grad(U, x, _g5(x), k, dims, mu)
            j = j - (dU.conj() * U).sum((-1, -2)).imag / len(s["ks"])
        back = torch.stack([_shift(j[nu], nu, dims, -1) for nu in range(4)])
        return j, (j - back).sum(0), (j + back).sum(0)
    # batch: S of the first source (the outputs of the others have no value here)
    S, _, _, _ = _sign_and_grad(U, psi[0], eta[0], s["ks"][0], dims, mu)
    return [float(S)] + [None] * (case["nsrc"] - 1), None, None
