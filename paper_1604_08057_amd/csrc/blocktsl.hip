// Two-sided Lanczos process on the block matrix B = [[H, dH], [0, H]] of Theorem 1
// (Sec. 2, eq. func_derivative_1): f(B) (0, x) = (d f(H) x, f(H) x), the paper's
// derivative of sgn(H) x along one link parameter, U_nu(x0) -> exp(i t X) U_nu(x0).
// Block vectors are pairs of float64 SoA fields (upper, lower); the products are
// B v = (H v1 + dH v2, H v2) and B^H w = (H^H w1, dH^H w1 + H^H w2), the inner products
// run over both halves, and the recursion is that of the plain process (both Krylov
// spaces from the source, v_1 = w_1 = x / |x|, no re-biorthogonalisation).  Its two
// kernels per step stand with the plain process's in fields.hip (k_blk_pair_*,
// k_blk_recur); here is the tangent dH alone, for the eigenvector derivatives.
#include "kernels.h"

namespace tslov {

// The tangent term at its two sites: with dU = i X U_nu(x0) (boundary sign folded
// into U as for the stencil),
//   dD_w psi (x0)        = -kappa e^{+mu d} (1 + g_nu) dU       psi(x0 + nu),
//   dD_w psi (x0 + nu)   = -kappa e^{-mu d} (1 - g_nu) dU^dag   psi(x0),
// and dH = g5 dD_w; dH^dag is the same at -mu.  out_a += dH in_a; out_b += dH^dag in_b
// (either pair may be null).  One thread.
template <int NU>
__device__ void tangent_one(const ZD (&u)[3][3], const BlockTangent& t, const Geom& g, double kappa, double emu,
                            const ZD* in_a, ZD* out_a, const ZD* in_b, ZD* out_b, int s0, int s1) {
    const double ef = NU == 3 ? emu : 1.0, eb = NU == 3 ? 1.0 / emu : 1.0;
    for (int which = 0; which < 2; ++which) {
        const ZD* in = which ? in_b : in_a;
        ZD* out = which ? out_b : out_a;
        if (!in) continue;
        // H(+mu) for the product, H(-mu) = H^dag for its adjoint
        const double cf = which ? eb : ef, cb = which ? ef : eb;
        Spinor<double> p1, p0, acc0, acc1;
        load_spinor(p1, in, g.ldv, s1);
        load_spinor(p0, in, g.ldv, s0);
        zero_spinor(acc0);
        zero_spinor(acc1);
        hop_fwd<NU>(acc0, u, p1, cf);
        hop_bwd<NU>(acc1, u, p0, cb);
        Spinor<double> o0, o1;
        load_spinor(o0, out, g.ldv, s0);
        load_spinor(o1, out, g.ldv, s1);
#pragma unroll
        for (int sp = 0; sp < 4; ++sp) {
            const double sg = sp < 2 ? -kappa : kappa;   // -kappa, then g5
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                o0.c[sp][c] = o0.c[sp][c] + sg * acc0.c[sp][c];
                o1.c[sp][c] = o1.c[sp][c] + sg * acc1.c[sp][c];
            }
        }
        store_spinor(out, g.ldv, s0, o0);
        store_spinor(out, g.ldv, s1, o1);
    }
    (void)t;
}

__global__ __launch_bounds__(64) void k_blk_tangent(const ZD* __restrict__ U, BlockTangent t, Geom g, double kappa,
                                                    double emu, const ZD* in_a, ZD* out_a, const ZD* in_b,
                                                    ZD* out_b) {
    if (threadIdx.x != 0) return;
    const Nbr n = neighbours(g, t.site);
    const int s0 = t.site, s1 = n.fwd[t.nu];
    // dU = i X U_nu(x0)
    ZD u0[3][3], du[3][3];
    load_link(u0, U, g.ldv, t.nu, s0);
#pragma unroll
    for (int a = 0; a < 3; ++a)
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            ZD acc = mk<double>(0, 0);
#pragma unroll
            for (int c = 0; c < 3; ++c) acc = acc + mk<double>(t.X[a][c][0], t.X[a][c][1]) * u0[c][b];
            du[a][b] = timesI(acc);
        }
    switch (t.nu) {
        case 0: tangent_one<0>(du, t, g, kappa, emu, in_a, out_a, in_b, out_b, s0, s1); break;
        case 1: tangent_one<1>(du, t, g, kappa, emu, in_a, out_a, in_b, out_b, s0, s1); break;
        case 2: tangent_one<2>(du, t, g, kappa, emu, in_a, out_a, in_b, out_b, s0, s1); break;
        default: tangent_one<3>(du, t, g, kappa, emu, in_a, out_a, in_b, out_b, s0, s1); break;
    }
}

void launch_blk_tangent(const ZD* U, const BlockTangent& t, const Geom& g, double kappa, double mu, const ZD* in_a,
                        ZD* out_a, const ZD* in_b, ZD* out_b, hipStream_t st) {
    hipLaunchKernelGGL(k_blk_tangent, dim3(1), dim3(64), 0, st, U, t, g, kappa, std::exp(mu), in_a, out_a, in_b,
                       out_b);
}

}  // namespace tslov
