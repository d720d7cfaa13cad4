// Projected-matrix step of the sign calls in O(N k) work: c = sgn(T) e_1 of the
// tridiagonal T_k by the partial fractions of a rational approximation of the sign.  The
// N-point member of the Kenney-Laub principal Pade family (C. S. Kenney and A. J. Laub,
// "Rational iterative methods for the matrix sign function", SIAM J. Matrix Anal. Appl.
// 12 (1991); N. J. Higham, "Functions of Matrices", Sec. 5.4), r_N(x) = coth(N arcoth x), is
//     r_N(x) = x/N + (1/N) sum_m sec^2(phi_m) / (x - i tan phi_m),  phi_m = pi m / N,
// m = -(N/2 - 1) .. N/2 - 1, with error 2 rho^N, rho = |(1 - x)/(1 + x)| for x in the right
// half plane (its mirror image in the left).  Newton's iteration composes the members
// N = 2, 4, 8, ... by inverting full matrices; the partial fractions give one large member
// from N - 1 independent tridiagonal solves, one per thread:
//     c = T e_1/(s N) + sum_m W_m x_m,   (T - i s t_m) x_m = e_1,   t_m = tan phi_m.
// The even m are the member N/2 and the odd m its midpoint twin tanh(N/2 arcoth x).  Half
// their difference is 1/sinh(N h), h = arcoth x, of which exp(-N h) is left in their mean, so
// the difference bounds the result's error; the host accepts the result by it, at rounding
// level, or refuses it (then a larger N, then Newton).
// Bound: the chain of 2 k dependent complex steps of each thread, whatever N up to the
// chip's width: 49 us at k = 200, 94 us at k = 400 (both sweeps), in place of 1.3 ms and
// 4.5 ms of Gauss-Jordan sweeps and products.
#include "kernels.h"

#include <cmath>

namespace tslov {

namespace {

constexpr int kRT = 64;     // poles per block of the sweeps (one wavefront)
constexpr int kRR = 256;    // threads per block of the pole sums

// 1/x by two Newton steps on the hardware estimate (x is a sum of squares; 0 and
// overflow give NaN or inf, which the acceptance test refuses).
__device__ __forceinline__ double rcp_nr(double x) {
    double r = __builtin_amdgcn_rcp(x);
    r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
    return __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
}
__device__ __forceinline__ ZD zrcp_nr(ZD d) {
    const double n = rcp_nr(norm2(d));
    return mk<double>(n * d.re, -n * d.im);
}

// Scale s of r_N(x / s): half the root mean square of the eigenvalues (from
// tr T^2 = sum alpha^2 + 2 sum beta gamma), below the middle of the spectrum so that
// the small eigenvalues, which converge last, gain; bounded below where the traces
// cancel.  Called by whole wavefronts, the same value in every lane.
__device__ __forceinline__ double rat_scale(const Coef& coef, int k) {
    double re = 0.0, im = 0.0, ab = 0.0;
    for (int j = 1 + (int)(threadIdx.x % kWave); j <= k; j += kWave) {
        const ZD a = coef.alpha[j], a2 = a * a;
        re += a2.re;
        im += a2.im;
        ab += norm2(a);
        if (j > 1) {
            const ZD bg = coef.beta[j] * coef.gamma[j];
            re += 2.0 * bg.re;
            im += 2.0 * bg.im;
            ab += 2.0 * (fabs(bg.re) + fabs(bg.im));
        }
    }
    re = wave_sum(re);
    im = wave_sum(im);
    ab = wave_sum(ab);
    return 0.5 * sqrt(fmax(sqrt(re * re + im * im), 1e-4 * ab) / k);
}

}  // namespace

// Both sweeps of the tridiagonal solves, thread = pole n (m = n - (N/2 - 1)), no pivoting:
// from the last row up  d_j = alpha_j - t - beta_{j+1} gamma_{j+1} / d_{j+1},  then down
// x_1 = 1 / d_1, x_j = -beta_j x_{j-1} / d_j.  A small d_j does no harm: every d_j is that of
// a row whose alpha_j - t and beta gamma are changed by a few ulps, and the x_j are products
// (pivots of 1e-15 planted at a pole leave c good to 1e-15).  Row j of the plane (ld poles):
// 1/d_j after the first sweep, W x_j after the second.
__global__ __launch_bounds__(kRT) void k_rat_sweeps(Coef coef, int k, RatWork w, int N) {
    extern __shared__ ZD rs[];   // alpha_j, beta_j gamma_j and beta_j (index j - 1)
    ZD* const al = rs;
    ZD* const bg = rs + k;
    double* const be = reinterpret_cast<double*>(rs + 2 * k);
    for (int j = threadIdx.x; j < k; j += kRT) {
        al[j] = coef.alpha[j + 1];
        be[j] = j > 0 ? coef.beta[j + 1] : 0.0;
        bg[j] = j > 0 ? coef.beta[j + 1] * coef.gamma[j + 1] : mk<double>(0, 0);
    }
    const double s = rat_scale(coef, k);
    __syncthreads();
    const int n = blockIdx.x * kRT + threadIdx.x;
    if (n >= N - 1) return;
    double sn, cs;
    sincospi((double)(n - (N / 2 - 1)) / N, &sn, &cs);
    const double t = s * sn / cs, W = s / (cs * cs * N);
    ZD* const buf = w.buf + n;
    const size_t ld = w.ld;
    ZD r = mk<double>(0, 0);
    for (int j = k - 1; j >= 0; --j) {
        ZD d = al[j] - (j + 1 < k ? bg[j + 1] : mk<double>(0, 0)) * r;
        d.im -= t;
        r = zrcp_nr(d);
        buf[(size_t)j * ld] = r;
    }
    ZD x = W * r;
    buf[0] = x;
    constexpr int kAhead = 8;      // rows in flight
    for (int j0 = 1; j0 < k; j0 += kAhead) {
        ZD rb[kAhead];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) rb[i] = buf[(size_t)min(j0 + i, k - 1) * ld];
#pragma unroll
        for (int i = 0; i < kAhead; ++i) {
            if (j0 + i >= k) break;
            x = (-be[j0 + i]) * (x * rb[i]);
            buf[(size_t)(j0 + i) * ld] = x;
        }
    }
}

// Pole sum of row j (block = row): c_j.  A thread's poles n, n + 256, ... have one parity,
// so the sums signed by it give the two members' difference dc_j.  Row partials: |dc_j|^2,
// |c_j|^2.
__global__ __launch_bounds__(kRR) void k_rat_sums(Coef coef, int k, RatWork w, int N) {
    const int j = blockIdx.x;
    const ZD* const row = w.buf + (size_t)j * w.ld;
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    for (int n = threadIdx.x; n < N - 1; n += kRR) {
        v[0] += row[n].re;
        v[1] += row[n].im;
    }
    // N/2 is even, so an even n is an odd m
    const double sg = (threadIdx.x & 1) ? 1.0 : -1.0;
    v[2] = sg * v[0];
    v[3] = sg * v[1];
    const double lin = 1.0 / (rat_scale(coef, k) * N);
    block_sum<4, kRR>(v);
    if (threadIdx.x != 0) return;
    // the polynomial part x/N belongs to the even member (and the mean)
    ZD t = mk<double>(0, 0);
    if (j == 0) t = lin * coef.alpha[1];
    if (j == 1) t = mk<double>(lin * coef.beta[2], 0.0);
    const ZD c = mk<double>(v[0], v[1]) + t, dc = mk<double>(v[2], v[3]) + t;
    coef.c[j + 1] = c;
    double* const p = w.rows + 2 * j;
    p[0] = norm2(dc);
    p[1] = norm2(c);
}

// |dc|^2 and |c|^2 into acc.
__global__ __launch_bounds__(kRR) void k_rat_finish(int k, RatWork w) {
    double v[2];
    reduce_partials<2, kRR>(w.rows, k, v);
    if (threadIdx.x == 0) {
        w.acc[0] = v[0];
        w.acc[1] = v[1];
    }
}

void launch_ratsign(Coef coef, int k, const RatWork& w, int N, hipStream_t st) {
    const size_t lds = (size_t)k * (2 * sizeof(ZD) + sizeof(double));
    hipLaunchKernelGGL(k_rat_sweeps, dim3((N - 1 + kRT - 1) / kRT), dim3(kRT), lds, st, coef, k, w, N);
    hipLaunchKernelGGL(k_rat_sums, dim3(k), dim3(kRR), 0, st, coef, k, w, N);
    hipLaunchKernelGGL(k_rat_finish, dim3(1), dim3(kRR), 0, st, k, w);
}

}  // namespace tslov
