// Smallest |Re theta| over the eigenvalues of the projected matrix and its infinity norm,
// on the device, for the sign calls: what ritz.cpp computes on host threads, by the same
// method (Ehrlich-Aberth sweeps on the tridiagonal's three-term recurrence, starting points
// by divide and conquer), where no device work is left to hide the host's time behind.  One
// workgroup, one root per thread: in a sweep every unsettled root forms its Newton
// correction (n dependent steps for a block of n rows) and its Aberth sum, all at once.
// Bound: that chain, about twelve sweeps at the full size and half as much at all the
// halved ones together.
// Measured 1.0 ms at k = 200 and 2.6 ms at k = 400 beside the rest of the call
// (host threads: 1.1 and 3.8 ms, with nothing else left to wait for).
#include "kernels.h"

#include <cmath>

namespace tslov {

namespace {

constexpr int kLeaf = 24;        // block size at which the iteration starts from a circle
constexpr int kMaxSweeps = 500;

__device__ __forceinline__ double rcp2(double x) {   // as the division, to an ulp
    double r = __builtin_amdgcn_rcp(x);
    r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
    return __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
}

struct __align__(16) Row {
    double ar, ai, wr, wi;       // diagonal entry and T_{j,j-1} T_{j-1,j}, scaled
};

// p(z)/p'(z) of det(z - T) on rows lo .. lo + n - 1, from the ratios of the leading minors
// and the logarithmic derivatives (ritz.cpp newton_batch).
__device__ __forceinline__ ZD newton_correction(const Row* __restrict__ T, int lo, int n, ZD z) {
    double rr = z.re - T[lo].ar, ri = z.im - T[lo].ai;
    if (rr == 0.0 && ri == 0.0) rr = 1e-18;
    double d = rcp2(rr * rr + ri * ri);
    double ir = rr * d, ii = -ri * d, sr = ir, si = ii, pr = 0.0, pi = 0.0;
    Row t = T[lo + (n > 1 ? 1 : 0)];
    for (int j = 1; j < n; ++j) {
        const Row nx = T[lo + min(j + 1, n - 1)];
        const double xr = z.re - t.ar, xi = z.im - t.ai;
        const double qr = t.wr * ir - t.wi * ii, qi = t.wr * ii + t.wi * ir;
        rr = xr - qr;
        ri = xi - qi;
        if (rr == 0.0 && ri == 0.0) rr = 1e-18;
        d = rcp2(rr * rr + ri * ri);
        ir = rr * d;
        ii = -ri * d;
        const double tr = 1.0 + (xr * sr - xi * si) - (qr * pr - qi * pi);
        const double ti = (xr * si + xi * sr) - (qr * pi + qi * pr);
        pr = sr;
        pi = si;
        sr = tr * ir - ti * ii;
        si = tr * ii + ti * ir;
        t = nx;
    }
    d = rcp2(sr * sr + si * si);
    return mk<double>(sr * d, -si * d);
}

// sum over the block's other roots of 1 / (z_i - z_q), four partial sums in flight.
__device__ __forceinline__ ZD aberth_sum(const ZD* __restrict__ z, int lo, int n, int i, ZD zi) {
    double sr[4] = {0.0, 0.0, 0.0, 0.0}, si[4] = {0.0, 0.0, 0.0, 0.0};
    for (int q0 = 0; q0 < n; q0 += 4)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int q = lo + min(q0 + c, n - 1);
            const double dr = zi.re - z[q].re, di = zi.im - z[q].im;
            const double w = (q0 + c >= n || q == i) ? 0.0 : rcp2(dr * dr + di * di);
            sr[c] += w == 0.0 ? 0.0 : dr * w;
            si[c] -= w == 0.0 ? 0.0 : di * w;
        }
    return mk<double>((sr[0] + sr[1]) + (sr[2] + sr[3]), (si[0] + si[1]) + (si[2] + si[3]));
}

// Largest v >= 0 over the workgroup, NaN ignored.
__device__ __forceinline__ double group_max(double v, double* red) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, kWave));
    __syncthreads();
    if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = v;
    __syncthreads();
    double m = 0.0;
    for (int w = 0; w < (int)blockDim.x / kWave; ++w) m = fmax(m, red[w]);
    return m;
}

}  // namespace

__global__ __launch_bounds__(1024) void k_ritz(Coef coef, int k, double* __restrict__ out) {
    extern __shared__ char mem[];
    Row* const T = reinterpret_cast<Row*>(mem);
    ZD* const z = reinterpret_cast<ZD*>(T + k);
    __shared__ double red[1024 / kWave];
    const int i = threadIdx.x;
    const bool mine = i < k;
    const ZD a = mine ? coef.alpha[i + 1] : mk<double>(0, 0);
    const double b = mine && i > 0 ? coef.beta[i + 1] : 0.0;
    const ZD g = mine && i > 0 ? coef.gamma[i + 1] : mk<double>(0, 0);
    const ZD gn = mine && i + 1 < k ? coef.gamma[i + 2] : mk<double>(0, 0);
    const double norm = group_max(sqrt(norm2(a)) + fabs(b) + sqrt(norm2(gn)), red);
    const double scale = group_max(fmax(fmax(sqrt(norm2(a)), fabs(b)), sqrt(norm2(g))), red);
    if (!(scale > 0.0) || !std::isfinite(scale)) {   // uniform: the zero matrix, or not finite
        if (i == 0) {
            out[0] = scale == 0.0 ? 0.0 : __builtin_nan("");
            out[1] = norm;
            out[2] = scale == 0.0 ? 0.0 : -1.0;
        }
        return;
    }
    if (mine) {
        const double rs = 1.0 / scale;
        T[i].ar = a.re * rs;
        T[i].ai = a.im * rs;
        T[i].wr = b * rs * (g.re * rs);
        T[i].wi = b * rs * (g.im * rs);
    }
    int top = 0;   // the depth of the leaves (blocks of one depth differ by one row)
    for (int m = k; m > kLeaf; m -= m / 2) ++top;
    __syncthreads();
    int sweeps = 0;
#pragma unroll 1
    for (int d = top; d >= 0; --d) {
        int l0 = 0, m = k;   // this thread's block at depth d (one at most kLeaf long stays whole)
        for (int q = 0; q < d && m > kLeaf; ++q) {
            const int h = m / 2;
            if (i - l0 >= h) {
                l0 += h;
                m -= h;
            } else {
                m = h;
            }
        }
        ZD zi = mk<double>(0, 0);
        if (d == top) {
            if (mine) {
                ZD centre = mk<double>(0, 0);
                double radius = 0.0;
                for (int j = 0; j < m; ++j) centre = centre + mk<double>(T[l0 + j].ar, T[l0 + j].ai);
                centre = (1.0 / m) * centre;
                for (int j = 0; j < m; ++j) {
                    double r = sqrt(norm2(mk<double>(T[l0 + j].ar, T[l0 + j].ai) - centre));
                    if (j > 0) r += sqrt(sqrt(norm2(mk<double>(T[l0 + j].wr, T[l0 + j].wi))));
                    if (j + 1 < m) r += sqrt(sqrt(norm2(mk<double>(T[l0 + j + 1].wr, T[l0 + j + 1].wi))));
                    radius = fmax(radius, r);
                }
                if (!(radius > 0.0)) radius = 1.0;
                double sn, cs;
                sincos(6.283185307179586 * (i - l0 + 0.25) / m + 0.4, &sn, &cs);
                zi = centre + radius * mk<double>(cs, sn);
            }
        } else if (mine) {
            zi = z[i];
            // equal starting points would make the Aberth sum singular
            const int h = m / 2;
            bool same = false;
            if (m > kLeaf && i - l0 >= h)
                for (int q = 0; q < h; ++q) same |= z[l0 + q].re == zi.re && z[l0 + q].im == zi.im;
            if (same) zi = zi + mk<double>(1e-8 * fmax(1.0, sqrt(norm2(zi))), 1e-8);
        }
        __syncthreads();
        if (mine) z[i] = zi;
        __syncthreads();
        bool done = !mine;
        double prev = INFINITY;
        for (sweeps = 1; sweeps <= kMaxSweeps; ++sweeps) {
            if (!done) {
                const ZD N = newton_correction(T, l0, m, zi);
                const ZD step = zdiv(N, mk<double>(1.0, 0.0) - N * aberth_sum(z, l0, m, i, zi));
                if (std::isfinite(step.re) && std::isfinite(step.im)) {
                    zi = zi - step;
                    const double st = sqrt(norm2(step)), sc = fmax(1.0, sqrt(norm2(zi)));
                    // at rounding level, or a small step that no longer halves (below the top
                    // the roots only start the next stage: a step of 1e-5 leaves them far closer)
                    done = st <= (d == 0 ? 4.0 * 2.220446049250313e-16 : 1e-5) * sc ||
                           (st < 1e-10 * sc && st > 0.5 * prev);
                    prev = st;
                } else {
                    done = true;
                }
            }
            const int open = __syncthreads_or(!done);   // every sum has read the old roots
            if (mine) z[i] = zi;
            __syncthreads();
            if (!open) break;
        }
    }
    double mn = mine ? fabs(z[i].re) : INFINITY;
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) mn = fmin(mn, __shfl_xor(mn, o, kWave));
    if (i % kWave == 0) red[i / kWave] = mn;
    __syncthreads();
    if (i == 0) {
        for (int w = 0; w < (int)blockDim.x / kWave; ++w) mn = fmin(mn, red[w]);
        out[0] = mn * scale;
        out[1] = norm;
        out[2] = sweeps <= kMaxSweeps ? (double)sweeps : -1.0;
    }
}

void launch_ritz(Coef coef, int k, double* out, hipStream_t st) {
    hipLaunchKernelGGL(k_ritz, dim3(1), dim3((k + kWave - 1) / kWave * kWave), (size_t)k * (sizeof(Row) + sizeof(ZD)),
                       st, coef, k, out);
}

}  // namespace tslov
