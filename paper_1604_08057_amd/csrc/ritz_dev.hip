// Smallest |Re theta| over the eigenvalues of the projected matrix and its infinity norm,
// on the device, for the sign calls: what ritz.cpp computes on host threads, by the same
// method (Ehrlich-Aberth sweeps on the tridiagonal's three-term recurrence, starting points
// by divide and conquer), where no device work is left to hide the host's time behind.  In a
// sweep every unsettled root forms its Newton correction and its Aberth sum, all at once, a
// root per pair of lanes: one lane walks the leading minors, the other the trailing ones.
// Blocks of up to kOneGroup rows settle in a workgroup each; the longer ones, whose walks
// would queue on one compute unit, in a launch per sweep over the chip (15 us for blocks of
// 100 rows, 25 for 200, 45 for 400, 5 once every root has settled).
// Bound: the walk, a serial chain of 0.2 us per row.
// Measured beside the rest of the call: 0.5 ms at k = 200, 1.2 ms at k = 400 and 4.3 ms at
// k = 1024; one workgroup with a lane per root took 1.0 and 2.6 ms at the first two, host
// threads 1.1, 3.8 and 28 ms with nothing else left to wait for.
#include "kernels.h"

#include <cmath>

namespace tslov {

namespace {

constexpr int kLeaf = 24;        // block size at which the iteration starts from a circle
constexpr int kMaxSweeps = 500;
constexpr int kOneGroup = 64;    // block size up to which one workgroup sweeps
constexpr int kInnerSweeps = 6;  // launched at each longer size but the full one,
constexpr int kTopSweeps = kRitzTopSweeps;    // at the full one, and
constexpr int kMoreSweeps = kRitzMoreSweeps;  // there again while a root is open
static_assert(kInnerSweeps % 2 == 0 && kTopSweeps % 2 == 0 && kMoreSweeps % 2 == 0, "the roots end in z[0]");

__device__ __forceinline__ double rcp2(double x) {   // as the division, to an ulp
    double r = __builtin_amdgcn_rcp(x);
    r = __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
    return __builtin_fma(r, __builtin_fma(-x, r, 1.0), r);
}

struct __align__(16) Row {
    double ar, ai, wr, wi;       // diagonal entry and T_{j,j-1} T_{j-1,j}, scaled
};

// The value of lane l ^ 1.
__device__ __forceinline__ double swap_pair(double v) { return dpp_d<kDppSwap1>(v); }
__device__ __forceinline__ ZD swap_pair(ZD v) { return mk<double>(swap_pair(v.re), swap_pair(v.im)); }

// a b with the bits of b a: a fused product would round the exchanged operands differently.
__device__ __forceinline__ ZD mul_symmetric(ZD a, ZD b) {
#pragma clang fp contract(off)
    const double re = a.re * b.re - a.im * b.im, im = a.re * b.im + a.im * b.re;
    return mk<double>(re, im);
}

// p(z)/p'(z) of p = det(z - T) on rows lo .. lo + n - 1 by a pair of lanes, the same bits in
// both: what joins the sides (rq, ends and s1 + s1' below) is symmetric in them to the last
// bit, so zi, prev and done agree too, and no lane settles alone and leaves its partner half
// a matrix (near a root D is all cancellation).  Side 0 walks
// the leading minors P_1 .. P_h down from the first row, side 1 the trailing minors Q up from
// the last one, each by the ratios of successive minors and their logarithmic derivatives
// (ritz.cpp newton_batch); they meet in p = P_h Q - w P_{h-1} Q', w the coupling of rows
// h - 1 and h:
//   p / (P_{h-1} Q') = r q - w,   p'/p = s0 + t0 + r q (s1 - s0 + t1 - t0) / (r q - w),
// r, q the last ratios and s, t the logarithmic derivatives of P_{h-1}, P_h and Q', Q.
__device__ __forceinline__ ZD newton_correction(const Row* __restrict__ T, int lo, int n, int side, ZD z) {
    const int h = n / 2, len = side ? n - h : h, step = side ? -1 : 1;
    int at = side ? lo + n - 1 : lo;
    double rr = 1.0, ri = 0.0, sr = 0.0, si = 0.0, pr = 0.0, pi = 0.0;   // an empty side: the minor 1
    if (len > 0) {
        rr = z.re - T[at].ar, ri = z.im - T[at].ai;
        if (rr == 0.0 && ri == 0.0) rr = 1e-18;
        double d = rcp2(rr * rr + ri * ri);
        double ir = rr * d, ii = -ri * d;
        sr = ir;
        si = ii;
        for (int j = 1; j < len; ++j) {
            const Row& w = T[side ? at : at + 1];   // the coupling of the old row and the new
            at += step;
            const double xr = z.re - T[at].ar, xi = z.im - T[at].ai;
            const double qr = w.wr * ir - w.wi * ii, qi = w.wr * ii + w.wi * ir;
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
        }
    }
    const ZD r = mk<double>(rr, ri), s1 = mk<double>(sr, si), s0 = mk<double>(pr, pi);
    const ZD w = h > 0 ? mk<double>(T[lo + h].wr, T[lo + h].wi) : mk<double>(0, 0);
    const ZD rq = mul_symmetric(r, swap_pair(r)), D = rq - w, ends = s0 + swap_pair(s0);
    const ZD den = D * ends + rq * (s1 + swap_pair(s1) - ends);
    return D * mk<double>(den.re * rcp2(norm2(den)), -den.im * rcp2(norm2(den)));
}

// sum over the block's other roots of 1 / (z_i - z_q), every other one by each lane of the
// pair, four partial sums in flight (a root equal to z_i has no direction to push it in).
__device__ __forceinline__ ZD aberth_sum(const ZD* __restrict__ z, int lo, int n, int i, int side, ZD zi) {
    double sr[4] = {0.0, 0.0, 0.0, 0.0}, si[4] = {0.0, 0.0, 0.0, 0.0};
    for (int q0 = side; q0 < n; q0 += 8)
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int at = q0 + 2 * c, q = lo + min(at, n - 1);
            const double dr = zi.re - z[q].re, di = zi.im - z[q].im;
            const double d2 = dr * dr + di * di;
            const double w = (at >= n || q == i || d2 == 0.0) ? 0.0 : rcp2(d2);
            sr[c] += w == 0.0 ? 0.0 : dr * w;
            si[c] -= w == 0.0 ? 0.0 : di * w;
        }
    const double tr = (sr[0] + sr[1]) + (sr[2] + sr[3]), ti = (si[0] + si[1]) + (si[2] + si[3]);
    return mk<double>(tr + swap_pair(tr), ti + swap_pair(ti));   // the same in both lanes
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

// Thread i's block at depth d, rows l0 .. l0 + m - 1 (one at most kLeaf long stays whole).
__device__ __forceinline__ void block_at(int k, int d, int i, int& l0, int& m) {
    l0 = 0;
    m = k;
    for (int q = 0; q < d && m > kLeaf; ++q) {
        const int h = m / 2;
        if (i - l0 >= h) {
            l0 += h;
            m -= h;
        } else {
            m = h;
        }
    }
}

// A halved block's root as starting point: equal points would make the Aberth sum singular.
__device__ __forceinline__ ZD start_point(const ZD* __restrict__ z, int l0, int m, int i) {
    ZD zi = z[i];
    const int h = m / 2;
    bool same = false;
    if (m > kLeaf && i - l0 >= h)
        for (int q = 0; q < h; ++q) same |= z[l0 + q].re == zi.re && z[l0 + q].im == zi.im;
    if (same) zi = zi + mk<double>(1e-8 * fmax(1.0, sqrt(norm2(zi))), 1e-8);
    return zi;
}

// One step of an open root; returns whether it has settled: at rounding level, or a small
// step that no longer halves (below the top the roots only start the next stage: a step of
// 1e-5 leaves them far closer).
__device__ __forceinline__ bool root_step(const Row* __restrict__ T, const ZD* __restrict__ z, int l0, int m, int i,
                                          int side, bool top, ZD& zi, double& prev) {
    const ZD N = newton_correction(T, l0, m, side, zi);
    const ZD step = zdiv(N, mk<double>(1.0, 0.0) - N * aberth_sum(z, l0, m, i, side, zi));
    if (!(std::isfinite(step.re) && std::isfinite(step.im))) return true;
    zi = zi - step;
    const double st = sqrt(norm2(step)), sc = fmax(1.0, sqrt(norm2(zi)));
    const bool done = st <= (top ? 4.0 * 2.220446049250313e-16 : 1e-5) * sc || (st < 1e-10 * sc && st > 0.5 * prev);
    prev = st;
    return done;
}

// Smallest |Re z| over the workgroup's roots, valid in its first thread.
__device__ __forceinline__ double group_min_re(double mn, double* red) {
#pragma unroll
    for (int o = kWave / 2; o > 0; o >>= 1) mn = fmin(mn, __shfl_xor(mn, o, kWave));
    __syncthreads();
    if (threadIdx.x % kWave == 0) red[threadIdx.x / kWave] = mn;
    __syncthreads();
    for (int w = 0; w < (int)blockDim.x / kWave; ++w) mn = fmin(mn, red[w]);
    return mn;
}

// Roots and matrix between the launches, behind the result (out[3]: the scale, 0: no
// eigenvalues to find).
struct RitzState {
    double* out;
    Row* T;
    ZD* z[2];
    double* prev;
    int* done;
    __host__ __device__ RitzState(double* o, int k)
        : out(o), T(reinterpret_cast<Row*>(o + 8)), z{reinterpret_cast<ZD*>(T + k), reinterpret_cast<ZD*>(T + k) + k},
          prev(reinterpret_cast<double*>(z[1] + k)), done(reinterpret_cast<int*>(prev + k)) {}
};

}  // namespace

// The divide and conquer inside block blockIdx.x of depth nd, a workgroup per block; nd > 0
// leaves the roots there for the sweep launches.
constexpr int kGroupThreads = 2 * kOneGroup;
__global__ __launch_bounds__(kGroupThreads) void k_ritz(Coef coef, int k, int nd, double* __restrict__ out) {
    __shared__ Row T[kOneGroup];
    __shared__ ZD z[kOneGroup];
    __shared__ double red[kGroupThreads / kWave];
    int lo = 0, n = k;   // the workgroup's rows (blocks longer than kOneGroup are all split)
    for (int q = nd - 1; q >= 0; --q) {
        const int h = n / 2;
        if (blockIdx.x >> q & 1) {
            lo += h;
            n -= h;
        } else {
            n = h;
        }
    }
    const int i = threadIdx.x / 2, side = threadIdx.x % 2;   // a root per pair of lanes
    const bool mine = i < n;
    double norm = 0.0, scale = 0.0;
    for (int q = threadIdx.x; q < k; q += kGroupThreads) {
        const double a = sqrt(norm2(coef.alpha[q + 1])), b = q > 0 ? fabs(coef.beta[q + 1]) : 0.0;
        const double g = q > 0 ? sqrt(norm2(coef.gamma[q + 1])) : 0.0;
        const double gn = q + 1 < k ? sqrt(norm2(coef.gamma[q + 2])) : 0.0;
        norm = fmax(norm, a + b + gn);
        scale = fmax(scale, fmax(fmax(a, b), g));
    }
    norm = group_max(norm, red);
    scale = group_max(scale, red);
    if (!(scale > 0.0) || !std::isfinite(scale)) {   // uniform: the zero matrix, or not finite
        if (threadIdx.x == 0 && blockIdx.x == 0) {
            out[0] = scale == 0.0 ? 0.0 : __builtin_nan("");
            out[1] = norm;
            out[2] = scale == 0.0 ? 0.0 : -1.0;
            out[3] = 0.0;
        }
        return;
    }
    if (mine && side == 0) {
        const double rs = 1.0 / scale;
        const ZD a = coef.alpha[lo + i + 1], g = lo + i > 0 ? coef.gamma[lo + i + 1] : mk<double>(0, 0);
        const double b = lo + i > 0 ? coef.beta[lo + i + 1] : 0.0;
        T[i].ar = a.re * rs;
        T[i].ai = a.im * rs;
        T[i].wr = b * rs * (g.re * rs);
        T[i].wi = b * rs * (g.im * rs);
    }
    int top = 0;   // the depth of the leaves (blocks of one depth differ by one row)
    for (int m = n; m > kLeaf; m -= m / 2) ++top;
    __syncthreads();
    int sweeps = 0;
#pragma unroll 1
    for (int d = top; d >= 0; --d) {
        int l0, m;
        block_at(n, d, i, l0, m);
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
            zi = start_point(z, l0, m, i);
        }
        __syncthreads();
        if (mine && side == 0) z[i] = zi;
        __syncthreads();
        bool done = !mine;
        double prev = INFINITY;
        for (sweeps = 1; sweeps <= kMaxSweeps; ++sweeps) {
            if (!done) done = root_step(T, z, l0, m, i, side, nd == 0 && d == 0, zi, prev);
            const int open = __syncthreads_or(!done);   // every sum has read the old roots
            if (mine && side == 0) z[i] = zi;
            __syncthreads();
            if (!open) break;
        }
    }
    if (nd > 0) {
        const RitzState st(out, k);
        if (mine && side == 0) {
            st.T[lo + i] = T[i];
            st.z[0][lo + i] = z[i];
        }
        if (threadIdx.x == 0 && blockIdx.x == 0) {
            out[1] = norm;
            out[3] = scale;
        }
        return;
    }
    const double mn = group_min_re(mine ? fabs(z[i].re) : INFINITY, red);
    if (threadIdx.x == 0) {
        out[0] = mn * scale;
        out[1] = norm;
        out[2] = sweeps <= kMaxSweeps ? (double)sweeps : -1.0;
    }
}

// One sweep at depth d, 128 roots per workgroup (a wavefront per SIMD: the chain is all
// latency); the first one starts from the roots of the halved blocks.  Every operand is
// loaded ahead of the first test, all in one round trip (the compiler holds them in private
// memory until then, 256 bytes per thread).
constexpr int kSweepBlock = 256, kSweepRows = 4;   // k <= 1024
__global__ __launch_bounds__(kSweepBlock) void k_ritz_sweep(double* __restrict__ out, int k, int d, int cur,
                                                            int first) {
    extern __shared__ char mem[];
    Row* const T = reinterpret_cast<Row*>(mem);
    ZD* const z = reinterpret_cast<ZD*>(T + k);
    const RitzState st(out, k);
    const int i = (blockIdx.x * kSweepBlock + threadIdx.x) / 2, side = threadIdx.x % 2, ic = min(i, k - 1);
    const bool mine = i < k;
    const double scale = out[3];
    bool done = (!first && st.done[ic]) || !mine;
    ZD zi = st.z[cur][ic];
    double prev = first ? INFINITY : st.prev[ic];
    Row row[kSweepRows];
    ZD root[kSweepRows];
#pragma unroll
    for (int c = 0; c < kSweepRows; ++c) {
        const int q = min((int)threadIdx.x + c * kSweepBlock, k - 1);
        row[c] = st.T[q];
        root[c] = st.z[cur][q];
    }
    if (scale == 0.0) return;
    if (__syncthreads_or(!done)) {
#pragma unroll
        for (int c = 0; c < kSweepRows; ++c)
            if ((int)threadIdx.x + c * kSweepBlock < k) {
                T[threadIdx.x + c * kSweepBlock] = row[c];
                z[threadIdx.x + c * kSweepBlock] = root[c];
            }
        __syncthreads();
        if (!done) {
            int l0, m;
            block_at(k, d, i, l0, m);
            if (first) zi = start_point(z, l0, m, i);
            done = root_step(T, z, l0, m, i, side, d == 0, zi, prev);
            if (side == 0) {
                st.prev[i] = prev;
                st.done[i] = done;
            }
        }
    }
    if (mine && side == 0) st.z[cur ^ 1][i] = zi;
}

// The result, out[2] = -2 while a root is open.
__global__ __launch_bounds__(1024) void k_ritz_end(double* __restrict__ out, int k, int cur, int sweeps) {
    __shared__ double red[1024 / kWave];
    const RitzState st(out, k);
    if (out[3] == 0.0) return;
    const int i = threadIdx.x;
    const int open = __syncthreads_or(i < k && !st.done[i]);
    const double mn = group_min_re(i < k ? fabs(st.z[cur][i].re) : INFINITY, red);
    if (i == 0) {
        out[0] = mn * out[3];
        out[2] = !open ? (double)sweeps : sweeps < kMaxSweeps ? -2.0 : -1.0;
    }
}

size_t ritz_bytes(int k) { return 8 * sizeof(double) + (size_t)k * (sizeof(Row) + 2 * sizeof(ZD) + sizeof(double) + sizeof(int)); }

// Depths whose blocks are longer than kOneGroup go out as sweep launches over the chip.
static int ritz_depths(int k) {
    int d = 0;
    for (int m = k; m > kOneGroup; m -= m / 2) ++d;
    return d;
}

static void ritz_sweeps(double* out, int k, int d, int n, bool start, int& cur, hipStream_t st) {
    const size_t lds = (size_t)k * (sizeof(Row) + sizeof(ZD));
    for (int s = 0; s < n; ++s, cur ^= 1)
        hipLaunchKernelGGL(k_ritz_sweep, dim3((2 * k + kSweepBlock - 1) / kSweepBlock), dim3(kSweepBlock), lds, st, out, k, d, cur, start && s == 0);
}

void launch_ritz(Coef coef, int k, double* out, hipStream_t st) {
    const int nd = ritz_depths(k);
    hipLaunchKernelGGL(k_ritz, dim3(1 << nd), dim3(kGroupThreads), 0, st, coef, k, nd, out);
    int cur = 0;
    for (int d = nd - 1; d >= 0; --d) ritz_sweeps(out, k, d, d ? kInnerSweeps : kTopSweeps, true, cur, st);
    if (nd) hipLaunchKernelGGL(k_ritz_end, dim3(1), dim3((k + kWave - 1) / kWave * kWave), 0, st, out, k, cur, kTopSweeps);
}

void launch_ritz_more(int k, double* out, int sweeps, hipStream_t st) {
    int cur = 0;
    ritz_sweeps(out, k, 0, kMoreSweeps, false, cur, st);
    hipLaunchKernelGGL(k_ritz_end, dim3(1), dim3((k + kWave - 1) / kWave * kWave), 0, st, out, k, cur, sweeps);
}

}  // namespace tslov
