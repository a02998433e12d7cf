// hqr_tiny.hpp -- the smallest problems to factor: at most W = 16 or 32
// columns with the right-hand sides, one wave, everything in registers.
//
// Lane l owns rows l, l + 64, .. (QM of them) of [A | B].  Step k is the
// one-reflector loop's (hqr_wg.hpp's wg_panel_step without panels): one wave
// reduction of the pivot column's products with every column, the scalars,
// the update; then the columns move down by one register, so the pivot column
// always is register 0 and the step is a loop body of its own.
//
// Bound: latency and instruction fetch.  A launch this short runs its code
// once, from memory: the unrolled panel kernels are 50 KB and more, and even a
// 4 x 2 problem took them about 16 us.  These are 5 to 13 KB.  A 20 x 8 solve
// with one right-hand side, its inputs copied in first, went from 27.6 to
// 18.2 us on MI355X; 100 x 20 (32 columns, two rows a lane) from 48 to 34 us.
#pragma once

#include "hqr_wg.hpp"

namespace hqr {

template <int QM>
HQR_DEV double tiny_sum(double (&x)[QM], bool sq)
{
    double t = 0.0;
#pragma unroll
    for (int q = 0; q < QM; ++q) t = sq ? fma(x[q], x[q], t) : fmax(t, fabs(x[q]));
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double y = __shfl_xor(t, o);
        t = sq ? t + y : fmax(t, y);
    }
    return t;
}

template <int W, int QM>
__global__ void __launch_bounds__(64) wg_tiny_kernel(WgDesc d, int *info, int *iters)
{
    __shared__ double rs[W][W + 1];   // [column][row] of R
    __shared__ double prow[W];
    const int lane = threadIdx.x;
    const int m = (int)d.m, n = (int)d.n, r = (int)d.nrhs;
    if (iters && lane == 0) *iters = 0;
    double a[QM][W];
#pragma unroll
    for (int j = 0; j < W; ++j) {
        // columns past the last repeat it (and become zeros below)
        const int c = min(j, n + r - 1);
        const double *col = (c < n) ? d.A + (size_t)c * d.lda : d.B + (size_t)(c - n) * d.ldb;
#pragma unroll
        for (int q = 0; q < QM; ++q) a[q][j] = col[min(lane + 64 * q, m - 1)];
    }
#pragma unroll
    for (int j = 0; j < W; ++j)
#pragma unroll
        for (int q = 0; q < QM; ++q) a[q][j] = (lane + 64 * q < m && j < n + r) ? a[q][j] : 0.0;
    double myup = 0.0;
#pragma unroll 1
    for (int k = 0; k < n; ++k) {
        if (lane == k) {
#pragma unroll
            for (int j = 0; j < W; ++j) prow[j] = a[0][j];
        }
        double xm[QM], tot[W / 16];
        bool nz = false;
#pragma unroll
        for (int q = 0; q < QM; ++q) {
            const int row = lane + 64 * q;
            xm[q] = (row > k && row < m) ? a[q][0] : 0.0;
            nz = nz || xm[q] != 0.0;
        }
#pragma unroll
        for (int h = 0; h < W / 16; ++h) {
            double s[16];
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                s[j] = 0.0;
#pragma unroll
                for (int q = 0; q < QM; ++q) s[j] = fma(a[q][16 * h + j], xm[q], s[j]);
            }
            tot[h] = wave_sum<16>(s, lane);   // column 16 h + lane / 4
        }
        __syncthreads();
        const double x0 = prow[0], sxx = readlane_f64(tot[0], 0);
        double upk = 0.0, sk = x0, inv_b = 0.0;
        if (__ballot(nz) != 0ull) {
            const double t = x0 * x0 + sxx;
            if (t >= 0x1p-920 && t <= 0x1p920) {
                double nu, rnu;
                wg_sqrt_rsqrt(t, nu, rnu);
                sk = (x0 >= 0.0) ? -nu : nu;
                upk = x0 - sk;
                inv_b = wg_recip(upk) * ((x0 >= 0.0) ? -rnu : rnu);
            } else {
                // the squares under- or overflow: scaled by the largest entry
                const double c = fmax(fabs(x0), tiny_sum<QM>(xm, false));
                double y[QM];
#pragma unroll
                for (int q = 0; q < QM; ++q) y[q] = xm[q] / c;
                const double x0c = x0 / c, nu = c * sqrt(x0c * x0c + tiny_sum<QM>(y, true));
                sk = (x0 >= 0.0) ? -nu : nu;
                upk = x0 - sk;
                inv_b = 1.0 / (upk * sk);
            }
        }
        if (lane == k) myup = upk;
        double wl[W / 16];
#pragma unroll
        for (int h = 0; h < W / 16; ++h) wl[h] = fma(upk, prow[16 * h + (lane >> 2)], tot[h]) * inv_b;
        // the pivot column is final: R above and on the diagonal, the tail below
#pragma unroll
        for (int q = 0; q < QM; ++q) {
            const int row = lane + 64 * q;
            const double v = (row == k) ? sk : a[q][0];
            if (row < m) d.A[(size_t)k * d.lda + row] = v;
            if (q == 0 && lane <= k) rs[k][lane] = v;
        }
        // apply the reflector (rows from k on; the others keep their values
        // exactly) and move the columns down
        double vr[QM];
        bool act[QM];
#pragma unroll
        for (int q = 0; q < QM; ++q) {
            const int row = lane + 64 * q;
            act[q] = row >= k && row < m;
            vr[q] = (row == k) ? upk : a[q][0];
        }
#pragma unroll
        for (int j = 1; j < W; ++j) {
            const double wj = readlane_f64(wl[j / 16], 4 * (j % 16));
#pragma unroll
            for (int q = 0; q < QM; ++q) {
                const double t = fma(wj, vr[q], a[q][j]);
                a[q][j - 1] = act[q] ? t : a[q][j];
            }
        }
#pragma unroll
        for (int q = 0; q < QM; ++q) a[q][W - 1] = 0.0;
        __syncthreads();
    }
    if (lane < n) d.up[lane] = myup;
    // registers 0 .. r-1 hold Q^T B
    const bool solve = (d.flags & WG_SOLVE) != 0;
    double rinv = 1.0;
    bool ok = false;
    if (solve) {
        const double rd = (lane < n) ? rs[lane][lane] : 1.0;
        const unsigned long long bad = __ballot(rd == 0.0);
        ok = bad == 0ull;
        if (lane == 0) info[d.index] = ok ? 0 : (int)__ffsll((long long)bad);
        rinv = 1.0 / rd;
    }
#pragma unroll 1
    for (int c = 0; c < r; ++c) {
        if (d.resnorm) {
            double x[QM];
#pragma unroll
            for (int q = 0; q < QM; ++q) x[q] = (lane + 64 * q >= n) ? a[q][0] : 0.0;
            const double mx = tiny_sum<QM>(x, false);
            double nrm;
            if (mx != 0.0 && !norm_fast_path_ok(mx)) {
#pragma unroll
                for (int q = 0; q < QM; ++q) x[q] /= mx;
                nrm = mx * sqrt(tiny_sum<QM>(x, true));
            } else {
                nrm = sqrt(tiny_sum<QM>(x, true));
            }
            if (lane == 0) d.resnorm[c] = nrm;
        }
        double t = a[0][0];
        if (ok) {
#pragma unroll 1
            for (int k = n - 1; k >= 0; --k) {
                const double xk = readlane_f64(t * rinv, k);
                const double rv = rs[k][min(lane, k)];
                t = (lane < k) ? fma(-rv, xk, t) : ((lane == k) ? xk : t);
            }
        }
#pragma unroll
        for (int q = 0; q < QM; ++q) {
            const int row = lane + 64 * q;
            if (row < m) d.B[(size_t)c * d.ldb + row] = (q == 0) ? t : a[q][0];
        }
#pragma unroll
        for (int j = 1; j < W; ++j)
#pragma unroll
            for (int q = 0; q < QM; ++q) a[q][j - 1] = a[q][j];
    }
}

} // namespace hqr
