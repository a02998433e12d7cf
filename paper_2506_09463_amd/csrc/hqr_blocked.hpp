// hqr_blocked.hpp -- blocked in-place Householder QR for problems that do not
// fit one workgroup.
//
// The matrix is processed in panels of NB columns (the coarsened "Task 1"
// of the paper's Alg. 3: alpha pivots generated back to back) followed by a
// blocked trailing update (the coarsened "Task 2" of Alg. 4, all of a panel's
// reflectors applied to the trailing columns at once).  On the GPU the
// trailing update is a compact-WY contraction on FP64 MFMA:
//     W  = V^T X            (split over rows, partial sums per split)
//     W' = T^T W            (T upper triangular, Q_panel = I - V T V^T)
//     X <- X - V W'
// where X = [trailing columns of A | B].  V's columns are the stored
// reflectors: v_k = (0..0, up_k, A[k+1:m, k]) with up_k kept in `up`.
//
// Panel factorization, one launch per pivot (panel_col_kernel): launch k
// applies reflector k-1 (derived from the reduced partial dot products of
// launch k-1) to every row chunk, then writes this launch's partial dot
// products of pivot column k, so every reflector is derived from the same
// data, in the same order, by every workgroup.
#pragma once

#include <utility>

#include "hqr_args.hpp"

#define HQR_HD __host__ __device__
#include "hqr_refine_rule.hpp"

namespace hqr {



__global__ void __launch_bounds__(256) panel_col_kernel(PanelArgs p)
{
    __shared__ double S[NB][PC_ROWS + 1];
    __shared__ double red[4][PW];
    __shared__ double wsh[NB];
    __shared__ double scal[4];

    const int tid = threadIdx.x, lane = tid & 63, g = tid >> 6;
    const int bw = p.bw, k = p.k, c0 = p.c0;
    const int64_t row_lo = (int64_t)c0 + (int64_t)blockIdx.x * PC_ROWS;
    const int64_t mp = p.m;
    const int nrow = (int)min<int64_t>((int64_t)PC_ROWS, mp - row_lo);

    // load my chunk (column-major in LDS)
    for (int idx = tid; idx < nrow * bw; idx += 256) {
        const int j = idx / nrow, r = idx - j * nrow;
        S[j][r] = HQR_AT(p.A, row_lo + r, c0 + j, p.lda);
    }
    __syncthreads();

    // ---- apply reflector k-1
    if (k > 0) {
        const int kp = k - 1;
        const int par = kp & 1;
        const double *X = p.xbuf + (size_t)par * p.nchunk * PW;
        const double *prow = p.pbuf + (size_t)par * NB;
        // reduced partials, same order in every workgroup: thread (value v,
        // quarter g4) sums chunks q = g4, g4+4, ...; quarters then summed 0..3
        for (int t = tid; t < 4 * PW; t += 256) {
            const int v = t % PW, g4 = t / PW;
            double acc4 = 0.0;
            if (v == NB) {
                for (int q = g4; q < p.nchunk; q += 4) acc4 = fmax(acc4, X[(size_t)q * PW + v]);
            } else {
#pragma unroll 4
                for (int q = g4; q < p.nchunk; q += 4) acc4 += X[(size_t)q * PW + v];
            }
            red[g4][v] = acc4;
        }
        __syncthreads();
        double d_j = 0.0;
        if (tid < bw) d_j = ((red[0][tid] + red[1][tid]) + red[2][tid]) + red[3][tid];
        if (tid == 0) {
            scal[0] = ((red[0][kp] + red[1][kp]) + red[2][kp]) + red[3][kp];
            scal[1] = fmax(fmax(red[0][NB], red[1][NB]), fmax(red[2][NB], red[3][NB]));
            scal[2] = ((red[0][NB + 1] + red[1][NB + 1]) + red[2][NB + 1]) + red[3][NB + 1];
        }
        __syncthreads();
        const double x0 = prow[kp];
        double up_k, s_k;
        if (scal[2] == 0.0) {
            up_k = 0.0;
            s_k = x0;
        } else {
            const double c = fmax(fabs(x0), scal[1]);
            double nu;
            if (norm_fast_path_ok(c)) {
                nu = sqrt(x0 * x0 + scal[0]);
            } else {
                // rare: the partials of this launch's pivot were not scaled;
                // recompute the scaled norm from the tail in global memory
                // (a deterministic single-thread loop, identical in every WG)
                double t = 0.0;
                const int64_t pr = (int64_t)c0 + kp;
                for (int64_t i = pr + 1; i < mp; ++i) {
                    const double y = HQR_AT(p.A, i, c0 + kp, p.lda) / c;
                    t += y * y;
                }
                const double x0c = x0 / c;
                nu = c * sqrt(x0c * x0c + t);
            }
            s_k = (x0 >= 0.0) ? -nu : nu;
            up_k = x0 - s_k;
        }
        const bool skip = (up_k == 0.0);
        const double b_k = up_k * s_k;
        if (tid < NB) wsh[tid] = (!skip && tid > kp && tid < bw) ? (up_k * prow[tid] + d_j) / b_k : 0.0;
        const int64_t prow_g = (int64_t)c0 + kp;
        if (blockIdx.x == 0 && tid == 0) p.up[c0 + kp] = up_k;
        __syncthreads();
        // rows of my chunk that are >= the pivot row
        if (!skip) {
            for (int idx = tid; idx < nrow * bw; idx += 256) {
                const int j = idx / nrow, r = idx - j * nrow;
                const int64_t gi = row_lo + r;
                if (j <= kp || gi < prow_g) continue;
                const double v = (gi == prow_g) ? up_k : S[kp][r];
                S[j][r] += wsh[j] * v;
            }
        }
        if (prow_g >= row_lo && prow_g < row_lo + nrow && tid == 0) S[kp][prow_g - row_lo] = s_k;
        __syncthreads();
    }

    // ---- partials of pivot column k (x = A[c0+k+1 : m, c0+k])
    if (k < bw) {
        const int par = k & 1;
        double *X = p.xbuf + (size_t)par * p.nchunk * PW;
        double *prow = p.pbuf + (size_t)par * NB;
        const int64_t pr = (int64_t)c0 + k;
        // thread (column j = lane, row group g)
        double acc = 0.0, mx = 0.0, nz = 0.0;
        for (int r = g; r < nrow; r += 4) {
            const int64_t gi = row_lo + r;
            if (gi <= pr) continue;
            const double xi = S[k][r];
            if (lane < bw) acc += xi * S[lane][r];
            mx = fmax(mx, fabs(xi));
            nz += (xi != 0.0) ? 1.0 : 0.0;
        }
        red[g][lane] = acc;
        if (lane == 0) {
            red[g][NB] = mx;
            red[g][NB + 1] = nz;
        }
        __syncthreads();
        if (tid < PW) {
            double v;
            if (tid == NB) v = fmax(fmax(red[0][NB], red[1][NB]), fmax(red[2][NB], red[3][NB]));
            else v = ((red[0][tid] + red[1][tid]) + red[2][tid]) + red[3][tid];
            X[(size_t)blockIdx.x * PW + tid] = v;
        }
        if (pr >= row_lo && pr < row_lo + nrow && tid < NB)
            prow[tid] = (tid < bw) ? S[tid][pr - row_lo] : 0.0;
    }
    __syncthreads();

    // store the chunk back
    for (int idx = tid; idx < nrow * bw; idx += 256) {
        const int j = idx / nrow, r = idx - j * nrow;
        HQR_AT(p.A, row_lo + r, c0 + j, p.lda) = S[j][r];
    }
}


// F32: operands rounded to FP32, FP32 MFMA with FP32 accumulation (the
// partial sums are stored widened to FP64).  WITHV: the first bw X columns
// are the panel's own V columns (the per-column panel mode forms V^T V there).
//
// Register budget: the prefetch loads are unconditional, with rows and
// columns clamped into the matrix and column addresses formed at each fetch
// (no per-thread pointer tables); the rows past the split, the columns past
// nx and the triangle of V near the pivot rows are applied by selects when
// the chunk is stored.  This keeps two waves per SIMD.
template <bool F32, bool WITHV>
__global__ void __launch_bounds__(256, 2) vtx_kernel(VtxArgs p)
{
    __shared__ double Vs[KC][NB + 1];
    __shared__ double Xs[KC][VTX_COLS + 1];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int x0 = blockIdx.x * VTX_COLS;
    const int64_t r_begin = (int64_t)p.c0 + (int64_t)blockIdx.y * p.split_rows;
    const int64_t r_end = min<int64_t>(p.m, r_begin + p.split_rows);

    f64x4 acc[8];
    f32x4 acc32[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
        acc32[t] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }

    // staging layout: thread t loads row t % KC of V columns t / KC + 8 q
    // and of X columns x0 + t / KC + 8 q
    constexpr int VPT = KC * NB / 256;       // V elements per thread
    constexpr int XPT = KC * VTX_COLS / 256; // X elements per thread
    const int sr = tid % KC, sc = tid / KC;  // sc in [0, 8)
    const int bwm = p.bw - 1;
    double upq[VPT];                         // up of this thread's V columns
#pragma unroll
    for (int q = 0; q < VPT; ++q) upq[q] = p.up[p.c0 + min(sc + 8 * q, bwm)];
    double vreg[VPT], xreg[XPT];
    auto fetch = [&](int64_t r0) {
        const int64_t gi0 = r0 + sr;
        const int64_t gi = (gi0 < r_end) ? gi0 : r_end - 1;
#pragma unroll
        for (int q = 0; q < VPT; ++q) vreg[q] = HQR_AT(p.A, gi, p.c0 + min(sc + 8 * q, bwm), p.lda);
#pragma unroll
        for (int q = 0; q < XPT; ++q) {
            const int x = min(x0 + sc + 8 * q, p.nx - 1);
            const double *col;
            if (WITHV && x < p.bw) {
                col = p.A + (size_t)(p.c0 + x) * p.lda;
            } else {
                const int xa = WITHV ? x - p.bw : x;
                col = (xa < p.ncA) ? p.A + (size_t)(p.c0 + p.bw + p.aoff + xa) * p.lda
                                   : p.B + (size_t)(xa - p.ncA) * p.ldb;
            }
            xreg[q] = __builtin_nontemporal_load(col + gi);
        }
    };
    // waits for the chunk's loads, then zeroes what lies outside and applies
    // the triangle of V (row offset d from the panel's first row)
    auto finish = [&](int64_t r0) {
#pragma unroll
        for (int q = 0; q < VPT; ++q) pin_f64(vreg[q]);
#pragma unroll
        for (int q = 0; q < XPT; ++q) pin_f64(xreg[q]);
        const int64_t gi0 = r0 + sr;
        const bool ok = gi0 < r_end;
        const int64_t d = gi0 - p.c0;
#pragma unroll
        for (int q = 0; q < VPT; ++q) {
            const int c = sc + 8 * q;
            const double v = (d < c) ? 0.0 : ((d == c) ? upq[q] : vreg[q]);
            vreg[q] = (ok && c < p.bw) ? v : 0.0;
        }
#pragma unroll
        for (int q = 0; q < XPT; ++q) {
            const int x = x0 + sc + 8 * q;
            // WITHV: X column x < bw is V column x, held by this thread as
            // vreg[q] (x < 64 only in tile 0, where x = sc + 8 q)
            double v = xreg[q];
            if (WITHV && q < VPT && x < p.bw) v = vreg[q < VPT ? q : 0];
            xreg[q] = (ok && x < p.nx) ? v : 0.0;
        }
    };
    if (r_begin < r_end) fetch(r_begin);
    for (int64_t r0 = r_begin; r0 < r_end; r0 += KC) {
        finish(r0);
#pragma unroll
        for (int q = 0; q < VPT; ++q) Vs[sr][sc + 8 * q] = vreg[q];
#pragma unroll
        for (int q = 0; q < XPT; ++q) Xs[sr][sc + 8 * q] = xreg[q];
        __syncthreads();
        if (r0 + KC < r_end) fetch(r0 + KC);
#pragma unroll 2
        for (int kk = 0; kk < KC; kk += 4) {
            const int kr = kk + (lane >> 4);
            const double a = Vs[kr][16 * w + (lane & 15)];
#pragma unroll
            for (int t = 0; t < 8; ++t) {
                const double b = Xs[kr][16 * t + (lane & 15)];
                if (F32)
                    acc32[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(to_f32(a), to_f32(b), acc32[t], 0, 0, 0);
                else
                    acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[t], 0, 0, 0);
            }
        }
        __syncthreads();
    }
    // FP64 MFMA: D[i][j] at lane j + 16*(i%4), register i/4;
    // FP32 MFMA: D[i][j] at lane j + 16*(i/4), register i%4
    double *out = p.wpart + (size_t)blockIdx.y * NB * p.nxpad;
#pragma unroll
    for (int t = 0; t < 8; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int i = F32 ? 16 * w + 4 * (lane >> 4) + r : 16 * w + 4 * r + (lane >> 4);
            const int x = x0 + 16 * t + (lane & 15);
            if (x < p.nxpad) out[(size_t)i * p.nxpad + x] = F32 ? (double)acc32[t][r] : acc[t][r];
        }
}





// W' = T^T X (or T X) for COLS columns per workgroup: X summed from the
// splits in order, then one 16-row tile of the product per wave on MFMA,
// block columns beyond T's triangle skipped.
//
// Bound: latency (X is small).  The splits' loads of all of a thread's
// elements and T's are in flight together; with one element after the other
// and the product as scalar loops over LDS a launch took
// 13.2 us in the wide Q application at 6001 x 700, 6.7 so.
template <int COLS>
__global__ void __launch_bounds__(256) wsolve_kernel(WArgs p)
{
    __shared__ double Ws[NB][COLS + 1];
    __shared__ double Ts[NB][NB + 1];
    constexpr int E = NB * COLS / 256, RS = 256 / COLS, U = 32 / E;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int xb = p.xoff + blockIdx.x * COLS, xe = p.xoff + p.ncols;
    const int c = tid % COLS, i0 = tid / COLS;
    double tv[16];
#pragma unroll
    for (int t = 0; t < 16; ++t) tv[t] = p.T[tid + 256 * t];
    const double *src[E];
    double s[E];
#pragma unroll
    for (int k = 0; k < E; ++k) {
        src[k] = p.wpart + (size_t)min(i0 + RS * k, p.bw - 1) * p.nxpad + min(xb + c, xe - 1);
        s[k] = 0.0;
    }
    const size_t stride = (size_t)NB * p.nxpad;
    for (int q0 = 0; q0 < p.nsplit; q0 += U) {
        double v[E][U];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int k = 0; k < E; ++k) v[k][u] = src[k][(size_t)min(q0 + u, p.nsplit - 1) * stride];
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int k = 0; k < E; ++k) pin_f64(v[k][u]);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int k = 0; k < E; ++k) s[k] += (q0 + u < p.nsplit) ? v[k][u] : 0.0;
    }
#pragma unroll
    for (int t = 0; t < 16; ++t) pin_f64(tv[t]);
#pragma unroll
    for (int t = 0; t < 16; ++t) Ts[w + 4 * t][lane] = tv[t];
#pragma unroll
    for (int k = 0; k < E; ++k) {
        const int i = i0 + RS * k;
        Ws[i][c] = (i < p.bw && xb + c < xe) ? s[k] : 0.0;
    }
    __syncthreads();
    const int i16 = lane & 15, kk = lane >> 4, i = 16 * w + i16;
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
        if (p.tmode == 0 ? kb > w : kb < w) continue;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = 16 * kb + 4 * q + kk;
            const double tr = (p.tmode == 0) ? Ts[k][i] : Ts[i][k];
            const bool in = (p.tmode == 0) ? (k <= i && i < p.bw) : (k >= i && k < p.bw);
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(in ? tr : 0.0, Ws[k][i16 % COLS], acc, 0, 0, 0);
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int row = 16 * w + 4 * r + kk, x = xb + i16;
        if (i16 < COLS && x < xe) p.wp[(size_t)row * p.nxpad + x] = (row < p.bw) ? acc[r] : 0.0;
    }
}


HQR_DEV double *col_ptr(const UpdArgs &p, int c)
{
    if (c < p.ncA) return p.A + (size_t)(p.c0 + p.bw + p.aoff + c) * p.lda;
    return p.B + (size_t)(c - p.ncA) * p.ldb;
}


// F32: V and W' rounded to FP32, the product accumulated in FP32 by FP32
// MFMA from zero, then subtracted from the FP64 trailing matrix.
template <bool F32>
__global__ void __launch_bounds__(256, 2) update_kernel(UpdArgs p)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int wr = w & 1, wc = w >> 1;
    const int64_t rb = (int64_t)p.c0 + (int64_t)blockIdx.x * UPD_TILE + 64 * wr;
    const int cb = blockIdx.y * UPD_TILE + 64 * wc;
    const int ncols = p.ncA + p.nB;
    if (rb >= p.m || cb >= ncols) return;
    const int li = lane & 15, lk = lane >> 4;
    const bool masked = rb < (int64_t)p.c0 + p.bw; // rows that meet the triangle of V

    // Loads are unconditional: rows and columns are clamped into the matrix.
    // A lane outside it only ever feeds accumulator entries that are never
    // stored, except through k >= bw, which is zeroed after the loads.
    int64_t gr[4];
    bool rok[4];
#pragma unroll
    for (int ti = 0; ti < 4; ++ti) {
        const int64_t gi = rb + 16 * ti + li;
        rok[ti] = gi < p.m;
        gr[ti] = rok[ti] ? gi : p.m - 1;
    }
    f64x4 acc[4][4]; // [column tile][row tile]
    f32x4 acc32[4][4];
    double *cptr[4][4];
    bool cok[4][4];
    // accumulator register r of lane (li, lk) holds column cb + 16 tj + ccol(r), row li
#define HQR_CCOL(r) (F32 ? 4 * lk + (r) : 4 * (r) + lk)
#pragma unroll
    for (int tj = 0; tj < 4; ++tj)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int c = cb + 16 * tj + HQR_CCOL(r);
            cok[tj][r] = c < ncols;
            cptr[tj][r] = col_ptr(p, cok[tj][r] ? c : 0);
        }
#pragma unroll
    for (int tj = 0; tj < 4; ++tj)
#pragma unroll
        for (int ti = 0; ti < 4; ++ti) {
            acc32[tj][ti] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int r = 0; r < 4; ++r)
                acc[tj][ti][r] = F32 ? 0.0 : __builtin_nontemporal_load(&cptr[tj][r][gr[ti]]);
        }

    const double *wrow = p.wp + p.xoff + cb + li;
    int wofs[4];
#pragma unroll
    for (int tj = 0; tj < 4; ++tj) wofs[tj] = (cb + 16 * tj + li < ncols) ? 16 * tj : 0;
    // raw operands of a k-step: W' row k, V column k and up_k (plain loads,
    // no branch); the triangle of V and k >= bw are applied after the pins
    double an[4], bn[4], un;
    auto issue = [&](int k0) {
        const int k = k0 + lk;
        const int kc = (k < p.bw) ? k : 0;
#pragma unroll
        for (int tj = 0; tj < 4; ++tj) an[tj] = wrow[(size_t)kc * p.nxpad + wofs[tj]];
#pragma unroll
        for (int ti = 0; ti < 4; ++ti) bn[ti] = HQR_AT(p.A, gr[ti], p.c0 + kc, p.lda);
        un = p.up[p.c0 + kc];
    };
    issue(0);
#pragma unroll 1
    for (int k0 = 0; k0 < NB; k0 += 4) {
        const int k = k0 + lk;
        const bool kok = k < p.bw;
        double a[4], b[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            pin_f64(an[q]);
            pin_f64(bn[q]);
        }
        pin_f64(un);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t d = rb + 16 * q + li - p.c0;   // row offset from the panel's first row
            const double v = (masked && d <= k) ? ((d == k) ? un : 0.0) : bn[q];
            a[q] = kok ? -an[q] : 0.0;
            b[q] = kok ? v : 0.0;
        }
        if (k0 + 4 < NB) issue(k0 + 4);
#pragma unroll
        for (int tj = 0; tj < 4; ++tj)
#pragma unroll
            for (int ti = 0; ti < 4; ++ti) {
                if (F32)
                    acc32[tj][ti] = __builtin_amdgcn_mfma_f32_16x16x4f32(to_f32(a[tj]), to_f32(b[ti]), acc32[tj][ti], 0, 0, 0);
                else
                    acc[tj][ti] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[tj], b[ti], acc[tj][ti], 0, 0, 0);
            }
    }
    if (F32) {
        // C += the FP32 product: the old values are loaded together first
#pragma unroll
        for (int tj = 0; tj < 4; ++tj)
#pragma unroll
            for (int ti = 0; ti < 4; ++ti)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[tj][ti][r] = __builtin_nontemporal_load(&cptr[tj][r][gr[ti]]);
    }
#pragma unroll
    for (int tj = 0; tj < 4; ++tj)
#pragma unroll
        for (int ti = 0; ti < 4; ++ti)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t gi = rb + 16 * ti + li;
                if (cok[tj][r] && rok[ti]) {
                    if (F32) __builtin_nontemporal_store(acc[tj][ti][r] + (double)acc32[tj][ti][r], &cptr[tj][r][gi]);
                    else __builtin_nontemporal_store(acc[tj][ti][r], &cptr[tj][r][gi]);
                }
            }
#undef HQR_CCOL
}

// X <- X - V W' for at most 64 columns (the next panel's columns on the
// critical path): grid ceil(rows / 64); wave w owns rows [64 bx + 16 w, +16)
// and all columns (four 16-column MFMA tiles), so the 64-deep contraction is
// spread over many waves instead of a few 64 x 64 tiles.  Same operand
// layout as update_kernel (D' = -W'^T V^T).
template <bool F32>
__global__ void __launch_bounds__(256) update_narrow_kernel(UpdArgs p)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t rb = (int64_t)p.c0 + (int64_t)blockIdx.x * 64 + 16 * w;
    const int ncols = p.ncA + p.nB;
    if (rb >= p.m) return; // no barriers below
    const int li = lane & 15, lk = lane >> 4;
    const int64_t gi = rb + li;
    const bool rok = gi < p.m;
    const int64_t gr = rok ? gi : p.m - 1;   // loads are unconditional (clamped, zeroed after)
    const bool masked = rb < (int64_t)p.c0 + p.bw;
#define HQR_NCOL(r) (F32 ? 4 * lk + (r) : 4 * (r) + lk)
    f64x4 acc[4];
    f32x4 acc32[4];
    double *cptr[4][4];
    bool cok[4][4];
#pragma unroll
    for (int tj = 0; tj < 4; ++tj) {
        acc32[tj] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int c = 16 * tj + HQR_NCOL(r);
            cok[tj][r] = c < ncols;
            cptr[tj][r] = col_ptr(p, cok[tj][r] ? c : 0);
            const double v = cptr[tj][r][gr];
            acc[tj][r] = (cok[tj][r] && rok) ? v : 0.0;
        }
    }
    // every operand is loaded before the first MFMA (80 values per lane, plus
    // up_k): plain loads first, all pinned, then the selects
    const double *wrow = p.wp + p.xoff + li;
    double a[NB / 4][4], bv[NB / 4], uv[NB / 4];
#pragma unroll
    for (int k4 = 0; k4 < NB / 4; ++k4) {
        const int k = 4 * k4 + lk;
        const int kc = (k < p.bw) ? k : 0;
#pragma unroll
        for (int tj = 0; tj < 4; ++tj) a[k4][tj] = wrow[(size_t)kc * p.nxpad + ((16 * tj + li < ncols) ? 16 * tj : 0)];
        bv[k4] = HQR_AT(p.A, gr, p.c0 + kc, p.lda);
        uv[k4] = p.up[p.c0 + kc];
    }
#pragma unroll
    for (int k4 = 0; k4 < NB / 4; ++k4) {
#pragma unroll
        for (int tj = 0; tj < 4; ++tj) pin_f64(a[k4][tj]);
        pin_f64(bv[k4]);
        pin_f64(uv[k4]);
    }
    const int64_t d = gi - p.c0;   // row offset from the panel's first row
#pragma unroll
    for (int k4 = 0; k4 < NB / 4; ++k4) {
        const int k = 4 * k4 + lk;
        const bool kok = k < p.bw;
#pragma unroll
        for (int tj = 0; tj < 4; ++tj) a[k4][tj] = (kok && 16 * tj + li < ncols) ? -a[k4][tj] : 0.0;
        const double b = (masked && d <= k) ? ((d == k) ? uv[k4] : 0.0) : bv[k4];
        bv[k4] = (kok && rok) ? b : 0.0;
    }
#pragma unroll
    for (int k4 = 0; k4 < NB / 4; ++k4) {
        const double b = bv[k4];
#pragma unroll
        for (int tj = 0; tj < 4; ++tj) {
            if (F32)
                acc32[tj] = __builtin_amdgcn_mfma_f32_16x16x4f32(to_f32(a[k4][tj]), to_f32(b), acc32[tj], 0, 0, 0);
            else
                acc[tj] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[k4][tj], b, acc[tj], 0, 0, 0);
        }
    }
#pragma unroll
    for (int tj = 0; tj < 4; ++tj)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (cok[tj][r] && rok) {
                if (F32) cptr[tj][r][gi] = acc[tj][r] + (double)acc32[tj][r];
                else cptr[tj][r][gi] = acc[tj][r];
            }
#undef HQR_NCOL
}

// ------------------------------------------------------------ triangular
// Before a back-substitution, in one launch: workgroup 0 sets info = smallest
// k+1 with R[k][k] == 0 (0 if none; with check), the others fill the published
// slots with TRSV_EMPTY.  Latency-bound: as a launch each, and with the
// diagonal read one dependent load after the other, the two took 4.0 and
// 3.2 us and the gap between them (n = 2048); together 4.5.
__global__ void __launch_bounds__(256) trsv_begin_kernel(TrsvArgs p, int check)
{
    if (p.active && *((volatile int *)p.active) == 0) return;
    if (blockIdx.x > 0) {
        const int64_t count = 2 * p.n * (int64_t)p.nrhs, step = (int64_t)(gridDim.x - 1) * 256;
        for (int64_t i = (int64_t)(blockIdx.x - 1) * 256 + threadIdx.x; i < count; i += step)
            ((int *)p.xpub)[i] = TRSV_EMPTY_WORD;
        return;
    }
    if (!check) return;
    __shared__ int first;
    if (threadIdx.x == 0) first = 0x7fffffff;
    __syncthreads();
    for (int64_t k0 = threadIdx.x; k0 < p.n; k0 += 8 * 256) {
        double d[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t k = min<int64_t>(k0 + 256 * u, p.n - 1);
            d[u] = HQR_AT(p.A, k, k, p.lda);
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) pin_f64(d[u]);
#pragma unroll
        for (int u = 0; u < 8; ++u)   // past the end: the last one again
            if (d[u] == 0.0) atomicMin(&first, (int)min<int64_t>(k0 + 256 * u, p.n - 1) + 1);
    }
    __syncthreads();
    if (threadIdx.x == 0) *p.info = (first == 0x7fffffff) ? 0 : first;
}

// Workgroup b owns TRSV_ROWS = 128 rows (for TRANS, R^T x = b by forward
// substitution and the blocks above it).  Positions 0 .. 127 are its rows in
// the order in which they are solved.  Everything that does not depend on
// other blocks is loaded before the first wait: the diagonal block, the
// block's right-hand sides, and each 64-column off-diagonal block of R one
// iteration ahead, in registers.  The critical path per block is then: poll
// the predecessor's last 64 x values until none holds TRSV_EMPTY (one read of
// memory shared by all XCDs, no separate flag and no cache invalidation), one
// 128 x 64 block product, a 128-step substitution with multiplies by the
// precomputed reciprocals, and the stores that publish the results, 64 at a
// time (no release fence: no other data rides on them).
//
// Bound: the serial chain of n steps and the handoffs between workgroups
// (about 1.5 us each).  One wave solves one right-hand side, lane l holding
// positions l and 64 + l: a step is a multiply, two lane reads and an FMA on
// the chain, and the second position's FMA beside it.  No step masks the
// positions already solved: their entries are stored as zeros.  Zero times a
// value that is not finite would change them, so a half that holds one is
// solved again with the masks.  Against 64-row blocks with masked steps and
// 1 or 8 right-hand sides per pass: 221 -> 141 us at n = 4096, one right-hand
// side; 167 -> 82 at n = 2000, four; R^T x = b at n = 2048, two: 160 -> 67.
// NR: right-hand sides of a pass (1, 2, 4 or 8).
constexpr int TRSV_NT = 512;

typedef double f64x4u __attribute__((ext_vector_type(4), aligned(8)));   // any element address

struct TrsvLane {
    double t0, t1;     // the running right-hand sides of positions l, 64 + l
    double r0, r1;     // 1 / diagonal
};

// position Q (of the half HALF): solves it and updates the rest; e0, e1 are
// the matrix entries of this position's column at l and 64 + l
template <int HALF, int Q> HQR_DEV void trsv_step(TrsvLane &s, double e0, double e1)
{
    const double xi = readlane_f64(HALF ? s.t1 * s.r1 : s.t0 * s.r0, Q);
    if (HALF == 0) s.t0 = fma(-e0, xi, s.t0);
    s.t1 = fma(-e1, xi, s.t1);
}

template <int HALF, int G, int... I>
HQR_DEV void trsv_steps(TrsvLane &s, const double (&e0)[16], const double (&e1)[16], std::integer_sequence<int, I...>)
{
    (trsv_step<HALF, 16 * G + I>(s, e0[I], e1[I]), ...);
}

// 16 steps with the next 16 columns' entries being read meanwhile; ends early
// at the last group that holds one of the nr rows
template <int HALF, int G>
HQR_DEV void trsv_half(TrsvLane &s, const double *S, int nr, int lane, double (&e0)[16], double (&e1)[16])
{
    constexpr int LD = HALF ? 65 : 129;
    double f0[16], f1[16];
    if constexpr (G < 3) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const double *col = S + (16 * (G + 1) + i) * LD;
            if (HALF == 0) f0[i] = col[lane];
            f1[i] = col[(HALF ? 0 : 64) + lane];
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    trsv_steps<HALF, G>(s, e0, e1, std::make_integer_sequence<int, 16>{});
    if constexpr (G < 3) {
        if (nr > 64 * HALF + 16 * (G + 1)) trsv_half<HALF, G + 1>(s, S, nr, lane, f0, f1);
    }
}

// the same with the solved positions left alone, for values that are not
// finite: returns the solution of position lane of the half
template <int HALF> HQR_DEV double trsv_masked(TrsvLane &s, const double *S, int nr, int lane)
{
    constexpr int LD = HALF ? 65 : 129;
    double x = 0.0;
    const int nq = min(nr - 64 * HALF, 64);
    for (int q = 0; q < nq; ++q) {
        const double xi = readlane_f64(HALF ? s.t1 * s.r1 : s.t0 * s.r0, q);
        if (HALF == 0 && lane > q) s.t0 = fma(-S[q * LD + lane], xi, s.t0);
        if (HALF == 0 || lane > q) s.t1 = fma(-S[q * LD + (HALF ? 0 : 64) + lane], xi, s.t1);
        x = (lane == q) ? xi : x;
    }
    return x;
}

template <bool TRANS, int NR>
__global__ void __launch_bounds__(TRSV_NT) trsv_kernel(TrsvArgs p)
{
    // S1[q][l]: entry of position q < 64 in the row of position l; S2[q][l]:
    // of position 64 + q in that of 64 + l
    __shared__ double S1[64][129], S2[64][65];
    __shared__ double xs[2][NR][64];
    __shared__ double part[4][NR][TRSV_ROWS];
    __shared__ int bad[2];
    const int tid = threadIdx.x, lane = tid & 63, pos = tid & (TRSV_ROWS - 1);
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), g = w >> 1;
    if (*((volatile int *)p.info) != 0) return;
    if (p.active && *((volatile int *)p.active) == 0) return;
    const int nblk = (int)((p.n + TRSV_ROWS - 1) / TRSV_ROWS);
    const int ib = TRANS ? (int)blockIdx.x : nblk - 1 - (int)blockIdx.x;
    const int64_t r0 = (int64_t)ib * TRSV_ROWS;
    const int nr = (int)min<int64_t>(TRSV_ROWS, p.n - r0);
    const int nrhs = p.nrhs;
    // row of position q; positions past the block repeat its last one (their
    // values are computed last and go nowhere)
    auto row = [&](int q) { return r0 + (TRANS ? min(q, nr - 1) : nr - 1 - min(q, nr - 1)); };
    if (tid < 2) bad[tid] = 0;
    // off-diagonal 64-column block of iteration jj: thread (position fp, group
    // fg) takes 16 of its columns.  TRANS reads rows of R^T, which lie along
    // R's columns: the four groups of a position are lanes of one wave and
    // take 4 consecutive elements of each 16, so that a load covers whole
    // lines of 16 columns (one position per lane touches 64 lines per load:
    // 141 us against 67 at n = 2048)
    const int nhalf = (int)((p.n + 63) / 64);
    const int npred = TRANS ? 2 * ib : max(nhalf - 2 * (ib + 1), 0);
    const int fp = TRANS ? 16 * w + (lane & 15) : pos, fg = TRANS ? lane >> 4 : g;
    const int64_t prow = row(fp);
    auto col = [&](int q) { return TRANS ? 16 * (q >> 2) + 4 * fg + (q & 3) : 16 * fg + q; };
    auto fetch = [&](int jj, double (&rv)[16]) {
        const int64_t c0 = (int64_t)(TRANS ? jj : nhalf - 1 - jj) * 64;
        if constexpr (TRANS) {   // 64 columns: only the last block has fewer
            const double *src = p.A + (size_t)prow * p.lda + c0 + 4 * fg;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const f64x4u v = *(const f64x4u *)(src + 16 * q);
#pragma unroll
                for (int e = 0; e < 4; ++e) rv[4 * q + e] = v[e];
            }
        } else {
            const int nc = (int)min<int64_t>(64, p.n - c0);
#pragma unroll
            for (int q = 0; q < 16; ++q) rv[q] = HQR_AT(p.A, prow, c0 + min(col(q), nc - 1), p.lda);
        }
    };
    double rv[16], rn[16];
    if (npred > 0) fetch(0, rv);
    // independent of the other blocks: the diagonal block, reciprocals of its
    // diagonal and own right-hand sides (wave c: right-hand side c)
    {
        double v1[16], v2[8];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int q = TRANS ? lane : g + 4 * k, l = TRANS ? w + 8 * k : pos;
            v1[k] = TRANS ? HQR_AT(p.A, row(q), row(l), p.lda) : HQR_AT(p.A, row(l), row(q), p.lda);
        }
        if (nr > 64) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int q = TRANS ? lane : w + 8 * k, l = TRANS ? w + 8 * k : lane;
                v2[k] = TRANS ? HQR_AT(p.A, row(64 + q), row(64 + l), p.lda) : HQR_AT(p.A, row(64 + l), row(64 + q), p.lda);
            }
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            const int q = TRANS ? lane : g + 4 * k, l = TRANS ? w + 8 * k : pos;
            S1[q][l] = (l > q) ? v1[k] : 0.0;
        }
        if (nr > 64) {
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int q = TRANS ? lane : w + 8 * k, l = TRANS ? w + 8 * k : lane;
                S2[q][l] = (l > q) ? v2[k] : 0.0;
            }
        }
    }
    TrsvLane sl;
    const bool solver = w < nrhs && w < NR;
    if (solver) {
        const int64_t ra = row(lane), rb = row(64 + lane);
        sl.t0 = HQR_AT(p.B, ra, w, p.ldb);
        sl.t1 = HQR_AT(p.B, rb, w, p.ldb);
        sl.r0 = 1.0 / HQR_AT(p.A, ra, ra, p.lda);
        sl.r1 = 1.0 / HQR_AT(p.A, rb, rb, p.lda);
        pin_f64(sl.r0);
        pin_f64(sl.r1);
    }
    double acc[NR];
#pragma unroll
    for (int c = 0; c < NR; ++c) acc[c] = 0.0;
    __syncthreads();
    // two buffers of x and of the timeout flag, one barrier per iteration: a
    // buffer is written again only past the next iteration's barrier
    for (int jj = 0; jj < npred; ++jj) {
        if (jj + 1 < npred) fetch(jj + 1, rn);
        const int64_t c0 = (int64_t)(TRANS ? jj : nhalf - 1 - jj) * 64;
        const int nc = (int)min<int64_t>(64, p.n - c0);
        if (w < NR) {
            unsigned long long u = 0;   // the bits of +0.0
            if (lane < nc && w < nrhs) {
                unsigned long long *slot = (unsigned long long *)(p.xpub + (size_t)w * p.n + (size_t)(c0 + lane));
                long spins = 0;
                while ((u = __hip_atomic_load(slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) == TRSV_EMPTY) {
                    if (++spins > p.spin_limit) {
                        bad[jj & 1] = 1;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
            }
            xs[jj & 1][w][lane] = __longlong_as_double((long long)u);
        }
        __syncthreads();
        if (bad[jj & 1]) {
            if (tid == 0) atomicExch(p.info, HQR_INFO_TIMEOUT);
            return;
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const double a = (col(q) < nc) ? rv[q] : 0.0;
#pragma unroll
            for (int c = 0; c < NR; ++c) acc[c] = fma(a, xs[jj & 1][c][col(q)], acc[c]);
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) rv[q] = rn[q];
    }
#pragma unroll
    for (int c = 0; c < NR; ++c) part[fg][c][fp] = acc[c];
    __syncthreads();
    if (!solver) return;
    sl.t0 -= ((part[0][w][lane] + part[1][w][lane]) + part[2][w][lane]) + part[3][w][lane];
    sl.t1 -= ((part[0][w][64 + lane] + part[1][w][64 + lane]) + part[2][w][64 + lane]) + part[3][w][64 + lane];
    // publish first (the successors wait on it), then the result
    auto publish = [&](int q, double x) {
        if (q < nr) {
            const int64_t r = row(q);
            unsigned long long u = (unsigned long long)__double_as_longlong(x);
            if (u == TRSV_EMPTY) u = 0x7FF8000000000000ull;
            __hip_atomic_store((unsigned long long *)(p.xpub + (size_t)w * p.n + (size_t)r), u, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
            p.B[(size_t)r + (size_t)w * p.ldb] = x;
        }
    };
    TrsvLane s0 = sl;
    double e0[16], e1[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        e0[i] = S1[i][lane];
        e1[i] = S1[i][64 + lane];
    }
    trsv_half<0, 0>(sl, &S1[0][0], nr, lane, e0, e1);
    double x = sl.t0 * sl.r0;
    if (__ballot(lane < nr && !(fabs(x) < __builtin_inf()))) {
        sl = s0;
        x = trsv_masked<0>(sl, &S1[0][0], nr, lane);
    }
    publish(lane, x);
    if (nr <= 64) return;
    s0 = sl;
#pragma unroll
    for (int i = 0; i < 16; ++i) e1[i] = S2[i][lane];
    trsv_half<1, 0>(sl, &S2[0][0], nr, lane, e0, e1);
    x = sl.t1 * sl.r1;
    if (__ballot(64 + lane < nr && !(fabs(x) < __builtin_inf()))) {
        sl = s0;
        x = trsv_masked<1>(sl, &S2[0][0], nr, lane);
    }
    publish(64 + lane, x);
}

// resnorm[c] = ||B[n:m, c]||, one workgroup per column.
__global__ void __launch_bounds__(256) resnorm_kernel(const double *B, int64_t ldb, int64_t n, int64_t m, double *out)
{
    __shared__ double ss[4], mxs[4];
    const int tid = threadIdx.x, lane = tid & 63, g = tid >> 6;
    const double *col = B + (size_t)blockIdx.x * ldb;
    double s = 0.0, mx = 0.0;
    for (int64_t i = n + tid; i < m; i += 256) {
        s += col[i] * col[i];
        mx = fmax(mx, fabs(col[i]));
    }
    for (int o = 32; o > 0; o >>= 1) {
        s += __shfl_xor(s, o);
        mx = fmax(mx, __shfl_xor(mx, o));
    }
    if (lane == 0) {
        ss[g] = s;
        mxs[g] = mx;
    }
    __syncthreads();
    const double tot = ((ss[0] + ss[1]) + ss[2]) + ss[3];
    const double gmx = fmax(fmax(mxs[0], mxs[1]), fmax(mxs[2], mxs[3]));
    if (gmx == 0.0 || norm_fast_path_ok(gmx)) {
        if (tid == 0) out[blockIdx.x] = sqrt(tot);
        return;
    }
    double t = 0.0;
    for (int64_t i = n + tid; i < m; i += 256) {
        const double y = col[i] / gmx;
        t += y * y;
    }
    for (int o = 32; o > 0; o >>= 1) t += __shfl_xor(t, o);
    __syncthreads();
    if (lane == 0) ss[g] = t;
    __syncthreads();
    if (tid == 0) out[blockIdx.x] = gmx * sqrt(((ss[0] + ss[1]) + ss[2]) + ss[3]);
}

// ------------------------------------------------------------ refinement
// r = b - A0 x (FP64) for RESID_ROWS rows (blockIdx.x) and up to RESID_NR
// right-hand sides (blockIdx.y), so A0 is streamed once per RESID_NR columns
// of x.  Lane l of wave w takes row l % 32 and lane group k = 2w + l / 32,
// which owns columns [64k, 64k + 64) of each 512-column chunk of x (staged in
// LDS): a load instruction reads two 256-byte column segments, and every lane
// keeps 16 loads in flight with two partial sums per right-hand side.  The
// eight groups' sums are combined in a fixed order (deterministic).  Columns
// that are frozen are skipped unless `all`.
constexpr int RESID_ROWS = 32, RESID_NR = 4, RESID_CHUNK = 512, RESID_UNROLL = 16;
__global__ void __launch_bounds__(256) resid_kernel(RefineArgs a, int all)
{
    __shared__ double xs[RESID_CHUNK][RESID_NR];
    __shared__ double red[8][RESID_ROWS][RESID_NR];
    const int tid = threadIdx.x, lane = tid & 63, row = lane & 31, grp = 2 * (tid >> 6) + (lane >> 5);
    if (!all && *((volatile int *)a.active) == 0) return;
    const int c0 = (int)blockIdx.y * RESID_NR;
    int act = 0;   // bit c: right-hand side c0 + c is computed
#pragma unroll
    for (int c = 0; c < RESID_NR; ++c)
        if (c0 + c < a.nrhs && (all || a.stat[4 * (c0 + c) + 3] == 0)) act |= 1 << c;
    if (act == 0) return;
    const int64_t i = (int64_t)blockIdx.x * RESID_ROWS + row;
    const bool rok = i < a.m;
    const double *arow = a.A0 + (rok ? i : 0);   // rows past m read row 0; discarded
    double s0[RESID_NR], s1[RESID_NR];
#pragma unroll
    for (int c = 0; c < RESID_NR; ++c) s0[c] = s1[c] = 0.0;
    for (int64_t j0 = 0; j0 < a.n; j0 += RESID_CHUNK) {
        const int nj = (int)min<int64_t>(RESID_CHUNK, a.n - j0);
        __syncthreads();
        {
            // all loads first (unconditional, at a clamped address: X[0] when
            // not needed), then the selects: no wait between the loads
            constexpr int PER = RESID_CHUNK * RESID_NR / 256;
            double v[PER];
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int idx = tid + 256 * q, j = idx / RESID_NR, c = idx - j * RESID_NR;
                const bool ok = j < nj && ((act >> c) & 1);
                v[q] = a.X[ok ? (size_t)(c0 + c) * a.ldx + (size_t)(j0 + j) : 0];
            }
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                const int idx = tid + 256 * q, j = idx / RESID_NR, c = idx - j * RESID_NR;
                const bool ok = j < nj && ((act >> c) & 1);
                xs[j][c] = ok ? v[q] : 0.0;
            }
        }
        __syncthreads();
        const int jb = 64 * grp;
        const int cnt = max(0, min(64, nj - jb));   // uniform over the 32-lane group
        const double *ap = arow + (size_t)(j0 + jb) * a.lda0;
        int jj = 0;
        for (; jj + RESID_UNROLL <= cnt; jj += RESID_UNROLL) {
            double av[RESID_UNROLL];
#pragma unroll
            for (int u = 0; u < RESID_UNROLL; ++u) av[u] = ap[(size_t)(jj + u) * a.lda0];
#pragma unroll
            for (int u = 0; u < RESID_UNROLL; u += 2) {
#pragma unroll
                for (int c = 0; c < RESID_NR; ++c) {
                    s0[c] = fma(av[u], xs[jb + jj + u][c], s0[c]);
                    s1[c] = fma(av[u + 1], xs[jb + jj + u + 1][c], s1[c]);
                }
            }
        }
        for (; jj < cnt; ++jj) {
            const double av = ap[(size_t)jj * a.lda0];
#pragma unroll
            for (int c = 0; c < RESID_NR; ++c) s0[c] = fma(av, xs[jb + jj][c], s0[c]);
        }
    }
#pragma unroll
    for (int c = 0; c < RESID_NR; ++c) red[grp][row][c] = s0[c] + s1[c];
    __syncthreads();
    if (tid < RESID_ROWS * RESID_NR) {
        const int r = tid % RESID_ROWS, c = tid / RESID_ROWS;
        const int64_t ir = (int64_t)blockIdx.x * RESID_ROWS + r;
        if (ir < a.m && ((act >> c) & 1)) {
            const double t = ((red[0][r][c] + red[1][r][c]) + (red[2][r][c] + red[3][r][c])) +
                             ((red[4][r][c] + red[5][r][c]) + (red[6][r][c] + red[7][r][c]));
            a.rvec[(size_t)(c0 + c) * a.m + ir] = a.borig[(size_t)(c0 + c) * a.m + ir] - t;
        }
    }
}

// g = A0^T r for column blockIdx.y (FP64): one wave per column of A0, lanes
// down the rows.
__global__ void __launch_bounds__(256) gemvt_kernel(RefineArgs a)
{
    const int c = blockIdx.y;
    if (*((volatile int *)a.active) == 0 || a.stat[4 * c + 3]) return;
    const int lane = threadIdx.x & 63;
    const int64_t j = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (j >= a.n) return;
    const double *aj = a.A0 + (size_t)j * a.lda0;
    const double *r = a.rvec + (size_t)c * a.m;
    double s = 0.0;
    for (int64_t i = lane; i < a.m; i += 64) s += aj[i] * r[i];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
    if (lane == 0) a.gvec[(size_t)c * a.n + j] = s;
}

// One correction step for column blockIdx.x: x += dx, then the stopping rule
// of hqr_refine_rule.hpp on ||dx|| and ||x||.  A column that converges or
// fails is frozen (its x stays as it is) and leaves the active count.
__global__ void __launch_bounds__(1024) csne_update_kernel(RefineArgs a, int step)
{
    __shared__ double s1[16], s2[16];
    const int c = blockIdx.x;
    int *st = a.stat + 4 * c;
    if (*((volatile int *)a.active) == 0 || st[3]) return;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    double *x = a.X + (size_t)c * a.ldx;
    const double *dx = a.gvec + (size_t)c * a.n;
    double sa = 0.0, sb = 0.0;
    for (int64_t j = tid; j < a.n; j += 1024) {
        const double xn = x[j] + dx[j];
        x[j] = xn;
        sa += dx[j] * dx[j];
        sb += xn * xn;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        sa += __shfl_xor(sa, o);
        sb += __shfl_xor(sb, o);
    }
    if (lane == 0) {
        s1[w] = sa;
        s2[w] = sb;
    }
    __syncthreads();
    if (tid == 0) {
        double da = 0.0, xb = 0.0;
        for (int q = 0; q < 16; ++q) {
            da += s1[q];
            xb += s2[q];
        }
        RefineState rs{st[0], st[1], st[2], st[3], a.dxprev[c]};
        refine_rule_step(rs, step, sqrt(da), sqrt(xb), a.tol, REFINE_STALL_FLOOR);
        st[0] = rs.first;
        st[1] = rs.failed;
        st[2] = rs.stalls;
        st[3] = rs.frozen;
        a.dxprev[c] = rs.prev;
        if (rs.frozen) atomicSub(a.active, 1);
    }
}

// Initial state of a refinement run: every column active.
__global__ void refine_init_kernel(RefineArgs a)
{
    for (int i = threadIdx.x; i < 4 * a.nrhs; i += blockDim.x) a.stat[i] = 0;
    for (int i = threadIdx.x; i < a.nrhs; i += blockDim.x) a.dxprev[i] = 0.0;
    if (threadIdx.x == 0) *a.active = a.nrhs;
}

// Outcome of a refinement run: verdict[0] = 1 when every column converged;
// iters = the largest first-converged step (max_iter when some column did
// not converge); with or_info, HQR_INFO_NOCONV is ORed into *info when not
// every column converged.  One thread.
__global__ void refine_verdict_kernel(RefineArgs a, int *verdict, int *info, int *iters, int or_info)
{
    if (threadIdx.x != 0) return;
    int conv = 1, it = 0;
    for (int c = 0; c < a.nrhs; ++c) {
        const int *st = a.stat + 4 * c;
        if (st[0] == 0 || st[1]) conv = 0;
        it = max(it, st[0]);
    }
    if (!conv) it = a.max_iter;
    if (verdict) *verdict = conv;
    if (iters) *iters = it;
    if (or_info && !conv && info) *info |= HQR_INFO_NOCONV;
}

// Q (m x k, leading dimension ldq) <- the leading k columns of the m x m
// identity; grid-stride over the k columns.
__global__ void __launch_bounds__(256) eye_kernel(double *Q, int64_t ldq, int64_t m, int64_t k)
{
    for (int64_t j = blockIdx.x; j < k; j += gridDim.x) {
        double *col = Q + (size_t)j * ldq;
        for (int64_t i = threadIdx.x; i < m; i += 256) col[i] = (i == j) ? 1.0 : 0.0;
    }
}

// *p |= v (one thread).
__global__ void or_int_kernel(int *p, int v)
{
    if (threadIdx.x == 0) *p |= v;
}

__global__ void fill_int_kernel(int *p, int v, int64_t count)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

} // namespace hqr
