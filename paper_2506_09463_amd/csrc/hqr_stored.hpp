// hqr_stored.hpp -- applying a stored factorization (Q^T B or Q B from A and
// up): the compact-WY factors T of all panels at once, and the panel by panel
// application to few columns with one launch per panel.
#pragma once

#include "hqr_chol64.hpp"

namespace hqr {

// A 64 x 64 tile of the panel (c0, bw)'s V: rows r0 .. r0+63 (zero past m),
// columns past bw zero, up on the diagonal and zeros above it.  256 threads;
// loads clamped into the matrix, all in flight together.
// Thread tid takes row tid % 64 of every fourth column, so at most one of its
// elements is on the diagonal: one up per thread.
HQR_DEV void sv_issue(double (&v)[16], double &u, const double *A, int64_t lda, const double *up, int64_t m,
                      int64_t r0, int c0, int bw, int tid)
{
    const int64_t gi = r0 + (tid & 63), row = min<int64_t>(gi, m - 1);
    const int64_t d = min<int64_t>(max<int64_t>(gi - c0, 0), bw - 1);
#pragma unroll
    for (int q = 0; q < 16; ++q) v[q] = HQR_AT(A, row, c0 + min((tid >> 6) + 4 * q, bw - 1), lda);
    u = up[c0 + d];
}

HQR_DEV void sv_store(double (*M)[LD65], double (&v)[16], double &u, int64_t m, int64_t r0, int c0, int bw, int tid)
{
#pragma unroll
    for (int q = 0; q < 16; ++q) pin(v[q]);
    pin(u);
    const int r = tid & 63;
    const int64_t d = r0 + r - c0;   // row offset from the panel's first row
    const bool ok = r0 + r < m;
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int c = (tid >> 6) + 4 * q;
        const double e = (d < c) ? 0.0 : ((d == c) ? u : v[q]);
        M[r][c] = (ok && c < bw) ? e : 0.0;
    }
}

// grid: (panels, splits).  Partial V^T V of panel blockIdx.x over the rows of
// split blockIdx.y (whole 64-row tiles from the panel's first row).
__global__ void __launch_bounds__(256) stored_gram_kernel(StoredGramArgs p)
{
    __shared__ double V[NB][LD65];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int c0 = (int)blockIdx.x * NB, bw = min(NB, (int)p.n - c0);
    const int64_t tiles = (p.m - c0 + 63) / 64, per = (tiles + gridDim.y - 1) / gridDim.y;
    const int64_t t0 = (int64_t)blockIdx.y * per, t1 = min<int64_t>(tiles, t0 + per);
    f64x4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
    for (int64_t t = t0; t < t1; ++t) {
        double v[16], u;
        sv_issue(v, u, p.A, p.lda, p.up, p.m, c0 + 64 * t, c0, bw, tid);
        __syncthreads();
        sv_store(V, v, u, p.m, c0 + 64 * t, c0, bw, tid);
        __syncthreads();
#pragma unroll 4
        for (int k0 = 0; k0 < NB; k0 += 4) {
            const int kr = k0 + (lane >> 4);
            const double a = V[kr][16 * w + (lane & 15)];
#pragma unroll
            for (int q = 0; q < 4; ++q)
                acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, V[kr][16 * q + (lane & 15)], acc[q], 0, 0, 0);
        }
    }
    double *out = p.gpart + ((size_t)blockIdx.x * gridDim.y + blockIdx.y) * NB * NB;
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int r = 0; r < 4; ++r) out[(16 * w + 4 * r + (lane >> 4)) * NB + 16 * q + (lane & 15)] = acc[q][r];
}

// One step of the application to at most SN_COLS columns of B, one workgroup
// per SN part of `tiles` 64-row tiles from row `base`:
//   with a previous panel (bwp > 0): W = T^T X or T X from the parts' sums of
//     its X = V^T B, and B -= V W on the workgroup's rows;
//   with a next panel (bw > 0): the part's X = V^T B of the updated rows.
// So a panel costs one launch (rows of V are read twice, B once), where V^T B,
// T, W' and the update were four.  Every workgroup sums the same parts in the
// same order.  Bound: latency (launch, one round of loads, three 64-deep
// MFMA products, the stores).  2047 x 1500, three columns, on MI355X: 11.0 us a
// panel, Q^T b and the solve 0.376 ms; four launches of 7 to 20 us and 1.31 ms
// before.
__global__ void __launch_bounds__(256) stored_step_kernel(StoredStepArgs p)
{
    __shared__ double Vp[NB][LD65];
    __shared__ double Vc[NB][LD65];
    __shared__ double Ts[NB][LD65];
    __shared__ double Xs[4][NB][SN_COLS + 1];
    __shared__ double Ws[NB][SN_COLS + 1];
    __shared__ double Bt[NB][SN_COLS + 1];
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int i16 = lane & 15, kk = lane >> 4, nc = p.nrhs;
    const int64_t row0 = p.base + 64 * (int64_t)p.tiles * blockIdx.x;
    double pv[16], pu, cv[16], cu, tv[16], bv[4];
    auto issue = [&](int64_t r0) {
        if (p.bwp > 0) sv_issue(pv, pu, p.A, p.lda, p.up, p.m, r0, p.cp, p.bwp, tid);
        if (p.bw > 0) sv_issue(cv, cu, p.A, p.lda, p.up, p.m, r0, p.c0, p.bw, tid);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int idx = tid + 256 * q, c = min(idx >> 6, nc - 1);
            bv[q] = HQR_AT(p.B, min<int64_t>(r0 + (idx & 63), p.m - 1), c, p.ldb);
        }
    };
    issue(row0);
    if (p.bwp > 0) {
#pragma unroll
        for (int q = 0; q < 16; ++q) tv[q] = p.T[tid + 256 * q];
        // X: thread (reflector lane, quarter w) sums parts w, w + 4, ..; the
        // loads of eight parts and four columns in flight together
        for (int c0 = 0; c0 < nc; c0 += 4) {
            double sum[4] = {0.0, 0.0, 0.0, 0.0};
            for (int q0 = w; q0 < p.nparts; q0 += 32) {
                double x[8][4];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const int q = q0 + 4 * u;
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        x[u][c] = p.xin[((size_t)((q < p.nparts) ? q : w) * nc + min(c0 + c, nc - 1)) * NB + lane];
                }
#pragma unroll
                for (int u = 0; u < 8; ++u)
#pragma unroll
                    for (int c = 0; c < 4; ++c) pin(x[u][c]);
#pragma unroll
                for (int u = 0; u < 8; ++u)
#pragma unroll
                    for (int c = 0; c < 4; ++c) sum[c] += (q0 + 4 * u < p.nparts) ? x[u][c] : 0.0;
            }
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (c0 + c < nc) Xs[w][lane][c0 + c] = sum[c];
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) pin(tv[q]);
#pragma unroll
        for (int q = 0; q < 16; ++q) Ts[(tid + 256 * q) >> 6][tid & 63] = tv[q];
        __syncthreads();
        f64x4 acc = {0.0, 0.0, 0.0, 0.0};
        const int cc = min(i16, nc - 1);
#pragma unroll 4
        for (int k0 = 0; k0 < NB; k0 += 4) {
            const int k = k0 + kk, i = 16 * w + i16;
            const double a = p.tmode ? Ts[i][k] : Ts[k][i];
            const double x = ((Xs[0][k][cc] + Xs[1][k][cc]) + Xs[2][k][cc]) + Xs[3][k][cc];
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(a, (i16 < nc) ? x : 0.0, acc, 0, 0, 0);
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) Ws[16 * w + 4 * r + kk][i16] = acc[r];
    }
    f64x4 xacc = {0.0, 0.0, 0.0, 0.0};
    for (int t = 0; t < p.tiles; ++t) {
        const int64_t r0 = row0 + 64 * (int64_t)t;
        if (r0 >= p.m) break;
        if (t > 0) {
            issue(r0);
            __syncthreads();   // the previous tile's products have read the LDS tiles
        }
        if (p.bwp > 0) sv_store(Vp, pv, pu, p.m, r0, p.cp, p.bwp, tid);
        if (p.bw > 0) sv_store(Vc, cv, cu, p.m, r0, p.c0, p.bw, tid);
#pragma unroll
        for (int q = 0; q < 4; ++q) pin(bv[q]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int idx = tid + 256 * q, c = idx >> 6, r = idx & 63;
            Bt[r][c] = (c < nc && r0 + r < p.m) ? bv[q] : 0.0;
        }
        __syncthreads();
        if (p.bwp > 0) {
            f64x4 acc;
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] = Bt[16 * w + 4 * r + kk][i16];
#pragma unroll 4
            for (int k0 = 0; k0 < NB; k0 += 4)
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-Vp[16 * w + i16][k0 + kk], Ws[k0 + kk][i16], acc, 0, 0, 0);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                // rows above the previous panel are not its to change
                const int row = 16 * w + 4 * r + kk;
                if (r0 + row >= p.cp) Bt[row][i16] = acc[r];
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int idx = tid + 256 * q, c = idx >> 6, r = idx & 63;
                if (c < nc && r0 + r < p.m) HQR_AT(p.B, r0 + r, c, p.ldb) = Bt[r][c];
            }
        }
        if (p.bw > 0) {
#pragma unroll 4
            for (int k0 = 0; k0 < NB; k0 += 4) {
                // rows above the panel do not enter its sums (0 times a value
                // that is not finite would)
                const double b = (r0 + k0 + kk >= p.c0) ? Bt[k0 + kk][i16] : 0.0;
                xacc = __builtin_amdgcn_mfma_f64_16x16x4f64(Vc[k0 + kk][16 * w + i16], b, xacc, 0, 0, 0);
            }
        }
    }
    if (p.bw > 0 && i16 < nc) {
        double *out = p.xout + ((size_t)blockIdx.x * nc + i16) * NB + 16 * w;
#pragma unroll
        for (int r = 0; r < 4; ++r) out[4 * r + kk] = xacc[r];
    }
}

} // namespace hqr
