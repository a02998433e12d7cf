// hqr_chol.hpp -- Cholesky factorization S = R^T R of a symmetric positive
// definite matrix (the factored form in which SLSQP keeps its Hessian
// approximation) and the rank-one update R'^T R' = R^T R + v v^T (which is
// also the update of a QR factorization's R when a row is appended).
//
// Factorization, right-looking by 64-column blocks k, two launches each:
//   chol_panel_kernel  R_kj = R_kk^{-T} S_kj for the block row (FP64 MFMA)
//   chol_syrk_kernel   S_ij -= R_ki^T R_kj on the trailing upper blocks; the
//                      workgroup of the next diagonal block factors it and
//                      leaves R_kk^{-1} for the next block row
// (the first diagonal block by chol_syrk_kernel without an update).  Only the
// upper triangle of S is read or written.
#pragma once

#include "hqr_chol64.hpp"

namespace hqr {

// out[i][j] = sum_k A[k][i] B[k][j] for 64 x 64 LDS matrices (row-major,
// stride 65), FP64 MFMA; 256 threads, wave w computes rows 16w..16w+15.
// Returned in D layout: acc[t][r] = out[16w + 4r + l/16][16t + l%16].
HQR_DEV void ch_mm64(f64x4 (&acc)[4], const double (*A)[LD65], const double (*B)[LD65], int lane, int w)
{
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (int k0 = 0; k0 < 64; k0 += 4) {
        const int kr = k0 + (lane >> 4);
        const double a = A[kr][16 * w + (lane & 15)];
#pragma unroll
        for (int t = 0; t < 4; ++t)
            acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, B[kr][16 * t + (lane & 15)], acc[t], 0, 0, 0);
    }
}

struct CholArgsS {
    double *S;
    int64_t lds;
    int64_t n;
    int64_t k0;       // first row/column of the block row
    int bw;           // its height (<= 64; 0: no update, the first diagonal block)
    double *rinv;     // [64][64] row-major inverse of the newest diagonal block
    int *info;        // 0, or j+1 at the first non-positive pivot
};

// Whether a pivot before row `before` failed; the same answer for every thread
// of every workgroup: a launch passes the rows that were factored before it,
// so a failure that its own workgroup 0 reports meanwhile does not count, and
// each tile's update is either done in full or not at all.
HQR_DEV bool chol_failed(const int *info, int64_t before, int *sh)
{
    if (threadIdx.x == 0) *sh = *((volatile const int *)info);
    __syncthreads();
    return *sh != 0 && *sh <= before;
}

// A 64 x 64 tile of S at (r0, c0), rows < nr and columns < nc, zeros outside:
// unconditional loads (clamped into the tile), all 16 of a thread in flight.
HQR_DEV void chol_tile_issue(double (&v)[16], const double *S, int64_t lds, int64_t r0, int64_t c0, int nr, int nc,
                             int tid)
{
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int idx = tid + 256 * q, r = idx & 63, c = idx >> 6;
        v[q] = HQR_AT(S, r0 + ((r < nr) ? r : 0), c0 + ((c < nc) ? c : 0), lds);
    }
}

HQR_DEV void chol_tile_store(double (*M)[LD65], double (&v)[16], int nr, int nc, int tid)
{
#pragma unroll
    for (int q = 0; q < 16; ++q) pin(v[q]);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int idx = tid + 256 * q, r = idx & 63, c = idx >> 6;
        M[r][c] = (r < nr && c < nc) ? v[q] : 0.0;
    }
}

// grid: ceil((n - k0 - bw) / 64) column tiles j of the block row:
// R_kj = R_kk^{-T} S_kj (64 x 64 each), written over S_kj.  Bound: latency
// (one tile per workgroup: two loads, 64 MFMAs, a store).
__global__ void __launch_bounds__(256) chol_panel_kernel(CholArgsS a)
{
    __shared__ double Ri[64][LD65];
    __shared__ double Sk[64][LD65];
    __shared__ int failed;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int64_t c0 = a.k0 + a.bw + (int64_t)blockIdx.x * 64;
    const int nc = (int)min<int64_t>(64, a.n - c0);
    double rv[16], sv[16];
    chol_tile_issue(sv, a.S, a.lds, a.k0, c0, a.bw, nc, tid);
#pragma unroll
    for (int q = 0; q < 16; ++q) rv[q] = a.rinv[tid + 256 * q];
    if (chol_failed(a.info, a.k0 + a.bw, &failed)) return;
    chol_tile_store(Sk, sv, a.bw, nc, tid);
#pragma unroll
    for (int q = 0; q < 16; ++q) pin(rv[q]);
#pragma unroll
    for (int q = 0; q < 16; ++q) Ri[(tid + 256 * q) >> 6][tid & 63] = rv[q];
    __syncthreads();
    f64x4 acc[4];
    ch_mm64(acc, Ri, Sk, lane, w);
    // through LDS, so that the stores run down the columns
    __syncthreads();
#pragma unroll
    for (int t = 0; t < 4; ++t) st_blk(Sk, 16 * w, 16 * t, acc[t], 1.0, lane);
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int idx = tid + 256 * q, r = idx & 63, c = idx >> 6;
        if (r < a.bw && c < nc) HQR_AT(a.S, a.k0 + r, c0 + c, a.lds) = Sk[r][c];
    }
}

// What chol64_dpp does (ratio 0), with square roots and divisions that hold for
// infinite pivots: x / inf = 0, where chol64_dpp's reciprocal roots give
// inf * 0.  One column per step and four barriers: for blocks that have one.
HQR_DEV void chol64_inf(double (*G)[LD65], double (*X)[LD65], int n, int tid, int *bad)
{
    __syncthreads();
    if (tid == 0) *bad = 0;
    for (int e = tid; e < NB * NB; e += 256) {
        const int r = e >> 6, c = e & 63;
        X[r][c] = 0.0;
        if (r == c && r >= n) G[r][c] = 1.0;
    }
    __syncthreads();
    for (int p = 0; p < n; ++p) {
        const double piv = G[p][p];
        if (!(piv > 0.0)) {   // the same for every thread
            if (tid == 0) *bad = p + 1;
            break;
        }
        const double rpp = sqrt(piv);
        __syncthreads();
        if (tid >= p && tid < NB) G[p][tid] = (tid == p) ? rpp : G[p][tid] / rpp;
        __syncthreads();
        for (int e = tid; e < NB * NB; e += 256) {
            const int i = e >> 6, j = e & 63;
            if (i > p && j >= i) G[i][j] -= G[p][i] * G[p][j];
        }
        __syncthreads();
    }
    __syncthreads();
    if (*bad == 0 && tid < NB) {
        for (int i = tid; i >= 0; --i) {
            double t = (i == tid) ? 1.0 : 0.0;
            for (int l = i + 1; l <= tid; ++l) t -= G[i][l] * X[l][tid];
            X[i][tid] = t / G[i][i];
        }
    }
    __syncthreads();
}

// grid: the T (T + 1) / 2 upper tiles of the trailing matrix, T = ceil((n -
// k0 - bw) / 64), column by column (tile 0 is the next diagonal block; one
// tile when bw == 0): S_ij -= R_ki^T R_kj, on diagonal tiles the upper
// triangle.  Workgroup 0 then factors its block in LDS (chol64_dpp), writes R
// over its upper triangle and R^{-1} to rinv; a non-positive pivot p sets
// *info = (its first row) + p + 1 instead.
//
// Bound: the chain of diagonal blocks, so the factorization of block k + 1
// starts with the update of its own tile, beside the other tiles.  2000 x
// 2000 on MI355X: 0.91 ms (21 us per launch here, 15 of them the diagonal
// block, 7 us per block row), against 5.6 ms with a diagonal kernel of its
// own that worked through four barriers a pivot (141 us per block).
__global__ void __launch_bounds__(256) chol_syrk_kernel(CholArgsS a)
{
    __shared__ double Ri[64][LD65];
    __shared__ double Rj[64][LD65];
    __shared__ double gdiag[64], rdiag[64];
    __shared__ int sh;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    // column of the tile: largest by with by (by + 1) / 2 <= blockIdx.x
    int by = (int)((sqrtf(8.0f * (float)blockIdx.x + 1.0f) - 1.0f) * 0.5f);
    while ((by + 1) * (by + 2) / 2 <= (int)blockIdx.x) ++by;
    while (by * (by + 1) / 2 > (int)blockIdx.x) --by;
    const int bx = (int)blockIdx.x - by * (by + 1) / 2;
    const int64_t t0 = a.k0 + a.bw;
    const int64_t ri = t0 + (int64_t)bx * 64, cj = t0 + (int64_t)by * 64;
    const int ni = (int)min<int64_t>(64, a.n - ri), nj = (int)min<int64_t>(64, a.n - cj);
    const bool diag = bx == by;
    double iv[16], jv[16], sv[16];
    if (a.bw > 0) {
        chol_tile_issue(iv, a.S, a.lds, a.k0, ri, a.bw, ni, tid);
        chol_tile_issue(jv, a.S, a.lds, a.k0, cj, a.bw, nj, tid);
    }
    // of a diagonal tile's lower triangle only the mirrored entries are read
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int idx = tid + 256 * q, r = min(idx & 63, ni - 1), c = min(idx >> 6, nj - 1);
        const bool mirror = diag && r > c;
        sv[q] = HQR_AT(a.S, ri + (mirror ? c : r), cj + (mirror ? r : c), a.lds);
    }
    if (chol_failed(a.info, t0, &sh)) return;
    if (a.bw > 0) {
        chol_tile_store(Ri, iv, a.bw, ni, tid);
        chol_tile_store(Rj, jv, a.bw, nj, tid);
        __syncthreads();
        f64x4 acc[4];
        ch_mm64(acc, Ri, Rj, lane, w);
        __syncthreads();
#pragma unroll
        for (int t = 0; t < 4; ++t) st_blk(Rj, 16 * w, 16 * t, acc[t], 1.0, lane);
        __syncthreads();
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) pin(sv[q]);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int idx = tid + 256 * q, r = idx & 63, c = idx >> 6;
        if (a.bw > 0) sv[q] -= Rj[r][c];
        if (blockIdx.x > 0 && r < ni && c < nj && (!diag || r <= c)) HQR_AT(a.S, ri + r, cj + c, a.lds) = sv[q];
    }
    if (blockIdx.x > 0) return;
    // the next diagonal block; the two triangles of its update agree bitwise
    auto block = [&] {
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int idx = tid + 256 * q, r = idx & 63, c = idx >> 6;
            Ri[r][c] = (r < ni && c < nj) ? sv[q] : 0.0;
        }
    };
    block();
    chol64_dpp(Ri, Rj, ni, lane, w, 0.0, gdiag, rdiag, &sh);
    // an infinite pivot leaves a NaN in rdiag (every wave sees all 64)
    if (__ballot(lane < ni && !(rdiag[lane] < __builtin_inf()))) {
        __syncthreads();
        block();
        chol64_inf(Ri, Rj, ni, tid, &sh);
    }
    if (sh) {
        // the block stays as its update left it
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int idx = tid + 256 * q, r = idx & 63, c = idx >> 6;
            if (a.bw > 0 && r < ni && c < nj && r <= c) HQR_AT(a.S, ri + r, cj + c, a.lds) = sv[q];
        }
        if (tid == 0) *((volatile int *)a.info) = (int)(ri + sh);
        return;
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int idx = tid + 256 * q, r = idx & 63, c = idx >> 6;
        a.rinv[idx] = Rj[idx >> 6][idx & 63];
        if (r < ni && c < nj && r <= c) HQR_AT(a.S, ri + r, cj + c, a.lds) = Ri[r][c];
    }
}

// ------------------------------------------------------------ rank-one update
// Row k's rotation (c, s) turns (R_kk, v_k) into (r, 0) with r of R_kk's sign
// (so c >= 0) and is applied to (R_kj, v_j) for j > k.  The rotations of a row
// are kept in v's own slot (their v_k is 0 from then on), as one number rho
// from which both are recovered to rounding (Stewart's storage, c >= 0):
// s / 2 when |s| < c, else sign(s) 2 / c (infinite when c = 0).
HQR_DEV double rot_pack(double c, double s)
{
    return (fabs(s) < c) ? 0.5 * s : ((s == s) ? copysign(2.0 / c, s) : s);   // NaN stays one
}

HQR_DEV void rot_unpack(double rho, double &c, double &s)
{
    if (fabs(rho) < 1.0) {
        s = 2.0 * rho;
        c = sqrt(fma(-s, s, 1.0));
    } else {
        c = 2.0 / fabs(rho);
        s = copysign(sqrt(fma(-c, c, 1.0)), rho);
    }
}

// The rotation of (a, b): r = sgn(a) hypot(a, b) with sgn(0) = +1, c = a / r,
// s = b / r; (1, 0) and r = 0 when both are zero.  The fast form needs
// d = a^2 + b^2 in [2^-900, 2^900] (one reciprocal square root, no division);
// the other takes anything.  With b = 0 the fast form's c and r are 1 and a to
// rounding only: its caller puts the row back.
HQR_DEV void rot_fast(double a, double b, double d, double &c, double &s, double &r)
{
    const double ri = pivot_rsqrt(d), bs = (a >= 0.0) ? b : -b;
    c = fabs(a) * ri;
    s = bs * ri;
    const double h = d * ri;
    r = copysign(fma(0.5 * ri, fma(-h, h, d), h), (a >= 0.0) ? 1.0 : -1.0);
}

HQR_DEV void rot_safe(double a, double b, double &c, double &s, double &r)
{
    const double h = hypot(a, b);
    r = (a >= 0.0) ? h : -h;
    c = 1.0;
    s = 0.0;
    if (r != 0.0) {
        c = a / r;
        s = b / r;
    }
}

constexpr int CHU = 64;    // rows and columns per block of the update

// One launch per block of 64 rows k0 .. k0+63 (k0 = -64: none yet), one
// workgroup per 64 columns to its right: the rows' rotations, from v, are
// applied to the block's part of the columns and to their v.  Workgroup 0
// then forms the rotations of its own diagonal block and leaves them in v.
// Columns are staged through LDS, so that the global loads and stores run
// down them; then one wave takes a column per lane.
//
// Bound: the chain of rotations in workgroup 0, about 0.13 us each; the columns
// to the right wait for a block of 64, not for each row.  n = 2000 on MI355X:
// 0.40 ms (12.4 us per launch), against 3.59 ms for one workgroup with a
// barrier, a hypot and two divisions per row.
__global__ void __launch_bounds__(256) chol_update_kernel(double *R, int64_t ldr, double *v, int64_t n, int64_t k0)
{
    __shared__ double P[CHU][CHU + 1];   // [column][row]: rows k0 ..
    __shared__ double D[CHU][CHU + 1];   // [column][row]: the diagonal block
    __shared__ double cs[CHU][2];
    __shared__ unsigned long long keep;  // rows of D that stay as they are in R
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t c0 = k0 + CHU + (int64_t)blockIdx.x * CHU;
    const int nc = (int)min<int64_t>(CHU, n - c0);
    const bool apply = k0 >= 0, first = blockIdx.x == 0;
    double pv[16], dv[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int idx = tid + 256 * q, r = idx & 63, c = min(idx >> 6, nc - 1);
        if (apply) pv[q] = HQR_AT(R, k0 + r, c0 + c, ldr);
        // on or above the diagonal only
        if (first) dv[q] = HQR_AT(R, c0 + min(r, c), c0 + c, ldr);
    }
    double vj = v[c0 + min(lane, nc - 1)];
    if (apply && tid < CHU) {
        double c, s;
        rot_unpack(v[k0 + tid], c, s);
        cs[tid][0] = c;
        cs[tid][1] = s;
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int idx = tid + 256 * q, r = idx & 63, c = idx >> 6;
        if (apply) P[c][r] = pv[q];
        if (first) D[c][r] = dv[q];
    }
    __syncthreads();
    // rows of P or D to R, by nthr threads (whole waves, so a thread's row is
    // one): the LDS reads of a thread together
    auto put = [&](const double (*M)[CHU + 1], int64_t r0, bool upper, int t, int nthr, unsigned long long not_rows) {
        const bool skip = (not_rows >> (t & 63)) & 1;
        for (int i0 = t; i0 < CHU * CHU; i0 += 16 * nthr) {
            double x[16];
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const int idx = min(i0 + nthr * q, CHU * CHU - 1);
                x[q] = M[idx >> 6][idx & 63];
            }
#pragma unroll
            for (int q = 0; q < 16; ++q) pin(x[q]);
#pragma unroll
            for (int q = 0; q < 16; ++q) {
                const int idx = i0 + nthr * q, r = idx & 63, c = idx >> 6;
                if (c < nc && (!upper || r <= c) && !skip) HQR_AT(R, r0 + r, c0 + c, ldr) = x[q];
            }
        }
    };
    if (apply) {
        if (tid < 64) {
            // 16 rows of the column and of (c, s) in registers at a time
#pragma unroll 1
            for (int i0 = 0; i0 < CHU; i0 += 16) {
                double a[16], c[16], s[16];
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    a[i] = P[lane][i0 + i];
                    c[i] = cs[i0 + i][0];
                    s[i] = cs[i0 + i][1];
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    pin(a[i]);
                    pin(c[i]);
                    pin(s[i]);
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const double x = a[i];
                    a[i] = fma(c[i], x, s[i] * vj);
                    vj = fma(c[i], vj, -(s[i] * x));
                }
#pragma unroll
                for (int i = 0; i < 16; ++i) P[lane][i0 + i] = a[i];
            }
            if (!first && lane < nc) v[c0 + lane] = vj;
        }
        __syncthreads();
        // in workgroup 0 the first wave goes on with the diagonal block
        if (!first) put(P, k0, false, tid, 256, 0ull);
        else if (tid >= 64) put(P, k0, false, tid - 64, 192, 0ull);
    }
    if (!first) return;
    // the previous block's rotations were used by the launch before this one,
    // this block's by no other workgroup when this is the last column block
    const bool last = c0 + nc == n;
    if (tid >= 64 && tid < 128) {
        if (k0 >= CHU) v[k0 - CHU + lane] = 0.0;
        if (apply && last) v[k0 + lane] = 0.0;
    }
    if (tid < 64) {
        // Lanes at or left of the pivot rotate values that nothing reads
        // again (the lower triangle of D is not stored), so the steps need
        // no masks; 16 rows in registers at a time.  All steps take the fast
        // form, and a block in which some d left its range is done again
        // from its values in R (no branch on the chain of rotations).
        const double v0 = vj;
        double my_d = 1.0;     // lane k: rotation k's d
#pragma unroll 1
        for (int i0 = 0; i0 < nc; i0 += 16) {
            double a[16];
#pragma unroll
            for (int i = 0; i < 16; ++i) a[i] = D[lane][i0 + i];
#pragma unroll
            for (int i = 0; i < 16; ++i) pin(a[i]);
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                // pinned: in vector registers (the scalar unit's round trips
                // would lengthen the chain)
                const int k = i0 + i;
                const double x = a[i];
                double ak = readlane_f64(x, k), bk = readlane_f64(vj, k);
                pin(ak);
                pin(bk);
                double d = fma(ak, ak, bk * bk), c, s, r;
                pin(d);
                rot_fast(ak, bk, d, c, s, r);
                const double na = fma(c, x, s * vj);
                vj = fma(c, vj, -(s * x));
                a[i] = (lane == k) ? r : na;
                my_d = (lane == k) ? d : my_d;
                cs[k][0] = c;
                cs[k][1] = s;
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) D[lane][i0 + i] = a[i];
        }
        // a row whose rotation is none keeps its bits: it is not stored (a
        // select in the steps lengthened their chain by 0.8 us a launch)
        unsigned long long same = __ballot(lane < nc && cs[lane][1] == 0.0);
        if (__ballot(lane < nc && !(my_d >= 0x1p-900 && my_d <= 0x1p900))) {
            vj = v0;
            same = 0ull;
            const int64_t col = c0 + min(lane, nc - 1);
            for (int k = 0; k < nc; ++k) {
                const double x = HQR_AT(R, min(c0 + k, col), col, ldr);
                double c, s, r;
                rot_safe(readlane_f64(x, k), readlane_f64(vj, k), c, s, r);
                D[lane][k] = (lane == k) ? r : fma(c, x, s * vj);
                vj = (lane > k) ? fma(c, vj, -(s * x)) : vj;
                cs[k][0] = c;
                cs[k][1] = s;
            }
        }
        if (lane < nc) v[c0 + lane] = last ? 0.0 : rot_pack(cs[lane][0], cs[lane][1]);
        if (lane == 0) keep = same;
    }
    __syncthreads();
    put(D, c0, true, tid, 256, keep);
}

// The smallest updates, n <= CHU_SMALL: one wave, a column per lane, no steps
// past the last row.  Bound: the launch, then n rotations (n = 8:
// 9.9 us, 11.3 by the kernel above, whose group of 16 steps and 64 x 64 staging
// are longer than the update).
constexpr int CHU_SMALL = 15;

__global__ void __launch_bounds__(64) chol_update_small_kernel(double *R, int64_t ldr, double *v, int n)
{
    __shared__ double D[CHU_SMALL][64];   // [row][column]
    const int lane = threadIdx.x, col = min(lane, n - 1);
    double a[CHU_SMALL];
#pragma unroll
    for (int i = 0; i < CHU_SMALL; ++i) a[i] = HQR_AT(R, min(i, col), col, ldr);
    const double v0 = v[col];
#pragma unroll
    for (int i = 0; i < CHU_SMALL; ++i) D[i][lane] = a[i];
    double vj = v0, my_d = 1.0, my_s = 1.0;   // lane k: of rotation k
#pragma unroll 1
    for (int k = 0; k < n; ++k) {
        const double x = D[k][lane], ak = readlane_f64(x, k), bk = readlane_f64(vj, k), d = fma(ak, ak, bk * bk);
        double c, s, r;
        rot_fast(ak, bk, d, c, s, r);
        D[k][lane] = (lane == k) ? r : fma(c, x, s * vj);
        vj = fma(c, vj, -(s * x));
        my_d = (lane == k) ? d : my_d;
        my_s = (lane == k) ? s : my_s;
    }
    // as above: rows whose rotation is none stay, a d out of range does all again
    unsigned long long same = __ballot(lane < n && my_s == 0.0);
    if (__ballot(lane < n && !(my_d >= 0x1p-900 && my_d <= 0x1p900))) {
        vj = v0;
        same = 0ull;
#pragma unroll 1
        for (int k = 0; k < n; ++k) {
            const double x = HQR_AT(R, min(k, col), col, ldr);
            double c, s, r;
            rot_safe(readlane_f64(x, k), readlane_f64(vj, k), c, s, r);
            D[k][lane] = (lane == k) ? r : fma(c, x, s * vj);
            vj = (lane > k) ? fma(c, vj, -(s * x)) : vj;
        }
    }
#pragma unroll
    for (int i = 0; i < CHU_SMALL; ++i)
        if (i <= lane && lane < n && !((same >> i) & 1)) HQR_AT(R, i, lane, ldr) = D[i][lane];
    if (lane < n) v[lane] = 0.0;
}

} // namespace hqr
