// hqr_cqr.hpp -- panel factorization with a constant number of grid-wide
// steps: CholeskyQR2 followed by Householder reconstruction.
//
// For a panel A_p (m_p x bw, bw <= 64) the Householder reflectors of the
// paper's per-column loop (Section 3, Alg. 2 / Alg. 3, restated for a block
// of alpha pivots) are recovered without a reduction per column:
//   1. G = A_p^T A_p, R1 = chol(G)                    (pass 1)
//   2. Q1 = A_p R1^{-1}, G2 = Q1^T Q1, R2 = chol(G2)  (pass 2), R = R2 R1
//   3. Q = A_p R^{-1} has orthonormal columns.  Householder QR of Q gives the
//      same reflectors as Householder QR of A_p (each pivot vector of Q is a
//      positive multiple of the corresponding pivot vector of A_p, and a
//      reflector with the sign rule R_kk = -sgn(x_0)||x|| does not change
//      when x is scaled by a positive factor).  For orthonormal Q that
//      factorization is an LU factorization without pivoting of Q - [S; 0],
//      S = diag(s_k), s_k = -sgn(pivot of step k) with sgn(0) = +1:
//          Q - [S; 0] = Y U,  T_Y = -U S Y_1^{-T},  R_house = S R,
//      where Y is unit lower trapezoidal (the normalized reflectors), Y_1 its
//      top bw x bw block and H_0 ... H_{bw-1} = I - Y T_Y Y^T.
//   4. Convert to the stored form: tau_k = T_Y[k][k], up_k = -tau_k R_kk,
//      stored tail = Y[k+1:, k] * up_k, and T for v = up*y:
//      T_V[i][j] = T_Y[i][j] / (up_i up_j).
//   The bottom rows of Y are Q_bot U^{-1} = A_bot (R^{-1} U^{-1}).
//
// Panels for which this is not the stored factorization of the one-reflector
// loop, or not accurate, go to an exact one-workgroup Householder panel
// (exact_panel) instead:
//   - a column whose part below the pivot row is exactly zero (the loop then
//     keeps H_k = I; this includes an empty tail when m_p == bw);
//   - a Cholesky pivot whose squared ratio to the column's norm falls below
//     CQR_RATIO (conditioning beyond what two CholeskyQR passes repair, or
//     rank deficiency).
// The decision is taken on the device: `flag` then makes pass 2 run the exact
// loop instead.
//
// Each pass is a kernel that forms Gram partials (cqr_gram1_kernel, which also
// applies the previous panel's update to these columns; cqr_gram2_kernel), one
// that sums them (gram_reduce_kernel) and one workgroup for the small matrices
// (cqr_chol_kernel), and the bottom rows become V_bot = A_bot W^{-1} in narrow_vtx_kernel (which
// also forms W = T^T V^T C for the next panel's columns, with look-ahead) or
// cqr_finish_kernel.
#pragma once

#include <utility>

#include "hqr_chol64.hpp"

namespace hqr {


// ------------------------------------------------------------------ helpers
// out = A * B for 64 x 64 LDS matrices (row-major, stride 65), FP64 MFMA.
// 256 threads; wave w computes row tile w.  out must not alias A or B.
HQR_DEV void mm64(double (*out)[LD65], const double (*A)[LD65], const double (*B)[LD65], int lane, int w)
{
    f64x4 acc[4];
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k0 = 0; k0 < NB; k0 += 4) {
        const int kr = k0 + (lane >> 4);
        const double a = A[16 * w + (lane & 15)][kr];
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, B[kr][16 * t + (lane & 15)], acc[t], 0, 0, 0);
    }
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) out[16 * w + 4 * r + (lane >> 4)][16 * t + (lane & 15)] = acc[t][r];
}

// One block step of the LU below, in one wave.  Every 16-lane row holds a
// copy of the diagonal block in g; z holds an identity column in the lanes of
// row 0 and, in rows 1..3, the rest of the block row or block column, so the
// elimination that factors the block also yields one inverse and the
// off-diagonal blocks.
//   LPART = false: g lane j = column j of M_kk; eliminating [M_kk | I | M_k,..]
//     gives U_kk (into M), L_kk^{-1} (into DL) and U's block row.
//   LPART = true: the same elimination of [M_kk^T | I | M_..,k^T], with rows
//     scaled by 1/U_ii at the end: L_kk (into DLL), U_kk^{-1} (at XU, row
//     stride ldxu) and L's block column.  Its multipliers are formed so that every product has the
//     other wave's operands: the pivots, and the signs taken from them, are
//     bitwise the same.
// One broadcast and two (LPART: three) operations per multiplier.
template <bool LPART>
HQR_DEV void lu64_load(const double (*M)[LD65], int b0, int lane, double (&g)[16], double (&z)[16])
{
    const int jj = lane & 15, c = b0 + lane, cz = (c < NB) ? c : b0;
    const bool aug = lane < 16;
    // LPART walks along rows of M, the other along columns
    constexpr int st = LPART ? 1 : LD65;
    const double *gp = LPART ? &M[b0 + jj][b0] : &M[b0][b0 + jj], *zp = LPART ? &M[cz][b0] : &M[b0][cz];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        g[i] = gp[i * st];
        z[i] = zp[i * st];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        pin(g[i]);
        pin(z[i]);
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) z[i] = aug ? ((i == jj) ? 1.0 : 0.0) : z[i];
}

// Pivot state of lu64_block: the current pivot's s_k, U_kk and reciprocal,
// and the lane's own s_k and U_kk.
struct LuPivot {
    int jj;
    double sg, ukk, uinv, my_sg = 0.0, my_uk = 0.0;
    __device__ __forceinline__ void set(double q)
    {
        sg = (q >= 0.0) ? -1.0 : 1.0;
        ukk = q - sg;
    }
};

// One pivot of the 16 x 16 elimination (as chol16_pivot): multipliers
// M[i2][I] (LPART: M[I][i2] U_II^{-1}) by broadcast, rows I scaled by U_II^{-1}
// (LPART: not scaled) as the other factor.
template <bool LPART, int I, int U>
HQR_DEV void lu16_rows(double (&g)[16], double (&z)[16], double gm, double zm, double uinv, RecipChain &rc)
{
    constexpr int i2 = I + 2 + 2 * U;
    if constexpr (i2 < 16) {
        double ta = bc16c<I>(g[i2]), tb;
        if constexpr (i2 + 1 < 16) tb = bc16c<I>(g[i2 + 1]);
        if constexpr (LPART) {
            ta *= uinv;
            if constexpr (i2 + 1 < 16) tb *= uinv;
        }
        pin(ta);
        if constexpr (i2 + 1 < 16) pin(tb);
        g[i2] = fma(-ta, gm, g[i2]);
        z[i2] = fma(-ta, zm, z[i2]);
        pin(g[i2]);
        pin(z[i2]);
        if constexpr (i2 + 1 < 16) {
            g[i2 + 1] = fma(-tb, gm, g[i2 + 1]);
            z[i2 + 1] = fma(-tb, zm, z[i2 + 1]);
            pin(g[i2 + 1]);
            pin(z[i2 + 1]);
        }
    }
    rc.template stage<U>();
}

template <bool LPART, int I>
HQR_DEV void lu16_pivot(double (&g)[16], double (&z)[16], LuPivot &pv)
{
    const double uinv = pv.uinv;
    const double gs = g[I] * uinv, zs = z[I] * uinv;
    if (!LPART) {
        pv.my_sg = (pv.jj == I) ? pv.sg : pv.my_sg;
        pv.my_uk = (pv.jj == I) ? pv.ukk : pv.my_uk;
    }
    if constexpr (I < 15) {
        const double gm = LPART ? g[I] : gs, zm = LPART ? z[I] : zs;
        double t1 = bc16c<I>(g[I + 1]);
        if (LPART) t1 *= uinv;
        g[I + 1] = fma(-t1, gm, g[I + 1]);
        pin(g[I + 1]);
        double q = bc16c<I + 1>(g[I + 1]);
        pin(q);
        z[I + 1] = fma(-t1, zm, z[I + 1]);
        pv.set(q);
        RecipChain rc;
        rc.start(pv.ukk);
        lu16_rows<LPART, I, 0>(g, z, gm, zm, uinv, rc);
        lu16_rows<LPART, I, 1>(g, z, gm, zm, uinv, rc);
        lu16_rows<LPART, I, 2>(g, z, gm, zm, uinv, rc);
        lu16_rows<LPART, I, 3>(g, z, gm, zm, uinv, rc);
        lu16_rows<LPART, I, 4>(g, z, gm, zm, uinv, rc);
        lu16_rows<LPART, I, 5>(g, z, gm, zm, uinv, rc);
        lu16_rows<LPART, I, 6>(g, z, gm, zm, uinv, rc);
        pv.uinv = rc.y;
    }
    if (LPART) {
        g[I] = gs;
        z[I] = zs;
    }
    __builtin_amdgcn_sched_barrier(0);
}

template <bool LPART, int... Is>
HQR_DEV void lu16_pivots(double (&g)[16], double (&z)[16], LuPivot &pv, std::integer_sequence<int, Is...>)
{
    (lu16_pivot<LPART, Is>(g, z, pv), ...);
}

// The block step on the loaded values (after a barrier: the other wave's
// writes to M cannot race with these reads).
template <bool LPART>
HQR_DEV void lu64_block(double (*M)[LD65], double (*DL)[17], double (*DLL)[17], double *XU, int ldxu, int b0,
                        int lane, double *sgn, double *udiag, double (&g)[16], double (&z)[16])
{
    // opaque per block step: keeps the per-pivot lane masks from being
    // hoisted out of the caller's kb loop (they would occupy ~100 SGPRs)
    int ln = lane;
    asm volatile("" : "+v"(ln));
    const int jj = ln & 15, c = b0 + ln;
    const bool aug = ln < 16, act = c < NB;
    LuPivot pv;
    pv.jj = jj;
    pv.set(bc16c<0>(g[0]));
    pv.uinv = recip_nr(pv.ukk);
    lu16_pivots<LPART>(g, z, pv, std::make_integer_sequence<int, 16>{});
    const double my_sg = pv.my_sg, my_uk = pv.my_uk;
    // rows 1..3 write the off-diagonal blocks, row 0 the diagonal block
    // (U with its diagonal, L below it) and the inverse's block
    // straight runs of stores: the lower triangle of U's diagonal block and
    // the upper one of L's are not meant to be read
    if (aug) {
        if (LPART) {
            double *xp = XU + jj * ldxu, *dp = &DLL[b0 + jj][0];
#pragma unroll
            for (int i = 0; i < 16; ++i) xp[i] = z[i];      // U^{-1}[jj][i]
#pragma unroll
            for (int i = 0; i < 16; ++i) dp[i] = g[i];      // L[jj][i]
        } else {
            double *xp = &DL[b0][jj], *dp = &M[b0][c];
#pragma unroll
            for (int i = 0; i < 16; ++i) xp[i * 17] = z[i]; // L^{-1}[i][jj]
#pragma unroll
            for (int i = 0; i < 16; ++i) dp[i * LD65] = g[i];
            dp[jj * LD65] = my_uk;
        }
    } else if (act) {
        double *dp = LPART ? &M[c][b0] : &M[b0][c];
#pragma unroll
        for (int i = 0; i < 16; ++i) dp[i * (LPART ? 1 : LD65)] = z[i];
    }
    if (!LPART && aug) {
        sgn[b0 + jj] = my_sg;
        udiag[b0 + jj] = my_uk;
    }
}

// In place: M (n x n leading block; entries outside it zero) becomes L
// (below the diagonal blocks; within them in DLL, unit diagonal implied) and
// U (on and above the diagonal) of the LU factorization without pivoting of
// M - S, s_k = -sgn(pivot of step k) (sgn(0) = +1); beyond n the factors
// continue as the identity (s_k = -1, U_kk = 1).  Block step kb: wave 0
// computes U's block row and the diagonal block of L^{-1} (into DL, rows
// 16kb..16kb+15), wave 1 L's block column and the diagonal block of U^{-1}
// (XU), both by lu64_block, while waves 2 and 3 finish the previous step's
// trailing blocks and then do what the caller adds; between two barriers
// only the blocks of block row and column kb + 1 are updated on MFMA.  sgn
// and udiag get s_k and U_kk for all 64 steps.
HQR_DEV void lu_trail_blk(double (*M)[LD65], int b0, int ib, int jb, int lane)
{
    f64x4 acc = ld_blk(M, 16 * ib, 16 * jb, lane);
    const int i16 = lane & 15, kk = lane >> 4;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int k = b0 + 4 * q + kk;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-M[16 * ib + i16][k], M[k][16 * jb + i16], acc, 0, 0, 0);
    }
    st_blk(M, 16 * ib, 16 * jb, acc, 1.0, lane);
}

// The pivots of step kb (a barrier inside, for all waves).
HQR_DEV void lu64_pivots(double (*M)[LD65], double (*DL)[17], double (*DLL)[17], double *XU, int ldxu, int kb,
                         int lane, int w, double *sgn, double *udiag)
{
    const int b0 = 16 * kb;
    double g[16], z[16];
    if (w == 0) {
        lu64_load<false>(M, b0, lane, g, z);
        __syncthreads();
        lu64_block<false>(M, DL, DLL, XU, ldxu, b0, lane, sgn, udiag, g, z);
    } else if (w == 1) {
        lu64_load<true>(M, b0, lane, g, z);
        __syncthreads();
        lu64_block<true>(M, DL, DLL, XU, ldxu, b0, lane, sgn, udiag, g, z);
    } else {
        __syncthreads();
        const int rem = 3 - kb;
        if (kb > 0)
            for (int bidx = w - 2; bidx < rem * rem; bidx += 2)
                lu_trail_blk(M, b0 - 16, kb + 1 + bidx / rem, kb + 1 + bidx % rem, lane);
    }
}

// After a barrier: block row and column kb + 1, i.e. (kb+1, kb+1..3) and
// (kb+2..3, kb+1); ends with a barrier.
HQR_DEV void lu64_trail(double (*M)[LD65], int kb, int lane, int w)
{
    const int rem = 3 - kb;
    for (int t = w; t < 2 * rem - 1; t += 4) {
        const int ib = (t < rem) ? kb + 1 : kb + 2 + (t - rem), jb = (t < rem) ? kb + 1 + t : kb + 1;
        lu_trail_blk(M, 16 * kb, ib, jb, lane);
    }
    __syncthreads();
}

// Unit lower inverse whose diagonal blocks are in D (rows 16kb..) and whose
// blocks below them are in X: the sum over k = j .. i-1 of L_ik X_kj in D
// layout, and X_ij = -X_ii times that sum.
HQR_DEV f64x4 mma_blk_d(f64x4 acc, const double (*MA)[LD65], int ar, int ac, const double (*D)[17], int kb, int lane)
{
    const int i = lane & 15, kk = lane >> 4;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(MA[ar + i][ac + 4 * q + kk], D[16 * kb + 4 * q + kk][i], acc, 0, 0, 0);
    return acc;
}

HQR_DEV f64x4 mma_sum(const double (*L)[LD65], int i, const double (*X)[LD65], const double (*D)[17], int j, int lane)
{
    f64x4 t = mma_blk_d(f64x4{0.0, 0.0, 0.0, 0.0}, L, 16 * i, 16 * j, D, j, lane);
    for (int k = j + 1; k < i; ++k) t = mma_blk(t, L, 16 * i, 16 * k, X, 16 * k, 16 * j, lane);
    return t;
}

HQR_DEV void inv_lower_close(double (*X)[LD65], const double (*D)[17], int i, int j, f64x4 t, int lane)
{
    const int i16 = lane & 15, kk = lane >> 4;
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 4; ++q)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(D[16 * i + i16][4 * q + kk], t[q], acc, 0, 0, 0);
    st_blk(X, 16 * i, 16 * j, acc, -1.0, lane);
}

// Off-diagonal blocks of triangular inverses whose diagonal blocks are
// already in place, by distance from the diagonal on MFMA:
//   X_ij = -X_ii sum_{k=i+1..j} U_ik X_kj   (i < j)
// One 16 x 16 block task: t = sum of the products, X_ij = -X_ii t.
HQR_DEV void inv_upper_task(double (*X)[LD65], const double (*U)[LD65], int i, int j, int lane)
{
    f64x4 t = f64x4{0.0, 0.0, 0.0, 0.0};
    for (int k = i + 1; k <= j; ++k) t = mma_blk(t, U, 16 * i, 16 * k, X, 16 * k, 16 * j, lane);
    st_blk(X, 16 * i, 16 * j, mma_blk_reg(f64x4{0.0, 0.0, 0.0, 0.0}, X, 16 * i, 16 * i, t, lane), -1.0, lane);
}

// zero the blocks of X strictly below the diagonal
HQR_DEV void zero_lower_blocks(double (*X)[LD65], int tid)
{
    for (int idx = tid; idx < NB * NB; idx += 256) {
        const int r = idx / NB, c = idx % NB;
        if ((r >> 4) > (c >> 4)) X[r][c] = 0.0;
    }
}

// X = U^{-1} (64 x 64 upper U) given X's diagonal blocks.  Starts and ends
// with a barrier.
HQR_DEV void inv_upper_levels(double (*X)[LD65], const double (*U)[LD65], int lane, int w)
{
    __syncthreads();
    zero_lower_blocks(X, 64 * w + lane);
    if (w < 3) inv_upper_task(X, U, w, w + 1, lane);
    __syncthreads();
    if (w < 2) inv_upper_task(X, U, w, w + 2, lane);
    __syncthreads();
    if (w == 0) inv_upper_task(X, U, 0, 3, lane);
    __syncthreads();
}

// Products of 64 x 64 operands given by element functions fa(r, c), fb(r, c),
// into D-layout accumulators (acc[s][q] = C[16 bi + 4q + lane/16][16 bj +
// lane%16] for the wave's block (bi, bj) of slot s).
//
// Upper x upper: the 10 blocks bi <= bj, each summed over k = bi..bj (20
// block products), spread 5 per wave; uu_slot gives slot s of wave w as
// 4 bi + bj, or -1.
constexpr int uu_slot_c(int w, int s)
{
    // w0: (0,3) (3,3)  w1: (0,2) (1,2)  w2: (1,3) (0,1)  w3: (2,3) (0,0) (1,1) (2,2)
    const unsigned tab = (w == 0) ? 0xffff0f03u : (w == 1) ? 0xffff0602u : (w == 2) ? 0xffff0107u : 0x0a05000bu;
    const int e = (int)((tab >> (8 * s)) & 0xffu);
    return e == 0xff ? -1 : e;
}

// One wave's share, its blocks known at compile time: the five block
// products become straight code whose loads and MFMAs the compiler can
// overlap (with the wave as a runtime value each product was a loop round
// of its own, its loads waited for one after the other: about 0.4 us each).
template <int W, int S, class FA, class FB>
HQR_DEV void mm_uu_block(f64x4 &acc, FA fa, FB fb, int lane)
{
    constexpr int e = uu_slot_c(W, S);
    acc = f64x4{0.0, 0.0, 0.0, 0.0};
    if constexpr (e >= 0) {
        constexpr int bi = e >> 2, bj = e & 3;
        const int i16 = lane & 15, kk = lane >> 4;
#pragma unroll
        for (int kb = bi; kb <= bj; ++kb) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int k = 16 * kb + 4 * q + kk;
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(fa(16 * bi + i16, k), fb(k, 16 * bj + i16), acc, 0, 0, 0);
            }
        }
    }
}

template <int W, class FA, class FB>
HQR_DEV void mm_uu_wave(f64x4 (&acc)[4], FA fa, FB fb, int lane)
{
    mm_uu_block<W, 0>(acc[0], fa, fb, lane);
    mm_uu_block<W, 1>(acc[1], fa, fb, lane);
    mm_uu_block<W, 2>(acc[2], fa, fb, lane);
    mm_uu_block<W, 3>(acc[3], fa, fb, lane);
}

// w must be uniform over the wave (a scalar)
template <class FA, class FB>
HQR_DEV void mm_upper_upper(f64x4 (&acc)[4], FA fa, FB fb, int lane, int w)
{
    if (w == 0) mm_uu_wave<0>(acc, fa, fb, lane);
    else if (w == 1) mm_uu_wave<1>(acc, fa, fb, lane);
    else if (w == 2) mm_uu_wave<2>(acc, fa, fb, lane);
    else mm_uu_wave<3>(acc, fa, fb, lane);
}

// In place, one wave: block row I of A B over A's, for upper A and B.  Block
// (I, j) needs A's blocks up to column j only, so the row goes from right to
// left; rows are independent.
template <int I>
HQR_DEV void mul_upper_row(double (*A)[LD65], const double (*B)[LD65], int lane)
{
#pragma unroll
    for (int j = 3; j >= I; --j) {
        f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = I; k <= j; ++k) acc = mma_blk(acc, A, 16 * I, 16 * k, B, 16 * k, 16 * j, lane);
        st_blk(A, 16 * I, 16 * j, acc, 1.0, lane);
        __builtin_amdgcn_sched_barrier(0);   // one block's operands in registers at a time
    }
}

// In place, one wave: block column J of A B over B's, for upper A (64 x 64
// row-major in global memory) and B: from top to bottom, columns independent.
template <int J>
HQR_DEV void mul_upper_col(const double *A, double (*B)[LD65], int lane)
{
    const int i16 = lane & 15, kk = lane >> 4;
#pragma unroll
    for (int i = 0; i <= J; ++i) {
        f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k = i; k <= J; ++k)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = 16 * k + 4 * q + kk;
                acc = __builtin_amdgcn_mfma_f64_16x16x4f64(A[(16 * i + i16) * NB + r], B[r][16 * J + i16], acc, 0, 0, 0);
            }
        st_blk(B, 16 * i, 16 * J, acc, 1.0, lane);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Full x upper: wave w computes block row w, block (w, bj) summed over
// k = 0..bj (slot s = bj).
template <class FA, class FB>
HQR_DEV void mm_full_upper(f64x4 (&acc)[4], FA fa, FB fb, int lane, int w)
{
    const int i16 = lane & 15, kk = lane >> 4;
#pragma unroll
    for (int s = 0; s < 4; ++s) acc[s] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = 16 * kb + 4 * q + kk;
            const double a = fa(16 * w + i16, k);
#pragma unroll
            for (int s = kb; s < 4; ++s)
                acc[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, fb(k, 16 * s + i16), acc[s], 0, 0, 0);
        }
    }
}

// Visit the elements of the wave's upper x upper accumulators:
// f(row, col, value).
template <int W, int S, class F>
HQR_DEV void for_uu_block(const f64x4 &acc, F f, int lane)
{
    constexpr int e = uu_slot_c(W, S);
    if constexpr (e >= 0) {
        constexpr int bi = e >> 2, bj = e & 3;
#pragma unroll
        for (int q = 0; q < 4; ++q) f(16 * bi + 4 * q + (lane >> 4), 16 * bj + (lane & 15), acc[q]);
    }
}

template <int W, class F>
HQR_DEV void for_uu_wave(const f64x4 (&acc)[4], F f, int lane)
{
    for_uu_block<W, 0>(acc[0], f, lane);
    for_uu_block<W, 1>(acc[1], f, lane);
    for_uu_block<W, 2>(acc[2], f, lane);
    for_uu_block<W, 3>(acc[3], f, lane);
}

template <class F>
HQR_DEV void for_uu(const f64x4 (&acc)[4], F f, int lane, int w)
{
    if (w == 0) for_uu_wave<0>(acc, f, lane);
    else if (w == 1) for_uu_wave<1>(acc, f, lane);
    else if (w == 2) for_uu_wave<2>(acc, f, lane);
    else for_uu_wave<3>(acc, f, lane);
}

// M[r][c] = A[r0 + r][c0 + c] (r < 64, c < NB), zero for rows >= m or
// columns >= ncol.  256 threads; the loads are unconditional (clamped into
// the matrix, zeroed afterwards), so all 16 of a thread are in flight
// together instead of each waiting behind its own branch.
HQR_DEV void tile_issue(double (&v)[16], const double *A, int64_t lda, int64_t m, int64_t r0, int c0, int ncol,
                        int tid)
{
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int idx = tid + 256 * q, c = idx / 64, r = idx % 64;
        const int64_t gi = r0 + r;
        v[q] = HQR_AT(A, (gi < m) ? gi : m - 1, c0 + ((c < ncol) ? c : 0), lda);
    }
}

HQR_DEV void tile_store(double (*M)[LD65], double (&v)[16], int64_t m, int64_t r0, int ncol, int tid)
{
#pragma unroll
    for (int q = 0; q < 16; ++q) pin_f64(v[q]);
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int idx = tid + 256 * q, c = idx / 64, r = idx % 64;
        M[r][c] = (r0 + r < m && c < ncol) ? v[q] : 0.0;
    }
}

// M[r][c] = V[r0 + r][c] of the panel starting at cv (width NB; unit lower
// triangle with up on the diagonal in its top block), zero for rows >= m.
// The issue half loads A's entries and up; the store half applies the
// triangle.
HQR_DEV void vtile_issue(double (&v)[16], double (&u)[16], const double *A, int64_t lda, const double *up, int64_t m,
                         int64_t r0, int cv, int tid)
{
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int idx = tid + 256 * q, c = idx / 64, r = idx % 64;
        const int64_t gi = r0 + r;
        v[q] = HQR_AT(A, (gi < m) ? gi : m - 1, cv + c, lda);
        u[q] = up[cv + c];
    }
}

HQR_DEV void vtile_store(double (*M)[LD65], double (&v)[16], double (&u)[16], int64_t m, int64_t r0, int cv, int tid)
{
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        pin_f64(v[q]);
        pin_f64(u[q]);
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int idx = tid + 256 * q, c = idx / 64, r = idx % 64;
        const int64_t d = r0 + r - cv;   // row offset from the panel's first row
        const double e = (d < c) ? 0.0 : ((d == c) ? u[q] : v[q]);
        M[r][c] = (r0 + r < m) ? e : 0.0;
    }
}

// A 64 x 64 row-major matrix into LDS in two halves (transposed when TRANS),
// so that its loads can be issued together with a tile's.
HQR_DEV void mat64_issue(double (&v)[16], const double *src, int tid)
{
#pragma unroll
    for (int t = 0; t < 16; ++t) v[t] = src[tid + 256 * t];
}

template <bool TRANS>
HQR_DEV void mat64_store(double (*M)[LD65], double (&v)[16], int tid)
{
#pragma unroll
    for (int t = 0; t < 16; ++t) pin_f64(v[t]);
#pragma unroll
    for (int t = 0; t < 16; ++t) {
        const int idx = tid + 256 * t;
        if (TRANS)
            M[idx % NB][idx / NB] = v[t];
        else
            M[idx / NB][idx % NB] = v[t];
    }
}

// acc[t] (t = 0..3) += sign * A[16w:16w+16][:] * B[:][16t:16t+16] over k = 0..63
HQR_DEV void mm64_acc(f64x4 (&acc)[4], const double (*A)[LD65], const double (*B)[LD65], double sign, int lane, int w)
{
#pragma unroll
    for (int k0 = 0; k0 < NB; k0 += 4) {
        const int kr = k0 + (lane >> 4);
        const double a = sign * A[16 * w + (lane & 15)][kr];
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, B[kr][16 * t + (lane & 15)], acc[t], 0, 0, 0);
    }
}

// acc[t] = Z^T Z (rows 16w.., column tile t) for a 64 x 64 LDS tile Z.  One
// wave per SIMD: nothing hides an LDS read but the products before it, so the
// 64-deep loops here and above are unrolled in full (by four, each group of 16
// products waited for its reads: second Gram pass 9.8 us against 8.0 at
// 701 x 333)
HQR_DEV void gram64(f64x4 (&acc)[4], const double (*Z)[LD65], int lane, int w)
{
#pragma unroll
    for (int t = 0; t < 4; ++t) acc[t] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int k0 = 0; k0 < NB; k0 += 4) {
        const int kr = k0 + (lane >> 4);
        const double a = Z[kr][16 * w + (lane & 15)];
#pragma unroll
        for (int t = 0; t < 4; ++t) acc[t] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, Z[kr][16 * t + (lane & 15)], acc[t], 0, 0, 0);
    }
}

// D-layout accumulators of a full 64 x 64 product -> row-major global
HQR_DEV void st64_global(double *out, const f64x4 (&acc)[4], int lane, int w)
{
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) out[(16 * w + 4 * r + (lane >> 4)) * NB + 16 * t + (lane & 15)] = acc[t][r];
}

// ------------------------------------------------- exact one-workgroup panel
// The one-reflector-at-a-time loop on the panel (the arithmetic of the
// per-column launches, the dot products split over NG row groups), streamed
// from global memory by 64 NG threads, followed by T from V^T V.  Used when a
// panel is flagged (structurally exact reflectors, or conditioning beyond
// what two CholeskyQR passes repair).
struct ExactArgs {
    double *A;
    int64_t lda;
    int64_t m;
    int c0, bw;
    double *up;
    double *T;
};

template <int NG>
HQR_DEV void exact_panel(const ExactArgs &p, int tid, double (*red)[PW], double *wsh, double *sc, double (*G)[LD65],
                         double (*Ts)[LD65], double *tau, double *tmp)
{
    constexpr int NT = 64 * NG;
    const int j = tid & 63, g = tid >> 6;
    const int bw = p.bw, c0 = p.c0;
    const int64_t m = p.m;
    __syncthreads();
    for (int k = 0; k < bw; ++k) {
        const int64_t pr = (int64_t)c0 + k;
        // partial dots x . a_j over rows > pr, plus max|x| and #nonzero
        double acc = 0.0, mx = 0.0, nz = 0.0;
        for (int64_t i = pr + 1 + g; i < m; i += NG) {
            const double xi = HQR_AT(p.A, i, c0 + k, p.lda);
            if (j >= k && j < bw) acc += xi * HQR_AT(p.A, i, c0 + j, p.lda);
            mx = fmax(mx, fabs(xi));
            nz += (xi != 0.0) ? 1.0 : 0.0;
        }
        red[g][j] = acc;
        if (j == 0) {
            red[g][NB] = mx;
            red[g][NB + 1] = nz;
        }
        __syncthreads();
        if (tid < PW) {
            double v = 0.0;
            if (tid == NB) {
                for (int q = 0; q < NG; ++q) v = fmax(v, red[q][NB]);
            } else {
                for (int q = 0; q < NG; ++q) v += red[q][tid];
            }
            red[0][tid] = v;
        }
        __syncthreads();
        if (tid == 0) {
            const double x0 = HQR_AT(p.A, pr, c0 + k, p.lda);
            double upk, sk;
            if (red[0][NB + 1] == 0.0) {
                upk = 0.0;
                sk = x0;
            } else {
                const double c = fmax(fabs(x0), red[0][NB]);
                double nu;
                if (norm_fast_path_ok(c)) {
                    nu = sqrt(x0 * x0 + red[0][k]);
                } else {
                    double t = 0.0;
                    for (int64_t i = pr + 1; i < m; ++i) {
                        const double y = HQR_AT(p.A, i, c0 + k, p.lda) / c;
                        t += y * y;
                    }
                    const double x0c = x0 / c;
                    nu = c * sqrt(x0c * x0c + t);
                }
                sk = (x0 >= 0.0) ? -nu : nu;
                upk = x0 - sk;
            }
            sc[0] = upk;
            sc[1] = sk;
            p.up[c0 + k] = upk;
        }
        __syncthreads();
        const double upk = sc[0], sk = sc[1];
        if (upk != 0.0) {
            const double bk = upk * sk;
            if (tid < NB) wsh[tid] = (tid > k && tid < bw) ? (upk * HQR_AT(p.A, pr, c0 + tid, p.lda) + red[0][tid]) / bk : 0.0;
            __syncthreads();
            if (j > k && j < bw) {
                const double wj = wsh[j];
                for (int64_t i = pr + g; i < m; i += NG) {
                    const double v = (i == pr) ? upk : HQR_AT(p.A, i, c0 + k, p.lda);
                    HQR_AT(p.A, i, c0 + j, p.lda) += wj * v;
                }
            }
        }
        __syncthreads();
        if (tid == 0) HQR_AT(p.A, pr, c0 + k, p.lda) = sk;
        __syncthreads();
    }
    // G = V^T V (V masked: up on the diagonal), then T by the recurrence
    for (int e = tid; e < NB * NB; e += NT) {
        Ts[e / NB][e % NB] = 0.0;
        const int a = e / NB, b = e % NB;
        if (a > b) continue;
        double s = 0.0;
        if (b < bw) {
            const int64_t lo = (int64_t)c0 + b;
            s = p.up[c0 + b] * ((a == b) ? p.up[c0 + a] : HQR_AT(p.A, lo, c0 + a, p.lda));
            for (int64_t i = lo + 1; i < m; ++i) s += HQR_AT(p.A, i, c0 + a, p.lda) * HQR_AT(p.A, i, c0 + b, p.lda);
        }
        G[a][b] = s;
        G[b][a] = s;
    }
    if (tid < NB) {
        double t = 0.0;
        if (tid < bw) {
            const double u = p.up[c0 + tid];
            t = (u == 0.0) ? 0.0 : -1.0 / (u * HQR_AT(p.A, (int64_t)c0 + tid, c0 + tid, p.lda));
        }
        tau[tid] = t;
    }
    __syncthreads();
    for (int jj = 0; jj < bw; ++jj) {
        if (tid < jj) {
            double s = 0.0;
            for (int l = tid; l < jj; ++l) s += Ts[tid][l] * G[l][jj];
            tmp[tid] = s;
        }
        __syncthreads();
        if (tid < jj) Ts[tid][jj] = -tau[jj] * tmp[tid];
        if (tid == jj) Ts[jj][jj] = tau[jj];
        __syncthreads();
    }
    for (int e = tid; e < NB * NB; e += NT) p.T[e] = Ts[e / NB][e % NB];
}


__global__ void __launch_bounds__(256) cqr_gram1_kernel(Gram1Args p)
{
    __shared__ double M0[NB][LD65];
    __shared__ double M1[NB][LD65];
    __shared__ double M2[NB][LD65];
    __shared__ unsigned long long msk;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int bw = p.bw, t = blockIdx.x;
    const int64_t rbase = p.upd ? (int64_t)p.cp : (int64_t)p.c0;
    const int64_t r0 = rbase + 64 * (int64_t)t;
    const bool flagged = *((volatile int *)p.flag) != 0;
    if (tid == 0) msk = 0ull;
    // M0 = C tile (panel columns); with the update M1 = V tile, M2 = W; all
    // loads are issued before the first wait
    {
        double cv[16], vv[16], uv[16], wv[16];
        tile_issue(cv, p.A, p.lda, p.m, r0, p.c0, bw, tid);
        if (p.upd) {
            vtile_issue(vv, uv, p.A, p.lda, p.up, p.m, r0, p.cp, tid);
            mat64_issue(wv, p.Wt, tid);
        }
        tile_store(M0, cv, p.m, r0, bw, tid);
        if (p.upd) {
            vtile_store(M1, vv, uv, p.m, r0, p.cp, tid);
            mat64_store<true>(M2, wv, tid);
        }
    }
    __syncthreads();
    if (p.upd) {
        f64x4 acc[4];
        // C -= V W: each wave reads and rewrites only its own 16 rows of M0
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = ld_blk(M0, 16 * w, 16 * q, lane);
        mm64_acc(acc, M1, M2, -1.0, lane, w);
#pragma unroll
        for (int q = 0; q < 4; ++q) st_blk(M0, 16 * w, 16 * q, acc[q], 1.0, lane);
        __syncthreads();
    }
    // thread (row lane, columns w, w + 4, ..): all reads before the first use
    double mv[16];
    const int64_t gi = r0 + lane;
#pragma unroll
    for (int k = 0; k < 16; ++k) mv[k] = M0[lane][w + 4 * k];
#pragma unroll
    for (int k = 0; k < 16; ++k) pin_f64(mv[k]);
    if (p.upd && gi < p.m) {
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if (w + 4 * k < bw) HQR_AT(p.A, gi, p.c0 + w + 4 * k, p.lda) = mv[k];
    }
    if (flagged) return;                 // the exact loop factors this panel
    if (p.upd && t == 0) return;         // rows above the panel
    const int gidx = p.upd ? t - 1 : t;
    // a wave's columns have one bit each: a ballot per column and one LDS
    // atomic per wave.  The chain's latency binds here: with a branch and a
    // wait per element and 256 atomics on one word the kernel took 16.5 us at
    // 701 x 333, 13 so
    unsigned long long mymask = 0ull;
#pragma unroll
    for (int k = 0; k < 16; ++k) {
        const int c = w + 4 * k;
        const bool nz = c < bw && gi > (int64_t)p.c0 + c && gi < p.m && mv[k] != 0.0;
        mymask |= (__ballot(nz) != 0ull) ? (1ull << c) : 0ull;
    }
    if (lane == 0 && mymask) atomicOr(&msk, mymask);
    f64x4 acc[4];
    gram64(acc, M0, lane, w);
    st64_global(p.gpart + (size_t)gidx * NB * NB, acc, lane, w);
    __syncthreads();
    if (tid == 0) p.mask[gidx] = msk;
}


__global__ void __launch_bounds__(256) cqr_gram2_kernel(Gram2Args p)
{
    __shared__ double X[NB][LD65];
    __shared__ double Y[NB][LD65];
    __shared__ double Ri[NB][LD65];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (*((volatile int *)p.flag)) return;
    const int t = blockIdx.x;
    const int64_t r0 = (int64_t)p.c0 + 64 * (int64_t)t;
    {
        double xv[16], rv[16];
        tile_issue(xv, p.A, p.lda, p.m, r0, p.c0, p.bw, tid);
        mat64_issue(rv, p.r1inv, tid);
        tile_store(X, xv, p.m, r0, p.bw, tid);
        mat64_store<false>(Ri, rv, tid);
    }
    __syncthreads();
    mm64(Y, X, Ri, lane, w);
    __syncthreads();
    if (t == 0) {
        double qv[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) qv[k] = Y[w + 4 * k][lane];
#pragma unroll
        for (int k = 0; k < 16; ++k) pin_f64(qv[k]);
#pragma unroll
        for (int k = 0; k < 16; ++k) p.q1top[tid + 256 * k] = (w + 4 * k < p.bw && lane < p.bw) ? qv[k] : 0.0;
    }
    f64x4 acc[4];
    gram64(acc, Y, lane, w);
    st64_global(p.gpart + (size_t)t * NB * NB, acc, lane, w);
}


__global__ void __launch_bounds__(256) gram_reduce_kernel(GredArgs p)
{
    __shared__ double part[4][64];
    const int tid = threadIdx.x, e = blockIdx.x * 64 + (tid & 63), g4 = tid >> 6;
    if (p.flag && *((volatile int *)p.flag)) return;
    // thread (e, g4) sums partials q = g4, g4 + 4, ... in that order; 16
    // loads at a time are issued before any is used (clamped, zeroed after)
    double s = 0.0;
    for (int q0 = g4; q0 < p.ngroups; q0 += 64) {
        double v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int q = q0 + 4 * u;
            v[u] = p.gpart[(size_t)((q < p.ngroups) ? q : g4) * NB * NB + e];
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) pin_f64(v[u]);
#pragma unroll
        for (int u = 0; u < 16; ++u) s += (q0 + 4 * u < p.ngroups) ? v[u] : 0.0;
    }
    part[g4][tid & 63] = s;
    __syncthreads();
    if (tid < 64) p.G[e] = ((part[0][tid] + part[1][tid]) + part[2][tid]) + part[3][tid];
    if (p.with_mask && blockIdx.x == 0 && tid >= 64 && tid < 128) {
        // OR of the masks: 64 lanes, strided loads all in flight, then a
        // butterfly over the wave
        const int l = tid - 64;
        unsigned long long all = 0ull;
        for (int q = l; q < p.ngroups; q += 64) all |= p.mask[q];
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            const unsigned lo = (unsigned)all, hi = (unsigned)(all >> 32);
            all |= (unsigned long long)(unsigned)__shfl_xor((int)lo, off) |
                   ((unsigned long long)(unsigned)__shfl_xor((int)hi, off) << 32);
        }
        if (l == 0) *p.mask_all = all;
    }
}

// ------------------------------------ Cholesky of a near-identity Gram matrix
// For G = I + E with every |E_ij| <= CQR_SERIES_TAU, the upper factor is
// R = I + X with X + X^T + X^T X = E.  Writing Phi(M) for the strict upper
// part of a symmetric M plus half its diagonal, X0 = Phi(E) and
// X1 = Phi(E - X0^T X0) satisfy ||X1 - X||_F <= 2 eps^3 (eps = ||E||_F <=
// 64 tau), and R^{-1} = I - X1 + X1^2 up to eps^3: below 3e-22 for
// tau = 2^-30, far under FP64 rounding.  Three block products on MFMA replace
// the 64 sequential pivots.  The second CholeskyQR pass meets this bound
// unless the panel's condition number exceeds about 1e3 (its Gram matrix is
// then I + O(kappa^2 u)).
constexpr double CQR_SERIES_TAU = 0x1p-30;

template <int W>
HQR_DEV void near_gram(f64x4 (&acc)[4], const double (*X)[LD65], int lane)
{
    const int i16 = lane & 15, kk = lane >> 4;
#pragma unroll
    for (int s = 0; s < 4; ++s) acc[s] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int kb = 0; kb <= W; ++kb)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = 16 * kb + 4 * q + kk;
            const double a = X[k][16 * W + i16];
#pragma unroll
            for (int s = W; s < 4; ++s)
                acc[s] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, X[k][16 * s + i16], acc[s], 0, 0, 0);
        }
}

// On entry (after a barrier) G holds I + E in full and X holds Phi(E).  On
// exit G = R and X = R^{-1} (upper, zeros below), rdiag = diag(R); ends with
// a barrier.
HQR_DEV void chol_near_identity(double (*G)[LD65], double (*X)[LD65], double *rdiag, int lane, int w)
{
    const int i16 = lane & 15, kk = lane >> 4;
    // P = X0^T X0 on the wave's upper blocks (w, s >= w): k-blocks 0..w
    f64x4 acc[4];
    if (w == 0) near_gram<0>(acc, X, lane);
    else if (w == 1) near_gram<1>(acc, X, lane);
    else if (w == 2) near_gram<2>(acc, X, lane);
    else near_gram<3>(acc, X, lane);
    // X1 = Phi(E - P) on the wave's rows, kept in registers
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = 16 * w + 4 * q + kk, c = 16 * s + i16;
            const double e = (G[r][c] - ((r == c) ? 1.0 : 0.0)) - acc[s][q];
            acc[s][q] = (r > c) ? 0.0 : ((r == c) ? 0.5 * e : e);
        }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = 16 * w + 4 * q + kk, c = 16 * s + i16;
            X[r][c] = acc[s][q];
            G[r][c] = ((r == c) ? 1.0 : 0.0) + acc[s][q];
            if (r == c) rdiag[r] = 1.0 + acc[s][q];
        }
    __syncthreads();
    // X = I - X1 + X1^2 (X1^2 upper; the lower blocks keep X1's zeros)
    f64x4 sq[4];
    mm_upper_upper(sq, [&](int r, int c) { return X[r][c]; }, [&](int r, int c) { return X[r][c]; }, lane, w);
    __syncthreads();
    for_uu(sq, [&](int r, int c, double v) { X[r][c] = (((r == c) ? 1.0 : 0.0) - X[r][c]) + v; }, lane, w);
    __syncthreads();
}


// One workgroup, 256 threads.  Bound: latency (two of these per panel are
// about half of the panel chain): the pivots' dependent operations, then LDS
// round trips between small products.  Launch to end on MI355X, 64 columns:
// pass 1 17.1 us, pass 2 31.5 us (37 us with a pivoted Cholesky); 25.0 and
// 46.9 (59) us with every phase on all four waves one after the other.
//   pass 1: R1 = chol(G), R1^{-1}; flags the panel (structurally exact
//           reflectors, or a pivot below CQR_RATIO).
//   flagged panel, pass 2: the exact one-reflector loop instead.
//   pass 2: R2 = chol(G2), Q_top = Q1_top R2^{-1}, LU of Q_top - S, then
//           R_house = S R2 R1, up, the stored tails of the top block, T_V
//           and W^{-1} = R1^{-1} R2^{-1} U^{-1} diag(up).
__global__ void __launch_bounds__(256) cqr_chol_kernel(CholArgs p)
{
    __builtin_amdgcn_s_setprio(3);   // single workgroup on the critical path: issue ahead of co-resident bulk waves
    __shared__ double M0[NB][LD65];
    __shared__ double M1[NB][LD65];
    __shared__ double M2[NB][LD65];
    __shared__ double M3[NB][LD65];
    __shared__ double DU0[16][17], DL[NB][17], DLL[NB][17];
    __shared__ double gdiag[NB], rdiag[NB], sgn[NB], udiag[NB], upv[NB], rupv[NB];
    __shared__ int bad, structural_sh, nonid_sh;
    const int tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);   // a scalar: uniform branches
    const int bw = p.bw;
    if (tid == 0) {
        structural_sh = 0;
        nonid_sh = 0;
        bad = 0;
    }
    __shared__ double red[4][PW], wsh[NB], sc[4];
    const ExactArgs ex{p.A, p.lda, p.m, p.c0, bw, p.up, p.T};
    if (*((volatile int *)p.flag)) {
        // flagged up front or in pass 1: the exact loop factors the panel
        if (p.pass == 2) exact_panel<4>(ex, tid, red, wsh, sc, M0, M1, gdiag, rdiag);
        return;
    }
    int tsi = 0;
#define HQR_TS()                                                                 \
    do {                                                                         \
        if (p.tstamp && tid == 0) p.tstamp[tsi] = (long long)wall_clock64();     \
        ++tsi;                                                                   \
    } while (0)
    HQR_TS();
    // G -> M0, Q1_top -> M2 and R1 -> M3 (the last two idle until after the
    // Cholesky factorization; read in pass 1 too, where they are unused):
    // all 48 loads of a thread are issued before the first is waited for
    {
        double gl[16], ql[16], rl[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            const int idx = tid + 256 * t;
            gl[t] = p.G[idx];
            ql[t] = p.q1top[idx];
            rl[t] = p.r1[idx];
        }
        __syncthreads();   // the flags are clear before any thread sets nonid_sh (the loads stay in flight)
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            pin(gl[t]);
            pin(ql[t]);
            pin(rl[t]);
        }
        int far = 0;   // an entry of G - I beyond CQR_SERIES_TAU
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            const int idx = tid + 256 * t, i = idx / NB, j = idx % NB;
            const double g = (i < bw && j < bw) ? gl[t] : 0.0;
            M0[i][j] = g;
            M2[i][j] = ql[t];
            M3[i][j] = rl[t];
            if (p.pass == 2) {
                const double e = g - ((i == j) ? 1.0 : 0.0);
                far |= !(fabs(e) <= CQR_SERIES_TAU);
                M1[i][j] = (i < j) ? e : ((i == j) ? 0.5 * e : 0.0);   // Phi(E)
            }
        }
        if (far) nonid_sh = 1;
    }
    int structural = 0;
    if (p.pass == 1 && tid == 0) {
        const unsigned long long all = *p.mask_all;
        const unsigned long long need = (bw == 64) ? ~0ull : ((1ull << bw) - 1ull);
        structural = ((all & need) != need);
        structural_sh = structural;
    }
    __syncthreads();
    // pass 2 of a full-width panel whose Gram matrix is within the series
    // bound of the identity: no sequential pivots
    const bool series = p.pass == 2 && bw == NB && !nonid_sh;
    HQR_TS();
    if (series)
        chol_near_identity(M0, M1, rdiag, lane, w);
    else
        chol64_dpp(M0, M1, bw, lane, w, CQR_RATIO, gdiag, rdiag, &bad);
    HQR_TS();
    // 1: an exactly zero column tail (only the exact loop keeps H_k = I);
    // 2: a pivot below the ratio (a TSQR panel can still take over)
    if (tid == 0 && (bad || structural)) *((volatile int *)p.flag) = structural ? 1 : 2;
    __syncthreads();
    if (bad && p.pass == 2) {
        exact_panel<4>(ex, tid, red, wsh, sc, M0, M1, gdiag, rdiag);
        return;
    }
    if (bad || structural_sh) return;
    HQR_TS();

    if (p.pass == 1) {
        double rv[16], iv[16];
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            rv[t] = M0[w + 4 * t][lane];
            iv[t] = M1[w + 4 * t][lane];
        }
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            pin(rv[t]);
            pin(iv[t]);
        }
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            p.r1[tid + 256 * t] = rv[t];
            p.r1inv[tid + 256 * t] = iv[t];
        }
        return;
    }

    // ---- pass 2: M0 = R2, M1 = R2^{-1}, M2 = Q1_top, M3 = R1
    // M2 = Q_top = Q1_top R2^{-1}
    {
        f64x4 qacc[4];
        mm_full_upper(qacc, [&](int r, int c) { return M2[r][c]; }, [&](int r, int c) { return M1[r][c]; }, lane, w);
        __syncthreads();
#pragma unroll
        for (int s = 0; s < 4; ++s) st_blk(M2, 16 * w, 16 * s, qacc[s], 1.0, lane);
    }
    HQR_TS();
    // LU of Q_top - S in M2.  Waves 0 and 1 work on its pivots; waves 2 and 3
    // form beside them what does not wait for the pivots or waits for earlier
    // block steps only:
    //   step 0: R = R2 R1 over R2 (M0), half the products each
    //   step 1: P = R1^{-1} R2^{-1} over R2^{-1} (M1), R1^{-1} from global
    //           memory
    //   from step 1, in M3 (R1 until step 0): wave 2 U^{-1}'s block columns
    //           above the diagonal blocks wave 1 leaves there (step 0's comes
    //           through DU0), wave 3 L^{-1}'s block rows below them (L^{-1}'s
    //           diagonal blocks are in DL); each block's sum one step before
    //           its product with the new diagonal block
    // After the last pivot one product per block of the last column and row
    // and the products T and W^{-1} = P U^{-1} diag(up) are left.
    f64x4 y0 = {0.0, 0.0, 0.0, 0.0}, y1 = y0, y2 = y0;
    __syncthreads();
#pragma unroll 1
    for (int kb = 0; kb < 4; ++kb) {
        // opaque per step: the LDS addresses of the products below would
        // otherwise be computed before the loop and kept in ~150 registers
        int ln = lane;
        asm volatile("" : "+v"(ln));
        double *XU = (kb == 0) ? &DU0[0][0] : &M3[16 * kb][16 * kb];
        lu64_pivots(M2, DL, DLL, XU, (kb == 0) ? 17 : LD65, kb, ln, w, sgn, udiag);
        if (w >= 2) {
            if (kb == 0) {
                if (w == 2) {
                    mul_upper_row<0>(M0, M3, ln);
                } else {
                    mul_upper_row<1>(M0, M3, ln);
                    mul_upper_row<2>(M0, M3, ln);
                    mul_upper_row<3>(M0, M3, ln);
                }
            } else if (kb == 1) {
                if (w == 2) {
                    mul_upper_col<3>(p.r1inv, M1, ln);
                    const int i16 = ln & 15, kk = ln >> 4;
#pragma unroll
                    for (int q = 0; q < 4; ++q) M3[4 * q + kk][i16] = DU0[4 * q + kk][i16];
                    y0 = mma_sum_t(M3, 0, M2, 1, 0, 1, ln);
                } else {
                    mul_upper_col<0>(p.r1inv, M1, ln);
                    mul_upper_col<1>(p.r1inv, M1, ln);
                    mul_upper_col<2>(p.r1inv, M1, ln);
                    y0 = mma_sum(M2, 1, M3, DL, 0, ln);
                }
            } else if (kb == 2) {
                if (w == 2) {
                    inv_upper_close(M3, 0, 1, y0, ln);
                    y0 = mma_sum_t(M3, 0, M2, 2, 0, 2, ln);
                    y1 = mma_sum_t(M3, 1, M2, 2, 1, 2, ln);
                } else {
                    inv_lower_close(M3, DL, 1, 0, y0, ln);
                    y0 = mma_sum(M2, 2, M3, DL, 0, ln);
                    y1 = mma_sum(M2, 2, M3, DL, 1, ln);
                }
            } else if (kb == 3) {
                if (w == 2) {
                    inv_upper_close(M3, 0, 2, y0, ln);
                    inv_upper_close(M3, 1, 2, y1, ln);
                    y0 = mma_sum_t(M3, 0, M2, 3, 0, 3, ln);
                    y1 = mma_sum_t(M3, 1, M2, 3, 1, 3, ln);
                    y2 = mma_sum_t(M3, 2, M2, 3, 2, 3, ln);
                } else {
                    inv_lower_close(M3, DL, 2, 0, y0, ln);
                    inv_lower_close(M3, DL, 2, 1, y1, ln);
                    y0 = mma_sum(M2, 3, M3, DL, 0, ln);
                    y1 = mma_sum(M2, 3, M3, DL, 1, ln);
                    y2 = mma_sum(M2, 3, M3, DL, 2, ln);
                }
            }
        }
        __syncthreads();
        if (kb < 3) lu64_trail(M2, kb, ln, w);
    }
    HQR_TS();
    if (w == 2) {
        inv_upper_close(M3, 0, 3, y0, lane);
        inv_upper_close(M3, 1, 3, y1, lane);
        inv_upper_close(M3, 2, 3, y2, lane);
    } else if (w == 3) {
        inv_lower_close(M3, DL, 3, 0, y0, lane);
        inv_lower_close(M3, DL, 3, 1, y1, lane);
        inv_lower_close(M3, DL, 3, 2, y2, lane);
    } else if (w == 0 && tid < bw) {
        const double rkk = sgn[tid] * M0[tid][tid];   // diag of S R2 R1
        const double tau = -udiag[tid] * sgn[tid];    // = 1 + |pivot|
        const double u = -tau * rkk;
        upv[tid] = u;
        rupv[tid] = 1.0 / u;   // nonzero: tau >= 1 and R_kk != 0 on this path
        p.up[p.c0 + tid] = u;
    }
    __syncthreads();
    HQR_TS();
    // T_Y = -(U S) L^{-T}, T_V = T_Y / (up_i up_j); W^{-1} = P U^{-1} diag(up)
    // (both zero beyond bw and below the diagonal)
    {
        f64x4 tacc[4], wacc[4];
        // L^{-1}: diagonal blocks in DL, the blocks below them in M3
        mm_upper_upper(tacc, [&](int r, int c) { return (c >= r && c < bw) ? M2[r][c] * sgn[c] : 0.0; },
                       [&](int r, int c) {
                           const double *q = ((c >> 4) == (r >> 4)) ? &DL[c][r & 15] : &M3[c][r];
                           return *q;
                       }, lane, w);
        mm_upper_upper(wacc, [&](int r, int c) { return M1[r][c]; }, [&](int r, int c) { return M3[r][c]; }, lane, w);
        HQR_TS();
        for_uu(tacc, [&](int r, int c, double v) {
            p.T[r * NB + c] = (r <= c && c < bw) ? -v * (rupv[r] * rupv[c]) : 0.0;
        }, lane, w);
        for_uu(wacc, [&](int r, int c, double v) { p.winv[r * NB + c] = (c < bw) ? v * upv[c] : 0.0; }, lane, w);
#pragma unroll
        for (int t = 0; t < 16; ++t)
            if (((w + 4 * t) >> 4) > (lane >> 4)) {
                p.T[tid + 256 * t] = 0.0;
                p.winv[tid + 256 * t] = 0.0;
            }
    }
    HQR_TS();
    // the panel's top block: R_house = S R on and above the diagonal, the
    // stored tails L[i][j] * up_j below it
    {
        double tv[16], hv[16], uc[16], sr = sgn[lane];
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            const int c = w + 4 * t;
            const double *lp = ((lane >> 4) == (c >> 4)) ? &DLL[lane][c & 15] : &M2[lane][c];
            tv[t] = *lp;
            hv[t] = M0[lane][c];
            uc[t] = upv[c];
        }
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            pin(tv[t]);
            pin(hv[t]);
            pin(uc[t]);
        }
        if (lane < bw) {
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                const int c = w + 4 * t;
                if (c < bw) HQR_AT(p.A, (int64_t)p.c0 + lane, p.c0 + c, p.lda) = (lane > c) ? tv[t] * uc[t] : sr * hv[t];
            }
        }
    }
    HQR_TS();
#undef HQR_TS
}


__global__ void __launch_bounds__(256) cqr_finish_kernel(FinArgs p)
{
    __shared__ double X[NB][LD65];
    __shared__ double Wi[NB][LD65];
    __shared__ double Y[NB][LD65];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (*((volatile int *)p.flag)) return;
    const int64_t r0 = (int64_t)p.c0 + p.bw + (int64_t)blockIdx.x * 64;
    {
        double wv[16], xv[16];
        mat64_issue(wv, p.winv, tid);
        tile_issue(xv, p.A, p.lda, p.m, r0, p.c0, p.bw, tid);
        mat64_store<false>(Wi, wv, tid);
        tile_store(X, xv, p.m, r0, p.bw, tid);
    }
    __syncthreads();
    mm64(Y, X, Wi, lane, w);
    __syncthreads();
    double yv[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) yv[k] = Y[lane][w + 4 * k];
#pragma unroll
    for (int k = 0; k < 16; ++k) pin_f64(yv[k]);
    if (r0 + lane < p.m) {
#pragma unroll
        for (int k = 0; k < 16; ++k)
            if (w + 4 * k < p.bw) HQR_AT(p.A, r0 + lane, p.c0 + w + 4 * k, p.lda) = yv[k];
    }
}


__global__ void __launch_bounds__(256) narrow_vtx_kernel(NarrowArgs p)
{
    __shared__ double M0[NB][LD65];
    __shared__ double M1[NB][LD65];
    __shared__ double M2[NB][LD65];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t = blockIdx.x;
    const int64_t r0 = (int64_t)p.c0 + 64 * (int64_t)t;
    const bool flagged = *((volatile int *)p.flag) != 0;
    const bool fin = (t > 0) && !flagged;
    // M0 = V rows (top block: unit lower with up on the diagonal), or A_bot;
    // M2 = C; M1 = W^{-1} when finishing
    {
        // the V/A_bot tile and up are loaded alike (the triangle is applied
        // when t == 0), W^{-1} always: every load is issued before the first wait
        double av[16], uv[16], cv[16], wv[16];
        vtile_issue(av, uv, p.A, p.lda, p.up, p.m, r0, p.c0, tid);
        tile_issue(cv, p.A, p.lda, p.m, r0, p.c0 + NB, p.nc, tid);
        mat64_issue(wv, p.winv, tid);
#pragma unroll
        for (int q = 0; q < 16; ++q) pin_f64(wv[q]);   // keeps its loads out of the conditional store
        if (t == 0)
            vtile_store(M0, av, uv, p.m, r0, p.c0, tid);
        else
            tile_store(M0, av, p.m, r0, NB, tid);
        tile_store(M2, cv, p.m, r0, p.nc, tid);
        if (fin) mat64_store<false>(M1, wv, tid);
    }
    __syncthreads();
    double (*V)[LD65] = M0;
    if (fin) {
        // V rows = A_bot W^{-1}: into M1's place after the product
        f64x4 acc[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = f64x4{0.0, 0.0, 0.0, 0.0};
        mm64_acc(acc, M0, M1, 1.0, lane, w);
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 4; ++q) st_blk(M1, 16 * w, 16 * q, acc[q], 1.0, lane);
        __syncthreads();
        V = M1;
        double vv[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) vv[k] = M1[lane][w + 4 * k];
#pragma unroll
        for (int k = 0; k < 16; ++k) pin_f64(vv[k]);
        if (r0 + lane < p.m) {
#pragma unroll
            for (int k = 0; k < 16; ++k) HQR_AT(p.A, r0 + lane, p.c0 + w + 4 * k, p.lda) = vv[k];
        }
    }
    // partial V_t^T C_t
    {
        f64x4 acc[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) acc[q] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int k0 = 0; k0 < NB; k0 += 4) {
            const int kr = k0 + (lane >> 4);
            const double a = V[kr][16 * w + (lane & 15)];
#pragma unroll
            for (int q = 0; q < 4; ++q) acc[q] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, M2[kr][16 * q + (lane & 15)], acc[q], 0, 0, 0);
        }
        // stored transposed, [column j][reflector i], for xw_reduce_kernel
        double *out = p.gpart + (size_t)t * NB * NB;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < 4; ++r) out[(16 * q + (lane & 15)) * NB + 16 * w + 4 * r + (lane >> 4)] = acc[q][r];
    }
}


__global__ void __launch_bounds__(256) xw_reduce_kernel(XwArgs p)
{
    __shared__ double part[4][64];
    __shared__ double xc[64];
    const int tid = threadIdx.x, i = tid & 63, g4 = tid >> 6, j = blockIdx.x;
    const size_t e = (size_t)j * NB + i;
    double tl[16];   // T's loads are in flight beside the partials'
#pragma unroll
    for (int u = 0; u < 16; ++u) tl[u] = p.T[(16 * g4 + u) * NB + i];
    double s = 0.0;
    for (int q0 = g4; q0 < p.parts; q0 += 64) {
        double v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) {
            const int q = q0 + 4 * u;
            v[u] = p.gpart[(size_t)((q < p.parts) ? q : g4) * NB * NB + e];
        }
#pragma unroll
        for (int u = 0; u < 16; ++u) pin_f64(v[u]);
#pragma unroll
        for (int u = 0; u < 16; ++u) s += (q0 + 4 * u < p.parts) ? v[u] : 0.0;
    }
#pragma unroll
    for (int u = 0; u < 16; ++u) pin_f64(tl[u]);
    part[g4][i] = s;
    __syncthreads();
    if (tid < 64) xc[i] = ((part[0][i] + part[1][i]) + part[2][i]) + part[3][i];
    __syncthreads();
    double wv = 0.0;
#pragma unroll
    for (int u = 0; u < 16; ++u) {
        const int l = 16 * g4 + u;
        wv = (l <= i) ? fma(tl[u], xc[l], wv) : wv;
    }
    part[g4][i] = wv;
    __syncthreads();
    if (tid < 64) p.Wt[e] = ((part[0][i] + part[1][i]) + part[2][i]) + part[3][i];
}

// T of a stored panel (compact WY, T upper, Q_panel^T = I + V T^T V^T with
// T[k][k] = tau_k = -1/b_k) from G = V^T V, the splits' partial sums of the
// V^T X pass.  T^{-1} = diag(1/tau) + the strict upper triangle of G, so T
// is the inverse of that upper triangular matrix: its four 16 x 16 diagonal
// blocks by the column recurrence T[i][k] = -tau_k sum_{l=i}^{k-1} T[i][l]
// G[l][k] (one wave each, lane i < 16 keeping row i and adding T[i][l]
// G[l][k] into every later column's sum once T[i][l] is final), then the
// blocks above them by distance from the diagonal on MFMA
// (inv_upper_levels).  Zero taus (identity reflectors, columns past bw) give
// zero rows and columns.  One workgroup of 256 threads per panel.
__global__ void __launch_bounds__(256) tfactor_kernel(TArgs p)
{
    __shared__ double G[NB][LD65];
    __shared__ double Ts[NB][LD65];
    __shared__ double tau[NB];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int c0 = p.c0 + NB * (int)blockIdx.x, bw = min(NB, p.bw - NB * (int)blockIdx.x);
    const double *wpart = p.wpart + (size_t)blockIdx.x * p.wstride;
    double *T = p.T + (size_t)blockIdx.x * NB * NB;
    // G = the splits' partial V^T V summed in split order; a thread's 16
    // elements are loaded together for each split
    constexpr int EPT = NB * NB / 256;
    double gs[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) gs[e] = 0.0;
#pragma unroll 4
    for (int q = 0; q < p.nsplit; ++q) {
        const double *src = wpart + (size_t)q * NB * p.nxpad;
#pragma unroll
        for (int e = 0; e < EPT; ++e) {
            const int idx = tid + 256 * e, i = idx / NB, j = idx - i * NB;
            gs[e] += (i < bw && j < bw) ? src[(size_t)i * p.nxpad + j] : 0.0;
        }
    }
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
        const int idx = tid + 256 * e;
        G[idx / NB][idx % NB] = gs[e];
    }
    if (tid < NB) {
        double t = 0.0;
        if (tid < bw) {
            const double u = p.up[c0 + tid];
            const double rkk = HQR_AT(p.A, (int64_t)c0 + tid, c0 + tid, p.lda);
            t = (u == 0.0) ? 0.0 : -1.0 / (u * rkk);
        }
        tau[tid] = t;
    }
    __syncthreads();
    if (lane < 16) {
        const int b0 = 16 * w, i = lane;
        double acc[16], trow[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) acc[k] = 0.0;
#pragma unroll
        for (int l = 0; l < 16; ++l) {
            trow[l] = (i > l) ? 0.0 : ((i == l) ? tau[b0 + l] : -tau[b0 + l] * acc[l]);
#pragma unroll
            for (int k = l + 1; k < 16; ++k) acc[k] = fma(trow[l], G[b0 + l][b0 + k], acc[k]);
        }
#pragma unroll
        for (int l = 0; l < 16; ++l) Ts[b0 + i][b0 + l] = trow[l];
    }
    inv_upper_levels(Ts, G, lane, w);
    for (int idx = tid; idx < NB * NB; idx += 256) T[idx] = Ts[idx / NB][idx % NB];
}

} // namespace hqr
