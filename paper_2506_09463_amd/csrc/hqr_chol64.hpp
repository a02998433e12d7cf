// hqr_chol64.hpp -- one workgroup's Cholesky factorization and triangular
// inverse of a 64 x 64 block in LDS, and the 16 x 16 block helpers it shares
// with the panel algebra (hqr_cqr.hpp).
#pragma once

#include <utility>

#include "hqr_args.hpp"

namespace hqr {

// ------------------------------------------- 16 x 16 blocks on MFMA
// FP64 MFMA 16x16x4 layouts: A[i][k] at lane i + 16k, B[k][j] at lane
// j + 16k, D[i][j] at lane j + 16 (i % 4), register i / 4.  A product D
// feeds the next MFMA as its B operand directly: register q is the B operand
// of the k-chunk 4q..4q+3.

// acc += MA[ar:ar+16][ac:ac+16] * MB[br:br+16][bc:bc+16]
HQR_DEV f64x4 mma_blk(f64x4 acc, const double (*MA)[LD65], int ar, int ac, const double (*MB)[LD65], int br, int bc,
                      int lane)
{
    const int i = lane & 15, kk = lane >> 4;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int k = 4 * q + kk;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(MA[ar + i][ac + k], MB[br + k][bc + i], acc, 0, 0, 0);
    }
    return acc;
}

// acc += MA[ar:ar+16][ac:ac+16] * D  (D a 16 x 16 block in D layout)
HQR_DEV f64x4 mma_blk_reg(f64x4 acc, const double (*MA)[LD65], int ar, int ac, f64x4 d, int lane)
{
    const int i = lane & 15, kk = lane >> 4;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(MA[ar + i][ac + 4 * q + kk], d[q], acc, 0, 0, 0);
    return acc;
}

HQR_DEV void st_blk(double (*M)[LD65], int r0, int c0, f64x4 d, double scale, int lane)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) M[r0 + 4 * r + (lane >> 4)][c0 + (lane & 15)] = scale * d[r];
}

// 16 x 16 LDS block in D layout (to accumulate an MFMA update onto it)
HQR_DEV f64x4 ld_blk(const double (*M)[LD65], int r0, int c0, int lane)
{
    f64x4 d;
#pragma unroll
    for (int r = 0; r < 4; ++r) d[r] = M[r0 + 4 * r + (lane >> 4)][c0 + (lane & 15)];
    return d;
}

// ------------------------------------------------- in-row broadcasts
// The value that lane 16r + I holds, in every lane of the 16-lane row r
// (DPP row_newbcast; one v_mov_b64_dpp for a double).
template <int I> HQR_DEV double bc16c(double v)
{
    const long b = __builtin_bit_cast(long, v);
    const long r = __builtin_amdgcn_mov_dpp(b, 0x150 + I, 0xf, 0xf, false);
    return __builtin_bit_cast(double, r);
}

// Pins v in a register at this point of the program: the compiler may not
// move its computation past it (used to keep long update chains in order).
HQR_DEV void pin(double &v) { asm volatile("" : "+v"(v)); }

// i must be a constant once the caller's loops are unrolled
HQR_DEV double bc16(double v, int i)
{
    switch (i) {
    case 0: return bc16c<0>(v);
    case 1: return bc16c<1>(v);
    case 2: return bc16c<2>(v);
    case 3: return bc16c<3>(v);
    case 4: return bc16c<4>(v);
    case 5: return bc16c<5>(v);
    case 6: return bc16c<6>(v);
    case 7: return bc16c<7>(v);
    case 8: return bc16c<8>(v);
    case 9: return bc16c<9>(v);
    case 10: return bc16c<10>(v);
    case 11: return bc16c<11>(v);
    case 12: return bc16c<12>(v);
    case 13: return bc16c<13>(v);
    case 14: return bc16c<14>(v);
    default: return bc16c<15>(v);
    }
}

// s = sqrt(d) and r = 1/sqrt(d): the hardware reciprocal square root refined
// by two coupled Newton steps (Goldschmidt's iteration for s and 1/(2s)) and
// a final residual correction of s.  d below 2^-900 is scaled by 2^1000
// first; d <= 0 (or NaN) gives s = r = 1, the caller flags such pivots.
HQR_DEV void pivot_sqrt(double d, double &s, double &r)
{
    const bool pos = d > 0.0;
    const bool sc = pos && d < 0x1p-900;
    const double x = pos ? (sc ? d * 0x1p+1000 : d) : 1.0;
    const double y = __builtin_amdgcn_rsq(x);
    double sv = x * y, h = 0.5 * y;
    double e = fma(-sv, h, 0.5);
    sv = fma(sv, e, sv);
    h = fma(h, e, h);
    e = fma(-sv, h, 0.5);
    sv = fma(sv, e, sv);
    h = fma(h, e, h);
    sv = fma(h, fma(-sv, sv, x), sv);
    s = sc ? sv * 0x1p-500 : sv;
    r = sc ? (2.0 * h) * 0x1p+500 : 2.0 * h;
}

// 1/u from the hardware reciprocal and two Newton steps (|u| >= 1 here).
HQR_DEV double recip_nr(double u)
{
    double y = __builtin_amdgcn_rcp(u);
    double e = fma(-u, y, 1.0);
    y = fma(y, e, y);
    e = fma(-u, y, 1.0);
    return fma(y, e, y);
}

// r = 1/sqrt(d) on a pivot chain: the hardware reciprocal square root (about
// 2^-24 relative) and one cubic step, r = y (1 + e/2 + 3 e^2/8) with
// e = 1 - d y^2, exact to below FP64 rounding in four dependent operations
// (two coupled Newton steps take seven).  d <= 0 (or NaN) gives a value that
// is not finite or not meaningful; the caller flags such pivots.
HQR_DEV double pivot_rsqrt(double d)
{
    const double y = __builtin_amdgcn_rsq(d);
    const double e = fma(-(d * y), y, 1.0);
    return fma(y * e, fma(e, 0.375, 0.5), y);
}

// pivot_rsqrt cut into its dependent stages, so that independent updates can
// be placed between them (y holds the result after stage 3).
struct PivotChain {
    double d, y, t, e, a, b;
    __device__ __forceinline__ void start(double dv)
    {
        d = dv;
        y = __builtin_amdgcn_rsq(d);
        pin(y);
    }
    template <int U> __device__ __forceinline__ void stage()
    {
        if constexpr (U == 0) {
            t = d * y;
            pin(t);
        } else if constexpr (U == 1) {
            e = fma(-t, y, 1.0);
            pin(e);
        } else if constexpr (U == 2) {
            a = y * e;
            b = fma(e, 0.375, 0.5);
            pin(a);
            pin(b);
        } else if constexpr (U == 3) {
            y = fma(a, b, y);
            pin(y);
        }
    }
};

// recip_nr in stages, the same way.
struct RecipChain {
    double u0, y, e;
    __device__ __forceinline__ void start(double u)
    {
        u0 = u;
        y = __builtin_amdgcn_rcp(u);
        pin(y);
    }
    template <int U> __device__ __forceinline__ void stage()
    {
        if constexpr (U == 0 || U == 2) {
            e = fma(-u0, y, 1.0);
            pin(e);
        } else if constexpr (U == 1 || U == 3) {
            y = fma(y, e, y);
            pin(y);
        }
    }
};

// The transposed block product Y^T = sum_k MB[16k.., 16j..]^T MA[16i.., 16k..]^T
// (k = k0 .. k1-1) in D layout, i.e. D[a][b] = Y[b][a] with
// Y = sum_k MA_ik MB_kj.
HQR_DEV f64x4 mma_sum_t(const double (*MA)[LD65], int i, const double (*MB)[LD65], int j, int k0, int k1, int lane)
{
    const int i16 = lane & 15, kk = lane >> 4;
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
    for (int k = k0; k < k1; ++k) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = 16 * k + 4 * q + kk;
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(MB[r][16 * j + i16], MA[16 * i + i16][r], acc, 0, 0, 0);
        }
    }
    return acc;
}

// X_ij = -Y X_jj for an upper inverse whose diagonal block X_jj is in place,
// from Y^T in D layout (mma_sum_t): X_ij^T = -X_jj^T Y^T.
HQR_DEV void inv_upper_close(double (*X)[LD65], int i, int j, f64x4 yt, int lane)
{
    const int i16 = lane & 15, kk = lane >> 4;
    f64x4 acc = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
    for (int q = 0; q < 4; ++q)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(X[16 * j + 4 * q + kk][16 * j + i16], yt[q], acc, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < 4; ++q) X[16 * i + i16][16 * j + 4 * q + kk] = -acc[q];
}

// Trailing block update M_ij -= MA_i^T-or-L rows of block step b0 on MFMA:
// the Cholesky form M_ij -= G_bi^T G_bj over the rows b0 .. b0 + 15.
HQR_DEV void chol_trail_blk(double (*G)[LD65], int b0, int ib, int jb, int lane)
{
    const int i16 = lane & 15, kk = lane >> 4;
    f64x4 acc = ld_blk(G, 16 * ib, 16 * jb, lane);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int k = b0 + 4 * q + kk;
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(-G[k][16 * ib + i16], G[k][16 * jb + i16], acc, 0, 0, 0);
    }
    st_blk(G, 16 * ib, 16 * jb, acc, 1.0, lane);
}

// One pivot of the 16 x 16 elimination in chol64_dpp: on entry d is pivot I
// and r its reciprocal root, on exit those of pivot I + 1.  Row I + 1 is
// updated first; its pivot's reciprocal root is then formed, a stage at a
// time, between the updates of the other rows (two rows' broadcasts together,
// so no FMA waits for its broadcast).  Templates rather than unrolled loops:
// every register index has to be static.
template <int I, int U>
HQR_DEV void chol16_rows(double (&g)[16], double (&z)[16], double vg, double vz, PivotChain &pc)
{
    constexpr int i2 = I + 2 + 2 * U;
    if constexpr (i2 < 16) {
        double ta = bc16c<i2>(vg), tb;
        pin(ta);
        if constexpr (i2 + 1 < 16) {
            tb = bc16c<i2 + 1>(vg);
            pin(tb);
        }
        g[i2] = fma(-ta, vg, g[i2]);
        z[i2] = fma(-ta, vz, z[i2]);
        pin(g[i2]);
        pin(z[i2]);
        if constexpr (i2 + 1 < 16) {
            g[i2 + 1] = fma(-tb, vg, g[i2 + 1]);
            z[i2 + 1] = fma(-tb, vz, z[i2 + 1]);
            pin(g[i2 + 1]);
            pin(z[i2 + 1]);
        }
    }
    pc.template stage<U>();
}

template <int I>
HQR_DEV void chol16_pivot(double (&g)[16], double (&z)[16], double &d, double &r, double &my_d, int jj)
{
    const double vg = g[I] * r, vz = z[I] * r;
    g[I] = vg;
    z[I] = vz;
    my_d = (jj == I) ? d : my_d;
    if constexpr (I < 15) {
        const double t1 = bc16c<I + 1>(vg);
        g[I + 1] = fma(-t1, vg, g[I + 1]);
        pin(g[I + 1]);
        d = bc16c<I + 1>(g[I + 1]);
        pin(d);
        z[I + 1] = fma(-t1, vz, z[I + 1]);
        PivotChain pc;
        pc.start(d);
        chol16_rows<I, 0>(g, z, vg, vz, pc);
        chol16_rows<I, 1>(g, z, vg, vz, pc);
        chol16_rows<I, 2>(g, z, vg, vz, pc);
        chol16_rows<I, 3>(g, z, vg, vz, pc);
        chol16_rows<I, 4>(g, z, vg, vz, pc);
        chol16_rows<I, 5>(g, z, vg, vz, pc);
        chol16_rows<I, 6>(g, z, vg, vz, pc);
        r = pc.y;
    }
    __builtin_amdgcn_sched_barrier(0);
}

template <int... Is>
HQR_DEV void chol16_pivots(double (&g)[16], double (&z)[16], double &d, double &r, double &my_d, int jj,
                           std::integer_sequence<int, Is...>)
{
    (chol16_pivot<Is>(g, z, d, r, my_d, jj), ...);
}

// In-place upper Cholesky G = R^T R of the n x n leading block of G (R in the
// upper triangle, zeros below, identity beyond n; G's entries outside the
// block must be zero) and X = R^{-1} (zeros below), right-looking by
// 16-column block steps; 256 threads.
//
// Bound: the serial chain of 64 pivots in one wave.  Block step kb: wave 0
// eliminates [G_kk | I | G_k,kb+1.. ] in registers: every 16-lane row holds a
// copy of the diagonal block (lane 16r + j: its column j, array g), and array
// z holds an identity column in the lanes of row 0 and the columns of the
// block row in rows 1..3, so one broadcast and two FMAs per entry of R give
// R_kk, R_kk^{-T} and the block row; R_kk^{-T}'s column j is row j of
// X_kk.  No lane masks inside: entries of g left of the pivot are never read.
// Waves 1..3 meanwhile do what the next pivots do not need: the trailing
// blocks outside block row kb (of the previous step) and X's block column kb,
// X_ik = -(sum_l X_il R_lk) X_kk, whose sums need only earlier steps.
// Only the blocks of block row kb + 1 are updated between two barriers.
// 9.4 us for 64 columns on MI355X, against 17.5 us for a factorization with
// three FMAs and two lane masks per entry, seven dependent operations per
// reciprocal root and the inverse's off-diagonal blocks after it.
//
// gdiag gets G's diagonal (1 beyond n), rdiag R's; *bad is set to one plus
// the smallest pivot index whose pivot is not above ratio * G_kk (ratio 0: not
// positive).  Starts and ends with a barrier.
HQR_DEV void chol64_dpp(double (*G)[LD65], double (*X)[LD65], int n, int lane, int w, double ratio,
                        double *gdiag, double *rdiag, int *bad)
{
    const int tid = 64 * w + lane;
    __syncthreads();
    if (tid < NB) {
        gdiag[tid] = (tid < n) ? G[tid][tid] : 1.0;
        if (tid >= n) G[tid][tid] = 1.0;
    }
    if (tid == 0) *bad = 0;
    f64x4 yt = {0.0, 0.0, 0.0, 0.0};   // wave w >= 1: Y^T of X's block (w - 1, kb)
    __syncthreads();
#pragma unroll 1
    for (int kb = 0; kb < 4; ++kb) {
        const int b0 = 16 * kb;
        if (w == 0) {
            // opaque per block step: keeps the per-pivot lane masks from being
            // hoisted out of the kb loop (they would occupy ~100 SGPRs)
            int ln = lane;
            asm volatile("" : "+v"(ln));
            const int jj = ln & 15, c = b0 + ln;
            const bool aug = ln < 16, act = c < NB;
            // 32 loads in flight from two addresses per lane, pinned before
            // the selects (a conditional load becomes a branch and a wait of
            // its own); the stores below likewise in two straight runs
            double g[16], z[16];
            const double *gp = &G[b0][b0 + jj], *zp = &G[b0][act ? c : b0 + jj];
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                g[i] = gp[i * LD65];
                z[i] = zp[i * LD65];
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                pin(g[i]);
                pin(z[i]);
            }
#pragma unroll
            for (int i = 0; i < 16; ++i) z[i] = aug ? ((i == jj) ? 1.0 : 0.0) : z[i];
            double my_d = 1.0;         // lane i (and 16r + i): pivot i
            double d = bc16c<0>(g[0]), r = pivot_rsqrt(d);
            chol16_pivots(g, z, d, r, my_d, jj, std::make_integer_sequence<int, 16>{});
            double my_s, my_r;
            pivot_sqrt(my_d, my_s, my_r);
            // row 0: R_kk's column jj and row jj of X_kk; rows 1..3: the block row
            if (aug) {
                double *xp = &X[b0 + jj][b0], *rp = &G[b0][b0 + jj];
#pragma unroll
                for (int i = 0; i < 16; ++i) xp[i] = z[i];
#pragma unroll
                for (int i = 0; i < 16; ++i) rp[i * LD65] = (i < jj) ? g[i] : 0.0;
                rp[jj * LD65] = my_s;
            } else if (act) {
                double *rp = &G[b0][c];
#pragma unroll
                for (int i = 0; i < 16; ++i) rp[i * LD65] = z[i];
            }
            const double least = (ratio > 0.0) ? ratio * gdiag[b0 + jj] : 0.0;
            const bool badl = aug && b0 + jj < n && !(my_d > least);
            if (aug) rdiag[b0 + jj] = my_s;
            const unsigned long long bm = __ballot(badl);
            if (bm && lane == 0 && *bad == 0) *bad = b0 + (int)__ffsll((long long)bm);
        } else {
            // the previous step's trailing blocks below block row kb
            if (kb > 0) {
                int cnt = 0;
                for (int a = kb + 1; a <= 3; ++a)
                    for (int b = a; b <= 3; ++b, ++cnt)
                        if (cnt % 3 == w - 1) chol_trail_blk(G, b0 - 16, a, b, lane);
            }
            // X's column kb - 1 closed (its sums are from the previous step)
            if (w - 1 < kb - 1) inv_upper_close(X, w - 1, kb - 1, yt, lane);
            if (kb == 0) {
                // zeros below the diagonal blocks, of G and X
                for (int idx = tid - 64; idx < NB * NB; idx += 192) {
                    const int r = idx / NB, cc = idx % NB;
                    if ((r >> 4) > (cc >> 4)) {
                        G[r][cc] = 0.0;
                        X[r][cc] = 0.0;
                    }
                }
            }
            // sums of column kb need X's columns < kb in row w - 1, which
            // this wave itself wrote, and its diagonal block (wave 0, before
            // the last barrier)
            if (w - 1 < kb) yt = mma_sum_t(X, w - 1, G, kb, w - 1, kb, lane);
        }
        __syncthreads();
        if (kb < 3) {
            const int jb = kb + 1 + w;
            if (jb <= 3) chol_trail_blk(G, b0, kb + 1, jb, lane);
            __syncthreads();
        }
    }
    if (w > 0) inv_upper_close(X, w - 1, 3, yt, lane);
    __syncthreads();
}

} // namespace hqr
