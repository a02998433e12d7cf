// k_chol.hip -- launch functions of the Cholesky factorization and the
// rank-one factor update (hqr_chol.hpp).
#include "hqr_chol.hpp"

namespace hqr {

hipError_t k_chol_first(hipStream_t s, double *S, int64_t lds, int64_t n, double *rinv, int *info)
{
    const CholArgsS a{S, lds, n, 0, 0, rinv, info};
    HQR_LAUNCH(K_CQR_CHOL, chol_syrk_kernel, dim3(1), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t k_chol_block(hipStream_t s, double *S, int64_t lds, int64_t n, int64_t k0, int bw, double *rinv,
                        int *info)
{
    const CholArgsS a{S, lds, n, k0, bw, rinv, info};
    const unsigned T = (unsigned)((n - k0 - bw + 63) / 64);
    HQR_LAUNCH(K_PANEL, chol_panel_kernel, dim3(T), dim3(256), 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    HQR_LAUNCH(K_UPDATE, chol_syrk_kernel, dim3(T * (T + 1) / 2), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t k_chol_update(hipStream_t s, double *R, int64_t ldr, double *v, int64_t n)
{
    if (n <= CHU_SMALL) {
        HQR_LAUNCH(K_REFINE, chol_update_small_kernel, dim3(1), dim3(64), 0, s, R, ldr, v, (int)n);
        return hipGetLastError();
    }
    for (int64_t k0 = -CHU; k0 + CHU < n; k0 += CHU) {
        const unsigned T = (k0 < 0) ? 1u : (unsigned)((n - k0 - CHU + CHU - 1) / CHU);
        HQR_LAUNCH(K_REFINE, chol_update_kernel, dim3(T), dim3(256), 0, s, R, ldr, v, n, k0);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

} // namespace hqr
