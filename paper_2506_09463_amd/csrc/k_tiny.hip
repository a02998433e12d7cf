// k_tiny.hip -- launch function of the smallest problems' kernel
// (hqr_tiny.hpp).
#include "hqr_tiny.hpp"

namespace hqr {

hipError_t k_wg_tiny(hipStream_t s, const WgDesc &d, int *info, int *iters)
{
    const bool narrow = d.n + d.nrhs <= 16;
    if (d.m <= 64) {
        if (narrow) HQR_LAUNCH(K_SMALL, (wg_tiny_kernel<16, 1>), dim3(1), dim3(64), 0, s, d, info, iters);
        else HQR_LAUNCH(K_SMALL, (wg_tiny_kernel<32, 1>), dim3(1), dim3(64), 0, s, d, info, iters);
    } else {
        if (narrow) HQR_LAUNCH(K_SMALL, (wg_tiny_kernel<16, 2>), dim3(1), dim3(64), 0, s, d, info, iters);
        else HQR_LAUNCH(K_SMALL, (wg_tiny_kernel<32, 2>), dim3(1), dim3(64), 0, s, d, info, iters);
    }
    return hipGetLastError();
}

} // namespace hqr
