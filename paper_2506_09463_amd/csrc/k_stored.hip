// k_stored.hip -- launch functions of the stored-factor kernels
// (hqr_stored.hpp).
#include "hqr_stored.hpp"

namespace hqr {

hipError_t k_stored_gram(int panels, int nsplit, hipStream_t s, const StoredGramArgs &a)
{
    HQR_LAUNCH(K_TFACTOR, stored_gram_kernel, dim3(panels, nsplit), dim3(256), 0, s, a);
    return hipGetLastError();
}

hipError_t k_stored_step(int parts, hipStream_t s, const StoredStepArgs &a)
{
    HQR_LAUNCH(K_UPDATE, stored_step_kernel, dim3(parts), dim3(256), 0, s, a);
    return hipGetLastError();
}

} // namespace hqr
