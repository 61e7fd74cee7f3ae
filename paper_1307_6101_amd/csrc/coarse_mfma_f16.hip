// Matrix-core kernels of the coarse level on FP16 operator storage.
#include "coarse_mfma_dev.h"

namespace ddamg {

template void coarse_apply_mfma<__half2>(const CoarseOpView<float, __half2>&, const int*, int, const float2*, const float2*,
                                     float2*, hipStream_t, int);
template void coarse_sap_q_mfma<__half2>(const CoarseOpView<float, __half2>&, const SapTables&, const int*, int, int, int,
                                     float2*, const SapScratch<float>&, hipStream_t, int);

}  // namespace ddamg
