// Coarse operator and SAP steps of batches on the matrix cores (FP32
// arithmetic): the calls of coarse.hip, defined per operator storage in
// coarse_mfma_f16.hip and coarse_mfma_f32.hip from coarse_mfma_dev.h.
#pragma once

#include "coarse.h"

namespace ddamg {

// out = K in over the sites of `sites` (nullptr: every site) for nb fields, or
// with b given out = b - K in
template <typename S>
void coarse_apply_mfma(const CoarseOpView<float, S>& op, const int* sites, int nsites, const float2* in,
                       const float2* b, float2* out, hipStream_t s, int nb);

// MR step `step` of a SAP colour pass for nb fields (see coarse_sap_colour)
template <typename S>
void coarse_sap_q_mfma(const CoarseOpView<float, S>& op, const SapTables& tb, const int* csites, int nsites, int pos0,
                       int step, float2* z, const SapScratch<float>& ws, hipStream_t s, int nb);

}  // namespace ddamg
