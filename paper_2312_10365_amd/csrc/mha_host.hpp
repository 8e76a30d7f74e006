// Host-side declarations shared by the attention translation units (mha.hip, mha_dense.hip).
#pragma once
#include "../../include/spt_mha.h"
#include "spt_host.hpp"

namespace spt {

// Attention on the matrix cores (mha_dense.hip): a query block's products as dense tiles in LDS.
hipError_t mha_dense_fwd(const spt_mha_shape_t& s, const void* Q, const void* K, const void* V, const int32_t* idx,
                         float* A, void* Y, hipStream_t st);
hipError_t mha_dense_bwd_q(const spt_mha_shape_t& s, const void* K, const void* V, const void* dY, const int32_t* idx,
                           const float* A, float* dS, void* dQ, hipStream_t st);
hipError_t mha_dense_bwd_kv(const spt_mha_shape_t& s, const void* Q, const void* dY, const int32_t* idx,
                            const float* A, const float* dS, void* dK, void* dV, hipStream_t st);

}  // namespace spt
