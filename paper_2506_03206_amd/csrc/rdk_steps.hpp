// The top-k sparse product for a few positions at a time out of LDS (rdk_steps.hip): its table and its launch.
#pragma once
#include "rdk_slab.hpp"

namespace rdk {

// Whether the form is taken for a batch of B positions.
bool steps_taken(const KernelHandle &h, int32_t B);

// Arguments as launch_slab_product.
rdk_status_t launch_steps_product(const KernelHandle &h, RowInput q, int32_t B, float *out, int64_t ldo, SoftStat *qrow, int kind,
                                 const FuseArgs &f, hipStream_t st);

}  // namespace rdk
