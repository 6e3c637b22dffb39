// uniform.hpp -- launch of the uniform kernels (uniform.hip): models of shallow trees whose nodes
// are all evaluated for every document (see UniformPlan in pack.hpp).
#pragma once

#include <cstdint>

#include <hip/hip_runtime.h>

#include "pack.hpp"
#include "planner.hpp"

namespace treeens {

// codes: rows of n_cols 16-bit threshold codes. Blocks past the head leave partial sums
// [split][doc - head * docs_per_block] in `partials` (splits > 1).
void launch_uniform(const UniformPlan &u, hipStream_t stream, const uint16_t *codes, int64_t n_docs, int32_t n_cols,
                    const uint32_t *nodes, const double *leaves, const LaunchShape &shape, double *partials,
                    float *scores, double scale);

} // namespace treeens
