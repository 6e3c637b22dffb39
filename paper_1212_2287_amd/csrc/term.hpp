// term.hpp -- launch of the scoring kernel of terminal packets (term.hip; see TermPlan in pack.hpp).
#pragma once

#include <cstdint>

#include <hip/hip_runtime.h>

#include "pack.hpp"

namespace treeens {

// codes: rows of n_cols codes, each staged as code << kCompactCodeShift | 31. Blocks of 64 documents:
// `head` of them walk all packets, the others are split over `splits` workgroups that leave partial
// sums [split][doc - head * 64].
void launch_term(const TermPlan &t, hipStream_t stream, const uint16_t *codes, int64_t n_docs, int32_t n_cols,
                 const uint32_t *packets, const uint32_t *slots, int64_t head, int splits, double *partials,
                 float *scores, double scale);

} // namespace treeens
