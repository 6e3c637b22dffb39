// score.hpp -- what the scoring kernels (score.hip) and the code that launches them share.
#pragma once

#include <cstdint>

#include <hip/hip_runtime.h>

#include "pack.hpp"
#include "planner.hpp"

namespace treeens {

constexpr int kXcds = 8; // accelerator complex dies, each with its own L2
// s_waitcnt immediate for gfx9: vmcnt(0), expcnt and lgkmcnt left at their maxima (no wait)
constexpr int kWaitVmcnt0 = 0x0F70;
// the same with lgkmcnt(0) (LDS and scalar memory) and vmcnt, expcnt at their maxima
constexpr int kWaitLgkmcnt0 = 0xC07F;
constexpr int kPrefetchDepth = 2; // tiles in flight with one workgroup per CU
constexpr int kThreads = 1024; // workgroup size of the scoring kernel (16 waves)
// what a launch of the scoring kernel produces
constexpr int kModeScore = 0;  // scores
constexpr int kModeLeaves = 1; // leaf ids
constexpr int kModeUsage = 2;  // per-document feature bitmasks and their popcounts
constexpr int kModeUsageSlot = 4; // the same with the bitmasks in the unused end of the tile slot
constexpr int kModeVector = 3; // four components of vector-valued scores
constexpr int kModeRows = 5;   // the lower 16 bits of each leaf's row of the leaf-vector table
constexpr int kVecPerLaunch = 4;

using ScoreFn = void (*)(const void *, int64_t, int32_t, int32_t, const uint2 *, int32_t,
                         const uint32_t *, int32_t, int32_t, int32_t, int32_t, int32_t, double *,
                         float *, int32_t *, const int32_t *, const uint32_t *, const int32_t *,
                         int32_t, uint32_t *, int32_t, int32_t, const float4 *, int32_t,
                         int32_t, int32_t, double, int32_t, const uint2 *, int32_t, uint32_t,
                         const uint32_t *, const int32_t *, uint16_t *);

// The scoring kernel of a plan for one mode (nullptr: none). Each mode's kernels are compiled from
// score.hip by themselves.
template <int MODE>
ScoreFn pick_kernel(const LdsPlan &p, bool compact);

} // namespace treeens
