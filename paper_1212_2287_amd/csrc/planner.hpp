// planner.hpp -- launch shapes of the scoring kernels (host code, no HIP call).
#pragma once

#include <algorithm>
#include <cstdint>

#include "pack.hpp"

namespace treeens {

constexpr int kNumCus = 256;

// Launch shape for a batch of n_blocks document blocks: a tiling level, a number of head blocks walked
// whole by one workgroup each, and the split count of the remaining (tail) blocks, each split over that
// many workgroups that walk a contiguous share of the tiles (or packets) each.
struct LaunchShape {
    int level = 0;
    int64_t head = 0;
    int splits = 1;
};

// What a launch does with the leaves it reaches.
enum class Work {
    kScores,    // adds their values: split blocks take a second kernel
    kVector,    // adds four values of each, gathered from the leaf-vector table
    kPositions, // stores them (leaf ids, leaf rows)
    kTerminal,  // scores by terminal packets
};

// What the planner knows of a model's tiles or packets (see LaunchShape), per tiling level: their number
// and the rounds of the fullest one and on average (a round: every walker walks one group of trees);
// what switching to the next costs, in rounds.
struct Tiling {
    int n_levels = 1;
    int tiles[kTileLevels] = {};
    int max_rounds[kTileLevels] = {};
    double mean_rounds[kTileLevels] = {};
    double switch_rounds = 0.0;
};
struct PlanFacts {
    Tiling walk, term;
    bool pairs = false, full = false; // two workgroups on a CU; four trees per lane
    double mean_steps = 0.0;
};

constexpr double kTileRounds = 0.5;   // switching tiles (barriers, the copy into LDS), in walker rounds
constexpr double kPacketRounds = 0.1; // switching packets (no barrier), in walker rounds

inline PlanFacts plan_facts(const Packed &p) {
    PlanFacts f;
    f.pairs = p.plan.lds_bytes <= kLdsPerCu / 2;
    f.full = p.plan.interleave == 4;
    f.mean_steps = p.mean_steps;
    auto packets = [](int per_wave, int max_groups, double mean_groups) {
        Tiling t;
        t.tiles[0] = per_wave, t.max_rounds[0] = max_groups, t.mean_rounds[0] = mean_groups;
        t.switch_rounds = kPacketRounds;
        return t;
    };
    if (p.cp_k > 0) {
        f.walk = packets(p.cp_per_walker, p.cp_max_groups, p.cp_mean_groups);
    } else if (p.pk_recs > 0) {
        f.walk = packets(p.pk_per_walker, p.pk_max_groups, p.pk_mean_groups);
    } else {
        f.walk.n_levels = kTileLevels;
        f.walk.switch_rounds = kTileRounds;
        for (int k = 0; k < kTileLevels; ++k) {
            f.walk.tiles[k] = p.level_begin[k + 1] - p.level_begin[k];
            f.walk.max_rounds[k] = p.level_max_rounds[k];
            f.walk.mean_rounds[k] = p.level_mean_rounds[k];
        }
    }
    f.term = packets(p.term.per_wave, p.term.max_groups, p.term.mean_groups);
    return f;
}

// The estimate, in microseconds, is that of the fullest place: its workgroups' rounds, the first
// workgroup's staging, prologue and reduction (kFirst), what each further one adds, and the second
// kernel. 1,000 trees of 32 leaves (16 rounds of 1.21 us), times of a call against the estimate plus 6 us
// of launch: 16,000 documents whole 31.8 (28.9), in halves 37.3 (34.4); 20,000 whole 49.1 (49.1);
// 40,000 whole 70.1 (69.2); 100,000 whole 144.5 (149.8), with 27 blocks split 132.8 (134).
// A share of t tiles takes their rounds on average, and once those of the fullest beyond that (600 trees
// of 5 to 300 leaves, 3,000 documents: tiles of up to 6 rounds, 1.25 on average; one per workgroup 28.3
// us, four 22.7).
// Candidates: all blocks split alike (small batches spread over the GPU), and whole rounds of one
// block per place as head, the rest split to fill the places evenly (313 blocks on 256 CUs whole would
// take as long as 512).
//
// Two workgroups on a CU with four trees per lane keep both its pipes busy, so they take twice as long
// as one would: the CU is one place, 350 cycles a step, and the second one's staging is mostly hidden.
// With fewer trees per lane they wait for latency and run side by side. Gathers of leaf vectors
// lie between: a lone workgroup takes a little longer than one of two.
// The other plans' steps and staging take longer than these figures say, both by about the same
// factor: 0.15 to 0.3 us a step and 5 to 18 us. Their ratio is what chooses. Over 542 batches of 40
// models, each measured in all its shapes, the shapes picked take 1 to 3% longer than the fastest on
// average (two workgroups of fewer than four trees per lane: 13%, most of it in batches below 1,000
// documents).
struct PlanTimes {
    int64_t places;
    double round_us, next_us, lone, reduce_us;
};
inline PlanTimes plan_times(const PlanFacts &f, Work work) {
    const bool full_pairs = f.pairs && f.full && work != Work::kTerminal;
    const bool vector = full_pairs && work == Work::kVector;
    PlanTimes t;
    t.places = f.pairs && !f.full && work != Work::kTerminal ? 2 * kNumCus : kNumCus;
    t.round_us = f.mean_steps * (vector ? 0.17 : 0.147);
    t.next_us = full_pairs ? 1.75 : 4.5;
    t.lone = vector ? 1.1 : 1.0;
    t.reduce_us = work == Work::kPositions ? 0.0 : 3.75;
    return t;
}

inline LaunchShape choose_launch(const PlanFacts &f, Work work, int64_t n_blocks) {
    constexpr double kFirst = 4.5;
    constexpr double kPerWorkgroup = 1e-5;
    constexpr double kPerSplit = 0.015; // of the second kernel
    const Tiling &tl = work == Work::kTerminal ? f.term : f.walk;
    const PlanTimes pt = plan_times(f, work);
    auto rounds_of = [&](int level, int tiles) {
        return double(tiles) * (tl.mean_rounds[level] + tl.switch_rounds) + (tl.max_rounds[level] - tl.mean_rounds[level]);
    };
    double best = 1e300;
    LaunchShape pick;
    auto consider = [&](int level, int64_t head, int sp) {
        const int nt = tl.tiles[level];
        const int64_t tail = n_blocks - head;
        const int64_t heads = (head + pt.places - 1) / pt.places, tails = (tail * sp + pt.places - 1) / pt.places;
        const double rounds = double(heads) * rounds_of(level, nt) + double(tails) * rounds_of(level, (nt + sp - 1) / sp);
        const double cost = kFirst + double(heads + tails - 1) * pt.next_us +
                            rounds * pt.round_us * (heads + tails == 1 ? pt.lone : 1.0) + (sp > 1 && pt.reduce_us > 0.0 ? pt.reduce_us + kPerSplit * sp : 0.0) +
                            kPerWorkgroup * double(head + tail * sp);
        if (cost < best - 1e-9) {
            best = cost;
            pick = LaunchShape{level, head, sp};
        }
    };
    for (int k = 0; k < tl.n_levels; ++k)
        for (int sp = 1; sp <= std::min(tl.tiles[k], 1024); ++sp)
            consider(k, 0, sp);
    for (int64_t head = n_blocks / pt.places * pt.places; head > 0 && head + 2 * pt.places > n_blocks; head -= pt.places)
        for (int sp = 2; head < n_blocks && sp <= std::min(tl.tiles[0], 64); ++sp)
            consider(0, head, sp);
    return pick;
}

} // namespace treeens
