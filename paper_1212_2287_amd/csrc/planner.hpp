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
    double us = 0.0; // the estimate it was chosen by
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
    Tiling walk, term; // term.tiles[0] == 0: no terminal packets
    UniformPlan uniform{};
    bool pairs = false, full = false; // two workgroups on a CU; four trees per lane
    bool compact = false;             // the walk takes compact packets
    double mean_steps = 0.0;
    int32_t n_trees = 0, n_cols = 0, n_outputs = 1, docs_per_block = 0;
};

constexpr double kTileRounds = 0.5;   // switching tiles (barriers, the copy into LDS), in walker rounds
constexpr double kPacketRounds = 0.1; // switching packets (no barrier), in walker rounds

inline PlanFacts plan_facts(const Packed &p) {
    PlanFacts f;
    f.pairs = p.plan.lds_bytes <= kLdsPerCu / 2;
    f.full = p.plan.interleave == 4;
    f.compact = p.cp_k > 0;
    f.mean_steps = p.mean_steps;
    f.n_trees = p.n_trees;
    f.n_cols = p.n_cols;
    f.n_outputs = p.n_outputs;
    f.docs_per_block = p.plan.docs_per_block;
    f.uniform = p.uniform;
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
// lie between: a lone workgroup takes a fifth longer than one of two (4 outputs, 4,096 trees of 16
// leaves, 256 blocks: 135 us whole, 121 in halves; 1,000 trees of 32 leaves: 45.2, 47.7).
// The other plans' steps and staging take longer than these figures say, both by about the same
// factor: 0.15 to 0.3 us a step and 5 to 18 us. Their ratio is what chooses. Over 542 batches of 40
// models, each measured in all its shapes, the shapes picked take 1 to 3% longer than the fastest on
// average (two workgroups of fewer than four trees per lane: 13%, most of it in batches below 1,000
// documents).
// Terminal packets are bound by latency and the L2s: workgroups whose shares are a packet short leave the
// others more of both, so a fifth of the average share counts (5,000 trees, 500 documents, 80
// packets: 27 shares of 2 or 3 58.9 us, 32 such shares 51.3).
struct PlanTimes {
    int64_t places;
    double round_us, next_us, lone, reduce_us, average;
};
inline PlanTimes plan_times(const PlanFacts &f, Work work) {
    const bool full_pairs = f.pairs && f.full && work != Work::kTerminal;
    const bool vector = full_pairs && work == Work::kVector;
    PlanTimes t;
    t.places = f.pairs && !f.full && work != Work::kTerminal ? 2 * kNumCus : kNumCus;
    t.round_us = f.mean_steps * (vector ? 0.17 : 0.147);
    t.next_us = full_pairs ? 1.75 : 4.5;
    t.lone = vector ? 1.2 : 1.0;
    t.reduce_us = work == Work::kPositions ? 0.0 : 3.75;
    t.average = work == Work::kTerminal ? 0.2 : 0.0;
    return t;
}

inline LaunchShape choose_launch(const PlanFacts &f, Work work, int64_t n_blocks) {
    constexpr double kFirst = 4.5;
    constexpr double kPerWorkgroup = 1e-5;
    constexpr double kPerSplit = 0.015; // of the second kernel
    const Tiling &tl = work == Work::kTerminal ? f.term : f.walk;
    const PlanTimes pt = plan_times(f, work);
    auto rounds_of = [&](int level, double tiles) {
        return tiles * (tl.mean_rounds[level] + tl.switch_rounds) + (tl.max_rounds[level] - tl.mean_rounds[level]);
    };
    double best = 1e300;
    LaunchShape pick;
    auto consider = [&](int level, int64_t head, int sp) {
        const int nt = tl.tiles[level];
        const int64_t tail = n_blocks - head;
        const int64_t heads = (head + pt.places - 1) / pt.places, tails = (tail * sp + pt.places - 1) / pt.places;
        const double share = (1.0 - pt.average) * double((nt + sp - 1) / sp) + pt.average * double(nt) / double(sp);
        const double rounds = double(heads) * rounds_of(level, nt) + double(tails) * rounds_of(level, share);
        const double cost = kFirst + double(heads + tails - 1) * pt.next_us +
                            rounds * pt.round_us * (heads + tails == 1 ? pt.lone : 1.0) + (sp > 1 && pt.reduce_us > 0.0 ? pt.reduce_us + kPerSplit * sp : 0.0) +
                            kPerWorkgroup * double(head + tail * sp);
        if (cost < best - 1e-9) {
            best = cost;
            pick = LaunchShape{level, head, sp, cost};
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

// Uniform launches: `head` document blocks walk all chunks of trees, the others are split over
// `splits` workgroups that leave partial sums.
inline LaunchShape uniform_shape(const UniformPlan &u, int64_t n_docs) {
    // one workgroup per CU; time in units of 16 chunks (one per wave)
    constexpr double kItem = 3.0; // staging and reduction of one workgroup (measured)
    constexpr double kReduce = 1.0;
    const int64_t n_blocks = (n_docs + u.docs_per_block - 1) / u.docs_per_block;
    const double all = double(u.n_chunks) / 16.0;
    LaunchShape best{0, n_blocks, 1};
    double least = 1e300;
    auto consider = [&](int64_t head, int splits) {
        const double share = double((u.n_chunks + splits - 1) / splits + 15) / 16.0; // fullest wave
        const double cost = double((head + kNumCus - 1) / kNumCus) * (all + kItem) +
                            double(((n_blocks - head) * splits + kNumCus - 1) / kNumCus) * (share + kItem) +
                            (splits > 1 ? kReduce : 0.0);
        if (cost < least - 1e-9) {
            least = cost;
            best = LaunchShape{0, head, splits, cost};
        }
    };
    consider(n_blocks, 1);
    const int most = int(std::max<int64_t>(1, std::min<int64_t>(u.n_chunks / 16, 256)));
    for (int s = 2; s <= most; ++s) {
        consider(0, s);
        if (n_blocks > kNumCus && n_blocks % kNumCus != 0)
            consider(n_blocks / kNumCus * kNumCus, s);
    }
    return best;
}

// Which kernels a call takes.

// Shallow models by uniform evaluation, or by the walk: models of at least 40 trees per column in calls
// of at least 1e8 walks (us by the walk against this; 136 columns, 3,000 trees, 400,000 documents 576,
// 624; 5,440 trees, 9,191 documents 42.7, 49.3), where the estimates of both agree with it. Both
// go in whole rounds of blocks, of 512 to 128 documents here and 64 or 32 there, and a batch
// that just fills rounds of one may leave the other's nearly empty (25 columns, 1,000 trees of depth 2:
// 100,000 documents 47.8, 42.7, 140,000 59.6, 73.8, 200,000 83.2, 76.9; 300 columns, 12,000 trees: 16,666
// documents 145, 184, 37,500 305, 294).
// The estimates: microseconds of uniform evaluation by depth and block, within 6% at the median
// of 305 measured batches; the walk's by the planner, scaled to complete trees.
inline double uniform_us(const PlanFacts &f, int64_t n_docs) {
    const int width = f.uniform.docs_per_block;
    const double unit = f.uniform.depth == 3 ? (width == 512 ? 9.6 : width == 256 ? 6.1 : 4.1)   // 16 chunks of trees
                                             : (width == 512 ? 10.4 : width == 256 ? 5.5 : 4.0);
    const double item = width == 128 ? 8.0 : 4.0;                     // a further workgroup's staging
    const double call = 9.5, coding = 3.5e-6 * double(n_docs) * f.n_cols, reduce = 4.0;
    const LaunchShape s = uniform_shape(f.uniform, n_docs);
    const int64_t n_blocks = (n_docs + width - 1) / width;
    const double heads = double((s.head + kNumCus - 1) / kNumCus);
    const double tails = double(((n_blocks - s.head) * s.splits + kNumCus - 1) / kNumCus);
    const double share = double((f.uniform.n_chunks + s.splits - 1) / s.splits + 15) / 16.0;
    return call + coding + unit * (heads * f.uniform.n_chunks / 16.0 + tails * share) + item * (heads + tails) +
           (s.splits > 1 ? reduce : 0.0);
}
inline bool uniform_pays(const PlanFacts &f, int64_t n_docs) {
    if (f.uniform.depth == 0 || f.n_trees < 40 * int64_t(f.n_cols) || double(n_docs) * f.n_trees < 1.0e8)
        return false;
    const int64_t n_blocks = (n_docs + f.docs_per_block - 1) / f.docs_per_block;
    const double scale = f.pairs ? (f.uniform.depth == 3 ? 0.8 : 0.65) : (f.uniform.depth == 3 ? 1.05 : 0.95);
    return uniform_us(f, n_docs) < 1.03 * (8.0 + scale * choose_launch(f, Work::kScores, n_blocks).us);
}

// Coded models by terminal packets, or by the walk. The packer makes them for coded models only: those
// code their documents anyway, where models of float documents would pay for it (1,000 trees of 64
// leaves, 700 features, 50,000 documents: 215 us on floats, 86 + 206 us on codes). Small batches of
// fewer than kTermTreesAlways trees keep the compact packets, whose walk ends without the terminals' two
// loads (us by compact packets against terminal ones: 1,024 trees of 256 leaves, 1,000 documents 42.3,
// 48.9, 2,000 49.6, 52.8, 6,700 76.9, 74.8; 300 trees of 200 leaves, 6,700 documents 51.0, 54.0, 10,000
// 56.4, 54.6; 2,000 trees of 150 leaves, 64 documents 24.7, 21.3, 1,000 35.5, 33.5). Trees beyond the
// compact packets (over 256 leaves) always take the terminal ones (1,000 trees of 512 leaves, 50,000
// documents: 912 us by 8-byte records, 524; 300 trees, 100 documents: 34.4, 32.2).
constexpr int32_t kTermTreesAlways = 1536;
inline bool term_pays(const PlanFacts &f, int64_t n_docs) {
    return f.term.tiles[0] > 0 &&
           (!f.compact || f.n_trees >= kTermTreesAlways || double(n_docs) * f.n_trees >= 2.5e6);
}

// Leaf ids: whether the walk stores them directly.
// It does where that is as fast (us stored directly against two kernels): outputs of at most
// kLeafDirectBytes (the L2s hold them until their lines are full; 1,000 trees of 32 leaves x 1,048
// documents 18.2, 18.5, x 2,621 38.5, 24.8; 256 x 8,192 18.3, 20.8, x 16,384 57.8, 27.5), twice that below
// 256 trees (128 x 24,576 21.3, 21.5), and rows of fewer than kLeafDirectTrees ids at any size (the
// L2s then hold the rows of all resident blocks; 100 x 31,457 22.1, 24.4), or four times as many in blocks
// of 8 documents, of which fewer are resident (300 trees x 41,943 312, 337; 400 x 31,457 201, 196; 1,000 x
// 12,582 135, 124).
constexpr int32_t kLeafDirectTrees = 128;
constexpr int64_t kLeafDirectBytes = int64_t(8) << 20;
constexpr int64_t kPositionBytes = int64_t(256) << 20;
inline bool leaves_direct(const PlanFacts &f, int64_t n_docs) {
    const int64_t most = f.n_trees < 2 * kLeafDirectTrees ? 2 * kLeafDirectBytes : kLeafDirectBytes;
    return f.n_trees < (f.docs_per_block == 8 ? 4 : 1) * kLeafDirectTrees || n_docs <= most / 4 / f.n_trees;
}

// Vector-valued scores: whether the walk stores each leaf's row once and sum_rows_kernel adds up to eight
// outputs per pass; else one walk per four (up to four outputs one walk does it all).
// Smaller batches do not pay for the second launch (us by walks against rows; 8 outputs, 1,000 trees of 32
// leaves: 2,000 documents 31.6, 38.7, 4,096 43.7, 44.0, 8,192 63.0, 53.2), nor do many trees of few
// documents (6 outputs, 4,000 trees of 8 leaves: 8,192 documents 118, 127, 12,000 151, 137; 64 outputs,
// 1,000 trees: 4,096 documents 342, 368, 6,000 488, 378).
// Nor do models whose chunks hold fewer than kRowDocs documents (64 of them fill a workgroup; 10,000
// trees of 8 leaves, 6 outputs, 50,000 documents in chunks of 6,500: 1,474, 2,194), and many trees of few
// steps, whose walks cost less than the gathers of the rows, beyond one chunk of documents (8 leaves,
// 50,000 documents: 4,000 trees, 6 outputs 483, 601, 16 outputs 1,011, 1,188; 3,000 trees, 6 outputs 362,
// 395, 12 outputs 544, 522; 2,000 trees 256, 248; 4,000 trees, 6 outputs, 16,384 documents 205, 162,
// 24,000 240, 246, 32,000 327, 282).
constexpr int64_t kRowDocs = 32768;
constexpr double kCheapSteps = 6.0; // 8 leaves: 5.3, 16: 6.8
inline bool rows_pay(const PlanFacts &f, int64_t n_docs) {
    if (f.n_outputs <= 4 || f.n_trees * kRowDocs * int64_t(sizeof(uint16_t)) > kPositionBytes)
        return false;
    const bool cheap_walks = f.pairs && f.full && f.mean_steps < kCheapSteps;
    if (cheap_walks && f.n_trees > (f.n_outputs <= 8 ? 2048 : 3072) && n_docs > kRowDocs)
        return false;
    return n_docs >= std::max<int64_t>(4096, (f.n_outputs <= 32 ? 4 : 5) * int64_t(f.n_trees));
}

} // namespace treeens
