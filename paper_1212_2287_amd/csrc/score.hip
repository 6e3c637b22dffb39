// score.hip -- the scoring kernels, compiled once per mode (TREE_ENS_SCORE_MODE).
//
// Work decomposition (one scoring launch per predict call):
//   * a workgroup owns a block of DL consecutive documents and stages their features into LDS
//     once, feature-major ([column][DL] values, column 0 = NaN, column f+1 = feature f), so a
//     lane's read of any feature of its own document is a conflict-free LDS access whatever
//     feature the lane's current node names;
//   * the trees are streamed through an LDS slot in tiles: self-describing images (header,
//     root copies, node records with absolute child links) copied global -> registers -> LDS,
//     the next one loading while the current one is walked;
//   * lanes are documents; each group of DL lanes (a "walker", a whole wave when DL = 64) walks
//     K trees of the tile at a time so that their LDS latencies overlap (the vectorisation
//     idea of Section 3, VPred, applied to trees instead of instances);
//   * each step is the branch-free predicated update of Section 3 (Pred) over explicit,
//     sibling-adjacent children: idx = left(idx) + (x[fid(idx)] >= theta(idx)); a wave stops
//     as soon as all its lanes sit on leaves (trees are unbalanced; most paths are short);
//   * leaf values are summed per lane in double precision, then reduced across walkers through
//     LDS in a fixed order and rounded once to float.
// Blocks of a last, partial round of workgroups (and every block of a small batch) are split
// over the tiles; the per-split partial sums are reduced by a second, tiny kernel in a fixed
// order, so results are deterministic.
// The same kernel has three more modes: leaf ids (the reached leaf of every (document, tree)),
// the feature-access trace (the set of distinct features each document's walks compare, the
// measure of Section 6 / Table 4: per-document bitmasks in LDS, set with an LDS atomic OR at
// every internal step), and vector-valued leaves (a leaf names a row of a leaf-vector table in
// global memory; a launch sums four of its components).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "score.hpp"

namespace treeens {

namespace {

// (w & mask) | b in one VALU op. The feature column offset is a multiple of DL * 4 and the lane
// offset is below DL * 4, so the OR is the sum the address needs.
__device__ __forceinline__ uint32_t and_or(uint32_t w, uint32_t mask, uint32_t b) {
    uint32_t r;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(w), "s"(mask), "v"(b));
    return r;
}
// One 8-byte node record from LDS, as one ds_read_b64, kept as one 64-bit value (threshold or
// leaf value in the low half, w in the high half) so that the pair stays in one register pair. A
// relaxed atomic load cannot be split: plain loads of the record get split by the compiler into
// two 4-byte reads (the threshold half sunk past the wave-wide leaf test), doubling the LDS
// reads per step.
__device__ __forceinline__ uint64_t read_record(const unsigned char *p) {
    return __hip_atomic_load(reinterpret_cast<const uint64_t *>(p), __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ uint32_t rec_thr(uint64_t r) { return uint32_t(r); }
__device__ __forceinline__ uint32_t rec_w(uint64_t r) { return uint32_t(r >> 32); }

// Child index of a narrow record plus the comparison bit, in two VALU ops: the compare writes
// VCC and an SDWA add-with-carry adds it to the high half-word of w. The s_nop covers the
// VALU-writes-VCC / VALU-reads-carry hazard (two wait states, as the compiler itself emits).
__device__ __forceinline__ uint32_t narrow_child(uint32_t w, float x, float thr) {
    uint32_t r;
    asm("v_cmp_ge_f32 vcc, %1, %2\n\t"
        "s_nop 1\n\t"
        "v_addc_co_u32_sdwa %0, vcc, %3, 0, vcc dst_sel:DWORD dst_unused:UNUSED_PAD "
        "src0_sel:WORD_1 src1_sel:DWORD"
        : "=v"(r)
        : "v"(x), "v"(thr), "v"(w)
        : "vcc");
    return r;
}

// The same for coded documents: unsigned compare of 16-bit codes.
[[maybe_unused]] __device__ __forceinline__ uint32_t narrow_child_coded(uint32_t w, uint32_t code, uint32_t q) {
    uint32_t r;
    asm("v_cmp_ge_u32 vcc, %1, %2\n\t"
        "s_nop 1\n\t"
        "v_addc_co_u32_sdwa %0, vcc, %3, 0, vcc dst_sel:DWORD dst_unused:UNUSED_PAD "
        "src0_sel:WORD_1 src1_sel:DWORD"
        : "=v"(r)
        : "v"(code), "v"(q), "v"(w)
        : "vcc");
    return r;
}

// Compact records: the side of the children pair {lo, hi} that a 4-byte record r sends a
// document to, whose staged value is x = code << 5 | 31: x >= the record's upper half is
// code >= threshold. Plain code: the compiler reads the upper half in place with an SDWA
// compare and places the compare-to-select wait states itself (filling them with the other
// trees' work).
[[maybe_unused]] __device__ __forceinline__ uint32_t compact_child(uint32_t x, uint32_t r, uint32_t lo, uint32_t hi) {
    return x >= (r >> 16) ? hi : lo;
}

template <int DL, int K, bool HALF, bool NARROW, bool CODED, int MODE, bool COMPACT>
// min waves per SIMD: 2 or 1 workgroups per CU (a feature trace holds a CU alone)
__global__ void __launch_bounds__(kThreads, HALF && MODE != kModeUsage ? 8 : 4)
score_kernel(const void *__restrict__ Xv, int64_t n_docs, int32_t n_features, int32_t n_cols,
             const uint2 *__restrict__ images, int32_t slot_recs,
             const uint32_t *__restrict__ tile_recs, int32_t n_tiles, int32_t head_blocks,
             int32_t tail_splits,
             int32_t xs_bytes, int32_t zero_rec, double *__restrict__ partials,
             float *__restrict__ scores, int32_t *__restrict__ leaf_ids,
             const int32_t *__restrict__ orig_id, const uint32_t *__restrict__ tree_node_off,
             const int32_t *__restrict__ tree_orig, int32_t n_trees,
             uint32_t *__restrict__ masks, int32_t mask_words, int32_t usage_off,
             const float4 *__restrict__ leaf_vec, int32_t vec_stride4, int32_t n_out,
             int32_t chunk, double out_scale, int32_t pk_recs, const uint2 *__restrict__ big,
             int32_t n_small, uint32_t big_off0, const uint32_t *__restrict__ cleaf,
             const int32_t *__restrict__ cleaf_id, uint16_t *__restrict__ leaf_pos) {
    // Static allocation: the LDS base is address 0, so feature and node addresses need no add.
    // HALF = half a CU's LDS, so that two workgroups share a CU. CODED = documents arrive as
    // 16-bit threshold codes (rows of n_features codes) instead of floats. Layout:
    //   [0, xs_bytes)            document tile, [(n_cols + 1) x DL] values
    //   [xs_bytes, zero_rec)     tile slot: the current tile image (header, then node records);
    //                            after the last tile, the cross-walker reduction (1,024 doubles,
    //                            4 x 1,024 with vector-valued leaves)
    //   zero_rec (8 bytes)       all-zero self-linked leaf of value 0, for idle walker slots
    //                            (walker packets of one-workgroup plans fill the LDS from
    //                            xs_bytes up to a zero record of their own, passed here)
    //   usage_off                usage modes: word j of document lane dl's feature bitmask at
    //                            [j * DL + dl] (32 feature ids a word); in the slot past the
    //                            largest tile image when it fits there (kModeUsageSlot, two
    //                            workgroups per CU as for scoring), else past the 80 KB half of
    //                            two-workgroup plans (kModeUsage: the launch holds a CU alone)
    constexpr bool LEAVES = MODE == kModeLeaves;
    constexpr bool USAGE = MODE == kModeUsage || MODE == kModeUsageSlot;
    constexpr bool VEC = MODE == kModeVector;
    constexpr bool ROWS = MODE == kModeRows;
    constexpr int kLds = HALF ? treeens::kLdsPerCu / 2 + (MODE == kModeUsage ? treeens::kUsageHalfBytes : 0)
                              : treeens::kLdsPerCu;
    __shared__ __align__(16) unsigned char lds[kLds];
    constexpr int kPre = HALF ? treeens::kPrefetchHalf : treeens::kPrefetchFull; // records per thread
    constexpr int kShift = NARROW ? 16 : treeens::kWideChildShift;
    uint2 *slot = reinterpret_cast<uint2 *>(lds + xs_bytes);
    const uint32_t *hdr = reinterpret_cast<const uint32_t *>(lds + xs_bytes);
    using Elem = std::conditional_t<CODED, uint16_t, float>;
    const Elem *X = reinterpret_cast<const Elem *>(Xv);
    Elem *xs = reinterpret_cast<Elem *>(lds);

    const int tid = threadIdx.x;
    const int nthr = kThreads;
    const int dl = tid & (DL - 1);
    // with 64-document blocks a walker is a whole wave: make that visible to the compiler so
    // the group loop is scalar
    const int walker = DL == 64 ? __builtin_amdgcn_readfirstlane(tid / DL) : tid / DL;
    const int n_walkers = nthr / DL;
    const uint32_t lane_off = uint32_t(dl) * uint32_t(sizeof(Elem));
    // a feature address is column * DL * sizeof(Elem) + lane offset (below DL * sizeof(Elem))
    constexpr int kColShift = __builtin_ctz(unsigned(DL * sizeof(Elem)));
    uint32_t *umask = reinterpret_cast<uint32_t *>(lds + usage_off);
    const int model_words = (n_cols + 31) / 32;

    const uint32_t col_mask =
        __builtin_amdgcn_readfirstlane(NARROW ? treeens::kNarrowColMask : treeens::kWideColMask);
    // column offsets below this are column 0 (NaN, or code 0), which only leaves name
    constexpr uint32_t kLeafCol = uint32_t(DL) * uint32_t(sizeof(Elem));
    // Workgroups [0, head_blocks) each walk all tiles for one document block; after them, each
    // remaining block is split over tail_splits workgroups that walk a contiguous share of the
    // tiles each and leave fp64 partial sums (the tail fills what would be a last, mostly idle
    // round of workgroups; small batches have no head at all).
    // After a head of whole rounds (a multiple of the XCD count), the splits of one tail block
    // are given workgroup indices of one residue mod kXcds: workgroups are dealt to the XCDs in
    // index order, so all splits of a block share one XCD's L2 and its document rows come from
    // HBM once. Indices past the last block (padding to whole XCD columns) exit at once.
    int64_t block = blockIdx.x;
    int split = 0, n_splits = 1;
    if (block >= head_blocks) {
        const int64_t t = block - head_blocks;
        if (head_blocks > 0) {
            const int64_t x = t % kXcds, r = t / kXcds;
            block = head_blocks + (r / tail_splits) * kXcds + x;
            split = int(r % tail_splits);
            if (block * DL >= n_docs)
                return;
        } else {
            block = head_blocks + t / tail_splits;
            split = int(t % tail_splits);
        }
        n_splits = tail_splits;
    }
    const int64_t doc0 = block * DL;
    const int t_lo = int((int64_t(n_tiles) * split) / n_splits);
    const int t_hi = int((int64_t(n_tiles) * (split + 1)) / n_splits);

    // Tile images are loaded into registers while the previous tile is walked, so the
    // global-memory latency of a tile load is hidden; the tile loop issues no scalar memory load
    // (those share a wait counter with LDS reads and would stall the walk).
    //  * HALF (two workgroups per CU, walk-bound): one tile in flight, its exact record count
    //    taken from the current tile's header.
    //  * full CU: two tiles in flight (one per register half), each a fixed window of
    //    kWin x kThreads records (the packer caps these tiles at that size and pads the images),
    //    loaded unconditionally so that the compiler counts the outstanding loads exactly.
    constexpr int kWin = treeens::kPrefetchFull / 2;
    constexpr int kDepth = HALF ? 1 : kPrefetchDepth; // tiles in flight
    constexpr int kPreA = kPre; // shared tiles of two-workgroup plans, or walker packets
    uint2 pa[kPreA], win[kDepth][HALF ? 1 : kWin];
    int cur_recs = 0;
    const int chunks = (slot_recs + kThreads - 1) / kThreads;
    auto fetch = [&](int ti, int n_rec) {
        const uint2 *src = images + int64_t(ti) * slot_recs;
#pragma unroll
        for (int j = 0; j < kPre; ++j) {
            const int i = tid + j * kThreads;
            if (i < n_rec)
                pa[j] = src[i];
        }
    };
    auto fetch_window = [&](uint2 (&dst)[kWin], int ti) {
        // unconditional: past the last tile it reloads that tile (exact wait counts)
        const uint2 *src = images + int64_t(min(ti, t_hi - 1)) * slot_recs + tid;
#pragma unroll
        for (int j = 0; j < kWin; ++j)
            dst[j] = src[(j < chunks ? j : 0) * kThreads];
    };
    // Walker packets (pk_recs > 0, plans of 64- or 32-document blocks): wave v's packet q is
    // images[(v * n_tiles + q) * pk_recs, ...), one part of pk_recs * DL / 64 records for each
    // of its walkers; each lane loads pk_recs / 64 records of it.
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int pk_lane = pk_recs / 64;
    // The loads are raw buffer loads: the packet's offset in a scalar register, each lane's
    // record offset in a vector register and the record's position in the instruction's
    // immediate, so no address arithmetic runs per packet (the packer keeps the packets below
    // 2 GiB).
    const __amdgpu_buffer_rsrc_t pk_rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint2 *>(images), 0, 0x7fffffff, 0x00020000);
    const int pk_lane_off = lane * 8;
    auto fetch_packet = [&](int q) {
        const int soff = (wave * n_tiles + q) * pk_recs * 8;
#pragma unroll
        for (int j = 0; j < kPre; ++j) {
            if (j < pk_lane) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b64(pk_rsrc, pk_lane_off + j * 512, soff, 0);
                pa[j] = make_uint2(v[0], v[1]);
            }
        }
    };
    // Compact packets: kCompactPacketBytes per packet, one 8-byte row of 64 lanes per 512 bytes,
    // read with raw buffer loads as above.
    constexpr int kCpRows = treeens::kCompactPacketBytes / 512;
    auto fetch_compact = [&](int q) {
        const int soff = (wave * n_tiles + q) * treeens::kCompactPacketBytes;
#pragma unroll
        for (int j = 0; j < kCpRows; ++j) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b64(pk_rsrc, pk_lane_off + j * 512, soff, 0);
            pa[j] = make_uint2(v[0], v[1]);
        }
    };
    if constexpr (COMPACT) {
        if (t_lo < t_hi)
            fetch_compact(t_lo);
    } else if constexpr (HALF) {
        if (pk_recs > 0) {
            if (t_lo < t_hi)
                fetch_packet(t_lo);
        } else {
            cur_recs = t_lo < t_hi ? int(tile_recs[t_lo]) : 0;
            if (t_lo < t_hi)
                fetch(t_lo, cur_recs);
        }
    } else {
        if (pk_recs > 0) {
            if (t_lo < t_hi)
                fetch_packet(t_lo);
        } else if (t_lo < t_hi) {
#pragma unroll
            for (int d = 0; d < kDepth; ++d)
                fetch_window(win[d], t_lo + d);
        }
    }

    if constexpr (USAGE) {
        for (int i = tid; i < model_words * DL; i += kThreads)
            umask[i] = 0u;
    }
    // Stage the document tile: lane = document, so each LDS write is conflict-free (bank =
    // lane). The workgroup size is a multiple of DL, so a thread's document (and row) is fixed
    // and it takes every (kThreads / DL)-th group of columns. When rows are 16-byte aligned a
    // lane reads 16 bytes of its row at a time (4 floats or 8 codes: a quarter or an eighth of
    // the strided row reads), else one value. Loads are unconditional (clamped to the row) so
    // that a pass's loads are in flight together before any is written.
    {
        constexpr int kColStep = kThreads / DL;
        constexpr int kUnroll = 8;
        constexpr int kVec = 16 / int(sizeof(Elem)); // values per 16-byte load
        const int64_t doc = doc0 + dl;
        const bool live = doc < n_docs;
        const Elem *row = X + (live ? doc : n_docs - 1) * int64_t(n_features);
        // (compact packets: code 0 staged as 0 << 5 | 31)
        const Elem leaf_col = COMPACT ? Elem(31) : CODED ? Elem(0) : Elem(__builtin_nanf(""));
        if (tid < DL)
            xs[dl] = leaf_col;
        const bool vec = (n_features % kVec) == 0 && (reinterpret_cast<uintptr_t>(X) & 15u) == 0;
        if (vec) {
            const uint4 *row4 = reinterpret_cast<const uint4 *>(row);
            const int n_groups = (n_cols + kVec - 1) / kVec; // within the row: n_features % kVec == 0
            const int last = n_groups > 0 ? n_groups - 1 : 0;
            constexpr int kVecUnroll = 4;
            for (int q0 = tid / DL; q0 < n_groups; q0 += kColStep * kVecUnroll) {
                uint4 v[kVecUnroll];
#pragma unroll
                for (int u = 0; u < kVecUnroll; ++u)
                    v[u] = row4[min(q0 + u * kColStep, last)];
#pragma unroll
                for (int u = 0; u < kVecUnroll; ++u) {
                    const int q = q0 + u * kColStep;
                    if (q < n_groups) {
                        const Elem *e = reinterpret_cast<const Elem *>(&v[u]);
#pragma unroll
                        for (int k = 0; k < kVec; ++k) {
                            const int c = q * kVec + k + 1; // tile column of feature q * kVec + k
                            if (c <= n_cols)
                                xs[c * DL + dl] = live ? e[k] : Elem(0);
                        }
                    }
                }
            }
        } else {
            const int last = n_cols > 0 ? n_cols - 1 : 0;
            for (int c0 = tid / DL + 1; c0 <= n_cols; c0 += kColStep * kUnroll) {
                Elem v[kUnroll];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u)
                    v[u] = row[min(c0 + u * kColStep - 1, last)];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    const int c = c0 + u * kColStep;
                    if (c <= n_cols)
                        xs[c * DL + dl] = live ? v[u] : Elem(0);
                }
            }
        }
    }
    if (!COMPACT && tid == 0) {
        // value 0 (as -0.0 for codes, whose leaves never hold zero bits; the all-zero row 0 of
        // the leaf-vector table for vector-valued leaves), column 0, self link
        const uint32_t thr = VEC || ROWS ? 1u : CODED ? 0x80000000u : 0u;
        *reinterpret_cast<uint2 *>(lds + zero_rec) = make_uint2(thr, (uint32_t(zero_rec) / 8u) << kShift);
    }

    double acc = 0.0;
    double accv[kVecPerLaunch] = {0.0, 0.0, 0.0, 0.0};
    // Walk one group of K trees whose K root copies are the records at rc. tree_of(i) gives the
    // packed index of the tree in slot i (-1: an idle slot) and, for leaf ids, the LDS record
    // index of that tree's first record.
    auto walk_group = [&](const unsigned char *rc, auto complete_tag, int complete_depth, auto &&tree_of) {
        constexpr bool kComplete = decltype(complete_tag)::value;
        // the K root records (broadcast reads)
        uint64_t nd[K];
        if constexpr (K % 2 == 0) {
            // two roots per 16-byte read (a group's roots start 16-byte aligned when K is even)
#pragma unroll
            for (int i = 0; i < K; i += 2) {
                const uint4 r2 = *reinterpret_cast<const uint4 *>(rc + 8 * i);
                nd[i] = uint64_t(r2.x) | uint64_t(r2.y) << 32;
                nd[i + 1] = uint64_t(r2.z) | uint64_t(r2.w) << 32;
            }
        } else {
#pragma unroll
            for (int i = 0; i < K; ++i)
                nd[i] = read_record(rc + 8 * i);
        }
        // One predicated step: feature addresses fa from the records, read the features
        // xv, compare, child link + bit (the right child follows the left one), read
        // that record.
        uint32_t fa[K];
        std::conditional_t<CODED, uint32_t, float> xv[K];
        auto read_features = [&]() {
#pragma unroll
            for (int i = 0; i < K; ++i) {
                fa[i] = and_or(rec_w(nd[i]), col_mask, lane_off);
                if constexpr (CODED)
                    xv[i] = *reinterpret_cast<const uint16_t *>(lds + fa[i]);
                else
                    xv[i] = *reinterpret_cast<const float *>(lds + fa[i]);
                if constexpr (USAGE) {
                    // column c > 0 holds feature c - 1; column 0 is a leaf's (no
                    // comparison, nothing recorded)
                    const uint32_t col = fa[i] >> kColShift;
                    if (col > 0u)
                        atomicOr(&umask[((col - 1u) >> 5) * DL + dl], 1u << ((col - 1u) & 31u));
                }
            }
        };
        uint32_t addr[K]; // byte addresses of the records read by the last step
        auto descend = [&]() {
#pragma unroll
            for (int i = 0; i < K; ++i) {
                uint32_t child;
                const uint32_t w = rec_w(nd[i]), thr = rec_thr(nd[i]);
                if constexpr (CODED) {
                    if constexpr (NARROW)
                        child = narrow_child_coded(w, xv[i], thr);
                    else
                        child = (w >> kShift) + (xv[i] >= thr ? 1u : 0u);
                } else {
                    if constexpr (NARROW)
                        child = narrow_child(w, xv[i], __uint_as_float(thr));
                    else
                        child = (w >> kShift) + (xv[i] >= __uint_as_float(thr) ? 1u : 0u);
                }
                addr[i] = child * 8u;
            }
#pragma unroll
            for (int i = 0; i < K; ++i)
                nd[i] = read_record(lds + addr[i]);
        };
        if constexpr (kComplete) {
            // every path has the same length: no leaf test needed
            for (int s = 0; s < complete_depth; ++s) {
                read_features();
                descend();
            }
        } else {
            // Every lane steps until all lanes of the wave sit on leaves (a leaf's
            // feature address is the NaN column, below kLeafCol); the record that shows
            // a lane is at a leaf holds the leaf's value. Every path of a validated tree
            // reaches a leaf and leaves link to themselves, so the exit is always taken.
            // The next feature reads are issued before the test, so the test overlaps
            // their latency (after the last step they read the NaN column: harmless).
            auto any_internal = [&]() {
                bool internal = false;
#pragma unroll
                for (int i = 0; i < K; ++i)
                    internal |= fa[i] >= kLeafCol;
                return __builtin_amdgcn_ballot_w64(internal) != 0;
            };
            // Trees sit in the packed order longest expected lockstep walk first, so the
            // group's first tree usually ends last: step while its lanes are not all on
            // leaves (one compare per step), then while any of the K trees is not (the full
            // test, rarely true by then). The first step is taken untested: a group whose K
            // roots are all leaves (single-leaf trees, idle slots) is rare, and a leaf absorbs
            // the extra step.
            auto lead_internal = [&]() {
                return __builtin_amdgcn_ballot_w64(fa[0] >= kLeafCol) != 0;
            };
            read_features();
            for (;;) {
                descend();
                read_features();
                if (!lead_internal() && (K == 1 || !any_internal()))
                    break;
            }
            // The exit path "uses" the last feature reads, so the compiler cannot sink
            // them below the test (where they would serialise with it again).
#pragma unroll
            for (int i = 0; i < K; ++i)
                asm volatile("" ::"v"(xv[i]));
        }
        if constexpr (LEAVES) {
            const int64_t doc = doc0 + dl;
#pragma unroll
            for (int i = 0; i < K; ++i) {
                // a leaf's link is its own LDS record index; minus that of its tree's
                // first record, it is the leaf's position in the tree
                const int2 tr = tree_of(i);
                const int gt = tr.x;
                // complete trees: the leaf's record index is the address the last step
                // read (their leaf records carry no link); else the leaf's own link
                const uint32_t rec = kComplete ? (complete_depth > 0 ? addr[i] / 8u : uint32_t(tr.y))
                                               : rec_w(nd[i]) >> kShift;
                const uint32_t self = rec - uint32_t(tr.y);
                if (leaf_pos) {
                    if (gt >= 0)
                        leaf_pos[(block * n_trees + gt) * DL + dl] = uint16_t(self);
                } else if (gt >= 0 && doc < n_docs) {
                    leaf_ids[doc * n_trees + tree_orig[gt]] = orig_id[tree_node_off[gt] + self];
                }
            }
        } else if constexpr (ROWS) {
            // a leaf's threshold slot holds its table row + 1
#pragma unroll
            for (int i = 0; i < K; ++i) {
                const int gt = tree_of(i).x;
                if (gt >= 0)
                    leaf_pos[(block * n_trees + gt) * DL + dl] = uint16_t(rec_thr(nd[i]) - 1u);
            }
        } else if constexpr (VEC) {
            // a leaf's threshold slot holds its table row + 1 (idle slots: row 0, zeros);
            // each component added to its double accumulator in tree order
#pragma unroll
            for (int i = 0; i < K; ++i) {
                const float4 v = leaf_vec[int64_t(rec_thr(nd[i]) - 1u) * vec_stride4 + chunk];
                accv[0] += double(v.x);
                accv[1] += double(v.y);
                accv[2] += double(v.z);
                accv[3] += double(v.w);
            }
        } else if constexpr (!USAGE) {
            // the K leaf values, each added to the double accumulator in tree order (a
            // float sum of the group first can miss the tolerance when a score cancels
            // near zero); idle slots hold the zero record. Complete trees' leaf records hold
            // the value as a double (tiles and packets with an idle slot are never complete).
#pragma unroll
            for (int i = 0; i < K; ++i) {
                if constexpr (kComplete)
                    acc += __longlong_as_double(static_cast<long long>(nd[i]));
                else
                    acc += double(__uint_as_float(rec_thr(nd[i])));
            }
        }
    };
    // Walk the tile image in the LDS slot: walker w takes groups w, w + n_walkers, ... of K
    // consecutive trees (the packer sizes tiles to a multiple of n_walkers * K trees where it
    // can, and pads the header's root copies to a multiple of K with the zero record).
    auto walk_tile = [&]() {
        const uint4 h = *reinterpret_cast<const uint4 *>(hdr);
        const int ntr = __builtin_amdgcn_readfirstlane(int(h.x));
        const int complete_depth = __builtin_amdgcn_readfirstlane(int(h.y));
        const int tree_begin = __builtin_amdgcn_readfirstlane(int(h.z));
        const int n_groups = (ntr + K - 1) / K;
        // records of the tile's trees start after the fixed header words and the root copies
        const uint32_t rec0 = uint32_t(xs_bytes) / 8u + uint32_t(treeens::kHeaderFixedWords / 2 + n_groups * K);
        auto walk_groups = [&](auto complete_tag) {
            for (int g = walker; g < n_groups; g += n_walkers) {
                const unsigned char *rc = lds + xs_bytes + 8 * (treeens::kHeaderFixedWords / 2 + g * K);
                auto tree_of = [&](int i) {
                    const int t = g * K + i;
                    return t < ntr ? make_int2(tree_begin + t,
                                               int(rec0 + tree_node_off[tree_begin + t] - tree_node_off[tree_begin]))
                                   : make_int2(-1, 0);
                };
                walk_group(rc, complete_tag, complete_depth, tree_of);
            }
        };
        // the branch on the tile's complete depth outside the group loop, so that each loop
        // keeps its records in the registers it reads them into
        if (complete_depth >= 0)
            walk_groups(std::true_type{});
        else
            walk_groups(std::false_type{});
    };
    // Walk one of this walker's packets in its sub-slot, which starts at LDS record base: its
    // groups are first_group, first_group + n_walkers, ...
    auto walk_packet = [&](uint32_t base) {
        const uint2 h0 = *reinterpret_cast<const uint2 *>(lds + 8 * base);
        const uint2 h1 = *reinterpret_cast<const uint2 *>(lds + 8 * (base + 1));
        const int ng = __builtin_amdgcn_readfirstlane(int(h0.x));
        const int complete_depth = __builtin_amdgcn_readfirstlane(int(h0.y));
        // group count and complete depth are common to the walkers of a wave; first groups not
        const int first_group = DL == 64 ? __builtin_amdgcn_readfirstlane(int(h1.x)) : int(h1.x);
        const uint16_t *first_rec =
            reinterpret_cast<const uint16_t *>(lds + 8 * (base + treeens::kPacketHeaderRecs + ng * K));
        auto walk_groups = [&](auto complete_tag) {
            for (int j = 0; j < ng; ++j) {
                const unsigned char *rc = lds + 8 * (base + treeens::kPacketHeaderRecs + j * K);
                auto tree_of = [&](int i) {
                    const int gt = (first_group + j * n_walkers) * K + i;
                    return gt < n_small ? make_int2(gt, int(first_rec[j * K + i])) : make_int2(-1, 0);
                };
                walk_group(rc, complete_tag, complete_depth, tree_of);
            }
        };
        // as in walk_tile, the branch on the complete depth outside the group loop
        if (complete_depth >= 0)
            walk_groups(std::true_type{});
        else
            walk_groups(std::false_type{});
    };
    // Each walker streams its own packets through its own sub-slot: no barrier between packets,
    // so a walker never waits for the slowest one of a tile.
    auto walk_packets = [&]() {
        const uint32_t my_base = uint32_t(xs_bytes) / 8u + uint32_t(wave * pk_recs);
        uint2 *my = reinterpret_cast<uint2 *>(lds) + my_base;
        // this walker's part of the wave's sub-slot
        const uint32_t part_base = my_base + uint32_t(DL == 64 ? 0 : (lane / DL) * (pk_recs * DL / 64));
        __syncthreads(); // the document tile and the zero record are written
        for (int q = t_lo; q < t_hi; ++q) {
            // this packet's records (and, before the first, the document rows) have landed
            __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
#pragma unroll
            for (int j = 0; j < kPre; ++j)
                if (j < pk_lane)
                    my[lane + j * 64] = pa[j];
            // the wave's own writes complete before it reads the packet back
            __builtin_amdgcn_s_waitcnt(kWaitLgkmcnt0);
            if (q + 1 < t_hi)
                fetch_packet(q + 1);
            walk_packet(part_base);
        }
    };
    // Compact packets (4-byte records): wave v owns K windows of kCompactWindowBytes / K bytes past
    // the document tile; the packet's header row stays in registers. A step reads the lane's staged value and
    // the current record's whole children pair together (one dependent LDS round trip) and keeps
    // the side the comparison picks. Leaves hold no value: the leaf's position in its window
    // locates its payload (value bits, leaf-vector row + 1 or input node id) in arrays shaped
    // like the packets in device memory. Scores add each group's payloads after the next group
    // is walked, so their loads have a whole walk to land (the sum keeps tree order).
    auto walk_compact = [&]() {
        if constexpr (COMPACT) {
            constexpr uint32_t kCpWin = treeens::kCompactWindowBytes / K;
            static_assert(K == treeens::kCompactTrees && kCpWin == 2048, "compact windows of 2 KiB");
            const uint32_t cw = (uint32_t(xs_bytes) + 2047u) & ~2047u;
            const uint32_t my_win = cw + uint32_t(wave) * treeens::kCompactWindowBytes;
            const __amdgpu_buffer_rsrc_t leaf_rsrc =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(cleaf), 0, 0x7fffffff, 0x00020000);
            const __amdgpu_buffer_rsrc_t id_rsrc =
                __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t *>(cleaf_id), 0, 0x7fffffff, 0x00020000);
            // the column field moved to a feature address (column * DL * 2 bytes), the pair offset
            const uint32_t col_sel = __builtin_amdgcn_readfirstlane(0x1FF80u);
            const uint32_t pair_sel = __builtin_amdgcn_readfirstlane(0x7F8u);
            // window bases (aligned to the window size: OR adds the pair offset), held in vector
            // registers for the whole walk (opaque to the compiler, which would otherwise copy
            // one from a scalar register at every step)
            uint32_t tb[K];
#pragma unroll
            for (int i = 0; i < K; ++i)
                asm volatile("v_mov_b32 %0, %1" : "=v"(tb[i]) : "s"(my_win + uint32_t(i) * kCpWin));
            uint32_t pend[K]; // leaf payloads of the last group walked (scores)
#pragma unroll
            for (int i = 0; i < K; ++i)
                pend[i] = 0u;
            if constexpr (MODE == kModeScore) {
                // Loads of the zero pairs' payloads (0.0) before the first packet, so that every
                // packet's copy finds K payload loads issued after its rows, as on later packets.
                if (t_lo < t_hi) {
                    const int soff = (wave * n_tiles + t_lo) * treeens::kCompactPacketBytes;
#pragma unroll
                    for (int i = 0; i < K; ++i)
                        pend[i] = __builtin_amdgcn_raw_buffer_load_b32(leaf_rsrc, i * kCpWin + kCpWin - 8, soff, 0);
                }
            }
            __syncthreads(); // the document tile is written
            for (int q = t_lo; q < t_hi; ++q) {
                const int soff = (wave * n_tiles + q) * treeens::kCompactPacketBytes;
                // this packet's rows have landed (the last group's payload loads may not have)
                __builtin_amdgcn_s_waitcnt(MODE == kModeScore ? kWaitVmcnt0 | K : kWaitVmcnt0);
#pragma unroll
                for (int j = 0; j < kCpRows - 1; ++j)
                    *reinterpret_cast<uint2 *>(lds + my_win + uint32_t(j) * 512u + uint32_t(pk_lane_off)) = pa[j];
                // The header row stays in registers (lane l holds header words 2l and 2l + 1):
                // its fields and the groups' roots are read from there with v_readlane.
                const uint2 hrow = pa[kCpRows - 1];
                // the wave's own writes complete before it reads the packet back
                __builtin_amdgcn_s_waitcnt(kWaitLgkmcnt0);
                // the next packet (the last one again after the last: the loads stay
                // unconditional, so the compiler counts them exactly when it waits for payloads)
                fetch_compact(min(q + 1, t_hi - 1));
                const int ng = __builtin_amdgcn_readlane(int(hrow.x), 0);
                const int complete_depth = __builtin_amdgcn_readlane(int(hrow.y), 0);
                const int first_group = __builtin_amdgcn_readlane(int(hrow.x), 1);
                auto walk_groups = [&](auto complete_tag) {
                    constexpr bool kComplete = decltype(complete_tag)::value;
                    for (int j = 0; j < ng; ++j) {
                        // group j's roots: header words 4 + 2j and 5 + 2j, lane 2 + j
                        static_assert(treeens::kCompactHeaderWords == 4 && K == 2, "root lane");
                        uint32_t r[K];
                        r[0] = uint32_t(__builtin_amdgcn_readlane(int(hrow.x), 2 + j));
                        r[1] = uint32_t(__builtin_amdgcn_readlane(int(hrow.y), 2 + j));
                        uint32_t fa[K], xv[K], lo[K], hi[K];
                        auto issue = [&]() {
#pragma unroll
                            for (int i = 0; i < K; ++i) {
                                fa[i] = and_or(r[i] >> 4, col_sel, lane_off);
                                const uint32_t pa_i = and_or(r[i], pair_sel, tb[i]);
                                xv[i] = *reinterpret_cast<const uint16_t *>(lds + fa[i]);
                                const uint64_t pr = read_record(lds + pa_i);
                                lo[i] = uint32_t(pr);
                                hi[i] = uint32_t(pr >> 32);
                            }
                        };
                        auto select = [&]() {
#pragma unroll
                            for (int i = 0; i < K; ++i)
                                r[i] = compact_child(xv[i], r[i], lo[i], hi[i]);
                        };
                        if constexpr (kComplete) {
                            for (int s = 0; s < complete_depth; ++s) {
                                issue();
                                select();
                            }
                        } else {
                            // as in walk_group: the first step untested, then step until the lead
                            // tree's lanes, then all K trees' lanes, sit on leaves (column 0); the
                            // next reads are issued before the test
                            issue();
                            for (;;) {
                                select();
                                issue();
                                if (__builtin_amdgcn_ballot_w64(fa[0] >= kLeafCol) == 0) {
                                    bool internal = false;
#pragma unroll
                                    for (int i = 1; i < K; ++i)
                                        internal |= fa[i] >= kLeafCol;
                                    if (__builtin_amdgcn_ballot_w64(internal) == 0)
                                        break;
                                }
                            }
#pragma unroll
                            for (int i = 0; i < K; ++i)
                                asm volatile("" ::"v"(xv[i]), "v"(lo[i]), "v"(hi[i]));
                        }
                        // byte offset of each leaf's payload in the packet
                        uint32_t voff[K];
#pragma unroll
                        for (int i = 0; i < K; ++i)
                            voff[i] = (r[i] & 0x7FCu) + uint32_t(i) * kCpWin;
                        if constexpr (MODE == kModeScore) {
#pragma unroll
                            for (int i = 0; i < K; ++i)
                                acc += double(__uint_as_float(pend[i]));
#pragma unroll
                            for (int i = 0; i < K; ++i)
                                pend[i] = __builtin_amdgcn_raw_buffer_load_b32(leaf_rsrc, voff[i], soff, 0);
                        } else if constexpr (LEAVES) {
                            const int64_t doc = doc0 + dl;
#pragma unroll
                            for (int i = 0; i < K; ++i) {
                                const int gt = (first_group + j * treeens::kPacketWalkers) * K + i;
                                if (gt >= n_trees)
                                    continue; // an idle slot
                                const int id = __builtin_amdgcn_raw_buffer_load_b32(id_rsrc, voff[i], soff, 0);
                                if (leaf_pos)
                                    leaf_pos[(block * n_trees + gt) * DL + dl] = uint16_t(id);
                                else if (doc < n_docs)
                                    leaf_ids[doc * n_trees + tree_orig[gt]] = id;
                            }
                        } else if constexpr (ROWS) {
#pragma unroll
                            for (int i = 0; i < K; ++i) {
                                const int gt = (first_group + j * treeens::kPacketWalkers) * K + i;
                                const uint32_t row = __builtin_amdgcn_raw_buffer_load_b32(leaf_rsrc, voff[i], soff, 0);
                                if (gt < n_trees)
                                    leaf_pos[(block * n_trees + gt) * DL + dl] = uint16_t(row - 1u);
                            }
                        } else if constexpr (VEC) {
#pragma unroll
                            for (int i = 0; i < K; ++i) {
                                const uint32_t row = __builtin_amdgcn_raw_buffer_load_b32(leaf_rsrc, voff[i], soff, 0);
                                const float4 v = leaf_vec[int64_t(row - 1u) * vec_stride4 + chunk];
                                accv[0] += double(v.x);
                                accv[1] += double(v.y);
                                accv[2] += double(v.z);
                                accv[3] += double(v.w);
                            }
                        }
                    }
                };
                if (complete_depth >= 0)
                    walk_groups(std::true_type{});
                else
                    walk_groups(std::false_type{});
            }
            if constexpr (MODE == kModeScore) {
#pragma unroll
                for (int i = 0; i < K; ++i)
                    acc += double(__uint_as_float(pend[i]));
            }
        }
    };
    if constexpr (COMPACT) {
        walk_compact();
    } else if constexpr (HALF) {
        if (pk_recs > 0)
            walk_packets();
        else
        for (int ti = t_lo; ti < t_hi; ++ti) {
            __syncthreads(); // the previous tile is fully walked (and the document tile written)
            // All outstanding global loads (this tile's records, and the document rows before
            // the first tile) land here, unconditionally: otherwise the compiler cannot prove
            // them complete on every path and waits for them again inside the walk.
            __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
#pragma unroll
            for (int j = 0; j < kPre; ++j) {
                const int i = tid + j * kThreads;
                if (i < cur_recs)
                    slot[i] = pa[j];
            }
            __syncthreads();
            cur_recs = __builtin_amdgcn_readfirstlane(int(hdr[3])); // the next tile's size
            if (ti + 1 < t_hi)
                fetch(ti + 1, cur_recs);
            walk_tile();
        }
    } else if (pk_recs > 0) {
        walk_packets();
    } else {
        // the document rows (loaded after the first two tiles) land before the first barrier
        __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
        // windows are written as whole 1,024-record chunks: the packer sizes the slot of these
        // plans to whole chunks, so the zero record and the trace's bitmasks after it are safe
        auto write_window = [&](const uint2 (&src)[kWin]) {
#pragma unroll
            for (int j = 0; j < kWin; ++j)
                if (j < chunks)
                    slot[tid + j * kThreads] = src[j];
        };
        for (int ti = t_lo; ti < t_hi; ti += kDepth) {
#pragma unroll
            for (int d = 0; d < kDepth; ++d) {
                __syncthreads(); // the previous tile is fully walked (and the document tile written)
                write_window(win[d]);
                __syncthreads();
                fetch_window(win[d], ti + d + kDepth);
                if (d == 0 || ti + d < t_hi)
                    walk_tile();
            }
        }
    }
    // Big trees (too large for a tile; packed after the tiled ones): walked from device memory,
    // one tree per walker at a time, the records staying in L2. A record is {thr, w} with
    // w = (tree-relative left child << 16) | column index; the features come from the LDS
    // document tile as for every other tree, and leaves absorb further steps (column 0). Big
    // tree b goes to split b % n_splits and, within it, to walker (b / n_splits) % n_walkers.
    if (!COMPACT && n_small < n_trees) {
        __syncthreads(); // the document tile is written (no tile may have been walked)
        const int n_big = n_trees - n_small;
        for (int b = split + n_splits * walker; b < n_big; b += n_splits * n_walkers) {
            const int gt = n_small + b;
            const uint2 *tr = big + (tree_node_off[gt] - big_off0);
            uint2 r = tr[0];
            for (;;) {
                const uint32_t fa = ((r.y & treeens::kBigColMask) << kColShift) | lane_off;
                const Elem x = *reinterpret_cast<const Elem *>(lds + fa);
                if constexpr (USAGE) {
                    const uint32_t col = r.y & treeens::kBigColMask;
                    if (col > 0u)
                        atomicOr(&umask[((col - 1u) >> 5) * DL + dl], 1u << ((col - 1u) & 31u));
                }
                if (__builtin_amdgcn_ballot_w64(fa >= kLeafCol) == 0)
                    break;
                bool right;
                if constexpr (CODED)
                    right = uint32_t(x) >= r.x;
                else
                    right = x >= __uint_as_float(r.x);
                r = tr[(r.y >> treeens::kBigLinkShift) + (right ? 1u : 0u)];
            }
            if constexpr (LEAVES) {
                const int64_t doc = doc0 + dl;
                const uint32_t self = r.y >> treeens::kBigLinkShift;
                if (leaf_pos)
                    leaf_pos[(block * n_trees + gt) * DL + dl] = uint16_t(self);
                else if (doc < n_docs)
                    leaf_ids[doc * n_trees + tree_orig[gt]] = orig_id[tree_node_off[gt] + self];
            } else if constexpr (ROWS) {
                leaf_pos[(block * n_trees + gt) * DL + dl] = uint16_t(r.x - 1u);
            } else if constexpr (VEC) {
                const float4 v = leaf_vec[int64_t(r.x - 1u) * vec_stride4 + chunk];
                accv[0] += double(v.x);
                accv[1] += double(v.y);
                accv[2] += double(v.z);
                accv[3] += double(v.w);
            } else if constexpr (!USAGE) {
                acc += double(__uint_as_float(r.x));
            }
        }
    }
    if constexpr (USAGE) {
        __syncthreads();
        // rows of mask_words words (>= model_words; the words past the model's are zero)
        const int64_t n_here = min<int64_t>(DL, n_docs - doc0);
        if (masks) {
            for (int e = tid; e < n_here * mask_words; e += kThreads) {
                const int d = e / mask_words, j = e - d * mask_words;
                masks[(doc0 + d) * mask_words + j] = j < model_words ? umask[j * DL + d] : 0u;
            }
        }
        if (walker == 0 && dl < n_here) {
            int count = 0;
            for (int j = 0; j < model_words; ++j)
                count += __popc(umask[j * DL + dl]);
            leaf_ids[doc0 + dl] = count;
        }
    }
    if constexpr (VEC) {
        __syncthreads();
        double *red = reinterpret_cast<double *>(lds + xs_bytes); // 4 x 1,024 doubles (32 KiB)
#pragma unroll
        for (int c = 0; c < kVecPerLaunch; ++c)
            red[(c * n_walkers + walker) * DL + dl] = accv[c];
        __syncthreads();
        if (walker == 0) {
            const int64_t doc = doc0 + dl;
            for (int c = 0; c < kVecPerLaunch; ++c) {
                double sum = 0.0;
                for (int w = 0; w < n_walkers; ++w)
                    sum += red[(c * n_walkers + w) * DL + dl];
                const int oc = kVecPerLaunch * chunk + c;
                if (doc < n_docs) {
                    if (n_splits == 1) {
                        if (oc < n_out)
                            scores[doc * n_out + oc] = float(sum * out_scale);
                    } else {
                        const int64_t tail0 = int64_t(head_blocks) * DL;
                        partials[(int64_t(split) * (n_docs - tail0) + (doc - tail0)) * kVecPerLaunch + c] = sum;
                    }
                }
            }
        }
    }
    if constexpr (MODE == kModeScore) {
        __syncthreads();
        double *red = reinterpret_cast<double *>(lds + xs_bytes);
        red[walker * DL + dl] = acc;
        __syncthreads();
        if (walker == 0) {
            const int64_t doc = doc0 + dl;
            double sum = 0.0;
            for (int w = 0; w < n_walkers; ++w)
                sum += red[w * DL + dl];
            if (doc < n_docs) {
                if (n_splits == 1) {
                    scores[doc] = float(sum * out_scale);
                } else {
                    const int64_t tail0 = int64_t(head_blocks) * DL;
                    partials[int64_t(split) * (n_docs - tail0) + (doc - tail0)] = sum;
                }
            }
        }
    }
}

template <int DL, bool HALF, bool NARROW, bool CODED, int MODE>
ScoreFn pick_k(int k) {
    switch (k) {
    case 1: return score_kernel<DL, 1, HALF, NARROW, CODED, MODE, false>;
    case 2: return score_kernel<DL, 2, HALF, NARROW, CODED, MODE, false>;
    case 4: return score_kernel<DL, 4, HALF, NARROW, CODED, MODE, false>;
    default: return nullptr;
    }
}

template <bool NARROW, bool CODED, int MODE>
ScoreFn pick_dl(const treeens::LdsPlan &p) {
    if (p.lds_bytes == treeens::kLdsPerCu / 2) {
        // two workgroups per CU: only small float tiles of 64-document blocks
        if constexpr (CODED)
            return nullptr;
        else
            return p.docs_per_block == 64 ? pick_k<64, true, NARROW, false, MODE>(p.interleave) : nullptr;
    }
    if constexpr (MODE == kModeUsageSlot)
        return nullptr; // one-workgroup plans keep room for the bitmasks after the zero record
    else
    switch (p.docs_per_block) {
    case 64: return pick_k<64, false, NARROW, CODED, MODE>(p.interleave);
    case 32: return pick_k<32, false, NARROW, CODED, MODE>(p.interleave);
    case 16: return pick_k<16, false, NARROW, CODED, MODE>(p.interleave);
    case 8: return pick_k<8, false, NARROW, CODED, MODE>(p.interleave);
    default: return nullptr;
    }
}

} // namespace

template <int MODE>
ScoreFn pick_kernel(const treeens::LdsPlan &p, bool compact) {
    if (compact) {
        // compact packets: coded 64-document blocks, one workgroup per CU (not the trace)
        if constexpr (MODE == kModeScore || MODE == kModeLeaves || MODE == kModeVector || MODE == kModeRows)
            return p.coded && p.docs_per_block == 64 && p.lds_bytes == treeens::kLdsPerCu
                       ? score_kernel<64, treeens::kCompactTrees, false, false, true, MODE, true>
                       : nullptr;
        else
            return nullptr;
    }
    if (p.lds_bytes != treeens::kLdsPerCu / 2 && p.lds_bytes != treeens::kLdsPerCu)
        return nullptr;
    if (p.coded)
        return p.narrow ? pick_dl<true, true, MODE>(p) : pick_dl<false, true, MODE>(p);
    return p.narrow ? pick_dl<true, false, MODE>(p) : pick_dl<false, false, MODE>(p);
}

template ScoreFn pick_kernel<TREE_ENS_SCORE_MODE>(const LdsPlan &p, bool compact);

} // namespace treeens
