// uniform.hip -- scoring kernels for models of shallow trees (depth at most 3).
//
// The walk of score.hip reads one record and one feature per step and document from LDS, both
// gathers. Here every node of a (complete, padded) tree is evaluated for every document instead:
// node data is the same for all lanes, so it comes through scalar registers, a lane's features of
// 8 (4, 2) documents come with one LDS read, and two documents share one 32-bit register of 16-bit
// threshold codes. A node takes one packed subtraction for two documents (code - threshold: the
// sign decides, and fills the bits above the 11 bits of a code); a node picks its subtree's signs
// with one bit-select (v_bfi). The signs of the three levels form the leaf's place in the tree's
// table of 8 doubles in LDS, whose 16 words lie in different banks.
//
// Bound by VALU issue: 10 instructions per (64 documents, tree of depth 3), 83% of the issue slots
// busy, LDS 47%; the walk takes 13.7 and 6.9 LDS instructions. 20,000 trees, 136 features,
// 1,000,000 documents: 9.0 ms by the walk, 6.1 ms here and 0.35 ms of coding. Blocks of 512
// documents (one 16-byte read per node and lane) halve the address arithmetic of 128.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "score.hpp"
#include "uniform.hpp"

namespace treeens {

namespace {

// a where the bit of m is set, else b (v_bfi_b32)
__device__ __forceinline__ uint32_t select_bits(uint32_t m, uint32_t a, uint32_t b) { return (m & a) | (~m & b); }

// The same with a constant mask, kept as one v_bfi_b32 (the compiler would merge chains of these into
// an AND per operand).
__device__ __forceinline__ uint32_t select_const(uint32_t m, uint32_t a, uint32_t b) {
    uint32_t r;
    asm("v_bfi_b32 %0, %1, %2, %3" : "=v"(r) : "s"(m), "v"(a), "v"(b));
    return r;
}

// (w & mask) | b and bits 10 to 25 of w, each as the one instruction it is (the compiler would
// split them into masks of the parts it knows).
__device__ __forceinline__ uint32_t and_or(uint32_t w, uint32_t mask, uint32_t b) {
    uint32_t r;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(w), "s"(mask), "v"(b));
    return r;
}
__device__ __forceinline__ uint32_t bits_10_25(uint32_t w) {
    uint32_t r;
    asm("v_bfe_u32 %0, %1, 10, 16" : "=v"(r) : "v"(w));
    return r;
}

// Two documents' codes minus the threshold in the upper half of a node word.
__device__ __forceinline__ uint32_t sub2(uint32_t x, uint32_t w) {
    uint32_t r;
    asm("v_pk_sub_i16 %0, %1, %2 op_sel:[0,1] op_sel_hi:[1,1]" : "=v"(r) : "v"(x), "s"(w));
    return r;
}

template <int WORDS> struct Codes { // the codes of 2 * WORDS documents
    uint32_t w[WORDS];
};
template <int WORDS>
__device__ __forceinline__ Codes<WORDS> read_codes(const unsigned char *p) {
    Codes<WORDS> c;
    if constexpr (WORDS == 4) {
        const uint4 v = *reinterpret_cast<const uint4 *>(p);
        c.w[0] = v.x, c.w[1] = v.y, c.w[2] = v.z, c.w[3] = v.w;
    } else if constexpr (WORDS == 2) {
        const uint2 v = *reinterpret_cast<const uint2 *>(p);
        c.w[0] = v.x, c.w[1] = v.y;
    } else {
        c.w[0] = *reinterpret_cast<const uint32_t *>(p);
    }
    return c;
}

// DEPTH: 2 or 3. WORDS: registers of two documents' codes per lane (4, 2, 1: blocks of 512, 256,
// 128 documents).
template <int DEPTH, int WORDS>
__global__ void __launch_bounds__(kThreads, 4)
uniform_kernel(const uint16_t *__restrict__ codes, int64_t n_docs, int32_t n_cols, const uint32_t *__restrict__ nodes,
               const double *__restrict__ leaves, int32_t n_chunks, int32_t head_blocks, int32_t tail_splits,
               double *__restrict__ partials, float *__restrict__ scores, double scale) {
    constexpr int kDocs = 128 * WORDS;         // documents of a block
    constexpr int kLeaves = 1 << DEPTH;        // leaves of a tree
    constexpr int kNodes = kLeaves - 1;        // nodes of a tree
    constexpr int kTrees = uniform_trees(DEPTH); // trees of a chunk
    constexpr int kStep = 4;                   // trees whose node words load together
    constexpr int kWaves = kThreads / 64;
    typedef uint32_t NodeWords __attribute__((ext_vector_type(kLeaves)));
    // [0, kUniformLeafBytes x waves): each wave's leaf tables of one chunk; then the document
    // tile, [column][kDocs] codes
    __shared__ __align__(16) unsigned char lds[kLdsPerCu];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // head and tail blocks as in score_kernel: the splits of one tail block after a head share an
    // XCD's L2
    int64_t block = blockIdx.x;
    int split = 0, n_splits = 1;
    if (block >= head_blocks) {
        const int64_t t = block - head_blocks;
        if (head_blocks > 0) {
            const int64_t x = t % kXcds, r = t / kXcds;
            block = head_blocks + (r / tail_splits) * kXcds + x;
            split = int(r % tail_splits);
            if (block * kDocs >= n_docs)
                return;
        } else {
            block = head_blocks + t / tail_splits;
            split = int(t % tail_splits);
        }
        n_splits = tail_splits;
    }
    const int64_t doc0 = block * kDocs;
    const int c_lo = int((int64_t(n_chunks) * split) / n_splits);
    const int c_hi = int((int64_t(n_chunks) * (split + 1)) / n_splits);

    // Stage the document tile: neighbouring lanes hold neighbouring documents, so the 16-bit
    // writes fill whole words. 16-byte reads where rows are whole multiples of 8 codes.
    {
        constexpr int kGroups = kThreads / kDocs;
        const int d = tid % kDocs, g = tid / kDocs;
        const uint16_t *row = codes + min<int64_t>(doc0 + d, n_docs - 1) * n_cols;
        uint16_t *dst = reinterpret_cast<uint16_t *>(lds + kUniformDocBase) + d;
        if (n_cols % 8 == 0) {
            const uint4 *row4 = reinterpret_cast<const uint4 *>(row);
            constexpr int kUnroll = 4;
            for (int q0 = g; q0 < n_cols / 8; q0 += kGroups * kUnroll) {
                uint4 v[kUnroll];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u)
                    v[u] = row4[min(q0 + u * kGroups, n_cols / 8 - 1)];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    const int q = q0 + u * kGroups;
                    if (q < n_cols / 8) {
                        const uint16_t *e = reinterpret_cast<const uint16_t *>(&v[u]);
#pragma unroll
                        for (int k = 0; k < 8; ++k)
                            dst[(q * 8 + k) * kDocs] = e[k];
                    }
                }
            }
        } else {
            constexpr int kUnroll = 8;
            for (int c0 = g; c0 < n_cols; c0 += kGroups * kUnroll) {
                uint16_t v[kUnroll];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u)
                    v[u] = row[min(c0 + u * kGroups, n_cols - 1)];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u)
                    if (c0 + u * kGroups < n_cols)
                        dst[(c0 + u * kGroups) * kDocs] = v[u];
            }
        }
    }

    double acc[2 * WORDS];
#pragma unroll
    for (int i = 0; i < 2 * WORDS; ++i)
        acc[i] = 0.0;
    const uint32_t lane_off = uint32_t(lane) * uint32_t(4 * WORDS);
    // Wave v takes chunks c_lo + v, c_lo + v + 16, ...; a chunk's leaf tables (1 KiB) are one
    // 16-byte load per lane, the next chunk's in flight while this one is evaluated. kStep trees'
    // node words load at a time, the next ones' while these trees are evaluated. A tree's codes are
    // read while the tree before it is evaluated, and its leaves are added after the next tree's
    // are read, so that a wave has LDS reads in flight all the time.
    static_assert(kTrees * kLeaves * 8 == kUniformLeafBytes && kUniformLeafBytes == 64 * 16, "one load per lane");
    static_assert(kTrees % kStep == 0 && kStep % 2 == 0, "whole steps");
    const uint4 *leaf4 = reinterpret_cast<const uint4 *>(leaves) + lane;
    struct Step {
        NodeWords w[kStep];
    };
    auto load_step = [&](int chunk, int t0) {
        Step st;
        int first = chunk * kTrees + t0;
        asm volatile("" : "+s"(first)); // the loads stay where they are written
        const NodeWords *p = reinterpret_cast<const NodeWords *>(nodes) + first;
#pragma unroll
        for (int t = 0; t < kStep; ++t)
            st.w[t] = p[t];
        return st;
    };
    Codes<WORDS> x[2][kNodes];
    auto read_tree = [&](Codes<WORDS> (&dst)[kNodes], const NodeWords &w) {
#pragma unroll
        for (int n = 0; n < kNodes; ++n)
            dst[n] = read_codes<WORDS>(lds + (((w[n] & 0xFFFFu) << 6) + lane_off));
    };
    double leaf[2][2 * WORDS];
#pragma unroll
    for (int i = 0; i < 2 * WORDS; ++i)
        leaf[1][i] = 0.0;
    const int c0 = c_lo + wave;
    uint4 next_leaf{0, 0, 0, 0};
    Step st{};
    if (c0 < c_hi) {
        next_leaf = leaf4[int64_t(c0) * 64];
        st = load_step(c0, 0);
    }
    __syncthreads(); // the document tile is written
    if (c0 < c_hi)
        read_tree(x[0], st.w[0]);
    for (int c = c0; c < c_hi; c += kWaves) {
        *reinterpret_cast<uint4 *>(lds + wave * kUniformLeafBytes + lane * 16) = next_leaf;
        const int next_chunk = min(c + kWaves, n_chunks - 1); // past the last: loaded, not used
        next_leaf = leaf4[int64_t(next_chunk) * 64];
        for (int t0 = 0; t0 < kTrees; t0 += kStep) {
            Step after;
            // LDS base of these trees' tables: 64-byte units, placed where the extraction of the
            // first document's place finds them (bit 16 of the merged signs is bit 6 of its
            // address), and as the upper word of the second document's shift
            const uint32_t base = uint32_t(wave * kUniformLeafBytes + t0 * (kLeaves * 8)) >> 6;
            uint32_t base_lo;
            asm("v_mov_b32 %0, %1" : "=v"(base_lo) : "s"(base << 16));
#pragma unroll
            for (int t = 0; t < kStep; ++t) {
                // (fences keep the compiler from hoisting the next trees' reads up here: it ran out
                // of registers)
                __builtin_amdgcn_sched_barrier(0);
                if (t + 1 < kStep)
                    read_tree(x[(t + 1) & 1], st.w[t + 1]);
                else
                    read_tree(x[(t + 1) & 1], after.w[0]);
                Codes<WORDS>(&d)[kNodes] = x[t & 1];
#pragma unroll
                for (int n = 0; n < kNodes; ++n)
#pragma unroll
                    for (int i = 0; i < WORDS; ++i)
                        d[n].w[i] = sub2(d[n].w[i], st.w[t][n]);
                // The next step's node words load from here: scalar loads return out of order with
                // LDS reads, so the next wait for a read waits for them too, and from here it is a
                // tree's selections away.
                if (t == 0) {
                    __builtin_amdgcn_sched_barrier(0);
                    const bool last = t0 + kStep == kTrees;
                    after = load_step(last ? next_chunk : c, last ? 0 : t0 + kStep);
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
                for (int i = 0; i < WORDS; ++i) {
                    // a set sign sends left: node n's children are 2n + 1 (left) and 2n + 2
                    const uint32_t s1 = select_bits(d[0].w[i], d[1].w[i], d[2].w[i]);
                    uint32_t place;
                    if constexpr (DEPTH == 3) {
                        const uint32_t a = select_bits(d[0].w[i], d[3].w[i], d[5].w[i]);
                        const uint32_t b = select_bits(d[0].w[i], d[4].w[i], d[6].w[i]);
                        const uint32_t s2 = select_bits(s1, a, b);
                        place = select_const(0x80008000u, d[0].w[i], select_const(0x40004000u, s1, s2));
                    } else {
                        place = select_const(0x40004000u, d[0].w[i], s1);
                    }
                    place = and_or(place, DEPTH == 3 ? 0xE000E000u : 0x60006000u, base_lo);
                    const uint32_t lo = bits_10_25(place);
                    const uint32_t hi = __builtin_amdgcn_alignbit(base, place, 26);
                    leaf[t & 1][2 * i] = *reinterpret_cast<const double *>(lds + lo + t * (kLeaves * 8));
                    leaf[t & 1][2 * i + 1] = *reinterpret_cast<const double *>(lds + hi + t * (kLeaves * 8));
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int i = 0; i < 2 * WORDS; ++i)
                    acc[i] += leaf[(t + 1) & 1][i];
            }
            st = after;
        }
    }
#pragma unroll
    for (int i = 0; i < 2 * WORDS; ++i)
        acc[i] += leaf[1][i];

    // sums of the waves, in wave order
    __syncthreads();
    double *red = reinterpret_cast<double *>(lds + kUniformDocBase);
#pragma unroll
    for (int i = 0; i < 2 * WORDS; ++i)
        red[wave * kDocs + lane * (2 * WORDS) + i] = acc[i];
    __syncthreads();
    if (tid < kDocs && doc0 + tid < n_docs) {
        double sum = 0.0;
        for (int w = 0; w < kWaves; ++w)
            sum += red[w * kDocs + tid];
        if (n_splits == 1) {
            scores[doc0 + tid] = float(sum * scale);
        } else {
            const int64_t tail0 = int64_t(head_blocks) * kDocs;
            partials[int64_t(split) * (n_docs - tail0) + (doc0 + tid - tail0)] = sum;
        }
    }
}

} // namespace

void launch_uniform(const UniformPlan &u, hipStream_t stream, const uint16_t *codes, int64_t n_docs, int32_t n_cols,
                    const uint32_t *nodes, const double *leaves, const LaunchShape &shape, double *partials,
                    float *scores, double scale) {
    const int words = u.docs_per_block / 128;
    auto *fn = u.depth == 3 ? (words == 4 ? uniform_kernel<3, 4> : words == 2 ? uniform_kernel<3, 2> : uniform_kernel<3, 1>)
                            : (words == 4 ? uniform_kernel<2, 4> : words == 2 ? uniform_kernel<2, 2> : uniform_kernel<2, 1>);
    const int64_t n_blocks = (n_docs + u.docs_per_block - 1) / u.docs_per_block;
    const int64_t tail = n_blocks - shape.head;
    const int64_t slots = shape.head > 0 ? (tail + kXcds - 1) / kXcds * kXcds : tail;
    hipLaunchKernelGGL(fn, dim3(unsigned(shape.head + slots * shape.splits)), dim3(kThreads), 0, stream, codes, n_docs,
                       n_cols, nodes, leaves, u.n_chunks, int32_t(shape.head), shape.splits, partials, scores, scale);
}

} // namespace treeens
