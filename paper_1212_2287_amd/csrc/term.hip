// term.hip -- scoring kernel of terminal packets: threshold-coded documents, 64 per block, one
// workgroup per CU (see TermPlan in pack.hpp).
//
// The walk of the compact packets (score.hip) is bound by latency: 32 walks of 64 documents per CU is
// what their windows leave room for next to the document tile. Ending the walks at subtrees of depth
// 2 halves the records of a tree, so a CU holds 64 walks, each about two steps shorter. What is left
// of a walk runs beside the next ones: the terminal's slot is loaded when its group ends, its one or
// two splits are taken (two features from LDS) when the next group ends, and the leaf value, loaded
// then, is added one group later.
//
// Still bound by latency, closer to issue: 5,000 trees of 256 leaves, 700 features, 1,000,000
// documents in 14.1 ms (16.7 ms by compact packets), VALU 66% and LDS 62% busy (a quarter of that
// in bank conflicts of the pair reads), 42% of wave time in waits (compact packets: 52%, 58%, 52%).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "score.hpp"
#include "term.hpp"

namespace treeens {

namespace {

// (w & mask) | b in one VALU op.
__device__ __forceinline__ uint32_t and_or(uint32_t w, uint32_t mask, uint32_t b) {
    uint32_t r;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(w), "s"(mask), "v"(b));
    return r;
}

// A children pair, as one ds_read_b64 (a plain load gets split).
__device__ __forceinline__ uint64_t read_pair(const unsigned char *p) {
    return __hip_atomic_load(reinterpret_cast<const uint64_t *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

__global__ void __launch_bounds__(kThreads, 4)
term_kernel(const uint16_t *__restrict__ codes, int64_t n_docs, int32_t n_cols, const uint32_t *__restrict__ packets,
            const uint32_t *__restrict__ slots, int32_t per_wave, int32_t head_blocks, int32_t tail_splits,
            double *__restrict__ partials, float *__restrict__ scores, double scale) {
    constexpr int K = kTermTrees, DL = 64;
    // [0, (n_cols + 1) x 128): the document tile, [column][64] staged codes, column 0 code 0; then each
    // wave's K windows
    __shared__ __align__(16) unsigned char lds[kLdsPerCu];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t lane_off = uint32_t(lane) * 2u;

    // head and tail blocks as in score_kernel
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
    const int q_lo = int((int64_t(per_wave) * split) / n_splits);
    const int q_hi = int((int64_t(per_wave) * (split + 1)) / n_splits);

    // A packet is nine 8-byte rows of 64 lanes, read with raw buffer loads (offset of the packet in a
    // scalar register); the next one is in flight while this one is walked.
    constexpr int kRows = kCompactPacketBytes / 512;
    const __amdgpu_buffer_rsrc_t pk_rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(packets), 0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t slot_rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(slots), 0, 0x7fffffff, 0x00020000);
    uint2 pa[kRows];
    auto fetch = [&](int q) {
        const int soff = (wave * per_wave + q) * kCompactPacketBytes;
#pragma unroll
        for (int j = 0; j < kRows; ++j) {
            const auto v = __builtin_amdgcn_raw_buffer_load_b64(pk_rsrc, lane * 8 + j * 512, soff, 0);
            pa[j] = make_uint2(v[0], v[1]);
        }
    };
    const bool any = q_lo < q_hi;
    if (any)
        fetch(q_lo);

    // Stage the document tile: lane = document. 16-byte reads where rows are whole multiples of 8
    // codes.
    {
        const uint16_t *row = codes + min<int64_t>(doc0 + lane, n_docs - 1) * n_cols;
        uint16_t *xs = reinterpret_cast<uint16_t *>(lds) + lane;
        constexpr int kWaves = kThreads / 64;
        if (tid < DL)
            xs[0] = uint16_t(31);
        if (n_cols % 8 == 0) {
            const uint4 *row4 = reinterpret_cast<const uint4 *>(row);
            constexpr int kUnroll = 4;
            for (int q0 = wave; q0 < n_cols / 8; q0 += kWaves * kUnroll) {
                uint4 v[kUnroll];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u)
                    v[u] = row4[min(q0 + u * kWaves, n_cols / 8 - 1)];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u) {
                    const int q = q0 + u * kWaves;
                    if (q < n_cols / 8) {
                        const uint16_t *e = reinterpret_cast<const uint16_t *>(&v[u]);
#pragma unroll
                        for (int k = 0; k < 8; ++k)
                            xs[(q * 8 + k + 1) * DL] = e[k];
                    }
                }
            }
        } else {
            constexpr int kUnroll = 8;
            for (int c0 = wave; c0 < n_cols; c0 += kWaves * kUnroll) {
                uint16_t v[kUnroll];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u)
                    v[u] = row[min(c0 + u * kWaves, n_cols - 1)];
#pragma unroll
                for (int u = 0; u < kUnroll; ++u)
                    if (c0 + u * kWaves < n_cols)
                        xs[(c0 + u * kWaves + 1) * DL] = v[u];
            }
        }
    }

    double acc = 0.0;
    if (any) {
        const uint32_t my_win = uint32_t(term_window_base(n_cols)) + uint32_t(wave) * kCompactWindowBytes;
        const uint32_t col_sel = __builtin_amdgcn_readfirstlane(0x1FF80u); // column * 128 bytes
        const uint32_t pair_sel = __builtin_amdgcn_readfirstlane(0x3F8u);
        constexpr uint32_t kLeafCol = 128u; // feature addresses below this are column 0
        // window bases, opaque to the compiler (it would copy them from scalar registers at every step)
        uint32_t tb[K];
#pragma unroll
        for (int i = 0; i < K; ++i)
            asm volatile("v_mov_b32 %0, %1" : "=v"(tb[i]) : "s"(my_win + uint32_t(i) * kTermWindowBytes));
        auto feature = [&](uint32_t r) {
            return uint32_t(*reinterpret_cast<const uint16_t *>(lds + and_or(r >> 4, col_sel, lane_off)));
        };
        // of the last group walked: byte offset of each terminal's slot, its splits; of the one before:
        // the leaf values
        uint32_t off[K];
        uint32_t s0[K], s1[K], s2[K];
        uint32_t val[K];
        auto load_slots = [&]() {
#pragma unroll
            for (int i = 0; i < K; ++i) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b96(slot_rsrc, off[i], 0, 0);
                s0[i] = v[0], s1[i] = v[1], s2[i] = v[2];
            }
        };
        // the last group's splits, up to the load of its leaf values
        auto finish = [&]() {
            uint32_t x[K], at[K];
#pragma unroll
            for (int i = 0; i < K; ++i)
                x[i] = feature(s0[i]);
#pragma unroll
            for (int i = 0; i < K; ++i) {
                const bool right = x[i] >= (s0[i] >> 16);
                s1[i] = right ? s2[i] : s1[i];
                at[i] = right ? 24u : 16u; // the values' place in the slot
            }
#pragma unroll
            for (int i = 0; i < K; ++i)
                x[i] = feature(s1[i]);
#pragma unroll
            for (int i = 0; i < K; ++i) {
                const uint32_t value_at = off[i] + at[i] + (x[i] >= (s1[i] >> 16) ? 4u : 0u);
                val[i] = __builtin_amdgcn_raw_buffer_load_b32(slot_rsrc, value_at, 0, 0);
            }
        };
        auto add_values = [&]() {
#pragma unroll
            for (int i = 0; i < K; ++i)
                acc += double(__uint_as_float(val[i]));
        };
        // before the first group: the zero pair of the first packet, value 0
        const uint32_t slot0 = uint32_t(wave * per_wave + q_lo) * (kTermSlotPacketWords * 4);
#pragma unroll
        for (int i = 0; i < K; ++i) {
            off[i] = slot0 + (kTermWindowBytes - 8) * (kTermSlotWords);
            val[i] = 0u;
        }
        load_slots();
        __syncthreads(); // the document tile is written
        for (int q = q_lo; q < q_hi; ++q) {
            const uint32_t slot_base = uint32_t(wave * per_wave + q) * (kTermSlotPacketWords * 4);
#pragma unroll
            for (int j = 0; j < kRows - 1; ++j)
                *reinterpret_cast<uint2 *>(lds + my_win + uint32_t(j) * 512u + uint32_t(lane * 8)) = pa[j];
            // the header row stays in registers: lane l holds words 2l and 2l + 1
            const uint2 hrow = pa[kRows - 1];
            // the wave's own writes complete before it reads the packet back
            __builtin_amdgcn_s_waitcnt(kWaitLgkmcnt0);
            fetch(min(q + 1, q_hi - 1)); // after the last: that one again, not used
            const int ng = __builtin_amdgcn_readlane(int(hrow.x), 0);
            int j = 0;
            do {
                // group j's roots: header words 4 + 4j ..., lanes 2 + 2j and 3 + 2j
                static_assert(kCompactHeaderWords == 4 && K == 4, "root lanes");
                uint32_t r[K];
                r[0] = uint32_t(__builtin_amdgcn_readlane(int(hrow.x), 2 + 2 * j));
                r[1] = uint32_t(__builtin_amdgcn_readlane(int(hrow.y), 2 + 2 * j));
                r[2] = uint32_t(__builtin_amdgcn_readlane(int(hrow.x), 3 + 2 * j));
                r[3] = uint32_t(__builtin_amdgcn_readlane(int(hrow.y), 3 + 2 * j));
                uint32_t fa[K], xv[K], lo[K], hi[K];
                auto issue = [&]() {
#pragma unroll
                    for (int i = 0; i < K; ++i) {
                        fa[i] = and_or(r[i] >> 4, col_sel, lane_off);
                        const uint32_t pair = and_or(r[i], pair_sel, tb[i]);
                        xv[i] = *reinterpret_cast<const uint16_t *>(lds + fa[i]);
                        const uint64_t pr = read_pair(lds + pair);
                        lo[i] = uint32_t(pr);
                        hi[i] = uint32_t(pr >> 32);
                    }
                };
                // as in score_kernel: the first step untested, then until the lead tree's lanes, then
                // all K trees' lanes, sit on terminals; the next reads are issued before the test
                issue();
                for (;;) {
#pragma unroll
                    for (int i = 0; i < K; ++i)
                        r[i] = xv[i] >= (r[i] >> 16) ? hi[i] : lo[i];
                    issue();
                    if (__builtin_amdgcn_ballot_w64(fa[0] >= kLeafCol) == 0) {
                        bool inner = false;
#pragma unroll
                        for (int i = 1; i < K; ++i)
                            inner |= fa[i] >= kLeafCol;
                        if (__builtin_amdgcn_ballot_w64(inner) == 0)
                            break;
                    }
                }
#pragma unroll
                for (int i = 0; i < K; ++i)
                    asm volatile("" ::"v"(xv[i]), "v"(lo[i]), "v"(hi[i]));
                add_values();
                finish();
#pragma unroll
                for (int i = 0; i < K; ++i)
                    off[i] = ((r[i] & 0x3FCu) << 3) + (slot_base + uint32_t(i) * (kTermWindowBytes * kTermSlotWords));
                load_slots();
            } while (++j < ng);
        }
        add_values();
        finish();
        add_values();
    } else {
        __syncthreads();
    }

    // sums of the waves, in wave order
    __syncthreads();
    double *red = reinterpret_cast<double *>(lds);
    red[wave * DL + lane] = acc;
    __syncthreads();
    if (tid < DL && doc0 + tid < n_docs) {
        double sum = 0.0;
        for (int w = 0; w < kThreads / 64; ++w)
            sum += red[w * DL + tid];
        if (n_splits == 1) {
            scores[doc0 + tid] = float(sum * scale);
        } else {
            const int64_t tail0 = int64_t(head_blocks) * DL;
            partials[int64_t(split) * (n_docs - tail0) + (doc0 + tid - tail0)] = sum;
        }
    }
}

} // namespace

void launch_term(const TermPlan &t, hipStream_t stream, const uint16_t *codes, int64_t n_docs, int32_t n_cols,
                 const uint32_t *packets, const uint32_t *slots, int64_t head, int splits, double *partials,
                 float *scores, double scale) {
    const int64_t n_blocks = (n_docs + 63) / 64, tail = n_blocks - head;
    const int64_t tail_slots = head > 0 ? (tail + kXcds - 1) / kXcds * kXcds : tail;
    hipLaunchKernelGGL(term_kernel, dim3(unsigned(head + tail_slots * splits)), dim3(kThreads), 0, stream, codes, n_docs,
                       n_cols, packets, slots, t.per_wave, int32_t(head), splits, partials, scores, scale);
}

} // namespace treeens
