// tree_ens.hip -- the C ABI of the tree-ensemble scorer, the launch planner, and the kernels around
// the scoring ones (score.hip): threshold codes, split reduction, leaf id rows.

#include <hip/hip_runtime.h>
#include <hip/hiprtc.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "pack.hpp"
#include "planner.hpp"
#include "score.hpp"
#include "scratch.hpp"
#include "status.hpp"
#include "term.hpp"
#include "tree_ens.h"
#include "uniform.hpp"

using treeens::NodeRec;
using treeens::Packed;

namespace {

thread_local std::string g_err;

int fail(int code, const std::string &msg) {
    g_err = msg;
    return code;
}

int hip_fail(hipError_t e, const char *what) {
    return fail(TREE_ENS_E_DEVICE, std::string(what) + ": " + hipGetErrorString(e));
}

using namespace treeens;

// ------------------------------------------------------------------------------------------
// kernels
// ------------------------------------------------------------------------------------------

// Sum of the split partials of each entry in a fixed order (so the rounding never changes).
// Entry j is component j % comps of document j / comps; it goes to output column
// c_base + j % comps of a row of n_out scores (if that column exists), scaled by out_scale.
// Few splits: one thread per entry, in split order. Many splits (small batches): one wave per
// entry, lanes interleave the splits, then a fixed butterfly.
struct ReduceOut {
    float *scores;
    int32_t comps, n_out, c_base;
    double scale;
    __device__ void store(int64_t j, double s) const {
        const int64_t doc = j / comps;
        const int c = c_base + int(j - doc * comps);
        if (c < n_out)
            scores[doc * n_out + c] = float(s * scale);
    }
};

__global__ void reduce_partials_thread_kernel(const double *__restrict__ partials, int32_t n_splits,
                                              int64_t n_docs, ReduceOut out) {
    const int64_t d = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (d < n_docs) {
        // eight independent loads in flight, then summed in split order
        double s = 0.0;
        int k = 0;
        for (; k + 8 <= n_splits; k += 8) {
            double v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                v[u] = partials[int64_t(k + u) * n_docs + d];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                s += v[u];
        }
        for (; k < n_splits; ++k)
            s += partials[int64_t(k) * n_docs + d];
        out.store(d, s);
    }
}

__global__ void __launch_bounds__(64)
reduce_partials_wave_kernel(const double *__restrict__ partials, int32_t n_splits, int64_t n_docs,
                            ReduceOut out) {
    const int64_t d = blockIdx.x;
    double s = 0.0;
    for (int k = threadIdx.x; k < n_splits; k += 64)
        s += partials[int64_t(k) * n_docs + d];
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1)
        s += __shfl_xor(s, off);
    if (threadIdx.x == 0)
        out.store(d, s);
}

__global__ void fill_zero_kernel(float *__restrict__ scores, int64_t n) {
    const int64_t d = int64_t(blockIdx.x) * blockDim.x + threadIdx.x;
    if (d < n)
        scores[d] = 0.0f;
}

// Threshold codes of a block of documents for a chunk of features: code_f(x) is the number of
// f's sorted distinct thresholds t with x >= t (a NaN x compares false everywhere and gets 0).
// The chunk's search tables are staged in LDS: feature j's 2^s - 1 entries hold its list as a
// complete search tree in breadth-first order (slot i at entry i - 1), padded with NaN (which
// never compares true), so the count is s steps of i = 2i + (x >= slot i) from i = 1, the same
// for every lane, and code = i - 2^s. Thread e takes elements e, e + 1,024, ... of the block's [doc][feature] order,
// stepping its (document, feature) pair without a division. Output rows hold n_cols 16-bit
// codes, each stored as code << code_shift with the shifted-out bits set (code_shift 5 for the
// compact records' comparison, else 0).
constexpr int kCodeThreads = 1024;
// One step of the search: 2i + (x >= t) as a compare into VCC and an add-with-carry of i to
// itself (two VALU ops; the s_nop as in narrow_child).
__device__ __forceinline__ uint32_t search_step(uint32_t i, float x, float t) {
    uint32_t r;
    asm("v_cmp_ge_f32 vcc, %1, %2\n\t"
        "s_nop 1\n\t"
        "v_addc_co_u32 %0, vcc, %3, %3, vcc"
        : "=v"(r)
        : "v"(x), "v"(t), "v"(i)
        : "vcc");
    return r;
}
__global__ void __launch_bounds__(kCodeThreads)
code_kernel(const float *__restrict__ X, int64_t n_docs, int32_t n_features, int32_t n_cols,
            int32_t docs_per_wg, const float *__restrict__ table,
            const treeens::CodeChunk *__restrict__ chunks, int32_t n_chunks, int32_t code_shift,
            uint16_t *__restrict__ codes) {
    __shared__ float tab[treeens::kCodeTableFloats];
    // Workgroups are dealt to the XCDs in index order: index L runs chunk (L % (8C)) / 8 of
    // document block (L / (8C)) * 8 + L % 8, so all C chunks of a block share one XCD and run
    // one after another there, and the cache lines of a row that two neighbouring chunks
    // share come from HBM once.
    const int64_t L = blockIdx.x;
    const int64_t per = int64_t(kXcds) * n_chunks;
    const int chunk = int((L % per) / kXcds);
    const int64_t block = (L / per) * kXcds + L % kXcds;
    if (block * docs_per_wg >= n_docs)
        return;
    const treeens::CodeChunk ch = chunks[chunk];
    const int nf = ch.f_end - ch.f_begin;
    const int steps = ch.search_steps;
    for (int i = threadIdx.x; i < ch.table_end - ch.table_begin; i += kCodeThreads)
        tab[i] = table[ch.table_begin + i];
    __syncthreads();
    const int64_t d0 = block * docs_per_wg;
    const int n = int(min<int64_t>(docs_per_wg, n_docs - d0)) * nf;
    // nf <= 256: every step moves at least 4 documents on
    const int step_d = kCodeThreads / nf, step_j = kCodeThreads - step_d * nf;
    int d = int(threadIdx.x) / nf, j = int(threadIdx.x) - d * nf;
    const uint32_t leaf0 = 1u << steps;
    // kCodeBatch elements per thread at a time: their feature values load together, then their
    // searches interleave (independent LDS round trips in flight)
    constexpr int kCodeBatch = 4;
    for (int e0 = threadIdx.x; e0 < n; e0 += kCodeBatch * kCodeThreads) {
        float x[kCodeBatch];
        int64_t at[kCodeBatch];
        int t0[kCodeBatch];
        uint32_t i[kCodeBatch];
#pragma unroll
        for (int u = 0; u < kCodeBatch; ++u) {
            const bool live = e0 + u * kCodeThreads < n;
            const int64_t doc = d0 + d;
            at[u] = live ? doc * n_cols + ch.f_begin + j : -1;
            x[u] = live ? X[doc * n_features + ch.f_begin + j] : 0.0f;
            t0[u] = j * int(leaf0 - 1u) - 1; // slot i of feature j is tab[t0 + i]
            i[u] = 1u;
            d += step_d;
            j += step_j;
            if (j >= nf) {
                j -= nf;
                ++d;
            }
        }
        for (int s = 0; s < steps; ++s) {
#pragma unroll
            for (int u = 0; u < kCodeBatch; ++u)
                i[u] = search_step(i[u], x[u], tab[t0[u] + int(i[u])]);
        }
#pragma unroll
        for (int u = 0; u < kCodeBatch; ++u) {
            const uint32_t code = i[u] - leaf0;
            if (at[u] >= 0)
                codes[at[u]] = uint16_t((code << code_shift) | ((1u << code_shift) - 1u));
        }
    }
}

// Leaf ids of whole document blocks from the packed-order leaf positions the walk left in
// pos[block][packed tree][DL documents] (16 bits each): out[doc][input tree]. A workgroup takes
// one block and kIdTrees consecutive input trees: reads DL positions of each tree (one row,
// coalesced), maps them to input node ids (orig_id is null when the walk stored ids already) and
// writes them transposed through LDS, 64 consecutive trees of a document per wave store.
// Bound by memory: 2 bytes read, 4 written per (document, tree). The walk's lanes hold documents,
// and its trees are packed in another order than the output's, so storing ids from the walk
// writes single 4-byte pieces of 64 rows per instruction, most lines leaving L2 before they are
// full.
constexpr int kIdThreads = 256;
constexpr int kIdTrees = 64;
template <int DL>
__global__ void __launch_bounds__(kIdThreads)
leaf_ids_kernel(const uint16_t *__restrict__ pos, int64_t n_docs, int32_t n_trees,
                const int32_t *__restrict__ tree_pos, const uint32_t *__restrict__ tree_node_off,
                const int32_t *__restrict__ orig_id, int32_t *__restrict__ out) {
    // row stride DL + 2: an odd number of dwords, so a column of 64 trees spreads over the banks
    __shared__ uint16_t tile[kIdTrees * (DL + 2)];
    // all tree tiles of a block on one XCD (workgroups are dealt to them in index order): the
    // lines two neighbouring tiles share are completed in one L2
    const int64_t L = blockIdx.x;
    const int n_tiles = (n_trees + kIdTrees - 1) / kIdTrees;
    const int64_t per = int64_t(kXcds) * n_tiles;
    const int64_t block = (L / per) * kXcds + L % kXcds;
    const int t0 = int((L % per) / kXcds) * kIdTrees;
    if (block * DL >= n_docs)
        return;
    const int nt = min(kIdTrees, n_trees - t0);
    constexpr int kRows = kIdThreads / DL; // trees read at a time
    const int d = int(threadIdx.x) % DL;
    // eight rows at a time: their loads (tree, position, id) are in flight together
    constexpr int kBatch = 8;
    const bool live = block * DL + d < n_docs; // documents past the last one hold no position
    for (int r0 = int(threadIdx.x) / DL; r0 < nt; r0 += kRows * kBatch) {
        int pt[kBatch];
        uint32_t id[kBatch];
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            pt[u] = tree_pos[t0 + min(r0 + u * kRows, nt - 1)];
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            id[u] = live ? uint32_t(pos[(block * n_trees + pt[u]) * DL + d]) : 0u;
        if (orig_id) {
#pragma unroll
            for (int u = 0; u < kBatch; ++u)
                id[u] = uint32_t(orig_id[tree_node_off[pt[u]] + id[u]]);
        }
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
            if (r0 + u * kRows < nt)
                tile[(r0 + u * kRows) * (DL + 2) + d] = uint16_t(id[u]);
    }
    __syncthreads();
    const int lane = int(threadIdx.x) % kIdTrees;
    if (lane < nt) {
        const int64_t n_here = min<int64_t>(DL, n_docs - block * DL);
        for (int k = int(threadIdx.x) / kIdTrees; k < n_here; k += kIdThreads / kIdTrees)
            out[(block * DL + k) * n_trees + t0 + lane] = tile[lane * (DL + 2) + k];
    }
}

} // namespace

namespace treeens {
int set_error(int code, const std::string &message) {
    g_err = message;
    return code;
}
void clear_error() { g_err.clear(); }
} // namespace treeens

// ------------------------------------------------------------------------------------------
// handle
// ------------------------------------------------------------------------------------------
struct tree_ens {
    int device = 0;
    int32_t n_trees = 0;
    int32_t n_cols = 0;
    int32_t max_depth = 0;
    int64_t n_nodes = 0;
    treeens::LdsPlan plan{};
    int32_t level_begin[treeens::kTileLevels + 1] = {};
    treeens::PlanFacts facts{};  // what the launch planner goes by
    int32_t usage_slot_off = -1; // feature-trace bitmasks in the tile slot (two-workgroup plans)
    int64_t level_image_off[treeens::kTileLevels] = {};
    int32_t level_slot_recs[treeens::kTileLevels] = {};
    void *d_model = nullptr; // the one allocation that every array below lies in
    uint2 *d_images = nullptr;      // tile images of every tiling
    uint32_t *d_tile_recs = nullptr; // records of each tile image
    // walker packets (plans of 64- and 32-document blocks): records per sub-slot (0: the plan
    // walks shared tiles), the packets' zero record, packets per wave, and the
    // images
    int32_t pk_recs = 0;
    int32_t pk_zero_rec = 0;
    int32_t pk_per_walker = 0;
    uint2 *d_packets = nullptr;
    // compact packets (coded 64-document plans; in place of the packets above for scores, leaf
    // ids and vector-valued leaves): trees per lane (0: none), packets per wave, the
    // packets, and the leaf payloads and input node ids at the leaves' positions
    int32_t cp_k = 0;
    int32_t cp_per_walker = 0;
    uint32_t *d_cpackets = nullptr;
    uint32_t *d_cleaf = nullptr;
    int32_t *d_cleaf_id = nullptr;
    // big trees (packed indices [n_small, n_trees)): their records in the big-tree format, the
    // first at packed node offset big_off0
    int32_t n_small = 0;
    uint32_t big_off0 = 0;
    uint2 *d_big = nullptr;
    // leaf-id output: packed tree -> input tree, packed node -> input node id
    uint32_t *d_tree_node_off = nullptr;
    int32_t *d_tree_orig = nullptr;
    int32_t *d_tree_pos = nullptr; // input tree -> packed tree
    int32_t *d_orig_id = nullptr;
    // vector-valued leaves and bagging: outputs per document, the table of leaf rows, and the
    // factor 1 / n_bags applied to every sum
    int32_t n_outputs = 1;
    int32_t n_bags = 1;
    int32_t vec_stride = 0;
    float *d_leaf_vec = nullptr;
    uint32_t *d_tree_row0 = nullptr; // each packed tree's first row
    // coded models
    float *d_code_search = nullptr; // the coding chunks' search tables
    treeens::CodeChunk *d_code_chunks = nullptr;
    int32_t n_code_chunks = 0;
    // terminal packets (coded documents, scores only): packets and terminal slots
    treeens::TermPlan term{};
    uint32_t *d_term_packets = nullptr;
    uint32_t *d_term_slots = nullptr;
    // uniform evaluation (shallow trees): node words and leaf tables
    treeens::UniformPlan uniform{};
    uint32_t *d_uniform_nodes = nullptr;
    double *d_uniform_leaves = nullptr;
    // kernel specialised for the model (TREE_ENS_CODEGEN), used by tree_ens_predict
    hipModule_t cg_module = nullptr;
    hipFunction_t cg_fn = nullptr;
    // Small batches: partial sums of the tile splits, reused by every eager call (no
    // allocation per call). Eager calls from different streams are ordered with an event, so
    // they never share the scratch at the same time.
    double *d_scratch = nullptr;
    hipEvent_t scratch_done = nullptr;
    mutable std::mutex scratch_mu;
    mutable bool scratch_used = false;
    // Calls captured into a HIP graph take none of the above (a replay is ordered with nothing
    // the handle records): each captured call gets a buffer of its own for its partial sums and
    // threshold codes, allocated when it is captured and kept until destroy.
    mutable std::mutex capture_mu;
    mutable std::vector<void *> capture_bufs;
    // Kernel timing (tree_ens_kernel_timing): while `timing` is set, eager predicts record
    // t_start[i] / t_stop[i] around the i-th scoring launch, i < t_used <= kMaxTimedLaunches.
    mutable std::mutex timing_mu;
    mutable bool timing = false;
    mutable std::vector<hipEvent_t> t_start, t_stop;
    mutable int32_t t_used = 0;
    // launch shapes of the last batch sizes seen (callers usually repeat a few), by the kind of
    // work (a treeens::Work, or kUniformWork) and the batch's blocks, replaced in turn
    struct Shape {
        int work = -1;
        int64_t blocks = 0;
        treeens::LaunchShape shape;
    };
    mutable std::mutex shape_mu;
    mutable Shape shapes[8];
    mutable unsigned next_shape = 0;
    mutable std::atomic<int32_t> last_path{TREE_ENS_PATH_NONE};
};

namespace {
constexpr size_t kScratchDoubles = size_t(1) << 17; // 1 MiB of split partials
constexpr int kMaxTimedLaunches = 1024;             // event pairs of tree_ens_kernel_timing

// Scratch of the allocation-free entry point (tree_ens_predict_noalloc): split partial sums and
// threshold codes in one static array, which every device the library runs on holds until the
// process ends. In host code `scratch` is only a stand-in for the symbol: its device address
// comes from hipGetSymbolAddress, once per device, and only that address reaches a kernel or a
// copy.
constexpr size_t kStaticScratchBytes = size_t(16) << 20; // 16 MiB
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

constexpr int kMaxDevices = 64;
std::mutex g_static_mu;
unsigned char *g_static_ptr[kMaxDevices] = {};

// Device address of `scratch` on `device` (the current device), looked up on the first use.
int static_scratch(int device, unsigned char **out) {
    if (device < 0 || device >= kMaxDevices)
        return fail(TREE_ENS_E_DEVICE, "device index beyond the allocation-free scratch table");
    std::lock_guard<std::mutex> lock(g_static_mu);
    if (!g_static_ptr[device]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p)
            return hip_fail(e != hipSuccess ? e : hipErrorInvalidSymbol, "hipGetSymbolAddress(scratch)");
        g_static_ptr[device] = static_cast<unsigned char *>(p);
    }
    *out = g_static_ptr[device];
    return TREE_ENS_OK;
}
} // namespace

namespace {

void free_device(tree_ens *h) {
    (void)hipFree(h->d_model);
    if (h->scratch_done)
        (void)hipEventDestroy(h->scratch_done);
    for (void *b : h->capture_bufs)
        (void)hipFree(b);
    for (hipEvent_t ev : h->t_start)
        (void)hipEventDestroy(ev);
    for (hipEvent_t ev : h->t_stop)
        (void)hipEventDestroy(ev);
    if (h->cg_module)
        (void)hipModuleUnload(h->cg_module);
}

// Compile generated HIP source for gfx950 with hiprtc (host only: no device is needed).
int compile_codegen(const std::string &src, std::vector<char> &code, std::string &err) {
    hiprtcProgram prog;
    hiprtcResult r = hiprtcCreateProgram(&prog, src.c_str(), "tree_ens_cg.hip", 0, nullptr, nullptr);
    if (r != HIPRTC_SUCCESS) {
        err = std::string("hiprtcCreateProgram: ") + hiprtcGetErrorString(r);
        return TREE_ENS_E_DEVICE;
    }
    // the same code-generation settings as the library's own kernels
    const char *opts[] = {"--offload-arch=gfx950", "-O3", "-fno-gpu-flush-denormals-to-zero",
                          "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"};
    r = hiprtcCompileProgram(prog, int(sizeof opts / sizeof opts[0]), opts);
    if (r != HIPRTC_SUCCESS) {
        size_t n = 0;
        std::string log;
        if (hiprtcGetProgramLogSize(prog, &n) == HIPRTC_SUCCESS && n > 1) {
            log.resize(n);
            if (hiprtcGetProgramLog(prog, &log[0]) != HIPRTC_SUCCESS)
                log.clear();
        }
        err = std::string("code generation: hiprtc failed (") + hiprtcGetErrorString(r) + ")" +
              (log.empty() ? "" : ": " + log.substr(0, 2000));
        (void)hiprtcDestroyProgram(&prog);
        return TREE_ENS_E_DEVICE;
    }
    size_t size = 0;
    r = hiprtcGetCodeSize(prog, &size);
    if (r == HIPRTC_SUCCESS) {
        code.resize(size);
        r = hiprtcGetCode(prog, code.data());
    }
    (void)hiprtcDestroyProgram(&prog);
    if (r != HIPRTC_SUCCESS) {
        err = std::string("code generation: ") + hiprtcGetErrorString(r);
        return TREE_ENS_E_DEVICE;
    }
    return TREE_ENS_OK;
}

// The model's device arrays, in one allocation: the small ones (first, gathered) take one copy together,
// the others one each.
class DeviceArrays {
public:
    // src must outlive upload(); count elements from the first-th on
    template <typename D, typename S>
    void add(D **dst, const std::vector<S> &src, size_t first = 0) {
        static_assert(sizeof(D) == sizeof(S), "same records");
        reserve(reinterpret_cast<void **>(dst), src.data() + first, (src.size() - first) * sizeof(S));
    }
    void reserve(void **dst, const void *src, size_t bytes) { items_.push_back(Item{dst, src, bytes, 0}); }

    hipError_t upload(void **base) {
        std::stable_partition(items_.begin(), items_.end(), [](const Item &i) { return i.src && i.bytes <= kSmall; });
        size_t total = 0, small = 0;
        for (Item &i : items_) {
            i.at = total;
            total += (std::max<size_t>(i.bytes, 1) + 255) & ~size_t(255);
            if (i.src && i.bytes <= kSmall)
                small = total;
        }
        hipError_t e = hipMalloc(base, std::max<size_t>(total, 256));
        if (e != hipSuccess)
            return e;
        unsigned char *at = static_cast<unsigned char *>(*base);
        std::vector<unsigned char> gathered(small);
        for (const Item &i : items_) {
            *i.dst = at + i.at;
            if (!i.src || i.bytes == 0)
                continue;
            if (i.bytes <= kSmall)
                std::memcpy(gathered.data() + i.at, i.src, i.bytes);
            else if (e == hipSuccess)
                e = hipMemcpy(at + i.at, i.src, i.bytes, hipMemcpyHostToDevice);
        }
        if (e == hipSuccess && small > 0)
            e = hipMemcpy(at, gathered.data(), small, hipMemcpyHostToDevice);
        return e;
    }

private:
    static constexpr size_t kSmall = size_t(256) << 10;
    struct Item {
        void **dst;
        const void *src;
        size_t bytes, at;
    };
    std::vector<Item> items_;
};

// The pool's memory (scratch.hpp) on the current device. The capture mode is relaxed where another
// stream may be capturing: none of this is part of a capture.
struct HipScratch {
    using Stream = hipStream_t;
    using Event = hipEvent_t;
    struct Relaxed {
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        Relaxed() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
        ~Relaxed() { (void)hipThreadExchangeStreamCaptureMode(&mode); }
    };
    static bool ok(hipError_t e) {
        if (e != hipSuccess)
            (void)hipGetLastError(); // the caller falls back
        return e == hipSuccess;
    }
    void *allocate(size_t bytes) {
        const Relaxed relaxed;
        void *p = nullptr;
        return ok(hipMalloc(&p, bytes)) ? p : nullptr;
    }
    void release(void *p, Event done) {
        const Relaxed relaxed;
        ok(hipEventSynchronize(done));
        ok(hipFree(p));
        ok(hipEventDestroy(done));
    }
    bool make_event(Event *ev) { return ok(hipEventCreateWithFlags(ev, hipEventDisableTiming)); }
    bool record(Event ev, Stream s) { return ok(hipEventRecord(ev, s)); }
    bool wait(Stream s, Event ev) { return ok(hipStreamWaitEvent(s, ev, 0)); }
    void finish(Stream s) { ok(hipStreamSynchronize(s)); }
};
using Pool = treeens::ScratchPool<HipScratch>;

// The device's pool; never destroyed (handles may outlive static objects), empty without handles.
Pool *pool_of(int device) {
    static Pool *const pools = new (std::nothrow) Pool[kMaxDevices];
    return pools && device >= 0 && device < kMaxDevices ? pools + device : nullptr;
}

// The handle's kept shape for this work and number of blocks, or that of `choose`.
constexpr int kUniformWork = 100;
constexpr int kUniformRule = 101; // (level: whether it pays; by documents)
template <typename Choose>
LaunchShape kept_shape(const tree_ens *h, int work, int64_t n_blocks, Choose &&choose) {
    std::lock_guard<std::mutex> lock(h->shape_mu);
    for (const tree_ens::Shape &s : h->shapes)
        if (s.work == work && s.blocks == n_blocks)
            return s.shape;
    const LaunchShape shape = choose();
    h->shapes[h->next_shape++ % (sizeof h->shapes / sizeof h->shapes[0])] = tree_ens::Shape{work, n_blocks, shape};
    return shape;
}

// Where a call's scratch (split partial sums, threshold codes, leaf positions) comes from.
enum class ScratchSource {
    kHandle, // the handle's shared buffer or the device's pool (eager calls), a buffer
             // of the call's own kept by the handle (calls captured into a graph)
    kStatic, // the library's static device array only (tree_ens_predict_noalloc)
};

bool capturing(hipStream_t stream) {
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(stream, &cap) != hipSuccess)
        cap = hipStreamCaptureStatusNone;
    (void)hipGetLastError();
    return cap != hipStreamCaptureStatusNone;
}

// Device memory of one call on `stream`. Eager calls: from the pool, or a stream-ordered allocation
// where the pool has none to lend; it goes back when the object ends, after the work enqueued until then.
// Captured calls: a buffer of the call's own, kept by the handle, so that replays of the graph never
// share it with eager calls or other graphs. Allocation-free calls: the static array.
class CallScratch {
public:
    CallScratch(const tree_ens *h, hipStream_t stream, ScratchSource source)
        : h_(h), pool_(pool_of(h->device)), stream_(stream), source_(source) {}
    CallScratch(const CallScratch &) = delete;
    ~CallScratch() {
        if (block_)
            pool_->give(block_);
        else if (async_)
            (void)hipFreeAsync(async_, stream_);
    }
    // nullptr: no memory, `error` says why
    unsigned char *take(size_t bytes) {
        if (source_ == ScratchSource::kStatic) {
            unsigned char *base = nullptr;
            error = hipErrorOutOfMemory;
            return bytes <= kStaticScratchBytes && static_scratch(h_->device, &base) == TREE_ENS_OK ? base : nullptr;
        }
        if (capturing(stream_))
            return take_captured(bytes);
        if (pool_ && (block_ = pool_->lend(bytes, stream_)))
            return static_cast<unsigned char *>(block_->p);
        error = hipMallocAsync(&async_, bytes, stream_);
        if (error != hipSuccess && pool_ && pool_->trim())
            error = hipMallocAsync(&async_, bytes, stream_);
        if (error != hipSuccess) {
            async_ = nullptr;
            (void)hipGetLastError();
        }
        return static_cast<unsigned char *>(async_);
    }
    hipError_t error = hipSuccess;

private:
    unsigned char *take_captured(size_t bytes) {
        std::lock_guard<std::mutex> lock(h_->capture_mu);
        try {
            h_->capture_bufs.reserve(h_->capture_bufs.size() + 1);
        } catch (const std::bad_alloc &) {
            error = hipErrorOutOfMemory;
            return nullptr;
        }
        void *buf = HipScratch().allocate(bytes);
        if (!buf && pool_ && pool_->trim())
            buf = HipScratch().allocate(bytes);
        if (!buf) {
            error = hipErrorOutOfMemory;
            return nullptr;
        }
        h_->capture_bufs.push_back(buf);
        return static_cast<unsigned char *>(buf);
    }

    const tree_ens *h_;
    Pool *pool_;
    hipStream_t stream_;
    ScratchSource source_;
    Pool::Block *block_ = nullptr;
    void *async_ = nullptr;
};

struct DeviceGuard {
    int prev = -1;
    hipError_t err = hipSuccess;
    explicit DeviceGuard(int dev) {
        err = hipGetDevice(&prev);
        if (err == hipSuccess && prev != dev)
            err = hipSetDevice(dev);
        else
            prev = -1;
    }
    ~DeviceGuard() {
        if (prev >= 0)
            (void)hipSetDevice(prev);
    }
};

int check_predict_args(const tree_ens *h, const float *X, int64_t n_docs, int32_t n_features,
                       const void *out) {
    if (!h)
        return fail(TREE_ENS_E_ARG, "handle is NULL");
    if (n_docs < 0)
        return fail(TREE_ENS_E_ARG, "n_docs must be >= 0");
    if (n_docs == 0)
        return TREE_ENS_OK;
    if (!X || !out)
        return fail(TREE_ENS_E_ARG, "X or the output pointer is NULL");
    if ((reinterpret_cast<uintptr_t>(X) & 3u) != 0 || (reinterpret_cast<uintptr_t>(out) & 3u) != 0)
        return fail(TREE_ENS_E_ARG, "X and the output must be 4-byte aligned");
    if (n_features < h->n_cols)
        return fail(TREE_ENS_E_SHAPE, "documents carry " + std::to_string(n_features) +
                                          " features; the model reads feature " +
                                          std::to_string(h->n_cols - 1));
    if (n_features < 1)
        return fail(TREE_ENS_E_SHAPE, "n_features must be >= 1");
    return TREE_ENS_OK;
}

// Sums of leaf vectors from the rows the walk left in pos[block][packed tree][DL documents] (the lower
// 16 bits of each): up to 4 * NV outputs in one pass over the trees. A workgroup takes 64 documents
// (lanes), each of its waves a run of trees; kRowTrees trees' rows load together, their positions
// while the trees before them are summed. Waves' sums are added in wave order.
// Bound by the texture addresser: 25 cycles per 16-byte gather of a wave keep it 96% busy while a CU
// has waves, and that is 69% of the launch (782 workgroups, 512 at a time): 50,000 documents, 1,000
// trees, 8 outputs in 95 us, against 110 us for each of the two walks it replaces, next to one
// walk of 83 us that stores the rows.
constexpr int kRowThreads = 1024;
constexpr int kRowTrees = 4;
template <int DL, int NV>
__global__ void __launch_bounds__(kRowThreads, 8)
sum_rows_kernel(const uint16_t *__restrict__ pos, int64_t n_docs, int32_t n_trees, const uint32_t *__restrict__ tree_row0,
                const float4 *__restrict__ leaf_vec, int32_t stride4, int32_t chunk, int32_t n_out, double scale,
                float *__restrict__ scores) {
    constexpr int kWaves = kRowThreads / 64;
    __shared__ double red[4 * NV][kWaves][64];
    const int lane = int(threadIdx.x) & 63;
    const int wave = __builtin_amdgcn_readfirstlane(int(threadIdx.x) >> 6);
    const int64_t doc = min<int64_t>(int64_t(blockIdx.x) * 64 + lane, n_docs - 1);
    const uint16_t *my = pos + (doc / DL) * n_trees * DL + doc % DL;
    const int lo = int(int64_t(n_trees) * wave / kWaves), hi = int(int64_t(n_trees) * (wave + 1) / kWaves);
    double acc[4 * NV];
#pragma unroll
    for (int c = 0; c < 4 * NV; ++c)
        acc[c] = 0.0;
    uint32_t next[kRowTrees], first[kRowTrees];
    auto fetch = [&](int t) { // past the last tree: the last one again, not used
#pragma unroll
        for (int u = 0; u < kRowTrees; ++u) {
            next[u] = my[int64_t(min(t + u, n_trees - 1)) * DL];
            first[u] = tree_row0[min(t + u, n_trees - 1)];
        }
    };
    auto add = [&](const float4 (&v)[NV]) {
#pragma unroll
        for (int c = 0; c < NV; ++c) {
            acc[4 * c] += double(v[c].x);
            acc[4 * c + 1] += double(v[c].y);
            acc[4 * c + 2] += double(v[c].z);
            acc[4 * c + 3] += double(v[c].w);
        }
    };
    auto load_row = [&](float4 (&v)[NV], int u) {
        const uint32_t row = first[u] + ((next[u] - first[u]) & 0xFFFFu);
#pragma unroll
        for (int c = 0; c < NV; ++c)
            v[c] = leaf_vec[int64_t(row) * stride4 + chunk + c];
    };
    fetch(lo);
    int t = lo;
    for (; t + kRowTrees <= hi; t += kRowTrees) {
        float4 v[kRowTrees][NV];
#pragma unroll
        for (int u = 0; u < kRowTrees; ++u)
            load_row(v[u], u);
        fetch(t + kRowTrees);
#pragma unroll
        for (int u = 0; u < kRowTrees; ++u)
            add(v[u]);
    }
#pragma unroll
    for (int u = 0; u < kRowTrees - 1; ++u) {
        if (t + u < hi) {
            float4 v[NV];
            load_row(v, u);
            add(v);
        }
    }
#pragma unroll
    for (int c = 0; c < 4 * NV; ++c)
        red[c][wave][lane] = acc[c];
    __syncthreads();
    const int c = wave, oc = 4 * chunk + c; // one wave per output
    if (c < 4 * NV && oc < n_out && int64_t(blockIdx.x) * 64 + lane < n_docs) {
        double sum = 0.0;
        for (int w = 0; w < kWaves; ++w)
            sum += red[c][w][lane];
        scores[doc * n_out + oc] = float(sum * scale);
    }
}

// Threshold codes of all documents, rows of n_cols.
void launch_coding(const tree_ens *h, hipStream_t stream, const float *X, int64_t n_docs, int32_t n_features,
                   int32_t code_shift, uint16_t *codes) {
    // documents per coding workgroup: enough workgroups to fill the GPU twice over, but
    // each one long enough to pay for loading its chunk's thresholds into LDS
    int64_t per_wg = 256;
    while (per_wg < 4096 && ((n_docs + per_wg - 1) / per_wg) * h->n_code_chunks > 4 * kNumCus)
        per_wg *= 2;
    const int64_t code_blocks = (n_docs + per_wg - 1) / per_wg;
    hipLaunchKernelGGL(code_kernel, dim3(unsigned((code_blocks + kXcds - 1) / kXcds * kXcds * h->n_code_chunks)),
                       dim3(kCodeThreads), 0, stream, X, n_docs, n_features, h->n_cols, int32_t(per_wg),
                       h->d_code_search, h->d_code_chunks, h->n_code_chunks, code_shift, codes);
}

// Kernel timing (tree_ens_kernel_timing): the event pair of the next scoring launch on `stream`, if
// launches are being timed (eager calls only).
struct TimedLaunch {
    hipEvent_t start = nullptr, stop = nullptr;
    TimedLaunch(const tree_ens *h, hipStream_t stream) {
        std::lock_guard<std::mutex> lock(h->timing_mu);
        if (h->timing && h->t_used < int32_t(h->t_start.size())) {
            hipStreamCaptureStatus tc = hipStreamCaptureStatusNone;
            if (hipStreamIsCapturing(stream, &tc) != hipSuccess)
                tc = hipStreamCaptureStatusActive;
            (void)hipGetLastError();
            if (tc == hipStreamCaptureStatusNone) {
                start = h->t_start[size_t(h->t_used)];
                stop = h->t_stop[size_t(h->t_used)];
                h->t_used++;
            }
        }
    }
};

// Tail blocks' split partial sums to scores, in a fixed order.
hipError_t launch_reduce(hipStream_t stream, const double *partials, int splits, int64_t n_entries, const ReduceOut &out) {
    if (splits <= 64)
        hipLaunchKernelGGL(reduce_partials_thread_kernel, dim3(unsigned((n_entries + 255) / 256)), dim3(256), 0, stream,
                           partials, splits, n_entries, out);
    else
        hipLaunchKernelGGL(reduce_partials_wave_kernel, dim3(unsigned(n_entries)), dim3(64), 0, stream, partials, splits,
                           n_entries, out);
    return hipGetLastError();
}

// MODE kModeScore writes scores; kModeVector writes scores [n_docs][n_outputs] (one launch per
// four outputs); kModeLeaves writes leaf_ids [n_docs][n_trees]; kModeUsage writes per-document
// feature counts into leaf_ids and, if masks is not NULL, the bitmasks (rows of mask_words
// words).
// Memory of a call that launches the walk as its first step.
struct WalkBuffers {
    uint16_t *leaf_pos = nullptr; // leaf positions or rows go here (kModeLeaves, kModeRows)
    uint16_t *codes = nullptr;    // room for the threshold codes (coded models)
};

template <int MODE>
int launch_predict(const tree_ens *h, hipStream_t stream, const float *X, int64_t n_docs,
                   int32_t n_features, float *scores, int32_t *leaf_ids, uint32_t *masks = nullptr,
                   int32_t mask_words = 0, ScratchSource source = ScratchSource::kHandle,
                   const WalkBuffers &given = {}) {
    constexpr bool kScores = MODE == kModeScore || MODE == kModeVector; // split partial sums
    // entries per document in the partial sums, and launches (four outputs each)
    const int comps = MODE == kModeVector ? kVecPerLaunch : 1;
    const int n_chunks = MODE == kModeVector ? (h->n_outputs + kVecPerLaunch - 1) / kVecPerLaunch : 1;
    if (MODE == kModeVector && h->plan.tile_bytes < kThreads * kVecPerLaunch * int(sizeof(double)))
        return fail(TREE_ENS_E_ARG, "the tile slot cannot hold the vector reduction");
    const int dl = h->plan.docs_per_block;
    const int64_t n_blocks = (n_docs + dl - 1) / dl;
    if (n_blocks > 0x7fffffff)
        return fail(TREE_ENS_E_ARG, "too many documents for one launch");
    LaunchShape shape;
    int32_t usage_off = h->plan.usage_off;
    if (MODE == kModeUsage || MODE == kModeUsageSlot) {
        // one workgroup walks every tile of its block: its bitmasks are complete in LDS
        shape = LaunchShape{0, n_blocks, 1};
        const int64_t mask_bytes = int64_t((h->n_cols + 31) / 32) * dl * 4;
        if (MODE == kModeUsageSlot) {
            usage_off = h->usage_slot_off;
            if (usage_off < 0 || usage_off + mask_bytes > h->plan.zero_rec)
                return fail(TREE_ENS_E_ARG, "feature bitmasks do not fit the tile slot");
        } else {
            const int64_t lds_end = h->plan.lds_bytes == treeens::kLdsPerCu
                                        ? treeens::kLdsPerCu
                                        : treeens::kLdsPerCu / 2 + treeens::kUsageHalfBytes;
            if (usage_off + mask_bytes > lds_end)
                return fail(TREE_ENS_E_ARG, "feature bitmasks do not fit the LDS plan");
        }
    } else {
        const Work work = MODE == kModeScore ? Work::kScores : MODE == kModeVector ? Work::kVector : Work::kPositions;
        shape = kept_shape(h, int(work), n_blocks, [&] { return choose_launch(h->facts, work, n_blocks); });
    }
    {
        // grid of the chosen shape (the no-split shape the allocation-free path may fall back
        // to is never larger): every tail block split into the shape's splits, plus the padding
        // to whole XCD columns
        const int64_t tail_blocks = n_blocks - shape.head;
        const int64_t tail_slots = shape.head > 0 ? (tail_blocks + kXcds - 1) / kXcds * kXcds : tail_blocks;
        if (shape.head + tail_slots * shape.splits > 0x7fffffff)
            return fail(TREE_ENS_E_ARG, "too many documents for one launch");
    }
    // compact packets, where the model has them, for every mode but the feature trace
    const bool cp = h->cp_k > 0 && MODE != kModeUsage && MODE != kModeUsageSlot;
    ScoreFn fn = pick_kernel<MODE>(h->plan, cp);
    if (!fn)
        return fail(TREE_ENS_E_ARG, "unsupported document block size");
    hipError_t e = hipSuccess;
    // scratch of this call: split partial sums (score modes with splits) and threshold codes
    // (coded models), each 256-byte aligned
    auto align256 = [](size_t b) { return (b + 255) & ~size_t(255); };
    const size_t codes_bytes = h->plan.coded && !given.codes ? align256(size_t(n_docs) * size_t(h->n_cols) * sizeof(uint16_t)) : 0;
    auto partial_bytes = [&](const LaunchShape &sh) {
        return kScores && sh.splits > 1
                   ? align256(size_t(sh.splits) * size_t(n_docs - sh.head * dl) * size_t(comps) * sizeof(double))
                   : size_t(0);
    };
    bool shared_scratch = false; // partials in the handle's event-ordered buffer
    CallScratch lent(h, stream, source);
    std::unique_lock<std::mutex> scratch_lock;
    if (source == ScratchSource::kStatic) {
        // a shape whose partials do not fit takes no splits (every workgroup walks all tiles of its
        // block); codes that do not fit are an error
        if (codes_bytes > kStaticScratchBytes)
            return fail(TREE_ENS_E_ARG,
                        "the batch's threshold codes (" + std::to_string(codes_bytes) +
                            " bytes) exceed the allocation-free scratch of " +
                            std::to_string(kStaticScratchBytes) + " bytes");
        if (codes_bytes + partial_bytes(shape) > kStaticScratchBytes)
            shape = LaunchShape{0, n_blocks, 1};
    }
    const size_t pb = partial_bytes(shape);
    unsigned char *buf = nullptr;
    if (source == ScratchSource::kHandle && pb > 0 && pb <= kScratchDoubles * sizeof(double) && codes_bytes == 0 &&
        !capturing(stream)) {
        scratch_lock = std::unique_lock<std::mutex>(h->scratch_mu);
        // also where the last call named the same stream: one handle value can stand for several (each
        // thread's own default stream, a destroyed stream's)
        if (h->scratch_used) {
            e = hipStreamWaitEvent(stream, h->scratch_done, 0);
            if (e != hipSuccess)
                return hip_fail(e, "hipStreamWaitEvent");
        }
        buf = reinterpret_cast<unsigned char *>(h->d_scratch);
        shared_scratch = true;
    } else if (codes_bytes + pb > 0) {
        buf = lent.take(codes_bytes + pb);
        if (!buf)
            return hip_fail(lent.error, "scratch of the call");
    }
    uint16_t *codes = given.codes ? given.codes : reinterpret_cast<uint16_t *>(buf);
    double *partials = pb > 0 ? reinterpret_cast<double *>(buf + codes_bytes) : nullptr;
    const int level = shape.level, splits = shape.splits;
    const int64_t tail_docs = n_docs - shape.head * dl;
    // tail blocks after a head are laid out in whole XCD columns (see the kernel)
    const int64_t tail_blocks = n_blocks - shape.head;
    const int64_t tail_slots = shape.head > 0 ? (tail_blocks + kXcds - 1) / kXcds * kXcds : tail_blocks;
    const int64_t n_wgs = shape.head + tail_slots * splits;
    // walker packets (pk_recs > 0) stand in for the tiles: n_tiles is then packets per walker.
    // The feature trace of one-workgroup plans keeps the shared tiles: its bitmasks sit past
    // their zero record, where the packets' sub-slots reach.
    const bool pk = h->pk_recs > 0 && !(MODE == kModeUsage && h->plan.lds_bytes == treeens::kLdsPerCu);
    const uint2 *images = cp   ? reinterpret_cast<const uint2 *>(h->d_cpackets)
                          : pk ? h->d_packets
                               : h->d_images + h->level_image_off[level];
    const uint32_t *tile_recs = h->d_tile_recs + (pk || cp ? 0 : h->level_begin[level]);
    const int n_tiles = cp   ? h->cp_per_walker
                        : pk ? h->pk_per_walker
                             : h->level_begin[level + 1] - h->level_begin[level];
    const int32_t slot_recs = cp ? treeens::kCompactPacketBytes / 8 : pk ? h->pk_recs : h->level_slot_recs[level];
    (void)hipGetLastError();
    // coded models: one pass turns the float features into 16-bit threshold codes
    const void *docs = X;
    int32_t row_stride = n_features;
    if (h->plan.coded) {
        launch_coding(h, stream, X, n_docs, n_features, cp ? treeens::kCompactCodeShift : 0, codes);
        docs = codes;
        row_stride = h->n_cols;
    }
    const double scale = 1.0 / double(h->n_bags);
    const int n_out = MODE == kModeVector ? h->n_outputs : 1;
    for (int chunk = 0; chunk < n_chunks && e == hipSuccess; ++chunk) {
        const TimedLaunch timed(h, stream);
        if (timed.start && (e = hipEventRecord(timed.start, stream)) != hipSuccess)
            break;
        hipLaunchKernelGGL(fn, dim3(unsigned(n_wgs)), dim3(kThreads), 0, stream, docs, n_docs,
                           row_stride, h->n_cols, images, slot_recs, tile_recs,
                           n_tiles, int32_t(shape.head), splits, h->plan.xs_bytes,
                           pk ? h->pk_zero_rec : h->plan.zero_rec,
                           partials, scores, leaf_ids, h->d_orig_id, h->d_tree_node_off,
                           h->d_tree_orig, h->n_trees, masks, mask_words, usage_off,
                           reinterpret_cast<const float4 *>(h->d_leaf_vec), h->vec_stride / 4, n_out,
                           chunk, scale, cp ? treeens::kCompactPacketBytes / 8 : pk ? h->pk_recs : 0,
                           h->d_big, h->n_small, h->big_off0, h->d_cleaf, h->d_cleaf_id, given.leaf_pos);
        e = hipGetLastError();
        if (e == hipSuccess && timed.stop)
            e = hipEventRecord(timed.stop, stream);
        if (e == hipSuccess && partials) {
            // the tail blocks' entries, in [doc][component] order
            const int64_t n_entries = tail_docs * comps;
            const ReduceOut out{scores + shape.head * dl * n_out, comps, n_out, chunk * comps, scale};
            e = launch_reduce(stream, partials, splits, n_entries, out);
        }
    }
    if (shared_scratch) {
        // the next eager call waits for this one's reduction
        if (e == hipSuccess)
            e = hipEventRecord(h->scratch_done, stream);
        h->scratch_used = true;
    }
    h->last_path.store(given.leaf_pos ? TREE_ENS_PATH_ROWS : TREE_ENS_PATH_WALK, std::memory_order_relaxed);
    if (e != hipSuccess)
        return hip_fail(e, "kernel launch");
    return TREE_ENS_OK;
}

// Scores of a shallow model by uniform evaluation, or of a coded one by terminal packets. `taken` is
// false (and nothing was launched) for calls that keep the walk (uniform_pays, term_pays), and when the
// scratch cannot be had (allocation-free calls: batches beyond the static array).
// Launch shape of `n_docs` coded documents: uniform blocks or terminal packets.
LaunchShape coded_shape(const tree_ens *h, bool uniform, int64_t n_docs) {
    const int docs = uniform ? h->uniform.docs_per_block : 64;
    const int64_t n_blocks = (n_docs + docs - 1) / docs;
    return kept_shape(h, uniform ? kUniformWork : int(Work::kTerminal), n_blocks, [&] {
        LaunchShape shape = uniform ? treeens::uniform_shape(h->uniform, n_docs)
                                    : choose_launch(h->facts, Work::kTerminal, n_blocks);
        if (shape.splits == 1)
            shape.head = n_blocks;
        return shape;
    });
}

// Bytes of a chunk's codes.
constexpr int64_t kCodeChunkBytes = int64_t(256) << 20;

int launch_coded_predict(const tree_ens *h, hipStream_t stream, const float *X, int64_t n_docs, int32_t n_features,
                         float *scores, ScratchSource source, bool *taken) {
    *taken = false;
    const bool uniform =
        h->uniform.depth > 0 &&
        kept_shape(h, kUniformRule, n_docs, [&] { return LaunchShape{uniform_pays(h->facts, n_docs)}; }).level != 0;
    const bool term = !uniform && term_pays(h->facts, n_docs);
    if ((!uniform && !term) || n_docs > int64_t(64) * 0x7ffffff)
        return TREE_ENS_OK;
    // Shallow models of any batch borrow a bounded amount: their documents go in chunks of whole rounds
    // (a block for every CU) whose codes take at most kCodeChunkBytes; a chunk but the last has no
    // tail to split (20,000 trees, 1,000,000 documents: 6.47 ms in two chunks, 6.48 in one). Coded models
    // take the codes of the whole batch, as every call of theirs does (5,000 trees of 256 leaves, 700
    // features, 1,000,000 documents: 15.46 ms whole, 15.69 in seven chunks).
    const int docs = uniform ? h->uniform.docs_per_block : 64;
    const int64_t round = int64_t(docs) * kNumCus, row_bytes = int64_t(h->n_cols) * int64_t(sizeof(uint16_t));
    const int64_t per =
        uniform ? std::min(n_docs, std::max<int64_t>(1, kCodeChunkBytes / (round * row_bytes)) * round) : n_docs;
    auto align256 = [](size_t b) { return (b + 255) & ~size_t(255); };
    const size_t codes_bytes = align256(size_t(per * row_bytes));
    const int64_t last_docs = n_docs - (n_docs - 1) / per * per; // 1 .. per
    const LaunchShape whole = coded_shape(h, uniform, per);
    const LaunchShape last = last_docs == per ? whole : coded_shape(h, uniform, last_docs);
    // documents past the head blocks (a split launch has some)
    auto tail_docs = [&](const LaunchShape &sh, int64_t nd) { return std::max<int64_t>(0, nd - sh.head * docs); };
    auto partial_bytes = [&](const LaunchShape &sh, int64_t nd) {
        return sh.splits > 1 ? size_t(sh.splits) * size_t(tail_docs(sh, nd)) * sizeof(double) : size_t(0);
    };
    CallScratch lent(h, stream, source);
    unsigned char *buf = lent.take(codes_bytes + std::max(partial_bytes(whole, per), partial_bytes(last, last_docs)));
    if (!buf)
        return TREE_ENS_OK;
    (void)hipGetLastError();
    *taken = true;
    h->last_path.store(uniform ? TREE_ENS_PATH_UNIFORM : TREE_ENS_PATH_TERMINAL, std::memory_order_relaxed);
    uint16_t *codes = reinterpret_cast<uint16_t *>(buf);
    double *partials = reinterpret_cast<double *>(buf + codes_bytes);
    const double scale = 1.0 / double(h->n_bags);
    hipError_t e = hipSuccess;
    for (int64_t doc0 = 0; doc0 < n_docs && e == hipSuccess; doc0 += per) {
        const int64_t nd = std::min(per, n_docs - doc0);
        const LaunchShape &sh = nd == per ? whole : last;
        float *out = scores + doc0;
        launch_coding(h, stream, X + doc0 * n_features, nd, n_features, uniform ? 0 : treeens::kCompactCodeShift, codes);
        const TimedLaunch timed(h, stream);
        if (timed.start && (e = hipEventRecord(timed.start, stream)) != hipSuccess)
            break;
        if (uniform)
            treeens::launch_uniform(h->uniform, stream, codes, nd, h->n_cols, h->d_uniform_nodes, h->d_uniform_leaves,
                                    sh, partials, out, scale);
        else
            treeens::launch_term(h->term, stream, codes, nd, h->n_cols, h->d_term_packets, h->d_term_slots, sh.head,
                                 sh.splits, partials, out, scale);
        e = hipGetLastError();
        if (e == hipSuccess && timed.stop)
            e = hipEventRecord(timed.stop, stream);
        if (e == hipSuccess && sh.splits > 1)
            e = launch_reduce(stream, partials, sh.splits, tail_docs(sh, nd),
                              ReduceOut{out + sh.head * docs, 1, 1, 0, scale});
    }
    return e == hipSuccess ? TREE_ENS_OK : hip_fail(e, "kernel launch");
}

// Leaf ids. Large outputs: the walk stores 16-bit leaf positions in its own (block, packed tree)
// order and leaf_ids_kernel turns them into the output's rows, in chunks of documents whose
// positions (and codes) take at most kPositionBytes (they stay in the last-level cache). 1,000 trees of 32
// leaves, 30,011 documents: 383 us with ids stored by the walk, 103 us this way (62 us the walk,
// 37 us the second kernel at 4.8 TB/s).
// Where that does not pay (leaves_direct), in calls captured into a graph and where the scratch cannot
// be had, the walk stores the ids directly.
// The walk's leaf positions in chunks of documents (MODE: kModeLeaves or kModeRows), each chunk
// followed by `then(pos, first document, documents)`. `taken` is false (and nothing was launched)
// when the scratch cannot be had.
template <int MODE, typename Then>
int walk_positions(const tree_ens *h, hipStream_t stream, const float *X, int64_t n_docs, int32_t n_features,
                   ScratchSource source, bool *taken, Then &&then) {
    const int dl = h->plan.docs_per_block;
    const int64_t n_blocks = (n_docs + dl - 1) / dl;
    // positions and, for coded models, threshold codes
    const int64_t pos_bytes = int64_t(h->n_trees) * dl * int64_t(sizeof(uint16_t));
    const int64_t block_bytes = pos_bytes + (h->plan.coded ? int64_t(h->n_cols) * dl * int64_t(sizeof(uint16_t)) : 0);
    const int64_t per = std::min(n_blocks, std::max<int64_t>(1, kPositionBytes / block_bytes / (64 / dl) * (64 / dl)));
    *taken = false;
    CallScratch lent(h, stream, source);
    unsigned char *buf = lent.take(size_t(per * block_bytes));
    if (!buf)
        return TREE_ENS_OK;
    *taken = true;
    // block_bytes are a multiple of 16 (8 documents at least): so is the codes' place
    uint16_t *pos = reinterpret_cast<uint16_t *>(buf);
    const WalkBuffers given{pos, h->plan.coded ? reinterpret_cast<uint16_t *>(buf + per * pos_bytes) : nullptr};
    int rc = TREE_ENS_OK;
    for (int64_t b = 0; b < n_blocks && rc == TREE_ENS_OK; b += per) {
        const int64_t doc0 = b * dl, nd = std::min(std::min(per, n_blocks - b) * dl, n_docs - doc0);
        rc = launch_predict<MODE>(h, stream, X + doc0 * n_features, nd, n_features, nullptr, nullptr, nullptr, 0,
                                  source, given);
        if (rc != TREE_ENS_OK)
            break;
        then(pos, doc0, nd);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess)
            rc = hip_fail(e, "kernel launch");
    }
    return rc;
}

// The kernel for a plan's document blocks.
template <typename Fn>
Fn pick_block(int dl, Fn f64, Fn f32, Fn f16, Fn f8) {
    return dl == 64 ? f64 : dl == 32 ? f32 : dl == 16 ? f16 : f8;
}

int launch_leaves(const tree_ens *h, hipStream_t stream, const float *X, int64_t n_docs,
                  int32_t n_features, int32_t *leaf_ids) {
    bool taken = false;
    if (!leaves_direct(h->facts, n_docs) && !capturing(stream)) {
        const int dl = h->plan.docs_per_block;
        // compact packets store input node ids, the other records positions in the packed tree
        const int32_t *map = h->cp_k > 0 ? nullptr : h->d_orig_id;
        auto *fn = pick_block(dl, leaf_ids_kernel<64>, leaf_ids_kernel<32>, leaf_ids_kernel<16>, leaf_ids_kernel<8>);
        const int64_t tiles = (h->n_trees + kIdTrees - 1) / kIdTrees;
        const int rc = walk_positions<kModeLeaves>(
            h, stream, X, n_docs, n_features, ScratchSource::kHandle, &taken, [&](const uint16_t *pos, int64_t doc0, int64_t nd) {
                const int64_t nb = (nd + dl - 1) / dl;
                hipLaunchKernelGGL(fn, dim3(unsigned((nb + kXcds - 1) / kXcds * kXcds * tiles)), dim3(kIdThreads), 0,
                                   stream, pos, nd, h->n_trees, h->d_tree_pos, h->d_tree_node_off, map,
                                   leaf_ids + doc0 * h->n_trees);
            });
        if (taken)
            return rc;
    }
    return launch_predict<kModeLeaves>(h, stream, X, n_docs, n_features, nullptr, leaf_ids);
}

// Vector-valued scores: the walk stores each leaf's row once and sum_rows_kernel adds up to eight outputs
// per pass, or (rows_pay) one walk per four outputs.
int launch_vector(const tree_ens *h, hipStream_t stream, const float *X, int64_t n_docs, int32_t n_features, float *scores,
                  ScratchSource source) {
    bool taken = false;
    if (rows_pay(h->facts, n_docs)) {
        const int dl = h->plan.docs_per_block, n_out = h->n_outputs;
        auto *two = pick_block(dl, sum_rows_kernel<64, 2>, sum_rows_kernel<32, 2>, sum_rows_kernel<16, 2>, sum_rows_kernel<8, 2>);
        auto *one = pick_block(dl, sum_rows_kernel<64, 1>, sum_rows_kernel<32, 1>, sum_rows_kernel<16, 1>, sum_rows_kernel<8, 1>);
        const double scale = 1.0 / double(h->n_bags);
        const int rc = walk_positions<kModeRows>(
            h, stream, X, n_docs, n_features, source, &taken, [&](const uint16_t *pos, int64_t doc0, int64_t nd) {
                const int chunks = (n_out + kVecPerLaunch - 1) / kVecPerLaunch;
                for (int c = 0; c < chunks; c += 2)
                    hipLaunchKernelGGL(c + 1 < chunks ? two : one, dim3(unsigned((nd + 63) / 64)), dim3(kRowThreads), 0,
                                       stream, pos, nd, h->n_trees, h->d_tree_row0,
                                       reinterpret_cast<const float4 *>(h->d_leaf_vec), h->vec_stride / 4, c, n_out,
                                       scale, scores + doc0 * n_out);
            });
        if (taken)
            return rc;
    }
    return launch_predict<kModeVector>(h, stream, X, n_docs, n_features, scores, nullptr, nullptr, 0, source);
}

int launch_scores(const tree_ens *h, hipStream_t stream, const float *X, int64_t n_docs, int32_t n_features, float *scores,
                  ScratchSource source) {
    if (h->n_outputs > 1)
        return launch_vector(h, stream, X, n_docs, n_features, scores, source);
    bool taken = false;
    const int rc = launch_coded_predict(h, stream, X, n_docs, n_features, scores, source, &taken);
    if (taken)
        return rc;
    return launch_predict<kModeScore>(h, stream, X, n_docs, n_features, scores, nullptr, nullptr, 0, source);
}

} // namespace

extern "C" {

int tree_ens_create(tree_ens_t **out, int32_t n_trees, const int64_t *tree_offsets,
                    const int32_t *feature, const float *threshold, const int32_t *left,
                    const int32_t *right, const float *value, uint32_t flags) {
    return tree_ens_create_multi(out, n_trees, tree_offsets, feature, threshold, left, right, value,
                                 1, 1, flags);
}

int tree_ens_create_multi(tree_ens_t **out, int32_t n_trees, const int64_t *tree_offsets,
                          const int32_t *feature, const float *threshold, const int32_t *left,
                          const int32_t *right, const float *value, int32_t n_outputs,
                          int32_t n_bags, uint32_t flags) {
    g_err.clear();
    if (!out)
        return fail(TREE_ENS_E_ARG, "out is NULL");
    *out = nullptr;
    if (n_bags < 1)
        return fail(TREE_ENS_E_ARG, "n_bags must be >= 1");
    const bool codegen = (flags & TREE_ENS_CODEGEN) != 0;
    if (codegen && n_outputs != 1)
        return fail(TREE_ENS_E_ARG, "code generation supports one value per leaf");
    Packed p;
    std::string err;
    int rc;
    try {
        rc = treeens::pack_model(n_trees, tree_offsets, feature, threshold, left, right, value, n_outputs, flags,
                                 p, err);
    } catch (const std::bad_alloc &) {
        return fail(TREE_ENS_E_NOMEM, "host allocation failed while packing");
    }
    if (rc != treeens::kOk)
        return fail(rc, err);
    std::vector<char> cg_code;
    if (codegen && n_trees > 0) {
        std::string src;
        try {
            rc = treeens::codegen_source(n_trees, tree_offsets, feature, threshold, left, right, value,
                                         flags, src, err);
        } catch (const std::bad_alloc &) {
            return fail(TREE_ENS_E_NOMEM, "host allocation failed while generating code");
        }
        if (rc != treeens::kOk)
            return fail(rc, err);
        rc = compile_codegen(src, cg_code, err);
        if (rc != TREE_ENS_OK)
            return fail(rc, err);
    }

    tree_ens *h = new (std::nothrow) tree_ens();
    if (!h)
        return fail(TREE_ENS_E_NOMEM, "host allocation failed");
    h->n_trees = p.n_trees;
    h->n_cols = p.n_cols;
    h->max_depth = p.max_depth;
    h->n_nodes = int64_t(p.nodes.size());
    h->plan = p.plan;
    h->n_outputs = p.n_outputs;
    h->n_bags = n_bags;
    h->vec_stride = p.vec_stride;
    std::memcpy(h->level_begin, p.level_begin, sizeof h->level_begin);
    hipError_t e = hipGetDevice(&h->device);
    std::memcpy(h->level_image_off, p.level_image_off, sizeof h->level_image_off);
    h->facts = treeens::plan_facts(p);
    h->usage_slot_off = p.usage_slot_off;
    h->pk_recs = p.pk_recs;
    h->pk_zero_rec = p.pk_zero_rec;
    h->pk_per_walker = p.pk_per_walker;
    std::memcpy(h->level_slot_recs, p.level_slot_recs, sizeof h->level_slot_recs);
    h->cp_k = p.cp_k;
    h->cp_per_walker = p.cp_per_walker;
    h->n_small = p.n_small;
    h->big_off0 = p.tree_node_off[size_t(p.n_small)];
    h->term = p.term;
    h->uniform = p.uniform;
    try {
        DeviceArrays arrays;
        std::vector<int32_t> tree_pos(p.tree_orig.size());
        for (size_t t = 0; t < tree_pos.size(); t++)
            tree_pos[size_t(p.tree_orig[t])] = int32_t(t);
        arrays.add(&h->d_images, p.images);
        arrays.add(&h->d_tile_recs, p.tile_recs);
        if (p.cp_k > 0) {
            // the compact packets replace the 8-byte ones (the feature trace walks the shared tiles)
            h->pk_recs = 0;
            arrays.add(&h->d_cpackets, p.cp_packets);
            arrays.add(&h->d_cleaf, p.cp_leaf);
            arrays.add(&h->d_cleaf_id, p.cp_leaf_id);
        } else if (p.pk_recs > 0) {
            arrays.add(&h->d_packets, p.packets);
        }
        if (p.n_small < p.n_trees)
            arrays.add(&h->d_big, p.nodes, h->big_off0);
        arrays.add(&h->d_tree_node_off, p.tree_node_off);
        arrays.add(&h->d_tree_orig, p.tree_orig);
        arrays.add(&h->d_tree_pos, tree_pos);
        arrays.add(&h->d_orig_id, p.orig_id);
        arrays.reserve(reinterpret_cast<void **>(&h->d_scratch), nullptr, kScratchDoubles * sizeof(double));
        if (p.n_outputs > 1) {
            p.leaf_vec.resize(size_t(p.leaf_rows) * size_t(p.vec_stride));
            arrays.add(&h->d_leaf_vec, p.leaf_vec);
            arrays.add(&h->d_tree_row0, p.tree_row0);
        }
        if (p.term.per_wave > 0) {
            arrays.add(&h->d_term_packets, p.term_packets);
            arrays.add(&h->d_term_slots, p.term_slots);
        }
        if (p.uniform.depth > 0) {
            arrays.add(&h->d_uniform_nodes, p.uniform_nodes);
            arrays.add(&h->d_uniform_leaves, p.uniform_leaves);
        }
        if (p.plan.coded || p.uniform.depth > 0) {
            arrays.add(&h->d_code_search, p.code_search);
            arrays.add(&h->d_code_chunks, p.code_chunks);
            h->n_code_chunks = int32_t(p.code_chunks.size());
        }
        if (e == hipSuccess)
            e = arrays.upload(&h->d_model);
        if (e == hipErrorOutOfMemory && !h->d_model && pool_of(h->device) && pool_of(h->device)->trim()) {
            (void)hipGetLastError();
            e = arrays.upload(&h->d_model);
        }
    } catch (const std::bad_alloc &) {
        e = hipErrorOutOfMemory;
    }
    if (e == hipSuccess)
        e = hipEventCreateWithFlags(&h->scratch_done, hipEventDisableTiming);
    if (e == hipSuccess && !cg_code.empty()) {
        e = hipModuleLoadData(&h->cg_module, cg_code.data());
        if (e == hipSuccess)
            e = hipModuleGetFunction(&h->cg_fn, h->cg_module, "tree_ens_cg");
    }
    if (e != hipSuccess) {
        free_device(h);
        delete h;
        return fail(e == hipErrorOutOfMemory ? TREE_ENS_E_NOMEM : TREE_ENS_E_DEVICE,
                    std::string("device upload failed: ") + hipGetErrorString(e));
    }
    if (Pool *pool = pool_of(h->device))
        pool->add_user();
    *out = h;
    return TREE_ENS_OK;
}

int tree_ens_predict(const tree_ens_t *h, void *stream, const float *X, int64_t n_docs,
                     int32_t n_features, float *scores) {
    g_err.clear();
    int rc = check_predict_args(h, X, n_docs, n_features, scores);
    if (rc != TREE_ENS_OK || n_docs == 0)
        return rc;
    DeviceGuard g(h->device);
    if (g.err != hipSuccess)
        return hip_fail(g.err, "hipSetDevice");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (h->n_trees == 0) {
        const int bs = 256;
        const int64_t n = n_docs * h->n_outputs;
        hipLaunchKernelGGL(fill_zero_kernel, dim3(unsigned((n + bs - 1) / bs)), dim3(bs), 0, s,
                           scores, n);
        hipError_t e = hipGetLastError();
        return e == hipSuccess ? TREE_ENS_OK : hip_fail(e, "kernel launch");
    }
    if (h->cg_fn) {
        // the model's own kernel: one document per thread
        const float *x = X;
        long long n = n_docs;
        int nf = n_features;
        float *out = scores;
        double scale = 1.0 / double(h->n_bags);
        void *args[] = {&x, &n, &nf, &out, &scale};
        const int64_t blocks = (n_docs + treeens::kCodegenThreads - 1) / treeens::kCodegenThreads;
        if (blocks > 0x7fffffff)
            return fail(TREE_ENS_E_ARG, "too many documents for one launch");
        (void)hipGetLastError();
        h->last_path.store(TREE_ENS_PATH_CODEGEN, std::memory_order_relaxed);
        hipError_t e = hipModuleLaunchKernel(h->cg_fn, unsigned(blocks), 1, 1, treeens::kCodegenThreads,
                                             1, 1, 0, s, args, nullptr);
        return e == hipSuccess ? TREE_ENS_OK : hip_fail(e, "specialised kernel launch");
    }
    return launch_scores(h, s, X, n_docs, n_features, scores, ScratchSource::kHandle);
}

int tree_ens_predict_noalloc(const tree_ens_t *h, void *stream, const float *X, int64_t n_docs,
                             int32_t n_features, float *scores) {
    g_err.clear();
    int rc = check_predict_args(h, X, n_docs, n_features, scores);
    if (rc != TREE_ENS_OK || n_docs == 0)
        return rc;
    DeviceGuard g(h->device);
    if (g.err != hipSuccess)
        return hip_fail(g.err, "hipSetDevice");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (h->n_trees == 0 || h->cg_fn)
        return tree_ens_predict(h, stream, X, n_docs, n_features, scores); // no scratch used
    return launch_scores(h, s, X, n_docs, n_features, scores, ScratchSource::kStatic);
}

int tree_ens_predict_leaves(const tree_ens_t *h, void *stream, const float *X, int64_t n_docs,
                            int32_t n_features, int32_t *leaf_ids) {
    g_err.clear();
    int rc = check_predict_args(h, X, n_docs, n_features, leaf_ids);
    if (rc != TREE_ENS_OK || n_docs == 0 || h->n_trees == 0)
        return rc;
    DeviceGuard g(h->device);
    if (g.err != hipSuccess)
        return hip_fail(g.err, "hipSetDevice");
    return launch_leaves(h, reinterpret_cast<hipStream_t>(stream), X, n_docs, n_features, leaf_ids);
}

int tree_ens_predict_topk(const tree_ens_t *h, void *stream, const float *X, int64_t n_docs,
                          int32_t n_features, const int64_t *group_offsets, int64_t n_groups,
                          int32_t k, float *scores, int32_t *top_idx, float *top_scores) {
    if (h && h->n_outputs != 1)
        return fail(TREE_ENS_E_ARG, "reranking needs one score per document (n_outputs = 1)");
    int rc = tree_ens_predict(h, stream, X, n_docs, n_features, scores);
    if (rc != TREE_ENS_OK)
        return rc;
    return tree_ens_topk(stream, scores, n_docs, group_offsets, n_groups, k, top_idx, top_scores);
}

int tree_ens_feature_usage(const tree_ens_t *h, void *stream, const float *X, int64_t n_docs,
                           int32_t n_features, int32_t *counts, uint32_t *masks) {
    g_err.clear();
    int rc = check_predict_args(h, X, n_docs, n_features, counts);
    if (rc != TREE_ENS_OK || n_docs == 0)
        return rc;
    if (masks && (reinterpret_cast<uintptr_t>(masks) & 3u) != 0)
        return fail(TREE_ENS_E_ARG, "masks must be 4-byte aligned");
    DeviceGuard g(h->device);
    if (g.err != hipSuccess)
        return hip_fail(g.err, "hipSetDevice");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const int32_t words = (n_features + 31) / 32;
    if (h->n_trees == 0) {
        const int bs = 256;
        hipLaunchKernelGGL(fill_zero_kernel, dim3(unsigned((n_docs + bs - 1) / bs)), dim3(bs), 0, s,
                           reinterpret_cast<float *>(counts), n_docs);
        if (masks)
            hipLaunchKernelGGL(fill_zero_kernel, dim3(unsigned((n_docs * words + bs - 1) / bs)),
                               dim3(bs), 0, s, reinterpret_cast<float *>(masks), n_docs * words);
        hipError_t e = hipGetLastError();
        return e == hipSuccess ? TREE_ENS_OK : hip_fail(e, "kernel launch");
    }
    // two-workgroup plans whose level-0 tiles leave room in the slot keep two workgroups per CU
    if (h->usage_slot_off >= 0)
        return launch_predict<kModeUsageSlot>(h, s, X, n_docs, n_features, nullptr, counts, masks,
                                              words);
    return launch_predict<kModeUsage>(h, s, X, n_docs, n_features, nullptr, counts, masks, words);
}

int tree_ens_info(const tree_ens_t *h, int32_t *n_trees, int32_t *min_features, int32_t *max_depth,
                  int64_t *packed_bytes, int32_t *n_tiles, int32_t *docs_per_block) {
    g_err.clear();
    if (!h)
        return fail(TREE_ENS_E_ARG, "handle is NULL");
    if (n_trees)
        *n_trees = h->n_trees;
    if (min_features)
        *min_features = h->n_cols;
    if (max_depth)
        *max_depth = h->max_depth;
    if (packed_bytes)
        *packed_bytes = h->n_nodes * int64_t(sizeof(NodeRec));
    if (n_tiles)
        *n_tiles = h->level_begin[1] - h->level_begin[0];
    if (docs_per_block)
        *docs_per_block = h->plan.docs_per_block;
    return TREE_ENS_OK;
}

int tree_ens_codegen_source(int32_t n_trees, const int64_t *tree_offsets, const int32_t *feature,
                            const float *threshold, const int32_t *left, const int32_t *right,
                            const float *value, uint32_t flags, char *buf, int64_t buf_size,
                            int64_t *src_len) {
    g_err.clear();
    if (buf_size < 0 || (buf_size > 0 && !buf))
        return fail(TREE_ENS_E_ARG, "buf is NULL with a positive buf_size");
    std::string src, err;
    int rc;
    try {
        rc = treeens::codegen_source(n_trees, tree_offsets, feature, threshold, left, right, value,
                                     flags | TREE_ENS_CODEGEN, src, err);
    } catch (const std::bad_alloc &) {
        return fail(TREE_ENS_E_NOMEM, "host allocation failed while generating code");
    }
    if (rc != treeens::kOk)
        return fail(rc, err);
    if (src_len)
        *src_len = int64_t(src.size());
    if (buf_size > 0) {
        const size_t n = std::min(src.size(), size_t(buf_size - 1));
        std::memcpy(buf, src.data(), n);
        buf[n] = '\0';
    }
    return TREE_ENS_OK;
}

int tree_ens_kernel_timing(const tree_ens_t *h, int32_t enable) {
    g_err.clear();
    if (!h)
        return fail(TREE_ENS_E_ARG, "handle is NULL");
    std::lock_guard<std::mutex> lock(h->timing_mu);
    if (!enable) {
        h->timing = false;
        return TREE_ENS_OK;
    }
    if (h->t_start.empty()) {
        DeviceGuard g(h->device);
        if (g.err != hipSuccess)
            return hip_fail(g.err, "hipSetDevice");
        for (int i = 0; i < kMaxTimedLaunches; ++i) {
            hipEvent_t a = nullptr, b = nullptr;
            hipError_t e = hipEventCreate(&a);
            if (e == hipSuccess)
                e = hipEventCreate(&b);
            if (e != hipSuccess) {
                if (a)
                    (void)hipEventDestroy(a);
                for (hipEvent_t ev : h->t_start)
                    (void)hipEventDestroy(ev);
                for (hipEvent_t ev : h->t_stop)
                    (void)hipEventDestroy(ev);
                h->t_start.clear();
                h->t_stop.clear();
                return hip_fail(e, "hipEventCreate");
            }
            h->t_start.push_back(a);
            h->t_stop.push_back(b);
        }
    }
    h->t_used = 0;
    h->timing = true;
    return TREE_ENS_OK;
}

int tree_ens_kernel_time(const tree_ens_t *h, double *total_ms, int32_t *launches) {
    g_err.clear();
    if (!h)
        return fail(TREE_ENS_E_ARG, "handle is NULL");
    std::lock_guard<std::mutex> lock(h->timing_mu);
    double sum = 0.0;
    for (int32_t i = 0; i < h->t_used; ++i) {
        hipError_t e = hipEventSynchronize(h->t_stop[size_t(i)]);
        float ms = 0.0f;
        if (e == hipSuccess)
            e = hipEventElapsedTime(&ms, h->t_start[size_t(i)], h->t_stop[size_t(i)]);
        if (e != hipSuccess)
            return hip_fail(e, "timing events");
        sum += double(ms);
    }
    if (total_ms)
        *total_ms = sum;
    if (launches)
        *launches = h->t_used;
    return TREE_ENS_OK;
}

int tree_ens_last_path(const tree_ens_t *h, int32_t *path) {
    g_err.clear();
    if (!h || !path)
        return fail(TREE_ENS_E_ARG, "handle or path is NULL");
    *path = h->last_path.load(std::memory_order_relaxed);
    return TREE_ENS_OK;
}

int tree_ens_outputs(const tree_ens_t *h, int32_t *n_outputs, int32_t *n_bags) {
    g_err.clear();
    if (!h)
        return fail(TREE_ENS_E_ARG, "handle is NULL");
    if (n_outputs)
        *n_outputs = h->n_outputs;
    if (n_bags)
        *n_bags = h->n_bags;
    return TREE_ENS_OK;
}

void tree_ens_destroy(tree_ens_t *h) {
    if (!h)
        return;
    DeviceGuard g(h->device);
    if (Pool *pool = pool_of(h->device))
        pool->drop_user();
    free_device(h);
    delete h;
}

const char *tree_ens_last_error(void) { return g_err.c_str(); }

} // extern "C"
