// scratch.hpp -- device memory lent to calls and kept between them (one pool per device).
//
// A stream-ordered allocation per call makes the host wait for the stream's work, and memory that
// goes back at every synchronisation is mapped again by the next call: two kernels of 1 MiB (64, 256)
// in a call that is waited for take 36 us (86, 302) with hipMallocAsync and hipFreeAsync, 15 us (34, 96)
// with a kept block ordered by an event, and the host enqueues them in 23 us (35, 93) against 6.
#pragma once

#include <algorithm>
#include <cstddef>
#include <memory>
#include <mutex>
#include <new>
#include <vector>

namespace treeens {

constexpr size_t kScratchKept = size_t(512) << 20;   // bytes a device's pool keeps at most
constexpr size_t kScratchGranule = size_t(2) << 20;  // block sizes are multiples of this

// Rt: Stream, Event and
//   void *allocate(size_t)      device memory, nullptr if there is none
//   void release(void *, Event) free it once the event's work is done, and the event
//   bool make_event(Event *), bool record(Event, Stream), bool wait(Stream, Event)
//   void finish(Stream)         wait on the host for the stream's work
//
// A block's last work is always waited for, also on the stream it ran on (one handle value can stand
// for several streams: a destroyed one's, each thread's own default stream).
template <typename Rt> class ScratchPool {
public:
    using Stream = typename Rt::Stream;
    struct Block {
        void *p;
        size_t bytes;
        typename Rt::Event done;
        Stream stream;
        bool used, lent;
    };

    explicit ScratchPool(Rt rt = Rt()) : rt_(rt) {}

    // A block of at least `bytes`, ordered after its last work for `stream`; nullptr: none to lend
    // (more than the pool may keep, every block lent, or no memory). A block last used on the same
    // stream is taken first, then a new one while the pool may grow, so that streams don't wait
    // for one another; then any.
    Block *lend(size_t bytes, Stream stream) {
        const size_t size = (std::max<size_t>(bytes, 1) + kScratchGranule - 1) / kScratchGranule * kScratchGranule;
        if (size > kScratchKept)
            return nullptr;
        std::lock_guard<std::mutex> lock(mu_);
        Block *b = smallest(bytes, [&](const Block &x) { return x.used && x.stream == stream; });
        if (!b)
            b = grow(size);
        if (!b)
            b = smallest(bytes, [](const Block &) { return true; });
        while (!b && drop_one())
            b = grow(size);
        if (!b || (b->used && !rt_.wait(stream, b->done)))
            return nullptr;
        b->lent = true;
        b->stream = stream;
        return b;
    }

    // Back from its call: everything that uses it is enqueued on its stream.
    void give(Block *b) {
        if (!rt_.record(b->done, b->stream))
            rt_.finish(b->stream);
        std::lock_guard<std::mutex> lock(mu_);
        b->used = true;
        b->lent = false;
    }

    // Blocks that are not lent go back, for an allocation elsewhere that found no memory; false if
    // there were none.
    bool trim() {
        std::lock_guard<std::mutex> lock(mu_);
        bool any = false;
        while (drop_one())
            any = true;
        return any;
    }

    // Handles of the device: the last one gives the memory back.
    void add_user() {
        std::lock_guard<std::mutex> lock(mu_);
        ++users_;
    }
    void drop_user() {
        std::lock_guard<std::mutex> lock(mu_);
        if (--users_ == 0)
            while (drop_one()) {
            }
    }

    size_t kept() const { return kept_; }

private:
    template <typename Pred> Block *smallest(size_t bytes, Pred &&pred) {
        Block *best = nullptr;
        for (auto &b : blocks_)
            if (!b->lent && b->bytes >= bytes && pred(*b) && (!best || b->bytes < best->bytes))
                best = b.get();
        return best;
    }

    Block *grow(size_t size) {
        if (kept_ + size > kScratchKept)
            return nullptr;
        try {
            blocks_.reserve(blocks_.size() + 1);
            auto b = std::make_unique<Block>(Block{nullptr, size, {}, {}, false, false});
            if (!rt_.make_event(&b->done))
                return nullptr;
            b->p = rt_.allocate(size);
            if (!b->p) {
                rt_.release(nullptr, b->done);
                return nullptr;
            }
            blocks_.push_back(std::move(b));
        } catch (const std::bad_alloc &) {
            return nullptr;
        }
        kept_ += size;
        return blocks_.back().get();
    }

    // The smallest block that is not lent goes back; false if there is none.
    bool drop_one() {
        Block *b = smallest(0, [](const Block &) { return true; });
        if (!b)
            return false;
        rt_.release(b->p, b->done);
        kept_ -= b->bytes;
        blocks_.erase(std::find_if(blocks_.begin(), blocks_.end(), [&](const auto &x) { return x.get() == b; }));
        return true;
    }

    Rt rt_;
    std::mutex mu_;
    std::vector<std::unique_ptr<Block>> blocks_;
    size_t kept_ = 0;
    int users_ = 0;
};

} // namespace treeens
