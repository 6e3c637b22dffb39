// The scratch pool (scratch.hpp) over a runtime that only records what is asked of it.
#include "scratch.hpp"

#include <cstdio>
#include <cstdlib>
#include <map>
#include <thread>

#define CHECK(c)                                                        \
    do {                                                                \
        if (!(c)) {                                                     \
            std::printf("line %d: %s\n", __LINE__, #c);                 \
            std::exit(1);                                               \
        }                                                               \
    } while (0)

namespace {

struct Log {
    std::mutex mu;
    size_t live = 0, most = 0, limit = ~size_t(0);
    int next_event = 1, allocations = 0, waits = 0, finishes = 0;
    bool refuse_record = false;
    std::map<void *, size_t> sizes;
    std::map<int, int> recorded; // event -> stream of its last record
    int waited_event = 0, waiting_stream = 0;
};

struct FakeRt {
    using Stream = int;
    using Event = int;
    Log *log = nullptr;
    void *allocate(size_t n) {
        std::lock_guard<std::mutex> lock(log->mu);
        if (log->live + n > log->limit)
            return nullptr;
        void *p = std::malloc(1);
        log->sizes[p] = n;
        log->live += n;
        log->most = std::max(log->most, log->live);
        log->allocations++;
        return p;
    }
    void release(void *p, Event) {
        std::lock_guard<std::mutex> lock(log->mu);
        if (p)
            log->live -= log->sizes[p], log->sizes.erase(p), std::free(p);
    }
    bool make_event(Event *e) {
        std::lock_guard<std::mutex> lock(log->mu);
        *e = log->next_event++;
        return true;
    }
    bool record(Event e, Stream s) {
        std::lock_guard<std::mutex> lock(log->mu);
        log->recorded[e] = s;
        return !log->refuse_record;
    }
    bool wait(Stream s, Event e) {
        std::lock_guard<std::mutex> lock(log->mu);
        CHECK(log->recorded.count(e));
        log->waits++, log->waited_event = e, log->waiting_stream = s;
        return true;
    }
    void finish(Stream) { log->finishes++; }
};
using Pool = treeens::ScratchPool<FakeRt>;
constexpr size_t MB = size_t(1) << 20;

void one_stream() {
    Log log;
    Pool pool(FakeRt{&log});
    pool.add_user();
    auto *a = pool.lend(30 * MB + 1, 1);
    CHECK(a && a->bytes == 32 * MB && log.waits == 0);
    pool.give(a);
    for (int i = 0; i < 5; i++) { // smaller calls of the stream: the same block, after its last work
        auto *b = pool.lend((i + 1) * MB, 1);
        CHECK(b == a && log.waits == i + 1 && log.waited_event == a->done && log.waiting_stream == 1);
        pool.give(b);
    }
    CHECK(log.allocations == 1);
    auto *big = pool.lend(100 * MB, 1);
    CHECK(big != a && log.allocations == 2);
    pool.give(big);
    CHECK(pool.lend(20 * MB, 1) == a); // the smallest that fits
    CHECK(pool.lend(20 * MB, 1) == big);
    auto *more = pool.lend(20 * MB, 1); // both lent: never lent twice
    CHECK(more && more != a && more != big);
    pool.give(a), pool.give(big), pool.give(more);
    pool.drop_user();
    CHECK(log.live == 0 && pool.kept() == 0);
}

void streams_and_bound() {
    Log log;
    Pool pool(FakeRt{&log});
    pool.add_user(), pool.add_user();
    auto *a = pool.lend(256 * MB, 1);
    pool.give(a);
    auto *b = pool.lend(256 * MB, 2); // another stream does not wait while the pool may grow
    CHECK(b != a && log.waits == 0);
    pool.give(b);
    auto *c = pool.lend(256 * MB, 3); // full: an idle block, after its last work
    CHECK((c == a || c == b) && log.waits == 1 && log.waiting_stream == 3 && log.waited_event == c->done);
    auto *d = pool.lend(256 * MB, 4);
    CHECK(d && d != c);
    CHECK(!pool.lend(2 * MB, 5)); // full and all lent
    pool.give(c), pool.give(d);
    CHECK(!pool.lend(512 * MB + 1, 1) && log.allocations == 2); // more than is ever kept
    auto *e = pool.lend(300 * MB, 6); // too small ones go back first
    CHECK(e && e->bytes == 300 * MB && log.most <= 512 * MB);
    pool.give(e);
    pool.drop_user();
    CHECK(log.live > 0);
    pool.drop_user();
    CHECK(log.live == 0 && log.sizes.empty());
    pool.add_user(); // and the pool can be used again
    auto *f = pool.lend(1, 1);
    CHECK(f && f->bytes == 2 * MB);
    pool.give(f);
    pool.drop_user();
    CHECK(log.live == 0);
}

void failures() {
    Log log;
    Pool pool(FakeRt{&log});
    pool.add_user();
    log.limit = 64 * MB;
    auto *a = pool.lend(40 * MB, 1);
    CHECK(a);
    CHECK(!pool.lend(40 * MB, 2) && pool.kept() == 40 * MB); // no memory
    log.refuse_record = true;
    pool.give(a); // no event: the host waits
    CHECK(log.finishes == 1);
    log.refuse_record = false;
    auto *b = pool.lend(60 * MB, 2); // room is made
    CHECK(b && pool.kept() == 60 * MB && log.live == 60 * MB);
    CHECK(!pool.trim() && log.live == 60 * MB); // lent: stays
    pool.give(b);
    CHECK(pool.trim() && log.live == 0 && !pool.trim());
    auto *c = pool.lend(10 * MB, 1);
    CHECK(c);
    pool.give(c);
    pool.drop_user();
    CHECK(log.live == 0);
}

void threads() {
    Log log;
    Pool pool(FakeRt{&log});
    pool.add_user();
    std::mutex mu;
    std::map<void *, int> owner;
    std::vector<std::thread> ts;
    for (int t = 0; t < 8; t++)
        ts.emplace_back([&, t] {
            unsigned r = unsigned(t) * 2654435761u + 1;
            for (int i = 0; i < 2000; i++) {
                r = r * 1664525u + 1013904223u;
                auto *b = pool.lend((r >> 8) % (200 * MB), t % 3);
                if (!b)
                    continue;
                {
                    std::lock_guard<std::mutex> lock(mu);
                    CHECK(owner[b->p]++ == 0);
                }
                std::this_thread::yield();
                {
                    std::lock_guard<std::mutex> lock(mu);
                    owner[b->p]--;
                }
                pool.give(b);
            }
        });
    for (auto &t : ts)
        t.join();
    CHECK(log.most <= treeens::kScratchKept);
    pool.drop_user();
    CHECK(log.live == 0);
}

} // namespace

int main() {
    one_stream();
    streams_and_bound();
    failures();
    threads();
    std::puts("ok");
}
