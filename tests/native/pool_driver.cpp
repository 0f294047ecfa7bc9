// Host-only checks of the device allocator's block pool (pool.hpp) over a
// device of fixed capacity whose blocks remember the stream that used them
// last.  Prints one line per check: "ok <name>" or "FAIL <name>: <detail>".
#include <atomic>
#include <cstdint>
#include <cstdio>
#include <map>
#include <mutex>
#include <random>
#include <set>
#include <string>
#include <thread>
#include <vector>

#include "pool.hpp"

static int failures = 0;
static void check(bool c, const std::string &name, const std::string &detail = "")
{
    std::printf("%s %s%s%s\n", c ? "ok" : "FAIL", name.c_str(), c ? "" : ": ", c ? "" : detail.c_str());
    if (!c) ++failures;
}

constexpr size_t MB = size_t(1) << 20;

// The shared state of a device: what is taken, and which streams have been
// waited for since each block was last used.
struct World {
    std::mutex mu;
    size_t capacity = 0, used = 0;
    uintptr_t next = 1;
    std::map<void *, size_t> taken;
    std::map<void *, std::set<int>> busy;  // block -> streams that may still touch it
    std::vector<int> waits;
    int unsafe_gives = 0;
    void touch(void *p, int stream)
    {
        std::lock_guard<std::mutex> lk(mu);
        busy[p].insert(stream);
    }
    bool idle(void *p, int stream)  // only work on `stream` may still touch it
    {
        std::lock_guard<std::mutex> lk(mu);
        for (int s : busy[p])
            if (s != stream) return false;
        return true;
    }
};

struct FakeDevice {
    using Stream = int;
    World *w = nullptr;
    void *take(size_t bytes)
    {
        std::lock_guard<std::mutex> lk(w->mu);
        if (w->used + bytes > w->capacity) return nullptr;
        w->used += bytes;
        void *p = reinterpret_cast<void *>(w->next++);
        w->taken[p] = bytes;
        return p;
    }
    void give(void *p)
    {
        std::lock_guard<std::mutex> lk(w->mu);
        w->used -= w->taken[p];
        w->taken.erase(p);
        if (!w->busy[p].empty()) ++w->unsafe_gives;
        w->busy.erase(p);
    }
    void wait(int s)
    {
        std::lock_guard<std::mutex> lk(w->mu);
        w->waits.push_back(s);
        for (auto &kv : w->busy) kv.second.erase(s);
    }
};
using Pool = tp::BlockPool<FakeDevice>;

int main()
{
    {
        World w;
        w.capacity = 100 * MB;
        Pool pool(FakeDevice{&w});
        Pool::Scope sc, none;
        pool.open(sc, 1);
        void *a = pool.alloc(20 * MB, 1, &sc);
        w.touch(a, 1);
        pool.release(a, 1, &sc);
        check(w.waits.empty(), "a scope's release does not wait");
        check(pool.live() == 0 && pool.cached() == 20 * MB, "a held block is released, and cached");
        check(pool.alloc(20 * MB, 1, &sc) == a, "its own stream gets it again");
        pool.release(a, 1, &sc);
        void *b = pool.alloc(20 * MB, 2, &sc);
        check(b && b != a, "another stream of the thread does not");
        void *c = pool.alloc(20 * MB, 1, &none);
        check(c && c != a, "another thread does not, while there is memory");
        w.touch(b, 2);
        pool.release(b, 2, &sc);
        check(w.waits == std::vector<int>{2}, "a release with another stream waits for it");
        pool.release(c, 1, nullptr);
        w.waits.clear();
        pool.close(sc);
        check(w.waits == std::vector<int>{1}, "the scope's end waits once");
        check(pool.cached() == 60 * MB && pool.live() == 0, "its blocks are in the cache");
        pool.trim();
        check(w.used == 0 && w.unsafe_gives == 0, "trim gives them back");
        pool.open(sc, 3);
        pool.close(sc);
        check(w.waits == std::vector<int>{1}, "an empty scope does not wait");
    }
    {
        // two calls near the device's capacity on two threads: what one has
        // released serves the other, after a wait for the stream that used it
        World w;
        w.capacity = 100 * MB;
        Pool pool(FakeDevice{&w});
        Pool::Scope first, second;
        pool.open(first, 1);
        void *a = pool.alloc(60 * MB, 1, &first);
        w.touch(a, 1);
        pool.release(a, 1, &first);
        void *b = nullptr;
        std::thread([&] {
            pool.open(second, 2);
            b = pool.alloc(80 * MB, 2, &second);
            if (b) pool.release(b, 2, &second);
            pool.close(second);
        }).join();
        check(b != nullptr, "a second call near capacity gets what the first has released");
        check(w.unsafe_gives == 0 && !w.waits.empty() && w.waits[0] == 1, "after a wait for the first one's stream");
        a = pool.alloc(90 * MB, 1, &first);
        check(a != nullptr, "and the other way round");
        check(pool.alloc(20 * MB, 1, &first) == nullptr, "live blocks are not given back");
        pool.release(a, 1, &first);
        pool.close(first);
        pool.trim();
        check(pool.live() == 0 && w.used == 0 && w.unsafe_gives == 0, "nothing is left");
    }
    {
        // threads with a scope and a stream each, on a device that holds what
        // they use at most, but not what they hold besides
        World w;
        constexpr int kThreads = 6, kBlocks = 3;
        w.capacity = (size_t)kThreads * kBlocks * 16 * MB;
        Pool pool(FakeDevice{&w});
        std::atomic<int> refused{0}, shared{0}, dirty{0};
        std::mutex mu;
        std::set<void *> out;
        std::vector<std::thread> threads;
        for (int t = 0; t < kThreads; ++t)
            threads.emplace_back([&, t] {
                std::mt19937 rng(t + 1);
                for (int call = 0; call < 60; ++call) {
                    Pool::Scope sc;
                    pool.open(sc, t);
                    std::vector<void *> mine;
                    for (int i = 0; i < 40; ++i) {
                        if (mine.size() < kBlocks && rng() % 2) {
                            void *p = pool.alloc((1 + rng() % 12) * MB, t, &sc);
                            if (!p) {
                                ++refused;
                                continue;
                            }
                            if (!w.idle(p, t)) ++dirty;
                            w.touch(p, t);
                            std::lock_guard<std::mutex> lk(mu);
                            if (!out.insert(p).second) ++shared;
                            mine.push_back(p);
                        } else if (!mine.empty()) {
                            const size_t k = rng() % mine.size();
                            void *p = mine[k];
                            mine.erase(mine.begin() + (long)k);
                            {
                                std::lock_guard<std::mutex> lk(mu);
                                out.erase(p);
                            }
                            pool.release(p, t, rng() % 4 ? &sc : nullptr);
                        }
                    }
                    for (void *p : mine) {
                        {
                            std::lock_guard<std::mutex> lk(mu);
                            out.erase(p);
                        }
                        pool.release(p, t, &sc);
                    }
                    pool.close(sc);
                }
            });
        for (auto &t : threads) t.join();
        check(shared == 0, "no block is handed out twice", std::to_string(shared.load()));
        check(dirty == 0, "no block is handed out while another stream may touch it", std::to_string(dirty.load()));
        check(refused == 0, "no call is refused memory that others only hold", std::to_string(refused.load()));
        check(w.unsafe_gives == 0, "no block is given back while a stream may touch it");
        check(pool.live() == 0, "all blocks are released");
        pool.trim();
        check(w.used == 0 && pool.cached() == 0, "and given back");
    }
    std::printf(failures ? "%d FAILED\n" : "all PASSED\n", failures);
    return failures ? 1 : 0;
}
