// pool.hpp -- the caching block pool behind the device allocator, as plain C++
// over a small device interface, so that its rules can be exercised on the
// host alone.
//
// Blocks are kept after release and handed out again for requests of similar
// size.  A released block may still be touched by work on its stream, so it
// enters the cache after a wait for that stream; a block released within a
// thread's scope with the scope's stream is held for the scope's own later
// requests instead, which are ordered after that work by the stream itself,
// and enters the cache when the scope closes, after one wait.  Held blocks are
// no thread's property: when the device has no memory left, every scope's are
// given back with the cache, after a wait for their streams.
#pragma once

#include <algorithm>
#include <cstddef>
#include <map>
#include <mutex>
#include <unordered_map>
#include <vector>

namespace tp {

// Dev: Stream, void *take(size_t) (null: out of memory), void give(void *),
// void wait(Stream).
template <class Dev>
class BlockPool {
public:
    using Stream = typename Dev::Stream;
    using Blocks = std::multimap<size_t, void *>;  // by size

    // What one thread holds during a call on one stream.
    struct Scope {
        Stream stream{};
        BlockPool *pool = nullptr;  // null: not open
        Blocks held;                // guarded by the pool's mutex
    };

    explicit BlockPool(Dev dev = Dev()) : dev_(dev) {}

    void open(Scope &sc, Stream stream)
    {
        std::lock_guard<std::mutex> lk(mu_);
        scopes_.push_back(&sc);
        sc.stream = stream;
        sc.pool = this;
    }

    void close(Scope &sc)
    {
        bool any;
        {
            std::lock_guard<std::mutex> lk(mu_);
            any = !sc.held.empty();
        }
        if (any) dev_.wait(sc.stream);
        std::lock_guard<std::mutex> lk(mu_);
        free_.merge(sc.held);
        scopes_.erase(std::find(scopes_.begin(), scopes_.end(), &sc));
        sc.pool = nullptr;
    }

    // A block of at least `bytes`, for work on `stream`; `own` is the calling
    // thread's scope.  Null: out of memory.
    void *alloc(size_t bytes, Stream stream, Scope *own)
    {
        const size_t sz = round_size(bytes ? bytes : 1);
        std::lock_guard<std::mutex> lk(mu_);
        if (holds(own, stream))
            if (void *p = reuse(own->held, sz)) return p;
        if (void *p = reuse(free_, sz)) return p;
        void *p = dev_.take(sz);
        if (!p) {
            give_back();
            p = dev_.take(sz);
        }
        if (p) {
            Blocks one;
            one.emplace(sz, p);
            live_.emplace(p, one.extract(one.begin()));
        }
        return p;
    }

    void release(void *p, Stream stream, Scope *own)
    {
        const bool held = holds(own, stream);
        if (!held) dev_.wait(stream);
        std::lock_guard<std::mutex> lk(mu_);
        auto it = live_.find(p);
        if (it == live_.end()) return;
        (held ? own->held : free_).insert(std::move(it->second));
        live_.erase(it);
    }

    // Give all released blocks back to the device.
    void trim()
    {
        std::lock_guard<std::mutex> lk(mu_);
        give_back();
    }

    size_t cached()  // bytes released and not given back
    {
        std::lock_guard<std::mutex> lk(mu_);
        size_t b = 0;
        for (const auto &kv : free_) b += kv.first;
        for (const Scope *sc : scopes_)
            for (const auto &kv : sc->held) b += kv.first;
        return b;
    }

    size_t live()  // bytes handed out and not yet released
    {
        std::lock_guard<std::mutex> lk(mu_);
        size_t b = 0;
        for (const auto &kv : live_) b += kv.second.key();
        return b;
    }

private:
    static size_t round_size(size_t bytes)
    {
        const size_t small = 512, big = size_t(2) << 20;
        return bytes < big ? (bytes + small - 1) / small * small : (bytes + big - 1) / big * big;
    }

    // The smallest block that is large enough, unless it is much larger.
    void *reuse(Blocks &blocks, size_t sz)
    {
        auto it = blocks.lower_bound(sz);
        if (it == blocks.end() || it->first > sz + sz / 4 + (size_t(8) << 20)) return nullptr;
        void *p = it->second;
        live_.emplace(p, blocks.extract(it));
        return p;
    }

    bool holds(const Scope *own, Stream stream) const { return own && own->pool == this && own->stream == stream; }

    void give_back()
    {
        for (Scope *sc : scopes_) {
            if (sc->held.empty()) continue;
            dev_.wait(sc->stream);
            free_.merge(sc->held);
        }
        for (const auto &kv : free_) dev_.give(kv.second);
        free_.clear();
    }

    Dev dev_;
    std::mutex mu_;
    Blocks free_;
    std::unordered_map<void *, typename Blocks::node_type> live_;
    std::vector<Scope *> scopes_;  // open ones
};

}  // namespace tp
