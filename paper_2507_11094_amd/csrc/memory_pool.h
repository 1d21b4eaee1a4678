// Device memory kept between objects: blocks that were given up, for later allocations of
// about the same size.  Nothing here throws: where the host's memory runs out, blocks are
// not kept and not known, and go back to the device instead.
#pragma once

#include <cstddef>
#include <cstdint>
#include <map>
#include <mutex>
#include <new>
#include <unordered_map>

namespace dg {

class MemoryPool {
    struct Block {
        void *p;
        int dev;
        uint64_t age;
    };
    typedef std::multimap<size_t, Block> Blocks;  // by size
    struct InUse {
        size_t bytes;
        int dev;
    };
    std::mutex mu;
    Blocks idle;
    std::unordered_map<void *, InUse> in_use;
    size_t held = 0;
    uint64_t clock = 0;
    const size_t most;
    void (*const free_fn)(void *);

public:
    MemoryPool(size_t most_, void (*free_)(void *)) : most(most_), free_fn(free_) {}

    // Sizes step by an eighth of their power of two, so that blocks of about the same
    // size are of the same size, but by 64 KiB at most: what the device has goes to the
    // graphs (steps of an eighth at any size took up to 12 % more than was asked for).
    static size_t round(size_t n) {
        size_t g = 256;
        while (g * 16 <= n && g < ((size_t)64 << 10)) g *= 2;
        return (n + g - 1) / g * g;
    }
    // A kept block of at least `bytes`, or null.
    void *take(size_t bytes, int dev) noexcept {
        std::lock_guard<std::mutex> l(mu);
        for (auto it = idle.lower_bound(bytes); it != idle.end() && it->first <= bytes + bytes / 4; ++it) {
            if (it->second.dev != dev) continue;
            void *p = it->second.p;
            if (!know(p, it->first, dev)) return nullptr;
            held -= it->first;
            idle.erase(it);
            return p;
        }
        return nullptr;
    }
    // A block that came from the device.
    void note(void *p, size_t bytes, int dev) noexcept {
        std::lock_guard<std::mutex> l(mu);
        (void)know(p, bytes, dev);
    }
    // A block is given up.  False: the caller frees it itself.
    bool give(void *p, bool keep) noexcept {
        Blocks out;
        bool kept = false;
        {
            std::lock_guard<std::mutex> l(mu);
            auto it = in_use.find(p);
            if (it == in_use.end()) return false;
            const InUse b = it->second;
            in_use.erase(it);
            if (keep && b.bytes <= most) {
                while (held + b.bytes > most) {
                    auto old = idle.begin();
                    for (auto i = idle.begin(); i != idle.end(); ++i)
                        if (i->second.age < old->second.age) old = i;
                    held -= old->first;
                    out.insert(idle.extract(old));
                }
                try {
                    idle.emplace(b.bytes, Block{p, b.dev, ++clock});
                    held += b.bytes;
                    kept = true;
                } catch (const std::bad_alloc &) {
                }
            }
        }
        for (auto &b : out) free_fn(b.second.p);
        return kept;
    }
    void trim() noexcept {
        Blocks out;
        {
            std::lock_guard<std::mutex> l(mu);
            out.swap(idle);
            held = 0;
        }
        for (auto &b : out) free_fn(b.second.p);
    }

private:
    bool know(void *p, size_t bytes, int dev) noexcept {
        try {
            in_use[p] = InUse{bytes, dev};
            return true;
        } catch (const std::bad_alloc &) {
            return false;
        }
    }
};

}  // namespace dg
