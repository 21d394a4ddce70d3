// Freed device blocks kept for later allocations: the bookkeeping alone (no
// HIP, no lock), so that it can be checked on the CPU.
//
// A block may still be in use by work queued before it was freed.  It is idle,
// and handed out as it is, when a device-wide wait followed its last use or
// its free, or when all its uses and the next ones are ordered on one stream.  A stream is known
// by its handle, so a handle must stand for one stream only: the per-thread
// default stream, one handle for a stream of each thread, is never that.
#pragma once

#include <cstddef>
#include <cstdint>
#include <deque>

namespace dsm {

// Sizes are rounded up so that blocks of nearly equal size serve each other:
// by less than 1/8, and only to 256 bytes under a budget, which then bounds the
// memory held to the byte rounding.
inline size_t block_class(size_t bytes, bool budget) {
    size_t step = 256;
    if (!budget)
        while (step * 16 < bytes) step <<= 1;
    return (bytes + step - 1) / step * step;
}

// New device memory for `bytes`: a block of their class, if need be after the
// kept blocks have been given back, or else, where the device has room for the
// bytes but not for the class, one of the bytes alone (*tight: it must not be
// kept as one of the class).  obtain(n): a block of n bytes or null.
template <class Obtain, class GiveBack>
void *new_block(size_t bytes, size_t cls, Obtain &&obtain, GiveBack &&give_back, bool *tight) {
    *tight = false;
    if (void *p = obtain(cls)) return p;
    give_back();
    if (void *p = obtain(cls)) return p;
    if (bytes >= cls) return nullptr;
    *tight = true;
    return obtain(bytes);
}

class BlockPool {
public:
    using Stream = const void *;
    static Stream unknown() { return (Stream)(uintptr_t)-1; }
    static Stream per_thread() { return (Stream)(uintptr_t)2; }

    struct Block {
        void *p;
        size_t bytes;    // size class
        Stream stream;   // every use was ordered on it; unknown() otherwise
        uint64_t seq;    // position in the order of frees; 0: idle
    };

    size_t bytes() const { return held; }
    uint64_t frees() const { return last; }

    // unused: the device has been waited for since the last use
    void put(void *p, size_t bytes, Stream s, bool unused = false) {
        blocks.push_back({p, bytes, ordered(s) ? s : unknown(), unused ? 0 : last + 1});
        last++;
        held += bytes;
    }

    // A block of this class, an idle one if there is any; false without one.
    // *wait: it is not idle.
    bool take(size_t bytes, Stream s, Block *out, bool *wait) {
        auto best = blocks.end();
        for (auto it = blocks.begin(); it != blocks.end(); ++it)
            if (it->bytes == bytes && (best == blocks.end() || (idle(*it, s) && !idle(*best, s)))) best = it;
        if (best == blocks.end()) return false;
        *out = *best;
        *wait = !idle(*best, s);
        held -= bytes;
        blocks.erase(best);
        return true;
    }

    bool take_oldest(Block *out) {
        if (blocks.empty()) return false;
        *out = blocks.front();
        held -= out->bytes;
        blocks.pop_front();
        return true;
    }

    // The device has been waited for after the `upto`-th free.
    void waited(uint64_t upto) { synced = upto > synced ? upto : synced; }

private:
    std::deque<Block> blocks;  // oldest first
    size_t held = 0;
    uint64_t last = 0, synced = 0;

    static bool ordered(Stream s) { return s != unknown() && s != per_thread(); }
    bool idle(const Block &b, Stream s) const { return b.seq <= synced || (ordered(s) && b.stream == s); }
};

}  // namespace dsm
