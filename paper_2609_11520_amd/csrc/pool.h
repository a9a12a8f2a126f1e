// The bookkeeping of the device blocks kept between handles (pool.cpp): which are kept, which one serves a
// request, which are given back.  Nothing here calls the device: blocks to be freed leave in a Blocks, freed by the
// caller, so that no lock is held while the device is waited for.
#pragma once
#include <cstddef>
#include <iterator>
#include <map>

namespace fio {

struct PoolBlock {
    void *p;
    int dev;
    long tick;                          // end_call() count when it was kept
    long epoch;                         // order of keeping
};
using PoolBlocks = std::multimap<size_t, PoolBlock>;      // by capacity

struct PoolBounds {
    size_t bytes;                       // kept at most
    size_t blocks;
    long age;                           // calls for which a block is kept unused
};

class BlockPool {
  public:
    explicit BlockPool(PoolBounds b) : bound(b) {}
    size_t bytes() const { return total; }
    size_t count() const { return kept.size(); }

    // The smallest block of `dev` that holds `bytes` and wastes at most a quarter (and 64 KiB) of them; false: none.
    // *wait: kernels that were launched before the block was kept may still use it.
    bool take(size_t bytes, int dev, size_t *cap, PoolBlock *out, bool *wait) {
        for (auto it = kept.lower_bound(bytes); it != kept.end() && it->first <= bytes + bytes / 4 + 65536; ++it) {
            if (it->second.dev != dev) continue;
            *cap = it->first;
            *out = it->second;
            *wait = it->second.epoch > idle[dev];
            total -= it->first;
            kept.erase(it);
            return true;
        }
        return false;
    }
    // the order of the last block kept: what a wait that begins now covers
    long epoch() const { return last; }
    // the device has been waited for, from epoch() == e on
    void waited(int dev, long e) {
        long &i = idle[dev];
        if (e > i) i = e;
    }
    // Keeps a block; what the bounds push out, the least recently kept first, goes to `out`.  May throw
    // std::bad_alloc, keeping nothing.
    void keep(void *p, size_t cap, int dev, PoolBlocks &out) {
        kept.emplace(cap, PoolBlock{p, dev, tick, last + 1});
        ++last;
        total += cap;
        shrink(bound.bytes, bound.blocks, out);
    }
    // one call that builds or destroys a handle has ended: blocks unused for too long go to `out`
    void end_call(PoolBlocks &out) {
        ++tick;
        for (auto it = kept.begin(); it != kept.end();) {
            const auto cur = it++;
            if (tick - cur->second.tick > bound.age) drop(cur, out);
        }
    }
    // at most so many bytes and blocks stay
    void shrink(size_t max_bytes, size_t max_blocks, PoolBlocks &out) {
        while (!kept.empty() && (total > max_bytes || kept.size() > max_blocks)) {
            auto old = kept.begin();
            for (auto it = kept.begin(); it != kept.end(); ++it)
                if (it->second.epoch < old->second.epoch) old = it;
            drop(old, out);
        }
    }

  private:
    void drop(PoolBlocks::iterator it, PoolBlocks &out) {
        total -= it->first;
        out.insert(kept.extract(it));                     // moves the node: no allocation
    }
    const PoolBounds bound;
    PoolBlocks kept;
    size_t total = 0;
    long tick = 0, last = 0;
    std::map<int, long> idle;           // per device: blocks kept up to this epoch are not in use
};

}  // namespace fio
