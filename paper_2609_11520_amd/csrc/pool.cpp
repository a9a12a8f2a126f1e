// Device memory of the calls that build and destroy handles.
//
// The kernel driver hands out memory it has cleared: once a process has cycled through the card's free memory,
// hipFree or hipMalloc waits for the clearing of what it frees or takes (2 GiB blocks on MI355X: 0.3 ms each
// for the first 200 GB, then 20 to 320 ms), and an offline stage of N = 2^16 goes through about 6 GB: 31 ms
// in the first 28 of a row, 194 ms in the next.  Blocks released while a handle is built or destroyed are
// therefore kept for the next one, at most kPoolBytes of them; they are given back when they have not
// been used for kPoolAge such calls, when newer ones need the room and when the device runs out of memory.
//
// A kept block may still be read or written by kernels in flight (on any stream).  hipFree would have
// waited for them; here the next owner does, once, before it takes a block that was kept after the
// last such wait.
#include <iterator>
#include <map>
#include <new>

#include "common.h"

namespace fio {
namespace {

constexpr size_t kPoolBytes = (size_t)8 << 30;    // under 3 % of the card
constexpr size_t kPoolBlocks = 1024;
constexpr long kPoolAge = 64;

struct Kept {
    void *p;
    int dev;
    long tick;                                    // PoolScope count when it was kept
    long epoch;                                   // order of keeping
};

using It = std::multimap<size_t, Kept>::iterator;

struct Pool {
    std::mutex mu;
    std::multimap<size_t, Kept> kept;             // by capacity
    size_t bytes = 0;
    long tick = 0, epoch = 0;
    std::map<int, long> waited;                   // per device: blocks up to this epoch are idle

    It drop(It it) {
        (void)hipFree(it->second.p);
        bytes -= it->first;
        return kept.erase(it);
    }
};

// never destroyed: handles may outlive the static objects of the library
Pool &pool() {
    static Pool *p = new Pool;
    return *p;
}

thread_local int t_depth = 0;

// the least recently kept blocks beyond the bounds
void evict(Pool &q) {
    while (!q.kept.empty() && (q.bytes > kPoolBytes || q.kept.size() > kPoolBlocks)) {
        It old = q.kept.begin();
        for (It it = q.kept.begin(); it != q.kept.end(); ++it)
            if (it->second.epoch < old->second.epoch) old = it;
        q.drop(old);
    }
}

// a block of at least `bytes` that wastes at most a quarter (and 64 KiB) of its size
void *take(size_t bytes, int dev, size_t *cap) {
    Pool &q = pool();
    std::lock_guard<std::mutex> lk(q.mu);
    for (It it = q.kept.lower_bound(bytes); it != q.kept.end() && it->first <= bytes + bytes / 4 + 65536; ++it) {
        if (it->second.dev != dev) continue;
        if (it->second.epoch > q.waited[dev]) {
            if (hipDeviceSynchronize() != hipSuccess) {
                (void)hipGetLastError();
                return nullptr;
            }
            q.waited[dev] = q.epoch;
        }
        void *p = it->second.p;
        *cap = it->first;
        q.bytes -= it->first;
        q.kept.erase(it);
        return p;
    }
    return nullptr;
}

}  // namespace

void *dev_alloc(size_t bytes, size_t *cap, int *dev) {
    FIO_HIP(hipGetDevice(dev));
    size_t c = bytes;
    void *p = t_depth > 0 ? take(bytes, *dev, &c) : nullptr;
    if (!p) {
        hipError_t e = hipMalloc(&p, bytes);
        if (e == hipErrorOutOfMemory) {
            (void)hipGetLastError();
            Pool &q = pool();
            std::lock_guard<std::mutex> lk(q.mu);
            for (It it = q.kept.begin(); it != q.kept.end();) it = q.drop(it);
            e = hipMalloc(&p, bytes);
        }
        FIO_HIP(e);
    }
    *cap = c;
    return p;
}

void dev_free(void *p, size_t cap, int dev) {
    if (t_depth > 0 && cap <= kPoolBytes) {
        Pool &q = pool();
        std::lock_guard<std::mutex> lk(q.mu);
        try {
            q.kept.emplace(cap, Kept{p, dev, q.tick, q.epoch + 1});
            ++q.epoch;
            q.bytes += cap;
            evict(q);
            return;
        } catch (const std::bad_alloc &) {
        }
    }
    (void)hipFree(p);
}

PoolScope::PoolScope() { ++t_depth; }

PoolScope::~PoolScope() {
    if (--t_depth > 0) return;
    Pool &q = pool();
    std::lock_guard<std::mutex> lk(q.mu);
    ++q.tick;
    for (It it = q.kept.begin(); it != q.kept.end();)
        it = q.tick - it->second.tick > kPoolAge ? q.drop(it) : std::next(it);
}

}  // namespace fio
