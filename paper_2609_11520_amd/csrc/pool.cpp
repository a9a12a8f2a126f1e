// Device memory of the calls that build and destroy handles.
//
// The kernel driver hands out memory it has cleared: once a process has cycled through the card's free memory,
// hipFree or hipMalloc waits for the clearing of what it frees or takes (2 GiB blocks on MI355X: 0.3 ms each
// for the first 200 GB, then 20 to 320 ms), and an offline stage of N = 2^16 goes through about 6 GB: 31 ms
// in the first 28 of a row, 194 ms in the next.  Blocks released while a handle is built or destroyed are
// therefore kept for the next one, at most kBounds.bytes of them; they are given back when they have not
// been used for kBounds.age such calls, when newer ones need the room, when the device runs out of memory, and by
// fio_memory_trim.
//
// A kept block may still be read or written by kernels in flight (on any stream).  hipFree would have
// waited for them; here the next owner does, once, before it takes a block that was kept after the
// last such wait.  The lock is not held while the device is waited for, here or in hipFree.
#include "pool.h"

#include <new>

#include "common.h"

namespace fio {
namespace {

constexpr PoolBounds kBounds{(size_t)8 << 30, 1024, 64};    // 8 GiB: under 3 % of the card

struct Pool {
    std::mutex mu;
    BlockPool q{kBounds};
};

// never destroyed: handles may outlive the static objects of the library
Pool &pool() {
    static Pool *p = new Pool;
    return *p;
}

thread_local int t_depth = 0;

void release(const PoolBlocks &b) {
    for (const auto &x : b) (void)hipFree(x.second.p);
}

void trim(size_t keep) {
    PoolBlocks out;
    {
        Pool &pl = pool();
        std::lock_guard<std::mutex> lk(pl.mu);
        pl.q.shrink(keep, kBounds.blocks, out);
    }
    release(out);
}

// a kept block of at least `bytes` that nothing uses any more, or null
void *take(size_t bytes, int dev, size_t *cap) {
    Pool &pl = pool();
    PoolBlock b;
    bool wait = false;
    long upto = 0;
    {
        std::lock_guard<std::mutex> lk(pl.mu);
        if (!pl.q.take(bytes, dev, cap, &b, &wait)) return nullptr;
        upto = pl.q.epoch();
    }
    if (wait) {
        if (hipDeviceSynchronize() != hipSuccess) {
            (void)hipGetLastError();
            dev_free(b.p, *cap, dev);
            return nullptr;
        }
        std::lock_guard<std::mutex> lk(pl.mu);
        pl.q.waited(dev, upto);
    }
    return b.p;
}

}  // namespace

void *dev_alloc(size_t bytes, size_t *cap, int *dev) {
    FIO_HIP(hipGetDevice(dev));
    size_t c = bytes;
    void *p = t_depth > 0 ? take(bytes, *dev, &c) : nullptr;
    if (!p) {
        c = bytes;
        hipError_t e = hipMalloc(&p, bytes);
        if (e == hipErrorOutOfMemory) {
            (void)hipGetLastError();
            trim(0);
            e = hipMalloc(&p, bytes);
        }
        FIO_HIP(e);
    }
    *cap = c;
    return p;
}

void dev_free(void *p, size_t cap, int dev) {
    if (t_depth > 0 && cap <= kBounds.bytes) {
        PoolBlocks out;
        bool kept = true;
        try {
            Pool &pl = pool();
            std::lock_guard<std::mutex> lk(pl.mu);
            pl.q.keep(p, cap, dev, out);
        } catch (const std::bad_alloc &) {
            kept = false;
        }
        release(out);
        if (kept) return;
    }
    (void)hipFree(p);
}

PoolScope::PoolScope() { ++t_depth; }

PoolScope::~PoolScope() {
    if (--t_depth > 0) return;
    PoolBlocks out;
    {
        Pool &pl = pool();
        std::lock_guard<std::mutex> lk(pl.mu);
        pl.q.end_call(out);
    }
    release(out);
}

}  // namespace fio

extern "C" void fio_memory_trim(size_t keep_bytes) { fio::trim(keep_bytes); }

extern "C" size_t fio_memory_kept(void) {
    fio::Pool &pl = fio::pool();
    std::lock_guard<std::mutex> lk(pl.mu);
    return pl.q.bytes();
}
