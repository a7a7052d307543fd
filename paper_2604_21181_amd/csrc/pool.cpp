// Device and pinned host memory of the library's handles and workspaces.
//
// hipMalloc and hipFree of operator-sized blocks map, clear and unmap pages:
// a program that fills one operator after another spent more time there than
// in the fill (1280-triangle sphere, complex64 blocks: 24 ms per fill in a
// loop, 5.6 ms of it kernels).  A context therefore keeps what its handles
// release, up to 1/16 of the device's memory, and hands it out again:
//  - a block only goes back to the context it was allocated under, whose work
//    all runs on one stream, so a new user's work follows the last one's;
//  - handles that other contexts may have used, and the parts of them that a
//    later call replaces, are released after a device synchronisation (as
//    hipFree does by itself);
//  - a failed allocation releases what every context keeps and is tried again;
//  - destroying the context gives everything back.  Blocks still in use then
//    are freed when their handle is.
#include <algorithm>
#include <map>
#include <mutex>
#include <new>
#include <unordered_map>
#include <vector>

#include "mbem_internal.h"

namespace mbem {

namespace {

enum Kind { kDevice = 0, kPinned = 1, kMapped = 2, kKinds = 3 };

struct Block {
    MemPool *pool;
    size_t size;
    Kind kind;
};

}  // namespace

struct MemPool {
    int device = 0;
    size_t limit[kKinds] = {0, 0, 0}, kept[kKinds] = {0, 0, 0};
    std::multimap<size_t, void *> idle[kKinds];
};

namespace {

// One lock for the table of blocks and every pool: allocations are rare.
// Never destroyed: handles may be released during the program's exit.
std::mutex &g_mu = *new std::mutex;
std::unordered_map<void *, Block> &g_blocks = *new std::unordered_map<void *, Block>;
std::vector<MemPool *> &g_pools = *new std::vector<MemPool *>;
thread_local MemPool *t_pool = nullptr;

hipError_t raw_alloc(Kind k, void **p, size_t n) {
    if (k == kDevice) return hipMalloc(p, n);
    return hipHostMalloc(p, n, k == kMapped ? hipHostMallocMapped | hipHostMallocCoherent : hipHostMallocDefault);
}

hipError_t raw_free(Kind k, void *p) { return k == kDevice ? hipFree(p) : hipHostFree(p); }

void release_idle(MemPool *q) {   // g_mu held
    int was = 0;
    (void)hipGetDevice(&was);
    (void)hipSetDevice(q->device);
    for (int k = 0; k < kKinds; ++k) {
        for (auto &b : q->idle[k]) (void)raw_free((Kind)k, b.second);
        q->idle[k].clear();
        q->kept[k] = 0;
    }
    (void)hipSetDevice(was);
}

hipError_t alloc(Kind k, void **p, size_t n) {
    *p = nullptr;
    try {
        std::lock_guard<std::mutex> lock(g_mu);
        MemPool *q = std::find(g_pools.begin(), g_pools.end(), t_pool) != g_pools.end() ? t_pool : nullptr;
        if (q) {
            // the smallest kept block that fits without wasting a quarter
            auto it = q->idle[k].lower_bound(n);
            if (it != q->idle[k].end() && it->first <= n + n / 4 + 4096) {
                *p = it->second;
                g_blocks[*p] = {q, it->first, k};
                q->kept[k] -= it->first;
                q->idle[k].erase(it);
                return hipSuccess;
            }
        }
        hipError_t e = raw_alloc(k, p, n);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            for (MemPool *o : g_pools) release_idle(o);
            e = raw_alloc(k, p, n);
        }
        if (e != hipSuccess) {
            (void)hipGetLastError();
            *p = nullptr;
            return e;
        }
        try {
            g_blocks[*p] = {q, n, k};
        } catch (...) {
            (void)raw_free(k, *p);
            *p = nullptr;
            throw;
        }
        return hipSuccess;
    } catch (const std::bad_alloc &) {
        return hipErrorOutOfMemory;
    }
}

hipError_t release(void *p) {
    if (!p) return hipSuccess;
    std::lock_guard<std::mutex> lock(g_mu);
    auto it = g_blocks.find(p);
    if (it == g_blocks.end()) return hipErrorInvalidValue;
    const Block b = it->second;
    g_blocks.erase(it);
    if (b.pool && b.pool->kept[b.kind] + b.size <= b.pool->limit[b.kind]) {
        try {
            b.pool->idle[b.kind].emplace(b.size, p);
            b.pool->kept[b.kind] += b.size;
            return hipSuccess;
        } catch (const std::bad_alloc &) {
        }
    }
    return raw_free(b.kind, p);
}

}  // namespace

hipError_t dev_malloc(void **p, size_t n) { return alloc(kDevice, p, std::max<size_t>(n, 1)); }
hipError_t dev_free(void *p) { return release(p); }
hipError_t dev_free_wait(void *p) {
    const hipError_t e = hipDeviceSynchronize();
    const hipError_t f = release(p);
    return e != hipSuccess ? e : f;
}
hipError_t pin_malloc(void **p, size_t n, bool mapped) {
    return alloc(mapped ? kMapped : kPinned, p, std::max<size_t>(n, 1));
}
hipError_t pin_free(void *p) { return release(p); }

MemPool *pool_create(int device) {
    MemPool *q = new (std::nothrow) MemPool;
    if (!q) return nullptr;
    q->device = device;
    size_t total = 0;
    if (hipDeviceTotalMem(&total, device) == hipSuccess) q->limit[kDevice] = total / 16;
    q->limit[kPinned] = q->limit[kMapped] = (size_t)16 << 20;
    std::lock_guard<std::mutex> lock(g_mu);
    try {
        g_pools.push_back(q);
    } catch (const std::bad_alloc &) {
        delete q;
        return nullptr;
    }
    return q;
}

void pool_use(MemPool *q) { t_pool = q; }

void pool_destroy(MemPool *q) {
    if (!q) return;
    std::lock_guard<std::mutex> lock(g_mu);
    release_idle(q);
    for (auto &b : g_blocks)
        if (b.second.pool == q) b.second.pool = nullptr;
    g_pools.erase(std::remove(g_pools.begin(), g_pools.end(), q), g_pools.end());
    if (t_pool == q) t_pool = nullptr;
    delete q;
}

}  // namespace mbem
