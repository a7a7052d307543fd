// Device and pinned host memory of the library's handles and workspaces.
//
// hipMalloc and hipFree of operator-sized blocks map, clear and unmap pages:
// a program that fills one operator after another spent more time there than
// in the fill (1280-triangle sphere, complex64 blocks, a fill and its release in
// a loop: 16 to 24 ms where the process held other operators, 6.5 in a fresh one,
// 5.6 of it kernels).  A context therefore keeps what its handles
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
    std::multimap<size_t, void *> idle[kKinds];
};

namespace {

// What the contexts of a device may keep together, and what they do
struct Kept {
    size_t limit[kKinds] = {0, 0, 0}, now[kKinds] = {0, 0, 0};
};

// One lock for the tables, held for their updates alone: hipMalloc and hipFree,
// which may wait for a device, run outside it.  Never destroyed: handles may be
// released during the program's exit.
std::mutex &g_mu = *new std::mutex;
std::unordered_map<void *, Block> &g_blocks = *new std::unordered_map<void *, Block>;
std::vector<MemPool *> &g_pools = *new std::vector<MemPool *>;
std::map<int, Kept> &g_kept = *new std::map<int, Kept>;
thread_local MemPool *t_pool = nullptr;

hipError_t raw_alloc(Kind k, void **p, size_t n) {
    if (k == kDevice) return hipMalloc(p, n);
    return hipHostMalloc(p, n, k == kMapped ? hipHostMallocMapped | hipHostMallocCoherent : hipHostMallocDefault);
}

hipError_t raw_free(Kind k, void *p) { return k == kDevice ? hipFree(p) : hipHostFree(p); }

// The idle blocks of one pool, taken out of it
struct Idle {
    int device = 0;
    std::multimap<size_t, void *> blocks[kKinds];
    void take(MemPool *q) {   // g_mu held
        device = q->device;
        for (int k = 0; k < kKinds; ++k) {
            blocks[k].swap(q->idle[k]);
            for (auto &b : blocks[k]) g_kept[device].now[k] -= b.first;
        }
    }
    void free_all() {
        int was = 0;
        (void)hipGetDevice(&was);
        (void)hipSetDevice(device);
        for (int k = 0; k < kKinds; ++k)
            for (auto &b : blocks[k]) (void)raw_free((Kind)k, b.second);
        (void)hipSetDevice(was);
    }
};

void release_all_idle() {
    for (;;) {
        Idle idle;
        {
            std::lock_guard<std::mutex> lock(g_mu);
            auto q = std::find_if(g_pools.begin(), g_pools.end(), [](MemPool *o) {
                return std::any_of(o->idle, o->idle + kKinds, [](auto &m) { return !m.empty(); });
            });
            if (q == g_pools.end()) return;
            idle.take(*q);
        }
        idle.free_all();
    }
}

MemPool *thread_pool() {   // g_mu held
    return std::find(g_pools.begin(), g_pools.end(), t_pool) != g_pools.end() ? t_pool : nullptr;
}

hipError_t alloc(Kind k, void **p, size_t n) {
    *p = nullptr;
    try {
        {
            std::lock_guard<std::mutex> lock(g_mu);
            if (MemPool *q = thread_pool()) {
                // the smallest kept block that fits without wasting a quarter
                auto it = q->idle[k].lower_bound(n);
                if (it != q->idle[k].end() && it->first <= n + n / 4 + 4096) {
                    g_blocks[it->second] = {q, it->first, k};
                    *p = it->second;
                    g_kept[q->device].now[k] -= it->first;
                    q->idle[k].erase(it);
                    return hipSuccess;
                }
            }
        }
        void *b = nullptr;
        hipError_t e = raw_alloc(k, &b, n);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            release_all_idle();
            e = raw_alloc(k, &b, n);
        }
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return e;
        }
        try {
            std::lock_guard<std::mutex> lock(g_mu);
            g_blocks[b] = {thread_pool(), n, k};
        } catch (...) {
            (void)raw_free(k, b);
            throw;
        }
        *p = b;
        return hipSuccess;
    } catch (const std::bad_alloc &) {
        return hipErrorOutOfMemory;
    }
}

hipError_t release(void *p) {
    if (!p) return hipSuccess;
    Block b;
    {
        std::lock_guard<std::mutex> lock(g_mu);
        auto it = g_blocks.find(p);
        if (it == g_blocks.end()) return hipErrorInvalidValue;
        b = it->second;
        g_blocks.erase(it);
        if (b.pool) {
            Kept &kept = g_kept[b.pool->device];   // made with the pool
            if (kept.now[b.kind] + b.size <= kept.limit[b.kind]) {
                try {
                    b.pool->idle[b.kind].emplace(b.size, p);
                    kept.now[b.kind] += b.size;
                    return hipSuccess;
                } catch (const std::bad_alloc &) {
                }
            }
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
    const bool known = hipDeviceTotalMem(&total, device) == hipSuccess;
    std::lock_guard<std::mutex> lock(g_mu);
    try {
        Kept &kept = g_kept[device];
        if (known) kept.limit[kDevice] = total / 16;
        kept.limit[kPinned] = kept.limit[kMapped] = (size_t)16 << 20;
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
    Idle idle;
    {
        std::lock_guard<std::mutex> lock(g_mu);
        idle.take(q);
        for (auto &b : g_blocks)
            if (b.second.pool == q) b.second.pool = nullptr;
        g_pools.erase(std::remove(g_pools.begin(), g_pools.end(), q), g_pools.end());
        if (t_pool == q) t_pool = nullptr;
    }
    idle.free_all();
    delete q;
}

}  // namespace mbem
