// Device memory kept between calls (pool.h).
#include "pool.h"

#include <algorithm>
#include <new>

namespace tgdk {

// one lock for all pools, so that an allocation can empty every one of a device
static std::mutex pools_mutex;
static std::vector<DevPool*> pools;
static unsigned long long puts = 0;

DevPool::DevPool(int dev) : device(dev) {
    std::lock_guard<std::mutex> lock(pools_mutex);
    pools.push_back(this);
}

DevPool::~DevPool() {
    std::lock_guard<std::mutex> lock(pools_mutex);
    pools.erase(std::remove(pools.begin(), pools.end(), this), pools.end());
    drop_all();
}

void DevPool::drop(size_t i) {
    held -= idle[i].bytes;
    (void)hipFree(idle[i].p);
    idle.erase(idle.begin() + i);
}

void DevPool::drop_all() {
    while (!idle.empty()) drop(idle.size() - 1);
}

void DevPool::trim(size_t room) {
    while (!idle.empty() && now - idle[0].stamp > POOL_AGE) drop(0);  // (in the order of their put)
    for (;;) {
        size_t sum = room;
        DevPool* oldest = nullptr;
        for (DevPool* p : pools) {
            if (p->device != device || p->idle.empty()) continue;
            sum += p->held;
            if (!oldest || p->idle[0].order < oldest->idle[0].order) oldest = p;
        }
        if (sum <= POOL_BYTES || !oldest) return;
        oldest->drop(0);
    }
}

void DevPool::flush() {
    std::lock_guard<std::mutex> lock(pools_mutex);
    drop_all();
}

void DevPool::close() {
    std::lock_guard<std::mutex> lock(pools_mutex);
    closed = true;
    drop_all();
}

hipError_t dev_malloc(int device, void** p, size_t bytes) {
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipSuccess) return e;
    (void)hipGetLastError();
    std::lock_guard<std::mutex> lock(pools_mutex);
    for (DevPool* pool : pools)
        if (pool->device == device) pool->drop_all();
    e = hipMalloc(p, bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        *p = nullptr;
    }
    return e;
}

static bool record(std::unordered_map<void*, size_t>& taken, void* p, size_t bytes) {
    try {
        taken[p] = bytes;
        return true;
    } catch (const std::bad_alloc&) {
        return false;
    }
}

void* DevPool::get(size_t bytes) noexcept {
    {
        std::lock_guard<std::mutex> lock(pools_mutex);
        ++now;
        size_t best = idle.size();
        for (size_t i = 0; i < idle.size(); ++i)
            if (idle[i].bytes >= bytes && idle[i].bytes - bytes <= idle[i].bytes / 8 &&
                (best == idle.size() || idle[i].bytes < idle[best].bytes))
                best = i;
        if (best < idle.size()) {
            void* p = idle[best].p;
            if (!record(taken, p, idle[best].bytes)) return nullptr;
            held -= idle[best].bytes;
            idle.erase(idle.begin() + best);
            trim(0);
            return p;
        }
        trim(0);
    }
    void* p = nullptr;
    if (dev_malloc(device, &p, bytes) != hipSuccess) return nullptr;
    std::lock_guard<std::mutex> lock(pools_mutex);
    if (record(taken, p, bytes)) return p;
    (void)hipFree(p);
    return nullptr;
}

void DevPool::put(void* p) noexcept {
    if (!p) return;
    std::lock_guard<std::mutex> lock(pools_mutex);
    const auto it = taken.find(p);
    const size_t bytes = it == taken.end() ? POOL_BYTES + 1 : it->second;
    if (it != taken.end()) taken.erase(it);
    if (closed || bytes > POOL_BYTES) {
        (void)hipFree(p);
        return;
    }
    trim(bytes);
    try {
        idle.push_back({p, bytes, now, ++puts});
    } catch (const std::bad_alloc&) {
        (void)hipFree(p);
        return;
    }
    held += bytes;
}

}  // namespace tgdk
