// Device memory kept between calls.
#pragma once

#include <hip/hip_runtime.h>

#include <mutex>
#include <unordered_map>
#include <vector>

namespace tgdk {

// Device memory of deflation spaces and of the calls that build and use them,
// kept for the next call.  Handing large blocks back to the driver and taking
// them again costs little in one call, but the driver clears what it is handed
// back, and a program that moves one space after another waits for that: moving
// 30 vectors to 1023^2 takes 2.8 ms the first times and 21 ms from then on
// (2.3 GB a call handed back and cleared).
//
// A block is reused for requests of its size or up to an eighth less.  All
// contexts of a device together hold at most POOL_BYTES free (the oldest goes
// first, whoever's it is), a block that no one took for POOL_AGE requests goes
// back to the driver, and so does everything free on flush() and when an
// allocation fails.  The pool belongs to a context, hence to one stream:
// whatever still uses a block's old contents is ordered before its next use.
// Handles may be destroyed from any thread (a garbage collector's), so the
// pools have a lock.
constexpr size_t POOL_BYTES = (size_t)2 << 30;
constexpr unsigned POOL_AGE = 64;
class DevPool {
public:
    explicit DevPool(int device);
    ~DevPool();
    DevPool(const DevPool&) = delete;
    DevPool& operator=(const DevPool&) = delete;
    // Both are called from C entry points and throw nothing: where there is no
    // host memory for its record, a block is not handed out (null, as without
    // device memory), or goes back to the driver.
    void* get(size_t bytes) noexcept;
    void put(void* p) noexcept;
    void flush();  // hands back what is free
    void close();  // the context goes: flush(), and nothing is kept from now on

private:
    friend hipError_t dev_malloc(int device, void** p, size_t bytes);
    struct Block {
        void* p;
        size_t bytes;
        unsigned long long stamp, order;  // of put(): this pool's requests, the process's
    };
    void drop(size_t i);
    void drop_all();
    void trim(size_t room);  // hands back old blocks, and the device's oldest until `room` more bytes fit
    const int device;
    std::vector<Block> idle;
    std::unordered_map<void*, size_t> taken;
    size_t held = 0;
    bool closed = false;
    unsigned long long now = 0;
};

// hipMalloc on the (current) device; where there is no memory, what the
// device's pools hold free is handed back first and the call made again.
hipError_t dev_malloc(int device, void** p, size_t bytes);

}  // namespace tgdk
