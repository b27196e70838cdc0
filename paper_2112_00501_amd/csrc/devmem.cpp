// Device memory kept between handles (see devmem.hpp).
#include "devmem.hpp"

#include <list>
#include <map>
#include <mutex>
#include <unordered_map>

namespace cs {

namespace {

struct Block {
    void* p;
    size_t bytes;
    int dev;
    bool quiet;  // the device has been waited for since the block was freed
};

struct Cache {
    std::mutex mu;
    std::unordered_map<void*, Block> live;  // handed out
    std::list<Block> kept;                  // longest-kept first
    std::map<int, size_t> kept_bytes, limit;
    long long lattices = 0;
};

// Never destroyed: the blocks that are left go with the process, and the HIP
// runtime may be gone before this would be.
Cache& cache() {
    static Cache* c = new Cache;
    return *c;
}

// The current device made dev for the lifetime of the object.
struct OnDevice {
    int was = -1;
    explicit OnDevice(int dev) {
        int cur = 0;
        if (hipGetDevice(&cur) == hipSuccess && cur != dev && hipSetDevice(dev) == hipSuccess) was = cur;
    }
    ~OnDevice() {
        if (was >= 0) (void)hipSetDevice(was);
    }
};

// Calls that are not capturable are allowed in this thread for the lifetime of
// the object, without ending a stream capture that is open in it.
struct BesideCapture {
    hipStreamCaptureMode was = hipStreamCaptureModeRelaxed;
    bool set;
    BesideCapture() : set(hipThreadExchangeStreamCaptureMode(&was) == hipSuccess) {}
    ~BesideCapture() {
        if (set) (void)hipThreadExchangeStreamCaptureMode(&was);
    }
};

void free_block(const Block& b) {
    OnDevice on(b.dev);
    (void)hipFree(b.p);
}

// Frees kept blocks of dev (all devices: -1), longest-kept first, until at
// most `most` bytes of it are kept.  The caller holds the lock.
void trim(Cache& c, int dev, size_t most) {
    for (auto it = c.kept.begin(); it != c.kept.end();) {
        if ((dev >= 0 && it->dev != dev) || c.kept_bytes[it->dev] <= most) {
            ++it;
            continue;
        }
        c.kept_bytes[it->dev] -= it->bytes;
        free_block(*it);
        it = c.kept.erase(it);
    }
}

// Waits for all work on dev and marks its kept blocks quiet.  hipFree is what
// waits: hipDeviceSynchronize would invalidate a stream capture that another
// thread has open.  The caller holds the lock.  A failure (device memory full)
// is the caller's to act on and not left behind for its next launch check.
hipError_t wait_for_device(Cache& c, int dev) {
    OnDevice on(dev);
    void* q = nullptr;
    hipError_t e = hipMalloc(&q, 256);
    if (e == hipSuccess) e = hipFree(q);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return e;
    }
    for (Block& b : c.kept)
        if (b.dev == dev) b.quiet = true;
    return hipSuccess;
}

}  // namespace

// No exception leaves these functions (the bookkeeping allocates host memory):
// a block that cannot be entered is not handed out, or not kept.
hipError_t dev_alloc(void** p, size_t bytes) try {
    *p = nullptr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    Cache& c = cache();
    std::lock_guard<std::mutex> lk(c.mu);
    // the block freed last among those of this size
    for (auto it = c.kept.rbegin(); it != c.kept.rend(); ++it)
        if (it->dev == dev && it->bytes == bytes) {
            if (!it->quiet && wait_for_device(c, dev) != hipSuccess) break;
            c.live[it->p] = *it;
            c.kept_bytes[dev] -= bytes;
            *p = it->p;
            c.kept.erase(std::next(it).base());
            return hipSuccess;
        }
    e = hipMalloc(p, bytes);
    if (e != hipSuccess && c.kept_bytes[dev] > 0) {
        (void)hipGetLastError();
        trim(c, dev, 0);
        e = hipMalloc(p, bytes);
    }
    if (e != hipSuccess) {
        *p = nullptr;
        return e;
    }
    if (c.limit.find(dev) == c.limit.end()) {
        size_t avail = 0, total = 0;
        c.limit[dev] = hipMemGetInfo(&avail, &total) == hipSuccess ? total / 16 : 0;
        c.kept_bytes[dev] = 0;  // the entries dev_free and trim look up
    }
    if (*p) c.live[*p] = Block{*p, bytes, dev, false};
    return hipSuccess;
} catch (...) {
    if (*p) (void)hipFree(*p);
    *p = nullptr;
    return hipErrorOutOfMemory;
}

void dev_free(void* p) {
    if (!p) return;
    Cache& c = cache();
    std::lock_guard<std::mutex> lk(c.mu);
    auto it = c.live.find(p);
    if (it == c.live.end()) return;
    Block b = it->second;
    c.live.erase(it);
    const size_t limit = c.limit[b.dev];
    if (c.lattices == 0 || b.bytes > limit) {
        free_block(b);
        return;
    }
    b.quiet = false;
    try {
        c.kept.push_back(b);
    } catch (...) {
        free_block(b);
        return;
    }
    c.kept_bytes[b.dev] += b.bytes;
    trim(c, b.dev, limit);
}

void dev_wait(const void* p) {
    if (!p) return;
    Cache& c = cache();
    std::lock_guard<std::mutex> lk(c.mu);
    auto it = c.live.find(const_cast<void*>(p));
    if (it == c.live.end()) return;
    const int dev = it->second.dev;
    BesideCapture beside;  // a handle may go while its thread captures
    if (wait_for_device(c, dev) == hipSuccess) return;
    // no memory left for the wait: returning kept blocks waits too
    if (c.kept_bytes[dev] > 0) {
        trim(c, dev, 0);
    } else {
        OnDevice on(dev);
        (void)hipDeviceSynchronize();
    }
}

void dev_release() {
    Cache& c = cache();
    std::lock_guard<std::mutex> lk(c.mu);
    BesideCapture beside;
    trim(c, -1, 0);
}

void dev_lattice_created() {
    Cache& c = cache();
    std::lock_guard<std::mutex> lk(c.mu);
    ++c.lattices;
}

void dev_lattice_destroyed() {
    Cache& c = cache();
    std::lock_guard<std::mutex> lk(c.mu);
    if (--c.lattices == 0) trim(c, -1, 0);
}

}  // namespace cs
