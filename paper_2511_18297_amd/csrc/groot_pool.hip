// Device memory of the library's own objects and of the scratch inside its calls.  A part of a partition and its
// plan take about 40 allocations, and hipMalloc and hipFree of a few megabytes cost 60 and 25 us each: eight parts of a
// 512-bit multiplier x 4 took 27 ms, 5 of them kernels.  So freed blocks are kept for the next allocation:
//   * A kept block is handed out again only after the device has been waited for once since it was freed, so whatever
//     was still running on any stream when its owner let it go has ended.  Freeing itself waits for nothing.
//   * At most 1 / 128 of the device's memory is kept; a block beyond that goes back to the device at once, and so do
//     all of them when the library's last block has been freed, or when an allocation fails.
//   * A request takes the smallest kept block that is large enough and at most a quarter larger.
// One table per device behind one mutex.
#include <map>
#include <mutex>
#include <unordered_map>

#include <hip/hip_runtime.h>

#include "groot_internal.h"

namespace groot {

namespace {

constexpr int kPoolDevices = 64;

struct Kept {
    void *p;
    bool idle;                               // the device has been waited for since it was freed
};

struct DevicePool {
    std::multimap<size_t, Kept> kept;        // by size
    size_t kept_bytes = 0, cap = 0;
    int64_t in_use = 0;                      // blocks handed out
};

struct Pool {
    std::mutex m;
    DevicePool dev[kPoolDevices];
    std::unordered_map<void *, std::pair<size_t, int>> out;   // block -> size, device
};

Pool &pool()
{
    static Pool *p = new Pool;               // never destroyed: objects may be freed while the process ends
    return *p;
}

// to a multiple of 256 bytes, and of 1/64 to 1/32 of the size, so that arrays of parts of nearly the same size fit one another
size_t pool_round(size_t bytes)
{
    size_t step = 256;
    while (step * 64 <= bytes) step *= 2;
    return (bytes + step - 1) / step * step;
}

void give_back(DevicePool &d)
{
    for (auto &k : d.kept) (void)hipFree(k.second.p);
    d.kept.clear();
    d.kept_bytes = 0;
}

}  // namespace

static int alloc_block(Pool &pl, int dev, void **p, size_t bytes)
{
    DevicePool &d = pl.dev[dev];
    if (!d.cap) {
        size_t free_bytes = 0, total = 0;
        const hipError_t e = hipMemGetInfo(&free_bytes, &total);
        if (e != hipSuccess) return (int)e;
        d.cap = total / 128 + 1;
    }
    const size_t size = bytes <= d.cap / 8 ? pool_round(bytes ? bytes : 1) : bytes;   // what would not be kept is not rounded
    const auto out = pl.out.emplace(nullptr, std::make_pair(size, dev)).first;        // a place in the table before the memory
    auto node = pl.out.extract(out);
    auto hand_out = [&](void *q, size_t have) {
        node.key() = q;
        node.mapped().first = have;
        pl.out.insert(std::move(node));
        ++d.in_use;
        *p = q;
        return 0;
    };
    const auto it = d.kept.lower_bound(size);
    if (it != d.kept.end() && it->first <= size + size / 4) {
        if (!it->second.idle) {
            if (hipDeviceSynchronize() == hipSuccess)
                for (auto &k : d.kept) k.second.idle = true;
            else
                (void)hipGetLastError();     // the device cannot be waited for now: a new block
        }
        if (it->second.idle) {
            void *const q = it->second.p;
            const size_t have = it->first;
            d.kept_bytes -= have;
            d.kept.erase(it);
            return hand_out(q, have);
        }
    }
    void *q = nullptr;
    hipError_t e = hipMalloc(&q, size);
    if (e == hipErrorOutOfMemory && !d.kept.empty()) {
        (void)hipGetLastError();
        give_back(d);
        e = hipMalloc(&q, size);
    }
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return (int)e;
    }
    return hand_out(q, size);
}

int dev_alloc(void **p, size_t bytes)
{
    *p = nullptr;
    int dev = 0;
    const hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return (int)e;
    if (dev < 0 || dev >= kPoolDevices) return (int)hipErrorInvalidDevice;
    try {
        Pool &pl = pool();
        std::lock_guard<std::mutex> lock(pl.m);
        return alloc_block(pl, dev, p, bytes);
    } catch (...) {                          // no host memory for the tables
        return (int)hipErrorOutOfMemory;
    }
}

void dev_free(void *p)
{
    if (!p) return;
    Pool &pl = pool();
    std::lock_guard<std::mutex> lock(pl.m);
    const auto it = pl.out.find(p);
    if (it == pl.out.end()) return;
    const size_t size = it->second.first;
    DevicePool &d = pl.dev[it->second.second];
    pl.out.erase(it);
    bool keep = size <= d.cap / 8 && d.kept_bytes + size <= d.cap;
    if (keep) {
        try {
            d.kept.emplace(size, Kept{p, false});
            d.kept_bytes += size;
        } catch (...) {
            keep = false;
        }
    }
    if (!keep) (void)hipFree(p);
    if (--d.in_use == 0) give_back(d);
}

}  // namespace groot
