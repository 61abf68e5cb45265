// Device memory of the library's own objects and of the scratch inside its calls.  A part of a partition and its
// plan take about 40 allocations, and hipMalloc and hipFree of a few megabytes cost 60 and 25 us each: eight parts of a
// 512-bit multiplier x 4 took 27 ms, 5 of them kernels.  So freed blocks are kept for the next allocation:
//   * A kept block is handed out again only after the device has been waited for once since it was freed, so whatever
//     was still running on any stream when its owner let it go has ended.  Freeing a block that is kept waits for nothing.
//   * At most 1 / 128 of the device's memory is kept, in blocks of at most an eighth of that; a block beyond that goes back to
//     the device at once, and so do all of them when the library's last block has been freed, or when an allocation fails.
//     hipFree waits for the device.
//   * A request takes the smallest kept block that is large enough and at most a quarter larger.
// One table and one mutex per device, held neither while the device is waited for nor while it allocates or frees.
#include <algorithm>
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
    uint64_t freed;                          // the device's count of freed blocks, this one included
};
typedef std::multimap<size_t, Kept> KeptBlocks;   // by size

struct DevicePool {
    std::mutex m;
    KeptBlocks kept;
    size_t kept_bytes = 0, cap = 0;
    int64_t in_use = 0;                      // blocks handed out or about to be
    uint64_t freed = 0;                      // blocks freed and kept so far
    uint64_t idle = 0;                       // of these, the device has been waited for since the first `idle` were freed
};

struct Pool {
    DevicePool dev[kPoolDevices];
    std::mutex m;                            // of out
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

// all kept blocks of a device (its mutex is held): the caller frees them after letting go of the mutex
void take_all(DevicePool &d, KeptBlocks &drop)
{
    drop.swap(d.kept);
    for (auto &k : drop) d.kept_bytes -= k.first;
}

void give_back(const KeptBlocks &drop)
{
    for (auto &k : drop) (void)hipFree(k.second.p);
}

// A kept block that the device has not been waited for since it was freed: waits, and hands it out.  NULL if that is not
// possible now; the block is kept on.
void *wait_for(DevicePool &d, KeptBlocks::node_type node, uint64_t upto)
{
    const bool waited = hipDeviceSynchronize() == hipSuccess;
    if (!waited) (void)hipGetLastError();
    std::lock_guard<std::mutex> lock(d.m);
    if (!waited) {
        d.kept.insert(std::move(node));
        return nullptr;
    }
    d.idle = std::max(d.idle, upto);
    d.kept_bytes -= node.key();
    return node.mapped().p;
}

int new_block(DevicePool &d, size_t size, void **q)
{
    hipError_t e = hipMalloc(q, size);
    if (e == hipErrorOutOfMemory) {
        KeptBlocks drop;
        {
            std::lock_guard<std::mutex> lock(d.m);
            take_all(d, drop);
        }
        if (!drop.empty()) {
            (void)hipGetLastError();
            give_back(drop);
            e = hipMalloc(q, size);
        }
    }
    if (e != hipSuccess) (void)hipGetLastError();
    return (int)e;
}

}  // namespace

int dev_alloc(void **p, size_t bytes)
{
    *p = nullptr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return (int)e;
    if (dev < 0 || dev >= kPoolDevices) return (int)hipErrorInvalidDevice;
    Pool *pl;
    try {
        pl = &pool();
    } catch (...) {
        return (int)hipErrorOutOfMemory;
    }
    DevicePool &d = pl->dev[dev];
    size_t size = 0, have = 0;
    void *q = nullptr;
    KeptBlocks::node_type node;
    uint64_t upto = 0;
    {
        std::lock_guard<std::mutex> lock(d.m);
        if (!d.cap) {
            size_t free_bytes = 0, total = 0;
            e = hipMemGetInfo(&free_bytes, &total);
            if (e != hipSuccess) return (int)e;
            d.cap = total / 128 + 1;
        }
        size = bytes <= d.cap / 8 ? pool_round(bytes ? bytes : 1) : bytes;   // what would not be kept is not rounded
        ++d.in_use;
        const auto it = d.kept.lower_bound(size);
        if (it != d.kept.end() && it->first <= size + size / 4) {
            have = it->first;
            if (it->second.freed <= d.idle) {
                q = it->second.p;
                d.kept_bytes -= have;
                d.kept.erase(it);
            } else {
                node = d.kept.extract(it);   // still counted in kept_bytes: it may come back
                upto = d.freed;
            }
        }
    }
    if (node) q = wait_for(d, std::move(node), upto);
    int err = 0;
    if (q) size = have;
    else err = new_block(d, size, &q);
    if (!err) {
        try {
            std::lock_guard<std::mutex> lock(pl->m);
            pl->out.emplace(q, std::make_pair(size, dev));
            *p = q;
            return 0;
        } catch (...) {                      // no host memory for the table
            (void)hipFree(q);
            err = (int)hipErrorOutOfMemory;
        }
    }
    KeptBlocks drop;
    {
        std::lock_guard<std::mutex> lock(d.m);
        if (--d.in_use == 0) take_all(d, drop);
    }
    give_back(drop);
    return err;
}

void dev_free(void *p)
{
    if (!p) return;
    Pool &pl = pool();
    size_t size = 0;
    int dev = 0;
    {
        std::lock_guard<std::mutex> lock(pl.m);
        const auto it = pl.out.find(p);
        if (it == pl.out.end()) return;
        size = it->second.first;
        dev = it->second.second;
        pl.out.erase(it);
    }
    DevicePool &d = pl.dev[dev];
    bool keep = false;
    KeptBlocks drop;
    {
        std::lock_guard<std::mutex> lock(d.m);
        if (size <= d.cap / 8 && d.kept_bytes + size <= d.cap) {
            try {
                d.kept.emplace(size, Kept{p, d.freed + 1});
                ++d.freed;
                d.kept_bytes += size;
                keep = true;
            } catch (...) {                  // no host memory for the table
            }
        }
        if (--d.in_use == 0) take_all(d, drop);   // with the last block in use, what is kept goes back
    }
    if (!keep) (void)hipFree(p);
    give_back(drop);
}

}  // namespace groot
