// device_memory.cpp -- device blocks kept between calls (device_memory.hpp).
#include "device_memory.hpp"

#include <mutex>
#include <vector>

namespace ul {

namespace {

struct Kept {
    DeviceBlock block;
    unsigned long long given;   // the count of takes when it was handed back
};

struct Store {
    std::mutex mu;
    std::vector<Kept> kept;
    size_t bytes = 0;
    unsigned long long takes = 0;
};

// never destroyed: the runtime may be gone when static objects are
Store &store()
{
    static Store *s = new Store;
    return *s;
}

void free_block(DeviceBlock *b)
{
    if (b->host) (void)hipHostFree(b->host);
    if (b->ptr) (void)hipFree(b->ptr);
    *b = DeviceBlock{};
}

void drop(Store &s, size_t i)
{
    s.bytes -= s.kept[i].block.bytes;
    free_block(&s.kept[i].block);
    s.kept.erase(s.kept.begin() + (ptrdiff_t)i);
}

}  // namespace

hipError_t take_block(size_t bytes, DeviceBlock *out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    Store &s = store();
    {
        std::lock_guard<std::mutex> lock(s.mu);
        ++s.takes;
        // the smallest that fits, not more than twice what is asked for (small ones: any up to 1 MB)
        size_t best = s.kept.size();
        for (size_t i = 0; i < s.kept.size(); ++i) {
            const DeviceBlock &b = s.kept[i].block;
            if (b.device != dev || b.bytes < bytes || (b.bytes > 2 * bytes && b.bytes > ((size_t)1 << 20))) continue;
            if (best == s.kept.size() || b.bytes < s.kept[best].block.bytes) best = i;
        }
        if (best < s.kept.size()) {
            *out = s.kept[best].block;
            s.bytes -= out->bytes;
            s.kept.erase(s.kept.begin() + (ptrdiff_t)best);
        }
        for (size_t i = s.kept.size(); i-- > 0;)
            if (s.takes - s.kept[i].given > kKeptTakes) drop(s, i);
        if (out->ptr) return hipSuccess;
    }
    DeviceBlock b;
    b.device = dev;
    b.bytes = bytes;
    e = hipMalloc(&b.ptr, bytes > 0 ? bytes : 1);
    if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation) {
        (void)hipGetLastError();
        {
            std::lock_guard<std::mutex> lock(s.mu);
            while (!s.kept.empty()) drop(s, s.kept.size() - 1);
        }
        e = hipMalloc(&b.ptr, bytes > 0 ? bytes : 1);
    }
    if (e != hipSuccess) return e;
    e = hipHostMalloc((void **)&b.host, kHostBytes, hipHostMallocDefault);
    if (e != hipSuccess) {
        (void)hipFree(b.ptr);
        return e;
    }
    *out = b;
    return hipSuccess;
}

void give_block(DeviceBlock *b, bool reuse)
{
    if (!b->ptr) return;
    if (!reuse || b->bytes > kKeptBytes) {
        free_block(b);
        return;
    }
    Store &s = store();
    std::lock_guard<std::mutex> lock(s.mu);
    try {
        s.kept.push_back(Kept{*b, s.takes});
    } catch (...) {
        free_block(b);
        return;
    }
    s.bytes += b->bytes;
    *b = DeviceBlock{};
    while (s.bytes > kKeptBytes) drop(s, 0);   // the one handed back first
}

}  // namespace ul
