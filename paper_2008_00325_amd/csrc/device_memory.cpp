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

// Takes block i out of the store (the mutex is held).
DeviceBlock remove(Store &s, size_t i)
{
    const DeviceBlock b = s.kept[i].block;
    s.bytes -= b.bytes;
    s.kept.erase(s.kept.begin() + (ptrdiff_t)i);
    return b;
}

// Frees kept blocks for which `which(store, block)` holds, one at a time and not under
// the mutex: freeing can wait for the device, and other threads' calls with it.
template <typename Which>
void free_where(Which which)
{
    Store &s = store();
    for (;;) {
        DeviceBlock b;
        {
            std::lock_guard<std::mutex> lock(s.mu);
            for (size_t i = 0; i < s.kept.size() && !b.ptr; ++i)
                if (which(s, s.kept[i])) b = remove(s, i);
        }
        if (!b.ptr) return;
        free_block(&b);
    }
}

}  // namespace

hipError_t take_block(size_t bytes, Held held, DeviceBlock *out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    // the smallest that fits: a handle's block not much larger than asked for, a
    // call's at most twice that (small ones: any up to 1 MB)
    size_t most = held == Held::kByHandle ? bytes + bytes / 8 : 2 * bytes;
    if (most < (size_t)1 << 20) most = (size_t)1 << 20;
    Store &s = store();
    {
        std::lock_guard<std::mutex> lock(s.mu);
        ++s.takes;
        size_t best = s.kept.size();
        for (size_t i = 0; i < s.kept.size(); ++i) {
            const DeviceBlock &b = s.kept[i].block;
            if (b.device != dev || b.bytes < bytes || b.bytes > most) continue;
            if (best == s.kept.size() || b.bytes < s.kept[best].block.bytes) best = i;
        }
        if (best < s.kept.size()) *out = remove(s, best);
    }
    free_where([](const Store &st, const Kept &k) { return st.takes - k.given > kKeptTakes; });
    if (out->ptr) return hipSuccess;
    DeviceBlock b;
    b.device = dev;
    b.bytes = bytes;
    e = hipMalloc(&b.ptr, bytes > 0 ? bytes : 1);
    if (e == hipErrorOutOfMemory || e == hipErrorMemoryAllocation) {
        (void)hipGetLastError();
        free_kept_blocks();
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
    try {
        std::lock_guard<std::mutex> lock(s.mu);
        s.kept.push_back(Kept{*b, s.takes});
        s.bytes += b->bytes;
    } catch (...) {
        free_block(b);
        return;
    }
    *b = DeviceBlock{};
    free_where([](const Store &st, const Kept &) { return st.bytes > kKeptBytes; });   // the one handed back first
}

void free_kept_blocks()
{
    free_where([](const Store &, const Kept &) { return true; });
}

}  // namespace ul
