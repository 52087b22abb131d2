// device_memory.hpp -- device blocks kept between calls.
//
// A layout at a million vertices takes about 1 GB for its handle and as much
// for its ingest.  Mapping and unmapping that for every handle costs from a few
// hundred microseconds to 35 ms of host time (the driver's work on the freed
// pages is waited for by the next allocation), more than the ingest's kernels.
// So freed blocks are kept and handed out again, up to a bound.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

namespace ul {

// Most bytes of free blocks kept per process (a larger block is not kept), and
// the number of blocks handed out after which one that was not needed is freed.
constexpr size_t kKeptBytes = (size_t)4 << 30;
constexpr unsigned kKeptTakes = 64;

// A block of device memory of the current device with at least `bytes` bytes
// (contents undefined), and a small pinned host buffer of its own.  All calls
// are safe from several threads; a block belongs to one holder at a time.
struct DeviceBlock {
    void *ptr = nullptr;
    size_t bytes = 0;
    int device = 0;
    unsigned *host = nullptr;   // kHostBytes of pinned host memory
};
constexpr size_t kHostBytes = 256;

// A handle keeps its block for as long as the caller keeps the handle, so it gets
// one at most an eighth larger than it needs; a call's scratch at most twice.
enum class Held { kByHandle, kByCall };
hipError_t take_block(size_t bytes, Held held, DeviceBlock *out);
// Hands a block back: no work that uses it may be pending.  `reuse` false: the
// device may be in an error state, the memory is freed.
void give_block(DeviceBlock *b, bool reuse);
// Frees every kept block.
void free_kept_blocks();

}  // namespace ul
