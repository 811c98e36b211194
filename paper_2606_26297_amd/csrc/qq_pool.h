// qq_pool.h -- device memory of calls and problem handles, kept for reuse.
//
// A call on host buffers needs device memory for its own length (states, partial sums, outputs), and a
// handle needs a diagonal and tables for its life.  hipMalloc and hipFree of these cost more than the
// kernels of most calls: measured on MI355X, 0.2 ms for the blocks of an n = 18 handle and 3 to 9 ms for
// the 0.5 GiB of states of a complex128 n = 22 gradient, whose kernels take 3 ms.  So a block that is
// given up while nothing on the device uses it is kept per device, up to kPoolKeep bytes in all (kPoolRest
// once no problem lives on the device), and handed to the next request that it fits.
//
// A block enters the pool only idle: its owner has synchronised the stream (or the device) that used it,
// so any thread may take it for any stream.  A block of unknown state is freed with hipFree, which waits
// for the device.  Its contents are whatever the last owner left.
//
// A request for a call takes a kept block of up to twice its size (1 MiB for the small ones); one for a handle,
// which may live as long as the program, of at most an eighth more, so that a handle does not sit on memory
// that it has no use for.  pool_trim gives every kept block back to the device, as a failing allocation of the
// library's own does before it is tried again.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

namespace qq {

constexpr size_t kPoolKeep = 4ull << 30;
constexpr size_t kPoolRest = 256ull << 20;

// One block of device memory, released by the destructor: to the pool after done(), else with hipFree.
struct DevBuf {
    void *p = nullptr;
    size_t bytes = 0;
    int device = 0;
    bool idle = false;

    DevBuf() = default;
    DevBuf(const DevBuf &) = delete;
    DevBuf &operator=(const DevBuf &) = delete;
    ~DevBuf() { release(); }
    // At least n bytes on `device` (made current by the caller); lasting: for a handle.
    hipError_t get(int dev, size_t n, bool lasting = false);
    // Nothing on the device uses the block any more.
    void done() { idle = true; }
    void release();
};

// Frees every kept block of the (current) device; their bytes.
size_t pool_trim(int device);

// Problems alive on a device, for the pool's bound.
void pool_problem_added(int device);
void pool_problem_removed(int device);

}  // namespace qq
