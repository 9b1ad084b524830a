// Device memory that outlives a call or a tree, kept in the process for the
// next one (memory.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>

namespace ot {

// Memory of a tree or of a build.
struct Block {
    void *p = nullptr;
    size_t bytes = 0;
    int device = 0;
};
Block block_take(size_t bytes);    // at least `bytes` on the current device; p = null: none to be had
void block_give(const Block &b);   // no work on it is left

// Working memory of a plain call that sorts its points, on a tree's device.
struct Scratch {
    void *p;   // null: none to be had
    int slot;  // -1: allocated for this call
};
Scratch scratch_take(int device, size_t bytes, hipStream_t s);
void scratch_give(int device, const Scratch &m, hipStream_t s);   // the call's kernels are enqueued
void scratch_trees(int device, int change);                       // a tree was built (1) or destroyed (-1)

// hipMalloc on the current device and hipMallocAsync on a stream of `device`;
// where there is no room, once more after what is kept on it is given back.
hipError_t device_malloc(void **p, size_t bytes);
hipError_t device_malloc_async(int device, void **p, size_t bytes, hipStream_t s);

}  // namespace ot
