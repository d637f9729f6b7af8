// Reads of large device arrays into host memory, and the pinned staging buffers they go through.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>

namespace btrth {

// Copies behind the work already on s and returns when complete. `device` is the current device; s may be
// any stream, hipStreamPerThread among them.
hipError_t copy_to_host(void* dst, const void* src, size_t bytes, int device, hipStream_t s);

// A pinned buffer and its size, or null where none is to be had (the caller then stages through memory of
// its own); give it back with staging_put.
void* staging_get(size_t* bytes);
void staging_put(void* p);
// Counts the handles, batches and servers that may copy; the last to go frees the idle staging memory.
void staging_retain();
void staging_release();
struct StagingUser {
    StagingUser() { staging_retain(); }
    ~StagingUser() { staging_release(); }
    StagingUser(const StagingUser&) = delete;
    StagingUser& operator=(const StagingUser&) = delete;
};

}  // namespace btrth
