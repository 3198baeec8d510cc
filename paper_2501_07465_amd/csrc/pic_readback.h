// pic_readback.h -- copies of device arrays to host memory in another layout (exports of libpic).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>

#include <functional>
#include <vector>

namespace pic {

// n elements of several device arrays that belong together: put(arrays, first, count) writes elements
// first .. first + count - 1 to where the caller wants them, arrays[k] pointing at element `first` of
// source k in host memory.  Called from several threads, on disjoint ranges.
struct ReadbackJob {
    struct Source {
        const void* dev;
        size_t elem;  // bytes per element
    };
    std::vector<Source> src;
    size_t n = 0;
    std::function<void(const char* const* arrays, size_t first, size_t count)> put;
};

// Runs the jobs: chunks copied on stream st into a ring of pinned buffers and put from there by worker
// threads while the next chunks are on their way.  Returns once everything is put (or the error).
hipError_t readback(const std::vector<ReadbackJob>& jobs, hipStream_t st);

// The pinned rings outlive a simulation; they are kept while any simulation is alive and freed with the
// last one.
void readback_retain();
void readback_release();

}  // namespace pic
